// adjoint.hip -- checkpoints of the forward push and the reverse sweep of K
// push + deposit steps (FP64).
//
// The loss is L = sum over steps n and particles of
// lambda . (F^r, F^th, G^ph)_n, lambda being given per grid element (the
// cotangent of the accumulated current).  Particles are independent given the
// fields, so the reverse sweep runs one thread per particle:
//   for each checkpoint segment, last first:
//     recompute the segment's start-of-step states from its checkpoint
//     (stored in the workspace), then for each step of the segment, last
//     first: replay the step into a tape and run its reverse
//     (grpic_adjoint.hpp), carrying the state cotangent in registers and
//     adding field cotangents to the gradient arrays with FP64 atomics.
// d L / d u_i(0) is the state cotangent left after the first step.  A
// prepass marks the rows and columns where lambda is non-zero; particles and
// steps whose deposits cannot reach them while their cotangent is zero are
// skipped (exactly: their contribution is zero).
#include "grpic_backward.hpp"

namespace grpic {

size_t checkpoint_slot_bytes(int64_t n) { return slot_cell_bytes(n) + (size_t)n * 5 * 8; }
int adj_max_corr() { return adj::kMaxCorr; }

// The state before a step, in double whatever the particles' precision (a
// float state is promoted exactly).
template <class T>
__global__ __launch_bounds__(256) void save_state(const StepArgs A, char* slot) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= A.n) return;
    int32_t* cell = reinterpret_cast<int32_t*>(slot);
    double* d = reinterpret_cast<double*>(slot + slot_cell_bytes(A.n));
    cell[p] = A.cell[p];
    const T* src[5] = {static_cast<const T*>(A.xr), static_cast<const T*>(A.xth), static_cast<const T*>(A.ur),
                       static_cast<const T*>(A.uth), static_cast<const T*>(A.uph)};
    for (int k = 0; k < 5; ++k) d[(int64_t)k * A.n + p] = (double)src[k][p];
}

hipError_t launch_save_state(const StepArgs& A, bool split, void* slot, hipStream_t stream) {
    if (A.n <= 0) return hipSuccess;
    const dim3 g((unsigned)((A.n + 255) / 256));
    if (split) hipLaunchKernelGGL(save_state<float>, g, dim3(256), 0, stream, A, static_cast<char*>(slot));
    else hipLaunchKernelGGL(save_state<double>, g, dim3(256), 0, stream, A, static_cast<char*>(slot));
    return hipGetLastError();
}

// ---------------------------------------------------------------- lambda support
// Rows and columns (storage indices, guards included) holding a non-zero
// lambda entry, as exclusive prefix counts, so that "is lambda zero on this
// box" is two subtractions.  A conservative test: a box is reported non-zero
// when some row and some column in its ranges hold non-zeros.
__global__ __launch_bounds__(256) void lam_clear(int* __restrict__ flags, int n) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) flags[t] = 0;
}

// Flags of the rows and columns: a workgroup reads kLamRows rows of 256
// columns (a pass over lambda with every CU busy; one thread per column took
// 0.28 ms for a dense 512 x 512).  Every writer of a flag writes 1.
constexpr int kLamRows = 8;
__global__ __launch_bounds__(256) void lam_any(const BackArgs B, int* __restrict__ row_flag, int* __restrict__ col_flag) {
    const int j = blockIdx.x * 256 + threadIdx.x, i0 = blockIdx.y * kLamRows;
    bool col = false;
    for (int i = i0; i < min(i0 + kLamRows, B.rows); ++i) {
        bool any = false;
        if (j < B.pitch) {
            const int64_t e = (int64_t)i * B.pitch + j;
            any = (B.lam[0][e] != 0.0) | (B.lam[1][e] != 0.0) | (B.lam[2][e] != 0.0);
        }
        col |= any;
        if (__ballot(any) && (threadIdx.x & 63) == 0) row_flag[i] = 1;
    }
    if (col) col_flag[j] = 1;
}

// flag[0..len) -> pre[0..len], a wave per array: rows, columns.
__global__ __launch_bounds__(128) void lam_prefix(const BackArgs B, const int* __restrict__ row_flag,
                                                  const int* __restrict__ col_flag, int* __restrict__ row_pre,
                                                  int* __restrict__ col_pre) {
    const bool rows = threadIdx.x < 64;
    const int* flag = rows ? row_flag : col_flag;
    int* pre = rows ? row_pre : col_pre;
    const int len = rows ? B.rows : B.pitch, lane = threadIdx.x & 63;
    int acc = 0;
    for (int k0 = 0; k0 < len; k0 += 64) {
        const int k = k0 + lane;
        const unsigned long long set = __ballot(k < len && flag[k] != 0);
        if (k < len) pre[k] = acc + __popcll(set & ((1ull << lane) - 1ull));
        acc += __popcll(set);
    }
    if (lane == 0) pre[len] = acc;
}

// Field cotangents of one particle are summed in LDS (one slot per thread)
// while successive steps gather from the same 2 x 2 block of a component,
// and added to the gradient arrays with atomics when the block changes and
// at the end: a particle stays in a cell for a few steps, so this takes a
// few times fewer global atomics than adding every step.
//
// What bounds the sweep: FP64 issue, 61 % of the time with two waves per SIMD
// (255 VGPRs; 1e6 particles x 32 steps with a dense lambda on 512 x 512 in
// 4.9 ms, 1.63e9 VALU instructions; at one wave per SIMD 6.7 ms; with a tape
// that spilled to scratch 15 GB of traffic and 7.3 ms).  A workgroup is one
// wave (nothing is shared between its particles), so that small sets spread
// over the CUs: 20 KB of LDS each, eight per CU.  Workgroup b, on XCD b % 8,
// takes block (b % 8) per + b / 8: of particles in cell order each XCD then
// gathers from one band of rows, which its L2 holds.
constexpr int kBackThreads = 64;

// The three-corrector kernel's points: a thread's column of an LDS array.
struct PointSlots {
    double* p;
    __device__ double& at(int it, int c) { return p[(it * 4 + c) * kBackThreads]; }
};

template <int NC, bool SMALL>
__global__ __launch_bounds__(kBackThreads) __attribute__((amdgpu_waves_per_eu(2))) void push_deposit_backward_f64(
    const BackArgs B) {
    __shared__ double acc[6][4][kBackThreads];
    __shared__ uint32_t base[6][kBackThreads];
    __shared__ double slots[NC == kFastCorr ? 4 * kFastCorr : 1][kBackThreads];
    const int t = threadIdx.x;
    const int64_t block = ((int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * kBackThreads;
    if (block + t >= B.count) return;                   // (no barrier below: the slots are per thread)
    constexpr uint32_t kNone = ~0u;             // (a grid array is below 4 GiB)
    for (int c = 0; c < 6; ++c) base[c][t] = kNone;
    auto add4 = [&](double* g, uint32_t e, const double v[4]) {
        const uint32_t off[4] = {0u, (uint32_t)B.pitch, 1u, (uint32_t)B.pitch + 1u};
        for (int k = 0; k < 4; ++k)
            if (v[k] != 0.0) atomicAdd(g + e + off[k], v[k]);
    };
    auto flush = [&](int c) {
        const uint32_t e = base[c][t];
        if (e == kNone || !B.gradF[c]) return;
        const double v[4] = {acc[c][0][t], acc[c][1][t], acc[c][2][t], acc[c][3][t]};
        add4(B.gradF[c], e, v);
    };
    constexpr bool kSlots = NC == kFastCorr;
    adj::StepTape<typename std::conditional<kSlots, PointSlots, adj::PointArray<NC>>::type> T;
    if constexpr (kSlots) T.pts.p = &slots[0][t];
    backward_particle<NC, SMALL>(B, block, t, [&](int c, uint32_t e, size_t step, const double v[4]) {
        if (step) {                             // an array per step: nothing to sum over steps
            if (B.gradF[c]) add4(B.gradF[c] + step, e, v);
            return;
        }
        const bool same = base[c][t] == e;
        if (!same) {
            flush(c);
            base[c][t] = e;
        }
        for (int k = 0; k < 4; ++k) acc[c][k][t] = same ? acc[c][k][t] + v[k] : v[k];
    }, T);
    for (int c = 0; c < 6; ++c) flush(c);
}

size_t backward_aux_bytes(int rows, int pitch) {
    return (size_t)(2 * rows + 2 * pitch + 2) * sizeof(int);
}

hipError_t launch_push_deposit_backward(BackArgs B, void* aux, hipStream_t stream) {
    if (B.count <= 0) return hipSuccess;
    int* row_flag = static_cast<int*>(aux);
    int* col_flag = row_flag + B.rows;
    int* row_pre = col_flag + B.pitch;
    int* col_pre = row_pre + B.rows + 1;
    B.row_pre = row_pre;
    B.col_pre = col_pre;
    const int flags = B.rows + B.pitch;
    hipLaunchKernelGGL(lam_clear, dim3((unsigned)((flags + 255) / 256)), dim3(256), 0, stream, row_flag, flags);
    hipLaunchKernelGGL(lam_any, dim3((unsigned)((B.pitch + 255) / 256), (unsigned)((B.rows + kLamRows - 1) / kLamRows)),
                       dim3(256), 0, stream, B, row_flag, col_flag);
    hipLaunchKernelGGL(lam_prefix, dim3(1), dim3(128), 0, stream, B, row_flag, col_flag, row_pre, col_pre);
    const dim3 grid((unsigned)((B.count + 8 * kBackThreads - 1) / (8 * kBackThreads) * 8));   // a multiple of 8
    const bool small = 2.0 * B.dlnr <= kSmallArg && 2.0 * B.dth <= kSmallArg;
    const dim3 block(kBackThreads);
    if (B.ncorr == kFastCorr && small)
        hipLaunchKernelGGL((push_deposit_backward_f64<kFastCorr, true>), grid, block, 0, stream, B);
    else if (B.ncorr == kFastCorr)
        hipLaunchKernelGGL((push_deposit_backward_f64<kFastCorr, false>), grid, block, 0, stream, B);
    else if (small)
        hipLaunchKernelGGL((push_deposit_backward_f64<adj::kMaxCorr, true>), grid, block, 0, stream, B);
    else
        hipLaunchKernelGGL((push_deposit_backward_f64<adj::kMaxCorr, false>), grid, block, 0, stream, B);
    return hipGetLastError();
}

}  // namespace grpic
