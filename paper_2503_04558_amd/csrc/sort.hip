// sort.hip -- counting sort of particles by cell, and the tiling the tiled
// push kernel runs on.
//
// histogram of live cells -> exclusive scan (4096 entries per block, two
// launches, three on the largest grids) -> [tiling: per-tile slice counts of both cuts -> scan -> slice
// tables] ->
// scatter.  Histogram and scatter take a chunk of consecutive particles per
// workgroup and count its cells in an LDS hash table first, so each distinct
// cell of the chunk costs one global atomic: on the almost sorted input of a
// re-sort a chunk holds a few dozen cells, and per-particle (or per-run)
// atomics would queue on the same few counters.  Removed particles
// (cell < 0) are dropped and the tail of the output is marked removed; the
// order inside a cell is not specified.
#include "grpic_launch.hpp"

#include <algorithm>
#include <mutex>

namespace grpic {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;
// Up to this many tiles every block of the scan's second launch sums the totals
// before it (a launch fewer: sort of 1e3 particles on 4096 x 4096, 4097 tiles, 251
// us against 261); the sums grow with the square of the tiles, so beyond it the
// totals are scanned by a block of their own (8192 x 4096, 8193 tiles, 475 against
// 466; 23000 x 23000, 129,151 tiles, 11.2 against 7.1 ms).
constexpr unsigned kScanSelfSum = 8192;

int64_t sort_scan_blocks(int64_t len) { return (len + kScanTile - 1) / kScanTile; }

size_t sort_workspace_bytes(int nr, int nth) {
    const int64_t len = (int64_t)nr * nth + 1;
    const int64_t ntiles = (int64_t)nr * tiles_per_row(nth);
    return (size_t)(len + sort_scan_blocks(len) + 1 + ntiles + 1) * sizeof(unsigned long long);
}

// Before the histogram: the counts cleared and, with a tiling, its two slice
// tables emptied and its anchor table written (from the same anchor_r /
// anchor_sc as the untiled kernels' anchors).
__global__ __launch_bounds__(256) void sort_setup(const SortArgs S, int64_t len, Slice* __restrict__ slices, int64_t cap,
                                                  Slice* __restrict__ slices3, int64_t cap3,
                                                  double* __restrict__ anchors, int rows, int cols) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < len) S.counts[t] = 0ull;
    if (t < cap) slices[t] = Slice{-1, 0, 0};
    if (t < cap3) slices3[t] = Slice{-1, 0, 0};
    if (t >= rows && t >= cols) return;                 // without a tiling all four are zero
    StepArgs A;
    A.lnr0 = S.lnr0;
    A.dlnr = S.dlnr;
    A.dth = S.dth;
    if (t < rows) anchors[t] = anchor_r(A, (int)t - kMarginRows);
    if (t < cols) {
        double s, c;
        anchor_sc(A, (int)t - kMarginCols, s, c);
        anchors[rows + t] = s;
        anchors[rows + cols + t] = c;
    }
}

// Chunk of consecutive particles per histogram / scatter workgroup, and the
// LDS hash table that counts its cells: at most half full, so an empty slot
// is always found.  A scatter workgroup waits for its cells' atomics (with
// return, at the memory side) and writes a run per distinct cell; both are per
// chunk, and 2048-particle chunks beat 1024 (scatter of a drifted 2e8 5.8
// against 7.2 ms; 2e7 particles at 5 per cell, drifted by several rows, 1.20
// against 1.34 ms).  What bounds the scatter is the memory side, where chunks
// meet on the counters' lines: a thread's 16 atomics in flight together instead
// of one after another, 1.20 -> 1.45 ms; the particles exchanged through LDS
// and written in cell order, 1.20 -> 1.23 ms; chunks dealt to the XCDs in bands
// (neighbouring ones through one L2), 5.8 -> 7.0 ms for 2e8.  A slot's 8 bytes
// hold its cell and count and then, in the scatter, the cell's reserved output
// index.
constexpr int kChunkThreads = 256;
constexpr int kChunkItems = 8;
constexpr int kChunk = kChunkThreads * kChunkItems;
static_assert(kHashSlots == 2 * kChunk, "at most half full");
constexpr int kEmpty = -1;

union CellSlot {
    struct {
        int key;                       // cell, or kEmpty
        int count;                     // particles of the chunk in that cell
    };
    unsigned long long base;           // the scatter's output index of the first of them
};

__device__ __forceinline__ void table_clear(CellSlot* T) {
    for (int e = threadIdx.x; e < kHashSlots; e += kChunkThreads) T[e].base = 0x00000000FFFFFFFFull;   // kEmpty, 0
}

// Slot of cell c (inserted if new); adds inc to its count and returns the
// count before the add in old.  The cells of a 128-byte line of counters lie
// in neighbouring slots (CellPlace), so that consecutive threads of the flush
// add to consecutive counters: an atomic per line instead of one per cell
// (histogram of 2e7 drifted particles on 2048 x 2048 0.58 -> 0.20 ms, re-sort
// of 2e8 0.80 -> 0.54 ms).
__device__ __forceinline__ int table_insert(CellSlot* T, int c, int inc, int& old) {
    CellPlace at(c);
    for (int probe = 0; probe < kHashSlots; ++probe, at.next()) {
        const int slot = at.slot();
        const int k = atomicCAS(&T[slot].key, kEmpty, c);
        if (k == kEmpty || k == c) {
            old = atomicAdd(&T[slot].count, inc);
            return slot;
        }
    }
    old = 0;                           // not reached: at most kChunk keys in 2 * kChunk slots
    return -1;
}

// Runs of equal valid cells among adjacent lanes of a wave: the first lane
// of each run (head) and the run's last lane (tail).  Every lane of the
// wave must call it.
__device__ __forceinline__ void wave_runs(int c, bool valid, int& head, int& tail) {
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(c, 1);
    const int next = __shfl_down(c, 1);
    const unsigned long long heads = __ballot(valid && (lane == 0 || prev != c));
    const unsigned long long tails = __ballot(valid && (lane == 63 || next != c));
    head = 0;
    tail = 0;
    if (valid) {
        const unsigned long long upto = lane == 63 ? ~0ull : ((1ull << (lane + 1)) - 1ull);
        head = 63 - __clzll(heads & upto);
        const unsigned long long from = ~((1ull << head) - 1ull);
        tail = __ffsll((long long)(tails & from)) - 1;
    }
}

// Inserts the valid cells of one item per lane, one table access per run of
// equal cells; returns the lane's slot (-1 if not valid) and its rank among
// the chunk's particles of that cell.  Every lane of the wave must call it.
__device__ __forceinline__ int wave_insert(CellSlot* T, int c, bool valid, int& rank) {
    const int lane = threadIdx.x & 63;
    int head, tail;
    wave_runs(c, valid, head, tail);
    int slot = -1, old = 0;
    if (valid && lane == head) slot = table_insert(T, c, tail - head + 1, old);
    slot = __shfl(slot, head);
    old = __shfl(old, head);
    rank = old + (lane - head);
    return valid ? slot : -1;
}

__device__ __forceinline__ int64_t chunk_index(int k) {
    return (int64_t)blockIdx.x * kChunk + (int64_t)k * kChunkThreads + threadIdx.x;
}

// Histogram of live cells: counts[c] += number of particles in cell c.
__global__ __launch_bounds__(kChunkThreads) void sort_hist(const int32_t* __restrict__ cell, int64_t n, int ncell,
                                                           unsigned long long* __restrict__ counts) {
    __shared__ CellSlot T[kHashSlots];
    int c[kChunkItems];
    for (int k = 0; k < kChunkItems; ++k) {
        const int64_t p = chunk_index(k);
        c[k] = p < n ? cell[p] : -1;
    }
    table_clear(T);
    __syncthreads();
    for (int k = 0; k < kChunkItems; ++k) {
        int rank;
        wave_insert(T, c[k], c[k] >= 0 && c[k] < ncell, rank);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kHashSlots; e += kChunkThreads)
        if (T[e].key != kEmpty) atomicAdd(counts + T[e].key, (unsigned long long)T[e].count);
}

// Inclusive scan of one value per thread across a 256-thread block.
__device__ __forceinline__ unsigned long long block_inclusive_scan(unsigned long long v, unsigned long long* sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const unsigned long long add = threadIdx.x >= (unsigned)off ? sh[threadIdx.x - off] : 0ull;
        __syncthreads();
        sh[threadIdx.x] += add;
        __syncthreads();
    }
    return sh[threadIdx.x];
}

// What scan_tiles sums at entry i: the array itself, or the slice counts of
// tile i in both cuts, the cubic cut's in the upper 32 bits (their totals are
// at most n / 192 + ntiles, far below 2^32).
struct ScanSelf {
    const unsigned long long* a;
    __device__ unsigned long long operator()(int64_t i) const { return a[i]; }
};
struct ScanSlices {
    const unsigned long long* offs;     // the scanned cell counts
    int nth, tpr;
    int64_t ntiles;
    __device__ unsigned long long operator()(int64_t t) const {
        if (t >= ntiles) return 0ull;
        const int64_t i = t / tpr, jb = t - i * tpr;
        const int64_t c0 = i * nth + jb * kTileCells;
        const int64_t c1 = c0 + min((int64_t)kTileCells, nth - jb * kTileCells);
        const unsigned long long cnt = offs[c1] - offs[c0];
        return (cnt + kSliceThreads - 1) / kSliceThreads | ((cnt + kSliceThreads3 - 1) / kSliceThreads3) << 32;
    }
};

// Exclusive scan of each 4096-entry tile of v into a; the tile total goes to blocksums.
template <class V>
__global__ __launch_bounds__(256) void scan_tiles(V values, unsigned long long* a, int64_t len,
                                                  unsigned long long* __restrict__ blocksums) {
    __shared__ unsigned long long sh[kScanThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    unsigned long long v[kScanItems];
    unsigned long long tot = 0;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + k;
        v[k] = i < len ? values(i) : 0ull;
        tot += v[k];
    }
    const unsigned long long incl = block_inclusive_scan(tot, sh);
    unsigned long long run = incl - tot;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + k;
        if (i < len) a[i] = run;
        run += v[k];
    }
    if (threadIdx.x == kScanThreads - 1) blocksums[blockIdx.x] = incl;
}

// Exclusive scan of the tile totals in place, by one block.
__global__ __launch_bounds__(256) void scan_totals(unsigned long long* __restrict__ blocksums, int64_t nb) {
    __shared__ unsigned long long sh[kScanThreads];
    unsigned long long carry = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += kScanTile) {
        const int64_t base = c0 + (int64_t)threadIdx.x * kScanItems;
        unsigned long long v[kScanItems];
        unsigned long long tot = 0;
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = base + k < nb ? blocksums[base + k] : 0ull;
            tot += v[k];
        }
        const unsigned long long incl = block_inclusive_scan(tot, sh);
        unsigned long long run = carry + incl - tot;
        for (int k = 0; k < kScanItems; ++k) {
            if (base + k < nb) blocksums[base + k] = run;
            run += v[k];
        }
        carry += sh[kScanThreads - 1];
        __syncthreads();                                 // sh is written again
    }
}

// Adds the totals of the tiles before it to each tile: their sum, which every
// block forms itself, or the scanned totals' entry (SCANNED); copies of the
// result go to offsets and its last entry to last, where given.
template <bool SCANNED>
__global__ __launch_bounds__(256) void scan_finish(unsigned long long* __restrict__ a, int64_t len,
                                                   const unsigned long long* __restrict__ blocksums,
                                                   int64_t* __restrict__ offsets, int64_t* __restrict__ last) {
    __shared__ unsigned long long part[4];
    unsigned long long v = 0;
    if constexpr (SCANNED) {
        v = blocksums[blockIdx.x];
    } else {
        for (unsigned i = threadIdx.x; i < blockIdx.x; i += 256) v += blocksums[i];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
        __syncthreads();
        v = part[0] + part[1] + part[2] + part[3];
    }
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = (int64_t)blockIdx.x * kScanTile + k * 256 + threadIdx.x;
        if (i >= len) return;
        const unsigned long long x = a[i] + v;
        a[i] = x;
        if (offsets) offsets[i] = (int64_t)x;
        if (last && i == len - 1) *last = (int64_t)x;
    }
}

static inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

// Exclusive scan of v[0..len) into a (v[len-1] should be a zero sentinel so
// that a[len-1] receives the total).
template <class V>
static void scan_into(V v, unsigned long long* a, int64_t len, unsigned long long* blocksums, int64_t* offsets,
                      int64_t* last, hipStream_t stream) {
    const dim3 nb((unsigned)sort_scan_blocks(len));
    hipLaunchKernelGGL(scan_tiles<V>, nb, dim3(kScanThreads), 0, stream, v, a, len, blocksums);
    if (nb.x > kScanSelfSum) {
        hipLaunchKernelGGL(scan_totals, dim3(1), dim3(kScanThreads), 0, stream, blocksums, (int64_t)nb.x);
        hipLaunchKernelGGL(scan_finish<true>, nb, dim3(256), 0, stream, a, len, blocksums, offsets, last);
    } else {
        hipLaunchKernelGGL(scan_finish<false>, nb, dim3(256), 0, stream, a, len, blocksums, offsets, last);
    }
}

void scan_exclusive(unsigned long long* a, int64_t len, unsigned long long* blocksums, hipStream_t stream) {
    scan_into(ScanSelf{a}, a, len, blocksums, nullptr, nullptr, stream);
}

// Slice tables: tile t's particles cut into ns balanced slices; slice L (in
// tile order) goes to entry (L % per_xcd) * 8 + L / per_xcd, the workgroup
// that runs the L % per_xcd-th slice of XCD L / per_xcd's band.  Both cuts,
// whose counts ScanSlices packed; the header.
__global__ __launch_bounds__(256) void tile_slices(const unsigned long long* __restrict__ offs,
                                                   const unsigned long long* __restrict__ base, int nr, int nth,
                                                   int tpr, int64_t n, TilingHeader* hdr, Slice* __restrict__ slices,
                                                   int64_t cap, Slice* __restrict__ slices3, int64_t cap3) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t ntiles = (int64_t)nr * tpr;
    const unsigned long long all = base[ntiles];
    if (t == 0) {
        hdr->nslices = (int64_t)(all & 0xFFFFFFFFull);
        hdr->n = n;
        hdr->n_sorted = (int64_t)offs[(int64_t)nr * nth];
        hdr->nr = nr;
        hdr->nth = nth;
        hdr->tiles_per_row = tpr;
        hdr->tile_cells = kTileCells;
    }
    if (t >= ntiles) return;
    const int i = (int)(t / tpr), jb = (int)(t - (int64_t)i * tpr);
    const int64_t c0 = (int64_t)i * nth + (int64_t)jb * kTileCells;
    const int64_t c1 = c0 + min(kTileCells, nth - jb * kTileCells);
    const int64_t start = (int64_t)offs[c0];
    const int64_t cnt = (int64_t)offs[c1] - start;
    const unsigned long long b0 = base[t], b1 = base[t + 1];
    for (int cut = 0; cut < 2; ++cut) {
        const int64_t b = (int64_t)(b0 >> (32 * cut) & 0xFFFFFFFFull);
        const int64_t ns = (int64_t)(b1 >> (32 * cut) & 0xFFFFFFFFull) - b;
        if (ns <= 0) continue;
        const int64_t per_xcd = ((int64_t)(all >> (32 * cut) & 0xFFFFFFFFull) + 7) / 8;
        const int64_t each = (cnt + ns - 1) / ns;
        Slice* out = cut == 0 ? slices : slices3;
        const int64_t room = cut == 0 ? cap : cap3;
        for (int64_t s = 0; s < ns; ++s) {
            const int64_t s0 = s * each;
            Slice sl;
            sl.start = start + s0;
            sl.len = (int32_t)(cnt - s0 < each ? cnt - s0 : each);
            sl.tile = (int32_t)t;
            const int64_t L = b + s;
            const int64_t e = (L % per_xcd) * 8 + L / per_xcd;
            if (e < room) out[e] = sl;                   // always: room >= nslices + 8
        }
    }
}

// Scatter: counts[] holds each cell's next free output index; a chunk
// reserves its particles' range of every cell with one atomic and places
// them by their rank inside the chunk.  Elements of the output beyond the
// live count (counts[ncell], which no cell adds to) are marked removed by the
// chunk of the same elements.
template <class T>
__global__ __launch_bounds__(kChunkThreads) void sort_scatter(const SortArgs S) {
    __shared__ CellSlot Tb[kHashSlots];
    int c[kChunkItems];
    for (int k = 0; k < kChunkItems; ++k) {
        const int64_t p = chunk_index(k);
        c[k] = p < S.n ? S.cell_in[p] : -1;
    }
    // the particles' data is read first, so its latency overlaps the counting
    T v[kChunkItems][6], ph[kChunkItems];
    uint8_t spv[kChunkItems];
    uint64_t tg[kChunkItems];
    for (int k = 0; k < kChunkItems; ++k) {
        const int64_t p = chunk_index(k);
        const bool valid = c[k] >= 0 && c[k] < S.ncell;
        for (int a = 0; a < 6; ++a) v[k][a] = valid ? static_cast<const T*>(S.in[a])[p] : T(0);
        spv[k] = valid ? S.sp_in[p] : 0;
        ph[k] = valid && S.phi_in ? static_cast<const T*>(S.phi_in)[p] : T(0);
        tg[k] = valid && S.tag_in ? S.tag_in[p] : 0ull;
    }
    const int64_t total = (int64_t)S.counts[S.ncell];
    table_clear(Tb);
    __syncthreads();
    int slot[kChunkItems], rank[kChunkItems];
    for (int k = 0; k < kChunkItems; ++k) slot[k] = wave_insert(Tb, c[k], c[k] >= 0 && c[k] < S.ncell, rank[k]);
    __syncthreads();
    for (int e = threadIdx.x; e < kHashSlots; e += kChunkThreads) {
        const CellSlot sl = Tb[e];
        if (sl.key != kEmpty) Tb[e].base = atomicAdd(S.counts + sl.key, (unsigned long long)sl.count);
    }
    __syncthreads();
    for (int k = 0; k < kChunkItems; ++k) {
        const int64_t p = chunk_index(k);
        if (p >= total && p < S.n) S.cell_out[p] = -1;
        if (slot[k] < 0) continue;
        const int64_t q = (int64_t)Tb[slot[k]].base + rank[k];
        S.cell_out[q] = c[k];
        for (int a = 0; a < 6; ++a) static_cast<T*>(S.out[a])[q] = v[k][a];
        S.sp_out[q] = spv[k];
        if (S.phi_in) static_cast<T*>(S.phi_out)[q] = ph[k];
        if (S.tag_in) S.tag_out[q] = tg[k];
    }
}

static inline unsigned nchunk(int64_t n) { return (unsigned)((n + kChunk - 1) / kChunk); }

hipError_t launch_sort(const SortArgs& S, hipStream_t stream) {
    const int64_t len = (int64_t)S.ncell + 1;
    const int tpr = tiles_per_row(S.nth);
    const int64_t ntiles = (int64_t)S.nr * tpr;
    const TilingLayout L = S.tiling ? tiling_layout(S.n, S.nr, S.nth) : TilingLayout{};
    Slice *slices = nullptr, *slices3 = nullptr;
    double* anchors = nullptr;
    if (S.tiling) {
        slices = tiling_at<Slice>(S.tiling, L.slices);
        slices3 = tiling_at<Slice>(S.tiling, L.slices3);
        anchors = tiling_at<double>(S.tiling, L.anchors);
    }
    const int rows = S.tiling ? anchor_table_rows(S.nr) : 0, cols = S.tiling ? anchor_table_cols(S.nth) : 0;
    const int64_t setup = std::max(std::max(len, std::max(L.cap, L.cap3)), (int64_t)std::max(rows, cols));
    hipLaunchKernelGGL(sort_setup, dim3(nblk(setup)), dim3(256), 0, stream, S, len, slices, L.cap, slices3, L.cap3,
                       anchors, rows, cols);
    if (S.n > 0)
        hipLaunchKernelGGL(sort_hist, dim3(nchunk(S.n)), dim3(kChunkThreads), 0, stream, S.cell_in, S.n, S.ncell, S.counts);
    scan_into(ScanSelf{S.counts}, S.counts, len, S.blocksums, S.cell_offsets, S.n_alive, stream);
    if (S.tiling) {
        scan_into(ScanSlices{S.counts, S.nth, tpr, ntiles}, S.tile_slices, ntiles + 1, S.blocksums, nullptr, nullptr,
                  stream);
        hipLaunchKernelGGL(tile_slices, dim3(nblk(ntiles)), dim3(256), 0, stream, S.counts, S.tile_slices, S.nr, S.nth,
                           tpr, S.n, static_cast<TilingHeader*>(S.tiling), slices, L.cap, slices3, L.cap3);
    }
    if (S.n > 0) {
        if (S.elem == 8) hipLaunchKernelGGL(sort_scatter<double>, dim3(nchunk(S.n)), dim3(kChunkThreads), 0, stream, S);
        else hipLaunchKernelGGL(sort_scatter<float>, dim3(nchunk(S.n)), dim3(kChunkThreads), 0, stream, S);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- no-allocation sort
// The workspace of grpic_sort_noalloc: a file-scope device array that every
// GPU the library runs on holds until the process ends.  Host code never
// passes its name to a kernel (on the host the name is only a stand-in):
// its device address is looked up once per device, with that device
// current, and kept.
static __device__ __align__(256) unsigned char scratch[kSortScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t sort_scratch(void** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace grpic
