// grpic_fields.hpp -- arguments and table layout of the field-solver kernels
// (fields.hip), shared with the C ABI in api.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace grpic {

// Planes of the table: inverse area elements per unit phi of the six
// components at their locations (zero where a component is not updated).
enum FieldTable { kT_iADr, kT_iADt, kT_iADp, kT_iABr, kT_iABt, kT_iABp, kTablePlanes };
// Radial edge lengths per row i = -2 .. nr + 1 (index i + 2): primal
// r_{i+1} - r_i and dual r_{i+1/2} - r_{i-1/2}.
enum { kDrPrimal, kDrDual, kDrRows };
constexpr int kTableRowLo = -2;                  // tables cover rows -2 .. nr + 1
// Radii r(x) at half-integer steps x = -2, -1.5, .. nr + 2 (2 nr + 9
// values) and sin, cos of theta at y = 0, 0.5, .. nth (2 nth + 1 values each).
__host__ __device__ inline int field_nrad(int nr) { return 2 * nr + 9; }
__host__ __device__ inline int field_nang(int nth) { return 2 * nth + 1; }

struct FieldArgs {
    double a, M, lnr0, dlnr, dth;
    int nr, nth, guard, pitch;
    size_t plane;                                 // elements of one grid array
    int nrow;                                     // rows of the radial-length table (nr + 4)
    double* tab;                                  // kTablePlanes planes
    double* drow;                                 // kDrRows x nrow
    double* rad;                                  // field_nrad(nr) radii
    double* sn;                                   // field_nang(nth) sines, then as many cosines
    const double* J[3];                           // flux-form currents (or NULL)
    double dt, w0, w1;
    __host__ __device__ uint32_t at(int i, int j) const { return (uint32_t)((i + guard) * pitch + (j + guard)); }
};

struct FieldPtrs {
    double* c[6];                                 // D^r, D^th, D^ph, B^r, B^th, B^ph (or E, H)
};

inline size_t field_plane(int nr, int pitch, int guard) { return (size_t)(nr + 1 + 2 * guard) * pitch; }
inline size_t field_tables_bytes(int nr, int nth, int pitch, int guard) {
    return sizeof(double) * (kTablePlanes * field_plane(nr, pitch, guard) + (size_t)kDrRows * (nr + 4) +
                             field_nrad(nr) + 2 * (size_t)field_nang(nth));
}
// Workspace: the corrector's constant part X^n + dt (w0 C(X^n) - J) and two
// buffers of corrector iterates: 18 grid arrays.
inline size_t field_workspace_bytes(int nr, int pitch, int guard) {
    return sizeof(double) * 18 * field_plane(nr, pitch, guard);
}

// Strips of 64 columns that a launch of K passes cuts columns 0 .. nth into:
// strip s loads columns s (64 - 2 K) and the 63 after it and stores those of
// them whose K neighbours on either side it holds too (the axes have none).
// A workgroup of two strips may hold one past the last: it stores nothing.
struct FieldStrips {
    int K, nth, count;
    __host__ __device__ FieldStrips(int K_, int nth_) : K(K_), nth(nth_), count(1) {
        const int rest = nth + 1 - 64;
        if (rest > 0) count += (rest + 63 - 2 * K) / (64 - 2 * K);
    }
    __host__ __device__ int first_column(int s) const { return s * (64 - 2 * K); }
    __host__ __device__ bool stores(int s, int lane) const {
        return s < count && first_column(s) + lane <= nth && (s == 0 || lane >= K) &&
               (s == count - 1 || lane < 64 - K);
    }
    // Does strip s store columns within `guard` of an axis, whose values the
    // columns beyond it take too?  They need not lie in the first or the last
    // strip: the last one stores as few as K + 1 columns.
    __host__ __device__ bool mirrors(int s, int guard) const {
        return first_column(s) + (s == 0 ? 0 : K) <= guard ||
               (s == count - 1 ? nth : first_column(s) + 63 - K) >= nth - guard;
    }
};

// Workgroups of one launch of K passes: strips and segments of rows.
// A workgroup's LDS (73.7 to 76.8 KB per strip with four passes) and its odd
// number of waves let a CU hold one workgroup of two strips, or one of one
// strip (two five-wave workgroups do not share a CU: their first SIMDs collide,
// measured 695 against 475 us per 2048 x 2048 step).  So with four passes: one
// strip per workgroup while segments of kMinSegRows rows fit one round of 256
// workgroups (a step of 256 x 256: 38 us against 46), else two strips and
// segments cut for one round.
// With fewer passes two one-strip workgroups can share a CU, which halves the
// segments.  That pays where the march's steps are the bound and not HBM: where
// a launch's arrays (24 planes) fit the 256 MB Infinity Cache, and on grids of one
// or three strips, where workgroups of two would leave a half idle.  Four
// passes in two launches: 20000 x 16 (one strip) 195 us in workgroups of two
// strips, 108 so, 20000 x 130 (three) 406 and 302, 2000 x 500 (194 MB) 111 and 97;
// but two strips in step read their halo columns once: 20000 x 400 (1.55 GB,
// seven) 792 and 813, 2048 x 2048 (0.81 GB) 400 and 422.
struct FieldMarch {
    static constexpr int kCus = 256, kMinSegRows = 6, kNarrow = 3, kMaxPasses = 4;
    static constexpr size_t kCacheBytes = (size_t)256 << 20;
    int strips, seg_rows, workgroups;
    bool two;                                     // two strips per workgroup
    FieldMarch(int K, int nr, int nth, size_t plane) : strips(FieldStrips(K, nth).count) {
        const int most = (nr + kMinSegRows) / kMinSegRows;
        const bool narrow = strips <= kNarrow && strips % 2 == 1;
        const bool share = K < kMaxPasses && (narrow || 24 * sizeof(double) * plane <= kCacheBytes);
        two = !share && (int64_t)strips * most > kCus;
        const int units = two ? (strips + 1) / 2 : strips;
        int segs = (share ? 2 * kCus : kCus) / units;
        segs = segs < 1 ? 1 : segs > most ? most : segs;
        seg_rows = (nr + segs) / segs;            // ceil((nr + 1) / segs)
        workgroups = units * ((nr + seg_rows) / seg_rows);
    }
};

hipError_t launch_field_tables(const FieldArgs& F, const double* gx, const double* gw, hipStream_t stream);
hipError_t launch_field_step(const FieldArgs& F, FieldPtrs X, FieldPtrs R, FieldPtrs W1, FieldPtrs W2, int ncorr,
                             int damp_cells, double damp_max, hipStream_t stream);

}  // namespace grpic
