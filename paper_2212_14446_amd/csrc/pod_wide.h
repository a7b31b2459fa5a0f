// Energy path for models whose angular degree is above FAST_MAX_PA or whose
// radial-function count is above FAST_MAX_K (up to POD_MAX_P = 10 and
// POD_MAX_K = 12): one
// 256-thread workgroup per atom at a time, the atom's basis rows and their
// adjoint in LDS.  Internal to libpod; the host side of the energy path
// chooses it by the model's degree.
#pragma once

#include <hip/hip_runtime.h>

#include "pod_internal.h"
#include "pod_tables.h"

namespace pod {

constexpr int WIDE_THREADS = 256;
constexpr int WIDE_CHUNK = 32;          // pairs staged per step
constexpr int WIDE_MAX_BLOCKS = 2048;   // persistent workgroups
constexpr int WIDE_PARTS = 48;          // parts of a radial index's degree sums, at most

template <typename T>
struct WideArgs {
    ParamsT<T> prm;      // by value: read with scalar loads
    CellT<T> cell;
    int N, P;
    const T* pos;
    const int* offsets;
    const int* nbr_j;
    const int* shift;
    const T* coef;       // energy coefficients (mode 1)
    T* D;                // descriptors N x M (mode 0)
    T* E_atom;           // per-atom energy or null (mode 1)
    double* part;        // block partials [10 + M][nblk]: column 0 E, 10.. G (mode 1)
    double* wpart;       // block virial partials [9][nblk]
    T* gown;             // gather path: g of every pair
    double* Facc;        // atomic path: FP64 force accumulator (zero on entry)
    T* rec;              // pair records, P x rs (scratch)
    int rs;              // record stride: 4 + K, or 4 + 2 K with R'_k (mode 1)
    int want_G, want_back, want_W;
    int* err;
};

// LDS layout of one wide_kernel workgroup, in bytes: the energy coefficients
// (M), the monomial codes (NA ints) and factorials, 1 / a!, with 4-body terms the
// packed eq. (30a) tables (wide_tab_ints ints), the basis rows [K][row stride]
// (later the adjoint rows), the degree sums [K][PA + 1] and their parts
// [K][WIDE_PARTS], B_{k 0} (K), the pair records of a chunk [WIDE_CHUNK][4 +
// 2K], the divided powers of the unit vectors' components
// [WIDE_CHUNK][3][PA + 2], the wavefronts' gradient sums [4][WIDE_CHUNK][4],
// and a reduction area.
struct WideLds {
    size_t coef, code, fact, inv, tab, b, s, part, b0, r, pw, g, red, total;
};

__host__ __device__ constexpr size_t wide_align(size_t b) { return (b + 15) & ~size_t(15); }

// Row stride of the basis and adjoint rows: 17 modulo 32, so that two rows'
// runs of 16 doubles (the operand of a matrix instruction) fall into
// different LDS banks, and one entry of all rows (4-body terms) as well.
__host__ __device__ constexpr int wide_row(int NA) { return (NA + 15) / 32 * 32 + 17; }
// Stride of a pair's power table: three components with a leading zero
// (u^-1), made odd.
__host__ __device__ constexpr int wide_pw(int PA) { return (3 * (PA + 2)) | 1; }

// ints of the packed 4-body tables: per index p its triple and term range
// (3 KA4), the terms (NT4), the occurrence ranges (NA4 + 1), the
// occurrences (3 NT4) and the index of (a, 0, 0) per degree a
__host__ __device__ constexpr int wide_tab_ints() {
    return 3 * n_partitions(POD_MAX_P4) + 4 * D4Table<POD_MAX_P4>::NT + n_mono(POD_MAX_P4) + 1 + POD_MAX_P4 + 1;
}

// Of the packed tables, what the descriptors alone need: without the occurrences.
__host__ __device__ constexpr int wide_desc_ints() {
    return 3 * n_partitions(POD_MAX_P4) + D4Table<POD_MAX_P4>::NT;
}

// Descriptors alone (energy false) take no coefficients, radial derivatives and
// gradient sums, and keep the parts of the degree sums where the power table
// was: K = 12, P3 = 10, P4 = 6 in FP64 74 -> 50 KB, three workgroups per
// compute unit instead of two (15,840 atoms 330 -> 266 us without 4-body terms).
__host__ __device__ constexpr WideLds wide_lds(int K, int PA, int M, bool four, int tsize, bool energy) {
    const size_t ts = static_cast<size_t>(tsize);
    const size_t NA = static_cast<size_t>(n_mono(PA));
    WideLds L{};
    L.coef = 0;
    L.code = wide_align(L.coef + (energy ? static_cast<size_t>(M) * ts : 0));
    L.fact = wide_align(L.code + NA * sizeof(int));
    L.inv = wide_align(L.fact + NA * sizeof(float));
    L.tab = wide_align(L.inv + (POD_MAX_P + 1) * sizeof(double));
    L.b = wide_align(L.tab + (four ? static_cast<size_t>(energy ? wide_tab_ints() : wide_desc_ints()) * sizeof(int) : 0));
    L.s = wide_align(L.b + static_cast<size_t>(K) * wide_row(static_cast<int>(NA)) * ts);
    L.part = wide_align(L.s + static_cast<size_t>(K) * (PA + 1) * ts);
    const size_t part = wide_align(static_cast<size_t>(K) * WIDE_PARTS * ts);
    const size_t pw = wide_align(static_cast<size_t>(WIDE_CHUNK) * wide_pw(PA) * ts);
    L.b0 = L.part + (energy ? part : part > pw ? part : pw);
    L.r = wide_align(L.b0 + static_cast<size_t>(K) * ts);
    const size_t r = wide_align(L.r + static_cast<size_t>(WIDE_CHUNK) * (4 + (energy ? 2 : 1) * K) * ts);
    L.pw = energy ? r : L.part;
    L.g = energy ? L.pw + pw : r;
    L.red = wide_align(L.g + (energy ? 4 * static_cast<size_t>(WIDE_CHUNK) * 4 * ts : 0));
    L.total = wide_align(L.red + 16 * sizeof(double));
    return L;
}

inline int wide_blocks(int N) { return N < WIDE_MAX_BLOCKS ? N : WIDE_MAX_BLOCKS; }
// Descriptors leave no partials per workgroup, so with 4-body terms, whose long
// term lists dwarf a workgroup's start, four times as many even out the last
// turn of the chip (K = 12, P4 = 6 1,178 -> 1,132 us FP64, 861 -> 779 FP32;
// without 4-body terms 266 -> 290 us, so those keep wide_blocks).
inline int wide_desc_blocks(int N) { return N < 4 * WIDE_MAX_BLOCKS ? N : 4 * WIDE_MAX_BLOCKS; }

// The energy path of a model with K radial functions and angular degree PA
// runs here when either exceeds what the register-resident kernels hold.
inline bool wide_path(int K, int PA) { return PA > FAST_MAX_PA || K > FAST_MAX_K; }

// Pair-record stride and bytes for P pairs.
inline int wide_rec_stride(int K, bool deriv) { return 4 + (deriv ? 2 : 1) * K; }

// mode 0: descriptors; mode 1: energy, and with want_back the pair
// gradients.  The pair records go to a.rec (P x a.rs values); then nblk
// workgroups take the atoms i = blk, blk + nblk, ...
template <typename T>
hipError_t launch_wide(const WideArgs<T>& a, int mode, bool fast, int nblk, hipStream_t st);

}  // namespace pod
