// Linear fit of the POD coefficients (Sec. IV.A, eq. (63a)): the normal
// equations of the weighted, regularised least-squares problem, accumulated
// on the FP64 matrix cores, and their solution by a Cholesky factorisation
// in one workgroup.
//
// Rows of the problem: one energy row per configuration (G_c, E_ref_c) with
// weight w_e and one force row per atom coordinate (-dG/dr_{n,d}, F_ref_{n,d})
// with weight w_f; the weights multiply the squared residuals as in the loss
// of eq. (63b).  With every row augmented by its label, x = [a | b], the
// Gram matrix Z = sum_r w_r x_r^T x_r holds A^T W A, A^T W b and b^T W b in
// one (M+1) x (M+1) block.  The Gram sum is a dense contraction, so it runs
// on v_mfma_f64_16x16x4_f64: one MFMA adds the outer products of four rows
// for one 16 x 16 tile of Z.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "pod.h"
#include "pod_internal.h"

namespace pod {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int GRAM_WAVES = 4;          // waves per workgroup
constexpr int GRAM_THREADS = GRAM_WAVES * WAVE;
constexpr int GRAM_BLOCKS = 512;       // persistent: two workgroups per CU
constexpr int GRAM_ROWS = 32;          // rows per LDS chunk (8 MFMA k-steps)
constexpr int RED_SLICES = 16;         // first reduction pass: workgroup partials in 16 slices
constexpr int FIT_MAX_TILES = 8;       // M + 1 <= 128
constexpr int SOLVE_THREADS = 512;      // two waves per SIMD, 256 registers each
constexpr int SOLVE_MAX_M = 2 * WAVE;   // two right-hand-side rows per lane
static_assert(SOLVE_THREADS >= 4 * SOLVE_MAX_M, "four lanes per row of Z c");
constexpr int SOLVE_ROWS = SOLVE_THREADS / SOLVE_MAX_M;   // rows of Z loaded per turn, one column a thread
constexpr int SOLVE_Z = (SOLVE_MAX_M + SOLVE_ROWS) / SOLVE_ROWS;   // turns for M + 1 rows

// Upper-triangle tile pairs (ti <= tj) of a T x T tiling, row by row; pair
// p belongs to wave p % GRAM_WAVES.
template <int T>
struct TilePairs {
    static constexpr int n = T * (T + 1) / 2;
    int ti[n], tj[n];
    constexpr TilePairs() : ti{}, tj{} {
        int p = 0;
        for (int i = 0; i < T; ++i)
            for (int j = i; j < T; ++j) {
                ti[p] = i;
                tj[p] = j;
                ++p;
            }
    }
};

struct GramArgs {
    const double* X;   // R x M, leading dimension ldx
    const double* y;   // R labels (column M of the augmented rows), or null
    double ysign;      // label sign: +1 energy rows, -1 force rows (a = -dG/dr)
    long ldx;
    long R;
    int M;
    int vec;           // X is 16-byte aligned and ldx == M: 16-byte loads
    double* part;      // [gridDim.x][n pairs][256] workgroup partial tiles
};

// Value of a double held by lane `src` (uniform) of the wave.
__device__ __forceinline__ double lane_value(double x, int src) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(b & 0xffffffffLL), src);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), src);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// One wave's share of a chunk: for every k-step of four rows, the T tile
// operands of the rows (lane l: row k0 + l / 16, column 16 t + l % 16) from
// LDS, then one MFMA per owned tile pair.
template <int T, int W>
__device__ __forceinline__ void gram_chunk(const double* __restrict__ buf, int lane,
                                           f64x4 (&acc)[(TilePairs<T>::n + GRAM_WAVES - 1) / GRAM_WAVES]) {
    constexpr TilePairs<T> tp{};
    constexpr int NP = TilePairs<T>::n;
    constexpr int LDW = 16 * T + 2;
    const int rl = lane >> 4, cl = lane & 15;
#pragma unroll 1
    for (int k0 = 0; k0 < GRAM_ROWS; k0 += 4) {
        double v[T];
#pragma unroll
        for (int t = 0; t < T; ++t) v[t] = buf[(k0 + rl) * LDW + 16 * t + cl];
#pragma unroll
        for (int q = 0; W + GRAM_WAVES * q < NP; ++q) {
            const int p = W + GRAM_WAVES * q;
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[tp.ti[p]], v[tp.tj[p]], acc[q], 0, 0, 0);
        }
    }
}

// Gram partials of the augmented rows [X | ysign y]: chunks of GRAM_ROWS
// rows are dealt round-robin to the workgroups; the rows of a chunk are one
// contiguous block of GRAM_ROWS x M doubles, loaded in 16-byte pieces (T per
// thread) two chunks ahead of the products (register double-buffering, so
// two chunks per workgroup are in flight), then stored into a double-
// buffered LDS tile with padded rows; each wave accumulates its own tile
// pairs in registers.
template <int T>
__global__ __launch_bounds__(GRAM_THREADS, 2) void gram_kernel(GramArgs a) {
    constexpr int NP = TilePairs<T>::n;
    constexpr int QP = (NP + GRAM_WAVES - 1) / GRAM_WAVES;
    constexpr int LDW = 16 * T + 2;
    static_assert(GRAM_ROWS * 16 * T / 2 <= GRAM_THREADS * T, "T pieces of 16 bytes per thread cover a chunk");
    __shared__ double buf[2][GRAM_ROWS * LDW];
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int M = a.M;
    const long nchunks = (a.R + GRAM_ROWS - 1) / GRAM_ROWS;
    const long nfull = a.R / GRAM_ROWS;           // chunks without a ragged end
    const int npc = GRAM_ROWS * M / 2;            // 16-byte pieces per chunk
    const bool vec = a.vec != 0;                  // X 16-byte aligned with ldx == M

    for (int e = tid; e < 2 * GRAM_ROWS * LDW; e += GRAM_THREADS) (&buf[0][0])[e] = 0.0;
    // LDS position (row << 8 | column) of the first double of each piece
    int rc[T];
#pragma unroll
    for (int e = 0; e < T; ++e) {
        const int p = tid + GRAM_THREADS * e;
        rc[e] = p < npc ? (((2 * p) / M) << 8) | ((2 * p) % M) : -1;
    }
    f64x4 acc[QP];
#pragma unroll
    for (int q = 0; q < QP; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
    struct Regs {
        double2 x[T];
        double yv;
    };
    auto load = [&](long c, Regs& g) {
        const long r0 = c * GRAM_ROWS;
        if (vec && c < nfull) {
            const double2* base = reinterpret_cast<const double2*>(a.X + r0 * M);
#pragma unroll
            for (int e = 0; e < T; ++e) g.x[e] = rc[e] >= 0 ? base[tid + GRAM_THREADS * e] : double2{0.0, 0.0};
        } else {
#pragma unroll
            for (int e = 0; e < T; ++e) {
                double v0 = 0.0, v1 = 0.0;
                if (rc[e] >= 0) {
                    const int row = rc[e] >> 8, col = rc[e] & 255;
                    const int row1 = col + 1 < M ? row : row + 1, col1 = col + 1 < M ? col + 1 : 0;
                    if (r0 + row < a.R) v0 = a.X[(r0 + row) * a.ldx + col];
                    if (r0 + row1 < a.R) v1 = a.X[(r0 + row1) * a.ldx + col1];
                }
                g.x[e] = double2{v0, v1};
            }
        }
        g.yv = (tid < GRAM_ROWS && a.y && r0 + tid < a.R) ? a.ysign * a.y[r0 + tid] : 0.0;
    };
    auto store = [&](const Regs& g, double* b) {
#pragma unroll
        for (int e = 0; e < T; ++e) {
            if (rc[e] >= 0) {
                const int row = rc[e] >> 8, col = rc[e] & 255;
                b[row * LDW + col] = g.x[e].x;
                if (col + 1 < M) b[row * LDW + col + 1] = g.x[e].y;
                else b[(row + 1) * LDW] = g.x[e].y;
            }
        }
        if (tid < GRAM_ROWS) b[tid * LDW + M] = g.yv;
    };
    auto compute = [&](const double* b) {
        switch (wave) {
            case 0: gram_chunk<T, 0>(b, lane, acc); break;
            case 1: gram_chunk<T, 1>(b, lane, acc); break;
            case 2: gram_chunk<T, 2>(b, lane, acc); break;
            default: gram_chunk<T, 3>(b, lane, acc); break;
        }
    };
    const long G = gridDim.x;
    Regs ga, gb;
    long c = blockIdx.x;
    if (c < nchunks) load(c, ga);
    if (c + G < nchunks) load(c + G, gb);
    __syncthreads();
    int cur = 0;
    for (; c < nchunks; c += 2 * G) {
        store(ga, buf[cur]);
        __syncthreads();
        if (c + 2 * G < nchunks) load(c + 2 * G, ga);
        compute(buf[cur]);
        cur ^= 1;
        if (c + G >= nchunks) break;
        store(gb, buf[cur]);
        __syncthreads();
        if (c + 3 * G < nchunks) load(c + 3 * G, gb);
        compute(buf[cur]);
        cur ^= 1;
    }

    // result layout of the 16 x 16 x 4 FP64 product (checked on the device
    // with an in-bounds probe): lane l, element e holds tile entry
    // (row l / 16 + 4 e, column l % 16)
#pragma unroll
    for (int q = 0; q < QP; ++q) {
        const int p = wave + GRAM_WAVES * q;
        if (p < NP) {
            double* out = a.part + (static_cast<long>(blockIdx.x) * NP + p) * 256;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[((lane >> 4) + 4 * e) * 16 + (lane & 15)] = acc[q][e];
        }
    }
}

// First reduction pass: slice s of tile pair p sums the partials of
// workgroups s, s + S, s + 2S, ... (fixed order).
__global__ __launch_bounds__(256) void gram_slice_kernel(const double* __restrict__ part, int nb, int NP,
                                                         double* __restrict__ sl) {
    const int p = blockIdx.x, s = blockIdx.y, k = threadIdx.x;
    double v = 0.0;
    for (int b = s; b < nb; b += RED_SLICES) v += part[(static_cast<long>(b) * NP + p) * 256 + k];
    sl[(static_cast<long>(s) * NP + p) * 256 + k] = v;
}

struct ReduceArgs {
    const double* sl_e;     // [RED_SLICES][NP][256] energy-row slices
    const double* sl_f;     // [RED_SLICES][NP][256] force-row slices
    int has_e, has_f, NP, M, T;
    double w_e, w_f;
    int accumulate;
    double* Z;              // (M+1) x (M+1), row-major
};

// Z = w_e sum(energy slices) + w_f sum(force slices) (+ Z), fixed order;
// each element is written from its upper-triangle tile entry and mirrored.
__global__ __launch_bounds__(256) void gram_reduce_kernel(ReduceArgs a) {
    const int p = blockIdx.x;
    const int k = threadIdx.x;
    int ti = 0, rem = p;
    while (rem >= a.T - ti) {
        rem -= a.T - ti;
        ++ti;
    }
    const int tj = ti + rem;
    const int row = 16 * ti + k / 16, col = 16 * tj + k % 16;
    const int D = a.M + 1;
    if (row >= D || col >= D || row > col) return;
    double se = 0.0, sf = 0.0;
    for (int s = 0; s < RED_SLICES; ++s) {
        if (a.has_e) se += a.sl_e[(static_cast<long>(s) * a.NP + p) * 256 + k];
        if (a.has_f) sf += a.sl_f[(static_cast<long>(s) * a.NP + p) * 256 + k];
    }
    double v = a.w_e * se + a.w_f * sf;
    if (a.accumulate) v += a.Z[static_cast<long>(row) * D + col];
    a.Z[static_cast<long>(row) * D + col] = v;
    if (row != col) a.Z[static_cast<long>(col) * D + row] = v;
}

// (Z_AA + gamma I) c = Z_Ab by Cholesky on the symmetrically scaled matrix
// (unit diagonal, same solution), one workgroup with the matrix in LDS;
// loss = c^T Z_AA c - 2 c^T Z_Ab + Z_bb + gamma c^T c, the value of eq. (63a).
//
// Factorisation: blocked right-looking Cholesky with panels of 16 columns
// (three barriers per panel).  The right-hand side is one more row below the
// matrix, so the factorisation leaves L^-1 b in it and no forward sweep is
// left.  Wave 0 factors a diagonal block in registers (lane r holds row r,
// pivots and columns broadcast by readlane); the back substitution runs in
// wave 0 with the right-hand side in registers (lane l holds rows l and
// l + 64) and the factor's rows read eight steps ahead, so it needs no barrier.
// Z is read once, every load in flight together, and stays in registers for
// the objective.
// Bound by the serial chain of M pivots and M back-substitution steps:
// M = 103 144 -> 64 us (before: 256 threads, Z read twice, diagonal
// blocks and both sweeps through LDS).
__global__ __launch_bounds__(SOLVE_THREADS) void solve_kernel(int M, const double* __restrict__ Z, double gamma,
                                                              double* __restrict__ c, double* __restrict__ loss,
                                                              int* err) {
    extern __shared__ double lds[];
    const int D = M + 1;             // Z is D x D
    const int DS = D | 1;            // row stride in LDS (odd: columns without bank conflicts)
    double* S = lds;                 // D x DS: the matrix, below it the right-hand side
    double* sc = S + D * DS;         // M: 1 / sqrt(diag of the unscaled matrix)
    double* ipiv = sc + M;           // M: 1 / L_kk
    double* cv = ipiv + M;           // M: solution
    __shared__ int bad;
    __shared__ double red[SOLVE_THREADS / WAVE];
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1), wave = tid / WAVE;
    if (tid == 0) bad = 0;
    // columns 0 ... M - 1 of rows 0 ... M - 1 and, as row M, the right-hand side:
    // the interface puts it in column M; what the last row of Z holds left of
    // the corner is not read
    const int zr = tid / SOLVE_MAX_M, zc = tid % SOLVE_MAX_M;
    double z[SOLVE_Z];
#pragma unroll
    for (int q = 0; q < SOLVE_Z; ++q) {
        const int i = zr + q * SOLVE_ROWS;
        z[q] = i <= M && zc < M ? Z[i < M ? i * D + zc : zc * D + M] : 0.0;
    }
    const double zbb = Z[M * D + M];
    for (int i = tid; i < M; i += SOLVE_THREADS) sc[i] = Z[i * D + i];
    __syncthreads();
    if (tid < M) {
        const double d = sc[tid] + gamma;
        if (!(d > 0.0) || !isfinite(d)) {
            bad = 1;
            sc[tid] = 0.0;
        } else {
            sc[tid] = 1.0 / sqrt(d);
        }
    }
    __syncthreads();
    // scaled matrix, below it the scaled right-hand side
    if (zc < M) {
        const double sj = sc[zc];
#pragma unroll
        for (int q = 0; q < SOLVE_Z; ++q) {
            const int i = zr + q * SOLVE_ROWS;
            if (i <= M) S[i * DS + zc] = (z[q] + (i == zc ? gamma : 0.0)) * (i < M ? sc[i] : 1.0) * sj;
        }
    }
    __syncthreads();
    // blocked right-looking Cholesky, panels of 16 columns, lower triangle:
    // (1) wave 0 factors the diagonal block, (2) one thread per row below
    // solves the panel against it, (3) the trailing triangle takes the rank-16
    // update -- three barriers per panel
    for (int k0 = 0; k0 < M; k0 += 16) {
        const int kb = M - k0 < 16 ? M - k0 : 16;
        if (tid < WAVE) {
            const int r = tid & 15;                      // four copies of the block
            double a[16], pv = 1.0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                // (the last panel is completed with rows of the identity)
                const double s = S[(r < kb ? k0 + r : k0) * DS + (k0 + j < M ? k0 + j : M - 1)];
                a[j] = r >= kb || j >= kb ? (r == j ? 1.0 : 0.0) : s;
            }
            bool ok = true;                              // the same in every lane
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double d = lane_value(a[k], k);
                ok = ok && d > 0.0 && d < INFINITY;
                const double il = rsqrt(d);
                a[k] *= il;                              // row k: d / sqrt(d)
                pv = r == k ? il : pv;
#pragma unroll
                for (int j = k + 1; j < 16; ++j) a[j] -= a[k] * lane_value(a[k], j);
            }
            if (!ok) bad = 1;
            if (tid < kb) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (j <= r) S[(k0 + r) * DS + k0 + j] = a[j];
                ipiv[k0 + r] = pv;
            }
        }
        __syncthreads();
        if (bad) break;
        // the block's rows sit in the lanes of each working wave, so its entries
        // are readlanes, not loads
        const int b0 = k0 + kb;
        const int i = b0 + tid;
        if (b0 + wave * WAVE <= M) {
            const int is = i <= M ? i : M;
            const int fr = k0 + ((lane & 15) < kb ? (lane & 15) : 0);
            double x[16], f[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int col = k0 + q < M ? k0 + q : M - 1;   // (columns past the last are not kept)
                x[q] = S[is * DS + col];
                f[q] = S[fr * DS + col];
            }
            const double pl = ipiv[fr];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                x[q] *= lane_value(pl, q);
#pragma unroll
                for (int u = q + 1; u < 16; ++u) x[u] -= x[q] * lane_value(f[q], u);
            }
            if (i <= M) {
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (q < kb) S[i * DS + k0 + q] = x[q];
            }
        }
        if (b0 >= M) break;
        __syncthreads();
        // rank-16 update, one 16 x 16 tile of the trailing triangle per wave
        // and turn: four products of the FP64 matrix cores, whose operands
        // (lane l: row l % 16, column l / 16) are 8 loads a tile and lane
        // instead of 32 an entry
        const int nt = (M - b0 + 16) / 16;   // rows b0 ... M
        const int cl = lane & 15, rl = lane >> 4;
        for (int u = wave; u < nt * (nt + 1) / 2; u += SOLVE_THREADS / WAVE) {
            int ti = 0, rem = u;
            while (rem > ti) rem -= ++ti;
            const int r0 = b0 + 16 * ti, c0 = b0 + 16 * rem;
            const int ra = r0 + cl <= M ? r0 + cl : M, rb = c0 + cl <= M ? c0 + cl : M;
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 16; s += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(S[ra * DS + k0 + s + rl], S[rb * DS + k0 + s + rl], acc,
                                                           0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = r0 + rl + 4 * e, col = c0 + cl;
                if (row <= M && col <= row && col < M) S[row * DS + col] -= acc[e];
            }
        }
        __syncthreads();
    }
    __syncthreads();
    if (bad) {
        if (tid == 0) atomicOr(err, ERR_SINGULAR);
        for (int i = tid; i < M; i += SOLVE_THREADS) c[i] = 0.0;
        if (loss && tid == 0) *loss = NAN;
        return;
    }
    // back substitution L^T w = u: w_j = u_j / L_jj, u_i -= L_ji w_j for i < j
    if (tid < WAVE) {
        const int l = tid;
        const bool in0 = l < M, in1 = l + WAVE < M;
        const int l0 = in0 ? l : 0, l1 = in1 ? l + WAVE : 0;
        double r0 = S[M * DS + l0], r1 = S[M * DS + l1];
        constexpr int AHEAD = 8;
        double a0[AHEAD], a1[AHEAD], pj[AHEAD];
        auto rows = [&](int j) {                         // rows j, j - 1, ...
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                const int jq = j - q > 0 ? j - q : 0;
                a0[q] = S[jq * DS + l0];
                a1[q] = S[jq * DS + l1];
                pj[q] = ipiv[jq];
            }
        };
        rows(M - 1);
        for (int jb = M - 1; jb >= 0; jb -= AHEAD) {
            double b0[AHEAD], b1[AHEAD], pb[AHEAD];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                b0[q] = a0[q];
                b1[q] = a1[q];
                pb[q] = pj[q];
            }
            rows(jb - AHEAD);
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                const int j = jb - q;
                // (j < 0 changes no row)
                const double wj = lane_value(j < WAVE ? r0 : r1, j & (WAVE - 1)) * pb[q];
                const double d0 = r0 - b0[q] * wj, d1 = r1 - b1[q] * wj;
                r0 = l == j ? wj : l < j ? d0 : r0;
                r1 = l + WAVE == j ? wj : l + WAVE < j ? d1 : r1;
            }
        }
        if (in0) {
            cv[l] = r0 * sc[l];
            c[l] = cv[l];
        }
        if (in1) {
            cv[l + WAVE] = r1 * sc[l + WAVE];
            c[l + WAVE] = cv[l + WAVE];
        }
    }
    if (!loss) return;
    __syncthreads();
    // objective from the unmodified Gram blocks: the residual form
    // sum_i c_i ((Z c)_i - 2 Z_ib + gamma c_i) + Z_bb.  Z goes back to LDS and
    // four lanes share a row of Z c.
    if (zc < M) {
#pragma unroll
        for (int q = 0; q < SOLVE_Z; ++q) {
            const int i = zr + q * SOLVE_ROWS;
            if (i <= M) S[i * DS + zc] = z[q];
        }
    }
    __syncthreads();
    double part = 0.0;
    {
        const int i = tid >> 2, l = tid & 3;
        double q = 0.0;
        if (i < M)
            for (int j = l; j < M; j += 4) q += S[i * DS + j] * cv[j];
#pragma unroll
        for (int o = 1; o < 4; o <<= 1) q += __shfl_xor(q, o);
        if (i < M && l == 0) part = cv[i] * (q - 2.0 * S[M * DS + i] + gamma * cv[i]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) part += __shfl_xor(part, o);
    if ((tid & (WAVE - 1)) == 0) red[tid / WAVE] = part;
    __syncthreads();
    if (tid == 0) {
        double s = zbb;
        for (int w = 0; w < SOLVE_THREADS / WAVE; ++w) s += red[w];
        *loss = s;
    }
}

template <int T>
void launch_gram(const GramArgs& a, int nblk, hipStream_t s) {
    hipLaunchKernelGGL((gram_kernel<T>), dim3(nblk), dim3(GRAM_THREADS), 0, s, a);
}

void launch_gram_t(int T, const GramArgs& a, int nblk, hipStream_t s) {
    switch (T) {
        case 1: launch_gram<1>(a, nblk, s); break;
        case 2: launch_gram<2>(a, nblk, s); break;
        case 3: launch_gram<3>(a, nblk, s); break;
        case 4: launch_gram<4>(a, nblk, s); break;
        case 5: launch_gram<5>(a, nblk, s); break;
        case 6: launch_gram<6>(a, nblk, s); break;
        case 7: launch_gram<7>(a, nblk, s); break;
        default: launch_gram<8>(a, nblk, s); break;
    }
}

// Workgroups for R rows: one per chunk, at most GRAM_BLOCKS.
int gram_blocks(long R) {
    if (R <= 0) return 0;
    return static_cast<int>(std::min<long>(GRAM_BLOCKS, (R + GRAM_ROWS - 1) / GRAM_ROWS));
}

// The same for M <= 8: one wavefront, everything in registers (lane r < M holds
// row r, lane SOLVE_SMALL the right-hand side; unused rows are the identity's).
// The kernel above pays for a panel of 16 columns and eight wavefronts whatever
// M is: M = 2 11.4 us per call, 8 11.7; here 5.1 and 4.9.
constexpr int SOLVE_SMALL = 8;
__global__ __launch_bounds__(WAVE) void solve_small_kernel(int M, const double* __restrict__ Z, double gamma,
                                                           double* __restrict__ c, double* __restrict__ loss,
                                                           int* err) {
    constexpr int S = SOLVE_SMALL;
    const int D = M + 1;
    const int l = threadIdx.x;
    const bool row = l < M;
    double z[S], a[S], iv[S], w[S];
#pragma unroll
    for (int j = 0; j < S; ++j) {
        const bool in = j < M && (row || l == S);
        z[j] = in ? Z[row ? l * D + j : j * D + M] : 0.0;
    }
    const double zb = row ? Z[l * D + M] : 0.0, zbb = Z[M * D + M];
    const double d0 = row ? Z[l * D + l] + gamma : 1.0;
    bool ok = d0 > 0.0 && isfinite(d0);
    const double sc = ok ? 1.0 / sqrt(d0) : 0.0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
        const double v = (z[j] + (row && l == j ? gamma : 0.0)) * sc * lane_value(sc, j);
        a[j] = j < M && (row || l == S) ? v : l == j ? 1.0 : 0.0;
    }
    double pv = 1.0;
#pragma unroll
    for (int k = 0; k < S; ++k) {
        const double d = lane_value(a[k], k);
        ok = ok && d > 0.0 && d < INFINITY;
        const double il = rsqrt(d);
        a[k] *= il;
        pv = l == k ? il : pv;
#pragma unroll
        for (int j = k + 1; j < S; ++j) a[j] -= a[k] * lane_value(a[k], j);
    }
    if (__any(!ok)) {   // as above: c = 0, loss NaN
        if (l == 0) atomicOr(err, ERR_SINGULAR);
        if (row) c[l] = 0.0;
        if (loss && l == 0) *loss = NAN;
        return;
    }
#pragma unroll
    for (int j = 0; j < S; ++j) iv[j] = lane_value(pv, j);
    double cl = 0.0;
#pragma unroll
    for (int j = S - 1; j >= 0; --j) {
        w[j] = lane_value(a[j], S);
#pragma unroll
        for (int i = j + 1; i < S; ++i) w[j] -= lane_value(a[j], i) * w[i];
        w[j] *= iv[j];
        cl = l == j ? w[j] * sc : cl;
    }
    if (row) c[l] = cl;
    if (!loss) return;
    double q = 0.0;
#pragma unroll
    for (int j = 0; j < S; ++j) q += z[j] * lane_value(cl, j);
    double part = row ? cl * (q - 2.0 * zb + gamma * cl) : 0.0;
#pragma unroll
    for (int o = S / 2; o >= 1; o >>= 1) part += __shfl_xor(part, o);
    if (l == 0) *loss = zbb + part;
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

}  // namespace
}  // namespace pod

extern "C" {

int pod_fit_gram(pod_handle* h, int M, int n_cfg, const double* G, const double* E_ref, double w_e, long n_frows,
                 const double* dGdR, const double* F_ref, double w_f, int accumulate, double* Z) {
    using namespace pod;
    if (!h || M < 1 || n_cfg < 0 || n_frows < 0 || !Z) return POD_EINVAL;
    if (M + 1 > 16 * FIT_MAX_TILES) return POD_ENOTSUP;
    if ((n_cfg > 0 && (!G || !E_ref)) || (n_frows > 0 && (!dGdR || !F_ref))) return POD_EINVAL;
    if (!std::isfinite(w_e) || !std::isfinite(w_f) || w_e < 0.0 || w_f < 0.0) return POD_EINVAL;
    const int T = (M + 1 + 15) / 16;
    const int NP = T * (T + 1) / 2;
    const int nb_e = gram_blocks(n_cfg), nb_f = gram_blocks(n_frows);
    const size_t tile_bytes = sizeof(double) * 256 * NP;
    const size_t be = align256(tile_bytes * nb_e), bf = align256(tile_bytes * nb_f);
    const size_t bs = align256(tile_bytes * RED_SLICES);
    const int rc = ensure_scratch(h, be + bf + 2 * bs);
    if (rc != POD_OK) return rc;
    char* base = static_cast<char*>(h->d_scratch);
    double* part_e = reinterpret_cast<double*>(base);
    double* part_f = reinterpret_cast<double*>(base + be);
    double* sl_e = reinterpret_cast<double*>(base + be + bf);
    double* sl_f = reinterpret_cast<double*>(base + be + bf + bs);
    timing_begin(h, 3);
    const int vec_e = (reinterpret_cast<uintptr_t>(G) & 15) == 0;
    const int vec_f = (reinterpret_cast<uintptr_t>(dGdR) & 15) == 0;
    if (nb_e > 0) launch_gram_t(T, GramArgs{G, E_ref, 1.0, M, n_cfg, M, vec_e, part_e}, nb_e, h->stream);
    if (nb_f > 0) launch_gram_t(T, GramArgs{dGdR, F_ref, -1.0, M, n_frows, M, vec_f, part_f}, nb_f, h->stream);
    timing_end(h, 3);
    if (nb_e > 0)
        hipLaunchKernelGGL(gram_slice_kernel, dim3(NP, RED_SLICES), dim3(256), 0, h->stream, part_e, nb_e, NP, sl_e);
    if (nb_f > 0)
        hipLaunchKernelGGL(gram_slice_kernel, dim3(NP, RED_SLICES), dim3(256), 0, h->stream, part_f, nb_f, NP, sl_f);
    ReduceArgs r{sl_e, sl_f, nb_e > 0, nb_f > 0, NP, M, T, w_e, w_f, accumulate ? 1 : 0, Z};
    hipLaunchKernelGGL(gram_reduce_kernel, dim3(NP), dim3(256), 0, h->stream, r);
    return hipGetLastError() == hipSuccess ? POD_OK : POD_EHIP;
}

int pod_fit_solve(pod_handle* h, int M, const double* Z, double gamma, double* c, double* loss) {
    using namespace pod;
    if (!h || M < 1 || !Z || !c) return POD_EINVAL;
    if (!std::isfinite(gamma) || gamma < 0.0) return POD_EINVAL;
    const size_t lds = sizeof(double) * (static_cast<size_t>(M + 1) * ((M + 1) | 1) + 3 * static_cast<size_t>(M));
    if (M > SOLVE_MAX_M) return POD_ENOTSUP;
    if (lds > h->lds_max) return POD_ENOTSUP;
    if (M <= SOLVE_SMALL) {
        hipLaunchKernelGGL(solve_small_kernel, dim3(1), dim3(WAVE), 0, h->stream, M, Z, gamma, c, loss, h->d_err);
        return hipGetLastError() == hipSuccess ? POD_OK : POD_EHIP;
    }
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(solve_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(lds)) != hipSuccess)
        return POD_EHIP;
    hipLaunchKernelGGL(solve_kernel, dim3(1), dim3(SOLVE_THREADS), lds, h->stream, M, Z, gamma, c, loss, h->d_err);
    return hipGetLastError() == hipSuccess ? POD_OK : POD_EHIP;
}

}  // extern "C"
