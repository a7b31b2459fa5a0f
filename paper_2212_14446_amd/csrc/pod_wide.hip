// Energy path for angular degree 7 to 10 (and K up to 12): the largest POD
// models of Table 6, whose atomic-basis rows (up to 286 monomials per radial
// function, eq. (23b)) do not fit a lane's registers.  Two kernels:
//
// wide_pair_kernel (16 lanes per atom): one record per listed pair --
//   [rhat (3), r, R_k (K) (, R'_k (K))] (Sec. II.A, II.B) -- with R = R' = 0
//   and rhat = 0 for a listed pair beyond the cut-off.
// wide_kernel: one 256-thread workgroup serves one atom at a time
//   (persistent over the atoms i = blk, blk + nblk, ...):
//   1. basis (eq. (24b)) as a matrix product over the pairs on the matrix
//      cores, B_{k n} = sum_p R_k(p) A_n(p): the records of WIDE_CHUNK pairs and
//      the powers of their unit vectors' components are staged in LDS;
//      wavefront w takes the 16-monomial tiles w, w + 4, .. (16 radial rows, 4
//      pairs per instruction) and forms A_n from three powers; the rows then
//      go to LDS;
//   2. contraction: degree sums S_{k a} = sum_{|n| = a} c_n B_{k n}^2,
//      thread d forms descriptor d: D2 = B_{k 0} (eq. (25)), D3 = S
//      (eq. (26a)), D4 by eq. (27a) for (a, 0, 0) and by the merged terms of
//      eq. (30a) otherwise; the energy (eq. (57a)) and the G partials;
//   3. adjoint dE_i/dB_{k n} by the product rule on the same formulas, the
//      4-body part gathered per monomial from a table of its occurrences in
//      the eq. (30a) terms (fixed order, no atomics); row k overwrites basis
//      row k in LDS;
//   4. pair gradients (eq. (24c)): W'_n = sum_k Abar_{k n} R'_k and W_n = sum_k
//      Abar_{k n} R_k of 16 monomials and 16 pairs at a time on the matrix
//      cores; the lane that holds W', W of (n, p) adds W'_n A_n and W_n grad
//      A_n; g_ij = (sum W' A - rhat . q / r) rhat + q / r with q = sum W grad A
//      (Euler identity for the homogeneous A_n).  The sums over a pair's lanes
//      and wavefronts have a fixed order; g is stored at the pair's slot (or
//      added to the force accumulator).
// With divided powers u^a / a! the gradient of a monomial is another product of
// the same table (d/du lowers a); the basis rows are multiplied, and the
// adjoint rows pre-multiplied, by a! b! c!.
// Vector form of 1 and 4 (one monomial per thread with 12 radial values from
// LDS per pair; eight lanes per pair with K adjoint values from LDS per
// monomial), 15,840 atoms, K = 12, P3 = 10, FP64: 1,580 us of kernel; the operands
// now stay in registers: 730 us (per call 1,656 -> 791).
// E, G and the virial leave as per-workgroup partials that the energy path's
// finalize kernel sums in a fixed order.  Evaluating the radial functions in
// a kernel of their own keeps their constants and temporaries out of the
// per-atom kernel's registers and leaves it one dependent load (the record)
// per pair instead of three (index, position, then the arithmetic).
#include <hip/hip_runtime.h>

#include <cmath>

#include "pod.h"
#include "pod_device.h"
#include "pod_internal.h"
#include "pod_tables.h"
#include "pod_wide.h"

namespace pod {
namespace {

using namespace dev;

constexpr int WT = WIDE_THREADS;
constexpr int CH = WIDE_CHUNK;
constexpr int NWV = WT / WAVE;
constexpr int NA_MAX = n_mono(POD_MAX_P);                   // 286
constexpr int APT = (POD_MAX_K * n_mono(POD_MAX_P4) + WT - 1) / WT;   // 4-body adjoint entries per thread
constexpr int TPW = ((NA_MAX + 15) / 16 + NWV - 1) / NWV;   // 16-monomial tiles per wavefront
constexpr int KSTEP = (POD_MAX_K + 3) / 4;                  // matrix steps over the radial index
constexpr int DPT = 2;                                      // descriptor columns per thread
constexpr int NA4 = n_mono(POD_MAX_P4);                     // monomials that enter eq. (30a)
constexpr int KA4 = n_partitions(POD_MAX_P4);               // 23
constexpr int NT4 = D4Table<POD_MAX_P4>::NT;                // merged eq. (30a) terms

static_assert(1 + POD_MAX_K + POD_MAX_K * (POD_MAX_P + 1) + POD_MAX_K * KA4 <= DPT * WT,
              "descriptor columns per thread");
static_assert(CH % 16 == 0 && POD_MAX_K <= 16 && NWV == 4, "tiles of the matrix products");

// Monomial codes: a | b << 4 | c << 8 | degree << 12 | multinomial << 16
// (device order of pod_tables.h).  Packed eq. (30a) tables for 4-body indices
// p up to degree POD_MAX_P4 (Table 1 order, so a lower P4 uses a prefix):
// per p its triple a | b << 4 | c << 8 and term range; every merged term
// x | y << 7 | z << 14 | coefficient << 21 (sorted monomial indices); and for
// every monomial n < NA4 its occurrences in the terms, p | u << 5 | v << 12 |
// coefficient << 19 (u, v the other two monomials).  The packed layout is
// the one copied to LDS: [ptri KA4][tbeg KA4][tend KA4][term NT4][obeg NA4+1]
// [occ 3 NT4][index of (a, 0, 0) for a <= POD_MAX_P4].  The occurrences of a
// monomial are in term order, hence sorted by p.
struct WideTables {
    int code[NA_MAX];
    int tab[wide_tab_ints()];
};
constexpr int T_PTRI = 0, T_TBEG = KA4, T_TEND = 2 * KA4, T_TERM = 3 * KA4, T_OBEG = 3 * KA4 + NT4,
              T_OCC = 3 * KA4 + NT4 + NA4 + 1, T_PA00 = 3 * KA4 + 4 * NT4 + NA4 + 1;

constexpr WideTables make_wide_tables() {
    WideTables w{};
    constexpr MonoTable<POD_MAX_P> mt{};
    for (int n = 0; n < NA_MAX; ++n)
        w.code[n] = mt.ex[n][0] | (mt.ex[n][1] << 4) | (mt.ex[n][2] << 8) | (mt.deg[n] << 12) | (mt.mult[n] << 16);
    constexpr D4Build<POD_MAX_P4> d4{};
    for (int p = 0; p < KA4; ++p) {
        w.tab[T_PTRI + p] = d4.pa[p] | (d4.pb[p] << 4) | (d4.pc[p] << 8);
        w.tab[T_TBEG + p] = d4.tbeg[p];
        w.tab[T_TEND + p] = d4.tend[p];
    }
    for (int k = 0; k < NT4; ++k)
        w.tab[T_TERM + k] = d4.tx[k] | (d4.ty[k] << 7) | (d4.tz[k] << 14) | (d4.tc[k] << 21);
    for (int a = 0; a <= POD_MAX_P4; ++a) w.tab[T_PA00 + a] = n_partitions(a - 1);
    int cnt[NA4] = {};
    for (int k = 0; k < NT4; ++k) { ++cnt[d4.tx[k]]; ++cnt[d4.ty[k]]; ++cnt[d4.tz[k]]; }
    w.tab[T_OBEG] = 0;
    for (int n = 0; n < NA4; ++n) w.tab[T_OBEG + n + 1] = w.tab[T_OBEG + n] + cnt[n];
    int at[NA4] = {};
    for (int n = 0; n < NA4; ++n) at[n] = w.tab[T_OBEG + n];
    for (int k = 0; k < NT4; ++k) {
        const int x = d4.tx[k], y = d4.ty[k], z = d4.tz[k];
        const int own[3] = {x, y, z}, u[3] = {y, x, x}, v[3] = {z, z, y};
        for (int r = 0; r < 3; ++r)
            w.tab[T_OCC + at[own[r]]++] = d4.tp[k] | (u[r] << 5) | (v[r] << 12) | (d4.tc[k] << 19);
    }
    return w;
}

// field limits of the packing
constexpr int wide_max_term_coef() {
    constexpr D4Build<POD_MAX_P4> d4{};
    int mx = 0;
    for (int k = 0; k < NT4; ++k) mx = d4.tc[k] > mx ? d4.tc[k] : mx;
    return mx;
}
static_assert(NA4 <= 128 && KA4 <= 32 && POD_MAX_P <= 15 && wide_max_term_coef() < 2048, "packed table fields");

__device__ const WideTables kWide = make_wide_tables();

// 4-body index of the triple (a, 0, 0): the first triple of degree a.
__device__ __forceinline__ int p_a00(const int* tab, int a) { return tab[T_PA00 + a]; }

// 16 x 16 x 4 matrix instruction of the working precision: operands A[i][k] and
// B[k][j] in lane 16 k + i (j); element e of lane 16 g + j is row row(g, e),
// column j of the result.
template <typename T> struct Mx;
template <> struct Mx<double> {
    typedef double vec __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ vec mul(double a, double b, vec c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int e) { return g + 4 * e; }
};
template <> struct Mx<float> {
    typedef float vec __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ vec mul(float a, float b, vec c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int e) { return 4 * g + e; }
};

// Divided powers u^a / a!, a = 0 .. PA, behind a leading zero (inv[a] = 1 / a!).
// The power runs in double and is divided once, so that an FP32 entry has one
// rounding, and an FP64 entry the power's and one more (the quotient is corrected
// by its remainder).  With one factor u * (1 / a) per step the rounding of 1 / 3,
// 1 / 5, ... was the same for every pair and atom: degree 10 of the descriptors
// was off by 2.2e-7 on average in FP32, now by 2e-8 as with plain powers.
template <typename T>
__device__ __forceinline__ void divided_powers(T* pw, T u, int PA, const double* inv) {
    pw[0] = T(0);
    double v = 1.0, f = 1.0;
    pw[1] = T(1);
    for (int a = 1; a <= PA; ++a) {
        v *= static_cast<double>(u);
        f *= a;
        double q = v * inv[a];
        if (sizeof(T) == 8) q = fma(fma(-q, f, v), inv[a], q);
        pw[a + 1] = static_cast<T>(q);
    }
}

// Parts of the degree sums S_a = sum_{|n| = a} c_n B_n^2: runs of at most
// PART_LEN monomials of one degree, so that no thread adds a long run alone.
constexpr int PART_LEN = 8;
constexpr int part_begin(int a) {      // parts of the degrees below a
    int p = 0;
    for (int d = 0; d < a; ++d) p += (n_of_degree(d) + PART_LEN - 1) / PART_LEN;
    return p;
}
struct PartTable {
    int begin[POD_MAX_P + 2];
    constexpr PartTable() : begin{} {
        for (int a = 0; a < POD_MAX_P + 2; ++a) begin[a] = part_begin(a);
    }
};
__device__ const PartTable kParts = PartTable();
static_assert(part_begin(POD_MAX_P + 1) <= WIDE_PARTS, "parts of the degree sums");

// Sum over the workgroup in a fixed order (shuffles within each wavefront,
// then the four wavefront sums in order); every thread gets the result.
__device__ __forceinline__ double block_sum(double v, double* red) {
    v = wave_sum(v);
    const int tid = threadIdx.x;
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    const double s = (red[0] + red[1]) + (red[2] + red[3]);
    return s;
}

// Pair records: 16 lanes per atom walk its list range.
template <typename T, bool DERIV, bool FAST>
__global__ __launch_bounds__(WT) void wide_pair_kernel(WideArgs<T> g) {
    __shared__ T sQ[POD_MAX_L * POD_MAX_K];
    const ParamsT<T>& prm = g.prm;
    const int tid = threadIdx.x;
    if (FAST)
        for (int k = tid; k < POD_MAX_L * POD_MAX_K; k += WT) sQ[k] = (&prm.Q[0][0])[k];
    __syncthreads();
    const int K = prm.K, RS = g.rs;
    const int i = blockIdx.x * (WT / 16) + tid / 16, l = tid % 16;
    int eb = 0;
    if (i < g.N) {
        const int b = g.offsets[i], e = g.offsets[i + 1];
        if (b < 0 || e < b || e > g.P) {
            eb |= ERR_NEIGH;
        } else {
            const T pi[3] = {g.pos[3 * i], g.pos[3 * i + 1], g.pos[3 * i + 2]};
            for (int p = b + l; p < e; p += 16) {
                const SlotIdx si = slot_index(g, true, p);
                T pj[3], d[3], r;
                slot_pos<T>(g, si, pj);
                const bool ok = slot_geometry<T>(g, true, si, pj, pi, eb, d, r);
                const T ri = T(1) / r;
                T R[POD_MAX_K], dR[POD_MAX_K];
                if constexpr (FAST) radial_std<T, DERIV>(&prm, sQ, r, ri, R, dR);
                else radial<T, DERIV>(&prm, r, ri, R, dR);
                T* rec = g.rec + static_cast<size_t>(p) * RS;
                rec[0] = ok ? d[0] * ri : T(0);
                rec[1] = ok ? d[1] * ri : T(0);
                rec[2] = ok ? d[2] * ri : T(0);
                rec[3] = r;
#pragma unroll
                for (int k = 0; k < POD_MAX_K; ++k)
                    if (k < K) {
                        rec[4 + k] = ok ? R[k] : T(0);
                        if (DERIV) rec[4 + K + k] = ok ? dR[k] : T(0);
                    }
            }
        }
    }
    eb = wave_or(eb);
    if ((tid & 63) == 0 && eb) atomicOr(g.err, eb);
}

// VL: the virial's sums in LDS (one column per thread of the gradient's end)
// instead of 18 registers of every thread.
template <typename T, int MODE, bool VL, bool FOUR>
__device__ __forceinline__ void wide_body(const WideArgs<T>& g) {
    extern __shared__ __align__(16) unsigned char smem[];
    const ParamsT<T>& prm = g.prm;
    const int K = prm.K, PA = prm.PA, M = prm.M;
    const int NA = n_mono(PA);
    const int NR = wide_row(NA);       // row stride of the basis rows
    const int PA1 = PA + 1, PA2 = PA + 2, PST = wide_pw(PA);
    const int nt = (NA + 15) / 16;     // 16-monomial tiles
    const bool four = MODE == 1 ? FOUR : prm.K4 > 0;   // 4-body terms
    const WideLds L = wide_lds(K, PA, M, four, static_cast<int>(sizeof(T)), MODE == 1);
    T* sC = reinterpret_cast<T*>(smem + L.coef);
    int* sCode = reinterpret_cast<int*>(smem + L.code);
    int* sTab = reinterpret_cast<int*>(smem + L.tab);
    T* sB = reinterpret_cast<T*>(smem + L.b);
    T* sS = reinterpret_cast<T*>(smem + L.s);
    T* sPart = reinterpret_cast<T*>(smem + L.part);
    T* sB0 = reinterpret_cast<T*>(smem + L.b0);
    T* sR = reinterpret_cast<T*>(smem + L.r);      // [q][RS]: rhat, r, R_k (, R'_k)
    T* sP = reinterpret_cast<T*>(smem + L.pw);
    __shared__ int sPartDef[WIDE_PARTS];
    auto part_begin_of = [](int a) { return kParts.begin[a]; };   // parts of the degrees below a
    double* sInv = reinterpret_cast<double*>(smem + L.inv);
    T* sG4 = reinterpret_cast<T*>(smem + L.g);     // [wavefront][q][4]
    float* sFact = reinterpret_cast<float*>(smem + L.fact);   // a! b! c!
    double* sRed = reinterpret_cast<double*>(smem + L.red);
    const int tid = threadIdx.x;
    const int lane = tid % WAVE, wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int c16 = lane & 15, gq = lane >> 4;

    if (tid <= POD_MAX_P) {
        double f = 1.0;
        for (int a = 2; a <= tid; ++a) f *= a;
        sInv[tid] = 1.0 / f;
    }
    for (int n = tid; n < NA; n += WT) {
        const int cd = kWide.code[n];
        sCode[n] = cd;
        float f = 1.0f;                // exact: at most 10!
        for (int x = 0; x < 3; ++x)
            for (int a = 2; a <= ((cd >> (4 * x)) & 15); ++a) f *= static_cast<float>(a);
        sFact[n] = f;
    }
    if (MODE == 1)
        for (int k = tid; k < M; k += WT) sC[k] = g.coef[k];
    if (four)
        for (int k = tid; k < (MODE == 1 ? wide_tab_ints() : wide_desc_ints()); k += WT) sTab[k] = kWide.tab[k];
    __syncthreads();

    const int K2 = prm.K2, K3 = prm.K3, K4 = prm.K4, P3 = prm.P3, P4 = prm.P4, KA = prm.Ka4;
    const int off3 = prm.off3, off4 = prm.off4;
    // parts: first and end monomial and degree
    for (int a = 0; a < PA1; ++a) {
        const int p0 = part_begin_of(a);
        const int m0 = n_mono(a - 1), m1 = n_mono(a);
        for (int x = tid; x < part_begin_of(a + 1) - p0; x += WT) {
            const int x0 = m0 + x * PART_LEN;
            sPartDef[p0 + x] = x0 | ((x0 + PART_LEN < m1 ? x0 + PART_LEN : m1) << 10) | (a << 20);
        }
    }
    __syncthreads();
    // power-table offsets of this lane's monomial of each of the wavefront's tiles
    int moff[TPW];
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        const int n = 16 * (wv + NWV * j) + c16;
        const int cd = n < NA ? sCode[n] : 0;
        moff[j] = (1 + (cd & 15)) | ((PA2 + 1 + ((cd >> 4) & 15)) << 8) | ((2 * PA2 + 1 + ((cd >> 8) & 15)) << 16);
    }

    double gacc[DPT] = {0.0, 0.0};
    double eacc = 0.0;
    __shared__ double sVir[VL ? 9 * CH : 1];
    double vir[VL ? 1 : 9];
    if constexpr (VL) {
        for (int t = tid; t < 9 * CH; t += WT) sVir[t] = 0.0;
    } else {
#pragma unroll
        for (int c = 0; c < 9; ++c) vir[c] = 0.0;
    }
    int eb = 0;

    const int RS = g.rs;
    const int np = part_begin_of(PA1);
    // list range of atom i (empty when malformed)
    auto range = [&](int i, int& b, int& n) {
        b = 0;
        n = 0;
        if (i >= g.N) return;
        const int o0 = g.offsets[i], o1 = g.offsets[i + 1];
        if (o0 < 0 || o1 < o0 || o1 > g.P) {
            eb |= ERR_NEIGH;
            return;
        }
        b = o0;
        n = o1 - o0;
    };
    // the records of one chunk, NPRE values per thread, zero past its end
    constexpr int NPRE = (CH * (4 + 2 * POD_MAX_K) + WT - 1) / WT;
    T pre[NPRE];
    auto request = [&](int p, int n) {
        const int len = (n < CH ? n : CH) * RS;
        const T* rc = g.rec + static_cast<size_t>(p) * RS;
#pragma unroll
        for (int x = 0; x < NPRE; ++x) {
            const int t = tid + x * WT;
            pre[x] = t < len ? rc[t] : T(0);
        }
    };
    // records to LDS, then the divided powers of their unit vectors
    auto stage = [&]() {
#pragma unroll
        for (int x = 0; x < NPRE; ++x) {
            const int t = tid + x * WT;
            if (t < CH * RS) sR[t] = pre[x];
        }
        __syncthreads();
        if (tid < 3 * CH) {
            const int q = tid / 3, ax = tid - 3 * q;
            divided_powers(sP + q * PST + ax * PA2, sR[q * RS + ax], PA, sInv);
        }
        __syncthreads();
    };

    int b, n;
    range(blockIdx.x, b, n);
    request(b, n);
    for (int i = blockIdx.x; i < g.N; i += gridDim.x) {
        int bn, nn1;
        range(i + static_cast<int>(gridDim.x), bn, nn1);
        if (n == 0) __syncthreads();   // no stage() barrier before LDS is rewritten

        // ---- 1. atomic basis
        typename Mx<T>::vec acc[TPW];
#pragma unroll
        for (int j = 0; j < TPW; ++j) acc[j] = typename Mx<T>::vec{T(0), T(0), T(0), T(0)};
        for (int c0 = 0; c0 < n; c0 += CH) {
            if (c0 > 0) {
                __syncthreads();   // the previous chunk is no longer read
                request(b + c0, n - c0);
            }
            stage();
            const int nq = n - c0 < CH ? n - c0 : CH;
#pragma unroll 1
            for (int q0 = 0; q0 < nq; q0 += 4) {
                const int q = q0 + gq;
                const T Rk = c16 < K ? sR[q * RS + 4 + c16] : T(0);
                const T* pw = sP + q * PST;
#pragma unroll
                for (int j = 0; j < TPW; ++j)
                    if (wv + NWV * j < nt)
                        acc[j] = Mx<T>::mul(Rk, pw[moff[j] & 255] * pw[(moff[j] >> 8) & 255] * pw[moff[j] >> 16], acc[j]);
            }
        }
        // the next atom's records, in flight until its stage()
        if (n <= CH) request(bn, nn1);
#pragma unroll
        for (int j = 0; j < TPW; ++j) {
            const int nn = 16 * (wv + NWV * j) + c16;
            if (nn < NA) {
                const T f = T(sFact[nn]);
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const int k = Mx<T>::row(gq, e4);
                    if (k < K) sB[k * NR + nn] = acc[j][e4] * f;
                }
            }
        }
        __syncthreads();

        // ---- 2. parts of the degree sums; without 4-body terms the adjoint row
        // entries too (3.), which then depend on their own basis entry only
        const bool own_adj = MODE == 1 && !four && g.want_back;
        for (int t = tid; t < K * np; t += WT) {
            const int k = t / np, pt = t - k * np;
            const int pc = sPartDef[pt];
            const int a = pc >> 20, n0 = pc & 1023, n1 = (pc >> 10) & 1023;
            T* Bk = sB + k * NR;
            T s = T(0);
            const T c3 = own_adj && k < K3 && a <= P3 ? T(2) * sC[off3 + k * (P3 + 1) + a] : T(0);
            for (int nn = n0; nn < n1; ++nn) {
                const T v = Bk[nn], mv = T(sCode[nn] >> 16) * v;
                s += mv * v;
                if (own_adj) Bk[nn] = (c3 * mv + (nn == 0 && k < K2 ? sC[1 + k] : T(0))) * T(sFact[nn]);
                if (nn == 0) sB0[k] = v;
            }
            sPart[k * WIDE_PARTS + pt] = s;
        }
        __syncthreads();
        auto degree_sum = [&](int k, int a) {
            T s = T(0);
            for (int pt = part_begin_of(a); pt < part_begin_of(a + 1); ++pt) s += sPart[k * WIDE_PARTS + pt];
            return s;
        };
        if (four) {
            for (int w = tid; w < K * PA1; w += WT) sS[w] = degree_sum(w / PA1, w % PA1);
            __syncthreads();
        }
        double ep = 0.0;
#pragma unroll
        for (int j = 0; j < DPT; ++j) {
            const int dc = tid + j * WT;
            if (dc >= M) continue;
            T v;
            if (dc == 0) {
                v = T(1);
            } else if (dc < off3) {
                v = sB0[dc - 1];
            } else if (dc < off4) {
                const int k = (dc - off3) / (P3 + 1), a = (dc - off3) - k * (P3 + 1);
                v = degree_sum(k, a);
            } else {
                const int k = (dc - off4) / KA, p = (dc - off4) - k * KA;
                const T* Bk = sB + k * NR;
                const int tri = sTab[T_PTRI + p];
                if ((tri >> 4) == 0) {
                    v = Bk[0] * sS[k * PA1 + (tri & 15)];                           // eq. (27a)
                } else {
                    T v0 = T(0), v1 = T(0);
                    const int t1 = sTab[T_TEND + p];
                    int t = sTab[T_TBEG + p];
                    // four terms' twelve loads in flight (two: K = 12, P4 = 6
                    // FP64 1,132 us against 790, FP32 779 against 502)
                    for (; t + 3 < t1; t += 4) {                                    // eq. (30a)
                        const int ta = sTab[T_TERM + t], tb = sTab[T_TERM + t + 1];
                        const int tc = sTab[T_TERM + t + 2], td = sTab[T_TERM + t + 3];
                        const T xa = Bk[ta & 127], ya = Bk[(ta >> 7) & 127], za = Bk[(ta >> 14) & 127];
                        const T xb = Bk[tb & 127], yb = Bk[(tb >> 7) & 127], zb = Bk[(tb >> 14) & 127];
                        const T xc = Bk[tc & 127], yc = Bk[(tc >> 7) & 127], zc = Bk[(tc >> 14) & 127];
                        const T xd = Bk[td & 127], yd = Bk[(td >> 7) & 127], zd = Bk[(td >> 14) & 127];
                        v0 += T(ta >> 21) * xa * ya * za;
                        v1 += T(tb >> 21) * xb * yb * zb;
                        v0 += T(tc >> 21) * xc * yc * zc;
                        v1 += T(td >> 21) * xd * yd * zd;
                    }
                    for (; t < t1; ++t) {
                        const int ta = sTab[T_TERM + t];
                        v0 += T(ta >> 21) * Bk[ta & 127] * Bk[(ta >> 7) & 127] * Bk[(ta >> 14) & 127];
                    }
                    v = v0 + v1;
                }
            }
            if constexpr (MODE == 0) {
                g.D[static_cast<size_t>(i) * M + dc] = v;
            } else {
                ep += static_cast<double>(sC[dc]) * static_cast<double>(v);
                gacc[j] += static_cast<double>(v);
            }
        }
        if constexpr (MODE == 1) {
            ep = wave_sum(ep);
            if (lane == 0) sRed[wv] = ep;
            if (!g.want_back) __syncthreads();
        }
        if (MODE == 1 && g.want_back) {
            // ---- 3. adjoint dE_i/dB_{k n}, in place.  The 4-body part of an entry
            // reads other entries of its row, all with n < NA4: those parts are
            // formed first, for all rows at once, and kept over a barrier.
            // Neighbouring lanes take the radial indices of one monomial: they
            // walk the same occurrences and read rows an odd stride apart.  (One
            // row at a time left two thirds of the threads idle: 15,840 atoms,
            // K = 12, P4 = 6 FP64 5,100 -> 2,228 us per call.)
            if (four) {
                const T* cf = sC;
                const int n4 = NA < NA4 ? NA : NA4;
                T a4[APT];
#pragma unroll
                for (int j = 0; j < APT; ++j) {
                    a4[j] = T(0);
                    const int t = tid + j * WT;
                    if (t >= K * n4) continue;
                    const int nn = t / K, k = t - nn * K;
                    if (k >= K4) continue;
                    const T* Bk = sB + k * NR;
                    const T* c4 = cf + off4 + k * KA;
                    // occurrences are sorted by p: stop at the first p of a
                    // higher degree than the model's; four at a time
                    const int o0 = sTab[T_OBEG + nn], o1 = sTab[T_OBEG + nn + 1];
                    T v4 = T(0);
                    int o = o0;
                    for (; o + 3 < o1; o += 4) {                                      // eq. (30a)
                        const int oa = sTab[T_OCC + o], ob = sTab[T_OCC + o + 1];
                        const int oc = sTab[T_OCC + o + 2], od = sTab[T_OCC + o + 3];
                        if ((od & 31) >= KA) break;
                        v4 += c4[oa & 31] * T(oa >> 19) * Bk[(oa >> 5) & 127] * Bk[(oa >> 12) & 127];
                        v4 += c4[ob & 31] * T(ob >> 19) * Bk[(ob >> 5) & 127] * Bk[(ob >> 12) & 127];
                        v4 += c4[oc & 31] * T(oc >> 19) * Bk[(oc >> 5) & 127] * Bk[(oc >> 12) & 127];
                        v4 += c4[od & 31] * T(od >> 19) * Bk[(od >> 5) & 127] * Bk[(od >> 12) & 127];
                    }
                    for (; o < o1; ++o) {
                        const int oa = sTab[T_OCC + o];
                        if ((oa & 31) >= KA) break;
                        v4 += c4[oa & 31] * T(oa >> 19) * Bk[(oa >> 5) & 127] * Bk[(oa >> 12) & 127];
                    }
                    a4[j] = v4;
                }
                __syncthreads();   // every product of basis entries is formed
                // the parts that need the entry itself only
                auto entry = [&](int k, int nn, T v4) {
                    T* Bk = sB + k * NR;
                    const int cd = sCode[nn];
                    const int dg = (cd >> 12) & 15;
                    const T mult = T(cd >> 16);
                    const T Bn = Bk[nn];
                    T v = T(0);
                    if (nn == 0 && k < K2) v += cf[1 + k];
                    if (k < K3 && dg <= P3) v += T(2) * cf[off3 + k * (P3 + 1) + dg] * mult * Bn;
                    if (k < K4) {
                        const T* c4 = cf + off4 + k * KA;
                        if (nn == 0)
                            for (int a = 0; a <= P4; ++a) v += c4[p_a00(sTab, a)] * sS[k * PA1 + a];   // eq. (27a)
                        if (dg <= P4) v += c4[p_a00(sTab, dg)] * sB0[k] * T(2) * mult * Bn;
                    }
                    Bk[nn] = (v + v4) * T(sFact[nn]);
                };
#pragma unroll
                for (int j = 0; j < APT; ++j) {
                    const int t = tid + j * WT;
                    if (t < K * n4) entry(t - t / K * K, t / K, a4[j]);
                }
                for (int t = tid; t < K * (NA - n4); t += WT) entry(t - t / K * K, n4 + t / K, T(0));
                __syncthreads();
            }
            const T* sA = sB;   // adjoint rows [K][NR], times a! b! c!

            // ---- 4. pair gradients, eq. (24c)
            for (int c0 = 0; c0 < n; c0 += CH) {
                const int nc = n - c0 < CH ? n - c0 : CH;
                const int nq = (nc + 15) & ~15;
                if (n > CH) {
                    __syncthreads();
                    request(b + c0, n - c0);
                    stage();
                }
                for (int qt = 0; qt < nq; qt += 16) {
                    const int q = qt + c16;
                    const T* pw = sP + q * PST;
                    T Rk[KSTEP], dRk[KSTEP];
#pragma unroll
                    for (int s = 0; s < KSTEP; ++s) {
                        const int k = 4 * s + gq;
                        Rk[s] = k < K ? sR[q * RS + 4 + k] : T(0);
                        dRk[s] = k < K ? sR[q * RS + 4 + K + k] : T(0);
                    }
                    T sa = T(0), gv0 = T(0), gv1 = T(0), gv2 = T(0);
#pragma unroll 1
                    for (int tl = wv; tl < nt; tl += NWV) {
                        typename Mx<T>::vec w1{T(0), T(0), T(0), T(0)}, w2{T(0), T(0), T(0), T(0)};
                        const int na = 16 * tl + c16;
#pragma unroll
                        for (int s = 0; s < KSTEP; ++s) {
                            const int k = 4 * s + gq;
                            const T av = k < K && na < NA ? sA[k * NR + na] : T(0);
                            w1 = Mx<T>::mul(av, dRk[s], w1);
                            w2 = Mx<T>::mul(av, Rk[s], w2);
                        }
#pragma unroll
                        for (int e4 = 0; e4 < 4; ++e4) {
                            const int nn = 16 * tl + Mx<T>::row(gq, e4);
                            const int cd = sCode[nn < NA ? nn : 0];   // past the end W = 0
                            const T* px = pw + (cd & 15);
                            const T* py = pw + PA2 + ((cd >> 4) & 15);
                            const T* pz = pw + 2 * PA2 + ((cd >> 8) & 15);
                            const T xm = px[0], xa = px[1], ym = py[0], yb = py[1], zm = pz[0], zc = pz[1];
                            const T yz = yb * zc;
                            sa += w1[e4] * (xa * yz);
                            gv0 += w2[e4] * (xm * yz);
                            gv1 += w2[e4] * (ym * (xa * zc));
                            gv2 += w2[e4] * (zm * (xa * yb));
                        }
                    }
                    // sum over the pair's four lanes (fixed order)
#pragma unroll
                    for (int o = 16; o < WAVE; o <<= 1) {
                        sa += __shfl_xor(sa, o);
                        gv0 += __shfl_xor(gv0, o);
                        gv1 += __shfl_xor(gv1, o);
                        gv2 += __shfl_xor(gv2, o);
                    }
                    if (gq == 0) {
                        T* o4 = sG4 + (wv * CH + q) * 4;
                        o4[0] = sa; o4[1] = gv0; o4[2] = gv1; o4[3] = gv2;
                    }
                }
                // read before the barrier: the next stage() may overwrite the records
                const int q = tid < CH ? tid : 0, p = b + c0 + q;
                const T u[3] = {sR[q * RS + 0], sR[q * RS + 1], sR[q * RS + 2]};
                const T r = sR[q * RS + 3];
                __syncthreads();
                if (tid < nc) {
                    const T ri = T(1) / r;
                    const bool ok = u[0] * u[0] + u[1] * u[1] + u[2] * u[2] > T(0.5);
                    T sm[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        sm[x] = (sG4[q * 4 + x] + sG4[(CH + q) * 4 + x]) +
                                (sG4[(2 * CH + q) * 4 + x] + sG4[(3 * CH + q) * 4 + x]);
                    const T gv0 = sm[1], gv1 = sm[2], gv2 = sm[3];
                    const T sa = sm[0] - (u[0] * gv0 + u[1] * gv1 + u[2] * gv2) * ri;
                    const T gx = ok ? sa * u[0] + ri * gv0 : T(0);
                    const T gy = ok ? sa * u[1] + ri * gv1 : T(0);
                    const T gz = ok ? sa * u[2] + ri * gv2 : T(0);
                    {
                        if (g.gown) {
                            T* go = g.gown + 3 * static_cast<size_t>(p);
                            go[0] = gx; go[1] = gy; go[2] = gz;
                        } else if (ok && g.Facc) {
                            const int j = g.nbr_j[p];
                            atomicAdd(&g.Facc[3 * j + 0], -static_cast<double>(gx));
                            atomicAdd(&g.Facc[3 * j + 1], -static_cast<double>(gy));
                            atomicAdd(&g.Facc[3 * j + 2], -static_cast<double>(gz));
                            atomicAdd(&g.Facc[3 * i + 0], static_cast<double>(gx));
                            atomicAdd(&g.Facc[3 * i + 1], static_cast<double>(gy));
                            atomicAdd(&g.Facc[3 * i + 2], static_cast<double>(gz));
                        }
                        if (ok) {
                            const double dd[3] = {static_cast<double>(u[0] * r), static_cast<double>(u[1] * r),
                                                  static_cast<double>(u[2] * r)};
                            const double gg[3] = {static_cast<double>(gx), static_cast<double>(gy),
                                                  static_cast<double>(gz)};
    #pragma unroll
                            for (int x = 0; x < 3; ++x)
    #pragma unroll
                                for (int y = 0; y < 3; ++y) {
                                if constexpr (VL) sVir[(3 * x + y) * CH + tid] -= dd[x] * gg[y];
                                else vir[3 * x + y] -= dd[x] * gg[y];
                            }
                        }
                    }
                }
            }
        }
        if constexpr (MODE == 1) {
            // sRed was written before the last barrier
            if (n == 0 && g.want_back) __syncthreads();
            if (tid == 0) {
                const double Ei = (sRed[0] + sRed[1]) + (sRed[2] + sRed[3]);
                if (g.E_atom) g.E_atom[i] = static_cast<T>(Ei);
                eacc += Ei;
            }
        }
        if (n > CH) request(bn, nn1);
        b = bn;
        n = nn1;
    }
    if constexpr (MODE == 1) __syncthreads();

    // block partials (every thread takes part in the reductions)
    const int blk = blockIdx.x, nblk = gridDim.x;
    if constexpr (MODE == 1) {
        if (tid == 0) g.part[blk] = eacc;
        if (g.want_G) {
#pragma unroll
            for (int j = 0; j < DPT; ++j) {
                const int dc = tid + j * WT;
                if (dc < M) g.part[static_cast<size_t>(10 + dc) * nblk + blk] = gacc[j];
            }
        }
        if (g.want_W) {
#pragma unroll
            for (int c = 0; c < 9; ++c) {
                double v;
                if constexpr (VL) v = block_sum(tid < CH ? sVir[c * CH + tid] : 0.0, sRed);
                else v = block_sum(vir[c], sRed);
                if (tid == 0) g.wpart[static_cast<size_t>(c) * nblk + blk] = v;
                __syncthreads();
            }
        }
    }
    eb = wave_or(eb);
    if ((tid & 63) == 0 && eb) atomicOr(g.err, eb);
}

// Wavefronts per SIMD.  The energy kernel of a model whose LDS lets three
// workgroups share a compute unit is held to three (K = 10, P3 = 8 FP64: 526 ->
// 451 us, K = 12, P3 = 10 FP32: 473 -> 406 us); with K = 12, P3 = 10 in FP64 only
// two fit, and the same kernel took 793 us against 753 when it was held to three.
constexpr int wide_waves(int mode) { return mode == 0 ? 4 : 2; }

template <typename T, int MODE>
__global__ __launch_bounds__(WT) __attribute__((amdgpu_waves_per_eu(wide_waves(MODE)))) void wide_kernel(WideArgs<T> g) {
    wide_body<T, MODE, false, false>(g);
}

template <typename T>
__global__ __launch_bounds__(WT) __attribute__((amdgpu_waves_per_eu(3))) void wide_kernel_occ3(WideArgs<T> g) {
    wide_body<T, 1, true, false>(g);
}

// With 4-body terms: an instance of its own, whose adjoint needs registers that
// the others are faster without (K = 12, P3 = 10 FP32: 518 against 399 us); in
// FP32 at three wavefronts per SIMD (K = 12, P4 = 6: 2,506 -> 1,489 us).
template <typename T>
__global__ __launch_bounds__(WT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 2))) void wide_kernel_four(WideArgs<T> g) {
    wide_body<T, 1, sizeof(T) == 4, true>(g);
}

template <typename T, int MODE>
hipError_t launch_mode(const WideArgs<T>& a, bool fast, int nblk, hipStream_t st) {
    const int nrec = (a.N + WT / 16 - 1) / (WT / 16);
    constexpr bool DERIV = MODE == 1;
    if (a.N > 0) {
        if (fast) hipLaunchKernelGGL((wide_pair_kernel<T, DERIV, true>), dim3(nrec), dim3(WT), 0, st, a);
        else hipLaunchKernelGGL((wide_pair_kernel<T, DERIV, false>), dim3(nrec), dim3(WT), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const size_t lds = wide_lds(a.prm.K, a.prm.PA, a.prm.M, a.prm.K4 > 0, static_cast<int>(sizeof(T)), MODE == 1).total;
    constexpr size_t STATIC = WIDE_PARTS * sizeof(int) + 9 * CH * sizeof(double);
    if (MODE == 1 && a.prm.K4 > 0)
        hipLaunchKernelGGL((wide_kernel_four<T>), dim3(nblk), dim3(WT), lds, st, a);
    else if (MODE == 1 && lds + STATIC <= 163840 / 3)
        hipLaunchKernelGGL((wide_kernel_occ3<T>), dim3(nblk), dim3(WT), lds, st, a);
    else
        hipLaunchKernelGGL((wide_kernel<T, MODE>), dim3(nblk), dim3(WT), lds, st, a);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_wide(const WideArgs<T>& a, int mode, bool fast, int nblk, hipStream_t st) {
    if (nblk <= 0) return hipSuccess;
    return mode == 0 ? launch_mode<T, 0>(a, fast, nblk, st) : launch_mode<T, 1>(a, fast, nblk, st);
}

template hipError_t launch_wide<double>(const WideArgs<double>&, int, bool, int, hipStream_t);
template hipError_t launch_wide<float>(const WideArgs<float>&, int, bool, int, hipStream_t);

}  // namespace pod
