// Batched descriptor-matrix assembly for fitting (Sec. IV.A, eqs. (58a),
// (63a)): for many small periodic cells, the per-atom descriptors D, the
// global descriptors G = sum_i D_i of each cell and their derivatives
// dG/dr_n (Sec. II.G, eqs. (26c), (24c), product rule for the 2- and 4-body
// terms), in FP64.  Three kernels over the cells in order of decreasing pair
// count (batches beyond 2 GB of scratch, or what the device has, in several
// rounds of them):
//   1. pair records: (rhat, 1/r) per pair and, per radial index, (R_m, R'_m),
//      in slot-major order (see BArgs);
//   2. forward: lanes (atom, m) accumulate the atomic-basis rows (eq. (24b)),
//      contract them (eqs. (25)-(30a)), write D, sum G in LDS, keep B and the
//      degree sums D3_0 .. D3_PA;
//   3. dG/dR: one workgroup per (cell, radial index m, chunk of at most `cw`
//      of its descriptor columns), with the cell's dG/dR block [N_c][3][cw] in
//      LDS.  Work items are (atom i, row): the lane forms the Jacobian row
//      dD/dB_{i m .} in registers, walks the pairs of atom i, evaluates the
//      row's polynomial h(rhat) and its gradient by nested Horner recurrences
//      and v = dD_i/dr_ij by eq. (24c), adds +v to the LDS row of the
//      neighbour (atomic) and keeps -v for atom i in registers, added once at
//      the end.  The block is then written out.
// The records and basis rows cross HBM between the kernels (1.4 GB for 250,505
// atoms); in one persistent kernel, as before, every cell's phases ran at the
// two wavefronts per SIMD of the forward phase, and a batch of few cells left
// most of the chip idle.
//
// Rows.  The columns of a radial index need fewer polynomials than there are
// columns, and most of them have few terms:
//   * e_0 (D2 = B_0) also gives D3_0 = B_0^2 and D4_(0,0,0) = B_0^3, scaled by
//     2 B_0 and 3 B_0^2;
//   * the degree-n sphere row (D3_n, n >= 1) also gives D4_(n,0,0) = B_0 D3_n
//     as B_0 v + D3_n v_0 with v_0 = R' rhat the derivative of e_0;
//   * the 4-body functions (a, b, c), b >= 1, have terms of the degrees a + b,
//     a + c and b + c only (eq. (30a)).
// Rows are classed by their highest degree D (the degrees up to 2 together),
// a wavefront takes 64 items of one class, and the class fixes the length of
// the polynomial at compile time: at P3 = P4 = 4, 11 rows for 17 columns, 5 of
// them with 10 coefficients, 3 with 20 and 3 with 35.  Wavefronts draw tasks
// of 64 items from a counter, highest degree first.
//
// 2,000 cells of 2 to 250 atoms (250,505 atoms, 6.6 M pairs, 17 columns per
// radial index): 6.85 -> 3.78 ms of kernels (records 0.30, basis 0.62, dG/dR
// 2.8), 200 cells 1.69 -> 0.42 ms, against one pass over all 35 monomials for every
// column in a persistent kernel.  dG/dR is held by the record loads and the
// LDS atomics together (without either 2.0, without the polynomials 2.3 ms).
// The same product on the FP64 matrix cores (15 Jacobian rows as one tile of
// v_mfma_f64_16x16x4_f64 against tiles of 16 pairs) took 8.9 ms in all: those
// instructions run at the vector FP64 rate, do not overlap with vector FP64,
// and multiply the zeros.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "pod.h"
#include "pod_device.h"
#include "pod_internal.h"
#include "pod_plan.h"
#include "pod_tables.h"

namespace pod {
namespace {

using namespace dev;

struct BArgs {
    ParamsT<double> prm;  // by value: read with scalar loads
    int n_cell;           // cells of this launch
    int c_end;            // one past the last of them
    long ent_max;         // record entries of the largest
    const int* order;     // their processing order (decreasing pair count)
    const int* cfg_off;   // n_cfg + 1 atom offsets
    const double* pos;
    const double* cells;  // n_cfg x 9, lattice vectors as rows
    const int* offsets;
    const int* nbr_j;
    const int* shift;
    double* D;
    double* G;
    double* dGdR;
    // scratch of this launch's cells, whose atoms start at a_base: pair records
    // in slot-major order, entry ebase[c] + slot N_c + atom for the pair at
    // place `slot` of an atom's list: recU [entry][ux, uy, uz, 1/r], recR
    // [m][entry][R_m, R'_m] (n_ent of them), recJ [entry] the neighbour's index
    // within the cell (-1: not in it); basis rows Bs
    // [m][mu][atom] with the degree sums D3_n behind the NA monomials
    const long* ebase;
    double* recU;
    double* recR;
    int* recJ;
    double* Bs;
    int a_base;
    long n_ent, n_at;
    int cw, nch, nc_max;  // columns per chunk, chunks per radial index, atoms of the LDS accumulator
    int* err;
};

// Rows of a radial index: kind << 8 | index with kind ROW_E0 (e_0), ROW_S
// (sphere row of degree `index`), ROW_P (4-body function `index`).
constexpr int ROW_E0 = 0, ROW_S = 1, ROW_P = 2;
constexpr int MAX_ROWS = 32;

// Classes: class 0 holds the rows up to degree min(PA, 2), class q the rows of
// degree 2 + q.
constexpr int class_degree(int PA, int q) { return PA < 2 ? PA : 2 + q; }
constexpr int n_classes(int PA) { return PA <= 2 ? 1 : PA - 1; }

template <int PA>
struct RowTable {
    int n;
    int row[MAX_ROWS], cls[MAX_ROWS];
    constexpr RowTable() : n(0), row{}, cls{} {
        constexpr D4Build<PA> d4{};
        row[n++] = ROW_E0 << 8;
        for (int d = 1; d <= PA; ++d) {
            row[n] = (ROW_S << 8) | d;
            cls[n++] = d <= 2 ? 0 : d - 2;
            for (int p = 0; p < d4.KA; ++p)
                if (d4.pb[p] > 0 && d4.pa[p] + d4.pb[p] == d) {
                    row[n] = (ROW_P << 8) | p;
                    cls[n++] = d <= 2 ? 0 : d - 2;
                }
        }
    }
};

// The rows in use for the current radial index and chunk, per class.  An
// entry packs the row (10 bits) and its local columns (6 bits each, COL_NONE
// when not in the chunk): the row's own (D2, D3_n or D4_p), then D3_0 of e_0
// or D4_(n,0,0) of a sphere row, then D4_(0,0,0) of e_0.  The list takes the
// place of Q in LDS, which only the pair records need.
constexpr int COL_NONE = 63;
constexpr int CLASS_ROWS = 16;
struct RowList {
    int task, nc;                // next task; columns of the chunk
    int col[COL_NONE];           // global column of every local one
    int n[n_classes(FAST_MAX_PA)];
    int ent[n_classes(FAST_MAX_PA)][CLASS_ROWS];
};
static_assert(sizeof(RowList) <= POD_MAX_L * POD_MAX_K * sizeof(double), "row list in the place of Q");
static_assert(1 + FAST_MAX_PA + 1 + n_partitions(POD_MAX_P4) < COL_NONE, "packed columns");

// Row J_mu = dD/dB_{i m mu} (degree at most D) of one row, from the atomic-
// basis row b = B_{i m .}.  All indices are compile-time, so J stays in
// registers.
template <int PA, int D, bool LOW>
__device__ __forceinline__ void jacobian_row(int row, const double* __restrict__ brow, long bs, double (&J)[n_mono(D)]) {
    constexpr MonoTable<PA> mt{};
    constexpr int NA = n_mono(D);
    using Tab = D4Table<PA>;
    const int kind = row >> 8, idx = row & 255;
    double b[NA];
#pragma unroll
    for (int mu = 0; mu < NA; ++mu) b[mu] = brow[mu * bs];
#pragma unroll
    for (int mu = 0; mu < NA; ++mu) J[mu] = 0.0;
    if (LOW && kind == ROW_E0) {              // eq. (25): D2 = B_m0
        J[0] = 1.0;
    } else if (kind == ROW_S) {               // eq. (26c): D3_n = sum_{|mu|=n} c_mu B_mu^2
#pragma unroll
        for (int mu = LOW ? 1 : n_mono(D - 1); mu < NA; ++mu)
            if (!LOW || mt.deg[mu] == idx) J[mu] = 2.0 * mt.mult[mu] * b[mu];
    } else {                                  // eq. (30a): sum_t c_t B_x B_y B_z
#pragma unroll
        for (int p = 0; p < Tab::KA; ++p) {
            const int dp = Tab::build.pa[p] + Tab::build.pb[p];
            if (Tab::build.pb[p] > 0 && (LOW ? dp <= D : dp == D)) {
                if (idx == p) {
#pragma unroll
                    for (int t = Tab::build.tbeg[p]; t < Tab::build.tend[p]; ++t) {
                        const int x = Tab::build.tx[t], y = Tab::build.ty[t], z = Tab::build.tz[t];
                        const double cf = Tab::build.tc[t];
                        J[x] += cf * b[y] * b[z];
                        J[y] += cf * b[x] * b[z];
                        J[z] += cf * b[x] * b[y];
                    }
                }
            }
        }
    }
}

// 64 items (atom, row) of one class from the atoms [ab, ab + nb), the pairs part,
// part + parts, ... of each: adds dD/dr of the items' rows into sAcc[N_c][3][cw].
template <int PA, int D, bool LOW>
__device__ __forceinline__ void row_task(const int* __restrict__ recJ, const RowList* sL, int q, int first,
                                         int ab, int nb, const double* __restrict__ recU, const double* __restrict__ recR,
                                         const double* __restrict__ Bs, long bs, const int* sOff, double* sAcc,
                                         int m, int Nc, int cw, int part, int parts) {
    constexpr int NAF = n_mono(PA);
    constexpr int NB = NAF + PA + 1;
    constexpr int NA = n_mono(D);
    const int nrow = sL->n[q];
    const int it = first + static_cast<int>(threadIdx.x & 63);
    const int rr = it / nb, al = it - rr * nb;   // a full block's wavefront has one row
    if (rr >= nrow) return;
    const int a = ab + al;
    const int ent = sL->ent[q][rr];
    const int row = ent & 1023;
    const int c0 = (ent >> 10) & 63, c1 = (ent >> 16) & 63, c2 = LOW ? (ent >> 22) & 63 : COL_NONE;
    const bool e0 = LOW && (row >> 8) == ROW_E0;
    const double* brow = Bs + static_cast<long>(m) * NB * bs + a;
    // second column: f1 v + fe v_0, third: f2 v
    const double b0 = brow[0];
    const double f1 = e0 ? 2.0 * b0 : b0, f2 = 3.0 * b0 * b0;
    const double fe = (row >> 8) == ROW_S ? brow[(NAF + (row & 255)) * bs] : 0.0;
    double J[NA];
    jacobian_row<PA, D, LOW>(row, brow, bs, J);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;   // sums over the atom's pairs of v ...
    double e0s = 0.0, e1s = 0.0, e2s = 0.0;   // ... and of v_0
    const int cnt = sOff[a + 1] - sOff[a];
    // the next pair's record is requested before this pair's arithmetic
    const double2* U2 = reinterpret_cast<const double2*>(recU);
    const double2* R2 = reinterpret_cast<const double2*>(recR);
    double2 nA = {0.0, 0.0}, nB = {0.0, 0.0}, nR = {0.0, 0.0};
    int nj = -1;
    long e = a + static_cast<long>(part) * Nc;
    const long step = static_cast<long>(parts) * Nc;
    if (part < cnt) {
        nA = U2[2 * e]; nB = U2[2 * e + 1]; nR = R2[e];
        nj = recJ[e];
    }
    for (int s = part + parts; s < cnt + parts; s += parts) {
        const int jl = nj;
        const double ux = nA.x, uy = nA.y, uz = nB.x, Rr = nR.x * nB.y, dR = nR.y;
        e += step;
        if (s < cnt) {
            nA = U2[2 * e]; nB = U2[2 * e + 1]; nR = R2[e];
            nj = recJ[e];
        }
        // eq. (24c): v = R' h rhat + (R / r) (grad_u h - (rhat . grad_u h) rhat)
        double h, hx, hy, hz;
        poly_gradient<double, D>(J, ux, uy, uz, h, hx, hy, hz);
        const double w = dR * h - Rr * (ux * hx + uy * hy + uz * hz);
        const double v0 = w * ux + Rr * hx, v1 = w * uy + Rr * hy, v2 = w * uz + Rr * hz;
        const double d0 = dR * ux, d1 = dR * uy, d2 = dR * uz;   // v_0
        if (jl >= 0) {
            double* acc = sAcc + static_cast<size_t>(jl) * 3 * cw;
            if (c0 != COL_NONE) {
                atomicAdd(&acc[c0], v0);
                atomicAdd(&acc[cw + c0], v1);
                atomicAdd(&acc[2 * cw + c0], v2);
            }
            if (c1 != COL_NONE) {
                atomicAdd(&acc[c1], f1 * v0 + fe * d0);
                atomicAdd(&acc[cw + c1], f1 * v1 + fe * d1);
                atomicAdd(&acc[2 * cw + c1], f1 * v2 + fe * d2);
            }
            if (LOW && c2 != COL_NONE) {
                atomicAdd(&acc[c2], f2 * v0);
                atomicAdd(&acc[cw + c2], f2 * v1);
                atomicAdd(&acc[2 * cw + c2], f2 * v2);
            }
        }
        s0 += v0; s1 += v1; s2 += v2;
        e0s += d0; e1s += d1; e2s += d2;
    }
    double* acc = sAcc + static_cast<size_t>(a) * 3 * cw;
    if (c0 != COL_NONE) {
        atomicAdd(&acc[c0], -s0);
        atomicAdd(&acc[cw + c0], -s1);
        atomicAdd(&acc[2 * cw + c0], -s2);
    }
    if (c1 != COL_NONE) {
        atomicAdd(&acc[c1], -(f1 * s0 + fe * e0s));
        atomicAdd(&acc[cw + c1], -(f1 * s1 + fe * e1s));
        atomicAdd(&acc[2 * cw + c1], -(f1 * s2 + fe * e2s));
    }
    if (LOW && c2 != COL_NONE) {
        atomicAdd(&acc[c2], -f2 * s0);
        atomicAdd(&acc[cw + c2], -f2 * s1);
        atomicAdd(&acc[2 * cw + c2], -f2 * s2);
    }
}

// The class of a task, resolved to its compile-time degree: q counts down
// from the highest class.
template <int PA, int Q>
__device__ __forceinline__ void class_task(const int* recJ, const RowList* sL, int q, int first,
                                           int ab, int nb, const double* recU, const double* recR, const double* Bs, long bs,
                                           const int* sOff, double* sAcc, int m, int Nc, int cw, int part, int parts) {
    if constexpr (Q >= 0) {
        if (q == Q)
            row_task<PA, class_degree(PA, Q), Q == 0>(recJ, sL, q, first, ab, nb, recU, recR, Bs, bs, sOff, sAcc, m, Nc,
                                                           cw, part, parts);
        else
            class_task<PA, Q - 1>(recJ, sL, q, first, ab, nb, recU, recR, Bs, bs, sOff, sAcc, m, Nc, cw, part, parts);
    }
}

// ---- 1. pair records: workgroups (cell, part), one entry (slot, atom) per
// thread and turn, consecutive threads on consecutive entries of the cell ----
// Lanes on the atoms of a cell and its four wavefronts on the slots, as before,
// left most lanes idle and a serial chain of a quarter of the longest list: 64
// cells of 2 to 10 atoms 35 us, 200 cells up to 250 atoms (K = 2) 89 us.
// DERIV: with R'_m; without derivatives only R_m is read back.
constexpr int REC_THREADS = 256;
// Workgroups aimed at, one turn and a half of the chip: more of them read a cell's
// lists and positions into more caches (2,000 cells: one part each 303 us, four
// 351, sixteen 377; 314 before).
constexpr int REC_BLOCKS = 2048;

template <bool FAST, bool DERIV>
__global__ __launch_bounds__(REC_THREADS) void batch_record_kernel(BArgs g) {
    __shared__ double sQ[POD_MAX_L * POD_MAX_K];
    const ParamsT<double>* __restrict__ P = &g.prm;
    const int K = P->K;
    const unsigned tid = threadIdx.x;
    const int c = g.order[blockIdx.x];
    const int a0 = g.cfg_off[c], a1 = g.cfg_off[c + 1];
    const unsigned Nc = a1 - a0;
    const long eb0 = g.ebase[c];
    const long n_ent = (c + 1 < g.c_end ? g.ebase[c + 1] : g.n_ent) - eb0;
    const unsigned first = blockIdx.y * REC_THREADS, step = gridDim.y * REC_THREADS;
    if (first >= n_ent) return;   // empty cells too
    if (FAST) {
        for (unsigned i = tid; i < POD_MAX_L * POD_MAX_K; i += REC_THREADS) sQ[i] = (&P->Q[0][0])[i];
        __syncthreads();
    }
    const double* cell = g.cells + 9 * static_cast<size_t>(c);
    const double rin = P->rin, rcut = P->rcut;
    int eb = 0;
    const unsigned ds = step / Nc, da = step - ds * Nc;
    unsigned s = (first + tid) / Nc, al = first + tid - s * Nc;
    for (long q = eb0 + first + tid; q < eb0 + n_ent; q += step) {
        const int i = a0 + static_cast<int>(al);
        const int p = g.offsets[i] + static_cast<int>(s);
        if (p < g.offsets[i + 1]) {   // lists shorter than the cell's longest leave entries unused
            const double xi = g.pos[3 * i + 0], yi = g.pos[3 * i + 1], zi = g.pos[3 * i + 2];
            const int j = g.nbr_j[p];
            const int sh = g.shift[p];
            double d0 = 0, d1 = 0, d2 = 0, r = 0.5 * (rin + rcut);
            bool ok = false;
            if (j < a0 || j >= a1) {
                eb |= ERR_NEIGH;
            } else {
                const double sx = unpack_shift(sh, 0), sy = unpack_shift(sh, 1), sz = unpack_shift(sh, 2);
                d0 = g.pos[3 * j + 0] - xi + sx * cell[0] + sy * cell[3] + sz * cell[6];
                d1 = g.pos[3 * j + 1] - yi + sx * cell[1] + sy * cell[4] + sz * cell[7];
                d2 = g.pos[3 * j + 2] - zi + sx * cell[2] + sy * cell[5] + sz * cell[8];
                const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
                if (!isfinite(r2)) {
                    eb |= ERR_NONFINITE;
                } else {
                    const double rr = sqrt(r2);
                    if (rr <= rin) eb |= ERR_RANGE;
                    else if (rr < rcut) { r = rr; ok = true; }   // beyond rcut: not a neighbour
                }
            }
            const double ri = 1.0 / r;
            double R[FAST_MAX_K], dR[FAST_MAX_K];
            if constexpr (FAST) radial_std<double, DERIV>(P, sQ, r, ri, R, dR);
            else radial<double, DERIV>(P, r, ri, R, dR);
            g.recJ[q] = j >= a0 && j < a1 ? j - a0 : -1;
            double2* U2 = reinterpret_cast<double2*>(g.recU) + 2 * q;
            U2[0] = ok ? double2{d0 * ri, d1 * ri} : double2{0.0, 0.0};
            U2[1] = double2{ok ? d2 * ri : 0.0, ri};
#pragma unroll
            for (int k = 0; k < FAST_MAX_K; ++k)
                if (k < K)
                    reinterpret_cast<double2*>(g.recR)[k * g.n_ent + q] =
                        ok ? double2{R[k], DERIV ? dR[k] : 0.0} : double2{0.0, 0.0};
        }
        s += ds;
        al += da;
        if (al >= Nc) { al -= Nc; ++s; }
    }
    eb = wave_or(eb);
    if ((tid & 63) == 0 && eb) atomicOr(g.err, eb);
}

// ---- 2. atomic basis, descriptors, G: one workgroup per cell, lanes (atom, m) ----
constexpr int BASIS_THREADS = 256;
template <int PA>
__global__ __launch_bounds__(BASIS_THREADS) void batch_basis_kernel(BArgs g) {
    constexpr MonoTable<PA> mt{};
    constexpr int NA = n_mono(PA);
    using Tab = D4Table<PA>;
    constexpr int KA = Tab::KA;
    constexpr int NB = NA + PA + 1;   // basis row with the degree sums D3_0 .. D3_PA

    const ParamsT<double>* __restrict__ P = &g.prm;
    const int K = P->K, M = P->M;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    constexpr int nwv = BASIS_THREADS / WAVE;
    const int apw = WAVE / K;
    const int al = lane / K, m = lane - al * K;
    const int ka_used = P->K4 > 0 ? P->Ka4 : 0;
    extern __shared__ __align__(16) unsigned char smem[];
    double* sG = reinterpret_cast<double*>(smem);
    for (int k = tid; k < M; k += BASIS_THREADS) sG[k] = 0.0;
    __syncthreads();
    const int c = g.order[blockIdx.x];
    const int a0 = g.cfg_off[c], a1 = g.cfg_off[c + 1];
    const int Nc = a1 - a0;
    const double2* U2 = reinterpret_cast<const double2*>(g.recU) + 2 * g.ebase[c];
    const double2* R2 = reinterpret_cast<const double2*>(g.recR) + m * g.n_ent + g.ebase[c];
    for (int base = wv * apw; base < Nc; base += nwv * apw) {
        const int a = base + al;
        const bool act = al < apw && a < Nc;
        double acc[NA];
#pragma unroll
        for (int mu = 0; mu < NA; ++mu) acc[mu] = 0.0;
        if (act) {
            // four pairs' records in flight; a slot past the end reads the last pair
            constexpr int GP = 4;
            const int cnt = g.offsets[a0 + a + 1] - g.offsets[a0 + a];
            for (int s0 = 0; s0 < cnt; s0 += GP) {
                double2 uA[GP], uB[GP];
                double Rm[GP];
#pragma unroll
                for (int s = 0; s < GP; ++s) {
                    const long e = static_cast<long>(min(s0 + s, cnt - 1)) * Nc + a;
                    uA[s] = U2[2 * e]; uB[s] = U2[2 * e + 1];
                    Rm[s] = R2[e].x;
                }
#pragma unroll
                for (int s = 0; s < GP; ++s)
                    if (s0 + s < cnt) accumulate_basis<double, PA>(acc, Rm[s], uA[s].x, uA[s].y, uB[s].x);
            }
        }
        double d3[PA + 1];
#pragma unroll
        for (int n = 0; n <= PA; ++n) d3[n] = 0.0;
#pragma unroll
        for (int mu = 0; mu < NA; ++mu) d3[mt.deg[mu]] += double(mt.mult[mu]) * acc[mu] * acc[mu];
        double d4[KA];
#pragma unroll
        for (int p = 0; p < KA; ++p) d4[p] = (Tab::build.pb[p] == 0) ? acc[0] * d3[Tab::build.pa[p]] : 0.0;
        // eq. (30a) for the triples the model uses
#pragma unroll
        for (int p = 0; p < KA; ++p)
            if (p < ka_used) {
#pragma unroll
                for (int t = Tab::build.tbeg[p]; t < Tab::build.tend[p]; ++t)
                    d4[p] += double(Tab::build.tc[t]) * acc[Tab::build.tx[t]] * acc[Tab::build.ty[t]] *
                             acc[Tab::build.tz[t]];
            }
        if (act) {
            if (g.dGdR) {
                double* brow = g.Bs + static_cast<long>(m) * NB * g.n_at + (a0 + a - g.a_base);
#pragma unroll
                for (int mu = 0; mu < NA; ++mu) brow[mu * g.n_at] = acc[mu];
#pragma unroll
                for (int n = 0; n <= PA; ++n) brow[(NA + n) * g.n_at] = d3[n];
            }
            double* Drow = g.D ? g.D + static_cast<size_t>(a0 + a) * M : nullptr;
            if (m == 0) { if (Drow) Drow[0] = 1.0; atomicAdd(&sG[0], 1.0); }
            if (m < P->K2) { if (Drow) Drow[1 + m] = acc[0]; atomicAdd(&sG[1 + m], acc[0]); }
            if (m < P->K3) {
#pragma unroll
                for (int n = 0; n <= PA; ++n)
                    if (n <= P->P3) {
                        const int col = P->off3 + m * (P->P3 + 1) + n;
                        if (Drow) Drow[col] = d3[n];
                        atomicAdd(&sG[col], d3[n]);
                    }
            }
            if (m < P->K4) {
#pragma unroll
                for (int p = 0; p < KA; ++p)
                    if (p < P->Ka4) {
                        const int col = P->off4 + m * P->Ka4 + p;
                        if (Drow) Drow[col] = d4[p];
                        atomicAdd(&sG[col], d4[p]);
                    }
            }
        }
    }
    __syncthreads();
    if (g.G)
        for (int k = tid; k < M; k += BASIS_THREADS) g.G[static_cast<size_t>(c) * M + k] = sG[k];
}

// ---- 3. dG/dR: one workgroup per item (cell, radial index, chunk) ----
// Threads per workgroup at most: three wavefronts per SIMD up to degree 4 (168
// registers), two above (256; degree 6 spills 380 bytes a lane, and 1,936 in the
// former kernel).  By default two or more workgroups of 256 share a compute unit where the LDS allows.
constexpr int deriv_threads(int PA) { return PA <= 4 ? 768 : 512; }

template <int PA>
__global__ __launch_bounds__(deriv_threads(PA)) void batch_deriv_kernel(BArgs g) {
    constexpr int NB = n_mono(PA) + PA + 1;
    constexpr int NCL = n_classes(PA);
    const ParamsT<double>* __restrict__ P = &g.prm;
    const int K = P->K, M = P->M;
    const int nth = blockDim.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int cw = g.cw;
    extern __shared__ __align__(16) unsigned char smem[];
    const BatchLds LY = batch_lds(M, cw, g.nc_max);
    RowList& sL = *reinterpret_cast<RowList*>(smem + LY.q);
    double* sAcc = reinterpret_cast<double*>(smem + LY.acc);
    int* sOff = reinterpret_cast<int*>(smem + LY.off);

    // items (cell, radial index, chunk) are numbered so that those of one cell
    // run on one XCD (workgroup i runs on XCD i mod 8) and share its records in
    // that L2
    const int per_cell = K * g.nch;
    const unsigned n_item = (g.n_cell + 7u) / 8 * 8 * per_cell;   // at most 2^20 cells x 8 x 31
    for (unsigned w = blockIdx.x; w < n_item; w += gridDim.x) {
        const int rank = (w >> 3) / per_cell * 8 + (w & 7), im = (w >> 3) % per_cell;
        const int m = im / g.nch, ch = im - m * g.nch;
        if (rank >= g.n_cell) continue;
        const int c = g.order[rank];
        const int a0 = g.cfg_off[c], a1 = g.cfg_off[c + 1];
        const int Nc = a1 - a0;
        if (Nc <= 0) continue;
        for (int i = tid; i <= Nc; i += nth) sOff[i] = g.offsets[a0 + i];
        const long eb0 = g.ebase[c];
        const double* recU = g.recU + 4 * eb0;
        const double* recR = g.recR + 2 * (m * g.n_ent + eb0);
        const int* recJ = g.recJ + eb0;
        const double* Bs = g.Bs + (a0 - g.a_base);
        for (int t = tid; t < Nc * 3 * cw; t += nth) sAcc[t] = 0.0;
        if (tid == 0) {
            // the chunk's rows: columns in the order of the row table, cw at a
            // time (a row whose columns fall into two chunks is in both)
            constexpr RowTable<PA> rt{};
            const int n3 = m < P->K3 ? P->P3 + 1 : 0, n4 = m < P->K4 ? P->Ka4 : 0;
            for (int q = 0; q < NCL; ++q) sL.n[q] = 0;
            sL.task = 0;
            int at = -ch * cw;   // place of the next column in the chunk
            for (int k = 0; k < rt.n; ++k) {
                const int kind = rt.row[k] >> 8, idx = rt.row[k] & 255, q = rt.cls[k];
                int col[3] = {-1, -1, -1};
                if (kind == ROW_E0) {
                    if (m < P->K2) col[0] = 1 + m;
                    if (n3) col[1] = P->off3 + m * n3;
                    if (n4) col[2] = P->off4 + m * n4;
                } else if (kind == ROW_S) {
                    if (idx < n3) col[0] = P->off3 + m * n3 + idx;
                    const int p = n_partitions(idx - 1);   // (idx, 0, 0): the first triple of its degree
                    if (p < n4) col[1] = P->off4 + m * n4 + p;
                } else if (idx < n4) {
                    col[0] = P->off4 + m * n4 + idx;
                }
                int ent = rt.row[k];
                bool any = false;
                for (int c3 = 0; c3 < 3; ++c3) {
                    int lc = COL_NONE;
                    if (col[c3] >= 0) {
                        if (at >= 0 && at < cw) {
                            lc = at;
                            sL.col[at] = col[c3];
                            any = true;
                        }
                        ++at;
                    }
                    ent |= lc << (10 + 6 * c3);
                }
                if (any) sL.ent[q][sL.n[q]++] = ent;
            }
            sL.nc = max(0, min(at, cw));
        }
        {
            __syncthreads();
            // blocks of 64 atoms, all classes of a block in turn: the block's
            // records are read again from L2.  A small cell with fewer tasks than
            // wavefronts splits every task's pairs into parts (otherwise one
            // wavefront walks the lists: 64 cells of 2 to 10 atoms, K = 1, degree
            // 1 62.7 -> 56.5 us per call).
            int tpb = 0, tail = 0;
            const int nfull = Nc / WAVE;
            for (int q = 0; q < NCL; ++q) {
                tpb += sL.n[q];
                tail += ((Nc - nfull * WAVE) * sL.n[q] + WAVE - 1) / WAVE;
            }
            const int ntask = nfull * tpb + tail;
            const int parts = ntask > 0 ? max(nth / WAVE / ntask, 1) : 1;
            for (;;) {
                int t = 0;
                if (lane == 0) t = atomicAdd(&sL.task, 1);
                t = __builtin_amdgcn_readfirstlane(t);
                if (t >= ntask * parts) break;
                const int part = parts > 1 ? t / ntask : 0;
                t -= part * ntask;
                const int blk = tpb > 0 ? min(t / tpb, nfull) : nfull;
                const int nb = min(WAVE, Nc - blk * WAVE);
                t -= blk * tpb;
                int q = NCL - 1;
                for (; q > 0; --q) {
                    const int nt = (nb * sL.n[q] + WAVE - 1) / WAVE;
                    if (t < nt) break;
                    t -= nt;
                }
                class_task<PA, NCL - 1>(recJ, &sL, q, WAVE * t, blk * WAVE, nb, recU, recR, Bs,
                                        g.n_at, sOff, sAcc, m, Nc, cw, part, parts);
            }
            __syncthreads();
            // write the chunk out, row r = (atom, d); t / nc by the rounded-up
            // reciprocal (exact for t nc < 2^32)
            const int nc = sL.nc;
            const unsigned inv = nc > 0 ? 0xFFFFFFFFu / static_cast<unsigned>(nc) + 1u : 0u;
            for (int t = tid; t < Nc * 3 * nc; t += nth) {
                const int r = nc == 1 ? t : static_cast<int>(__umulhi(static_cast<unsigned>(t), inv));
                const int cl = t - r * nc;
                g.dGdR[(static_cast<size_t>(a0) * 3 + r) * M + sL.col[cl]] = sAcc[r * cw + cl];
            }
        }
        if (m == 0 && ch == 0)
            for (int t = tid; t < Nc * 3; t += nth) g.dGdR[(static_cast<size_t>(a0) * 3 + t) * M] = 0.0;
        __syncthreads();   // LDS is rewritten by the next item
    }
}

template <int PA>
hipError_t launch_batch(const BArgs& a, bool fast, int ncell, int nth, size_t lds, hipStream_t st) {
    const auto records = [&](auto kernel) {
        const long parts = std::min((a.ent_max + REC_THREADS - 1) / REC_THREADS, static_cast<long>(REC_BLOCKS / a.n_cell));
        hipLaunchKernelGGL(kernel, dim3(a.n_cell, static_cast<unsigned>(std::max(parts, 1L))), dim3(REC_THREADS), 0, st, a);
    };
    if (fast) records(a.dGdR ? batch_record_kernel<true, true> : batch_record_kernel<true, false>);
    else records(a.dGdR ? batch_record_kernel<false, true> : batch_record_kernel<false, false>);
    hipLaunchKernelGGL((batch_basis_kernel<PA>), dim3(a.n_cell), dim3(BASIS_THREADS),
                       static_cast<size_t>(a.prm.M) * sizeof(double), st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.dGdR) return e;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&batch_deriv_kernel<PA>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return hipErrorInvalidValue;
    // one workgroup per item, as far as a launch's 2^32 threads reach: the
    // kernel's loop takes the rest
    // (ncell: cells worked on at a time)
    const long per_cell = static_cast<long>(a.prm.K) * a.nch;
    const long all = ((ncell > 0 ? std::min(ncell, a.n_cell) : a.n_cell) + 7L) / 8 * 8 * per_cell;
    const int nitem = static_cast<int>(std::min(all, 1L << 22));
    if (nth <= 0) nth = deriv_threads(PA);
    if (nth > deriv_threads(PA)) nth = deriv_threads(PA);
    hipLaunchKernelGGL((batch_deriv_kernel<PA>), dim3(nitem), dim3(nth), lds, st, a);
    return hipGetLastError();
}

hipError_t dispatch_batch(int PA, const BArgs& a, bool fast, int ncell, int nth, size_t lds, hipStream_t st) {
    switch (PA) {
        case 0: return launch_batch<0>(a, fast, ncell, nth, lds, st);
        case 1: return launch_batch<1>(a, fast, ncell, nth, lds, st);
        case 2: return launch_batch<2>(a, fast, ncell, nth, lds, st);
        case 3: return launch_batch<3>(a, fast, ncell, nth, lds, st);
        case 4: return launch_batch<4>(a, fast, ncell, nth, lds, st);
        case 5: return launch_batch<5>(a, fast, ncell, nth, lds, st);
        case 6: return launch_batch<6>(a, fast, ncell, nth, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
}  // namespace pod

extern "C" {

int pod_batch_assemble(pod_handle* h, int n_cfg, int N, int P, const int* cfg_atom_off, const void* pos,
                       const double* cells, const int* offsets, const int* nbr_j, const int* shift, double* D,
                       double* G, double* dGdR, const pod_tune* tune) {
    using namespace pod;
    if (!h || n_cfg < 0 || N < 0 || P < 0) return POD_EINVAL;
    if (h->dtype != POD_F64 || h->PA > FAST_MAX_PA || h->K > FAST_MAX_K) return POD_ENOTSUP;
    if (n_cfg == 0 || N == 0) return POD_OK;
    if (!cfg_atom_off || !pos || !cells || !offsets || (P > 0 && (!nbr_j || !shift))) return POD_EINVAL;
    // plan on the host: cell sizes and pair counts
    std::vector<int> coff(n_cfg + 1), off(N + 1);
    if (hipMemcpyAsync(coff.data(), cfg_atom_off, sizeof(int) * (n_cfg + 1), hipMemcpyDeviceToHost, h->stream) !=
            hipSuccess ||
        hipMemcpyAsync(off.data(), offsets, sizeof(int) * (N + 1), hipMemcpyDeviceToHost, h->stream) != hipSuccess ||
        hipStreamSynchronize(h->stream) != hipSuccess)
        return POD_EHIP;
    BatchPlan plan;
    int rc = plan_batch(n_cfg, N, P, coff.data(), off.data(), h->M, h->lds_max, tune, &plan);
    if (rc != POD_OK) return rc;
    // The records and basis rows of a round's cells live in the handle's
    // scratch; batches that need more than SCRATCH_CAP run in several rounds of
    // consecutive cells, and where the device does not have that much, in
    // rounds of half the size, and so on down to one cell a round.
    constexpr size_t SCRATCH_CAP = size_t(2) << 30;
    const int NB = n_mono(h->PA) + h->PA + 1;
    const size_t per_ent = (4 + 2 * static_cast<size_t>(h->K)) * sizeof(double) + sizeof(int);
    const size_t per_atom = static_cast<size_t>(h->K) * NB * sizeof(double);
    const size_t order_bytes = ((sizeof(int) * n_cfg + 255) / 256) * 256;
    const size_t base_bytes = ((sizeof(long) * n_cfg + 255) / 256) * 256;
    BatchRounds rounds;
    rc = fit_rounds(
        n_cfg, coff.data(), plan.longest.data(), per_ent, per_atom, SCRATCH_CAP,
        [&](size_t bytes) {
            const int r = ensure_scratch(h, order_bytes + base_bytes + bytes + 256);
            if (r == POD_ENOMEM) (void)hipGetLastError();   // answered here, not by the next launch
            return r;
        },
        &rounds);
    if (rc != POD_OK) return rc;
    const std::vector<int>& first = rounds.first;
    // processing order (decreasing pair count) of each round's cells
    std::vector<int> order(n_cfg);
    if (first.size() == 2) {
        order = plan.order;
    } else {
        std::vector<int> at(first.begin(), first.end() - 1);
        for (int c : plan.order)
            order[at[std::upper_bound(first.begin(), first.end(), c) - first.begin() - 1]++] = c;
    }
    // both tables in one copy (a second one costs about 8 us)
    std::vector<char> tables(order_bytes + base_bytes);
    std::memcpy(tables.data(), order.data(), sizeof(int) * n_cfg);
    std::memcpy(tables.data() + order_bytes, rounds.ebase.data(), sizeof(long) * n_cfg);
    int* d_order = static_cast<int*>(h->d_scratch);
    long* d_ebase = reinterpret_cast<long*>(static_cast<char*>(h->d_scratch) + order_bytes);
    if (hipMemcpyAsync(h->d_scratch, tables.data(), tables.size(), hipMemcpyHostToDevice, h->stream) != hipSuccess)
        return POD_EHIP;
    BArgs a;
    a.prm = h->hp_d;
    a.cfg_off = cfg_atom_off;
    a.pos = static_cast<const double*>(pos); a.cells = cells;
    a.offsets = offsets; a.nbr_j = nbr_j; a.shift = shift;
    a.D = D; a.G = G; a.dGdR = dGdR;
    a.ebase = d_ebase;
    // Columns per chunk: without a tuning value, the widest chunk that lets
    // two workgroups of 256 threads share a compute unit's LDS (one large
    // workgroup leaves the unit idle at the barriers around the write-out), as
    // long as that is at least four columns; the chunks of a radial index are
    // then made equally wide.  Measured at P3 = P4 = 4, cells up to 250 atoms:
    // 2,000 cells 3.49 ms (two chunks of 9) against 3.47 (one of 17, 512
    // threads), 200 cells 0.426 / 0.433 ms, 1,000 cells without 4-body terms
    // 0.948 / 1.178 ms; 2,000 cells up to 100 atoms, one chunk either way: 1.32
    // ms with 256 threads, 1.71 with 512.
    const int ncol = (h->K2 > 0 ? 1 : 0) + (h->K3 > 0 ? h->P3 + 1 : 0) + (h->K4 > 0 ? h->Ka4 : 0);
    int cw = plan.cw, nth = tune ? tune->threads : 0;
    if (!(tune && tune->cw > 0)) {
        int c2 = ncol;
        while (c2 > 0 && batch_lds(h->M, c2, plan.nc_max).total > h->lds_max / 2) --c2;
        if (c2 >= 4) cw = c2;
    }
    a.nch = (ncol + cw - 1) / cw;
    a.cw = (ncol + a.nch - 1) / a.nch;
    a.nc_max = plan.nc_max;
    const size_t lds = batch_lds(h->M, a.cw, a.nc_max).total;
    if (nth <= 0 && lds <= h->lds_max / 2) nth = 256;
    a.err = h->d_err;
    timing_begin(h, 1);
    hipError_t e = hipSuccess;
    for (size_t k = 0; k + 1 < first.size() && e == hipSuccess; ++k) {
        const int c0 = first[k], c1 = first[k + 1];
        a.n_cell = c1 - c0;
        a.c_end = c1;
        a.ent_max = rounds.ent_max[k];
        a.order = d_order + c0;
        a.a_base = coff[c0];
        a.n_ent = rounds.n_ent[k];
        a.n_at = coff[c1] - coff[c0];
        a.recU = reinterpret_cast<double*>(static_cast<char*>(h->d_scratch) + order_bytes + base_bytes);
        a.recR = a.recU + 4 * a.n_ent;
        a.Bs = a.recR + 2 * h->K * a.n_ent;
        a.recJ = reinterpret_cast<int*>(a.Bs + static_cast<size_t>(coff[c1] - coff[c0]) * h->K * NB);
        e = dispatch_batch(h->PA, a, h->std_ok != 0, tune ? tune->nblocks : 0, nth, lds, h->stream);
    }
    timing_end(h, 1);
    return e == hipSuccess ? POD_OK : POD_EHIP;
}

}  // extern "C"
