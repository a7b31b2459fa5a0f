// Energy path and descriptors for few atoms (Sec. II.E, II.G): one workgroup
// per atom, every phase spread over its threads.
//
// The per-atom kernel gives an atom K lanes, which walk its neighbours in
// rounds of K and evaluate the contractions serially in registers: the best
// use of a full chip, but a chain of about 20 us (FP64) when there are only a
// few wavefronts, followed by the pair kernel's 8 us.  Here an atom's pairs are
// evaluated at once, one per thread, and the sums run over threads:
//   1. thread p: geometry, R_k and R'_k, monomials A_mu(rhat) of pair p -> LDS;
//   2. thread (k, mu): B_{k mu} = sum_p R_k(p) A_mu(p) (eq. (24b));
//   3. thread (k, n): degree sums D3_kn (eq. (26a)); then four threads per (k, p)
//      share the merged terms of eq. (30a); energy, G and D rows;
//   4. thread (k, mu): adjoint dE_i/dB_{k mu} (product rule; the 4-body part
//      gathered from a table of the monomial's occurrences);
//   5. thread (p, k): value and gradient of the adjoint row's polynomial (nested
//      Horner), combined with R'_k and R_k; thread p adds the K parts in order
//      (eq. (24c)) and stores the pair's gradient.
// Fixed orders throughout: results are reproducible.  Lists longer than the
// staged chunk are taken chunk by chunk (the gradient pass stages them again).
// Bound by the latency of that chain (17 us for 16 atoms with all outputs; the
// two kernels it replaces took 31).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pod.h"
#include "pod_device.h"
#include "pod_internal.h"
#include "pod_small.h"
#include "pod_tables.h"

namespace pod {
namespace {

using namespace dev;

constexpr int small_chunk(int PA) { return PA <= 4 ? 64 : 32; }   // pairs staged at a time

// Packed tables of degree PA: monomial codes (degree | multinomial << 8),
// merged terms of eq. (30a) x | y << 7 | z << 14 | coefficient << 21 with the
// range of every 4-body index p, and per monomial its occurrences p | u << 5 |
// v << 12 | coefficient << 19 (in term order, hence sorted by p).
template <int PA>
struct SmallTab {
    static constexpr int NA = n_mono(PA), KA = n_partitions(PA), NT = D4Table<PA>::NT;
    static constexpr int CODE = 0, TBEG = NA, PABC = TBEG + KA + 1, TERM = PABC + KA, OBEG = TERM + NT,
                         OCC = OBEG + NA + 1, N = OCC + 3 * NT;
    int v[N];
    constexpr SmallTab() : v{} {
        constexpr MonoTable<PA> mt{};
        constexpr D4Build<PA> d4{};
        for (int n = 0; n < NA; ++n) v[CODE + n] = mt.deg[n] | (mt.mult[n] << 8);
        for (int p = 0; p < KA; ++p) {
            v[TBEG + p] = d4.tbeg[p];
            v[PABC + p] = d4.pa[p] | (d4.pb[p] << 4);
        }
        v[TBEG + KA] = NT;
        int cnt[NA + 1] = {};
        for (int t = 0; t < NT; ++t) {
            v[TERM + t] = d4.tx[t] | (d4.ty[t] << 7) | (d4.tz[t] << 14) | (d4.tc[t] << 21);
            ++cnt[d4.tx[t]];
            ++cnt[d4.ty[t]];
            ++cnt[d4.tz[t]];
        }
        v[OBEG] = 0;
        for (int n = 0; n < NA; ++n) v[OBEG + n + 1] = v[OBEG + n] + cnt[n];
        int at[NA + 1] = {};
        for (int n = 0; n < NA; ++n) at[n] = v[OBEG + n];
        for (int t = 0; t < NT; ++t) {
            const int x = d4.tx[t], y = d4.ty[t], z = d4.tz[t];
            const int own[3] = {x, y, z}, u[3] = {y, x, x}, w[3] = {z, z, y};
            for (int r = 0; r < 3; ++r) v[OCC + at[own[r]]++] = d4.tp[t] | (u[r] << 5) | (w[r] << 12) | (d4.tc[t] << 19);
        }
    }
};

template <int PA>
__device__ const SmallTab<PA> kSmall = SmallTab<PA>();

// 4-body index of (a, 0, 0): the number of triples of lower degree (1, 1, 2, 3,
// 4, 5 triples of degree 0 .. 5).
__device__ __forceinline__ int n_partitions_below(int a) {
    constexpr int below[7] = {n_partitions(-1), n_partitions(0), n_partitions(1), n_partitions(2),
                              n_partitions(3),  n_partitions(4), n_partitions(5)};
    int v = below[0];
#pragma unroll
    for (int d = 1; d < 7; ++d)
        if (a == d) v = below[d];
    return v;
}

// LDS of one workgroup, in elements of T (then the table's ints).
struct SmallLds {
    int u, r, dr, a, b, ab, s, c, total;
};
__host__ __device__ constexpr int odd(int n) { return n | 1; }
__host__ __device__ constexpr SmallLds small_lds(int K, int PA, int M) {
    const int CH = small_chunk(PA), NA = n_mono(PA);
    SmallLds L{};
    L.u = 0;                                   // [p][5]: rhat, 1/r, r
    L.r = L.u + 5 * CH;                        // [p][odd(K)]
    L.dr = L.r + odd(K) * CH;
    L.a = L.dr + odd(K) * CH;                  // [p][odd(NA)]; later the gradient parts [k][p][4]
    const int mono = odd(NA) * CH, part = 4 * K * CH;
    L.b = L.a + (mono > part ? mono : part);   // [k][NA]
    L.ab = L.b + K * NA;
    L.s = L.ab + K * NA;                       // [k][PA + 1]
    L.c = L.s + K * (PA + 1);                  // coefficients
    L.total = L.c + M;
    return L;
}

template <typename T, int PA, int MODE, bool FAST, int ST>
__global__ __launch_bounds__(ST) void small_kernel(WideArgs<T> g) {
    constexpr int SW = ST / WAVE;
    constexpr int NA = n_mono(PA), KA = n_partitions(PA), PA1 = PA + 1, CH = small_chunk(PA);
    constexpr MonoTable<PA> mt{};
    using Tab = SmallTab<PA>;
    const ParamsT<T>* __restrict__ P = &g.prm;
    const int K = P->K, M = P->M, P3 = P->P3, Ka4 = P->Ka4;
    const int K2 = P->K2, K3 = P->K3, K4 = P->K4;
    const bool four = K4 > 0;
    const int tid = threadIdx.x, lane = tid % WAVE, wv = tid / WAVE;
    const int i = blockIdx.x;
    extern __shared__ __align__(16) unsigned char smem[];
    const SmallLds L = small_lds(K, PA, M);
    T* sm = reinterpret_cast<T*>(smem);
    T *sU = sm + L.u, *sR = sm + L.r, *sdR = sm + L.dr, *sA = sm + L.a, *sB = sm + L.b, *sAb = sm + L.ab, *sS = sm + L.s, *sC = sm + L.c;
    int* sTab = reinterpret_cast<int*>(smem + (L.total * sizeof(T) + 15) / 16 * 16);
    __shared__ double sRed[SW];
    const int KO = odd(K);
    constexpr int NO = NA | 1;

    for (int t = tid; t < (four ? Tab::N : NA); t += ST) sTab[t] = kSmall<PA>.v[t];
    if (MODE == 1)
        for (int t = tid; t < M; t += ST) sC[t] = g.coef[t];
    int eb = 0, beg = 0, n = 0;
    {
        const int o0 = g.offsets[i], o1 = g.offsets[i + 1];
        if (o0 < 0 || o1 < o0 || o1 > g.P) eb |= ERR_NEIGH;
        else { beg = o0; n = o1 - o0; }
    }
    const T pi[3] = {g.pos[3 * i], g.pos[3 * i + 1], g.pos[3 * i + 2]};

    // ---- 1. the pairs c0 .. c0 + nc - 1: geometry, radial functions, monomials
    T dv[3] = {T(0), T(0), T(0)};   // this thread's pair vector, for the virial
    auto stage = [&](int c0, int nc, bool mono, int& err) {
        if (tid < nc) {
            const SlotIdx si = slot_index(g, true, beg + c0 + tid);
            T pj[3], d[3], r;
            slot_pos<T>(g, si, pj);
            const bool ok = slot_geometry<T>(g, true, si, pj, pi, err, d, r);
            const T ri = T(1) / r;
            T R[FAST_MAX_K], dR[FAST_MAX_K];
            if constexpr (FAST) radial_std<T, MODE == 1>(P, &P->Q[0][0], r, ri, R, dR);
            else radial<T, MODE == 1>(P, r, ri, R, dR);
            const T u[3] = {d[0] * ri, d[1] * ri, d[2] * ri};   // zero for a pair that is not a neighbour
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                sU[5 * tid + x] = u[x];
                dv[x] = d[x];
            }
            sU[5 * tid + 3] = ri;
            sU[5 * tid + 4] = ok ? r : T(0);
#pragma unroll
            for (int k = 0; k < FAST_MAX_K; ++k)
                if (k < K) {
                    sR[tid * KO + k] = ok ? R[k] : T(0);
                    if (MODE == 1) sdR[tid * KO + k] = ok ? dR[k] : T(0);
                }
            if (mono) {
                T A[NA];
                A[0] = T(1);
                sA[tid * NO] = A[0];
#pragma unroll
                for (int mu = 1; mu < NA; ++mu) {
                    A[mu] = A[mt.par[mu]] * u[mt.axis[mu]];
                    sA[tid * NO + mu] = A[mu];
                }
            }
        }
    };

    // ---- 2. atomic basis
    constexpr int OPT = (FAST_MAX_K * NA + ST - 1) / ST;   // basis values per thread, at most
    int ok_[OPT], om_[OPT];
    T acc[OPT];
#pragma unroll
    for (int x = 0; x < OPT; ++x) {
        const int o = tid + x * ST;
        ok_[x] = o < K * NA ? o / NA : -1;
        om_[x] = o < K * NA ? o - ok_[x] * NA : 0;
        acc[x] = T(0);
    }
    for (int c0 = 0; c0 < n; c0 += CH) {
        const int nc = n - c0 < CH ? n - c0 : CH;
        if (c0 > 0) __syncthreads();
        stage(c0, nc, true, eb);
        __syncthreads();
#pragma unroll
        for (int x = 0; x < OPT; ++x)
            if (ok_[x] >= 0) {
                const T *a = sA + om_[x], *r = sR + ok_[x];
                T v = acc[x];
#pragma unroll 4
                for (int p = 0; p < nc; ++p) v += r[p * KO] * a[p * NO];
                acc[x] = v;
            }
    }
#pragma unroll
    for (int x = 0; x < OPT; ++x)
        if (ok_[x] >= 0) sB[tid + x * ST] = acc[x];
    __syncthreads();

    // ---- 3. degree sums, 4-body sums, energy
    for (int w = tid; w < K * PA1; w += ST) {
        const int k = w / PA1, a = w - k * PA1;
        const int m0 = n_mono(a - 1), m1 = n_mono(a);
        T s = T(0);
#pragma unroll 4
        for (int mu = m0; mu < m1; ++mu) {
            const T v = sB[k * NA + mu];
            s += T(sTab[mu] >> 8) * v * v;
        }
        sS[w] = s;
    }
    __syncthreads();
    double ep = 0.0;
    auto column = [&](int col, T v) {
        if constexpr (MODE == 0) {
            g.D[static_cast<size_t>(i) * M + col] = v;
        } else {
            ep += static_cast<double>(sC[col]) * static_cast<double>(v);
            if (g.want_G) g.part[static_cast<size_t>(10 + col) * g.N + i] = static_cast<double>(v);
        }
    };
    const int off3 = P->off3, off4 = P->off4;
    if (tid == 0) column(0, T(1));
    if (tid < K2) column(1 + tid, sB[tid * NA]);
    for (int w = tid; w < K3 * (P3 + 1); w += ST) {
        const int k = w / (P3 + 1);
        column(off3 + w, sS[k * PA1 + w - k * (P3 + 1)]);
    }
    if (four) {
        // four lanes per (k, p) share the terms; the loop bound is the same for
        // all lanes of a wavefront, so the shuffles see every lane
        const int nd = K4 * Ka4;
        for (int w0 = 0; w0 < nd; w0 += ST / 4) {
            const int w = w0 + tid / 4, part = tid & 3;
            const bool in = w < nd;
            const int k = in ? w / Ka4 : 0, p = in ? w - k * Ka4 : 0;
            const T* Bk = sB + k * NA;
            const int pabc = sTab[Tab::PABC + p];
            T v = T(0);
            if ((pabc >> 4) == 0) {
                if (part == 0) v = Bk[0] * sS[k * PA1 + (pabc & 15)];                        // eq. (27a)
            } else {
                const int t1 = sTab[Tab::TBEG + p + 1];
#pragma unroll 2
                for (int t = sTab[Tab::TBEG + p] + part; t < t1; t += 4) {                     // eq. (30a)
                    const int te = sTab[Tab::TERM + t];
                    v += T(te >> 21) * Bk[te & 127] * Bk[(te >> 7) & 127] * Bk[(te >> 14) & 127];
                }
            }
            v += __shfl_xor(v, 1);
            v += __shfl_xor(v, 2);
            if (in && part == 0) column(off4 + w, v);
        }
    }
    {
        const int ew = wave_or(eb);
        if (lane == 0 && ew) atomicOr(g.err, ew);
    }
    if constexpr (MODE == 0) return;
    ep = wave_sum(ep);
    if (lane == 0) sRed[wv] = ep;

    // ---- 4. adjoint
    if (g.want_back) {
        const T* c = sC;
        for (int o = tid; o < K * NA; o += ST) {
            const int k = o / NA, mu = o - k * NA;
            const T* Bk = sB + k * NA;
            const int deg = sTab[mu] & 255;
            const T B0 = Bk[0];
            T e3 = k < K3 && deg <= P3 ? c[off3 + k * (P3 + 1) + deg] : T(0);
            T v = mu == 0 && k < K2 ? c[1 + k] : T(0);
            if (k < K4) {
                const T* c4 = c + off4 + k * Ka4;
                const int pd = n_partitions_below(deg);          // (deg, 0, 0): the first triple of its degree
                if (pd < Ka4) e3 += c4[pd] * B0;
                if (mu == 0)
                    for (int a = 0; a <= PA; ++a)
                        if (n_partitions_below(a) < Ka4) v += c4[n_partitions_below(a)] * sS[k * PA1 + a];
                // occurrences, sorted by p: four at a time, up to the first p
                // the model does not have (its weight is taken as zero)
                const int o1 = sTab[Tab::OBEG + mu + 1];
                for (int x = sTab[Tab::OBEG + mu]; x < o1; x += 4) {
                    int oc[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) oc[q] = sTab[Tab::OCC + (x + q < o1 ? x + q : o1 - 1)];
                    if ((oc[0] & 31) >= Ka4) break;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int p = oc[q] & 31;
                        const T w = x + q < o1 && p < Ka4 ? c4[p < Ka4 ? p : 0] : T(0);
                        v += w * T(oc[q] >> 19) * Bk[(oc[q] >> 5) & 127] * Bk[(oc[q] >> 12) & 127];
                    }
                }
            }
            sAb[o] = v + T(2 * (sTab[mu] >> 8)) * e3 * Bk[mu];
        }
    }
    __syncthreads();
    if (tid == 0) {
        double e = sRed[0];
        for (int w = 1; w < SW; ++w) e += sRed[w];
        if (g.E_atom) g.E_atom[i] = static_cast<T>(e);
        g.part[i] = e;
    }
    if (!g.want_back) return;

    // ---- 5. pair gradients
    double vir[9];
#pragma unroll
    for (int x = 0; x < 9; ++x) vir[x] = 0.0;
    for (int c0 = 0; c0 < n; c0 += CH) {
        const int nc = n - c0 < CH ? n - c0 : CH;
        if (n > CH) {
            int again = 0;   // errors were reported by the first pass
            stage(c0, nc, false, again);
            __syncthreads();
        }
        for (int w = tid; w < K * nc; w += ST) {
            const int k = w / nc, p = w - k * nc;
            T h, hx, hy, hz;
            poly_gradient<T, PA>(sAb + k * NA, sU[5 * p], sU[5 * p + 1], sU[5 * p + 2], h, hx, hy, hz);
            const T R = sR[p * KO + k];
            T* o = sA + 4 * (k * CH + p);
            o[0] = sdR[p * KO + k] * h;
            o[1] = R * hx;
            o[2] = R * hy;
            o[3] = R * hz;
        }
        __syncthreads();
        if (tid < nc) {
            T s = T(0), q0 = T(0), q1 = T(0), q2 = T(0);
            for (int k = 0; k < K; ++k) {
                const T* o = sA + 4 * (k * CH + tid);
                s += o[0]; q0 += o[1]; q1 += o[2]; q2 += o[3];
            }
            const T ux = sU[5 * tid], uy = sU[5 * tid + 1], uz = sU[5 * tid + 2], ri = sU[5 * tid + 3], r = sU[5 * tid + 4];
            const bool ok = r > T(0);
            const T a1 = s - (ux * q0 + uy * q1 + uz * q2) * ri;
            const T gx = ok ? a1 * ux + ri * q0 : T(0), gy = ok ? a1 * uy + ri * q1 : T(0), gz = ok ? a1 * uz + ri * q2 : T(0);
            const int p = beg + c0 + tid;
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
                const double dd[3] = {double(dv[0]), double(dv[1]), double(dv[2])};
                const double gg[3] = {double(gx), double(gy), double(gz)};
#pragma unroll
                for (int x = 0; x < 3; ++x)
#pragma unroll
                    for (int y = 0; y < 3; ++y) vir[3 * x + y] -= dd[x] * gg[y];
            }
        }
        if (n > CH) __syncthreads();
    }
    if (g.want_W && tid < WAVE) {   // the pairs' threads are wavefront 0 (CH <= 64)
        int c;
        const double sw = wave_sum9(vir, lane, c);
        if (c < 9) g.wpart[static_cast<size_t>(c) * g.N + i] = sw;
    }
}

template <typename T, int PA>
hipError_t launch_pa(const WideArgs<T>& a, int mode, bool fast, hipStream_t st) {
    const SmallLds L = small_lds(a.prm.K, PA, a.prm.M);
    const size_t lds = (L.total * sizeof(T) + 15) / 16 * 16 + (a.prm.K4 > 0 ? SmallTab<PA>::N : n_mono(PA)) * sizeof(int);
    const dim3 grid(a.N);
    const auto go = [&](auto st_c) {
        constexpr int ST = decltype(st_c)::value;
        if (mode == 0) {
            if (fast) hipLaunchKernelGGL((small_kernel<T, PA, 0, true, ST>), grid, dim3(ST), lds, st, a);
            else hipLaunchKernelGGL((small_kernel<T, PA, 0, false, ST>), grid, dim3(ST), lds, st, a);
        } else {
            if (fast) hipLaunchKernelGGL((small_kernel<T, PA, 1, true, ST>), grid, dim3(ST), lds, st, a);
            else hipLaunchKernelGGL((small_kernel<T, PA, 1, false, ST>), grid, dim3(ST), lds, st, a);
        }
    };
    if constexpr (small_max(PA) > SMALL_WIDE_N) {
        if (a.N > SMALL_WIDE_N) {
            go(std::integral_constant<int, 128>{});
            return hipGetLastError();
        }
    }
    go(std::integral_constant<int, 256>{});
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_small(const WideArgs<T>& a, int PA, int mode, bool fast, hipStream_t st) {
    if (a.N <= 0) return hipSuccess;
    switch (PA) {
        case 0: return launch_pa<T, 0>(a, mode, fast, st);
        case 1: return launch_pa<T, 1>(a, mode, fast, st);
        case 2: return launch_pa<T, 2>(a, mode, fast, st);
        case 3: return launch_pa<T, 3>(a, mode, fast, st);
        case 4: return launch_pa<T, 4>(a, mode, fast, st);
        case 5: return launch_pa<T, 5>(a, mode, fast, st);
        case 6: return launch_pa<T, 6>(a, mode, fast, st);
        default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_small<double>(const WideArgs<double>&, int, int, bool, hipStream_t);
template hipError_t launch_small<float>(const WideArgs<float>&, int, int, bool, hipStream_t);

}  // namespace pod
