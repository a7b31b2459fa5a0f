// Full neighbour list on the device (Sec. II.A: the neighbours of atom i are
// the atoms, and periodic images, closer to atom i than the cut-off radius).
//
// Cell list in fractional coordinates of the (possibly triclinic) cell: a
// bin spans at least r_list perpendicular to each lattice plane, atoms are
// ordered by bin with a stable radix sort (positions copied into bin order,
// so a bin scan reads contiguous memory), and every atom scans the bins
// within ns_d bins of its own.  The bin offset carries the periodic image,
// so small cells produce their multiple images and self-images and no image
// is visited twice.  A count pass and a prefix sum give the offsets; a fill
// pass writes (j, packed image shift) in the same fixed order.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "pod.h"
#include "pod_internal.h"
#include "pod_plan.h"

namespace pod {
namespace {

constexpr int NB_THREADS = 256;
// Lanes per atom of the search.  List and reverse index together, 8 / 16 / 32
// lanes: 128 atoms 128 / 111 / 107 us, 15,840 atoms 164 / 151 / 151 us,
// 1,024,000 atoms (FP32) 2.48 / 2.56 / 2.77 ms (one thread per atom: 303, 324
// us and 4.25 ms), so one width serves the whole range.
constexpr int NB_LANES = 16;
constexpr int NB_SLICE = 1 << 27;      // atoms per launch of the search, which has at most 2^32 threads
constexpr int NB_MAX_WRAP = 1 << 20;   // |lattice vectors| between an atom and its home cell

__device__ __forceinline__ int floor_div(int a, int b) {
    const int q = a / b;
    return (a % b != 0 && (a < 0)) ? q - 1 : q;   // b > 0
}

// Bin of every atom; its position moved into the home cell (periodic) and
// the number of lattice vectors removed.
template <typename T>
__global__ __launch_bounds__(NB_THREADS) void bin_kernel(int N, const T* __restrict__ pos, NbGeom g,
                                                         int* __restrict__ key, int* __restrict__ idx,
                                                         double* __restrict__ wpos, int* __restrict__ wrap, int* err) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const double r[3] = {static_cast<double>(pos[3 * i]), static_cast<double>(pos[3 * i + 1]),
                         static_cast<double>(pos[3 * i + 2])};
    int c[3] = {0, 0, 0}, w[3] = {0, 0, 0};
    double rw[3] = {r[0], r[1], r[2]};
    if (!(isfinite(r[0]) && isfinite(r[1]) && isfinite(r[2]))) {
        atomicOr(err, ERR_NONFINITE);
    } else if (g.periodic) {
        double sw[3];
        for (int d = 0; d < 3; ++d) {
            const double s = r[0] * g.inv[0 * 3 + d] + r[1] * g.inv[1 * 3 + d] + r[2] * g.inv[2 * 3 + d];
            double f = floor(s);
            if (fabs(f) > NB_MAX_WRAP) {
                atomicOr(err, ERR_NEIGH);
                f = 0.0;
            }
            w[d] = static_cast<int>(f);
            sw[d] = s - f;
            c[d] = min(max(static_cast<int>(sw[d] * g.nb[d]), 0), g.nb[d] - 1);
        }
        for (int e = 0; e < 3; ++e) rw[e] = r[e] - (w[0] * g.a[0 * 3 + e] + w[1] * g.a[1 * 3 + e] + w[2] * g.a[2 * 3 + e]);
    } else {
        for (int d = 0; d < 3; ++d) c[d] = min(max(static_cast<int>((r[d] - g.lo[d]) / g.bw[d]), 0), g.nb[d] - 1);
    }
    key[i] = (c[2] * g.nb[1] + c[1]) * g.nb[0] + c[0];
    idx[i] = i;
    for (int d = 0; d < 3; ++d) {
        wpos[3 * i + d] = rw[d];
        wrap[3 * i + d] = w[d];
    }
}

__global__ __launch_bounds__(NB_THREADS) void fill_int_kernel(int* __restrict__ x, long n, int v) {
    const long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

// Bin ranges [start, end) in sorted order and the positions in sorted order.
__global__ __launch_bounds__(NB_THREADS) void order_kernel(int N, const int* __restrict__ ks,
                                                           const int* __restrict__ sidx,
                                                           const double* __restrict__ wpos, int* __restrict__ start,
                                                           int* __restrict__ end, double* __restrict__ spos) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    const int b = ks[k];
    if (k == 0 || ks[k - 1] != b) start[b] = k;
    if (k == N - 1 || ks[k + 1] != b) end[b] = k + 1;
    const int j = sidx[k];
    for (int d = 0; d < 3; ++d) spos[3 * k + d] = wpos[3 * j + d];
}

// FILL = false: number of neighbours of every atom into cnt[i];
// FILL = true: the neighbours themselves from offsets[i] on (same order).
//
// G lanes serve one atom.  The bins of one (y, z) row around the atom are
// consecutive in bin order, so a row's candidates are one range of the
// sorted atoms (one range per periodic image when the row wraps): lane s of
// the group looks up the range of segment s, then the group walks the
// segments together, G candidates per step, and a ballot gives every
// accepted candidate its place behind the earlier ones -- the order of a
// serial scan.  One thread per atom (the former split) left 247 wavefronts
// on the chip for 15,840 atoms, each serially waiting on ~200 dependent
// candidate loads.
// (Count and fill pass for 15,840 atoms: 95 + 118 us before.)
template <bool FILL, int G>
__global__ __launch_bounds__(NB_THREADS) void search_kernel(int i0, int N, NbGeom g, const int* __restrict__ key,
                                                            const int* __restrict__ sidx,
                                                            const int* __restrict__ start, const int* __restrict__ end,
                                                            const double* __restrict__ wpos,
                                                            const double* __restrict__ spos,
                                                            const int* __restrict__ wrap, long* __restrict__ cnt,
                                                            const int* __restrict__ offsets, int* __restrict__ nbr_j,
                                                            int* __restrict__ shift, int* err) {
    static_assert(G == 8 || G == 16 || G == 32, "lanes per atom");
    constexpr unsigned GM = G == 32 ? 0xFFFFFFFFu : (1u << G) - 1u;
    const int lane = threadIdx.x % WAVE, sub = threadIdx.x % G;
    const int i = i0 + static_cast<int>(blockIdx.x) * (NB_THREADS / G) + static_cast<int>(threadIdx.x) / G;
    if (i >= N) return;   // whole groups
    const int b = key[i];
    const int ci[3] = {b % g.nb[0], (b / g.nb[0]) % g.nb[1], b / (g.nb[0] * g.nb[1])};
    const double ri[3] = {wpos[3 * i], wpos[3 * i + 1], wpos[3 * i + 2]};
    int wi[3] = {0, 0, 0};
    if (FILL) { wi[0] = wrap[3 * i]; wi[1] = wrap[3 * i + 1]; wi[2] = wrap[3 * i + 2]; }
    int n = 0;
    const int out = FILL ? offsets[i] : 0;
    const int room = FILL ? offsets[i + 1] - out : 0;
    // segments of a row: one per image of the row it crosses
    const int x0 = ci[0] - g.ns[0], x1 = ci[0] + g.ns[0];
    const int s0 = g.periodic ? floor_div(x0, g.nb[0]) : 0;
    const int nseg = g.periodic ? floor_div(x1, g.nb[0]) - s0 + 1 : 1;
    const int ny = 2 * g.ns[1] + 1;
    const int total = ny * (2 * g.ns[2] + 1) * nseg;
    for (int base = 0; base < total; base += G) {
        int lo = 0, hi = 0, S = 0;   // S: image (x, y, z) as signed bytes
        const int s = base + sub;
        if (s < total) {
            const int row = s / nseg, sx = s0 + (s - row * nseg);
            int by = ci[1] + row % ny - g.ns[1], bz = ci[2] + row / ny - g.ns[2];
            int sy = 0, sz = 0;
            bool in = true;
            if (g.periodic) {
                sy = floor_div(by, g.nb[1]); by -= sy * g.nb[1];
                sz = floor_div(bz, g.nb[2]); bz -= sz * g.nb[2];
            } else {
                in = by >= 0 && by < g.nb[1] && bz >= 0 && bz < g.nb[2];
            }
            if (in) {
                const int bx0 = max(x0 - sx * g.nb[0], 0), bx1 = min(x1 - sx * g.nb[0], g.nb[0] - 1);
                const int br = (bz * g.nb[1] + by) * g.nb[0];
                lo = 0x7fffffff;
                for (int bx = bx0; bx <= bx1; ++bx) {
                    const int k0 = start[br + bx], k1 = end[br + bx];
                    if (k1 > k0) { lo = min(lo, k0); hi = max(hi, k1); }
                }
                S = (sx & 0xFF) | ((sy & 0xFF) << 8) | ((sz & 0xFF) << 16);
            }
        }
        const int live = min(G, total - base);
        for (int t = 0; t < live; ++t) {
            const int k0 = __shfl(lo, t, G), k1 = __shfl(hi, t, G);
            const int sp = __shfl(S, t, G);
            const int s3[3] = {static_cast<int>(static_cast<int8_t>(sp & 0xFF)),
                               static_cast<int>(static_cast<int8_t>((sp >> 8) & 0xFF)),
                               static_cast<int>(static_cast<int8_t>((sp >> 16) & 0xFF))};
            const bool home = sp == 0;
            double q[3] = {ri[0], ri[1], ri[2]};
            if (!home)
                for (int e = 0; e < 3; ++e)
                    q[e] = __dsub_rn(ri[e], __dadd_rn(__dadd_rn(__dmul_rn(s3[0], g.a[0 * 3 + e]),
                                                                __dmul_rn(s3[1], g.a[1 * 3 + e])),
                                                      __dmul_rn(s3[2], g.a[2 * 3 + e])));
            for (int kb = k0; kb < k1; kb += G) {
                const int k = kb + sub;
                bool hit = false;
                int j = 0;
                if (k < k1) {
                    // explicit roundings: the count and fill passes take the
                    // same decision for every pair
                    const double d0 = __dsub_rn(spos[3 * k], q[0]);
                    const double d1 = __dsub_rn(spos[3 * k + 1], q[1]);
                    const double d2 = __dsub_rn(spos[3 * k + 2], q[2]);
                    j = sidx[k];
                    const double r2 = __dadd_rn(__dadd_rn(__dmul_rn(d0, d0), __dmul_rn(d1, d1)), __dmul_rn(d2, d2));
                    hit = r2 < g.rl2 && !(home && j == i);
                }
                const unsigned m = static_cast<unsigned>(__ballot(hit) >> (lane - sub)) & GM;
                if (FILL && hit) {
                    const int at = n + __popc(m & ((1u << sub) - 1u));
                    if (at >= room) {   // the count pass saw fewer pairs: never write past the row
                        atomicOr(err, ERR_NEIGH);
                    } else {
                        // image in the caller's coordinates: r_ij = pos_j + n a - pos_i
                        const int n0 = s3[0] - wrap[3 * j] + wi[0];
                        const int n1 = s3[1] - wrap[3 * j + 1] + wi[1];
                        const int n2 = s3[2] - wrap[3 * j + 2] + wi[2];
                        if (n0 < -127 || n0 > 127 || n1 < -127 || n1 > 127 || n2 < -127 || n2 > 127)
                            atomicOr(err, ERR_NEIGH);   // beyond the signed-byte shift
                        nbr_j[out + at] = j;
                        shift[out + at] = (n0 & 0xFF) | ((n1 & 0xFF) << 8) | ((n2 & 0xFF) << 16);
                    }
                }
                n += __popc(m);
            }
        }
    }
    if (!FILL && sub == 0) cnt[i] = n;
}

// int32 offsets from the 64-bit prefix sum; total[0] = number of pairs.
__global__ __launch_bounds__(NB_THREADS) void offsets_kernel(int N, const long* __restrict__ off64,
                                                             int* __restrict__ offsets, long* __restrict__ total) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > N) return;
    const long v = off64[i];
    offsets[i] = v > 0x7fffffffL ? 0x7fffffff : static_cast<int>(v);
    if (i == N) total[0] = v;
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Bounding box of an open system (host copy of the positions).
int open_geometry_dev(pod_handle* h, int N, const void* pos, double rlist, NbGeom* g) {
    std::vector<double> hp(3 * static_cast<size_t>(N));
    if (h->dtype == POD_F64) {
        if (hipMemcpyAsync(hp.data(), pos, hp.size() * sizeof(double), hipMemcpyDeviceToHost, h->stream) !=
                hipSuccess ||
            hipStreamSynchronize(h->stream) != hipSuccess)
            return POD_EHIP;
    } else {
        std::vector<float> hf(hp.size());
        if (hipMemcpyAsync(hf.data(), pos, hf.size() * sizeof(float), hipMemcpyDeviceToHost, h->stream) !=
                hipSuccess ||
            hipStreamSynchronize(h->stream) != hipSuccess)
            return POD_EHIP;
        for (size_t k = 0; k < hf.size(); ++k) hp[k] = hf[k];
    }
    return open_geometry(hp.data(), N, rlist, g);
}

}  // namespace
}  // namespace pod

extern "C" {

int pod_build_neighbors(pod_handle* h, int N, const void* pos, const double* cell, double rlist, int* offsets,
                        int* nbr_j, int* shift, long capacity, long* n_pairs) {
    using namespace pod;
    if (!h || N < 0 || !offsets || !n_pairs || capacity < 0) return POD_EINVAL;
    if (N > 0 && !pos) return POD_EINVAL;
    if (capacity > 0 && (!nbr_j || !shift)) return POD_EINVAL;
    if (rlist == 0.0) rlist = h->rcut;
    if (!(rlist > 0.0) || !std::isfinite(rlist)) return POD_EINVAL;
    *n_pairs = 0;
    const dim3 tb(NB_THREADS);
    const dim3 gb(static_cast<unsigned>((static_cast<long>(N) + NB_THREADS) / NB_THREADS));   // N + 1 threads
    if (N == 0) {
        hipLaunchKernelGGL(fill_int_kernel, dim3(1), tb, 0, h->stream, offsets, 1L, 0);
        return hipStreamSynchronize(h->stream) == hipSuccess ? POD_OK : POD_EHIP;
    }
    NbGeom g{};
    {
        const int rc = cell ? periodic_geometry(cell, rlist, &g) : open_geometry_dev(h, N, pos, rlist, &g);
        if (rc != POD_OK) return rc;
    }
    const long nbins = static_cast<long>(g.nb[0]) * g.nb[1] * g.nb[2];
    int key_bits = 1;
    while ((1L << key_bits) < nbins) ++key_bits;

    size_t sort_bytes = 0, scan_bytes = 0;
    if (rocprim::radix_sort_pairs(nullptr, sort_bytes, static_cast<int*>(nullptr), static_cast<int*>(nullptr),
                                  static_cast<int*>(nullptr), static_cast<int*>(nullptr), N, 0u,
                                  static_cast<unsigned>(key_bits), h->stream) != hipSuccess ||
        rocprim::exclusive_scan(nullptr, scan_bytes, static_cast<long*>(nullptr), static_cast<long*>(nullptr), 0L,
                                static_cast<size_t>(N) + 1, rocprim::plus<long>(), h->stream) != hipSuccess)
        return POD_EHIP;
    const size_t n1 = static_cast<size_t>(N) + 1;
    const size_t sI = align256(sizeof(int) * n1), sL = align256(sizeof(long) * n1);
    const size_t sP = align256(sizeof(double) * 3 * n1), sW = align256(sizeof(int) * 3 * n1);
    const size_t sB = align256(sizeof(int) * static_cast<size_t>(nbins)), sT = align256(std::max(sort_bytes, scan_bytes));
    const int rc = ensure_scratch(h, 4 * sI + 2 * sL + 2 * sP + sW + 2 * sB + sT);
    if (rc != POD_OK) return rc;
    char* base = static_cast<char*>(h->d_scratch);
    auto take = [&base](size_t bytes) { char* p = base; base += bytes; return p; };
    int* key = reinterpret_cast<int*>(take(sI));
    int* key_s = reinterpret_cast<int*>(take(sI));
    int* idx = reinterpret_cast<int*>(take(sI));
    int* idx_s = reinterpret_cast<int*>(take(sI));
    long* cnt = reinterpret_cast<long*>(take(sL));
    long* off64 = reinterpret_cast<long*>(take(sL));
    double* wpos = reinterpret_cast<double*>(take(sP));
    double* spos = reinterpret_cast<double*>(take(sP));
    int* wrap = reinterpret_cast<int*>(take(sW));
    int* start = reinterpret_cast<int*>(take(sB));
    int* end = reinterpret_cast<int*>(take(sB));
    void* tmp = take(sT);

    if (h->dtype == POD_F64)
        hipLaunchKernelGGL((bin_kernel<double>), gb, tb, 0, h->stream, N, static_cast<const double*>(pos), g, key, idx,
                           wpos, wrap, h->d_err);
    else
        hipLaunchKernelGGL((bin_kernel<float>), gb, tb, 0, h->stream, N, static_cast<const float*>(pos), g, key, idx,
                           wpos, wrap, h->d_err);
    size_t tbytes = sT;
    if (rocprim::radix_sort_pairs(tmp, tbytes, key, key_s, idx, idx_s, N, 0u, static_cast<unsigned>(key_bits),
                                  h->stream) != hipSuccess)
        return POD_EHIP;
    const dim3 gbins(static_cast<unsigned>((nbins + NB_THREADS - 1) / NB_THREADS));
    hipLaunchKernelGGL(fill_int_kernel, gbins, tb, 0, h->stream, start, nbins, 0);
    hipLaunchKernelGGL(fill_int_kernel, gbins, tb, 0, h->stream, end, nbins, 0);
    hipLaunchKernelGGL(order_kernel, gb, tb, 0, h->stream, N, key_s, idx_s, wpos, start, end, spos);
    const auto search = [&](auto fill) {
        for (long i0 = 0; i0 < N; i0 += NB_SLICE) {
            const long n = std::min<long>(N - i0, NB_SLICE);
            const dim3 gs(static_cast<unsigned>((n * NB_LANES + NB_THREADS - 1) / NB_THREADS));
            hipLaunchKernelGGL((search_kernel<decltype(fill)::value, NB_LANES>), gs, tb, 0, h->stream,
                               static_cast<int>(i0), static_cast<int>(i0 + n), g, key, idx_s, start, end, wpos, spos, wrap,
                               cnt, offsets, nbr_j, shift, h->d_err);
        }
    };
    search(std::false_type{});
    hipLaunchKernelGGL(fill_int_kernel, dim3(1), tb, 0, h->stream, reinterpret_cast<int*>(cnt + N), 2L, 0);
    tbytes = sT;
    if (rocprim::exclusive_scan(tmp, tbytes, cnt, off64, 0L, static_cast<size_t>(N) + 1, rocprim::plus<long>(),
                                h->stream) != hipSuccess)
        return POD_EHIP;
    hipLaunchKernelGGL(offsets_kernel, gb, tb, 0, h->stream, N, off64, offsets, cnt);
    long P = 0;
    if (hipMemcpyAsync(&P, cnt, sizeof(long), hipMemcpyDeviceToHost, h->stream) != hipSuccess ||
        hipStreamSynchronize(h->stream) != hipSuccess)
        return POD_EHIP;
    *n_pairs = P;
    if (P > 0x7fffffffL) return POD_ENOTSUP;   // int32 offsets
    if (P > 0 && capacity >= P) {
        search(std::true_type{});
        if (hipStreamSynchronize(h->stream) != hipSuccess) return POD_EHIP;
    }
    return hipGetLastError() == hipSuccess ? POD_OK : POD_EHIP;
}

}  // extern "C"
