// Energy path and descriptors of small systems: one workgroup per atom.
// Internal to libpod; the host side of the energy path chooses it by the
// number of atoms.
#pragma once

#include <hip/hip_runtime.h>

#include "pod_internal.h"
#include "pod_wide.h"

namespace pod {

// Up to this many atoms one workgroup per atom is faster than the per-atom
// kernel, whose wavefronts take 64 / K atoms each and need about 20 us however
// few there are.  Energy and forces per call, per-atom and pair kernels / this
// path (FP64): K = 6, degree 4: 128 atoms 33.4 / 22.9 us, 686 34.1 / 26.5, 1,024
// 34.4 / 28.4, 1,458 35.3 / 47.6; 4-body degree 6: 128 atoms 65.4 / 42.2, 432
// 65.9 / 45.5, 1,024 66.5 / 85.5; K = 7, P3 = 6: 128 atoms 84.7 / 23.1.
// Descriptors, degree 4: 128 atoms 16.7 / 10.5 us, 1,024 16.9 / 13.1, 2,000 17.2
// / 23.9.  (About 23 us of a call are the caller's side.)
constexpr int small_max(int PA) { return PA <= 4 ? 1024 : 512; }

// Threads per workgroup: 256 while the chip holds every atom at once (two
// workgroups per compute unit), 128 above (1,024 atoms: 35.0 against 28.4 us).
constexpr int SMALL_WIDE_N = 512;

// With short lists the per-atom kernel has little left to do in turn: K lanes take
// an atom's list K pairs a round, P / (N K) rounds, while this path still brings
// the tables of the 4-body terms to every atom.  Per-atom kernel / this path, us:
//   forces: ahead from the first pair on (0.4 pairs per atom: at most 0.94 of the
//     other), so only 4-body models without any pair go the other way (K = 8, degree
//     6: 30 / 44);
//   descriptors and energy alone, degree up to 4, FP32: N <= 512 1.0 round (K = 8)
//     10.1 / 10.6, 1.8 rounds 10.6 / 10.7, 2.3 (K = 6) 11.1 / 9.7; above 512 atoms 1.8
//     rounds 10.6 / 12.5, 2.3 11.1 / 11.5, 2.8 (K = 5) 10.8 / 10.0, 3.3 (K = 8) 14.8 /
//     13.1; without 4-body terms 0.7 rounds (K = 6) 7.6 / 7.6 at any N;
//   above degree 4, descriptors with 4-body terms: 1.8 rounds 15.9 / 19.6, 2.5 18.1 /
//     19.7, 3.3 21.7 / 20.3; others 0.4 rounds 1.03 of the other, 0.6 0.88.
enum class SmallCall { descriptors, energy, forces };
inline bool small_path(int K, int K4, int PA, int N, int P, SmallCall call) {
    if (wide_path(K, PA) || N > small_max(PA)) return false;
    if (call == SmallCall::forces) return P > 0 || K4 == 0;
    const long p2 = 2L * P, round = static_cast<long>(K) * N;   // p2 / round: twice the rounds
    if (PA > 4) return p2 >= (call == SmallCall::descriptors && K4 > 0 ? 6 : 1) * round;
    return p2 >= (K4 == 0 ? 2 : N <= SMALL_WIDE_N ? 4 : 5) * round;
}

// mode 0: descriptors; mode 1: energy, and with want_back the pair gradients.
// One workgroup per atom; block partials [10 + M][N] and [9][N] (the layout of
// the finalize kernel with one block per atom).  a.rec is not used.
template <typename T>
hipError_t launch_small(const WideArgs<T>& a, int PA, int mode, bool fast, hipStream_t st);

}  // namespace pod
