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
inline int small_max(int PA) { return PA <= 4 ? 1024 : 512; }

// Threads per workgroup: 256 while the chip holds every atom at once (two
// workgroups per compute unit), 128 above (1,024 atoms: 35.0 against 28.4 us).
constexpr int SMALL_WIDE_N = 512;

inline bool small_path(int K, int PA, int N) { return !wide_path(K, PA) && N <= small_max(PA); }

// mode 0: descriptors; mode 1: energy, and with want_back the pair gradients.
// One workgroup per atom; block partials [10 + M][N] and [9][N] (the layout of
// the finalize kernel with one block per atom).  a.rec is not used.
template <typename T>
hipError_t launch_small(const WideArgs<T>& a, int PA, int mode, bool fast, hipStream_t st);

}  // namespace pod
