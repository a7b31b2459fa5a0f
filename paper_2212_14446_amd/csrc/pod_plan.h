// Host-only planning logic of libpod: parameter validation, the POD radial
// basis, the neighbour-list bin geometry and the batch-assembly plan.  Plain
// C++ with no HIP types, so that it also builds on its own with g++ for the
// host-code sanitizer tests; the kernels' sources use the plain structs and
// constexpr layouts declared here.
#pragma once

#include <cstddef>
#include <vector>

#include "pod.h"

namespace pod {

// Parameter checks of pod_init / pod_compute_basis (POD_OK, POD_EINVAL, POD_ENOTSUP).
int validate_params(const pod_params* p);

// Snapshot l of the family at distance r, eqs. (3)-(8), in double.
double snapshot_value(const pod_params* p, int l, double r);

// POD basis of the snapshot family (Sec. II.B, eqs. (9)-(12)): midpoint rule
// on (rin, rcut) with n_quad points (2000 when zero), eigenvectors of the L x L
// covariance by cyclic Jacobi, sorted by decreasing eigenvalue, each column's
// largest component made positive.  Q: L x L row-major (column k = mode k).
int compute_basis(const pod_params* p, std::vector<double>& Q, std::vector<double>& eig);

// Neighbour-list bin geometry, passed by value to the neighbour kernels.
constexpr int NB_MAX_BINS = 256;   // per direction (wider bins stay correct)
constexpr int NB_MAX_SPAN = 64;    // search half-width in bins

struct NbGeom {
    double a[9];     // periodic: lattice vectors as rows
    double inv[9];   // periodic: inverse of a, fractional s = r inv
    double lo[3];    // open: bounding-box origin
    double bw[3];    // open: bin width
    double rl2;      // r_list^2
    int nb[3];       // bins per direction
    int ns[3];       // search half-width in bins
    int periodic;
};

// Periodic cell (lattice vectors as rows): bins at least r_list apart
// perpendicular to each lattice plane and the search half-width that covers
// r_list.  POD_EINVAL for a singular or non-finite cell or r_list,
// POD_ENOTSUP when the search would span more than NB_MAX_SPAN bins.
int periodic_geometry(const double* cell, double rlist, NbGeom* g);

// Open system from a host copy of the positions (N x 3): bounding box of the
// finite coordinates, bins of at least r_list, search half-width 1.
int open_geometry(const double* pos, int N, double rlist, NbGeom* g);

// LDS layout of one batch-assembly workgroup: Q, the cell's G row, the
// dG/dR chunk accumulator (nc_max atoms x 3 x cw columns) and the atom offsets.
struct BatchLds {
    size_t q, gsum, acc, off, total;
};

constexpr BatchLds batch_lds(int M, int cw, int nc_max) {
    BatchLds L{};
    const size_t d = sizeof(double);
    L.q = 0;
    L.gsum = L.q + static_cast<size_t>(POD_MAX_L) * POD_MAX_K * d;
    L.acc = L.gsum + static_cast<size_t>(M + 1) * d;
    L.off = L.acc + static_cast<size_t>(nc_max) * 3 * cw * d;
    L.total = L.off + static_cast<size_t>(nc_max + 1) * sizeof(int);
    return L;
}

constexpr int BATCH_MAX_THREADS = 512;

// Rounds of pod_batch_assemble: the pair records and basis rows of one
// round's cells are in scratch at a time.  Cells are taken in order; a round
// ends before the cell that would take its scratch beyond cap bytes (a cell
// that needs more by itself has a round of its own) or after BATCH_MAX_CELLS
// cells (a launch has at most 2^32 threads).  A cell has longest[cell]
// x atoms record entries of per_ent bytes (lists padded to the cell's longest)
// and per_atom bytes for every atom.
constexpr int BATCH_MAX_CELLS = 1 << 20;

struct BatchRounds {
    std::vector<int> first;      // first cell of every round, then n_cfg
    std::vector<long> ebase;     // first record entry of every cell within its round
    std::vector<long> n_ent;     // record entries of every round
    std::vector<long> ent_max;   // record entries of its largest cell
    size_t bytes;                // scratch of the largest round
};

void plan_rounds(int n_cfg, const int* coff, const int* longest, size_t per_ent, size_t per_atom, size_t cap,
                 BatchRounds* r);

// The rounds for which alloc(bytes of scratch) does not answer POD_ENOMEM: of at
// most cap bytes, else of half as much, and so on down to the largest cell's own.
// Returns alloc's last answer.
template <typename Alloc>
int fit_rounds(int n_cfg, const int* coff, const int* longest, size_t per_ent, size_t per_atom, size_t cap, Alloc alloc,
               BatchRounds* r) {
    plan_rounds(n_cfg, coff, longest, per_ent, per_atom, cap, r);
    for (;;) {
        const int rc = alloc(r->bytes);
        if (rc != POD_ENOMEM) return rc;
        const size_t tried = r->bytes;
        plan_rounds(n_cfg, coff, longest, per_ent, per_atom, tried / 2, r);
        if (r->bytes >= tried) return rc;   // the largest cell alone
    }
}

// Launch plan of pod_batch_assemble from host copies of the cell atom
// offsets coff[n_cfg + 1] and the pair offsets off[N + 1]: the widest chunk
// (largest that fits lds_max, from the tuning value or 17 down), the atoms of
// the LDS accumulator, the processing order of the cells (decreasing pair
// count, stable) and the longest pair list of each cell.  The other fields describe the plan (cell and pair maxima, LDS
// bytes at that width, a workgroup and thread count); the launch itself takes
// its grid from the cells and its threads from the tuning value or its own rule.
struct BatchPlan {
    int cw, nblk, nth, nc_max, max_nc, max_pc;
    size_t lds;
    std::vector<int> order, longest;
};

// POD_EINVAL for offsets that do not start at 0, end at N / P or decrease
// between cells or for a bad thread count, POD_ENEIGH for pair offsets that
// decrease within a cell, POD_ENOTSUP when even one column does not fit LDS.
int plan_batch(int n_cfg, int N, int P, const int* coff, const int* off, int M, size_t lds_max,
               const pod_tune* tune, BatchPlan* plan);

}  // namespace pod
