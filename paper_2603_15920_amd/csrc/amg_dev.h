// Device form of the smoothed-aggregation AMG preconditioner (amg.hip).
#pragma once

#include "amg.h"
#include "internal.h"
#include "ops.h"

namespace difvm {

struct PcgCtl;
struct AmgDev;

// The update of a CG iteration, made by the first kernel of the cycle after it: with alpha from the segment's
// p.q partials (pq), x += alpha p and r_new = r - alpha q.
struct CgStep {
  double* x;
  const double *p, *r, *q, *pq;
  double* r_new;
};

// Builds the hierarchy from the symmetric cell-slot matrix K (copied to the host; synchronises) and
// uploads it.  No face joins two segments, so no aggregate does either and every level stays
// block-diagonal over the segments.  Throws Error.
AmgDev* amg_create(difvm_mesh* m, SellMatrix K, const AmgOptions& opt);
void amg_free(AmgDev* a);
// z = M^-1 r, one symmetric V-cycle (one degree-2 Chebyshev sweep on every level before and after
// each coarse correction, a dense solve on the coarsest; the finest level uses K, the coarser ones
// the stored Galerkin operators), queued on the mesh's stream.  part != nullptr: the last kernel stores per-tile partials of r.z at part[t].
// ctl != nullptr (the per-segment CG states): every kernel returns at once when all segments have
// stopped (iterations queued after the stop).  rr != nullptr: the first kernel also makes the stopping test
// of CG iterate k, whose r.r partials these are (as the product of iteration k + 1 does), so that the
// cycle after the last iteration ends there.  step != nullptr (with rr, on meshes of fine_spans): the first kernel
// also makes iteration k's update, storing r (= step->r_new) and the partials rr, and the second makes the test.
// res: scratch of one value per cell (may be step->q); the hierarchy has its own otherwise.
void amg_vcycle(const AmgDev* a, SellMatrix K, const double* r, double* z, double* part, PcgCtl* ctl,
                double* rr = nullptr, int k = 0, const CgStep* step = nullptr, double* res = nullptr);
// Whether a whole CG solve with this preconditioner fits one block (a mesh of one segment and at most four
// tiles, two levels), and that solve: at most `chunk` further iterations in one launch (the first makes the
// control state); r and p keep what the next launch needs.
bool amg_pcg_in_block(const AmgDev* a);
void amg_pcg_block(const AmgDev* a, SellMatrix K, const double* b, double* x, double* r, double* p, double tol,
                   int maxit, int chunk, bool first, PcgCtl* ctl);
// rows per level (finest first) into rows[0..cap); returns the number of levels
int amg_levels(const AmgDev* a, int* rows, int cap);
// Algorithmic bytes of one V-cycle: every kernel's distinct inputs read once and outputs written
// once, the finest level's matrix in its LDU form (diagonal, one coefficient and the owner /
// neighbour indices per internal face), coarse matrices in CSR (row pointers, 4-byte columns, 8-byte
// values, diagonal), the coarsest inverse dense.
double amg_vcycle_bytes(const AmgDev* a);

}  // namespace difvm
