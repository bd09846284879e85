// Host checks of the brick plans of resident solves: one problem per input line,
//   cus  n_outer[3]  fem_lo[3]  fem_cells[3]  n_steps  detector_faces  absorbing_faces  adjoint  recompute
// and one output line for it,
//   blocks  longest run  most nodes of an FEM brick  LDS bytes  threads' LDS rows outside their brick's box
// (0 blocks: the grid does not fit on chip).
#include <algorithm>
#include <cstdio>

#include "resident.hpp"

using namespace dd;

namespace {

// Threads of a brick whose rows, or the rows beside them, lie outside its LDS box.
int rows_outside(const ResBlock& b, size_t lds) {
  const int SZ = RES_SY * (b.dim[1] + 2), box = SZ * (b.dim[2] + 2);
  int bad = 4 * (size_t)box > lds;
  for (int t = 0; t < RES_THREADS; ++t) {
    const ResRows r = res_rows(b.dim, b.run, t);
    // the first plane's row and the planes below and above, in every plane of the run
    const int first = (int)r.base - SZ, last = (int)r.base + SZ * std::max(r.run, 1) + 4;
    bad += first < 0 || last >= box;
  }
  return bad;
}

}  // namespace

int main() {
  int cus, n[3], lo[3], cells[3], nt, det, damp, adj, rec;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", &cus, &n[0], &n[1], &n[2], &lo[0], &lo[1], &lo[2],
                    &cells[0], &cells[1], &cells[2], &nt, &det, &damp, &adj, &rec) == 15) {
    dd_problem_desc d{};
    std::vector<int> own;          // owned nodes in lattice order
    for (int a = 0; a < 3; ++a) {
      d.n_outer[a] = n[a];
      d.fem_lo[a] = lo[a];
      d.fem_cells[a] = cells[a];
    }
    for (int z = 1; z < cells[2]; ++z)
      for (int y = 1; y < cells[1]; ++y)
        for (int x = 1; x < cells[0]; ++x) own.push_back(x + (cells[0] + 1) * (y + (cells[1] + 1) * z));
    d.n_steps = nt;
    d.detector_faces = (uint32_t)det;
    d.absorbing_faces = (uint32_t)damp;
    ResPlan p;
    build_resident(d, own, cus, adj != 0, rec != 0, p);
    int fem = 0, bad = 0;
    for (const ResBlock& b : p.blocks) {
      if (b.fem) fem = std::max(fem, b.dim[0] * b.dim[1] * b.dim[2]);
      else bad += rows_outside(b, p.lds());
    }
    std::printf("%zu %d %d %zu %d\n", p.blocks.size(), p.max_run, fem, p.lds(), bad);
  }
  return 0;
}
