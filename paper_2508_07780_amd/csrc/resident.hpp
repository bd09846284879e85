// Resident solves: all time steps of one source in one launch, the fields kept on chip.
//
// A step of a grid of a few million nodes takes less time than its launch, its blocks' first
// loads and its drain.  Here the grid is cut into at most one brick per CU.  A block holds its
// brick's current level in LDS and the previous one in registers for the whole solve; per step
// it computes, publishes the values that other bricks read, and collects theirs.  Finite-
// difference bricks hold one component (the region's update couples none), so a brick's surface
// is small against its volume; finite-element bricks hold all three.
//
// Exchange: one 8-byte word per published node and component, {value, tag}, stored and polled
// with relaxed agent-scope atomics; the tag is the level's number, unique over the plan's
// solves (a direction has its own words and numbers: however often the other one runs, a word holds a tag of its
// plan's last solve, which the next one never awaits), so a word tells by itself whether it is the awaited level, and
// no flag or fence follows the data.  Words sit in a ring of two levels.  Bricks collect from each other mutually, so a
// block that publishes level n+2 has collected the level n+1 of each of its readers, which they published after
// collecting level n: the level n words it overwrites have been read.
//
// Blocks wait for each other, so all of them must be on the GPU at once.  Each announces
// itself first, and the last one to arrive starts the solve for all; if some do not get a place
// in time (the GPU is shared with other work), the launch is called off before anything is
// written, and a kernel that needs no number of blocks at once takes all steps, in two to five times the launches'
// time.  The state is decided by compare-and-swap, so every block sees the same outcome; waits during the solve are
// bounded the same way.
#pragma once

#include "dd_common.hpp"

namespace dd {

constexpr int RES_THREADS = 512;         // two waves per SIMD: 256 registers each, for the state and the operands
// Finite-difference brick: at most 32 x 32 nodes in (x, y).  LDS box with a one-node rim: rows of RES_SY
// floats (node x at 4 + x, so that four nodes are one aligned 16-byte access; the right rim of a full row is
// the next row's first float), planes of RES_SY (dim y + 2).
constexpr int RES_B = 32;
constexpr int RES_SY = RES_B + 4;
constexpr int RES_SINK = 1;             // a float that is no node's: words collected only for their order go here
constexpr int RES_RUN_MAX = 12;         // planes per thread
// special nodes per thread (and the dipole's) beside runs of up to `run` planes, as registers allow
constexpr int res_special(int run) { return run <= 8 ? 4 : 0; }
constexpr int RES_XCH = 12;           // exchange words per thread, each way
constexpr int RES_OUT = 4;              // trace / interface outputs per thread kept in registers
constexpr int RES_RING = 2;
constexpr int RES_NF_MAX = 3;             // FEM nodes per thread
constexpr int64_t RES_NODES_MAX = 11 << 18;   // 2.9 million: above, no cut fits on chip
constexpr size_t RES_LDS_MAX = 160 * 1024 - 512;
constexpr int RES_TAB = 440;            // source values per upload launch (by-value kernel argument)

// flags of a special node: outer faces, dipole
enum { RES_XL = 1, RES_XH = 2, RES_YL = 4, RES_YH = 8, RES_ZL = 16, RES_ZH = 32, RES_DIP = 64 };

struct ResBlock {
  int fem;                     // 0: finite-difference brick, 1: finite-element brick
  int lo[3], dim[3];           // brick origin (grid nodes; lattice nodes for FEM) and size
  int comp;                    // component of a finite-difference brick
  int run;                     // finite differences: planes per thread
  int sp_off, sp_n;            // special nodes: sp_meta, sp_det
  int pub_off, pub_n;          // published nodes: cells; word 3 pub_off + comp pub_n + i
  int con_off, con_n;          // collected nodes: {word, cell}
  int out_off, out_n;          // outputs: {cell | kind << 16, index}; kind 0 trace, 1 interface
  int con_fem;                 // FEM: the first con_fem collected nodes are FEM-owned, then layer 0
  int node_off;                // FEM: first of the brick's entries in fem_node
};

// The rows of thread t in a finite-difference brick: four nodes along x from 4 xq on of row ty, `run` planes (0: none)
// from z on; base: LDS float of its first node.  Runs are counted from the top: the lowest one may be shorter, and the
// top plane is every brick's plane run - 1 of its last run.  Threads without planes read the last run's rows, unused.
struct ResRows { int xq, ty, z, run; uint32_t base; };
__host__ __device__ inline ResRows res_rows(const int* dim, int run, int t) {
  ResRows r;
  const int nxq = (dim[0] + 3) / 4, tr = t / (nxq * dim[1]), runs = (dim[2] + run - 1) / run;
  r.xq = t % nxq;
  r.ty = (t / nxq) % dim[1];
  const int low = dim[2] - (tr < runs ? runs - tr : 1) * run;
  r.z = low > 0 ? low : 0;
  r.run = tr < runs ? low + run - r.z : 0;
  r.base = (uint32_t)(4 + 4 * r.xq + RES_SY * (r.ty + 1) + RES_SY * (dim[1] + 2) * (r.z + 1));
  return r;
}

struct ResCtl {
  unsigned epoch[2];           // tag of level 0 of the direction's current solve
  int arrive, state, end;      // RES_WAIT .. RES_DONE
  unsigned long long tickets, finished;   // of the last resort
  int skip;                    // a launch of this call has been called off: its other solves go to the last resort
  // per direction (forward, adjoint): solves taken by the resident kernel, launches called off, solves taken by the
  // last resort
  int solves[2], called_off[2], fallback[2];
};
enum { RES_WAIT = 0, RES_GO = 1, RES_OFF = 2, RES_FAILED = 3, RES_DONE = 4 };

// Host-built plan of a problem; empty blocks: not eligible.
struct ResPlan {
  std::vector<ResBlock> blocks;
  std::vector<uint32_t> sp_meta;       // cell | flags << 16
  std::vector<int> sp_det;             // detector index or -1
  std::vector<uint16_t> pub_cell;
  std::vector<uint32_t> con_word;      // word of component 0; the next component's is con_step further
  std::vector<uint16_t> con_step;
  std::vector<uint16_t> con_cell;
  std::vector<int> con_src;            // FEM bricks: owned id, or -1 - layer-0 index, of the node
  std::vector<uint32_t> out_cell;
  std::vector<int> out_idx;
  std::vector<int2> fem_node;          // FEM bricks: {owned id, box cell}, brick by brick (x fastest)
  int n_pub = 0;                       // published nodes
  bool adj = false, rec = false;
  int max_run = 0;                     // planes per thread
  int max_fem = 0;                     // nodes of the largest FEM brick
  size_t fem_lds = 0;                  // LDS of the largest FEM brick
  int fd_cells = 0;                    // largest FD box (cells)
  size_t lds() const { return fem_lds > 4 * (size_t)fd_cells ? fem_lds : 4 * (size_t)fd_cells; }
};

struct ResArgs {
  const ResBlock* blocks;
  const uint32_t* sp_meta; const int* sp_det; const uint16_t* pub_cell;
  const uint32_t* con_word; const uint16_t *con_step, *con_cell; const int* con_src;
  const uint32_t* out_cell; const int* out_idx; const int2* fem_node;
  unsigned long long *xbuf, *xbuf_rec;   // [RES_RING][3][n_pub]; the recompute's words
  ResCtl* ctl;
  int* off_host;                         // host word: launches called off so far
  int n_pub, n_blocks, need;
  long long wait_ticks, run_ticks;       // bounds of the waits (100 MHz clock)
  int nx, ny, nz, nt;
  int64_t N, n_l0, n_own, n_det;
  float *Efd[2], *Efem[2], *Vfem, *iring;
  const float *em1, *c1, *c2;
  const int* own_grid;
  float sk1, sk6, sb1, sb2, sb4, sb6, sb12;   // the assembled Kuhn star's entries (StarValues)
  float nu, nu2, dt2_h3;
  unsigned abs_mask, det_mask;
  int64_t top_det;                       // detector index of the top face's first node
  int blo[3], bhi[3];                    // FEM box, grid nodes
  double dt, t_switch;
  // source of a forward
  const double* tab; int n_tab;
  double pw_scale, dip_scale, pol[3];
  int plane, oblique, kind;
  float pw_amp[3], pw_kx, pw_ky, pw_omega, pw_iw, pw_sup;
  int pw_x0, pw_y0;
  double pw_t0;
  int64_t dip_idx;
  float* traces;                         // this source's rows
  float *ihist, *ckpt, *tail;            // saved forward of this source (null: not saved)
  int64_t K, n_ck, k_tail, nseg;
  // adjoint
  const float *cot, *obs;
  float *win, *win_b;
  double *g_eps, *g_sig;
  const double* mass_d;
  double inv_dt2, inv_2dt;
};

// Brick plan of a forward (or an adjoint, `rec`: one that recomputes segments) for `cus` compute
// units; an empty plan where the grid does not fit on chip.  own_api: lattice node of each FEM-owned node.
void build_resident(const dd_problem_desc& d, const std::vector<int>& own_api, int cus, bool adj, bool rec,
                    ResPlan& plan) noexcept;
// The assembled stencil of the Kuhn split has seven values up to sign: K is 6 h at the centre and -h at the
// axis neighbours, B's entries are +-1, 2, 4, 6 and 12 times h / 6 (kStarB).  False unless every
// entry of the mesh's table is one of seven floats, in that pattern.
struct StarValues { float k1, k6, b1, b2, b4, b6, b12; };
bool kuhn_star(const HostMesh& m, StarValues& v);
struct StarSlot { int x, y, z, k, b[9]; };
constexpr StarSlot kStar[15] = {
    {-1, -1, -1, 0, {0, -1, -1, -1, 0, -1, -1, -1, 0}}, {0, -1, -1, 0, {0, 1, 1, 1, 0, -2, 1, -2, 0}},
    {-1, 0, -1, 0, {0, 1, -2, 1, 0, 1, -2, 1, 0}},      {0, 0, -1, -1, {0, -1, 2, -1, 0, 2, 2, 2, -6}},
    {-1, -1, 0, 0, {0, -2, 1, -2, 0, 1, 1, 1, 0}},      {0, -1, 0, -1, {0, 2, -1, 2, -6, 2, -1, 2, 0}},
    {-1, 0, 0, -1, {-6, 2, 2, 2, 0, -1, 2, -1, 0}},     {0, 0, 0, 6, {12, -4, -4, -4, 12, -4, -4, -4, 12}},
    {1, 0, 0, -1, {-6, 2, 2, 2, 0, -1, 2, -1, 0}},      {0, 1, 0, -1, {0, 2, -1, 2, -6, 2, -1, 2, 0}},
    {1, 1, 0, 0, {0, -2, 1, -2, 0, 1, 1, 1, 0}},        {0, 0, 1, -1, {0, -1, 2, -1, 0, 2, 2, 2, -6}},
    {1, 0, 1, 0, {0, 1, -2, 1, 0, 1, -2, 1, 0}},        {0, 1, 1, 0, {0, 1, 1, 1, 0, -2, 1, -2, 0}},
    {1, 1, 1, 0, {0, -1, -1, -1, 0, -1, -1, -1, 0}}};
// Whether a forward's plan exists, by size alone.
bool resident_fits(const dd_problem_desc& d, int cus);
// Bytes of such a plan's device arrays and exchange words, at most.
size_t resident_bytes_bound(const dd_problem_desc& d, int cus, bool adj, bool rec);

// first: the call's first solve.
void launch_resident_begin(const ResArgs& a, bool adj, bool first, const double* tab, int n, hipStream_t s);
void launch_resident(const ResArgs& a, const ResPlan& plan, hipStream_t s);
// The last resort: takes all steps unless the solve is done (kernels.hip).
void launch_resident_rest(const ResArgs& a, const FdArgs& fa, const FemArgs& ea, bool adj, hipStream_t s);
int device_cus();

}  // namespace dd
