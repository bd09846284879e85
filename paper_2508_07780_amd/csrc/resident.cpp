// Host plans of resident solves: how the grid is cut into bricks, and per brick the lists of the
// nodes it updates, publishes, collects and writes out (resident.hpp).
#include "resident.hpp"

#include <algorithm>
#include <array>
#include <atomic>
#include <thread>

namespace dd {
namespace {

struct Cut {
  int dim[3] = {0, 0, 0};   // brick size (the last brick of an axis may be smaller)
  int num[3] = {0, 0, 0};
  int blocks = 0;
  double words = 0.0;       // published words of all bricks, roughly
  double us = 0.0;          // compute time of the fullest brick
};

// Cost model of a step's parts that depend on the cut, fitted on an MI355X to steps of 25^3 (FD bricks of 1, 2 and 3
// planes per thread: 2.43, 2.74 and 3.52 us), 64^3 (3, 4, 6, 8, 11 planes: 4.15, 4.46, 5.43, 6.28, 6.88 us) and
// 96^3, and for the FEM bricks to adjoint steps with the recompute (256, 512 nodes beside 37x35x41: 5.9, 6.8 us; 768,
// 1008, 1120 nodes at 96^3: 11.1, 11.7, 13.4 us): planes of a thread and waves of nodes per SIMD; per word of all
// bricks' exchange, 1.7 ps.
constexpr double kWordUs = 1.7e-6;
double fd_us(int run, bool adj) { return 0.45 * run + (adj ? 0.6 : 0.0); }
double fem_us(int nodes, bool adj, bool rec) {
  const int waves = (nodes + 255) / 256;
  return rec ? 2.9 + 0.9 * waves : adj ? 1.2 + 0.8 * waves : 0.75 * waves;
}

// Planes per thread of a brick: a thread takes four nodes along x and a run of planes.
int run_of(int bx, int by, int bz) {
  const int plane = (bx + 3) / 4 * by, runs = RES_THREADS / plane;
  return runs ? (bz + runs - 1) / runs : RES_RUN_MAX + 1;
}
// LDS of a finite-element brick: its box, and the recompute's
size_t fem_bytes(int bx, int by, int bz, bool rec) { return (rec ? 32 : 16) * (size_t)((bx + 2) * (by + 2) * (bz + 2)); }
size_t fd_floats(int by, int bz) { return (size_t)RES_SY * (by + 2) * (bz + 2); }

// FEM-owned nodes of axis a, as grid indices: lo + 1 .. lo + cells - 1.
void owned_range(const dd_problem_desc& d, int a, int& beg, int& end) {
  beg = d.fem_lo[a] + 1;
  end = d.fem_lo[a] + d.fem_cells[a];
}

bool inside(const dd_problem_desc& d, const int lo[3], const int hi[3]) {   // [lo, hi) all FEM-owned
  for (int a = 0; a < 3; ++a) {
    int b, e;
    owned_range(d, a, b, e);
    if (lo[a] < b || hi[a] > e) return false;
  }
  return true;
}

std::vector<int> sizes_of(int n, int most) {
  std::vector<int> s;
  for (int k = (n + most - 1) / most; k <= n; ++k) {
    const int b = (n + k - 1) / k;
    if (s.empty() || s.back() != b) s.push_back(b);
    if (b <= 2) break;
  }
  return s;
}

std::vector<Cut> fd_cuts(const dd_problem_desc& d, int most_blocks, bool adj) {
  std::vector<Cut> out;
  const int* n = d.n_outer;
  // side faces whose nodes are updated one by one
  const unsigned sides = d.absorbing_faces & ~(unsigned)(DD_FACE_TOP | DD_FACE_BOTTOM);
  const bool special = sides || (adj && (d.detector_faces & ~(unsigned)DD_FACE_TOP));
  // nodes that bricks have to hold: fewer blocks than this over the brick's size hold none of the others
  const int64_t nodes = 3 * ((int64_t)n[0] * n[1] * n[2] -
                             (int64_t)(d.fem_cells[0] - 1) * (d.fem_cells[1] - 1) * (d.fem_cells[2] - 1));
  const std::vector<int> sx = sizes_of(n[0], RES_B), sy = sizes_of(n[1], RES_B), sz = sizes_of(n[2], 64);
  for (int bx : sx)
    for (int by : sy)
      for (int bz : sz) {
        if (nodes > (int64_t)most_blocks * bx * by * bz) break;
        const int run = run_of(bx, by, bz);
        if (special && !res_special(run)) continue;
        // rim copies along the outer faces (RIM1, RIM4 per thread)
        if (2 * by * bz > 4 * RES_THREADS || 2 * ((bx + 3) / 4) * (by + bz) > 2 * RES_THREADS) continue;
        if (run > RES_RUN_MAX || 4 * fd_floats(by, bz) > RES_LDS_MAX) continue;
        Cut c;
        const int b[3] = {bx, by, bz};
        for (int a = 0; a < 3; ++a) {
          c.dim[a] = b[a];
          c.num[a] = (n[a] + b[a] - 1) / b[a];
        }
        // bricks whose nodes are all FEM-owned are dropped
        int64_t in = 1;
        for (int a = 0; a < 3; ++a) {
          int ob, oe, first, last;
          owned_range(d, a, ob, oe);
          first = (ob + b[a] - 1) / b[a];
          last = oe / b[a];                     // brick [last * b, ...) starts past the range's whole bricks
          in *= std::max(0, last - first);
        }
        const int64_t bricks = (int64_t)c.num[0] * c.num[1] * c.num[2] - in;
        if (3 * bricks > most_blocks) continue;
        c.blocks = (int)(3 * bricks);
        c.words = c.blocks * 2.0 * ((double)bx * by + (double)by * bz + (double)bx * bz);
        c.us = fd_us(run, adj);
        out.push_back(c);
      }
  return out;
}

std::vector<Cut> fem_cuts(const dd_problem_desc& d, int most_blocks, bool adj, bool rec) {
  std::vector<Cut> out;
  int n[3];
  for (int a = 0; a < 3; ++a) n[a] = d.fem_cells[a] - 1;
  const std::vector<int> sx = sizes_of(n[0], 32), sy = sizes_of(n[1], 32), sz = sizes_of(n[2], 32);
  for (int bx : sx)
    for (int by : sy)
      for (int bz : sz) {
        if ((int64_t)n[0] * n[1] * n[2] > (int64_t)most_blocks * bx * by * bz) break;
        if (bx * by * bz > RES_NF_MAX * RES_THREADS) continue;
        Cut c;
        const int b[3] = {bx, by, bz};
        int64_t blocks = 1;
        for (int a = 0; a < 3; ++a) {
          c.dim[a] = b[a];
          c.num[a] = (n[a] + b[a] - 1) / b[a];
          blocks *= c.num[a];
        }
        if (blocks > most_blocks) continue;
        const int cells = (bx + 2) * (by + 2) * (bz + 2);
        if (fem_bytes(bx, by, bz, rec) > RES_LDS_MAX) continue;
        if (3 * (cells - bx * by * bz) > RES_XCH * RES_THREADS) continue;
        c.blocks = (int)blocks;
        c.words = blocks * 3.0 * (cells - bx * by * bz) * (rec ? 2.0 : 1.0);
        c.us = fem_us(bx * by * bz, adj, rec);
        out.push_back(c);
      }
  return out;
}

int m_fx(const dd_problem_desc& d) { return d.fem_cells[0] + 1; }
int m_fy(const dd_problem_desc& d) { return d.fem_cells[1] + 1; }

int fd_cell(int x, int y, int z, int by) { return (x + 4) + RES_SY * ((y + 1) + (by + 2) * (z + 1)); }

// The cheapest pair of cuts with at most one block per CU; false where nothing fits on chip.
bool choose(const dd_problem_desc& d, int cus, bool adj, bool rec, Cut& fd, Cut& fe) {
  const int64_t N = (int64_t)d.n_outer[0] * d.n_outer[1] * d.n_outer[2];
  if (d.n_steps < 4 || N > RES_NODES_MAX) return false;
  // compute times take few values: per time and number of blocks, the cut with the fewest words of those with at
  // most as many blocks
  struct Best { double us; std::vector<const Cut*> by_blocks; };
  const auto table = [cus](const std::vector<Cut>& cuts) {
    std::vector<Best> t;
    for (const Cut& c : cuts) {
      auto it = std::find_if(t.begin(), t.end(), [&](const Best& b) { return b.us == c.us; });
      if (it == t.end()) it = t.insert(t.end(), Best{c.us, std::vector<const Cut*>(cus + 1)});
      const Cut*& at = it->by_blocks[c.blocks];
      if (!at || c.words < at->words) at = &c;
    }
    for (Best& b : t)
      for (int n = 1; n <= cus; ++n)
        if (b.by_blocks[n - 1] && (!b.by_blocks[n] || b.by_blocks[n - 1]->words <= b.by_blocks[n]->words))
          b.by_blocks[n] = b.by_blocks[n - 1];
    return t;
  };
  const std::vector<Cut> fds = fd_cuts(d, cus - 1, adj), fems = fem_cuts(d, cus - 3, adj, rec);
  double best = 1e30;
  const std::vector<Best> tfd = table(fds), tfe = table(fems);
  for (const Best& f : tfd)
    for (const Best& e : tfe)
      for (int n = 3; n < cus; n += 3) {
        const Cut *x = f.by_blocks[n], *y = e.by_blocks[cus - n];
        if (!x || !y) continue;
        const double t = std::max(f.us, e.us) + kWordUs * (x->words + y->words);
        if (t < best) { best = t; fd = *x; fe = *y; }
      }
  return best < 1e30;
}

}  // namespace

bool kuhn_star(const HostMesh& m, StarValues& v) {
  if (!m.stencil_ok || m.n_slots != 15) return false;
  v.k6 = m.slot_k[7];
  v.k1 = -m.slot_k[3];
  v.b1 = -m.slot_b[9 * 0 + 1];
  v.b2 = m.slot_b[9 * 3 + 2];
  v.b4 = -m.slot_b[9 * 7 + 1];
  v.b6 = -m.slot_b[9 * 3 + 8];
  v.b12 = m.slot_b[9 * 7];
  const auto value = [&](int k) {
    const int n = std::abs(k);
    const float f = n == 1 ? v.b1 : n == 2 ? v.b2 : n == 4 ? v.b4 : n == 6 ? v.b6 : n == 12 ? v.b12 : 0.f;
    return k < 0 ? -f : f;
  };
  for (int s = 0; s < 15; ++s) {
    const StarSlot& q = kStar[s];
    if (m.slot_off[4 * s] != q.x || m.slot_off[4 * s + 1] != q.y || m.slot_off[4 * s + 2] != q.z) return false;
    if (m.slot_k[s] != (q.k == 6 ? v.k6 : q.k ? -v.k1 : 0.f)) return false;
    for (int e = 0; e < 9; ++e)
      if (m.slot_b[9 * s + e] != value(q.b[e])) return false;
  }
  return true;
}

namespace {

// f(brick) for every brick, on several threads where there are many: the lists of a grid of 96^3 take about 4 ms on one
// thread, as long as a few hundred of its steps gain.  False where f fails or throws.
template <class F>
bool each_brick(int n, F&& f) {
  std::atomic<int> next{0};
  std::atomic<bool> ok{true};
  const auto work = [&]() noexcept {
    try {
      for (int b; ok && (b = next++) < n;)
        if (!f(b)) ok = false;
    } catch (...) {
      ok = false;
    }
  };
  std::thread pool[7];
  const int threads = std::min<int>({n / 16, 7, (int)std::thread::hardware_concurrency() - 1});
  for (int i = 0; i < threads; ++i) {
    try {
      pool[i] = std::thread(work);
    } catch (...) {
      break;          // as many as there are
    }
  }
  work();
  for (std::thread& t : pool)
    if (t.joinable()) t.join();
  return ok;
}

void build(const dd_problem_desc& d, const std::vector<int>& own_api, int cus, bool adj, bool rec, ResPlan& plan) {
  Cut cut_fd, cut_fe;
  if (!choose(d, cus, adj, rec, cut_fd, cut_fe)) return;
  const Cut *fd = &cut_fd, *fe = &cut_fe;
  const int nx = d.n_outer[0], ny = d.n_outer[1], nz = d.n_outer[2];
  const int64_t N = (int64_t)nx * ny * nz;
  // ---- bricks and ownership
  struct Brick { int lo[3], dim[3]; bool fem; };
  std::vector<Brick> br;
  std::vector<int> fd_of((size_t)fd->num[0] * fd->num[1] * fd->num[2], -1);
  for (int k = 0; k < fd->num[2]; ++k)
    for (int j = 0; j < fd->num[1]; ++j)
      for (int i = 0; i < fd->num[0]; ++i) {
        Brick b;
        const int at[3] = {i, j, k};
        int hi[3];
        for (int a = 0; a < 3; ++a) {
          b.lo[a] = at[a] * fd->dim[a];
          b.dim[a] = std::min(fd->dim[a], d.n_outer[a] - b.lo[a]);
          hi[a] = b.lo[a] + b.dim[a];
        }
        b.fem = false;
        if (inside(d, b.lo, hi)) continue;
        fd_of[i + (size_t)fd->num[0] * (j + (size_t)fd->num[1] * k)] = (int)br.size();
        br.push_back(b);
      }
  const int n_fd = (int)br.size();
  for (int k = 0; k < fe->num[2]; ++k)
    for (int j = 0; j < fe->num[1]; ++j)
      for (int i = 0; i < fe->num[0]; ++i) {
        Brick b;
        const int at[3] = {i, j, k};
        for (int a = 0; a < 3; ++a) {
          b.lo[a] = 1 + at[a] * fe->dim[a];            // lattice index
          b.dim[a] = std::min(fe->dim[a], d.fem_cells[a] - b.lo[a]);
        }
        b.fem = true;
        br.push_back(b);
      }
  const int n_br = (int)br.size();
  const int* lo = d.fem_lo;
  auto fem_owned = [&](int x, int y, int z) {
    return x > lo[0] && x < lo[0] + d.fem_cells[0] && y > lo[1] && y < lo[1] + d.fem_cells[1] && z > lo[2] &&
           z < lo[2] + d.fem_cells[2];
  };
  // the bricks of a coordinate along each axis
  std::vector<int> fd_at[3], fe_at[3];
  for (int a = 0, step_fd = 1, step_fe = 1; a < 3; ++a) {
    for (int x = 0; x < d.n_outer[a]; ++x) {
      fd_at[a].push_back(step_fd * (x / fd->dim[a]));
      fe_at[a].push_back(step_fe * std::max(0, (x - lo[a] - 1) / fe->dim[a]));
    }
    step_fd *= fd->num[a];
    step_fe *= fe->num[a];
  }
  auto owner = [&](int x, int y, int z) {
    if (fem_owned(x, y, z)) return n_fd + fe_at[0][x] + fe_at[1][y] + fe_at[2][z];
    return fd_of[fd_at[0][x] + fd_at[1][y] + fd_at[2][z]];
  };
  auto grid = [&](int x, int y, int z) { return (int)(x + (int64_t)nx * (y + (int64_t)ny * z)); };
  // ---- collected nodes per brick
  struct Need { int node, cell, owner, src; };
  std::vector<std::vector<Need>> need(n_br);
  std::vector<int> con_fem(n_br, 0);
  std::vector<int> own_of((size_t)m_fx(d) * m_fy(d) * (d.fem_cells[2] + 1), -1);
  for (size_t i = 0; i < own_api.size(); ++i) own_of[own_api[i]] = (int)i;
  const auto needs = [&](int b) {
    const Brick& q = br[b];
    std::vector<Need>& list = need[b];
    list.reserve(2 * (q.dim[0] * q.dim[1] + q.dim[1] * q.dim[2] + q.dim[2] * q.dim[0]));
    if (!q.fem) {
      // own: node updated by this brick
      auto own = [&](int x, int y, int z) {
        return x >= q.lo[0] && x < q.lo[0] + q.dim[0] && y >= q.lo[1] && y < q.lo[1] + q.dim[1] && z >= q.lo[2] &&
               z < q.lo[2] + q.dim[2] && !fem_owned(x, y, z);
      };
      auto add = [&](int x, int y, int z) {
        list.push_back({grid(x, y, z), fd_cell(x - q.lo[0], y - q.lo[1], z - q.lo[2], q.dim[1]), owner(x, y, z), 0});
      };
      const int n[3] = {nx, ny, nz};
      for (int a = 0; a < 3; ++a)
        for (int side = 0; side < 2; ++side) {
          int p[3];
          p[a] = side ? q.lo[a] + q.dim[a] : q.lo[a] - 1;
          if (p[a] < 0 || p[a] >= n[a]) continue;
          const int u = (a + 1) % 3 < (a + 2) % 3 ? (a + 1) % 3 : (a + 2) % 3, v = 3 - a - u;
          for (int j = 0; j < q.dim[v]; ++j)
            for (int i = 0; i < q.dim[u]; ++i) {
              p[u] = q.lo[u] + i;
              p[v] = q.lo[v] + j;
              int w[3] = {p[0], p[1], p[2]};
              w[a] += side ? -1 : 1;
              if (own(w[0], w[1], w[2])) add(p[0], p[1], p[2]);
            }
        }
      // FEM-owned nodes of lattice layer 1 within the brick, next to a node it updates
      int ib[3], ie[3];
      bool any = true;
      for (int a = 0; a < 3; ++a) {
        ib[a] = std::max(q.lo[a], lo[a] + 1);
        ie[a] = std::min(q.lo[a] + q.dim[a], lo[a] + d.fem_cells[a]);
        any = any && ib[a] < ie[a];
      }
      if (any)
        for (int z = ib[2]; z < ie[2]; ++z)
          for (int y = ib[1]; y < ie[1]; ++y) {
            const bool row = z == lo[2] + 1 || z == lo[2] + d.fem_cells[2] - 1 || y == lo[1] + 1 ||
                             y == lo[1] + d.fem_cells[1] - 1;
            for (int x = ib[0]; x < ie[0]; ++x) {
              if (!row && x != lo[0] + 1 && x != lo[0] + d.fem_cells[0] - 1) continue;
              if (own(x - 1, y, z) || own(x + 1, y, z) || own(x, y - 1, z) || own(x, y + 1, z) || own(x, y, z - 1) ||
                  own(x, y, z + 1))
                add(x, y, z);
            }
          }
      return (int)list.size() <= RES_XCH * RES_THREADS;
    } else {
      const int sx = q.dim[0] + 2, sy = q.dim[1] + 2;
      std::vector<Need> l0;
      // rim nodes that the star of one of the brick's nodes reads
      const auto used = [&](int x, int y, int z) {
        for (const StarSlot& s : kStar) {
          const int u = x - s.x, v = y - s.y, w = z - s.z;
          if (u >= 0 && u < q.dim[0] && v >= 0 && v < q.dim[1] && w >= 0 && w < q.dim[2]) return true;
        }
        return false;
      };
      const auto add = [&](int x, int y, int z) {
        if (!used(x, y, z)) return;
        const int lx = q.lo[0] + x, ly = q.lo[1] + y, lz = q.lo[2] + z;
        const int gx = lo[0] + lx, gy = lo[1] + ly, gz = lo[2] + lz;
        int src = own_of[lx + (int64_t)m_fx(d) * (ly + (int64_t)m_fy(d) * lz)];
        const bool fem = src >= 0;
        if (!fem) src = -1 - (int)face_lex_index(lx, ly, lz, d.fem_cells[0] + 1, d.fem_cells[1] + 1, d.fem_cells[2] + 1, 63u);
        (fem ? list : l0).push_back({grid(gx, gy, gz), (x + 1) + sx * ((y + 1) + sy * (z + 1)), owner(gx, gy, gz), src});
      };
      for (int z = -1; z <= q.dim[2]; ++z)
        for (int y = -1; y <= q.dim[1]; ++y) {
          const bool row = z < 0 || z == q.dim[2] || y < 0 || y == q.dim[1];
          for (int x = -1; x <= q.dim[0]; x += row ? 1 : q.dim[0] + 1) add(x, y, z);
        }
      con_fem[b] = (int)list.size();
      list.insert(list.end(), l0.begin(), l0.end());
      return 3 * (int)list.size() <= RES_XCH * RES_THREADS;
    }
  };
  if (!each_brick(n_br, needs)) return;
  // ---- published nodes: grouped by their owner, in grid order
  std::vector<int> word((size_t)N, -1);
  std::vector<std::vector<int>> pub(n_br);
  std::vector<std::vector<int>> from(n_br);     // bricks a brick collects from
  for (int b = 0; b < n_br; ++b) {
    std::vector<int>& f = from[b];
    for (const Need& e : need[b]) {
      if (f.empty() || f.back() != e.owner) f.push_back(e.owner);
      word[e.node] = e.owner;
    }
    std::sort(f.begin(), f.end());
    f.erase(std::unique(f.begin(), f.end()), f.end());
  }
  for (int64_t i = 0; i < N; ++i)
    if (word[i] >= 0) pub[word[i]].push_back((int)i);
  // A brick that another collects from has to collect from it too, so that it never runs further ahead
  // than the ring is deep.  Finite-element bricks read layer-0 nodes at the box's edges whose own
  // bricks read no FEM node: those bricks collect one word of the reader into the sink.
  auto collects = [&](int b, int o) { return std::binary_search(from[b].begin(), from[b].end(), o); };
  for (int b = 0; b < n_br; ++b)
    for (int o : from[b]) {
      if (collects(o, b)) continue;
      if (br[o].fem || pub[b].empty()) return;
      need[o].push_back({pub[b][0], RES_SINK, b, 0});
      from[o].insert(std::upper_bound(from[o].begin(), from[o].end(), b), b);
      if ((int)need[o].size() > RES_XCH * RES_THREADS) return;
    }
  int n_pub = 0;
  std::vector<int> pub_off(n_br);
  for (int b = 0; b < n_br; ++b) {
    pub_off[b] = n_pub;
    for (int node : pub[b]) word[node] = n_pub++;
    if ((int)pub[b].size() * (br[b].fem ? 3 : 1) > RES_XCH * RES_THREADS) return;
  }
  plan.n_pub = n_pub;
  // ---- lists (the kernel is chosen by the longest run)
  int longest = 0;
  for (int b = 0; b < n_fd; ++b) longest = std::max(longest, run_of(br[b].dim[0], br[b].dim[1], br[b].dim[2]));
  const int special_max = res_special(longest) * RES_THREADS;
  std::vector<ResBlock> bricks(n_br);
  std::vector<std::vector<uint32_t>> sp_meta(n_br), out_cell(n_br);
  std::vector<std::vector<int>> sp_det(n_br), out_idx(n_br);
  int n_con = 0, n_node = 0;
  for (int b = 0; b < n_br; ++b) {
    const Brick& q = br[b];
    ResBlock& r = bricks[b];
    r.fem = q.fem;
    for (int a = 0; a < 3; ++a) { r.lo[a] = q.lo[a]; r.dim[a] = q.dim[a]; }
    r.pub_off = pub_off[b];
    r.pub_n = (int)pub[b].size();
    r.con_off = n_con;
    r.con_n = (int)need[b].size();
    r.con_fem = con_fem[b];
    r.node_off = n_node;
    n_con += r.con_n;
    if (q.fem) n_node += q.dim[0] * q.dim[1] * q.dim[2];
  }
  plan.con_word.resize(n_con);
  plan.con_step.resize(n_con);
  plan.con_cell.resize(n_con);
  plan.con_src.resize(n_con);
  plan.pub_cell.resize(n_pub);
  plan.fem_node.resize(n_node);
  const auto lists = [&](int b) {
    const Brick& q = br[b];
    ResBlock& r = bricks[b];
    const int sx = q.dim[0] + 2, sy = q.dim[1] + 2;
    for (int i = 0; i < r.con_n; ++i) {
      const Need& e = need[b][i];
      const int o = e.owner, k = r.con_off + i;
      plan.con_word[k] = (uint32_t)(3 * pub_off[o] + (word[e.node] - pub_off[o]));
      plan.con_step[k] = (uint16_t)pub[o].size();
      plan.con_cell[k] = (uint16_t)e.cell;
      plan.con_src[k] = e.src;
    }
    uint16_t* cell = plan.pub_cell.data() + r.pub_off;
    for (int node : pub[b]) {
      int p[3] = {node % nx, (node / nx) % ny, (int)(node / ((int64_t)nx * ny))};
      if (q.fem) {
        for (int a = 0; a < 3; ++a) p[a] -= lo[a] + q.lo[a];
        *cell++ = (uint16_t)((p[0] + 1) + sx * ((p[1] + 1) + sy * (p[2] + 1)));
      } else {
        *cell++ = (uint16_t)fd_cell(p[0] - q.lo[0], p[1] - q.lo[1], p[2] - q.lo[2], q.dim[1]);
      }
    }
    if (q.fem) {
      int2* node = plan.fem_node.data() + r.node_off;
      for (int z = 0; z < q.dim[2]; ++z)
        for (int y = 0; y < q.dim[1]; ++y)
          for (int x = 0; x < q.dim[0]; ++x)
            *node++ = make_int2(own_of[(q.lo[0] + x) + (int64_t)m_fx(d) * ((q.lo[1] + y) + (int64_t)m_fy(d) * (q.lo[2] + z))],
                                (x + 1) + sx * ((y + 1) + sy * (z + 1)));
      return true;
    }
    r.run = run_of(q.dim[0], q.dim[1], q.dim[2]);
    // Nodes of the brick with something of their own: outputs (detectors, layer 0), and the special nodes:
    // those on absorbing side faces, and in an adjoint the detectors below the top plane
    const unsigned sides = d.absorbing_faces & (DD_FACE_XMIN | DD_FACE_XMAX | DD_FACE_YMIN | DD_FACE_YMAX);
    auto visit = [&](int x, int y, int z) {
      const int cell = fd_cell(x - q.lo[0], y - q.lo[1], z - q.lo[2], q.dim[1]);
      const uint32_t f = (x == 0 ? RES_XL : 0) | (x == nx - 1 ? RES_XH : 0) | (y == 0 ? RES_YL : 0) |
                         (y == ny - 1 ? RES_YH : 0) | (z == 0 ? RES_ZL : 0) | (z == nz - 1 ? RES_ZH : 0);
      if (f) {
        const int det = (int)face_lex_index(x, y, z, nx, ny, nz, d.detector_faces);
        if (det >= 0 && !adj) {
          out_cell[b].push_back((uint32_t)cell);
          out_idx[b].push_back(det);
        }
        const bool damped = ((sides & DD_FACE_XMIN) && x == 0) || ((sides & DD_FACE_XMAX) && x == nx - 1) ||
                            ((sides & DD_FACE_YMIN) && y == 0) || ((sides & DD_FACE_YMAX) && y == ny - 1);
        if (damped || (adj && det >= 0 && z != nz - 1)) {
          sp_meta[b].push_back((uint32_t)cell | f << 16);
          sp_det[b].push_back(det);
        }
      }
      if (!adj && x >= lo[0] && x <= lo[0] + d.fem_cells[0] && y >= lo[1] && y <= lo[1] + d.fem_cells[1] && z >= lo[2] &&
          z <= lo[2] + d.fem_cells[2] && !fem_owned(x, y, z)) {
        out_cell[b].push_back((uint32_t)cell | 1u << 16);
        out_idx[b].push_back((int)face_lex_index(x - lo[0], y - lo[1], z - lo[2], d.fem_cells[0] + 1,
                                                   d.fem_cells[1] + 1, d.fem_cells[2] + 1, 63u));
      }
    };
    for (int z = q.lo[2]; z < q.lo[2] + q.dim[2]; ++z)
      for (int y = q.lo[1]; y < q.lo[1] + q.dim[1]; ++y) {
        // whole rows on a face of the grid or the box, else the ends of the grid's and the box's rows
        const bool in_yz = z >= lo[2] && z <= lo[2] + d.fem_cells[2] && y >= lo[1] && y <= lo[1] + d.fem_cells[1];
        const bool row = z == 0 || z == nz - 1 || y == 0 || y == ny - 1 ||
                         (in_yz && (z == lo[2] || z == lo[2] + d.fem_cells[2] || y == lo[1] || y == lo[1] + d.fem_cells[1]));
        const int xe = q.lo[0] + q.dim[0];
        if (row) {
          for (int x = q.lo[0]; x < xe; ++x) visit(x, y, z);
          continue;
        }
        const int ends[4] = {0, lo[0], lo[0] + d.fem_cells[0], nx - 1};
        for (int e = 0; e < 4; ++e)
          if (ends[e] >= q.lo[0] && ends[e] < xe && (in_yz || e == 0 || e == 3)) visit(ends[e], y, z);
      }
    return (int)sp_meta[b].size() <= special_max;
  };
  if (!each_brick(n_br, lists)) return;
  for (int b = 0; b < n_br; ++b) {
    const Brick& q = br[b];
    ResBlock& r = bricks[b];
    if (q.fem) {
      plan.max_fem = std::max(plan.max_fem, q.dim[0] * q.dim[1] * q.dim[2]);
      plan.fem_lds = std::max(plan.fem_lds, fem_bytes(q.dim[0], q.dim[1], q.dim[2], rec));
      plan.blocks.push_back(r);
      continue;
    }
    const auto join = [](auto& to, const auto& from, int& off, int& n) {
      off = (int)to.size();
      n = (int)from.size();
      to.insert(to.end(), from.begin(), from.end());
    };
    join(plan.sp_meta, sp_meta[b], r.sp_off, r.sp_n);
    join(plan.sp_det, sp_det[b], r.sp_off, r.sp_n);
    join(plan.out_cell, out_cell[b], r.out_off, r.out_n);
    join(plan.out_idx, out_idx[b], r.out_off, r.out_n);
    plan.max_run = std::max(plan.max_run, r.run);
    plan.fd_cells = std::max(plan.fd_cells, (int)fd_floats(q.dim[1], q.dim[2]));
    for (int c = 0; c < 3; ++c) {
      r.comp = c;
      plan.blocks.push_back(r);
    }
  }
  plan.adj = adj;
  plan.rec = rec;
  if (plan.max_run > RES_RUN_MAX || plan.lds() > RES_LDS_MAX) plan.blocks.clear();
}

}  // namespace

void build_resident(const dd_problem_desc& d, const std::vector<int>& own_api, int cus, bool adj, bool rec,
                    ResPlan& plan) noexcept {
  try {
    plan = ResPlan();
    build(d, own_api, cus, adj, rec, plan);
  } catch (...) {
    plan.blocks.clear();        // no memory for the lists: the solve runs by launches
  }
}

bool resident_fits(const dd_problem_desc& d, int cus) {
  Cut fd, fe;
  return choose(d, cus, false, false, fd, fe);
}

size_t resident_bytes_bound(const dd_problem_desc& d, int cus, bool adj, bool rec) {
  Cut fd, fe;
  if (!choose(d, cus, adj, rec, fd, fe)) return 0;
  const int64_t n[3] = {d.n_outer[0], d.n_outer[1], d.n_outer[2]};
  const int64_t f[3] = {d.fem_cells[0] - 1, d.fem_cells[1] - 1, d.fem_cells[2] - 1};   // owned nodes
  // nodes on either side of the planes between bricks
  const auto between = [](const int64_t* n, const Cut& c) {
    return 2 * ((c.num[0] - 1) * n[1] * n[2] + (c.num[1] - 1) * n[0] * n[2] + (c.num[2] - 1) * n[0] * n[1]);
  };
  const int64_t own = f[0] * f[1] * f[2];
  const int64_t layer1 = own - std::max<int64_t>(f[0] - 2, 0) * std::max<int64_t>(f[1] - 2, 0) * std::max<int64_t>(f[2] - 2, 0);
  const int64_t layer0 = face_lex_count(d.fem_cells[0] + 1, d.fem_cells[1] + 1, d.fem_cells[2] + 1, 63u);
  const int64_t bricks = fd.blocks / 3;
  // published: beside the cuts, and between the two regions
  const int64_t pub = between(n, fd) + layer0 + between(f, fe) + layer1;
  // collected: beside the cuts (and by a brick of a node of its own that a finite-element brick updates), the boxes'
  // rims, and a word for its order by a brick from a finite-element brick that reads it
  const int64_t con = between(n, fd) + layer1 + fe.blocks * ((int64_t)(fe.dim[0] + 2) * (fe.dim[1] + 2) * (fe.dim[2] + 2) -
                                                             (int64_t)fe.dim[0] * fe.dim[1] * fe.dim[2]) +
                      (int64_t)bricks * fe.blocks;
  const unsigned sides = DD_FACE_XMIN | DD_FACE_XMAX | DD_FACE_YMIN | DD_FACE_YMAX;
  const unsigned special = (d.absorbing_faces & sides) | (adj ? d.detector_faces : 0u);
  const int64_t sp = face_lex_count(d.n_outer[0], d.n_outer[1], d.n_outer[2], special);
  const int64_t out = adj ? 0 : face_lex_count(d.n_outer[0], d.n_outer[1], d.n_outer[2], d.detector_faces) + layer0;
  int64_t b = (int64_t)sizeof(ResBlock) * (fd.blocks + fe.blocks) + 8 * (sp + out + own) + 2 * pub + 12 * con;
  b += (int64_t)8 * 3 * RES_RING * pub * (rec ? 2 : 1) + 1024;     // and the lists' alignment, the control block
  return (size_t)b;
}

}  // namespace dd
