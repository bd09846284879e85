// Resident solves (resident.hpp): one launch takes every time step of a source.
//
// A step costs compute, publish and collect with a barrier between them: the exchange's round trip through the
// memory side (1.15 us for a few words per block, 1.5 us for three per thread) plus the longest brick's
// compute, bound by vector and LDS instructions of one block per CU.  By launches a step costs the launch and its drain,
// 5 us and more.  us per step, forward / adjoint, by launches -> resident: 25^3 5.5 / 5.9 -> 2.7 / 4.0; with checkpoints
// recomputed 37x35x41 5.0 / 8.4 -> 2.9 / 5.7, 64^3 6.5 / 7.7 -> 4.0 / 6.2, 96^3 (FEM 48^3) 10.5 / 13.1 -> 7.2 / 10.3.
#include "resident.hpp"

#include <algorithm>

#include "kuhn_star.hpp"
#include "oblique.hpp"

namespace dd {
namespace {

typedef unsigned long long u64;

// Uniform data read with scalar loads.
typedef const __attribute__((address_space(4))) double* cdouble;

// ---- exchange -----------------------------------------------------------------------------------
__device__ __forceinline__ void put_word(u64* p, unsigned tag, float v) {
  __hip_atomic_store(p, (u64)tag << 32 | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get_word(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int load_state(const ResCtl* c) {
  return __hip_atomic_load(&c->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One outcome for all blocks: the first transition out of `from` holds.
__device__ __forceinline__ void decide(ResCtl* c, int from, int to) {
  int e = from;
  __hip_atomic_compare_exchange_strong(&c->state, &e, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
}

// The words a thread publishes and collects each step; the lists do not change during a solve,
// so they stay in registers.  A brick's published words follow each other (component by
// component), so only their LDS places are kept.
struct Exchange {
  uint32_t pub[RES_XCH / 2], cell[RES_XCH / 2];   // LDS float indices, two per register
  uint32_t con_w[RES_XCH];                        // byte offsets of the words, NO_WORD: none
  int first, n, n_con;                            // first published word; numbers of words
};
constexpr uint32_t NO_WORD = 0xFFFFFFFFu;

template <bool FEM>
__device__ __forceinline__ void exchange_lists(const ResArgs& a, const ResBlock& b, int con_n, Exchange& x) {
  const int t = threadIdx.x;
  x.first = 3 * b.pub_off + (FEM ? 0 : b.comp * b.pub_n);
  x.n = (FEM ? 3 : 1) * b.pub_n;
  x.n_con = (FEM ? 3 : 1) * con_n;
#pragma unroll
  for (int i = 0; i < RES_XCH; ++i) {
    const int e = t + i * RES_THREADS;
    // FEM: entry e is component e / n of node e % n
    uint32_t cell = 0;
    if (e < x.n) {
      const int c = FEM ? e / b.pub_n : 0, k = FEM ? e % b.pub_n : e;
      cell = a.pub_cell[b.pub_off + k];
      if (FEM) cell = 4 * cell + c;
    }
    x.pub[i / 2] = i % 2 ? x.pub[i / 2] | cell << 16 : cell;
    cell = 0;
    x.con_w[i] = NO_WORD;
    if (e < x.n_con) {
      const int c = FEM ? e / con_n : b.comp, k = b.con_off + (FEM ? e % con_n : e);
      x.con_w[i] = 8u * (a.con_word[k] + (uint32_t)c * a.con_step[k]);
      cell = a.con_cell[k];
      if (FEM) cell = 4 * cell + c;
    }
    x.cell[i / 2] = i % 2 ? x.cell[i / 2] | cell << 16 : cell;
  }
}
template <int N>
__device__ __forceinline__ uint32_t half_of(const uint32_t (&v)[N], int i) {
  const uint32_t w = fresh(v[i / 2]);
  return i % 2 ? w >> 16 : w & 0xFFFFu;
}

__device__ __forceinline__ void publish(u64* buf, const Exchange& x, unsigned tag, const float* L) {
  char* w = reinterpret_cast<char*>(buf + x.first);
  float v[RES_XCH];
#pragma unroll
  for (int i = 0; i < RES_XCH; ++i) {    // all reads, then all stores
    if (i * RES_THREADS >= x.n) break;
    v[i] = L[half_of(x.pub, i)];
    here(v[i]);
  }
#pragma unroll
  for (int i = 0; i < RES_XCH; ++i) {
    if (i * RES_THREADS >= x.n) break;
    const int e = fresh((int)threadIdx.x) + i * RES_THREADS;
    if (e < x.n) put_word(reinterpret_cast<u64*>(w + 8u * (uint32_t)e), tag, v[i]);
  }
}

// Collects the words of `tag` into LDS (and those of a second list); false when the solve has been given up.
__device__ __forceinline__ unsigned awaited(const Exchange& x) {
  unsigned todo = 0;
#pragma unroll
  for (int i = 0; i < RES_XCH; ++i) {
    if (i * RES_THREADS >= x.n_con) break;
    if (fresh((int)threadIdx.x) + i * RES_THREADS < x.n_con) todo |= 1u << i;
  }
  return todo;
}
__device__ __forceinline__ void ask(const u64* buf, const Exchange& x, unsigned todo, u64 (&w)[RES_XCH]) {
#pragma unroll
  for (int i = 0; i < RES_XCH; ++i) {
    if (i * RES_THREADS >= x.n_con) break;
    if (todo & 1u << i)
      w[i] = get_word(reinterpret_cast<const u64*>(reinterpret_cast<const char*>(buf) + fresh(x.con_w[i])));
  }
}
__device__ __forceinline__ void take(const Exchange& x, unsigned tag, unsigned& todo, const u64 (&w)[RES_XCH], float* L) {
#pragma unroll
  for (int i = 0; i < RES_XCH; ++i) {
    if (i * RES_THREADS >= x.n_con) break;
    if ((todo & 1u << i) && (unsigned)(w[i] >> 32) == tag) {
      L[half_of(x.cell, i)] = __uint_as_float((unsigned)w[i]);
      todo &= ~(1u << i);
    }
  }
}
__device__ __forceinline__ bool waiting(unsigned spin, ResCtl* ctl, long long limit) {
  if (spin & 255u) return true;
  if (wall_clock64() > limit) decide(ctl, RES_GO, RES_FAILED);
  return load_state(ctl) == RES_GO;
}
// meanwhile: work done while the first words are on their way.
template <class F>
__device__ __forceinline__ bool collect(const u64* buf, const Exchange& x, unsigned tag, float* L, ResCtl* ctl, long long limit,
                                        F&& meanwhile) {
  unsigned todo = awaited(x);
  u64 w[RES_XCH];
  ask(buf, x, todo, w);
  meanwhile();
  take(x, tag, todo, w, L);
  for (unsigned spin = 1; todo; ++spin) {
    if (!waiting(spin, ctl, limit)) return false;
    ask(buf, x, todo, w);
    take(x, tag, todo, w, L);
  }
  return true;
}
__device__ __forceinline__ bool collect(const u64* buf, const Exchange& x, unsigned tag, float* L, const u64* buf2,
                                        const Exchange& x2, unsigned tag2, float* L2, ResCtl* ctl, long long limit) {
  unsigned todo = awaited(x), todo2 = awaited(x2);
  for (unsigned spin = 1; todo | todo2; ++spin) {
    u64 w[RES_XCH], w2[RES_XCH];
    ask(buf, x, todo, w);
    ask(buf2, x2, todo2, w2);
    take(x, tag, todo, w, L);
    take(x2, tag2, todo2, w2, L2);
    if ((todo | todo2) && !waiting(spin, ctl, limit)) return false;
  }
  return true;
}

// All blocks are on the GPU (or none of them goes on).
__device__ __forceinline__ bool assemble(const ResArgs& a) {
  __shared__ int go;
  if (threadIdx.x == 0) {
    const long long limit = wall_clock64() + a.wait_ticks;
    const int before = __hip_atomic_fetch_add(&a.ctl->arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before + 1 == a.need) decide(a.ctl, RES_WAIT, RES_GO);
    int s;
    while ((s = load_state(a.ctl)) == RES_WAIT) {
      if (wall_clock64() > limit) decide(a.ctl, RES_WAIT, RES_OFF);
      __builtin_amdgcn_s_sleep(1);
    }
    go = s == RES_GO;
  }
  __syncthreads();
  return go;
}

// Every block has taken its last step: only then results that add to earlier ones are written.
__device__ __forceinline__ bool finish(const ResArgs& a, long long limit) {
  __shared__ int done;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int before = __hip_atomic_fetch_add(&a.ctl->end, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before + 1 == a.n_blocks) decide(a.ctl, RES_GO, RES_DONE);
    int s;
    while ((s = load_state(a.ctl)) == RES_GO) {
      if (wall_clock64() > limit) decide(a.ctl, RES_GO, RES_FAILED);
      __builtin_amdgcn_s_sleep(1);
    }
    done = s == RES_DONE;
  }
  __syncthreads();
  return done;
}

// Outer faces of the grid: their rim cells hold the face's own values.  A thread's copies of a step, {from, to} LDS
// floats, two per register: single values along the x faces, four at a time along the others.
constexpr int RIM1 = 4, RIM4 = 2;
struct Rims {
  uint32_t one[RIM1], four[RIM4];     // 0: none
};
__device__ __forceinline__ void rim_lists(const ResBlock& b, uint32_t faces, Rims& m) {
  const int bx = b.dim[0], by = b.dim[1], bz = b.dim[2], nxq = (bx + 3) / 4, SZ = RES_SY * (by + 2);
  const int nl = faces & RES_XL ? by * bz : 0, nr = faces & RES_XH ? by * bz : 0;
#pragma unroll
  for (int i = 0; i < RIM1; ++i) {
    int e = threadIdx.x + i * RES_THREADS;
    m.one[i] = 0;
    if (e < nl + nr) {
      const bool left = e < nl;
      e -= left ? 0 : nl;
      const int row = 4 + RES_SY * (e % by + 1) + SZ * (e / by + 1), from = left ? row : row + bx - 1;
      m.one[i] = from | (uint32_t)(left ? from - 1 : from + 1) << 16;
    }
  }
  const int n[4] = {faces & RES_YL ? nxq * bz : 0, faces & RES_YH ? nxq * bz : 0, faces & RES_ZL ? nxq * by : 0,
                    faces & RES_ZH ? nxq * by : 0};
#pragma unroll
  for (int i = 0; i < RIM4; ++i) {
    int e = threadIdx.x + i * RES_THREADS, side = 0;
    m.four[i] = 0;
    while (side < 4 && e >= n[side]) e -= n[side++];
    if (side < 4) {
      const int u = e / nxq, x = 4 + 4 * (e % nxq);
      const int from = side == 0 ? x + RES_SY + SZ * (u + 1) : side == 1 ? x + RES_SY * by + SZ * (u + 1)
                       : side == 2 ? x + RES_SY * (u + 1) + SZ : x + RES_SY * (u + 1) + SZ * bz;
      const int to = side == 0 ? from - RES_SY : side == 1 ? from + RES_SY : side == 2 ? from - SZ : from + SZ;
      m.four[i] = from | (uint32_t)to << 16;
    }
  }
}
__device__ __forceinline__ void copy_rims(const Rims& m, float* L) {
#pragma unroll
  for (int i = 0; i < RIM1; ++i) {
    const uint32_t w = fresh(m.one[i]);
    if (w) L[w >> 16] = L[w & 0xFFFFu];
  }
#pragma unroll
  for (int i = 0; i < RIM4; ++i) {
    const uint32_t w = fresh(m.four[i]);
    if (w) *reinterpret_cast<float4*>(L + (w >> 16)) = *reinterpret_cast<const float4*>(L + (w & 0xFFFFu));
  }
}

// ---- finite-difference bricks ---------------------------------------------------------------------
// One component of a brick.  A thread takes four nodes along x and a run of planes: rows are 16-byte LDS
// accesses, neighbours along z stay in registers, and a difference between two nodes serves both of them.  P
// holds the previous level.  Outer faces cost nothing but weights: a face's rim cells hold a copy of the face's own
// nodes (a difference of 0), and the difference to the inner neighbour counts twice.  The rows of the top and
// the bottom plane add damping, forcing and the cotangent.  Nodes on absorbing side faces, detectors below
// the top plane (adjoint) and the dipole are advanced once more, one by one, as `special` nodes, whose values replace
// the rows'.  The arithmetic is that of the step kernels' tiles (explicit fused multiply-adds, no other
// contraction; an exact difference, its negative and a factor of 1 change nothing), so both paths round alike.
template <int RUN, bool ADJ>
__device__ __forceinline__ void fd_brick(const ResArgs& a, const ResBlock& b, float* L, long long limit) {
#pragma clang fp contract(off)
  __shared__ int given_up;
  const int t = threadIdx.x, comp = b.comp, nt = a.nt;
  const int SZ = RES_SY * (b.dim[1] + 2);
  // ---- this thread's nodes
  const ResRows rows = res_rows(b.dim, b.run, t);
  const int xq = rows.xq, ty = rows.ty, z_beg = rows.z, run_ = rows.run;
  const uint32_t base = rows.base;
  const int gx = b.lo[0] + 4 * xq, gy = b.lo[1] + ty;                    // grid coordinates of its first node
  float wx[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) wx[e] = gx + e == 0 || gx + e == a.nx - 1 ? 2.f : 1.f;
  const float wy = gy == 0 || gy == a.ny - 1 ? 2.f : 1.f;
  // its run holds the grid's bottom (plane 0) or top plane (b.run - 1)
  const int ends = (b.lo[2] == 0 && z_beg == 0 ? 1 : 0) | (b.lo[2] + z_beg + run_ == a.nz && run_ > 0 ? 2 : 0);
  const int x_last = a.nx - 1 - gx;                                      // the grid's last node among the four
  float4 P[RUN];
#pragma unroll
  for (int k = 0; k < RUN; ++k) P[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  // ---- special nodes; the last one is the dipole's where this brick holds it
  constexpr int NSP = res_special(RUN);
  uint32_t meta[NSP + 1];
  int det[NSP + 1];
  float Q[NSP + 1], r[NSP + 1];
#pragma unroll
  for (int j = 0; j <= NSP; ++j) {
    const int e = j * RES_THREADS + t;
    meta[j] = 0;
    det[j] = -1;
    Q[j] = r[j] = 0.f;
    if (j < NSP && e < b.sp_n) {
      meta[j] = a.sp_meta[b.sp_off + e];
      det[j] = a.sp_det[b.sp_off + e];
    }
  }
  int n_sp = (b.sp_n + RES_THREADS - 1) / RES_THREADS;
  bool special = n_sp > 0;
  if (!ADJ && a.dip_idx >= 0) {
    const int x = (int)(a.dip_idx % a.nx), y = (int)((a.dip_idx / a.nx) % a.ny), z = (int)(a.dip_idx / ((int64_t)a.nx * a.ny));
    const int u = x - b.lo[0], v = y - b.lo[1], w = z - b.lo[2];
    if (u >= 0 && u < b.dim[0] && v >= 0 && v < b.dim[1] && w >= 0 && w < b.dim[2]) {
      special = true;
      const uint32_t cell = 4 + u + RES_SY * (v + 1) + SZ * (w + 1);
      const uint32_t f = (x == 0 ? RES_XL : 0) | (x == a.nx - 1 ? RES_XH : 0) | (y == 0 ? RES_YL : 0) |
                         (y == a.ny - 1 ? RES_YH : 0) | (z == 0 ? RES_ZL : 0) | (z == a.nz - 1 ? RES_ZH : 0) | RES_DIP;
#pragma unroll
      for (int j = 0; j < NSP; ++j)
        if ((meta[j] & 0xFFFFu) == cell) meta[j] = 0;      // on an absorbing side: once, with the force
      if (t == 0) meta[NSP] = cell | f << 16;
    }
  }
  // ---- trace and interface outputs
  constexpr int NO = RUN <= 8 ? RES_OUT : 1;
  uint32_t out_c[NO];
  int out_i[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int e = i * RES_THREADS + t;
    out_i[i] = -1;
    out_c[i] = 0;
    if (!ADJ && e < b.out_n) {
      out_c[i] = a.out_cell[b.out_off + e];
      out_i[i] = a.out_idx[b.out_off + e];
    }
  }
  Exchange xc;
  exchange_lists<false>(a, b, b.con_n, xc);
  for (int i = t; i < SZ * (b.dim[2] + 2); i += RES_THREADS) L[i] = 0.f;
  if (t == 0) given_up = 0;
  const unsigned tag0 = a.ctl->epoch[ADJ];
  if (!ADJ && a.ihist)   // layer-0 values of level 0
    for (int e = t; e < b.out_n; e += RES_THREADS)
      if (a.out_cell[b.out_off + e] >> 16) a.ihist[comp * a.n_l0 + a.out_idx[b.out_off + e]] = 0.f;
  // adjoint: the cotangent of a step is loaded one step ahead
  float rt[4] = {0.f, 0.f, 0.f, 0.f};
  const bool top_det = ADJ && (a.det_mask & DD_FACE_TOP) && (ends & 2);
  auto cotangent = [&](int k) {
    const int64_t row = (int64_t)(k - 1) * a.n_det * 3 + comp;
    if (top_det) {
      const int64_t o = row + 3 * (a.top_det + (int64_t)gy * a.nx + gx);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e <= x_last && 4 * xq + e < b.dim[0]) rt[e] = a.obs ? a.cot[o + 3 * e] - a.obs[o + 3 * e] : a.cot[o + 3 * e];
    }
#pragma unroll
    for (int j = 0; j < NSP; ++j)
      if (j < n_sp && det[j] >= 0) {
        const int64_t o = row + (int64_t)det[j] * 3;
        r[j] = a.obs ? a.cot[o] - a.obs[o] : a.cot[o];
      }
  };
  if (ADJ) cotangent(nt);
  const uint32_t fixed = (a.abs_mask & DD_FACE_BOTTOM ? RES_ZL : 0) | (a.abs_mask & DD_FACE_XMIN ? RES_XL : 0) |
                         (a.abs_mask & DD_FACE_XMAX ? RES_XH : 0) | (a.abs_mask & DD_FACE_YMIN ? RES_YL : 0) |
                         (a.abs_mask & DD_FACE_YMAX ? RES_YH : 0);
  const uint32_t grid_faces = (b.lo[0] == 0 ? RES_XL : 0) | (b.lo[0] + b.dim[0] == a.nx ? RES_XH : 0) |
                              (b.lo[1] == 0 ? RES_YL : 0) | (b.lo[1] + b.dim[1] == a.ny ? RES_YH : 0) |
                              (b.lo[2] == 0 ? RES_ZL : 0) | (b.lo[2] + b.dim[2] == a.nz ? RES_ZH : 0);
  Rims rims;
  rim_lists(b, grid_faces, rims);
  const cdouble tab = (cdouble)(uintptr_t)a.tab;
  double pulse = !ADJ && a.n_tab > 0 ? tab[0] : 0.0;
  __syncthreads();

  for (int n = 0; n < nt; ++n) {
    // forward: level n -> n + 1; adjoint: lambda^k -> lambda^{k-1}, k = nt - n
    const int k1 = nt - n;
    const int run = fresh(run_);
    const bool at_top = fresh(ends) & 2, at_bot = fresh(ends) & 1;
    uint32_t abs_a, abs_b;     // faces that absorb at the levels of D+ and D-
    float pw = 0.f, dip = 0.f, pw_t = 0.f;
    int pw_kind = 0;
    if (ADJ) {
      abs_a = fixed | ((a.abs_mask & DD_FACE_TOP) && (double)(k1 - 1) * a.dt > a.t_switch ? RES_ZH : 0);
      abs_b = fixed | ((a.abs_mask & DD_FACE_TOP) && (double)(k1 + 1) * a.dt > a.t_switch ? RES_ZH : 0);
    } else {
      const double time = (double)n * a.dt;
      abs_a = abs_b = fixed | ((a.abs_mask & DD_FACE_TOP) && time > a.t_switch ? RES_ZH : 0);
      if (a.plane && time <= a.t_switch) {
        if (a.oblique) {
          pw_kind = a.kind;
          pw_t = a.kind == DD_SRC_GAUSS_SINE ? (float)(time - a.pw_t0) : (float)time;
        } else {
          pw = (float)(a.pw_scale * pulse * a.pol[comp]);
        }
      }
      dip = (float)(pulse * a.pol[comp] * a.dip_scale);
      pulse = n + 1 < a.n_tab ? tab[n + 1] : 0.0;
    }
    // forcing of a top-face node
    auto top_source = [&](int x, int y) {
      float s = pw;
      if (pw_kind) s += a.pw_amp[comp] * oblique_pulse_at(a, pw_kind, pw_t, x, y);
      return s;
    };
    // out = increment of a node with sum S of weighted differences, previous level p, forcing src, na / nb absorbing faces
    auto update = [&](float v, float p, float S, float src, int na, int nb) {
      if (na == 0 && nb == 0) return v + (__builtin_fmaf(-a.nu2, S, v - p) + src);
      const float ba = a.nu * (float)na, bb = a.nu * (float)nb;
      return v + ((1.f - bb) * (v - p) - a.nu2 * S + src - (ba - bb) * v) / (1.f + ba);
    };
    // ---- special nodes: T becomes their next level, Q the current one
    float T[NSP + 1];
    if (special) {
#pragma unroll
      for (int j = 0; j <= NSP; ++j) {
        if (j < NSP && j >= n_sp) continue;
        const uint32_t mt = fresh(meta[j]), f = mt >> 16;
        if (!mt) continue;
        const float* p = L + (mt & 0xFFFFu);
        const float v = p[0];
        const float sx = (v - p[f & RES_XL ? 0 : -1]) + (v - p[f & RES_XH ? 0 : 1]);
        const float sy = (v - p[f & RES_YL ? 0 : -RES_SY]) + (v - p[f & RES_YH ? 0 : RES_SY]);
        const float sz = (v - p[f & RES_ZL ? 0 : -SZ]) + (v - p[f & RES_ZH ? 0 : SZ]);
        const float fx = f & (RES_XL | RES_XH) ? 2.f : 1.f, fy = f & (RES_YL | RES_YH) ? 2.f : 1.f,
                    fz = f & (RES_ZL | RES_ZH) ? 2.f : 1.f;
        const float S = __builtin_fmaf(fz, sz, __builtin_fmaf(fy, sy, fx * sx));
        float src = 0.f;
        if (!ADJ) {
          if (f & RES_ZH) {
            const int c = (int)(mt & 0xFFFFu);
            src = top_source(c % RES_SY - 4 + b.lo[0], c / RES_SY % (b.dim[1] + 2) - 1 + b.lo[1]);
          }
          if (f & RES_DIP) src += dip;
        } else if (det[j] >= 0) {
          // r dt^2 / m: a lumped mass of h^3 / 2 per outer face
          src -= r[j] * (a.dt2_h3 * (float)(1 << __popc(f & 63u)));
        }
        T[j] = update(v, Q[j], S, src, __popc(f & abs_a), __popc(f & abs_b));
        Q[j] = v;
        here(T[j]);
      }
    }
    // ---- the thread's rows: N becomes the next level, P the current one (long runs: P the next level, the
    // current one comes back from LDS as it is replaced; both would not fit the registers)
    constexpr bool KEEP = RUN <= 8;
    float4 N[RUN], n_top;
    {
      float tv[4], tp[4], tS[4];       // the last plane's operands: on the grid's top it is formed again below
      const float* p = L + fresh(base);
      float4 zc = *reinterpret_cast<const float4*>(p);
      float4 dz = *reinterpret_cast<const float4*>(p - SZ);      // differences to the plane below
      dz = make_float4(zc.x - dz.x, zc.y - dz.y, zc.z - dz.z, zc.w - dz.w);
      float4 ym, yp, zp;
      float xl, xr;
      auto load = [&]() {
        ym = *reinterpret_cast<const float4*>(p - RES_SY);
        yp = *reinterpret_cast<const float4*>(p + RES_SY);
        zp = *reinterpret_cast<const float4*>(p + SZ);
        xl = p[-1];
        xr = p[4];
      };
      load();
#pragma unroll
      for (int k = 0; k < RUN; ++k) {
        // (planes past a shorter run repeat its last one, unused)
        if (k < b.run) {
          const float v[4] = {zc.x, zc.y, zc.z, zc.w};
          const float d[5] = {v[0] - xl, v[1] - v[0], v[2] - v[1], v[3] - v[2], v[3] - xr};
          const float a0[4] = {ym.x, ym.y, ym.z, ym.w}, a1[4] = {yp.x, yp.y, yp.z, yp.w};
          const float4 zu = zp;
          const float up[4] = {zp.x, zp.y, zp.z, zp.w}, dn[4] = {dz.x, dz.y, dz.z, dz.w};
          const float pv[4] = {P[k].x, P[k].y, P[k].z, P[k].w};
          // the next plane's rows, in flight during this one's arithmetic (where registers allow)
          p += k + 1 < run ? SZ : 0;
          if (KEEP && k + 1 < RUN) load();
          float du[4], S[4], nv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float sx = e == 3 ? d[3] + d[4] : d[e] - d[e + 1];
            const float sy = (v[e] - a0[e]) + (v[e] - a1[e]);
            du[e] = v[e] - up[e];
            const float sz = dn[e] + du[e];
            S[e] = __builtin_fmaf(wy, sy, wx[e] * sx);
            if (k == 0) S[e] = __builtin_fmaf(at_bot || (at_top && b.run == 1) ? 2.f : 1.f, sz, S[e]);
            else if (k == b.run - 1) S[e] = __builtin_fmaf(at_top ? 2.f : 1.f, sz, S[e]);
            else S[e] = sz + S[e];
            nv[e] = v[e] + __builtin_fmaf(-a.nu2, S[e], v[e] - pv[e]);
          }
          if (k == 0 && at_bot) {
#pragma unroll
            for (int e = 0; e < 4; ++e) nv[e] = update(v[e], pv[e], S[e], 0.f, (abs_a & RES_ZL) != 0, (abs_b & RES_ZL) != 0);
          }
          if (k == b.run - 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              tv[e] = v[e];
              tp[e] = pv[e];
              tS[e] = S[e];
            }
          }
          N[k] = make_float4(nv[0], nv[1], nv[2], nv[3]);
          here(N[k].x), here(N[k].y), here(N[k].z), here(N[k].w);
          if (KEEP) P[k] = zc;
          else P[k] = N[k];
          dz = make_float4(-du[0], -du[1], -du[2], -du[3]);
          zc = zu;
          if (!KEEP && k + 1 < RUN) load();
        }
      }
      if (at_top) {    // with forcing and damping
        float nv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float src = 0.f;
          if (!ADJ) src = top_source(gx + e, gy);
          else src -= rt[e] * (a.dt2_h3 * (2.f * wx[e] * wy));
          nv[e] = update(tv[e], tp[e], tS[e], src, (abs_a & RES_ZH) != 0, (abs_b & RES_ZH) != 0);
        }
        n_top = make_float4(nv[0], nv[1], nv[2], nv[3]);
        here(n_top.x), here(n_top.y), here(n_top.z), here(n_top.w);
      }
    }
    __syncthreads();
    {
      float4* p = reinterpret_cast<float4*>(L + fresh(base));
#pragma unroll
      for (int k = 0; k < RUN; ++k)
        if (k < run) {
          float4 v = KEEP ? N[k] : P[k];
          if (!KEEP) P[k] = p[k * (SZ / 4)];
          if (k == b.run - 1 && at_top) v = n_top;
          p[k * (SZ / 4)] = v;
        }
    }
    __syncthreads();
    if (special) {
#pragma unroll
      for (int j = 0; j <= NSP; ++j) {
        if (j < NSP && j >= n_sp) continue;
        const uint32_t mt = fresh(meta[j]);
        if (!mt) continue;
        L[mt & 0xFFFFu] = T[j];
      }
      __syncthreads();
    }
    const unsigned tag = tag0 + n + 1;
    u64* buf = a.xbuf + (size_t)((n + 1) % RES_RING) * 3 * a.n_pub;
    if (n + 1 < nt) {
      publish(buf, xc, tag, L);
      const bool ok = collect(buf, xc, tag, L, a.ctl, limit, [&] {
        if (grid_faces) copy_rims(rims, L);
      });
      if (!ok) given_up = 1;
    }
    // (memory operations of a wave complete in order: these would hold up the words' answers above)
    if (!ADJ) {
      float* tr = a.traces + (int64_t)n * a.n_det * 3 + comp;
      float* ih = a.ihist ? a.ihist + ((int64_t)(n + 1) * 3 + comp) * a.n_l0 : nullptr;
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        if (i * RES_THREADS >= b.out_n) break;
        if (out_i[i] >= 0) {
          const uint32_t c = fresh(out_c[i]);
          const int o = fresh(out_i[i]);
          const float v = L[c & 0xFFFFu];
          if (c >> 16) { if (ih) ih[o] = v; }
          else tr[(int64_t)o * 3] = v;
        }
      }
      for (int e = NO * RES_THREADS + t; e < b.out_n; e += RES_THREADS) {
        const uint32_t c = a.out_cell[b.out_off + e];
        const int i = a.out_idx[b.out_off + e];
        const float v = L[c & 0xFFFFu];
        if (c >> 16) { if (ih) ih[i] = v; }
        else tr[(int64_t)i * 3] = v;
      }
    } else if (k1 > 1) {
      cotangent(k1 - 1);
    }
    __syncthreads();
    if (given_up) return;
  }
  if (!finish(a, limit)) return;
  // the last two levels, where the step kernels leave them
  float* now = a.Efd[ADJ ? 0 : nt & 1] + comp * a.N;
  float* before = a.Efd[ADJ ? 1 : (nt - 1) & 1] + comp * a.N;
#pragma unroll
  for (int k = 0; k < RUN; ++k)
    if (k < run_) {
      const float v[4] = {P[k].x, P[k].y, P[k].z, P[k].w};
      const int gz = b.lo[2] + z_beg + k;
      const bool in_yz = gy > a.blo[1] && gy < a.bhi[1] && gz > a.blo[2] && gz < a.bhi[2];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (4 * xq + e >= b.dim[0] || (in_yz && gx + e > a.blo[0] && gx + e < a.bhi[0])) continue;
        const int64_t g = gx + e + (int64_t)a.nx * (gy + (int64_t)a.ny * gz);
        now[g] = L[base + k * SZ + e];
        before[g] = v[e];
      }
    }
}

// ---- finite-element bricks ------------------------------------------------------------------------
// A brick's nodes sit in LDS, a box of float4 (E or lambda, eps - 1) with a one-node rim; a thread takes M of
// them, with their increments, coefficients and gradient sums in registers.
template <int M>
struct FemNodes {
  int own[M], cell[M];        // owned id (-1: none), box cell
  float c1[M], c2[M];
};
template <int M>
__device__ __forceinline__ void fem_nodes(const ResArgs& a, const ResBlock& b, FemNodes<M>& f) {
  const int n = b.dim[0] * b.dim[1] * b.dim[2];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int l = threadIdx.x + j * RES_THREADS;
    const int2 nd = a.fem_node[b.node_off + (l < n ? l : 0)];   // without a node: the first one's sums, unused
    f.own[j] = l < n ? nd.x : -1;
    f.cell[j] = nd.y;
    f.c1[j] = a.c1[nd.x];
    f.c2[j] = a.c2[nd.x];
  }
}

// Increments of a forward step (also the recompute's): V = c1 V - c2 (row sums).
template <int M>
__device__ __forceinline__ void fem_advance(const ResArgs& a, const FemNodes<M>& f, const float4* box, int sx, int sxy,
                                            float (&V)[M][3]) {
#pragma clang fp contract(off)
  float r[M][3] = {}, q[M][3] = {};
  StarSums<0, M, false>::run(a, box, f.cell, sx, sxy, r, q);
#pragma unroll
  for (int j = 0; j < M; ++j)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      V[j][c] = __builtin_fmaf(f.c1[j], V[j][c], -(f.c2[j] * r[j][c]));
      here(V[j][c]);
    }
}

template <int M>
__device__ __forceinline__ void fem_forward(const ResArgs& a, const ResBlock& b, float* L, long long limit) {
#pragma clang fp contract(off)
  __shared__ int given_up;
  const int t = threadIdx.x, nt = a.nt;
  const int64_t n_own = a.n_own;
  const int sx = b.dim[0] + 2, sxy = sx * (b.dim[1] + 2);
  float4* box = reinterpret_cast<float4*>(L);
  for (int i = t; i < sxy * (b.dim[2] + 2); i += RES_THREADS) box[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (t == 0) given_up = 0;
  Exchange xc;
  exchange_lists<true>(a, b, b.con_n, xc);
  FemNodes<M> f;
  fem_nodes(a, b, f);
  float V[M][3];
  __syncthreads();
  for (int e = t; e < b.con_fem; e += RES_THREADS) L[4 * a.con_cell[b.con_off + e] + 3] = a.em1[a.con_src[b.con_off + e]];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    V[j][0] = V[j][1] = V[j][2] = 0.f;
    if (f.own[j] < 0) continue;
    box[f.cell[j]].w = a.em1[f.own[j]];
    if (a.ckpt)
      for (int c = 0; c < 6; ++c) {
        a.ckpt[c * n_own + f.own[j]] = 0.f;
        if (a.k_tail == 0) a.tail[c * n_own + f.own[j]] = 0.f;
      }
  }
  const unsigned tag0 = a.ctl->epoch[0];
  __syncthreads();
  for (int n = 0; n < nt; ++n) {
    fem_advance(a, f, box, sx, sxy, V);
    __syncthreads();
    const bool last = n + 1 == nt;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      if (f.own[j] < 0) continue;
      float* e = L + 4 * fresh(f.cell[j]);
      const int own = fresh(f.own[j]), g = last ? a.own_grid[own] : -1;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float old = e[c];
        e[c] = old + V[j][c];
        if (last) {
          a.Efem[n & 1][c * n_own + own] = old;
          if (g >= 0) a.Efd[n & 1][c * a.N + g] = old;
        }
      }
    }
    __syncthreads();
    const unsigned tag = tag0 + n + 1;
    u64* buf = a.xbuf + (size_t)((n + 1) % RES_RING) * 3 * a.n_pub;
    if (!last) {
      publish(buf, xc, tag, L);
      if (!collect(buf, xc, tag, L, a.ctl, limit, [] {})) given_up = 1;
    }
    float* ck = nullptr;
    if (a.ckpt && n + 1 >= a.k_tail)
      ck = a.tail + (n + 1 - a.k_tail) * 6 * n_own;
    else if (a.ckpt && (n + 1) % a.K == 0 && (n + 1) / a.K < a.n_ck)
      ck = a.ckpt + ((n + 1) / a.K) * 6 * n_own;
    if (ck)
#pragma unroll
      for (int j = 0; j < M; ++j) {
        const int own = fresh(f.own[j]);
        if (own < 0) continue;
        const float* e = L + 4 * fresh(f.cell[j]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          __builtin_nontemporal_store(e[c], ck + c * n_own + own);
          __builtin_nontemporal_store(V[j][c], ck + (3 + c) * n_own + own);
        }
      }
    __syncthreads();
    if (given_up) return;
  }
  if (!finish(a, limit)) return;
#pragma unroll
  for (int j = 0; j < M; ++j) {
    if (f.own[j] < 0) continue;
    const int g = a.own_grid[f.own[j]];
    for (int c = 0; c < 3; ++c) {
      const float v = L[4 * f.cell[j] + c];
      a.Efem[nt & 1][c * n_own + f.own[j]] = v;
      a.Vfem[c * n_own + f.own[j]] = V[j][c];
      if (g >= 0) a.Efd[nt & 1][c * a.N + g] = v;
    }
  }
}

// REC: the forward state of the segment before the one the adjoint is in is recomputed beside it, a step per step,
// in a second box, into that segment's window (which the same threads read later).
template <int M, bool REC>
__device__ __forceinline__ void fem_adjoint(const ResArgs& a, const ResBlock& b, float* L, long long limit) {
#pragma clang fp contract(off)
  __shared__ int given_up;
  const int t = threadIdx.x, nt = a.nt;
  const int64_t n_own = a.n_own, n_l0 = a.n_l0;
  const int sx = b.dim[0] + 2, sxy = sx * (b.dim[1] + 2), cells = sxy * (b.dim[2] + 2);
  float4* box = reinterpret_cast<float4*>(L);
  float* LR = L + 4 * cells;
  float4* boxR = reinterpret_cast<float4*>(LR);
  for (int i = t; i < cells; i += RES_THREADS) box[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (t == 0) given_up = 0;
  Exchange xc, xr;
  exchange_lists<true>(a, b, b.con_n, xc);
  if (REC) exchange_lists<true>(a, b, b.con_fem, xr);
  FemNodes<M> f;
  fem_nodes(a, b, f);
  float V[M][3] = {}, VR[M][3] = {}, em[M], wV[M][3], wM[M][3];
  double m[M], ge[M], gs[M];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int own = f.own[j] < 0 ? 0 : f.own[j];
    em[j] = a.em1[own];
    m[j] = a.mass_d[own];
    ge[j] = a.g_eps[own];
    gs[j] = a.g_sig[own];
  }
  const unsigned tag0 = a.ctl->epoch[1];
  unsigned tag_rec = tag0;
  const int n_rim0 = b.con_n - b.con_fem;      // layer-0 nodes of the rim
  __syncthreads();
  int n = 0;
  for (int64_t seg = a.nseg - 1; seg >= 0; --seg) {
    const int64_t k0 = seg * a.K, k1 = min(k0 + a.K, (int64_t)nt);
    const float* win = seg == a.nseg - 1 ? a.tail : (seg & 1) ? a.win_b : a.win;
    const int n_adj = (int)(k1 - k0), n_rec = REC && seg > 0 ? (int)a.K : 0;
    float* winR = (seg & 1) ? a.win : a.win_b;
    const int64_t r0 = k0 - a.K;               // first level of the recomputed segment
    if (n_rec) {
      const float* ck = a.ckpt + (seg - 1) * 6 * n_own;
#pragma unroll
      for (int j = 0; j < M; ++j) {
        if (f.own[j] < 0) continue;
        float* e = LR + 4 * f.cell[j];
        for (int c = 0; c < 3; ++c) {
          const float x = ck[c * n_own + f.own[j]], v = ck[(3 + c) * n_own + f.own[j]];
          e[c] = x;
          VR[j][c] = v;
          winR[c * n_own + f.own[j]] = x;
          winR[(3 + c) * n_own + f.own[j]] = v;
        }
        e[3] = em[j];
      }
      for (int e = t; e < b.con_n; e += RES_THREADS) {
        float* p = LR + 4 * a.con_cell[b.con_off + e];
        const int src = a.con_src[b.con_off + e];
        for (int c = 0; c < 3; ++c) p[c] = src >= 0 ? ck[c * n_own + src] : a.ihist[(r0 * 3 + c) * n_l0 - 1 - src];
        p[3] = src >= 0 ? a.em1[src] : 0.f;
      }
      __syncthreads();
    }
    // V^k of a step is V^{k-1} of the one before: only the segment's first step reads it
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c) wM[j][c] = f.own[j] < 0 ? 0.f : win[(n_adj * 6 + 3 + c) * n_own + f.own[j]];
    const int steps = max(n_adj, n_rec);
    for (int i = 0; i < steps; ++i) {
      const bool adj = i < n_adj, rec = i < n_rec;
      // the step's forward state, E^k and V^{k-1}, on its way during the sums
      float wE[M][3];
      if (adj)
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const int own = fresh(f.own[j]);
          const float* w = win + (int64_t)(n_adj - i) * 6 * n_own + (own < 0 ? 0 : own);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            wV[j][c] = wM[j][c];
            wE[j][c] = w[c * n_own];
            wM[j][c] = w[(c - 3) * n_own];
          }
        }
      if (rec) fem_advance(a, f, boxR, sx, sxy, VR);
      if (adj) {
        float r[M][3] = {}, q[M][3] = {};
        StarSums<0, M, true>::run(a, box, f.cell, sx, sxy, r, q);
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const float* x = reinterpret_cast<const float*>(box + fresh(f.cell[j]));
          double e = 0.0, g = 0.0, s = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float sum = __builtin_fmaf(em[j], q[j][c], r[j][c]);
            const float inc = __builtin_fmaf(f.c1[j], V[j][c], -(f.c2[j] * sum));
            const float xn = x[c] + inc;
            V[j][c] = inc;
            const double wv = (double)wV[j][c];
            e = __builtin_fma((double)q[j][c], (double)wE[j][c], e);
            g = __builtin_fma((double)inc, wv, g);
            s = __builtin_fma((double)xn, wv + (double)wM[j][c], s);
          }
          ge[j] += __builtin_fma(m[j] * a.inv_dt2, g, e);
          gs[j] += m[j] * a.inv_2dt * s;
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < M; ++j) {
        if (f.own[j] < 0) continue;
        const int cell = fresh(f.cell[j]);
        if (adj) {
          float* e = L + 4 * cell;
#pragma unroll
          for (int c = 0; c < 3; ++c) e[c] += V[j][c];
        }
        if (rec) {
          float* e = LR + 4 * cell;
#pragma unroll
          for (int c = 0; c < 3; ++c) e[c] += VR[j][c];
        }
      }
      __syncthreads();
      bool ok = true;
      u64* buf = a.xbuf + (size_t)((n + 1) % RES_RING) * 3 * a.n_pub;
      const bool more = adj && n + 1 < nt, more_rec = rec && i + 1 < n_rec;
      if (more) publish(buf, xc, tag0 + n + 1, L);
      if (more_rec) {
        ++tag_rec;
        u64* bufR = a.xbuf_rec + (size_t)(tag_rec % RES_RING) * 3 * a.n_pub;
        publish(bufR, xr, tag_rec, LR);
        const float* ih = a.ihist + (r0 + i + 1) * 3 * n_l0;
        for (int e = t; e < n_rim0; e += RES_THREADS) {
          const int k = b.con_off + b.con_fem + e, src = -1 - a.con_src[k];
          float* to = LR + 4 * a.con_cell[k];
#pragma unroll
          for (int c = 0; c < 3; ++c) to[c] = ih[c * n_l0 + src];
        }
        if (more) ok = collect(buf, xc, tag0 + n + 1, L, bufR, xr, tag_rec, LR, a.ctl, limit);
        else ok = collect(bufR, xr, tag_rec, LR, a.ctl, limit, [] {});
      } else if (more) {
        ok = collect(buf, xc, tag0 + n + 1, L, a.ctl, limit, [] {});
      }
      if (!ok) given_up = 1;
      if (rec)
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const int own = fresh(f.own[j]);
          if (own < 0) continue;
          const float* e = LR + 4 * fresh(f.cell[j]);
          float* w = winR + (int64_t)(i + 1) * 6 * n_own + own;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            w[c * n_own] = e[c];
            w[(3 + c) * n_own] = VR[j][c];
          }
        }
      if (adj) ++n;
      __syncthreads();
      if (given_up) return;
    }
  }
  if (!finish(a, limit)) return;
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int own = f.own[j];
    if (own < 0) continue;
    const int g = a.own_grid[own];
    if (g < 0) {              // free nodes
      a.g_eps[own] = ge[j];
      a.g_sig[own] = gs[j];
    }
    for (int c = 0; c < 3; ++c) {
      const float v = L[4 * f.cell[j] + c], before = v - V[j][c];
      a.Efem[0][c * n_own + own] = v;
      a.Efem[1][c * n_own + own] = before;
      a.Vfem[c * n_own + own] = V[j][c];
      if (g >= 0) {
        a.Efd[0][c * a.N + g] = v;
        a.Efd[1][c * a.N + g] = before;
      }
    }
  }
}

template <bool ADJ, bool REC>
__device__ __forceinline__ void fem_brick(const ResArgs& a, const ResBlock& b, float* L, long long limit) {
  const int n = b.dim[0] * b.dim[1] * b.dim[2];
  if (n <= RES_THREADS) {
    if (ADJ) fem_adjoint<1, REC>(a, b, L, limit);
    else fem_forward<1>(a, b, L, limit);
  } else if (n <= 2 * RES_THREADS) {
    if (ADJ) fem_adjoint<2, REC>(a, b, L, limit);
    else fem_forward<2>(a, b, L, limit);
  } else {
    if (ADJ) fem_adjoint<RES_NF_MAX, REC>(a, b, L, limit);
    else fem_forward<RES_NF_MAX>(a, b, L, limit);
  }
}

template <int RUN, bool ADJ, bool REC>
__global__ __launch_bounds__(RES_THREADS) void resident_kernel(ResArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  if (!assemble(a)) return;
  const long long limit = wall_clock64() + a.run_ticks;
  const ResBlock b = a.blocks[blockIdx.x];
  float* L = reinterpret_cast<float*>(lds);
  if (!b.fem) fd_brick<RUN, ADJ>(a, b, L, limit);
  else fem_brick<ADJ, REC>(a, b, L, limit);
}

struct TabChunk { double v[RES_TAB]; };
__global__ void resident_begin_kernel(ResCtl* c, bool adj, int tags, bool first, double* tab, int off, int n, TabChunk v) {
  if (off == 0 && threadIdx.x == 0) {
    c->epoch[adj] += tags;
    c->arrive = c->end = 0;
    c->tickets = c->finished = 0;
    if (first) c->skip = 0;
    c->state = c->skip ? RES_OFF : RES_WAIT;
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) tab[off + i] = v.v[i];
}
template <int RUN, bool ADJ, bool REC>
void launch_t(const ResArgs& a, size_t lds, hipStream_t s) {
  (void)hipFuncSetAttribute((const void*)resident_kernel<RUN, ADJ, REC>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((resident_kernel<RUN, ADJ, REC>), dim3(a.n_blocks), dim3(RES_THREADS), lds, s, a);
}

}  // namespace

void launch_resident_begin(const ResArgs& a, bool adj, bool first, const double* tab, int n, hipStream_t s) {
  int off = 0;
  do {
    TabChunk v;
    const int m = std::min(n - off, RES_TAB);
    for (int i = 0; i < m; ++i) v.v[i] = tab[off + i];
    hipLaunchKernelGGL(resident_begin_kernel, dim3(1), dim3(512), 0, s, a.ctl, adj, 2 * a.nt + 64, first, const_cast<double*>(a.tab), off,
                       m, v);
    off += m;
  } while (off < n);
}

namespace {
template <bool ADJ, bool REC>
void launch_run(const ResArgs& a, const ResPlan& plan, hipStream_t s) {
  const size_t lds = plan.lds();
  if (plan.max_run <= 2) launch_t<2, ADJ, REC>(a, lds, s);
  else if (plan.max_run <= 4) launch_t<4, ADJ, REC>(a, lds, s);
  else if (plan.max_run <= 8) launch_t<8, ADJ, REC>(a, lds, s);
  else launch_t<12, ADJ, REC>(a, lds, s);
}
}  // namespace

void launch_resident(const ResArgs& a, const ResPlan& plan, hipStream_t s) {
  if (!plan.adj) launch_run<false, false>(a, plan, s);
  else if (plan.rec) launch_run<true, true>(a, plan, s);
  else launch_run<true, false>(a, plan, s);
}

}  // namespace dd
