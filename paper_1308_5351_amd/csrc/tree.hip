// Far-field compression of the Cauchy sums S_i = sum_{j != i} w_j/(eta_i - eta_j)
// for large N (the paper evaluates these sums with a fast multipole method;
// this is a treecode on the GPU, FP64 throughout):
//   * boxes: level 0 holds the leaves of up to kLeaf = 64 consecutive nodes of a
//     curve (of fewer than 64 nodes a curve: across curves), level l + 1 pairs the
//     boxes of level l; each box has a bounding circle;
//   * multipole moments of box b about its centre c_b in units of its radius r_b,
//     for one weight column: a_k = sum_{j in b} w_j ((eta_j - c_b)/r_b)^k, k < p;
//     leaves from their nodes, parents from their children by the binomial shift;
//   * a box far from a target tile (centre c_t, radius r_t) enters the tile's
//     local expansion sum_l L_l ((z - c_t)/r_t)^l: with D = c_t - c_b, x = r_b/D and
//     y = -r_t/D,  L_l += y^l sum_{k < p_e} C(k + l, l) a_k x^k / D,
//     truncated on the box's side with error below (r_b/(|D| - r_t))^p_e and on
//     the tile's side below (r_t/(|D| - r_b))^q_e, each times a factor of at most
//     2.4 and sum |w_j|/|z - eta_j|; the expansion is evaluated once per target;
//   * every other source is summed directly, leaf by leaf, by the
//     FP64 pair loops (j != i excluded);
//   * the order of the leaves (and of separate targets) along a Hilbert curve
//     and the interaction lists (far boxes and near blocks per target tile) are
//     made on the GPU; each (target tile, split) workgroup takes four equal
//     ranges of its tile's near sources, one per wavefront, and writes one partial
//     sum, which the consumer adds in split order like those of the direct
//     kernels.
// Local expansions instead of evaluating every far box at every target (4 p_e +
// 14 operations each), and leaves of 64 nodes instead of 256: at 1089 x 4096 nodes
// a target meets 506 near sources and 145 boxes instead of 1020 and 115, and a
// product took 2.6 ms instead of 5.3; now 2.2 (near sums 1.05, expansions 0.9, moments 0.2).
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>
#include <vector>

#include "gnk_device.h"
#include "gnk_internal.h"

namespace gnk {

namespace {

#include "pair_steps.inl"

// Bounding circles {cx, cy, r, 0} of the boxes of every level: the centre of
// the box's bounding box and the largest distance of its nodes from it. The
// leaves (up to kLeaf consecutive nodes) take the slots of level 0 in an order chosen
// by their centres (perm: slot -> leaf); the box of slots
// [b 2^l, (b + 1) 2^l) is box b of level l. Leaf bounding boxes come from
// their nodes (one wavefront per leaf), a parent's from its two children
// (exact: min and max), and the radii of all levels from one pass over the
// nodes (maxima over the waves, then an atomic maximum on the radius's bit
// pattern, which orders non-negative doubles as unsigned integers).
__global__ __launch_bounds__(64) void k_leaf_bbox(const double2* __restrict__ eta, int N, Pieces leaves,
                                                  double4* __restrict__ bbox) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int i0 = leaves.first(b), i1 = leaves.last(b, N);
  double xmin = 1e300, xmax = -1e300, ymin = 1e300, ymax = -1e300;
  for (int i = i0 + lane; i < i1; i += 64) {
    const double2 e = eta[i];
    xmin = fmin(xmin, e.x);
    xmax = fmax(xmax, e.x);
    ymin = fmin(ymin, e.y);
    ymax = fmax(ymax, e.y);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    xmin = fmin(xmin, __shfl_xor(xmin, off, 64));
    xmax = fmax(xmax, __shfl_xor(xmax, off, 64));
    ymin = fmin(ymin, __shfl_xor(ymin, off, 64));
    ymax = fmax(ymax, __shfl_xor(ymax, off, 64));
  }
  if (lane == 0) bbox[b] = make_double4(xmin, xmax, ymin, ymax);
}

__global__ __launch_bounds__(64) void k_piece_circles(const double2* __restrict__ eta, int N, Pieces tiles,
                                                      double4* __restrict__ out) {
  const int b = blockIdx.x;
  const double4 v = wave_circle(eta, tiles.first(b), tiles.last(b, N));
  if (threadIdx.x == 0) out[b] = v;
}

__global__ void k_bbox_gather(const double4* __restrict__ leafbox, const int* __restrict__ perm, int nleaf,
                              double4* __restrict__ slotbox) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nleaf) slotbox[s] = leafbox[perm[s]];
}

__global__ void k_bbox_merge(const double4* __restrict__ child, int nchild, double4* __restrict__ parent, int npar) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= npar) return;
  double4 v = child[2 * b];
  if (2 * b + 1 < nchild) {
    const double4 u = child[2 * b + 1];
    v = make_double4(fmin(v.x, u.x), fmax(v.y, u.y), fmin(v.z, u.z), fmax(v.w, u.w));
  }
  parent[b] = v;
}

// centres of all boxes; radii (as bits) cleared for the maximum that follows
__global__ void k_box_centres(const double4* __restrict__ bbox, int nbox, double4* __restrict__ out,
                              unsigned long long* __restrict__ rbits) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbox) return;
  const double4 v = bbox[b];
  out[b] = make_double4(0.5 * (v.x + v.y), 0.5 * (v.z + v.w), 0.0, 0.0);
  rbits[b] = 0ull;
}

struct LevelTable {
  int off[32];   // first box of each level
  int nb[32];    // boxes of each level
};

// A block takes 16 consecutive slots, one wavefront each: from level 4 on they
// lie in one box, whose maximum the block forms before its atomic (one atomic a
// leaf would queue 70000 of them on the top box of 4460544 nodes).
constexpr int kRadiiWaves = 16;
__global__ __launch_bounds__(64 * kRadiiWaves) void k_box_radii(const double2* __restrict__ eta, int N,
                                                                Pieces leaves, LevelTable lv, int levels, int nleaf,
                                                                const int* __restrict__ perm,
                                                                const double4* __restrict__ out,
                                                                unsigned long long* __restrict__ rbits) {
  static_assert(kLeaf == 64, "one node per lane");
  __shared__ double sh[32][kRadiiWaves];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int slot = blockIdx.x * kRadiiWaves + wv;
  const bool has = slot < nleaf;
  const int i = has ? leaves.first(perm[slot]) + lane : N;
  const bool in = has && i < leaves.last(perm[slot], N);
  const double2 e = in ? eta[i] : make_double2(0.0, 0.0);
  for (int l = 0; l < levels; ++l) {
    const double4 c = out[lv.off[l] + (has ? slot >> l : 0)];
    double r = in ? sqrt((e.x - c.x) * (e.x - c.x) + (e.y - c.y) * (e.y - c.y)) : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) r = fmax(r, __shfl_xor(r, off, 64));
    if (lane == 0) {
      if (l < 4) {
        if (has) atomicMax(rbits + lv.off[l] + (slot >> l), (unsigned long long)__double_as_longlong(r));
      } else {
        sh[l][wv] = r;
      }
    }
  }
  __syncthreads();
  const int l = threadIdx.x;
  if (l >= 4 && l < levels) {
    double r = 0.0;
    for (int w = 0; w < kRadiiWaves; ++w) r = fmax(r, sh[l][w]);
    atomicMax(rbits + lv.off[l] + ((blockIdx.x * kRadiiWaves) >> l), (unsigned long long)__double_as_longlong(r));
  }
}

// widen by a relative margin so rounding of the centre cannot hide a node
__global__ void k_box_finish(const unsigned long long* __restrict__ rbits, int nbox, double4* __restrict__ out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbox) return;
  const double r = __longlong_as_double((long long)rbits[b]);
  out[b].z = r * (1.0 + 1e-12) + 1e-300;
}

// Leaf moments of the launch's weight columns (record fields wo, wo + 1, .. by
// blockIdx.y): four lanes per level-0 slot (leaf perm[slot]), each CH moments from
// k = CH q on, the powers advanced from ((eta - c)/r)^(CH q), so that nothing is
// reduced across lanes and a leaf's records are read once. Bound by the records'
// loads (32 bytes a node with one column).
template <int CH>
__global__ __launch_bounds__(64) void k_leaf_moments(const double2* __restrict__ rec, int stride, int wo, int N,
                                                     Pieces leaves, const double4* __restrict__ bounds,
                                                     const int* __restrict__ perm, int nleaf, int p,
                                                     double2* __restrict__ mom, size_t colstride,
                                                     const int* __restrict__ active) {
  if (active != nullptr && active[blockIdx.y] == 0) return;
  const int b = blockIdx.x * 16 + (threadIdx.x >> 2), q = threadIdx.x & 3;
  if (b >= nleaf) return;
  const double4 c = bounds[b];
  const double inv = 1.0 / c.z;
  const int j0 = leaves.first(perm[b]), j1 = leaves.last(perm[b], N);
  const int w0 = wo + blockIdx.y;
  double ax[CH], ay[CH];
#pragma unroll
  for (int k = 0; k < CH; ++k) ax[k] = ay[k] = 0.0;
  constexpr int G = 8;   // nodes in flight
  for (int j = j0; j < j1; j += G) {
    double2 e[G], w[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double2* r = rec + (size_t)min(j + g, j1 - 1) * stride;
      e[g] = r[0];
      w[g] = j + g < j1 ? r[w0] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double x = (e[g].x - c.x) * inv, y = (e[g].y - c.y) * inv;
      double px = 1.0, py = 0.0;   // ((eta - c)/r)^CH
#pragma unroll
      for (int m = 0; m < CH; ++m) {
        const double nx = px * x - py * y;
        py = px * y + py * x;
        px = nx;
      }
      double tx = w[g].x, ty = w[g].y;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const double nx = tx * px - ty * py, ny = tx * py + ty * px;
        tx = m < q ? nx : tx;
        ty = m < q ? ny : ty;
      }
#pragma unroll
      for (int k = 0; k < CH; ++k) {
        ax[k] += tx;
        ay[k] += ty;
        const double nx = tx * x - ty * y;
        ty = tx * y + ty * x;
        tx = nx;
      }
    }
  }
  double2* o = mom + blockIdx.y * colstride + (size_t)b * p + CH * q;
#pragma unroll
  for (int k = 0; k < CH; ++k)
    if (CH * q + k < p) o[k] = make_double2(ax[k], ay[k]);
}

// ---------------------------------------------------- local expansions of tiles
// Workgroups go to the eight XCDs in turn: with this order each takes a contiguous
// run of the n items (n a multiple of 8), whose boxes and records its L2 shares.
__device__ __forceinline__ int xcd_order(int b, int n) { return (b & 7) * (n >> 3) + (b >> 3); }

constexpr int kLoc = kTreeMaxP;   // terms of a local expansion, in chunks of 16

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ double2 zsquare(double2 a) {
  return make_double2(a.x * a.x - a.y * a.y, 2.0 * (a.x * a.y));
}

// z^j for j = 0..15 (from the bits of j), and z^8 in z8
__device__ __forceinline__ double2 power16(double2 z, int j, double2& z8) {
  const double2 one = make_double2(1.0, 0.0);
  const double2 z2 = zsquare(z), z4 = zsquare(z2);
  z8 = zsquare(z4);
  double2 v = (j & 1) ? z : one;
  v = zmul(v, (j & 2) ? z2 : one);
  v = zmul(v, (j & 4) ? z4 : one);
  return zmul(v, (j & 8) ? z8 : one);
}

// lane K of the lane's row of 16
template <int K>
__device__ __forceinline__ double row_lane(double v) {
  const long long zero = 0, p = __builtin_bit_cast(long long, v);
  const long long q = __builtin_amdgcn_update_dpp(zero, p, 0x150 + K, 0xf, 0xf, true);   // row_newbcast:K
  return __builtin_bit_cast(double, q);
}

// Moments of levels l0 + 1 .. l0 + nlev from those of level l0. a_k of a child in its
// parent's terms, scaled by (r_child/r_parent)^k and shifted by e = (c_child -
// c_parent)/r_parent, is
//   sum_{q <= k} C(k, q) e^(k - q) a_q,
// formed as Horner's rule in e over q, the a_q broadcast by DPP: a row of 16 lanes per
// child, lane j of it the terms k = j, j + 16, j + 32 (P >= p in all). A workgroup
// takes 64 boxes of level l0, 32 rows at a time, up to their common ancestor six levels
// on; siblings lie in neighbouring rows, and parents pass on through LDS. Bound by
// these chains, P complex steps per level and row (a lane per box with its moments in
// registers and a_k += e a_(k-1), p^2/2 products a level in one chain, took 35-44 us a
// launch at 33 terms; at N = 4460544 95, 50 and 40 us, now 85, 23 and 20; at 614400
// 34.5, now 18).
constexpr int kM2MLevels = 6;

// the table's entries C(k, q) of the four q from 4 G on
template <int NCH, int P, int G>
__device__ __forceinline__ void m2m_table(double (&t)[4][NCH], const double* tab, int j) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int ch = G / 4; ch < NCH; ++ch)
      t[i][ch] = tab[(4 * G + i) * P + max(16 * ch + j - (4 * G + i), 0)];
}
template <int NCH, int P, int Q>
__device__ __forceinline__ void m2m_step(double2 (&s)[NCH], const double2 (&b)[NCH], double ex, double ey,
                                         const double (&t)[NCH], int j) {
  constexpr int QC = Q / 16, QI = Q % 16;
  const double bx = row_lane<QI>(b[QC].x), by = row_lane<QI>(b[QC].y);
#pragma unroll
  for (int ch = QC; ch < NCH; ++ch) {
    const double nx = __builtin_fma(ex, s[ch].x, __builtin_fma(-ey, s[ch].y, t[ch] * bx));
    const double ny = __builtin_fma(ex, s[ch].y, __builtin_fma(ey, s[ch].x, t[ch] * by));
    const bool on = ch > QC || j >= QI;
    s[ch].x = on ? nx : s[ch].x;
    s[ch].y = on ? ny : s[ch].y;
  }
}
// the steps of four q, the next four's entries loading meanwhile (the barriers keep the
// broadcasts and reads of all steps from going first, past the registers)
template <int NCH, int P, int G>
__device__ __forceinline__ void m2m_group(double2 (&s)[NCH], const double2 (&b)[NCH], double ex, double ey,
                                          double (&t)[2][4][NCH], const double* tab, int j) {
  if constexpr (4 * G + 4 < P) m2m_table<NCH, P, G + 1>(t[(G + 1) & 1], tab, j);
  __builtin_amdgcn_sched_barrier(0);
  m2m_step<NCH, P, 4 * G>(s, b, ex, ey, t[G & 1][0], j);
  m2m_step<NCH, P, 4 * G + 1>(s, b, ex, ey, t[G & 1][1], j);
  m2m_step<NCH, P, 4 * G + 2>(s, b, ex, ey, t[G & 1][2], j);
  m2m_step<NCH, P, 4 * G + 3>(s, b, ex, ey, t[G & 1][3], j);
  __builtin_amdgcn_sched_barrier(0);
}
template <int NCH, int P, int... G>
__device__ __forceinline__ void m2m_groups(double2 (&s)[NCH], const double2 (&b)[NCH], double ex, double ey,
                                           const double* tab, int j, std::integer_sequence<int, G...>) {
  double t[2][4][NCH];
  m2m_table<NCH, P, 0>(t[0], tab, j);
  (m2m_group<NCH, P, G>(s, b, ex, ey, t, tab, j), ...);
}

constexpr int kM2MT = 512;   // 32 rows
template <int P>
__global__ __launch_bounds__(kM2MT) void k_m2m_levels(const double4* __restrict__ bounds, LevelTable lt, int l0,
                                                    int nlev, int p, double2* __restrict__ mom, size_t colstride,
                                                    const double* __restrict__ binom, const int* __restrict__ active) {
  constexpr int NCH = (P + 15) / 16;
  __shared__ double tab[P * P];              // tab[q][d] = C(q + d, q)
  __shared__ double2 even[32 * P], odd[16 * P];   // parents after odd and even steps
  __shared__ double4 box[128];               // {c, r, 1/r}: level l0 + s from 128 - (128 >> s) on
  if (active != nullptr && active[blockIdx.y] == 0) return;
  for (int i = threadIdx.x; i < P * P; i += kM2MT) tab[i] = binom[(i / P) * kTreeMaxP + i % P];
  if (threadIdx.x < 127) {
    const int s = 6 - (31 - __clz(127 - threadIdx.x));
    const int b = blockIdx.x * (64 >> s) + threadIdx.x - (128 - (128 >> s));
    if (s <= nlev && b < lt.nb[l0 + s]) {
      const double4 v = bounds[lt.off[l0 + s] + b];
      box[threadIdx.x] = make_double4(v.x, v.y, v.z, 1.0 / v.z);
    }
  }
  __syncthreads();
  mom += blockIdx.y * colstride;
  const int row = threadIdx.x >> 4, j = threadIdx.x & 15;
  for (int s = 1; s <= nlev; ++s) {
    const int l = l0 + s, nc = 64 >> (s - 1), first = blockIdx.x * nc;
    const double2* src = (s & 1) ? odd : even;
    double2* dst = (s & 1) ? even : odd;
    for (int r0 = 0; r0 + (row & ~3) < nc; r0 += kM2MT / 16) {   // (whole waves)
      const int lc = r0 + row, cb = first + lc;
      const bool live = lc < nc && cb < lt.nb[l - 1];
      double2 b[NCH], a[NCH];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int k = 16 * ch + j;
        b[ch] = a[ch] = make_double2(0.0, 0.0);
        if (live && k < p) b[ch] = s == 1 ? mom[(size_t)(lt.off[l - 1] + cb) * p + k] : src[lc * P + k];
      }
      const int at = live ? lc : 0;
      const double4 cc = box[128 - (256 >> s) + at], cp = box[128 - (128 >> s) + (at >> 1)];
      const double ratio = live ? cc.z * cp.w : 0.0;
      const double ex = live ? (cc.x - cp.x) * cp.w : 0.0, ey = live ? (cc.y - cp.y) * cp.w : 0.0;
      const double f2 = ratio * ratio, f4 = f2 * f2, f8 = f4 * f4, f16 = f8 * f8;
      double f = (j & 1) ? ratio : 1.0;
      f *= (j & 2) ? f2 : 1.0;
      f *= (j & 4) ? f4 : 1.0;
      f *= (j & 8) ? f8 : 1.0;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        b[ch].x *= f;
        b[ch].y *= f;
        f *= f16;
      }
      m2m_groups<NCH, P>(a, b, ex, ey, tab, j, std::make_integer_sequence<int, P / 4>{});
      // the sibling's, of the neighbouring row
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        a[ch].x += __shfl_xor(a[ch].x, 16, 64);
        a[ch].y += __shfl_xor(a[ch].y, 16, 64);
      }
      if (live && (row & 1) == 0) {
        double2* o = mom + (size_t)(lt.off[l] + (cb >> 1)) * p;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
          const int k = 16 * ch + j;
          if (k < p) {
            dst[(lc >> 1) * P + k] = a[ch];
            o[k] = a[ch];
          }
        }
      }
    }
    __syncthreads();
  }
}

// s[ch] += sum over the four k from 4 G on (of the lane's chunk of 16) of
// C(k + l, l) b_k, l = j + 16 ch, ch < NQ; tab: the table's row of the chunk's
// first k at column j. The number of chunks is a template parameter so that the
// table's reads go out together (with a test per chunk and term instead, the
// kernel took 1.09 ms at 1089 x 4096 nodes).
template <int G, int NQ, int NC>
__device__ __forceinline__ void local_terms(double2 (&s)[3][NC], const double2 (&b)[NC], const double* tab) {
  double t[4][NQ];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int ch = 0; ch < NQ; ++ch) t[k][ch] = tab[(4 * G + k) * kLoc + 16 * ch];
  auto term = [&](const double (&tk)[NQ], int c, double bx, double by) {
#pragma unroll
    for (int ch = 0; ch < NQ; ++ch) {
      s[ch][c].x = __builtin_fma(tk[ch], bx, s[ch][c].x);
      s[ch][c].y = __builtin_fma(tk[ch], by, s[ch][c].y);
    }
  };
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    term(t[0], c, row_lane<4 * G>(b[c].x), row_lane<4 * G>(b[c].y));
    term(t[1], c, row_lane<4 * G + 1>(b[c].x), row_lane<4 * G + 1>(b[c].y));
    term(t[2], c, row_lane<4 * G + 2>(b[c].x), row_lane<4 * G + 2>(b[c].y));
    term(t[3], c, row_lane<4 * G + 3>(b[c].x), row_lane<4 * G + 3>(b[c].y));
  }
}

// s[ch] for ch < NQ from the moments a and x^j/D (X) of the row's box, pm terms
template <int NQ, int NC>
__device__ __forceinline__ void local_sums(double2 (&s)[3][NC], const double2 (&a)[3][NC], double2 X, double2 x16,
                                           int pm, const double* tab) {
#pragma unroll
  for (int kc = 0; kc < 3; ++kc) {
    if (16 * kc < pm) {
      if (kc > 0) X = zmul(X, x16);
      double2 b[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) b[c] = zmul(a[kc][c], X);
      const double* tk = tab + 16 * kc * kLoc;
      local_terms<0, NQ, NC>(s, b, tk);
      if (16 * kc + 4 < pm) local_terms<1, NQ, NC>(s, b, tk);
      if (16 * kc + 8 < pm) local_terms<2, NQ, NC>(s, b, tk);
      if (16 * kc + 12 < pm) local_terms<3, NQ, NC>(s, b, tk);
    }
  }
}

// The local expansions of the target tiles for NC weight columns, one wavefront
// per tile, four far boxes at a time, one per row of 16 lanes: lane j of a row
// holds x^j/D and the terms a_k x^k/D of its box for k = j, j + 16, j + 32 and
// forms L_l for l = j, j + 16, j + 32 (as many chunks of 16 as the largest p_e and
// q_e of the four need), each term broadcast over the row by DPP. binom: C(k + l,
// l), kLoc x kLoc. Bound by VALU issue (77 % of the cycles at 1089 x 4096 nodes):
// about 320 instructions per four boxes, where evaluating them at 128 targets took
// 870. loc: per tile and column kLoc coefficients, of which terms[tile] are used.
template <int NC>
__global__ __launch_bounds__(256) void k_tile_locals(const double4* __restrict__ tb, int tiles,
                                                     const int64_t* __restrict__ faroff, const int2* __restrict__ far,
                                                     const double4* __restrict__ bounds,
                                                     const double2* __restrict__ mom, size_t colstride, int p,
                                                     const double* __restrict__ binom, double2* __restrict__ loc,
                                                     int* __restrict__ terms, const int* __restrict__ active) {
  __shared__ double tab[kLoc * kLoc];
  if (active != nullptr) {
    bool any = false;
#pragma unroll
    for (int c = 0; c < NC; ++c) any = any || active[blockIdx.y * NC + c] != 0;
    if (!any) return;
  }
  // the launch's NC-column groups by blockIdx.y
  mom += (size_t)blockIdx.y * NC * colstride;
  loc += (size_t)blockIdx.y * NC * tiles * kLoc;
  for (int i = threadIdx.x; i < kLoc * kLoc; i += 256) tab[i] = binom[i];
  __syncthreads();
  const int lane = threadIdx.x & 63, row = lane >> 4, j = lane & 15;
  struct Box {
    double4 bb;
    double2 a[3][NC];
    int pe, nq;
  };
  const int groups = ((tiles + 3) / 4 + 7) & ~7;
  for (int gb = blockIdx.x; gb < groups; gb += gridDim.x) {
    const int t = xcd_order(gb, groups) * 4 + (threadIdx.x >> 6);
    if (t >= tiles) continue;
    const double4 tt = tb[t];
    const int e0 = __builtin_amdgcn_readfirstlane((int)faroff[t]);
    const int e1 = __builtin_amdgcn_readfirstlane((int)faroff[t + 1]);
    double2 acc[3][NC];
    int most = 1;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[ch][c] = make_double2(0.0, 0.0);
    auto entry = [&](int e) { return far[max(0, min(e + row, e1 - 1))]; };
    auto fetch = [&](int e, int2 ent) {
      Box B;
      const bool on = e + row < e1;
      B.pe = on ? (ent.y & 0xff) : 0;
      B.nq = on ? (ent.y >> 8) : 1;
      B.bb = bounds[ent.x];
      const double2* m = mom + (size_t)ent.x * p + j;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch)
#pragma unroll
        for (int c = 0; c < NC; ++c)
          B.a[ch][c] = 16 * ch + j < B.pe ? m[c * colstride + 16 * ch] : make_double2(0.0, 0.0);
      return B;
    };
    // the next four boxes' moments and the entries after them load during a step
    Box next{};
    int2 ent = make_int2(0, 0);
    if (e0 < e1) {
      next = fetch(e0, entry(e0));
      ent = entry(e0 + 4);
    }
    for (int e = e0; e < e1; e += 4) {
      const Box B = next;
      if (e + 4 < e1) {
        next = fetch(e + 4, ent);
        ent = entry(e + 8);
      }
      const double4 bb = B.bb;
      auto most_of = [&](int v) {
        return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                   max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
      };
      const int pm = most_of(B.pe), qm = most_of(B.nq);
      most = max(most, qm);
      const double dx = tt.x - bb.x, dy = tt.y - bb.y;
      const double d2 = __builtin_fma(dy, dy, dx * dx);
      double inv = refine_rcp(d2);
      inv = __builtin_fma(inv, __builtin_fma(-d2, inv, 1.0), inv);
      const double2 v = make_double2(dx * inv, -dy * inv);   // 1/D
      const double2 x = make_double2(v.x * bb.z, v.y * bb.z), y = make_double2(-v.x * tt.z, -v.y * tt.z);
      double2 x8, y8;
      const double2 X = zmul(power16(x, j, x8), v);
      double2 yl = power16(y, j, y8);
      double2 s[3][NC];
#pragma unroll
      for (int ch = 0; ch < 3; ++ch)
#pragma unroll
        for (int c = 0; c < NC; ++c) s[ch][c] = make_double2(0.0, 0.0);
      const double2 x16 = zsquare(x8);
      if (qm == 1) local_sums<1, NC>(s, B.a, X, x16, pm, tab + j);
      else if (qm == 2) local_sums<2, NC>(s, B.a, X, x16, pm, tab + j);
      else local_sums<3, NC>(s, B.a, X, x16, pm, tab + j);
#pragma unroll
      for (int ch = 0; ch < 3; ++ch)
        if (ch < qm) {
          if (ch > 0) yl = zmul(yl, zsquare(y8));
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const double2 u = zmul(yl, s[ch][c]);
            acc[ch][c].x += u.x;
            acc[ch][c].y += u.y;
          }
        }
    }
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        double2 u = acc[ch][c];
        u.x += __shfl_xor(u.x, 16, 64);
        u.y += __shfl_xor(u.y, 16, 64);
        u.x += __shfl_xor(u.x, 32, 64);
        u.y += __shfl_xor(u.y, 32, 64);
        if (row == 0) loc[((size_t)t * NC + c) * kLoc + 16 * ch + j] = u;
      }
    if (lane == 0) terms[t] = e1 > e0 ? 16 * most : 0;
  }
}

// One workgroup per (target tile, split), weight columns col .. col + NC - 1: wave
// wv takes the range 4 split + wv of 4 splits equal ranges (in fours) of the
// tile's near sources, leaf by leaf, summed directly. In the first split wave t
// adds the tile's local expansion at the targets of the lanes' t-th set. Partial
// sums go to slot split, like the direct kernels'.
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
using cptr = const __attribute__((address_space(4))) T*;   // read-only: scalar loads
#else
template <class T>
using cptr = const T*;
#endif

template <int TPT, int NC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NC == 1 ? 8 : 6))) void k_tree(
    const DomDev* __restrict__ doms, const int64_t* __restrict__ nearoff, const int* __restrict__ near_,
    const double4* __restrict__ tb, const double2* __restrict__ loc, const int* __restrict__ terms, int items,
    int tiles, int splits, int col, int wcols, const int* __restrict__ active, int lead, int ext, int curve,
    Pieces cut) {
  __shared__ double red[4][TPT][NC][2][64];
  const DomDev& D = doms[0];
  col += NC * blockIdx.y;
  loc += (size_t)blockIdx.y * NC * tiles * kLoc;
  if (active != nullptr) {
    bool any = false;
#pragma unroll
    for (int c = 0; c < NC; ++c) any = any || col + c < lead || active[D.c0 + col + c - lead] != 0;
    if (!any) return;
  }
  const int N = D.N;
  const int NT = ext ? D.Nt : N;   // targets: the points tz (ext) or the nodes
  const int item = xcd_order(blockIdx.x, gridDim.x);
  if (item >= items) return;
  const int tile = item / splits, g = item - tile * splits;
  const int base = cut.first(tile), end = cut.last(tile, NT);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int stride = D.slim ? slim_stride(wcols) : rec_stride(wcols);
  const int wo = (D.slim ? 1 : kRecHead) + col;
  const gptr<const double2> rec = (gptr<const double2>)D.rec;
  const cptr<int64_t> off = (cptr<int64_t>)nearoff + tile;
  const int n0 = (int)off[0];
  const int64_t units = 16 * (off[1] - n0);   // of four sources
  const int u0 = (int)(units * (4 * g + wv) / (4 * splits)) * 4;
  const int u1 = (int)(units * (4 * g + wv + 1) / (4 * splits)) * 4;

  double2 tg[TPT];
  int ti[TPT];
#pragma unroll
  for (int t = 0; t < TPT; ++t) {
    ti[t] = base + t * 64 + lane;
    tg[t] = ext ? D.tz[min(ti[t], end - 1)] : D.eta[min(ti[t], end - 1)];
  }
  Acc<NC, TPT> acc;
#pragma unroll
  for (int t = 0; t < TPT; ++t)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc.x[t][c] = acc.y[t][c] = 0.0;

  auto plain = [&](int ja, int jb) {
    int j = ja;
    for (; j + 3 < jb; j += 4) {
      gptr<const double2> r = rec + (size_t)j * stride;
      quad_step<NC, TPT>(acc, tg, r, r + stride, r + 2 * stride, r + 3 * stride, wo);
    }
    for (; j + 1 < jb; j += 2) {
      gptr<const double2> r = rec + (size_t)j * stride;
      pair_step<NC, TPT>(acc, tg, r, r + stride, wo);
    }
    if (j < jb) single_step<NC, TPT>(acc, tg, ti, rec + (size_t)j * stride, wo, j, false);
  };

  const cptr<int> nl = (cptr<int>)near_ + n0;
  for (int u = u0; u < u1;) {
    const int ue = min(u1, (u | 63) + 1);
    // (a short leaf ends its curve)
    const int v = nl[u >> 6], blk = v < 0 ? ~v : v;
    const int bend = v < 0 ? min(N, (blk / curve + 1) * curve) : blk + kLeaf;
    const int ja = min(bend, blk + (u & 63)), jb = min(bend, blk + ((ue - 1) & 63) + 1);
    u = ue;
    if (ext) {
      plain(ja, jb);
      continue;
    }
    plain(ja, min(jb, base));
    const int ma = max(ja, base), mb = min(jb, end);
    for (int j = ma; j < mb; ++j) single_step<NC, TPT>(acc, tg, ti, rec + (size_t)j * stride, wo, j, true);
    plain(max(ja, end), jb);
  }
#pragma unroll
  for (int t = 0; t < TPT; ++t)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      red[wv][t][c][0][lane] = acc.x[t][c];
      red[wv][t][c][1][lane] = acc.y[t][c];
    }
  __syncthreads();
  if (wv >= TPT) return;
  // wave t closes the sums of the t-th targets: the four waves' in order, then
  // the local expansion (Horner in (z - c_t)/r_t)
  double2 z = tg[0];
#pragma unroll
  for (int t = 1; t < TPT; ++t)
    if (wv == t) z = tg[t];
  const int i = base + wv * 64 + lane;
  const double4 tt = ((cptr<double4>)tb)[tile];
  const double inv = 1.0 / tt.z;
  const double zx = (z.x - tt.x) * inv, zy = (z.y - tt.y) * inv;
  const int nt = g == 0 ? ((cptr<int>)terms)[tile] : 0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    double x = 0.0, y = 0.0;
    const cptr<double2> L = (cptr<double2>)loc + ((size_t)tile * NC + c) * kLoc;
    for (int l = nt - 4; l >= 0; l -= 4) {
      const double2 l0 = L[l], l1 = L[l + 1], l2 = L[l + 2], l3 = L[l + 3];
      auto horner = [&](double2 a) {
        const double nx = __builtin_fma(zx, x, __builtin_fma(-zy, y, a.x));
        y = __builtin_fma(zx, y, __builtin_fma(zy, x, a.y));
        x = nx;
      };
      horner(l3);
      horner(l2);
      horner(l1);
      horner(l0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x += red[q][wv][c][0][lane];
      y += red[q][wv][c][1][lane];
    }
    if (i < end) D.parts[((size_t)g * wcols + col + c) * NT + i] = make_double2(x, y);
  }
}

// ------------------------------------------------ order along a Hilbert curve
// The points (or the centres of boxes) in the order of their positions along a
// Hilbert curve, 16 bits per coordinate over their bounding square, ties in
// index order: the curve has no jumps, so any run of consecutive entries lies in
// a compact region of the plane. The sort is bound by its launches: 0.2 ms for
// 200003 points (on the host about 15 ms of a 20.7 ms call).
constexpr int kMinMaxBlocks = 64;

__device__ __forceinline__ double2 point_at(const double2* pts, const double4* boxes, int i) {
  if (pts) return pts[i];
  const double4 b = boxes[i];
  return make_double2(0.5 * (b.x + b.y), 0.5 * (b.z + b.w));
}

// per block {xmin, xmax, ymin, ymax} of its share of the points
__global__ __launch_bounds__(256) void k_point_range(const double2* __restrict__ pts,
                                                     const double4* __restrict__ boxes, int n,
                                                     double4* __restrict__ range) {
  __shared__ double4 sh[4];
  double4 v = make_double4(1e300, -1e300, 1e300, -1e300);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double2 p = point_at(pts, boxes, i);
    v = make_double4(fmin(v.x, p.x), fmax(v.y, p.x), fmin(v.z, p.y), fmax(v.w, p.y));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.x = fmin(v.x, __shfl_xor(v.x, off, 64));
    v.y = fmax(v.y, __shfl_xor(v.y, off, 64));
    v.z = fmin(v.z, __shfl_xor(v.z, off, 64));
    v.w = fmax(v.w, __shfl_xor(v.w, off, 64));
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k)
      v = make_double4(fmin(v.x, sh[k].x), fmax(v.y, sh[k].y), fmin(v.z, sh[k].z), fmax(v.w, sh[k].w));
    range[blockIdx.x] = v;
  }
}

// position along the curve of cell (x, y) of the 2^16 x 2^16 grid
__device__ __forceinline__ uint32_t hilbert_position(uint32_t x, uint32_t y) {
  constexpr uint32_t side = 1u << 16;
  uint32_t d = 0;
  for (uint32_t h = side / 2; h > 0; h /= 2) {
    const uint32_t rx = (x & h) ? 1u : 0u, ry = (y & h) ? 1u : 0u;
    d += h * h * ((3u * rx) ^ ry);
    if (ry == 0) {   // rotate the quadrant
      if (rx == 1) {
        x = side - 1 - x;
        y = side - 1 - y;
      }
      const uint32_t t = x;
      x = y;
      y = t;
    }
  }
  return d;
}

// the points' bounding box from the blocks' (by every lane of a wave together)
__device__ __forceinline__ double4 whole_range(const double4* __restrict__ range) {
  static_assert(kMinMaxBlocks == 64, "one block's range per lane");
  double4 v = range[threadIdx.x & 63];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.x = fmin(v.x, __shfl_xor(v.x, off, 64));
    v.y = fmax(v.y, __shfl_xor(v.y, off, 64));
    v.z = fmin(v.z, __shfl_xor(v.z, off, 64));
    v.w = fmax(v.w, __shfl_xor(v.w, off, 64));
  }
  return v;
}

__device__ __forceinline__ uint32_t point_code(const double2* pts, const double4* boxes, int i, double4 v) {
  const double span = fmax(v.y - v.x, v.w - v.z);
  const double sc = span > 0.0 ? 65535.0 / span : 0.0;
  const double2 p = point_at(pts, boxes, i);
  const uint32_t qx = (uint32_t)fmin(65535.0, fmax(0.0, (p.x - v.x) * sc));
  const uint32_t qy = (uint32_t)fmin(65535.0, fmax(0.0, (p.y - v.z) * sc));
  return hilbert_position(qx, qy);
}

__global__ __launch_bounds__(256) void k_point_codes(const double2* __restrict__ pts,
                                                     const double4* __restrict__ boxes, int n,
                                                     const double4* __restrict__ range, uint32_t* __restrict__ key,
                                                     int* __restrict__ idx) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const double4 v = whole_range(range);
  if (i >= n) return;
  key[i] = point_code(pts, boxes, i, v);
  idx[i] = i;
}

// Up to kSmallSort points in one block: codes and indices as 64-bit keys
// (unique, so any sort keeps ties in index order), bitonic in LDS.
constexpr int kSmallSort = 4096;
__global__ __launch_bounds__(1024) void k_sort_small(const double2* __restrict__ pts,
                                                     const double4* __restrict__ boxes, int n,
                                                     const double4* __restrict__ range, int* __restrict__ perm) {
  __shared__ unsigned long long k[kSmallSort];
  const double4 v = whole_range(range);
  int m = 1;
  while (m < n) m *= 2;
  for (int i = threadIdx.x; i < m; i += blockDim.x)
    k[i] = i < n ? ((unsigned long long)point_code(pts, boxes, i, v) << 32) | (unsigned)i : ~0ull;
  __syncthreads();
  for (int len = 2; len <= m; len *= 2)
    for (int h = len / 2; h > 0; h /= 2) {
      for (int q = threadIdx.x; q < m / 2; q += blockDim.x) {
        const int a = 2 * h * (q / h) + q % h, b = a + h;
        const unsigned long long x = k[a], y = k[b];
        if ((x > y) == ((a & len) == 0)) {
          k[a] = y;
          k[b] = x;
        }
      }
      __syncthreads();
    }
  for (int i = threadIdx.x; i < n; i += blockDim.x) perm[i] = (int)(k[i] & 0xffffffffu);
}

// More points: least-significant-digit radix sort, eight bits a pass, stable.
// A block takes kSortTile consecutive entries in rounds of 256.
constexpr int kSortTile = 2048;
__global__ __launch_bounds__(256) void k_sort_count(const uint32_t* __restrict__ key, int n, int shift, int nblk,
                                                    int* __restrict__ hist) {
  __shared__ int cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int i0 = blockIdx.x * kSortTile;
  for (int r = 0; r < kSortTile; r += 256) {
    const int i = i0 + r + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(key[i] >> shift) & 255], 1);
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * nblk + blockIdx.x] = cnt[threadIdx.x];
}

// exclusive sums of v[0..n) in place, one block; the total to *total when given
template <class T>
__device__ __forceinline__ void block_scan(T* __restrict__ v, int64_t n, T* total) {
  __shared__ T wsum[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;   // 1024 threads
  T run = 0;
  for (int64_t base = 0; base < n; base += 4096) {
    T x[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = base + 4 * t + k;
      x[k] = i < n ? v[i] : (T)0;
      s += x[k];
    }
    T inc = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const T o = __shfl_up(inc, off, 64);
      if (lane >= off) inc += o;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    T before = run, all = 0;
    for (int k = 0; k < 16; ++k) {
      if (k < wv) before += wsum[k];
      all += wsum[k];
    }
    T e = before + inc - s;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = base + 4 * t + k;
      if (i < n) v[i] = e;
      e += x[k];
    }
    run += all;
    __syncthreads();
  }
  if (total && t == 0) *total = run;
}

__global__ __launch_bounds__(1024) void k_sort_scan(int* __restrict__ hist, int64_t n) {
  block_scan<int>(hist, n, nullptr);
}

__global__ __launch_bounds__(256) void k_sort_scatter(const uint32_t* __restrict__ key, const int* __restrict__ idx,
                                                      int n, int shift, int nblk, const int* __restrict__ hist,
                                                      uint32_t* __restrict__ key_out, int* __restrict__ idx_out) {
  __shared__ int next[256];       // where the block's next entry of a digit goes
  __shared__ int wcnt[4][256];    // entries of a digit in each wave of the round
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  next[t] = hist[(size_t)t * nblk + blockIdx.x];
  const int i0 = blockIdx.x * kSortTile;
  for (int r = 0; r < kSortTile && i0 + r < n; r += 256) {
    const int i = i0 + r + t;
    const bool in = i < n;
    const uint32_t k = in ? key[i] : 0u;
    const int dg = (k >> shift) & 255;
    for (int w = 0; w < 4; ++w) wcnt[w][t] = 0;
    __syncthreads();
    unsigned long long same = __ballot(in);   // lanes with this lane's digit
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const unsigned long long m = __ballot(in && ((dg >> b) & 1));
      same &= ((dg >> b) & 1) ? m : ~m;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    if (in && rank == 0) wcnt[wv][dg] = __popcll(same);
    __syncthreads();
    if (in) {
      int pos = next[dg] + rank;
      for (int w = 0; w < wv; ++w) pos += wcnt[w][dg];
      key_out[pos] = k;
      idx_out[pos] = idx[i];
    }
    __syncthreads();
    next[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
    __syncthreads();
  }
}

// --------------------------------------------------------- interaction lists
// One wavefront per target tile walks the boxes from the root, up to 64 of one
// level at a time (the stack holds at most 128 boxes of each level, since a level
// is pushed to only when nothing deeper is left). A box separated from the tile
// by (1 + theta)(r_t + r_b) becomes a far entry {box, p_e | chunks of 16 of q_e << 8}
// with the orders its own ratios need, a leaf that is not a near block (the index
// of its 64 nodes), any other box its two children. The first pass counts, the
// second writes. Bound by the latency of the box loads (on 16 host threads, with
// the copies both ways, the lists of 1089 x 4096 nodes took most of the 40 ms that
// a solve spent outside the GPU).
constexpr int kTreeLevels = 26;   // leaves < 2^25

struct TreeWalk {
  const double4* bounds;
  const double4* tb;
  const int* perm;
  int off[kTreeLevels + 1], nb[kTreeLevels + 1];
  double thr[kTreeMaxP + 1];   // far_tol^(1/k)
  double qthr[2];              // (far_tol/64)^(1/16), ^(1/32)
  double f2;                   // (1 + theta)^2
  int levels, p, N, NT, tiles;
  Pieces leaves, cut;
};

__device__ __forceinline__ int wave_prefix(int v, int lane, int* total) {
  int inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(inc, off, 64);
    if (lane >= off) inc += o;
  }
  *total = __shfl(inc, 63, 64);
  return inc - v;
}

template <bool FILL>
__global__ __launch_bounds__(256) void k_tree_lists(TreeWalk W, int64_t* __restrict__ nfar,
                                                    int64_t* __restrict__ nnear, double* __restrict__ work,
                                                    int2* __restrict__ far, int* __restrict__ near_) {
  extern __shared__ int stk[];                // 128 levels boxes per wave, deepest level last
  __shared__ int left[4][kTreeLevels];        // boxes of each level on the stack
  __shared__ double thr[kTreeMaxP + 1];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x <= (unsigned)W.p) thr[threadIdx.x] = W.thr[threadIdx.x];
  __syncthreads();
  const int t = blockIdx.x * 4 + wv;
  if (t >= W.tiles) return;
  int* st = stk + wv * 128 * W.levels;
  int* cnt = left[wv];
  const double4 tt = W.tb[t];
  const double nt = (double)(W.cut.last(t, W.NT) - W.cut.first(t));
  int64_t f = FILL ? nfar[t] : 0, n = FILL ? nnear[t] : 0;
  double wk = 0.0;
  int l = W.levels - 1, sp = 1;   // level of the stack's top, boxes on it
  if (lane < W.levels) cnt[lane] = lane == l ? 1 : 0;
  if (lane == 0) st[0] = 0;
  auto fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  fence();
  while (sp > 0) {
    const int have = __builtin_amdgcn_readfirstlane(cnt[l]);
    const int take = min(64, have);
    const int b = lane < take ? st[sp - 1 - lane] : 0;
    sp -= take;
    const int g = W.off[l] + b;
    bool is_far = false, is_near = false;
    int pe = 2, nq = 1, nch = 0;
    if (lane < take) {
      const double4 bb = W.bounds[g];
      const double dx = tt.x - bb.x, dy = tt.y - bb.y, rr = tt.z + bb.z;
      const double d2 = dx * dx + dy * dy;
      if (d2 > W.f2 * rr * rr) {
        is_far = true;
        const double d = sqrt(d2), rho = bb.z / (d - tt.z), rq = tt.z / (d - bb.z);
        while (pe < W.p && rho > thr[pe]) ++pe;
        nq = rq <= W.qthr[0] ? 1 : (rq <= W.qthr[1] ? 2 : 3);
        if (!FILL) wk += 64.0 * pe * nq;
      } else if (l == 0) {
        is_near = true;
        if (!FILL) wk += 16.0 * nt * (W.leaves.last(W.perm[b], W.N) - W.leaves.first(W.perm[b]));
      } else {
        nch = 2 * b + 1 < W.nb[l - 1] ? 2 : 1;
      }
    }
    const unsigned long long below = (1ull << lane) - 1ull, mf = __ballot(is_far), mn = __ballot(is_near);
    if (FILL) {
      if (is_far) far[f + __popcll(mf & below)] = make_int2(g, pe | (nq << 8));
      if (is_near) {
        const int a = W.leaves.first(W.perm[b]);
        near_[n + __popcll(mn & below)] = W.leaves.last(W.perm[b], W.N) - a < kLeaf ? ~a : a;
      }
    }
    f += __popcll(mf);
    n += __popcll(mn);
    int th;
    const int ph = wave_prefix(nch, lane, &th);
    // a box's children keep their order when they come off the stack
    for (int q = 0; q < nch; ++q) st[sp + th - 1 - ph - q] = 2 * b + q;
    sp += th;
    if (lane == 0) {
      cnt[l] = have - take;
      if (th > 0) cnt[l - 1] = th;   // (nothing of that level was left)
    }
    fence();
    if (th > 0) --l;
    else while (l + 1 < W.levels && __builtin_amdgcn_readfirstlane(cnt[l]) == 0) ++l;
  }
  if constexpr (!FILL) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wk += __shfl_xor(wk, off, 64);
    if (lane == 0) {
      nfar[t] = f;
      nnear[t] = n;
      work[t] = wk + (f > 0 ? 8.0 * kLoc * nt : 0.0);
    }
  }
}

// counts to offsets, the totals behind them and in host-mapped memory
__global__ __launch_bounds__(1024) void k_list_offsets(int64_t* __restrict__ nfar, int64_t* __restrict__ nnear,
                                                       int tiles, int64_t* total) {
  int64_t* v = blockIdx.x == 0 ? nfar : nnear;
  int64_t sum = 0;
  block_scan<int64_t>(v, tiles, &sum);
  if (threadIdx.x == 0) {
    v[tiles] = sum;
    total[blockIdx.x] = sum;
  }
}

}  // namespace

// scratch: 2 n uint32 keys, n ints, 256 ceil(n / 2048) ints, kMinMaxBlocks double4
size_t hilbert_scratch(int64_t n) {
  const int64_t nblk = (n + kSortTile - 1) / kSortTile;
  return (size_t)(n <= kSmallSort ? 0 : 12 * n + 1024 * nblk) + kMinMaxBlocks * sizeof(double4);
}

hipError_t launch_hilbert_order(const double2* pts, const double4* boxes, int n, void* scratch, int* perm,
                                hipStream_t st) {
  double4* range = static_cast<double4*>(scratch);
  k_point_range<<<kMinMaxBlocks, 256, 0, st>>>(pts, boxes, n, range);
  if (n <= kSmallSort) {
    k_sort_small<<<1, 1024, 0, st>>>(pts, boxes, n, range, perm);
    return hipGetLastError();
  }
  const int nblk = (n + kSortTile - 1) / kSortTile;
  uint32_t* key[2] = {reinterpret_cast<uint32_t*>(range + kMinMaxBlocks), nullptr};
  key[1] = key[0] + n;
  int* idx[2] = {perm, reinterpret_cast<int*>(key[1] + n)};   // four passes: back in perm
  int* hist = idx[1] + n;
  k_point_codes<<<(n + 255) / 256, 256, 0, st>>>(pts, boxes, n, range, key[0], idx[0]);
  for (int pass = 0; pass < 4; ++pass) {
    const int a = pass & 1, b = a ^ 1;
    k_sort_count<<<nblk, 256, 0, st>>>(key[a], n, 8 * pass, nblk, hist);
    k_sort_scan<<<1, 1024, 0, st>>>(hist, (int64_t)256 * nblk);
    k_sort_scatter<<<nblk, 256, 0, st>>>(key[a], idx[a], n, 8 * pass, nblk, hist, key[b], idx[b]);
  }
  return hipGetLastError();
}

static TreeWalk tree_walk(const TreeListArgs& A) {
  TreeWalk W{};
  W.bounds = A.bounds;
  W.tb = A.tb;
  W.perm = A.perm;
  for (int l = 0; l < A.levels; ++l) {
    W.off[l] = A.level_off[l];
    W.nb[l] = A.level_nb[l];
  }
  // rho^k <= far_tol exactly when rho <= far_tol^(1/k): the order of a far
  // entry is the least k >= 2 (at most p) whose threshold its ratio meets
  for (int k = 1; k <= A.p; ++k) W.thr[k] = std::pow(A.far_tol, 1.0 / k);
  W.qthr[0] = std::pow(A.far_tol / 64.0, 1.0 / 16.0);
  W.qthr[1] = std::pow(A.far_tol / 64.0, 1.0 / 32.0);
  W.f2 = (1.0 + A.theta) * (1.0 + A.theta);
  W.levels = A.levels;
  W.p = A.p;
  W.N = A.N;
  W.NT = A.NT;
  W.tiles = A.tiles;
  W.leaves = A.leaves;
  W.cut = A.cut;
  return W;
}

hipError_t launch_tree_count(const TreeListArgs& A, int64_t* nfar, int64_t* nnear, double* work, int64_t* total,
                             hipStream_t st) {
  if (A.levels < 1 || A.levels > kTreeLevels || A.p > kTreeMaxP) return hipErrorInvalidValue;
  k_tree_lists<false><<<(A.tiles + 3) / 4, 256, 4 * 128 * sizeof(int) * A.levels, st>>>(tree_walk(A), nfar, nnear,
                                                                                        work, nullptr, nullptr);
  k_list_offsets<<<2, 1024, 0, st>>>(nfar, nnear, A.tiles, total);
  return hipGetLastError();
}

hipError_t launch_tree_fill(const TreeListArgs& A, int64_t* nfar, int64_t* nnear, int2* far, int* near_,
                            hipStream_t st) {
  k_tree_lists<true><<<(A.tiles + 3) / 4, 256, 4 * 128 * sizeof(int) * A.levels, st>>>(tree_walk(A), nfar, nnear,
                                                                                       nullptr, far, near_);
  return hipGetLastError();
}

hipError_t launch_leaf_boxes(const double2* eta, int N, Pieces leaves, int nleaf, double4* leafbox, hipStream_t st) {
  k_leaf_bbox<<<nleaf, 64, 0, st>>>(eta, N, leaves, leafbox);
  return hipGetLastError();
}

hipError_t launch_piece_circles(const double2* eta, int N, Pieces tiles, int count, double4* out, hipStream_t st) {
  k_piece_circles<<<count, 64, 0, st>>>(eta, N, tiles, out);
  return hipGetLastError();
}

hipError_t launch_box_bounds(const double2* eta, int N, Pieces leaves, const int* level_off, const int* level_nb,
                             int levels, const double4* leafbox, const int* perm, double4* bbox,
                             unsigned long long* rbits, double4* out, hipStream_t st) {
  if (levels < 1 || levels > 32) return hipErrorInvalidValue;
  k_bbox_gather<<<(level_nb[0] + 255) / 256, 256, 0, st>>>(leafbox, perm, level_nb[0], bbox);
  hipError_t e = hipGetLastError();
  for (int l = 0; l + 1 < levels && e == hipSuccess; ++l) {
    const int npar = level_nb[l + 1];
    k_bbox_merge<<<(npar + 255) / 256, 256, 0, st>>>(bbox + level_off[l], level_nb[l], bbox + level_off[l + 1], npar);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  const int nbox = level_off[levels - 1] + level_nb[levels - 1];
  k_box_centres<<<(nbox + 255) / 256, 256, 0, st>>>(bbox, nbox, out, rbits);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  LevelTable lv{};
  for (int l = 0; l < levels; ++l) lv.off[l] = level_off[l];
  k_box_radii<<<(level_nb[0] + kRadiiWaves - 1) / kRadiiWaves, 64 * kRadiiWaves, 0, st>>>(
      eta, N, leaves, lv, levels, level_nb[0], perm, out, rbits);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_box_finish<<<(nbox + 255) / 256, 256, 0, st>>>(rbits, nbox, out);
  return hipGetLastError();
}

hipError_t launch_tree_moments(const double2* rec, int stride, int wo, int ncols, int N, Pieces leaves,
                               const double4* bounds,
                               const int* perm, const int* level_off, const int* level_nb, int levels, int p,
                               double2* mom, size_t colstride, const double* binom, const int* active,
                               hipStream_t st) {
  if (levels > 32 || p > kTreeMaxP) return hipErrorInvalidValue;
  LevelTable lt{};
  for (int l = 0; l < levels; ++l) {
    lt.off[l] = level_off[l];
    lt.nb[l] = level_nb[l];
  }
  // instances for 12, 24, 36 and 48 terms (four lanes' shares of a leaf's moments)
  auto run = [&](auto terms) {
    constexpr int P = decltype(terms)::value;
    const dim3 grid((unsigned)((level_nb[0] + 15) / 16), (unsigned)ncols);
    k_leaf_moments<P / 4><<<grid, 64, 0, st>>>(rec, stride, wo, N, leaves, bounds, perm, level_nb[0], p, mom, colstride,
                                               active);
    for (int l = 0; l + 1 < levels;) {
      const int nlev = std::min(kM2MLevels, levels - 1 - l);
      const dim3 g((unsigned)((level_nb[l] + 63) / 64), (unsigned)ncols);
      k_m2m_levels<P><<<g, kM2MT, 0, st>>>(bounds, lt, l, nlev, p, mom, colstride, binom, active);
      l += nlev;
    }
  };
  if (p <= 12) run(std::integral_constant<int, 12>{});
  else if (p <= 24) run(std::integral_constant<int, 24>{});
  else if (p <= 36) run(std::integral_constant<int, 36>{});
  else run(std::integral_constant<int, 48>{});
  return hipGetLastError();
}

std::vector<double> tree_binomials() {
  std::vector<double> b((size_t)kLoc * kLoc);
  for (int k = 0; k < kLoc; ++k)
    for (int l = 0; l < kLoc; ++l)
      b[k * kLoc + l] = k == 0 || l == 0 ? 1.0 : b[(k - 1) * kLoc + l] + b[k * kLoc + l - 1];
  return b;
}

hipError_t launch_tree_eval(const DomDev* doms, int tiles, int tpt, const TreeEvalArgs& A, int ncols, int splits,
                            int col, int wcols, const int* active, int lead, bool ext, const int* flag,
                            hipStream_t st) {
  const int groups = ((tiles + 3) / 4 + 7) & ~7, items = tiles * splits;
  const unsigned lg = (unsigned)std::min(groups, 4096), grid = (unsigned)((items + 7) & ~7);
  const int e = ext ? 1 : 0;
  // the columns in twos, the last of an odd number alone
  const int pairs = ncols / 2;
  auto run = [&](auto two, int c0, int ny) {
    constexpr int NC = decltype(two)::value;
    const double2* mom = A.mom + c0 * A.colstride;
    double2* loc = A.loc + (size_t)c0 * tiles * kLoc;
    k_tile_locals<NC><<<dim3(lg, (unsigned)ny), 256, 0, st>>>(A.tb, tiles, A.faroff, A.far, A.bounds, mom, A.colstride,
                                                              A.p, A.binom, loc, A.terms,
                                                              flag ? flag + c0 : nullptr);
    auto eval = [&](auto kern) {
      kern<<<dim3(grid, (unsigned)ny), 256, 0, st>>>(doms, A.nearoff, A.near, A.tb, loc, A.terms, items, tiles, splits,
                                                     col + c0, wcols, active, lead, e, A.leaves.n, A.cut);
    };
    if (tpt == 2) eval(k_tree<2, NC>);
    else eval(k_tree<1, NC>);
  };
  if (pairs > 0) run(std::integral_constant<int, 2>{}, 0, pairs);
  if (ncols & 1) run(std::integral_constant<int, 1>{}, ncols - 1, 1);
  return hipGetLastError();
}

}  // namespace gnk
