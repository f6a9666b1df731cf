// One-column FP64 Cauchy sums with every unordered pair of nodes evaluated
// once: S_i += w_j q and S_j -= w_i q from the same q = 1/(eta_i - eta_j).
//
// The direct sum is bound by FP64 VALU issue, and a third to a half of the
// one-sided kernel's operations per pair (k_pairs in cauchy.hip: 9.75 far, 13
// near) go into the distance and the reciprocal. Here these serve both nodes:
// per unordered pair a far tile takes 3 (distance) + 2.75 (a quarter of the
// shared reciprocal) + 8 (four FMAs per side) = 13.75, a near one 16.75, so
// 6.9 and 8.4 per (target, source).
//
// Mapping. A wavefront owns 64 T consecutive nodes, T per lane in registers
// with their weights; a workgroup of four waves owns a block of 256 T nodes.
// It streams the other blocks' nodes in chunks of 64, which lie in LDS: in
// step r = 0..63 of a chunk, lane l meets chunk node (l + r) mod 64, so that in
// each step the 64 lanes hold 64 different stream nodes and each of these
// nodes' sums sits in one lane, which hands it to its neighbour after the step
// (wave_rol; back in its own lane after 64 steps). The arrays in LDS are doubled,
// entry k + 64 standing for entry k, so that l + r needs no wrap. The owned
// nodes' sums stay in registers for the chunk. T = 8 (two waves per SIMD): 112
// FP64 operations and 9 others per step; T = 4 (three waves): 56 and 9. With T = 8
// 256 registers do not hold everything: 24 are spilled (68 bytes a lane), between the
// chunks but for three accesses per two far steps, which the FP64 issue covers; at
// N = 264192 12 % of the bytes written are not partial sums, but such registers.
//
// Measured (one column, launch us, one-sided / two-sided): 126 / 96 at N = 17408,
// 407 / 318 at 33792, 1695 / 1415 at 73729. At the last the VALU is busy 93 % of
// the cycles at 1.93 GHz, where the one-sided kernel ran at 2.08: the power limit
// sets the clock, so that operations and bytes count more than issue slots
// (sums of the stream nodes kept in LDS: 1526 us at 83 % and 1.90 GHz; stream
// nodes by scalar loads and their sums folded over the lanes by permlane swaps:
// 1549 us).
//
// Far chunks (all T 64-node tiles of the wave separated from the chunk's as in
// k_pairs' far form): coordinates relative to the chunk's centre c, z' = z_i - c
// and e' = eta_j - c, m = 1/|z' - e'|^2 from |z'|^2 + |e'|^2 - 2 z'.e':
//   S_i += conj(z') sum_j w_j m - sum_j w_j conj(e'_j) m
//   S_j += conj(e') sum_i w_i m - sum_i w_i conj(z'_i) m
// (the rounding that the differences amplify is bounded as for k_pairs). The
// other chunks take q = conj(d) m from d = z_i - eta_j itself.
//
// Which pairs: with nb blocks, block I streams the blocks I + 1 .. I + nb/2
// (mod nb; for even nb the last one only if I < nb/2), which covers every
// pair of different blocks once. Inside a block, wave tile w streams tile
// w + 1 (mod 4), tiles 0 and 1 also tiles 2 and 3, and each tile its own nodes
// one-sidedly (j != i). Every result is a partial sum in a slot of its own:
//   slots 0 .. F - 1          the block's items (ranges of its stream)
//   F .. F + H - 1            from the block d = 1..H before it
//   F + H .. F + H + P - 1    the P parts of the block's own pairs (3 T tasks)
//   F + H + P, F + H + P + 1  from the tiles one and two before it in the block
// which the consumer adds in this order: results are bitwise reproducible.
#include "gnk_device.h"
#include "gnk_internal.h"

namespace gnk {

namespace {

// Registers of the owned nodes and the wave's LDS area.
template <int T>
struct SymLds {
  double2 u[128], w[128], b[128];   // stream: -2 e' (far) or eta (near), weight, w conj(e')
  double a[128];                    // |e'|^2
  double2 s[64 * T];                // the owned nodes' sums
};

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// m[v] = 1/d[v], one reciprocal for the four (the product stays in range while
// every d lies in [1e-75, 1e75])
__device__ __forceinline__ void inverse4(const double (&d)[4], double (&m)[4]) {
  const double p0 = d[0] * d[1], p1 = d[2] * d[3];
  const double R = refine_rcp(p0 * p1);
  const double r0 = R * p1, r1 = R * p0;
  m[0] = r0 * d[1];
  m[1] = r0 * d[0];
  m[2] = r1 * d[3];
  m[3] = r1 * d[2];
}

// the same with a reciprocal for each: one zero distance leaves the others' inverses
__device__ __forceinline__ void inverse4_apart(const double (&d)[4], double (&m)[4]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) m[v] = refine_rcp(d[v]);
}

__device__ __forceinline__ double2 zmul_conj(double2 a, double2 b) {   // a conj(b)
  return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// the value of the next lane (lane 63: of lane 0)
__device__ __forceinline__ double from_next_lane(double v) {
  const int2 p = __builtin_bit_cast(int2, v);
  int2 q;
  q.x = __builtin_amdgcn_mov_dpp(p.x, 0x134, 0xf, 0xf, false);
  q.y = __builtin_amdgcn_mov_dpp(p.y, 0x134, 0xf, 0xf, false);
  return __builtin_bit_cast(double, q);
}
__device__ __forceinline__ double2 from_next_lane(double2 v) {
  return make_double2(from_next_lane(v.x), from_next_lane(v.y));
}

struct SymNodes {
  gptr<const double2> eta, w;
  int N;
};

__device__ __forceinline__ double2 node_at(const SymNodes& g, int i) { return g.eta[i]; }
__device__ __forceinline__ double2 weight_at(const SymNodes& g, int i) { return g.w[i]; }

// The chunk's 64 nodes against the wave's 64 T, far form. Returns the sum of
// chunk node `lane` (of the chunk) over the wave's nodes.
template <int T>
__device__ __forceinline__ double2 chunk_far(const SymNodes& g, SymLds<T>& L, int own0, int chunk, double2 c) {
  const int lane = threadIdx.x & 63;
  const int j = chunk * 64 + lane;
  const double2 e = node_at(g, min(j, g.N - 1));
  const double2 ep = make_double2(e.x - c.x, e.y - c.y);
  {
    const double2 wj = j < g.N ? weight_at(g, j) : make_double2(0.0, 0.0);
    L.u[lane] = L.u[lane + 64] = make_double2(-2.0 * ep.x, -2.0 * ep.y);
    L.w[lane] = L.w[lane + 64] = wj;
    L.b[lane] = L.b[lane + 64] = zmul_conj(wj, ep);
    L.a[lane] = L.a[lane + 64] = __builtin_fma(ep.y, ep.y, ep.x * ep.x);
  }
  double zx[T], zy[T], zz[T], wx[T], wy[T], bx[T], by[T];
  double ax[T], ay[T], cx[T], cy[T];   // sums of w m and of b m
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int i = own0 + t * 64 + lane;
    const double2 z = node_at(g, min(i, g.N - 1));
    const double2 w = i < g.N ? weight_at(g, i) : make_double2(0.0, 0.0);
    zx[t] = z.x - c.x;
    zy[t] = z.y - c.y;
    zz[t] = __builtin_fma(zy[t], zy[t], zx[t] * zx[t]);
    wx[t] = w.x;
    wy[t] = w.y;
    const double2 b = zmul_conj(w, make_double2(zx[t], zy[t]));
    bx[t] = b.x;
    by[t] = b.y;
    ax[t] = ay[t] = cx[t] = cy[t] = 0.0;
  }
  wave_fence();
  double2 u = L.u[lane], w = L.w[lane], b = L.b[lane];
  double a = L.a[lane];
  double2 ra = make_double2(0.0, 0.0), rb = ra;
#pragma unroll 2
  for (int r = 0; r < 64; ++r) {
    const int k = lane + r;
    const double2 un = L.u[k + 1], wn = L.w[k + 1], bn = L.b[k + 1];
    const double an = L.a[k + 1];
#pragma unroll
    for (int t = 0; t < T; t += 4) {
      double d[4], m[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) d[v] = __builtin_fma(u.x, zx[t + v], __builtin_fma(u.y, zy[t + v], a + zz[t + v]));
      inverse4(d, m);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        ax[t + v] = __builtin_fma(w.x, m[v], ax[t + v]);
        ay[t + v] = __builtin_fma(w.y, m[v], ay[t + v]);
        cx[t + v] = __builtin_fma(b.x, m[v], cx[t + v]);
        cy[t + v] = __builtin_fma(b.y, m[v], cy[t + v]);
        ra.x = __builtin_fma(wx[t + v], m[v], ra.x);
        ra.y = __builtin_fma(wy[t + v], m[v], ra.y);
        rb.x = __builtin_fma(bx[t + v], m[v], rb.x);
        rb.y = __builtin_fma(by[t + v], m[v], rb.y);
      }
    }
    ra = from_next_lane(ra);
    rb = from_next_lane(rb);
    u = un;
    w = wn;
    b = bn;
    a = an;
  }
#pragma unroll
  for (int t = 0; t < T; ++t) {
    double2 s = L.s[t * 64 + lane];
    s.x += __builtin_fma(zx[t], ax[t], zy[t] * ay[t]) - cx[t];
    s.y += __builtin_fma(zx[t], ay[t], -zy[t] * ax[t]) - cy[t];
    L.s[t * 64 + lane] = s;
  }
  const double2 out = make_double2(__builtin_fma(ep.x, ra.x, ep.y * ra.y) - rb.x,
                                   __builtin_fma(ep.x, ra.y, -ep.y * ra.x) - rb.y);
  wave_fence();   // the next chunk overwrites the area
  return out;
}

// The 64 steps of the plain form: adds to the owned nodes' sums sx, sy and returns
// the sum of the lane's stream node. SELF: the chunk lies in the wave's own tile; one
// side only, and pairs of equal (clamped) node indices are left out.
template <int T, bool SELF, bool APART>
__device__ __forceinline__ double2 near_steps(const SymNodes& g, const SymLds<T>& L, int own0, int chunk,
                                              const double (&zx)[T], const double (&zy)[T], const double (&wx)[T],
                                              const double (&wy)[T], double (&sx)[T], double (&sy)[T]) {
  const int lane = threadIdx.x & 63;
  double2 e = L.u[lane], w = L.w[lane];
  double2 ra = make_double2(0.0, 0.0);
#pragma unroll 2
  for (int r = 0; r < 64; ++r) {
    const int k = lane + r;
    const double2 en = L.u[k + 1], wn = L.w[k + 1];
    const int jk = min(chunk * 64 + (k & 63), g.N - 1);
#pragma unroll
    for (int t = 0; t < T; t += 4) {
      double dx[4], dy[4], d[4], m[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dx[v] = zx[t + v] - e.x;
        dy[v] = zy[t + v] - e.y;
        d[v] = __builtin_fma(dy[v], dy[v], dx[v] * dx[v]);
        // equal nodes: q = 0 from dx = dy = 0 and a finite m
        if constexpr (SELF) d[v] = (min(own0 + (t + v) * 64 + lane, g.N - 1) == jk) ? 1.0 : d[v];
      }
      if constexpr (APART) inverse4_apart(d, m);
      else inverse4(d, m);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double qx = dx[v] * m[v], qy = -dy[v] * m[v];
        sx[t + v] = __builtin_fma(w.x, qx, sx[t + v]);
        sx[t + v] = __builtin_fma(-w.y, qy, sx[t + v]);
        sy[t + v] = __builtin_fma(w.x, qy, sy[t + v]);
        sy[t + v] = __builtin_fma(w.y, qx, sy[t + v]);
        if constexpr (!SELF) {
          ra.x = __builtin_fma(-wx[t + v], qx, ra.x);
          ra.x = __builtin_fma(wy[t + v], qy, ra.x);
          ra.y = __builtin_fma(-wx[t + v], qy, ra.y);
          ra.y = __builtin_fma(-wy[t + v], qx, ra.y);
        }
      }
    }
    if constexpr (!SELF) ra = from_next_lane(ra);
    e = en;
    w = wn;
  }
  return ra;
}

// The chunk's 64 nodes against the wave's 64 T in the plain form. Two nodes in one
// place spoil the reciprocal that four of a lane's nodes share: a chunk that leaves a
// sum non-finite is taken again with a reciprocal for each pair, which keeps that to
// the two nodes' own sums.
template <int T, bool SELF>
__device__ __forceinline__ double2 chunk_near(const SymNodes& g, SymLds<T>& L, int own0, int chunk) {
  const int lane = threadIdx.x & 63;
  const int j = chunk * 64 + lane;
  {
    const double2 e = node_at(g, min(j, g.N - 1));
    const double2 wj = j < g.N ? weight_at(g, j) : make_double2(0.0, 0.0);
    L.u[lane] = L.u[lane + 64] = e;
    L.w[lane] = L.w[lane + 64] = wj;
  }
  double zx[T], zy[T], wx[T], wy[T], sx[T], sy[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int i = own0 + t * 64 + lane;
    const double2 z = node_at(g, min(i, g.N - 1));
    const double2 w = i < g.N ? weight_at(g, i) : make_double2(0.0, 0.0);
    zx[t] = z.x;
    zy[t] = z.y;
    wx[t] = w.x;
    wy[t] = w.y;
  }
  auto start = [&] {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const double2 s = L.s[t * 64 + lane];
      sx[t] = s.x;
      sy[t] = s.y;
    }
  };
  start();
  wave_fence();
  double2 ra = near_steps<T, SELF, false>(g, L, own0, chunk, zx, zy, wx, wy, sx, sy);
  double all = ra.x + ra.y;
#pragma unroll
  for (int t = 0; t < T; ++t) all += sx[t] + sy[t];
  if (__any(!isfinite(all))) {
    start();
    ra = near_steps<T, SELF, true>(g, L, own0, chunk, zx, zy, wx, wy, sx, sy);
  }
#pragma unroll
  for (int t = 0; t < T; ++t) L.s[t * 64 + lane] = make_double2(sx[t], sy[t]);
  wave_fence();
  return ra;
}

// both sides of (wave tile, chunk): far form where every 64-node tile of the
// wave is separated from the chunk's
template <int T>
__device__ __forceinline__ double2 chunk_pair(const SymNodes& g, SymLds<T>& L, gptr<const double4> sb, double far2,
                                              int own0, int chunk, int nchunk) {
  const int lane = threadIdx.x & 63;
  const double4 cb = sb[chunk];
  bool far = true;
  const int tile = own0 / 64 + lane;
  if (lane < T && tile < nchunk) {
    const double4 tb = sb[tile];
    const double dx = tb.x - cb.x, dy = tb.y - cb.y, rr = tb.z + cb.z;
    far = dx * dx + dy * dy > far2 * rr * rr;
  }
  if (__all(far)) return chunk_far<T>(g, L, own0, chunk, make_double2(cb.x, cb.y));
  return chunk_near<T, false>(g, L, own0, chunk);
}

// item {block, first, end, slot}: stream chunks [first, end) of the block's
// stream into forward slot `slot`; slot < 0: part `first` of `end` parts of the
// block's own pairs.
template <int T>
__global__ __launch_bounds__(256, T == 8 ? 2 : 3) void k_pairs_sym(const DomDev* __restrict__ doms,
                                                                   const int4* __restrict__ items, SymPlan P,
                                                                   const int* __restrict__ active) {
  __shared__ SymLds<T> lds[4];
  __shared__ double2 xch[4][64];
  const DomDev& D = doms[0];
  if (active != nullptr && active[D.c0] == 0) return;
  const int4 it = items[blockIdx.x];
  const int N = D.N;
  const SymNodes g{(gptr<const double2>)D.eta, (gptr<const double2>)D.w1, N};
  const gptr<const double4> sb = (gptr<const double4>)D.sb;
  const gptr<double2> part = (gptr<double2>)D.parts;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SymLds<T>& L = lds[wv];
  const int nchunk = (N + 63) / 64;
  const int tile0 = 4 * it.x;                 // the block's first wave tile
  const int own0 = (tile0 + wv) * 64 * T;
  const double far2 = D.far2d;
#pragma unroll
  for (int t = 0; t < T; ++t) L.s[t * 64 + lane] = make_double2(0.0, 0.0);
  auto put = [&](int slot, int i, double2 v) {
    typedef double nt2 __attribute__((ext_vector_type(2)));
    if (i < N) __builtin_nontemporal_store(nt2{v.x, v.y}, (gptr<nt2>)(part + (size_t)slot * N + i));
  };
  int slot = it.w;
  if (slot >= 0) {
    const int c0 = it.x + 1 == P.nb ? 0 : (it.x + 1) * 4 * T;
    for (int q = it.y; q < it.z; ++q) {
      int c = c0 + q;
      c -= c >= nchunk ? nchunk : 0;
      int d = c / (4 * T) - it.x;
      d += d < 0 ? P.nb : 0;
      // (a wave past the last node has no tile whose distance would tell far from near)
      xch[wv][lane] = own0 < N ? chunk_pair<T>(g, L, sb, far2, own0, c, nchunk) : make_double2(0.0, 0.0);
      __syncthreads();
      if (wv == (q & 3)) {
        const double2 a0 = xch[0][lane], a1 = xch[1][lane], a2 = xch[2][lane], a3 = xch[3][lane];
        put(P.F + d - 1, c * 64 + lane, make_double2((a0.x + a1.x) + (a2.x + a3.x), (a0.y + a1.y) + (a2.y + a3.y)));
      }
      __syncthreads();
    }
  } else {
    // 3 T tasks: chunk lc of the wave's own tile, of the tile one on and (first
    // two tiles) two on; a tile without nodes adds nothing to the others, whose
    // slots are written all the same
    slot = P.F + P.H + it.y;
    const int back = P.F + P.H + P.P;
    for (int task = it.y; task < 3 * T; task += it.z) {
      const int k = task / T, lc = task - k * T;
      if (k == 0) {
        const int c = (tile0 + wv) * T + lc;
        if (c < nchunk) {
          (void)chunk_near<T, true>(g, L, own0, c);
          // even block counts: the last backward slot is empty for the first half
          if (P.nb % 2 == 0 && it.x < P.nb / 2) put(P.F + P.H - 1, c * 64 + lane, make_double2(0.0, 0.0));
        }
      } else {
        const int c = (tile0 + (k == 1 ? ((wv + 1) & 3) : (wv ^ 2))) * T + lc;
        if (c < nchunk)
          put(back + k - 1, c * 64 + lane,
              own0 < N && (k == 1 || wv < 2) ? chunk_pair<T>(g, L, sb, far2, own0, c, nchunk)
                                              : make_double2(0.0, 0.0));
      }
    }
  }
#pragma unroll
  for (int t = 0; t < T; ++t) put(slot, own0 + t * 64 + lane, L.s[t * 64 + lane]);
}

}  // namespace

hipError_t launch_pairs_sym(const DomDev* doms, const int4* items, int nitems, const SymPlan& P, const int* active,
                            hipStream_t st) {
  if (P.T == 8) k_pairs_sym<8><<<nitems, 256, 0, st>>>(doms, items, P, active);
  else k_pairs_sym<4><<<nitems, 256, 0, st>>>(doms, items, P, active);
  return hipGetLastError();
}

}  // namespace gnk
