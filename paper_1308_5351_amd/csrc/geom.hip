// Derivatives of the discrete operators with respect to the boundary data, and
// Fourier boundary curves with their reverse-mode derivative.
//
// Geometry. Every geometry-dependent entry of f_B = 2I + diag(B1) - B and of
// fC = D - diag(D1) + Lhat comes from K_ij = (2/n) a_i b_j / (eta_j - eta_i),
// a = A, b = eta'/A (B = Im K, D = Re K, eqs. (e:B), (e:M); Lhat depends on n
// only). For s = sum_t c_t u_t^T Op_t v_t (Op_t = f_B or fC, u_t, v_t real)
//   s = const + Re sum_{i != j} K_ij W_ij,  W_ij = sum_t z_t u_t,i (v_t,j - v_t,i),
// with z_t = i c_t for f_B (B = Re(-i K), and the rows of diag(B1) - B give
// u_i (v_i - v_j)) and z_t = c_t for fC. Grouping the terms by v (groups g with
// vector V_g and U_g = sum_{t in g} z_t u_t, P = sum_g U_g V_g), the partial
// derivatives of F = sum_{i != j} K_ij W_ij need only row and column sums: with
// S1(w)_i = sum_{j != i} w_j/(eta_i - eta_j) (the matrix E of eq. (e:fmm-E)),
// kappa = 2/n, q = 1/(eta_i - eta_j) and e_g = V_g,i - V_g,j,
//   R1_i = sum_j K_ij W_ij = kappa a_i sum_g U_g,i F1_g,i,   F1_g,i = sum_j b_j e_g q
//   R2_i = sum_j K_ij W_ij / (eta_j - eta_i) = -kappa a_i sum_g U_g,i F2_g,i  (q^2 for q)
//   T1_i = sum_g V_g,i S1(a U_g)_i - S1(a P)_i = sum_j X q,  X = sum_g (a U_g)_j e_g
//   T2_i = sum_j X q^2,
//   dF/deta_i = R2_i - kappa b_i T2_i,  dF/deta'_i = kappa T1_i / A_i,
//   dF/dA_i = (R1_i - kappa b_i T1_i) / A_i.
// The gradients returned are conj(dF/dz) = ds/dRe z + i ds/dIm z.
//
// Working with the differences e_g (real) leaves 2 + 2 G complex sums per node, 44
// FP64 operations per pair for the two groups of a solve's gradient; the sums of the
// 2 G + 2 weights b V_g, b, a U_g, a P, each in both orders, took 65 and cancel where
// V varies slowly. The kernel is bound by the FP64 units: two targets per lane share
// one reciprocal and every fetched source, sources are wave-uniform records by scalar
// loads (the next one's in flight), only the tile's own 128 sources run the masked
// loop; four wavefronts split a workgroup's sources and add their sums through LDS in
// a fixed order, as the epilogue adds the source splits. Groups go two per launch
// plane (the last plane of an odd count one). N = 33792, two groups: 2.36 ms before,
// 1.65 now, 30 of the card's 34 T FP64 operations/s.
#include <cstdint>
#include <type_traits>

#include "gnk_device.h"
#include "gnk_internal.h"

namespace gnk {

namespace {

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zdiv(double2 a, double2 b) {
  const double m = 1.0 / (b.x * b.x + b.y * b.y);
  return make_double2((a.x * b.x + a.y * b.y) * m, (a.y * b.x - a.x * b.y) * m);
}
__device__ __forceinline__ double2 zadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 zsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 zscale(double s, double2 a) { return make_double2(s * a.x, s * a.y); }

// Records of plane z (groups 2z and, if there, 2z + 1), at rec + kGeomRec N z:
// {eta, b, a U_g, a U_g', V_g, V_g'} (10 doubles; a missing group has zeros).
constexpr int kGeomRec = 10;
__global__ void k_geom_weights(const double2* __restrict__ eta, const double2* __restrict__ etap,
                               const double2* __restrict__ A, int N, const GeomTerm* __restrict__ terms,
                               const GeomGroup* __restrict__ groups, int G, double* __restrict__ rec,
                               double2* __restrict__ Ut) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const double2 a = A[j];
  const double2 b = zdiv(etap[j], a);
  for (int g = 0; g < G; g += 2) {
    double2* r = reinterpret_cast<double2*>(rec + ((size_t)(g >> 1) * N + j) * kGeomRec);
    double v[2] = {0.0, 0.0};
    r[0] = eta[j];
    r[1] = b;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double2 U = make_double2(0.0, 0.0);
      if (g + h < G) {
        const GeomGroup gr = groups[g + h];
        for (int t = gr.t0; t < gr.t1; ++t) U = zadd(U, zscale(terms[t].u[j], terms[t].z));
        v[h] = gr.v[j];
        Ut[(size_t)(g + h) * N + j] = U;
      }
      r[2 + h] = zmul(a, U);
    }
    r[4] = make_double2(v[0], v[1]);
  }
}

struct GeomSrc {
  double2 eta, b, x[2];
  double v[2];
};
__device__ __forceinline__ GeomSrc load_src(gptr<const double2> r) {
  const double2 v = r[4];
  return GeomSrc{r[0], r[1], {r[2], r[3]}, {v.x, v.y}};
}

// sums of one target: T1, T2, then F1, F2 of each group
template <int NG>
struct GeomAcc {
  double2 s[2 + 2 * NG];
};

// one source against the lane's two targets; MASK: a target's own node counts nothing;
// APART: a reciprocal for each target
template <int NG, bool MASK, bool APART>
__device__ __forceinline__ void geom_step(GeomAcc<NG> (&acc)[2], const double2 (&z)[2], const double (&vt)[2][NG],
                                          const GeomSrc& s, bool own0, bool own1) {
  double dx[2], dy[2], m[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    dx[t] = z[t].x - s.eta.x;
    dy[t] = z[t].y - s.eta.y;
    m[t] = __builtin_fma(dy[t], dy[t], dx[t] * dx[t]);
  }
  if (MASK) {
    m[0] = own0 ? 1.0 : m[0];
    m[1] = own1 ? 1.0 : m[1];
  }
  double i0, i1;
  if (APART) {
    i0 = refine_rcp(m[0]);
    i1 = refine_rcp(m[1]);
  } else {
    const double R = refine_rcp(m[0] * m[1]);
    i0 = R * m[1];
    i1 = R * m[0];
  }
  m[0] = MASK && own0 ? 0.0 : i0;
  m[1] = MASK && own1 ? 0.0 : i1;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const double qx = dx[t] * m[t], ny = dy[t] * m[t];   // q = qx - i ny
    double2(&S)[2 + 2 * NG] = acc[t].s;
    double e[NG];
    double2 X;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      e[g] = vt[t][g] - s.v[g];
      X.x = g ? __builtin_fma(s.x[g].x, e[g], X.x) : s.x[g].x * e[g];
      X.y = g ? __builtin_fma(s.x[g].y, e[g], X.y) : s.x[g].y * e[g];
    }
    const double yx = __builtin_fma(X.y, ny, X.x * qx), yy = __builtin_fma(X.y, qx, -X.x * ny);
    S[0].x += yx;
    S[0].y += yy;
    S[1].x = __builtin_fma(yx, qx, __builtin_fma(yy, ny, S[1].x));
    S[1].y = __builtin_fma(yy, qx, __builtin_fma(-yx, ny, S[1].y));
    const double bx = __builtin_fma(s.b.y, ny, s.b.x * qx), by = __builtin_fma(s.b.y, qx, -s.b.x * ny);
    const double cx = __builtin_fma(by, ny, bx * qx), cy = __builtin_fma(by, qx, -bx * ny);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      S[2 + 2 * g].x = __builtin_fma(bx, e[g], S[2 + 2 * g].x);
      S[2 + 2 * g].y = __builtin_fma(by, e[g], S[2 + 2 * g].y);
      S[3 + 2 * g].x = __builtin_fma(cx, e[g], S[3 + 2 * g].x);
      S[3 + 2 * g].y = __builtin_fma(cy, e[g], S[3 + 2 * g].y);
    }
  }
}

// The sums of the 128 targets of blockIdx.x over the sources of split blockIdx.y and
// the groups of plane blockIdx.z (from `plane0` on):
// parts[((g nz + z) 6 + k) N + i], k: T1, T2, F1, F2 (, F1', F2')
template <int NG>
__global__ __launch_bounds__(256) void k_geom_sums(const double* __restrict__ rec_, int N, int plane0, int nz,
                                                   int chunk, double2* __restrict__ parts_) {
  __shared__ double2 red[3][2][64];
  constexpr int kStride = kGeomRec / 2;
  const int zp = plane0 + blockIdx.z;
  gptr<const double2> rec = (gptr<const double2>)rec_ + (size_t)zp * N * kStride;
  gptr<double2> parts = (gptr<double2>)parts_ + ((size_t)blockIdx.y * nz + zp) * 6 * N;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int base = blockIdx.x * 128;
  const int i0 = base + lane, i1 = i0 + 64;
  // targets past the end repeat node N - 1, of this tile, and skip it as source
  const int n0 = min(i0, N - 1), n1 = min(i1, N - 1);
  double2 z[2];
  double vt[2][NG];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const gptr<const double2> r = rec + (size_t)(t ? n1 : n0) * kStride;
    z[t] = r[0];
    const double2 v = r[4];
    vt[t][0] = v.x;
    if constexpr (NG > 1) vt[t][1] = v.y;
  }
  const int jb0 = blockIdx.y * chunk;
  const int jb1 = min(N, jb0 + chunk);
  const int wchunk = (chunk + 3) >> 2;
  const int j0 = min(jb1, jb0 + wv * wchunk);
  const int j1 = min(jb1, j0 + wchunk);
  GeomAcc<NG> acc[2] = {};
  auto sums = [&](auto apart) {
    constexpr bool APART = decltype(apart)::value;
    auto plain = [&](int ja, int jb) {
      if (ja >= jb) return;
      GeomSrc a = load_src(rec + (size_t)ja * kStride), b;
      int j = ja;
      for (; j + 1 < jb; j += 2) {
        b = load_src(rec + (size_t)(j + 1) * kStride);
        __builtin_amdgcn_sched_barrier(0);
        geom_step<NG, false, APART>(acc, z, vt, a, false, false);
        a = load_src(rec + (size_t)min(j + 2, jb - 1) * kStride);
        __builtin_amdgcn_sched_barrier(0);
        geom_step<NG, false, APART>(acc, z, vt, b, false, false);
      }
      if (j < jb) geom_step<NG, false, APART>(acc, z, vt, a, false, false);
    };
    plain(j0, min(j1, base));
    const int ma = max(j0, base), mb = min(j1, base + 128);
    for (int j = ma; j < mb; ++j)
      geom_step<NG, true, APART>(acc, z, vt, load_src(rec + (size_t)j * kStride), j == n0, j == n1);
    plain(max(j0, base + 128), j1);
  };
  sums(std::false_type{});
  // a node in the place of a target, or squared distances whose product leaves the
  // range, spoil the lane's two targets: sums left non-finite are formed again with a
  // reciprocal for each
  double all = 0.0;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int k = 0; k < 2 + 2 * NG; ++k) all += acc[t].s[k].x + acc[t].s[k].y;
  if (__any(!isfinite(all))) {
    acc[0] = acc[1] = GeomAcc<NG>{};
    sums(std::true_type{});
  }

#pragma unroll
  for (int k = 0; k < 2 + 2 * NG; ++k) {
    if (wv > 0) {
      red[wv - 1][0][lane] = acc[0].s[k];
      red[wv - 1][1][lane] = acc[1].s[k];
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        double2 s = acc[t].s[k];
#pragma unroll
        for (int w = 0; w < 3; ++w) s = zadd(s, red[w][t][lane]);
        const int i = t ? i1 : i0;
        if (i < N) parts[(size_t)k * N + i] = s;
      }
    }
    __syncthreads();
  }
}

__global__ void k_geom_epilogue(const double2* __restrict__ etap, const double2* __restrict__ A, int N, int n, int G,
                                const double2* __restrict__ Ut, const double2* __restrict__ parts, int splits,
                                double2* g_eta, double2* g_etap, double2* g_A) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int nz = (G + 1) / 2;
  // the six sums of a plane over the splits, their loads in flight together
  auto sums = [&](int z, double2 (&s)[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = make_double2(0.0, 0.0);
    for (int g = 0; g < splits; ++g) {
      const double2* p = parts + ((size_t)g * nz + z) * 6 * N + i;
      double2 v[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) v[k] = (k < 4 || 2 * z + 1 < G) ? p[(size_t)k * N] : make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 6; ++k) s[k] = zadd(s[k], v[k]);
    }
  };
  const double kappa = 2.0 / (double)n;
  const double2 a = A[i];
  const double2 b = zdiv(etap[i], a);
  double2 R1 = make_double2(0.0, 0.0), R2 = R1, T1 = R1, T2 = R1;
  for (int z = 0; z < nz; ++z) {
    double2 s[6];
    sums(z, s);
    T1 = zadd(T1, s[0]);
    T2 = zadd(T2, s[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (2 * z + h < G) {
        const double2 U = Ut[(size_t)(2 * z + h) * N + i];
        R1 = zadd(R1, zmul(U, s[2 + 2 * h]));
        R2 = zadd(R2, zmul(U, s[3 + 2 * h]));
      }
  }
  R1 = zscale(kappa, zmul(a, R1));
  R2 = zscale(-kappa, zmul(a, R2));
  const double2 C1 = zscale(kappa, zmul(b, T1));
  const double2 C2 = zscale(-kappa, zmul(b, T2));
  const double2 de = zadd(R2, C2);
  const double2 dp = zscale(kappa, zdiv(T1, a));
  const double2 da = zdiv(zsub(R1, C1), a);
  if (g_eta) g_eta[i] = make_double2(de.x, -de.y);
  if (g_etap) g_etap[i] = make_double2(dp.x, -dp.y);
  if (g_A) g_A[i] = make_double2(da.x, -da.y);
}

// e^{2 pi i m / n} for an integer m reduced into [0, n) (exact argument)
__device__ __forceinline__ double2 unit_root(int64_t m, int64_t n) {
  double s, c;
  sincospi(2.0 * (double)m / (double)n, &s, &c);
  return make_double2(c, s);
}

__device__ __forceinline__ int64_t mod_n(int64_t x, int64_t n) {
  int64_t r = x % n;
  return r < 0 ? r + n : r;
}

// eta_j(t_p) = sum_k c_{j,k} e^{i s k t_p}, t_p = 2 pi p / n, and the first two
// derivatives (factors i s k and -k^2); grid (blocks over n, m1)
__global__ void k_fourier_curve(const double2* __restrict__ coef, int n, int kmin, int nk, int sgn,
                                double2* __restrict__ eta, double2* __restrict__ etap, double2* __restrict__ etapp) {
  const int j = blockIdx.y;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  double2 e0 = make_double2(0.0, 0.0), e1 = e0, e2 = e0;
  for (int q = 0; q < nk; ++q) {
    const int64_t k = kmin + q;
    const double2 cp = zmul(coef[(size_t)j * nk + q], unit_root(mod_n((int64_t)sgn * k * p, n), n));
    const double sk = (double)(sgn * k);
    e0 = zadd(e0, cp);
    e1 = zadd(e1, make_double2(-sk * cp.y, sk * cp.x));
    e2 = zadd(e2, zscale(-(double)(k * k), cp));
  }
  const size_t o = (size_t)j * n + p;
  eta[o] = e0;
  if (etap) etap[o] = e1;
  if (etapp) etapp[o] = e2;
}

// g_c[j,k] = sum_p (g_eta + conj(i s k) g_eta' + conj(-k^2) g_eta'')_p e^{-i s k t_p};
// one 256-thread block per (coefficient, component), fixed-order reduction
__global__ __launch_bounds__(256) void k_fourier_vjp(const double2* __restrict__ g_eta,
                                                     const double2* __restrict__ g_etap,
                                                     const double2* __restrict__ g_etapp, int n, int kmin, int nk,
                                                     int sgn, double2* __restrict__ g_coef) {
  __shared__ double2 sh[256];
  const int q = blockIdx.x, j = blockIdx.y;
  const int64_t k = kmin + q;
  const double sk = (double)(sgn * k);
  double2 acc = make_double2(0.0, 0.0);
  for (int p = threadIdx.x; p < n; p += blockDim.x) {
    const size_t o = (size_t)j * n + p;
    double2 w = g_eta ? g_eta[o] : make_double2(0.0, 0.0);
    if (g_etap) {
      const double2 z = g_etap[o];
      w = zadd(w, make_double2(sk * z.y, -sk * z.x));     // (-i s k) z
    }
    if (g_etapp) w = zadd(w, zscale(-(double)(k * k), g_etapp[o]));
    acc = zadd(acc, zmul(w, unit_root(mod_n(-(int64_t)sgn * k * p, n), n)));
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] = zadd(sh[threadIdx.x], sh[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) g_coef[(size_t)j * nk + q] = sh[0];
}

}  // namespace

size_t geom_rec_doubles(int N, int G) { return (size_t)((G + 1) / 2) * N * kGeomRec; }
size_t geom_part_count(int N, int G, int splits) { return (size_t)((G + 1) / 2) * N * 6 * splits; }

hipError_t launch_geom_weights(const double2* eta, const double2* etap, const double2* A, int N,
                               const GeomTerm* terms, const GeomGroup* groups, int G, double* rec, double2* Ut,
                               hipStream_t st) {
  k_geom_weights<<<(unsigned)((N + 255) / 256), 256, 0, st>>>(eta, etap, A, N, terms, groups, G, rec, Ut);
  return hipGetLastError();
}

hipError_t launch_geom_sums(const double* rec, int N, int G, int chunk, int splits, double2* parts, hipStream_t st) {
  const int nz = (G + 1) / 2;
  const dim3 grid((unsigned)((N + 127) / 128), (unsigned)splits, (unsigned)(G / 2));
  if (G > 1) k_geom_sums<2><<<grid, 256, 0, st>>>(rec, N, 0, nz, chunk, parts);
  if (G & 1) k_geom_sums<1><<<dim3(grid.x, grid.y, 1), 256, 0, st>>>(rec, N, nz - 1, nz, chunk, parts);
  return hipGetLastError();
}

hipError_t launch_geom_epilogue(const double2* etap, const double2* A, int N, int n, int G, const double2* Ut,
                                const double2* parts, int splits, double2* g_eta, double2* g_etap, double2* g_A,
                                hipStream_t st) {
  k_geom_epilogue<<<(unsigned)((N + 63) / 64), 64, 0, st>>>(etap, A, N, n, G, Ut, parts, splits, g_eta, g_etap, g_A);
  return hipGetLastError();
}

hipError_t launch_fourier_curve(const double2* coef, int m1, int n, int kmin, int nk, int sgn, double2* eta,
                                double2* etap, double2* etapp, hipStream_t st) {
  dim3 grid((unsigned)((n + 255) / 256), (unsigned)m1);
  k_fourier_curve<<<grid, 256, 0, st>>>(coef, n, kmin, nk, sgn, eta, etap, etapp);
  return hipGetLastError();
}

hipError_t launch_fourier_vjp(const double2* g_eta, const double2* g_etap, const double2* g_etapp, int m1, int n,
                              int kmin, int nk, int sgn, double2* g_coef, hipStream_t st) {
  dim3 grid((unsigned)nk, (unsigned)m1);
  k_fourier_vjp<<<grid, 256, 0, st>>>(g_eta, g_etap, g_etapp, n, kmin, nk, sgn, g_coef);
  return hipGetLastError();
}

}  // namespace gnk
