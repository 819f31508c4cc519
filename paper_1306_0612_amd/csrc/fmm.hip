// 2D Coulomb FMM for the Cauchy part of the double-layer operator.
//
// The operator of Section 5 (eq. disc_sphere) splits, for target node i, as
//   (K sigma)_i = Re sum_{j != i} p_j / (xi_i - xi_j) + tau_i sigma_i + gamma
// with complex strengths p_j = -i q_j, q_j = (s h / pi) xi'_j sigma_j.
// The sum is the planar Coulomb/Cauchy potential that the paper evaluates
// with the 2D FMM (Section 5).  Expansions are stored scaled by the box
// half-width r so that same-level translations are level independent:
//   multipole  Psi(z) = sum_{k=1..P} a_k (r / (z - c))^k,
//              a_k = (1/r) sum_j p_j ((z_j - c)/r)^(k-1)
//   local      Psi(z) = sum_{l=0..P-1} b_l ((z - c)/r)^l
// Translations (binomial series of 1/(z - z_j)):
//   M2M  child c1 (half-width r/2) -> parent c0: d = c1 - c0 = (r/2) delta,
//        A_l = sum_{k<=l} a_k C(l-1,k-1) delta^(l-k) 2^-l
//   M2L  same-level, c_s - c_t = r tau, tau = 2 (dx + i dy):
//        b_l = tau^-l sum_k (-1)^k C(k+l-1,l) tau^-k a_k
//   L2L  parent c0 -> child c1 = c0 + (r/2) delta:
//        b'_m = sum_{l>=m} b_l C(l,m) delta^(l-m) 2^-l
//   P2L  b_l = -sum_j (p_j/u_j) (r/u_j)^l, u_j = z_j - c
//   M2P  Psi(z) = sum_k a_k (r_w/(z - c_w))^k
#include <cmath>
#include <type_traits>
#include <vector>

#include "cplx.h"
#include "lbs_internal.h"

namespace lbs {

// ----------------------------------------------------------------- tables
static double binom(int n, int k) {
  if (k < 0 || k > n) return 0.0;
  double r = 1.0;
  for (int i = 1; i <= k; ++i) r = r * (double)(n - k + i) / (double)i;
  return std::round(r);
}

static void cpow_host(double x, double y, int n, double &ox, double &oy) {
  double rx = 1, ry = 0;
  for (int i = 0; i < n; ++i) {
    double t = rx * x - ry * y;
    ry = rx * y + ry * x;
    rx = t;
  }
  ox = rx;
  oy = ry;
}

void build_tables(Tables &t, int P, hipStream_t s) {
  t.P = P;
  // M2M and L2L factorized as scale x Pascal x scale (quadrant offset
  // delta = (+-1, +-1), |delta|^2 = 2):
  //   M2M: A_lo = 1/2 (delta/2)^lo sum_{k <= lo} C(lo, k) (conj(delta)/2)^k a_k
  //   L2L: b'_m = (conj(delta)/2)^m sum_{l >= m} C(l, m) (delta/2)^l b_l
  // Tables: C (P x P, zero above the diagonal), pre[q][n] =
  // (conj(delta_q)/2)^n and post[q][n] = (delta_q/2)^n.
  std::vector<double> bc(P * P, 0.0), pre(4 * P * 2), post(4 * P * 2);
  for (int n = 0; n < P; ++n)
    for (int k = 0; k <= n; ++k) bc[n * P + k] = binom(n, k);
  for (int q = 0; q < 4; ++q) {
    const double dx = (q & 1) ? 1.0 : -1.0, dy = (q & 2) ? 1.0 : -1.0;
    for (int n = 0; n < P; ++n) {
      double ax, ay, bx, by;
      cpow_host(0.5 * dx, -0.5 * dy, n, ax, ay);
      cpow_host(0.5 * dx, 0.5 * dy, n, bx, by);
      pre[2 * (q * P + n)] = ax;
      pre[2 * (q * P + n) + 1] = ay;
      post[2 * (q * P + n)] = bx;
      post[2 * (q * P + n) + 1] = by;
    }
  }
  std::vector<double> h(P * P);
  for (int l = 0; l < P; ++l)
    for (int ki = 0; ki < P; ++ki) {
      int k = ki + 1;
      h[l * P + ki] = ((k & 1) ? -1.0 : 1.0) * binom(k + l - 1, l);
    }
  const int NP = 2 * P + 1;
  std::vector<double> itp(49 * NP * 2, 0.0);
  for (int code = 0; code < 49; ++code) {
    int dx = code / 7 - 3, dy = code % 7 - 3;
    if (std::abs(dx) <= 1 && std::abs(dy) <= 1) continue;
    double tx = 2.0 * dx, ty = 2.0 * dy, d = tx * tx + ty * ty;
    double ix = tx / d, iy = -ty / d;  // 1 / tau
    for (int n = 0; n < NP; ++n) {
      double px, py;
      cpow_host(ix, iy, n, px, py);
      itp[(code * NP + n) * 2] = px;
      itp[(code * NP + n) * 2 + 1] = py;
    }
  }
  auto to32 = [](const std::vector<double> &v) {
    return std::vector<float>(v.begin(), v.end());
  };
  t.bc64.upload(bc, s);
  t.pre64.upload(pre, s);
  t.post64.upload(post, s);
  t.h64.upload(h, s);
  t.bc32.upload(to32(bc), s);
  t.pre32.upload(to32(pre), s);
  t.post32.upload(to32(post), s);
  t.h32.upload(to32(h), s);
  t.itp32.upload(to32(itp), s);
  LBS_HIP(hipStreamSynchronize(s));
}

// ----------------------------------------------------------------- kernels
// v[0 .. NV) summed over the 64 lanes of a wave by recursive halving: at
// step s (partner lane ^ (32 >> s)) a lane keeps the upper half of its
// values when that lane bit is set, else the lower half, and adds its
// partner's copy of the half it keeps; once a single value is left the
// remaining steps add it whole.  Lane i returns the total of value
// i >> (6 - log2 NV); NV - 1 + 6 - log2 NV shuffles in all.
// One halving step at lane offset 32 or 16 for the pair (a, b): the
// permlane swaps exchange the upper 32 lanes of a with the lower 32 of b
// (the odd 16-lane rows of a with the even rows of b), after which a + b is,
// in every lane, its own plus its partner's copy of the value it keeps.
template <int O>
__device__ __forceinline__ float swap_add(float a, float b) {
  static_assert(O == 32 || O == 16, "lane offsets with a swap instruction");
  const auto r = O == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)
                         : __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <typename T, int NV, bool SWAP, int S = 0>
__device__ __forceinline__ void halving_steps(T (&v)[NV], int lane) {
  if constexpr (S < 6) {
    constexpr int o = 32 >> S, h = NV >> (S + 1);
    if constexpr (SWAP && h >= 1 && sizeof(T) == 4 && o >= 16) {
#pragma unroll
      for (int k = 0; k < h; ++k) v[k] = swap_add<o>(v[k], v[k + h]);
    } else if constexpr (h >= 1) {
      const bool up = (lane & o) != 0;
#pragma unroll
      for (int k = 0; k < h; ++k) {
        const T send = up ? v[k] : v[k + h];
        const T keep = up ? v[k + h] : v[k];
        v[k] = keep + __shfl_xor(send, o, 64);
      }
    } else {
      v[0] += __shfl_xor(v[0], o, 64);
    }
    halving_steps<T, NV, SWAP, S + 1>(v, lane);
  }
}

// SWAP: the steps at lane offsets 32 and 16 of FP32 values by permlane
// swaps (swap_add) instead of selects and a cross-lane read.
template <typename T, int NV, bool SWAP = true>
__device__ __forceinline__ T halving_sum(T (&v)[NV], int lane) {
  static_assert(NV >= 1 && NV <= 64 && (NV & (NV - 1)) == 0,
                "a power of two up to the wave size");
  halving_steps<T, NV, SWAP>(v, lane);
  return v[0];
}

constexpr int pow2_ceil(int n) { return n <= 1 ? 1 : 2 * pow2_ceil((n + 1) / 2); }
constexpr int log2_exact(int n) { return n <= 1 ? 0 : 1 + log2_exact(n / 2); }

// Coefficients per register pass of the P2M and P2L sums: 2 KB real
// accumulators per lane (KB of 16 FP64 or 32 FP32 terms keeps them within
// 64 registers); an order above KB takes several passes over the sources.
template <typename T, int P>
constexpr int kChunk() {
  return P < (sizeof(T) == 8 ? 16 : 32) ? P : (sizeof(T) == 8 ? 16 : 32);
}

// P2L sum of one box (centre (cxb, cyb), half-width rb) over the sources
// of its X list, xf_idx[x0 .. x0 + total) (concatenated at set-up), for
// coefficients K0 .. K0 + KB - 1: lane q accumulates t_q (r/u_q)^l,
// t_q = -p_q / u_q, u_q = z_q - c, for sources q, q + 64, ... in registers
// (parts of coefficient K0 + l as values 2l, 2l + 1); one halving sum.
// Lane i returns the total of value i >> (6 - log2 NV), NV = pow2 >= 2 KB.
template <typename T, int P, int K0, int KB>
__device__ __forceinline__ T p2l_sum(int64_t x0, int total,
                                     const int32_t *__restrict__ xf_idx,
                                     double cxb, double cyb, T rb,
                                     const double *__restrict__ sx,
                                     const double *__restrict__ sy,
                                     const cx<T> *__restrict__ pr, int lane) {
  constexpr int NV = pow2_ceil(2 * KB);
  T acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = T(0);
  for (int q = lane; q < total; q += 64) {
    const int64_t j = xf_idx[x0 + q];
    const cx<T> u{T(sx[j] - cxb), T(sy[j] - cyb)};
    cx<T> iu;
    if constexpr (sizeof(T) == 4) {  // FP32 expansions: hardware reciprocal
      const float d = __builtin_amdgcn_rcpf(u.x * u.x + u.y * u.y);
      iu = cx<T>{u.x * d, -u.y * d};
    } else {
      iu = cinv(u);
    }
    const cx<T> rho = rb * iu;
    cx<T> t = pr[j] * iu;
    t = cx<T>{-t.x, -t.y};
    if (K0 > 0) t = t * cpow(rho, K0);
#pragma unroll
    for (int l = 0; l < KB; ++l) {
      if (K0 + l < P) {
        acc[2 * l] += t.x;
        acc[2 * l + 1] += t.y;
        t = t * rho;
      }
    }
  }
  return halving_sum<T, NV>(acc, lane);
}

// Where the leaf multipole pass finds its strengths: with sigma set it
// forms p_j = -i q_j sigma_j itself (q-factor qfac_t in tree order, sigma in
// API order through perm, stride ldx per right-hand side) and stores them
// for the near field and P2L; otherwise it reads p as given.
struct StrengthSrc {
  const int64_t *perm = nullptr;
  const double *qfac_t = nullptr;
  const double *sigma = nullptr;
  int64_t ldx = 0;
  // with gpart set: gpart[r * (#leaves) + leaf] = sum over the leaf's
  // sources of gw_t[j] sigma_j (FP64), for GammaFused
  const double *gw_t = nullptr;
  double *gpart = nullptr;
  // optional, for the FP32 leaf multipoles: -i q_j as (Im q_j, -Re q_j)
  // rounded to FP32 and the permutation as 32-bit indices (half the bytes
  // of qfac_t and perm)
  const float2 *qm32 = nullptr;
  const int32_t *perm32 = nullptr;
};

// Leaf multipoles, one wave per leaf (every source lies in one leaf): lane
// j accumulates p_j w_j^k of sources j, j + 64, ... in registers, KB
// coefficients per pass (real and imaginary parts as values 2k, 2k + 1 of
// NV = pow2 >= 2 KB), and one halving sum per pass leaves the parts of
// coefficient k in lanes (2k + c) << SH.  The first pass forms the
// strengths (when asked to); later passes read them back.
template <typename T, int P>
__global__ void __launch_bounds__(64)
    k_p2m(const int32_t *__restrict__ leaves,
          const int64_t *__restrict__ ls_rng,
          const double4 *__restrict__ ls_geo,
          const double *__restrict__ sx, const double *__restrict__ sy,
          cx<T> *__restrict__ p, int64_t ns, cx<T> *__restrict__ M,
          int nbox, StrengthSrc ss) {
  constexpr int KB = kChunk<T, P>(), NV = pow2_ceil(2 * KB),
                SH = 6 - log2_exact(NV);
  // the leaf's source range and frame by work-group (one load level less
  // than through its box id, which only the final store needs)
  const int b = leaves[blockIdx.x];
  const int r = blockIdx.y;
  const int lane = threadIdx.x;
  const double4 geo = ls_geo[blockIdx.x];
  const double c_x = geo.x, c_y = geo.y, ir = geo.z;
  cx<T> *pr = p + (int64_t)r * ns;
  double gsum = 0.0;
  const int64_t e0 = ls_rng[2 * blockIdx.x], e1 = ls_rng[2 * blockIdx.x + 1];
  if (e1 == e0 && !ss.gpart) return;  // an empty range: the whole wave, M left as it is
  const int vi = lane >> SH;
  const bool writer = (lane & ((1 << SH) - 1)) == 0;
#pragma unroll
  for (int k0 = 0; k0 < P; k0 += KB) {
    T acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = T(0);
    for (int64_t j = e0 + lane; j < e1; j += 64) {
      const cx<T> w{T((sx[j] - c_x) * ir), T((sy[j] - c_y) * ir)};
      cx<T> pw;
      if (k0 == 0 && ss.sigma) {  // form the strength: p_j = -i q_j sigma_j
        const double sg = ss.sigma[(int64_t)r * ss.ldx + ss.perm[j]];
        const double qx = ss.qfac_t[2 * j], qy = ss.qfac_t[2 * j + 1];
        pw = cx<T>{T(qy * sg), T(-qx * sg)};
        pr[j] = pw;
        if (ss.gpart) gsum += ss.gw_t[j] * sg;
      } else {
        pw = pr[j];
      }
      if (k0 > 0) pw = pw * cpow(w, k0);
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        if (k0 + k < P) {
          acc[2 * k] += pw.x;
          acc[2 * k + 1] += pw.y;
          pw = pw * w;
        }
      }
    }
    const T tot = halving_sum<T, NV, false>(acc, lane);
    T *Mb = reinterpret_cast<T *>(M + ((int64_t)r * nbox + b) * P);
    if (writer && vi < 2 * KB && 2 * k0 + vi < 2 * P) Mb[2 * k0 + vi] = T(ir) * tot;
  }
  if (ss.gpart) {  // block-uniform
    for (int o = 32; o > 0; o >>= 1) gsum += __shfl_xor(gsum, o, 64);
    if (lane == 0) ss.gpart[(int64_t)r * gridDim.x + blockIdx.x] = gsum;
  }
}

// The FP32 leaf multipoles of two leaves per wave (list entries 2 w and
// 2 w + 1 on lanes 0-31 and 32-63): as k_p2m, with every source loop
// striding by 32 and the halving sum run inside each half (lane offsets
// 16 .. 1), so that the sum's fixed cost is shared by two leaves.  One
// pass: P <= 32 coefficients, NV = 2 P values.
template <typename T, int NV, int S = 0>
__device__ __forceinline__ void halving_steps_half(T (&v)[NV], int lane) {
  if constexpr (S < 5) {
    constexpr int o = 16 >> S, h = NV >> (S + 1);
    if constexpr (h >= 1) {
      const bool up = (lane & o) != 0;
#pragma unroll
      for (int k = 0; k < h; ++k) {
        const T send = up ? v[k] : v[k + h];
        const T keep = up ? v[k + h] : v[k];
        v[k] = keep + __shfl_xor(send, o, 64);
      }
    } else {
      v[0] += __shfl_xor(v[0], o, 64);
    }
    halving_steps_half<T, NV, S + 1>(v, lane);
  }
}

template <int P>
__global__ void __launch_bounds__(64)
    k_p2m_pair(const int32_t *__restrict__ leaves, int nleaf,
               const int64_t *__restrict__ ls_rng,
               const double4 *__restrict__ ls_geo,
               const double *__restrict__ sx, const double *__restrict__ sy,
               const float2 *__restrict__ w32,
               cx<float> *__restrict__ p, int64_t ns, cx<float> *__restrict__ M,
               int nbox, StrengthSrc ss) {
  constexpr int NV = pow2_ceil(2 * P), SH = 5 - log2_exact(NV);
  static_assert(P <= 16, "one pass of at most 32 values per lane");
  const int lane = threadIdx.x, half = lane >> 5, hl = lane & 31;
  const int e = 2 * blockIdx.x + half;  // this half's list entry
  const bool has = e < nleaf;           // uniform within the half
  const int r = blockIdx.y;
  cx<float> *pr = p + (int64_t)r * ns;
  float acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.f;
  double gsum = 0.0;
  int b = 0;
  double ir = 0.0;
  if (has) {
    b = leaves[e];
    const double4 geo = ls_geo[e];
    const double c_x = geo.x, c_y = geo.y;
    ir = geo.z;
    const int64_t e0 = ls_rng[2 * e], e1 = ls_rng[2 * e + 1];
    if (w32 && ss.sigma && ss.qm32) {  // uniform
      // sources j and j + 32 of this lane per step, every load issued
      // before the dependent gathers of sigma, the terms added in source
      // order as below
      const double *sgr = ss.sigma + (int64_t)r * ss.ldx;
      for (int64_t j = e0 + hl; j < e1; j += 64) {
        const bool two = j + 32 < e1;
        const int64_t jb = two ? j + 32 : j;
        const int ia = ss.perm32[j], ib = ss.perm32[jb];
        const float2 wa = w32[j], wb = w32[jb];
        const float2 qa = ss.qm32[j], qb = ss.qm32[jb];
        double ga = 0.0, gb = 0.0;
        if (ss.gpart) {
          ga = ss.gw_t[j];
          gb = ss.gw_t[jb];
        }
        const double sa = sgr[ia], sb = sgr[ib];
        cx<float> pa{float((double)qa.x * sa), float((double)qa.y * sa)};
        cx<float> pb{float((double)qb.x * sb), float((double)qb.y * sb)};
        pr[j] = pa;
        if (ss.gpart) gsum += ga * sa;
        if (two) {
          pr[jb] = pb;
          if (ss.gpart) gsum += gb * sb;
        } else {
          pb = cx<float>{0.f, 0.f};
        }
        const cx<float> wca{wa.x, wa.y}, wcb{wb.x, wb.y};
#pragma unroll
        for (int k = 0; k < P; ++k) {
          acc[2 * k] += pa.x;
          acc[2 * k + 1] += pa.y;
          pa = pa * wca;
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
          acc[2 * k] += pb.x;
          acc[2 * k + 1] += pb.y;
          pb = pb * wcb;
        }
      }
    } else
    for (int64_t j = e0 + hl; j < e1; j += 32) {
      cx<float> w;
      if (w32) {  // uniform: the leaf-relative positions of set-up
        const float2 t = w32[j];
        w = cx<float>{t.x, t.y};
      } else {
        w = cx<float>{float((sx[j] - c_x) * ir), float((sy[j] - c_y) * ir)};
      }
      cx<float> pw;
      if (ss.sigma) {  // form the strength: p_j = -i q_j sigma_j
        if (ss.qm32) {  // uniform
          const double sg = ss.sigma[(int64_t)r * ss.ldx + ss.perm32[j]];
          const float2 q = ss.qm32[j];
          pw = cx<float>{float((double)q.x * sg), float((double)q.y * sg)};
          if (ss.gpart) gsum += ss.gw_t[j] * sg;
        } else {
          const double sg = ss.sigma[(int64_t)r * ss.ldx + ss.perm[j]];
          const double qx = ss.qfac_t[2 * j], qy = ss.qfac_t[2 * j + 1];
          pw = cx<float>{float(qy * sg), float(-qx * sg)};
          if (ss.gpart) gsum += ss.gw_t[j] * sg;
        }
        pr[j] = pw;
      } else {
        pw = pr[j];
      }
#pragma unroll
      for (int k = 0; k < P; ++k) {
        acc[2 * k] += pw.x;
        acc[2 * k + 1] += pw.y;
        pw = pw * w;
      }
    }
  }
  halving_steps_half<float, NV>(acc, lane);
  const int vi = hl >> SH;
  if (has && (hl & ((1 << SH) - 1)) == 0 && vi < 2 * P) {
    float *Mb = reinterpret_cast<float *>(M + ((int64_t)r * nbox + b) * P);
    Mb[vi] = float(ir) * acc[0];
  }
  if (ss.gpart) {  // block-uniform
    for (int o = 16; o > 0; o >>= 1) gsum += __shfl_xor(gsum, o, 64);
    if (has && hl == 0) ss.gpart[(int64_t)r * nleaf + e] = gsum;
  }
}

// The FP64 leaf multipoles of two leaves per wave (list entries 2 w and
// 2 w + 1 on lanes 0-31 and 32-63): as k_p2m, KB coefficients per pass
// over the sources (the first pass forms the strengths, later passes read
// them back), every source loop striding by 32 and one halving sum per
// pass inside each half, so that the sums' fixed cost is shared by two
// leaves.
template <int P>
__global__ void __launch_bounds__(64)
    k_p2m_pair64(const int32_t *__restrict__ leaves, int nleaf,
                 const int64_t *__restrict__ ls_rng,
                 const double4 *__restrict__ ls_geo,
                 const double *__restrict__ sx, const double *__restrict__ sy,
                 cx<double> *__restrict__ p, int64_t ns, cx<double> *__restrict__ M,
                 int nbox, StrengthSrc ss) {
  constexpr int KB = kChunk<double, P>(), NV = pow2_ceil(2 * KB), SH = 5 - log2_exact(NV);
  static_assert(NV <= 32, "at most one value per lane of a half after the halving sum");
  const int lane = threadIdx.x, half = lane >> 5, hl = lane & 31;
  const int e = 2 * blockIdx.x + half;  // this half's list entry
  const bool has = e < nleaf;           // uniform within the half
  const int r = blockIdx.y;
  cx<double> *pr = p + (int64_t)r * ns;
  double gsum = 0.0, c_x = 0.0, c_y = 0.0, ir = 0.0;
  int b = 0;
  int64_t e0 = 0, e1 = 0;
  if (has) {
    b = leaves[e];
    const double4 geo = ls_geo[e];
    c_x = geo.x;
    c_y = geo.y;
    ir = geo.z;
    e0 = ls_rng[2 * e];
    e1 = ls_rng[2 * e + 1];
  }
  const int vi = hl >> SH;
  const bool writer = has && (hl & ((1 << SH) - 1)) == 0;
#pragma unroll
  for (int k0 = 0; k0 < P; k0 += KB) {
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    for (int64_t j = e0 + hl; j < e1; j += 32) {
      const cx<double> w{(sx[j] - c_x) * ir, (sy[j] - c_y) * ir};
      cx<double> pw;
      if (k0 == 0 && ss.sigma) {  // form the strength: p_j = -i q_j sigma_j
        const double sg = ss.sigma[(int64_t)r * ss.ldx + ss.perm[j]];
        const double qx = ss.qfac_t[2 * j], qy = ss.qfac_t[2 * j + 1];
        pw = cx<double>{qy * sg, -qx * sg};
        pr[j] = pw;
        if (ss.gpart) gsum += ss.gw_t[j] * sg;
      } else {
        pw = pr[j];
      }
      if (k0 > 0) pw = pw * cpow(w, k0);
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        if (k0 + k < P) {
          acc[2 * k] += pw.x;
          acc[2 * k + 1] += pw.y;
          pw = pw * w;
        }
      }
    }
    halving_steps_half<double, NV>(acc, lane);
    if (writer && vi < 2 * KB && 2 * k0 + vi < 2 * P) {
      double *Mb = reinterpret_cast<double *>(M + ((int64_t)r * nbox + b) * P);
      Mb[2 * k0 + vi] = ir * acc[0];
    }
  }
  if (ss.gpart) {  // block-uniform
    for (int o = 16; o > 0; o >>= 1) gsum += __shfl_xor(gsum, o, 64);
    if (has && hl == 0) ss.gpart[(int64_t)r * nleaf + e] = gsum;
  }
}

// gamma[r G + g] = the sum of the partial sums of geometry g's source
// leaves, positions gl_ptr[g] .. gl_ptr[g + 1] of the plan's leaf list.
// Block (c, g, r) sums chunk c of that range into csum; the last block of
// (g, r) to finish (a device-scope counter) adds the chunk sums in index
// order and resets the counter for the next application, so the result
// does not depend on the order in which blocks run.
constexpr int kGammaChunk = 2048;
__device__ __forceinline__ void gamma_chunk(int c, int g, int r, int nch,
                                            const int32_t *__restrict__ gl_ptr,
                                            const double *__restrict__ gpart,
                                            int nls, int G,
                                            double *__restrict__ csum,
                                            int32_t *__restrict__ cnt,
                                            double *__restrict__ gamma) {
  __shared__ double red[4];
  __shared__ bool last;
  const int tid = threadIdx.x, slot = r * G + g;  // (256 threads)
  const int a = gl_ptr[g] + c * kGammaChunk, b = min(gl_ptr[g + 1], a + kGammaChunk);
  double v = 0.0;
  for (int e = a + tid; e < b; e += 256) v += gpart[(int64_t)r * nls + e];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  if (tid == 0) {
    csum[(int64_t)slot * nch + c] = red[0] + red[1] + red[2] + red[3];
    __threadfence();
    last = atomicAdd(&cnt[slot], 1) == nch - 1;
  }
  __syncthreads();
  if (last && tid == 0) {
    __threadfence();
    double t = 0.0;
    for (int k = 0; k < nch; ++k)
      t += __hip_atomic_load(&csum[(int64_t)slot * nch + k], __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    gamma[slot] = t;
    cnt[slot] = 0;
  }
}

__global__ void __launch_bounds__(256)
    k_gamma_reduce(const int32_t *__restrict__ gl_ptr,
                   const double *__restrict__ gpart, int nls, int G,
                   double *__restrict__ csum, int32_t *__restrict__ cnt,
                   double *__restrict__ gamma) {
  gamma_chunk(blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x, gl_ptr, gpart,
              nls, G, csum, cnt, gamma);
}

// The correction sums of GammaFused for a kernel that takes them as extra
// work-groups: group x >= first (x - first = g nchunk + c) reduces chunk c
// of geometry g for right-hand side blockIdx.y.
struct GammaGroups {
  const int32_t *gl_ptr = nullptr;
  const double *gpart = nullptr;
  double *csum = nullptr;
  int32_t *cnt = nullptr;
  double *gamma = nullptr;
  int nls = 0, G = 0, nchunk = 0, first = 0;
};

// 1 / d in FP64: the hardware estimate (2^-22 or better) and one cubic
// correction, r (1 + e + e^2) with e = 1 - d r, which leaves e^3 < 2^-64:
// three fused multiply-adds where two Newton-Raphson steps take four.
__device__ __forceinline__ double rcp64(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Set-up of the FP64 M2L: each group's list entries as (source box, offset
// code), kM2LEnt per group
// (source -1 past the last), and its boxes as (box, number of entries up to
// and with it | box has an X list << 16), kM2LBoxes per group (box -1 past
// the last).  One wave per group.
__global__ void __launch_bounds__(64)
    k_m2l_pack(const int2 *__restrict__ grp, const int32_t *__restrict__ boxes,
               const int32_t *__restrict__ v_ptr, const int32_t *__restrict__ v_src,
               const uint8_t *__restrict__ v_code, const int64_t *__restrict__ xf_ptr,
               int2 *__restrict__ ent, int2 *__restrict__ box) {
  const int gi = blockIdx.x, lane = threadIdx.x;
  const int2 gr = grp[gi];
  int n = 0;
  int2 mine = make_int2(-1, 0);
  for (int i = 0; i < gr.y; ++i) {
    const int b = boxes[gr.x + i], v0 = v_ptr[b], len = v_ptr[b + 1] - v0;
    if (lane >= n && lane < n + len)
      mine = make_int2(v_src[v0 + lane - n], (int)v_code[v0 + lane - n]);
    n += len;
    const int hx = xf_ptr[b + 1] > xf_ptr[b];
    if (lane == 0) box[gi * kM2LBoxes + i] = make_int2(b, n | (hx << 16));
  }
  if (lane >= gr.y && lane < kM2LBoxes) box[gi * kM2LBoxes + lane] = make_int2(-1, n);
  if (lane < kM2LEnt) ent[(int64_t)gi * kM2LEnt + lane] = mine;
}

void build_m2l_groups(DevPlan &pl, const std::vector<int32_t> &grp, hipStream_t s) {
  pl.n_grp = (int)(grp.size() / 2);
  if (pl.n_grp == 0) return;
  pl.grp.upload(grp, s);
  pl.grp_ent.alloc((size_t)pl.n_grp * kM2LEnt);
  pl.grp_box.alloc((size_t)pl.n_grp * kM2LBoxes);
  hipLaunchKernelGGL(k_m2l_pack, dim3(pl.n_grp), dim3(64), 0, s,
                     reinterpret_cast<const int2 *>(pl.grp.p), pl.m2l_box.p, pl.v_ptr.p, pl.v_src.p,
                     pl.v_code.p, pl.xf_ptr.p, pl.grp_ent.p, pl.grp_box.p);
  LBS_HIP(hipGetLastError());
}

// P2L sums of two boxes with X lists per wave (entries 2 e and 2 e + 1 of
// xbox on lanes 0-31 and 32-63), stored to L: KB coefficients in registers
// per pass over a box's sources, one halving sum per pass inside each half;
// a source's index is read two steps and its data one step ahead.
struct XBoxes {
  int n = 0;                             // boxes with X lists
  const int32_t *box = nullptr;
  const int64_t *xf_ptr = nullptr;
  const int32_t *xf_idx = nullptr;
  const double *cx = nullptr, *cy = nullptr, *rad = nullptr, *sx = nullptr, *sy = nullptr;
  int64_t ns = 0;
};

template <int P, int KB>
__device__ __forceinline__ void p2l_pair64(int e, int r, const XBoxes &xb,
                                           const cx<double> *__restrict__ p,
                                           cx<double> *__restrict__ L, int nbox) {
  constexpr int NV = 2 * KB;
  static_assert(NV == 32 || NV == 64, "one or two values per lane of a half");
  const int lane = threadIdx.x & 63, hl = lane & 31;
  const int i = 2 * e + (lane >> 5);
  const bool has = i < xb.n;
  const int b = xb.box[has ? i : xb.n - 1];
  const int64_t x0 = xb.xf_ptr[b];
  const int nx = (int)(xb.xf_ptr[b + 1] - x0);
  const double cxb = xb.cx[b], cyb = xb.cy[b], rb = xb.rad[b];
  const cx<double> *pr = p + (int64_t)r * xb.ns;
  const int32_t *xi = xb.xf_idx + x0;
  double *o = reinterpret_cast<double *>(L + ((int64_t)r * nbox + b) * P);
  const int ql = nx - 1, steps = (nx + 31) >> 5;
  for (int k0 = 0; k0 < P; k0 += KB) {
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    // past the end the last source again, with strength 0
    int jn = xi[min(hl + 32, ql)];
    const int j0 = xi[min(hl, ql)];
    double zx = xb.sx[j0], zy = xb.sy[j0];
    cx<double> pj = pr[j0];
    if (hl > ql) pj = cx<double>{0.0, 0.0};
    for (int st = 0; st < steps; ++st) {
      const int q1 = hl + 32 * (st + 1);
      const double nzx = xb.sx[jn], nzy = xb.sy[jn];
      cx<double> npj = pr[jn];
      jn = xi[min(q1 + 32, ql)];
      if (q1 > ql) npj = cx<double>{0.0, 0.0};
      const double ux = zx - cxb, uy = zy - cyb;
      const double d = rcp64(fma(ux, ux, uy * uy));
      const cx<double> iu{ux * d, -uy * d};
      const cx<double> rho = rb * iu;
      cx<double> t = pj * iu;
      t = cx<double>{-t.x, -t.y};
      if (k0 > 0) t = t * cpow(rho, k0);
#pragma unroll
      for (int l = 0; l < KB; ++l) {
        acc[2 * l] += t.x;
        acc[2 * l + 1] += t.y;
        t = t * rho;
      }
      zx = nzx;
      zy = nzy;
      pj = npj;
    }
    halving_steps_half<double, NV>(acc, lane);
#pragma unroll
    for (int c = 0; c < NV / 32; ++c) {  // lane hl of a half: values hl NV / 32 ..
      const int x = 2 * k0 + hl * (NV / 32) + c;
      if (has && x < 2 * P) o[x] = acc[c];
    }
  }
}

// ------------------------------------------------ upward / downward passes
template <typename T>
struct Chunk16;
template <>
struct Chunk16<float> {
  using type = float4;
};
template <>
struct Chunk16<double> {
  using type = double2;
};

// v (coefficients k, k + 1 in FP32; k in FP64) times tab[k], tab[k + 1]
template <typename T>
__device__ __forceinline__ void scale_chunk(typename Chunk16<T>::type &v, const cx<T> *tab,
                                            int k) {
  if constexpr (sizeof(T) == 4) {
    const cx<T> a = cx<T>{v.x, v.y} * tab[k], b = cx<T>{v.z, v.w} * tab[k + 1];
    v = make_float4(a.x, a.y, b.x, b.y);
  } else {
    const cx<T> a = cx<T>{v.x, v.y} * tab[k];
    v = make_double2(a.x, a.y);
  }
}

// One component of a pass program per work-group (PassProgram in tree.h),
// for right-hand side blockIdx.y.  Its inputs are staged in LDS with every
// load in flight at once, scaled as the program says; then its work boxes
// are finished level by level from LDS only, each also written to E:
//   upward    A_lo = 1/2 sum_q post[q][lo] sum_{k <= lo} C(lo, k) a~_{q,k},
//             a~ a child's multipole times pre[q_child]; the result is kept
//             times pre[q_box] for the box's parent
//   downward  b_m = own_m + pre[q][m] sum_{l >= m} C(l, m) c_l, c the
//             parent's local times post[q]; the result is passed on times
//             post[q_child] to each child of the component
// (C is zero off its triangle, so the fixed-length sums add exact zeros).
// Upward, an absent child reads a slot of zeros (slot CAP), so that the
// four quadrant sums run side by side without branches.  XL: work-groups
// past ncomp form P2L sums (run_pass).
constexpr int kPassThreads = 1024;
template <typename T, int P, bool DOWN, bool XL = false>
__global__ void __launch_bounds__(kPassThreads)
    k_pass(const int32_t *__restrict__ hdr, const int2 *__restrict__ ext,
           const int4 *__restrict__ par, const int32_t *__restrict__ stp,
           const T *__restrict__ Cb, const cx<T> *__restrict__ Pre,
           const cx<T> *__restrict__ Post, cx<T> *__restrict__ E, int nbox, int ncomp,
           XBoxes xb, const cx<T> *__restrict__ p, cx<T> *__restrict__ L) {
  using V = typename Chunk16<T>::type;
  if constexpr (XL) {
    if ((int)blockIdx.x >= ncomp) {  // block-uniform: P2L sums, two boxes a wave
      const int e = ((int)blockIdx.x - ncomp) * (kPassThreads / 64) + (int)(threadIdx.x >> 6);
      if (2 * e < xb.n) p2l_pair64<P, 16>(e, blockIdx.y, xb, p, L, nbox);
      return;
    }
  }
  constexpr int NT = kPassThreads, CAP = pass_cap(P, (int)sizeof(cx<T>));
  static_assert(P * (int)sizeof(cx<T>) % 16 == 0, "expansions of whole 16-byte chunks");
  constexpr int CH = P * (int)sizeof(cx<T>) / 16, IT = (CAP * CH + NT - 1) / NT;
  constexpr int CPC = 16 / (int)sizeof(cx<T>);  // coefficients per chunk
  __shared__ __align__(16) cx<T> sl[(CAP + 1) * P];  // expansion slots + zeros
  __shared__ int4 spd[CAP];                          // work boxes in step order
  __shared__ int32_t sst[kPassMaxSteps + 1];
  __shared__ T sC[P * P];  // upward C(lo, k) at k P + lo; downward C(l, m) at l P + m
  __shared__ cx<T> sPre[4 * P], sPost[4 * P];
  const int tid = threadIdx.x;
  const int32_t *h = hdr + 8 * (int64_t)blockIdx.x;
  const int ne = h[1], p0 = h[2], np = h[3], s0 = h[4], ns = h[5];
  cx<T> *Er = E + (int64_t)blockIdx.y * nbox * P;
  int2 d[IT];
  V v[IT];
  // ext: this component's CAP input slots (box -1 past #ext), read
  // without waiting for the header
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int e = tid + i * NT;
    d[i] = e < CAP * CH ? ext[(int64_t)blockIdx.x * CAP + e / CH] : make_int2(-1, 0);
  }
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int e = tid + i * NT;
    if (d[i].x >= 0) v[i] = reinterpret_cast<const V *>(Er + (int64_t)d[i].x * P)[e % CH];
  }
  for (int i = tid; i < np; i += NT) spd[i] = par[p0 + i];
  for (int i = tid; i <= ns; i += NT) sst[i] = stp[s0 + i];
  for (int i = tid; i < P * P; i += NT) sC[i] = DOWN ? Cb[i] : Cb[(i % P) * P + i / P];
  for (int i = tid; i < 4 * P; i += NT) {
    sPre[i] = Pre[i];
    sPost[i] = Post[i];
  }
  if (tid < P) sl[CAP * P + tid] = cx<T>{T(0), T(0)};
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int e = tid + i * NT;
    if (e < ne * CH) {  // slot e / CH, chunk e % CH
      const int mode = d[i].y & 3, q = d[i].y >> 2, k = (e % CH) * CPC;
      if (mode == 1) scale_chunk<T>(v[i], sPre + q * P, k);
      else if (mode == 2) scale_chunk<T>(v[i], sPost + q * P, k);
      reinterpret_cast<V *>(sl)[e] = v[i];
    }
  }
  __syncthreads();
  for (int st = 0; st < ns; ++st) {
    const int a = sst[st], b = sst[st + 1];
    if constexpr (!DOWN) {
      if ((b - a) * P * 4 <= NT) {  // uniform
        // a step of few boxes: four lanes per (box, coefficient), one child
        // quadrant each, so that the chain per lane is short; the quadrant
        // sums meet by two cross-lane steps (it & 3 = tid & 3: NT is a
        // multiple of 4, and the four lanes of a group are active together)
        for (int it = tid; it < (b - a) * P * 4; it += NT) {
          const int qq = it & 3, jm = it >> 2;
          const int j = a + jm / P, m = jm % P;
          const int4 pd = spd[j];
          const int box = pd.x & 0x3FFFFFFF, q = (int)((uint32_t)pd.x >> 30);
          const int w = qq < 2 ? pd.z : pd.w;
          const int sq = (qq & 1) ? (int)((uint32_t)w >> 16) : (w & 0xFFFF);
          const cx<T> *ak = sl + (sq == kPassNone ? CAP : sq) * P;
          cx<T> sum{T(0), T(0)};
#pragma unroll
          for (int k = 0; k < P; ++k) sum = sum + sC[k * P + m] * ak[k];
          cx<T> acc = sPost[qq * P + m] * sum;
          acc.x += __shfl_xor(acc.x, 1, 64);
          acc.y += __shfl_xor(acc.y, 1, 64);
          acc.x += __shfl_xor(acc.x, 2, 64);
          acc.y += __shfl_xor(acc.y, 2, 64);
          if (qq == 0) {
            const cx<T> A = T(0.5) * acc;
            Er[(int64_t)box * P + m] = A;
            sl[(ne + j) * P + m] = A * sPre[q * P + m];
          }
        }
      } else {
        // one lane per (box, coefficient), the four quadrant sums side by side
        for (int it = tid; it < (b - a) * P; it += NT) {
          const int j = a + it / P, m = it % P;
          const int4 pd = spd[j];
          const int box = pd.x & 0x3FFFFFFF, q = (int)((uint32_t)pd.x >> 30);
          const int s4[4] = {pd.z & 0xFFFF, (int)((uint32_t)pd.z >> 16), pd.w & 0xFFFF,
                             (int)((uint32_t)pd.w >> 16)};
          cx<T> sum[4];
          const cx<T> *ak[4];
#pragma unroll
          for (int qq = 0; qq < 4; ++qq) {
            ak[qq] = sl + (s4[qq] == kPassNone ? CAP : s4[qq]) * P;
            sum[qq] = cx<T>{T(0), T(0)};
          }
#pragma unroll
          for (int k = 0; k < P; ++k) {
            const T c = sC[k * P + m];
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) sum[qq] = sum[qq] + c * ak[qq][k];
          }
          // the quadrant terms added as the four-lane form adds them
          const cx<T> t0 = sPost[m] * sum[0], t1 = sPost[P + m] * sum[1];
          const cx<T> t2 = sPost[2 * P + m] * sum[2], t3 = sPost[3 * P + m] * sum[3];
          const cx<T> A = T(0.5) * ((t0 + t1) + (t2 + t3));
          Er[(int64_t)box * P + m] = A;
          sl[(ne + j) * P + m] = A * sPre[q * P + m];
        }
      }
    } else {
      for (int it = tid; it < (b - a) * P; it += NT) {
        const int j = a + it / P, m = it % P;
        const int4 pd = spd[j];
        const int box = pd.x & 0x3FFFFFFF, q = (int)((uint32_t)pd.x >> 30);
        const int s4[4] = {pd.z & 0xFFFF, (int)((uint32_t)pd.z >> 16), pd.w & 0xFFFF,
                           (int)((uint32_t)pd.w >> 16)};
        const int own = pd.y & 0xFFFF, ver = (int)((uint32_t)pd.y >> 16);
        cx<T> val = sl[own * P + m];
        if (ver != kPassNone) {
          const cx<T> *cl = sl + ver * P;
          cx<T> s2[2] = {cx<T>{T(0), T(0)}, cx<T>{T(0), T(0)}};
#pragma unroll
          for (int l = 0; l < P; ++l) s2[l & 1] = s2[l & 1] + sC[l * P + m] * cl[l];
          val = val + sPre[q * P + m] * (s2[0] + s2[1]);
        }
        Er[(int64_t)box * P + m] = val;
#pragma unroll
        for (int qq = 0; qq < 4; ++qq)
          if (s4[qq] != kPassNone) sl[s4[qq] * P + m] = sPost[qq * P + m] * val;
      }
    }
    __syncthreads();
  }
}

// The rounds of a pass program, one launch each; the first launch of an
// upward FP64 pass also forms the P2L sums of the boxes xb (strengths p,
// stored to L) while they are at most kP2LGroups work-groups: the pass
// leaves most of the chip idle then and they cost no launch and no time
// ((I + K) at 20k nodes 68.9 us against 71.7 with a launch of their own, 77k
// the same; 1.02M, where the pass fills the chip, 442 against 426).  Returns
// whether it did.
constexpr int kP2LGroups = 128;
template <typename T, int P, bool DOWN>
static bool run_pass(const DevPass &pg, const T *bc, const cx<T> *pre, const cx<T> *post,
                     cx<T> *E, int nbox, int nrhs, hipStream_t s, XBoxes xb = XBoxes{},
                     const cx<T> *p = nullptr, cx<T> *L = nullptr) {
  bool p2l = false;
  if (pg.cap != pass_cap(P, (int)sizeof(cx<T>)))
    throw ApiError{LBS_ERR_UNSUPPORTED, "pass program built for another expansion order"};
  for (size_t k = 0; k + 1 < pg.round_ptr.size(); ++k) {
    const int a = pg.round_ptr[k], n = pg.round_ptr[k + 1] - a;
    if (n <= 0) continue;
    // (a wave takes two boxes, a work-group kPassThreads / 64 waves)
    const int per = kPassThreads / 32, xg = (xb.n + per - 1) / per;
    const int nx = !p2l && xg > 0 && xg * nrhs <= kP2LGroups ? xg : 0;
    p2l = p2l || nx > 0;
    const auto kern = nx > 0 ? k_pass<T, P, DOWN, sizeof(T) == 8 && !DOWN> : k_pass<T, P, DOWN>;
    hipLaunchKernelGGL(kern, dim3(n + nx, nrhs), dim3(kPassThreads), 0, s,
                       pg.hdr.p + 8 * (int64_t)a,
                       reinterpret_cast<const int2 *>(pg.ext.p) + (int64_t)a * pg.cap,
                       reinterpret_cast<const int4 *>(pg.par.p), pg.stp.p, bc, pre, post, E,
                       nbox, n, xb, p, L);
  }
  return p2l;
}

template <int P>
struct Groups {
  static constexpr int G = 64 / P;
};

// P2L parts of one box's local expansion into px (values 2k, 2k + 1 of
// coefficient k), KB coefficients per pass (p2l_sum).
template <typename T, int P, int K0>
__device__ __forceinline__ void p2l_pass_lds(int64_t xf0, int total,
                                             const int32_t *__restrict__ xf_idx,
                                             double cxb, double cyb, T rb,
                                             const double *__restrict__ sx,
                                             const double *__restrict__ sy,
                                             const cx<T> *__restrict__ pr, T *px, int lane) {
  if constexpr (K0 < P) {
    constexpr int KB = kChunk<T, P>(), NV = pow2_ceil(2 * KB),
                  SH = 6 - log2_exact(NV);
    const T tot = p2l_sum<T, P, K0, KB>(xf0, total, xf_idx, cxb, cyb, rb, sx,
                                        sy, pr, lane);
    const int vi = lane >> SH;
    if ((lane & ((1 << SH) - 1)) == 0 && vi < 2 * KB && 2 * K0 + vi < 2 * P)
      px[2 * K0 + vi] = tot;
    p2l_pass_lds<T, P, K0 + KB>(xf0, total, xf_idx, cxb, cyb, rb, sx, sy, pr, px, lane);
  }
}

// M2L over the V list of every box with targets at level >= 2 (vector ALU;
// FP32 orders other than 16).  One 64-lane block per box; lane (g, l)
// accumulates coefficient l from every G-th list entry with the factorized
// translation b_l += tau^-l sum_k H[l][k] (tau^-k a_k),
// H[l][k] = (-1)^k C(k+l-1, l).
// The box's P2L sum over its X list (every box with an X list whose local
// expansion is used is one of these boxes) follows in the same block and
// is added to the M2L result before the one store.
template <typename T, int P>
__global__ void __launch_bounds__(64)
    k_m2l(const int32_t *__restrict__ boxes,
          const int32_t *__restrict__ v_ptr, const int32_t *__restrict__ v_src,
          const uint8_t *__restrict__ v_code, const T *__restrict__ H,
          const cx<T> *__restrict__ itp, const cx<T> *__restrict__ M,
          cx<T> *__restrict__ L, int nbox, const int64_t *__restrict__ xf_ptr,
          const int32_t *__restrict__ xf_idx, const double *__restrict__ cxv,
          const double *__restrict__ cyv, const double *__restrict__ rad,
          const double *__restrict__ sx, const double *__restrict__ sy,
          const cx<T> *__restrict__ p, int64_t ns) {
  constexpr int G = Groups<P>::G;
  constexpr int NP = 2 * P + 1;
  __shared__ cx<T> ybuf[G][P];
  __shared__ cx<T> red[G][P];
  __shared__ T px[2 * P];
  const int b = boxes[blockIdx.x];
  const int r = blockIdx.y;
  const int lane = threadIdx.x;
  const int g = lane / P, l = lane % P;
  const bool act = g < G;
  T hrow[P];
#pragma unroll
  for (int k = 0; k < P; ++k) hrow[k] = act ? H[l * P + k] : T(0);
  cx<T> acc{T(0), T(0)};
  const cx<T> *Mr = M + (int64_t)r * nbox * P;
  const int vb = v_ptr[b], nv = v_ptr[b + 1] - vb;
  for (int base = 0; base < nv; base += G) {
    const int v = base + g;
    const bool ok = act && v < nv;
    int code = 0;
    if (ok) {
      const int src = v_src[vb + v];
      code = v_code[vb + v];
      ybuf[g][l] = itp[code * NP + l + 1] * Mr[(int64_t)src * P + l];
    }
    __syncthreads();
    if (ok) {
      cx<T> z{T(0), T(0)};
#pragma unroll
      for (int k = 0; k < P; ++k) z = z + hrow[k] * ybuf[g][k];
      acc = acc + itp[code * NP + l] * z;
    }
    __syncthreads();
  }
  if (act) red[g][l] = acc;
  const int64_t xf0 = xf_ptr[b];
  const int nx = (int)(xf_ptr[b + 1] - xf0);  // block-uniform
  if (nx > 0)
    p2l_pass_lds<T, P, 0>(xf0, nx, xf_idx, cxv[b], cyv[b], T(rad[b]), sx, sy,
                          p + (int64_t)r * ns, px, lane);
  __syncthreads();
  if (act && g == 0) {
    cx<T> s = red[0][l];
#pragma unroll
    for (int gg = 1; gg < G; ++gg) s = s + red[gg][l];
    if (nx > 0) s = s + cx<T>{px[2 * l], px[2 * l + 1]};
    L[((int64_t)r * nbox + b) * P + l] = s;
  }
}

// M2L for FP32 expansions of 16 terms on the matrix cores, followed by the
// box's P2L sum (p2l_sum).  One wave per target box.  For 8 V-list sources
// at a time the wave forms
// Y[k][2v + part] = part(tau_v^-(k+1) a_{v,k+1}) (16 x 16), multiplies
// Z = H Y with four v_mfma_f32_16x16x4f32 (H: 16 x 16, real), then scales
// column pair (2v, 2v+1) of Z by tau_v^-l and accumulates.  Lane layout of
// the 16x16x4 instruction: A[i][k] in lane i + 16 k, B[k][j] in lane
// j + 16 k, D[i][j] in lane j + 16 (i / 4), register i % 4.
typedef float v4f __attribute__((ext_vector_type(4)));

// The X-list sources of the boxes for the P2L sums folded into the FP32
// M2L (per-box ranges xf_ptr into the concatenated source indices xf_idx;
// box centres (bx, by) and half-widths rad).
struct XListSrc {
  const int64_t *xf_ptr;
  const int32_t *xf_idx;
  const double *bx, *by, *rad, *sx, *sy;
  const cx<float> *p;
  int64_t ns;
};

__global__ void __launch_bounds__(256)
    k_m2l_mfma16(int nb, const int32_t *__restrict__ boxes,
                 const int32_t *__restrict__ v_ptr,
                 const int32_t *__restrict__ v_src,
                 const uint8_t *__restrict__ v_code,
                 const float *__restrict__ H, const cx<float> *__restrict__ itp,
                 const cx<float> *__restrict__ M, cx<float> *__restrict__ L,
                 int nbox, XListSrc xs, GammaGroups gg) {
  constexpr int P = 16, NP = 2 * P + 1;
  if ((int)blockIdx.x >= gg.first) {  // block-uniform: a correction chunk
    const int x = blockIdx.x - gg.first;
    gamma_chunk(x % gg.nchunk, x / gg.nchunk, blockIdx.y, gg.nchunk, gg.gl_ptr,
                gg.gpart, gg.nls, gg.G, gg.csum, gg.cnt, gg.gamma);
    return;
  }
  // the 49 x (2P + 1) table of tau^-n, read by every pair, in LDS
  __shared__ cx<float> sItp[49 * NP];
  for (int i = threadIdx.x; i < 49 * NP; i += 256) sItp[i] = itp[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.y;
  const int col = lane & 15, kq = lane >> 4;
  const int vslot = col >> 1, part = col & 1;
  float a[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = H[col * P + 4 * s + kq];
  // each wave takes every (4 x #M2L groups)-th box, so that the table
  // above is read once per block for several boxes; the next box's id and
  // list offsets are loaded while this box is worked on (box ids two
  // ahead, offsets one ahead; past the end, box 0 stands in)
  const int stride = 4 * gg.first;
  int wv = blockIdx.x * 4 + (threadIdx.x >> 6);
  int b = wv < nb ? boxes[wv] : 0;
  int bn = wv + stride < nb ? boxes[wv + stride] : 0;
  int vb = v_ptr[b], ve = v_ptr[b + 1];
  int64_t xb0 = xs.xf_ptr[b], xb1 = xs.xf_ptr[b + 1];
  for (; wv < nb; wv += stride) {
    const int nv = ve - vb;
    const int64_t x0 = xb0;
    const int xt = (int)(xb1 - xb0);
    const int bc = b;
    b = bn;
    bn = wv + 2 * stride < nb ? boxes[wv + 2 * stride] : 0;
    const int vbc = vb;
    vb = v_ptr[b];
    ve = v_ptr[b + 1];
    xb0 = xs.xf_ptr[b];
    xb1 = xs.xf_ptr[b + 1];
    const cx<float> *Mr = M + (int64_t)r * nbox * P;
    // the box's list entries, lane e holding entry e (a V list has at most
    // 27 entries; any beyond 64 are read directly)
    int esrc = 0, ecode = 0;
    if (lane < nv) {
      esrc = v_src[vbc + lane];
      ecode = v_code[vbc + lane];
    }
    // multipole coefficients k = 4 s + kq of the batch's source vslot
    auto fetch = [&](int base, cx<float> (&mv)[4], int &code, bool &ok) {
      const int v = base + vslot;
      ok = v < nv;
      int src = __shfl(esrc, v & 63, 64);
      code = __shfl(ecode, v & 63, 64);
      if (ok && v >= 64) {
        src = v_src[vbc + v];
        code = v_code[vbc + v];
      }
      if (!ok) src = code = 0;
      const cx<float> *ms = Mr + (int64_t)src * P;
#pragma unroll
      for (int s = 0; s < 4; ++s) mv[s] = ok ? ms[4 * s + kq] : cx<float>{0.f, 0.f};
    };
    float accr[4] = {0.f, 0.f, 0.f, 0.f}, acci[4] = {0.f, 0.f, 0.f, 0.f};
    cx<float> mcur[4], mnxt[4];
    int ccur, cnxt = 0;
    bool okc, oknx = false;
    fetch(0, mcur, ccur, okc);
    for (int base = 0; base < nv; base += 8) {
      // the next batch's loads go out before this batch's products
      if (base + 8 < nv) fetch(base + 8, mnxt, cnxt, oknx);  // wave-uniform
      const bool ok = okc;
      const cx<float> *ip = sItp + ccur * NP;
      v4f d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = 4 * s + kq;
        const cx<float> y = ip[k + 1] * mcur[s];
        const float bv = ok ? (part ? y.y : y.x) : 0.f;
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bv, d, 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float mine = d[j];
        const float other = __shfl_xor(mine, 1, 64);
        if (ok && part == 0) {
          const cx<float> t = ip[4 * kq + j] * cx<float>{mine, other};
          accr[j] += t.x;
          acci[j] += t.y;
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) mcur[s] = mnxt[s];
      ccur = cnxt;
      okc = oknx;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      for (int off = 2; off < 16; off <<= 1) {
        accr[j] += __shfl_xor(accr[j], off, 64);
        acci[j] += __shfl_xor(acci[j], off, 64);
      }
    }
    // P2L over the box's X list: the real part of coefficient l ends in
    // lane 4 l, the imaginary part in lane 4 l + 2
    if (xt > 0) {  // wave-uniform
      const float v = p2l_sum<float, P, 0, P>(x0, xt, xs.xf_idx, xs.bx[bc],
                                              xs.by[bc], float(xs.rad[bc]),
                                              xs.sx, xs.sy,
                                              xs.p + (int64_t)r * xs.ns, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        accr[j] += __shfl(v, (lane & 48) + 4 * j, 64);
        acci[j] += __shfl(v, (lane & 48) + 4 * j + 2, 64);
      }
    }
    if (col == 0) {
      cx<float> *dst = L + ((int64_t)r * nbox + bc) * P + 4 * kq;
#pragma unroll
      for (int j = 0; j < 4; ++j) dst[j] = cx<float>{accr[j], acci[j]};
    }
  }
}

// x of the lane's neighbour (lane ^ 1)
__device__ __forceinline__ double lane_xor1(double x) {
  const unsigned long long u = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)u, 0xB1, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), 0xB1, 0xF, 0xF, true);
  return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

typedef double v4d __attribute__((ext_vector_type(4)));

// M2L over the V lists of a group of boxes at level >= 2 (FP64, matrix
// cores).  For eight list entries at a time a wave forms
// Y[k][2 v + part] = part(tau_v^-(k+1) a_{v,k+1}), multiplies Z = H Y with
// v_mfma_f64_16x16x4f64 (H[l][k] = (-1)^k C(k+l-1, l), held in registers),
// scales column pair v by tau_v^-l and writes it to LDS, where one lane per
// (box, coefficient part) adds the box's entries (and, with add_x, the P2L
// sum that boxes with an X list hold already).  Lane layout of the 16x16x4
// instruction: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k, D[i][j]
// in lane j + 16 (i % 4), register i / 4.
//
// Bound by the latency of the gathers and of the exchange; the matrix cores
// are 0.33 busy (counters over the benchmark's applications: 1.02M nodes,
// 536k entries, about 93 us a launch; the vector form that this replaces took 168
// with the P2L sums, which now take 43 in a launch of their own there).  That
// form broadcast y through LDS, 16 bytes read per two multiply-adds and lane,
// four times what the LDS delivers beside them.  Forms compared by repeated
// applications on warm caches, where this one took 83 us: rows of H in scalar
// registers with one entry per lane 105 (a wave waits for each row), a
// persistent form that reads one batch ahead 90 (158 registers, three waves a
// SIMD), two and eight waves a group 96 and 109; groups of 32 entries 80.
constexpr int kM2LWaves = 4;  // (gamma_chunk takes 256 threads)
template <int P>
__global__ void __launch_bounds__(64 * kM2LWaves)
    k_m2l64(int ngrp, const int2 *__restrict__ ent, const int2 *__restrict__ gbox,
            const double *__restrict__ H,
            const cx<double> *__restrict__ M, cx<double> *__restrict__ L, int nbox, int add_x,
            GammaGroups gg) {
  constexpr int NT = (P + 15) / 16, NS = (P + 3) / 4, ROW = kM2LEnt + 1;
  if ((int)blockIdx.x >= ngrp) {   // block-uniform: a correction chunk
    const int x = blockIdx.x - ngrp;
    gamma_chunk(x % gg.nchunk, x / gg.nchunk, blockIdx.y, gg.nchunk, gg.gl_ptr, gg.gpart,
                gg.nls, gg.G, gg.csum, gg.cnt, gg.gamma);
    return;
  }
  extern __shared__ __align__(16) double tb[];  // [2 P][entry]
  __shared__ int2 sbox[kM2LBoxes];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = kM2LWaves;
  const int lane = threadIdx.x & 63, r = blockIdx.y;
  const int col = lane & 15, kq = lane >> 4, part = col & 1;
  const int2 mine = ent[(int64_t)blockIdx.x * kM2LEnt + (lane & (kM2LEnt - 1))];
  const int2 bx = gbox[blockIdx.x * kM2LBoxes + (lane & (kM2LBoxes - 1))];
  if (threadIdx.x < kM2LBoxes) sbox[threadIdx.x] = bx;
  const int total = __shfl(bx.y, kM2LBoxes - 1, 64) & 0xFFFF;  // list entries of the group
  if (8 * wv < total) {
    double a[NT][NS];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int l = 16 * t + col, k = 4 * s + kq;
        a[t][s] = l < P && k < P ? H[l * P + k] : 0.0;
      }
    for (int v0 = 8 * wv; v0 < total; v0 += 8 * W) {
      const int v = v0 + (col >> 1);
      const int src = __shfl(mine.x, v, 64), code = __shfl(mine.y, v, 64);
      const cx<double> *ms = M + ((int64_t)r * nbox + max(src, 0)) * P;
      cx<double> m[NS];  // multipole coefficients k = 4 s + kq of the column's entry
#pragma unroll
      for (int s = 0; s < NS; ++s) m[s] = 4 * s + kq < P ? ms[4 * s + kq] : cx<double>{0.0, 0.0};
      const double tx = 2.0 * (code / 7 - 3), ty = 2.0 * (code % 7 - 3);
      const double id = src < 0 ? 0.0 : 1.0 / (tx * tx + ty * ty);
      const cx<double> w{tx * id, -ty * id};  // 1 / tau (0 past the last entry)
      const cx<double> w2 = w * w, w4 = w2 * w2;
      cx<double> q = kq & 1 ? w2 : w;         // w^(kq + 1), times -i for the
      if (kq & 2) q = q * w2;                 // imaginary column: Im y = Re(-i y)
      if (part) q = cx<double>{q.y, -q.x};
      v4d d[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) d[t] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double y = fma(q.x, m[s].x, -(q.y * m[s].y));
        q = q * w4;
#pragma unroll
        for (int t = 0; t < NT; ++t)
          d[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t][s], y, d[t], 0, 0, 0);
      }
      // row l = 16 t + 4 j + kq: part(tau^-l z) = u^l.x mine + u^l.y other
      // with u = conj(w) (real part) or w (imaginary part)
      const double sg = part ? 1.0 : -1.0;
      const cx<double> u4{w4.x, sg * w4.y}, u1{w.x, sg * w.y}, u2{w2.x, sg * w2.y};
      cx<double> ul = kq & 1 ? u1 : cx<double>{1.0, 0.0};
      if (kq & 2) ul = ul * u2;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double mz = d[t][j], other = lane_xor1(mz);
          const int l = 16 * t + 4 * j + kq;
          if (l < P) tb[(2 * l + part) * ROW + v] = fma(ul.x, mz, ul.y * other);
          ul = ul * u4;
        }
    }
  }
  __syncthreads();
  // one lane per (box, coefficient part): the box's entries, eight in flight
  for (int x = threadIdx.x; x < kM2LBoxes * 2 * P; x += blockDim.x) {
    const int i = x / (2 * P), c = x % (2 * P);
    const int2 gb = sbox[i];
    if (gb.x < 0) break;
    const int t1 = gb.y & 0xFFFF, t0 = i > 0 ? sbox[i - 1].y & 0xFFFF : 0;
    double *o = reinterpret_cast<double *>(L + ((int64_t)r * nbox + gb.x) * P) + c;
    double s = add_x && (gb.y >> 16) ? *o : 0.0;
    for (int t = t0; t < t1; t += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = tb[c * ROW + min(t + u, t1 - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += t + u < t1 ? v[u] : 0.0;
    }
    *o = s;
  }
}

template <int P>
__global__ void __launch_bounds__(64)
    k_p2l64(XBoxes xb, const cx<double> *__restrict__ p, cx<double> *__restrict__ L, int nbox) {
  p2l_pair64<P, 32>(blockIdx.x, blockIdx.y, xb, p, L, nbox);
}

// Launch of k_m2l64 over the plan's groups, with the correction sums of gg
// as extra work-groups when gg.nchunk > 0; add_x: boxes with an X list hold
// their P2L sum already.
template <int P>
static void launch_m2l64(const DevPlan &pl, const double *H, const cx<double> *M,
                         cx<double> *L, bool add_x, int nrhs, GammaGroups gg, hipStream_t s) {
  const int ng = pl.n_grp, W = kM2LWaves;
  const size_t lds = (size_t)2 * P * (kM2LEnt + 1) * sizeof(double);
  hipLaunchKernelGGL((k_m2l64<P>), dim3(ng + gg.nchunk * gg.G, nrhs), dim3(64 * W), lds, s, ng,
                     pl.grp_ent.p, pl.grp_box.p, H, M, L, pl.nbox, (int)add_x, gg);
}


// P2L over the X list of one box per wave (p2l_sum, KB coefficients per
// pass), added to the M2L result.
template <typename T, int P, int K0>
__device__ __forceinline__ void p2l_pass(int64_t xf0, int total,
                                         const int32_t *__restrict__ xf_idx,
                                         double cxb, double cyb, T rb,
                                         const double *__restrict__ sx,
                                         const double *__restrict__ sy,
                                         const cx<T> *__restrict__ pr,
                                         T *__restrict__ Lb, int lane) {
  if constexpr (K0 < P) {
    constexpr int KB = kChunk<T, P>(), NV = pow2_ceil(2 * KB),
                  SH = 6 - log2_exact(NV);
    const T tot = p2l_sum<T, P, K0, KB>(xf0, total, xf_idx, cxb, cyb, rb, sx,
                                        sy, pr, lane);
    const int vi = lane >> SH;
    if ((lane & ((1 << SH) - 1)) == 0 && vi < 2 * KB && 2 * K0 + vi < 2 * P)
      Lb[2 * K0 + vi] += tot;
    p2l_pass<T, P, K0 + KB>(xf0, total, xf_idx, cxb, cyb, rb, sx, sy, pr, Lb,
                            lane);
  }
}

template <typename T, int P>
__global__ void __launch_bounds__(64)
    k_p2l(const int32_t *__restrict__ boxes, const int64_t *__restrict__ xf_ptr,
          const int32_t *__restrict__ xf_idx, const double *__restrict__ cxv,
          const double *__restrict__ cyv, const double *__restrict__ rad,
          const double *__restrict__ sx, const double *__restrict__ sy,
          const cx<T> *__restrict__ p, int64_t ns, cx<T> *__restrict__ L,
          int nbox) {
  const int b = boxes[blockIdx.x];
  const int r = blockIdx.y;
  const int64_t xf0 = xf_ptr[b];
  if (xf_ptr[b + 1] == xf0) return;  // nothing to add (the whole wave)
  p2l_pass<T, P, 0>(xf0, (int)(xf_ptr[b + 1] - xf0), xf_idx, cxv[b], cyv[b],
                    T(rad[b]), sx, sy, p + (int64_t)r * ns,
                    reinterpret_cast<T *>(L + ((int64_t)r * nbox + b) * P),
                    (int)threadIdx.x);
}

__device__ __forceinline__ int pow2_at_least(int n) {
  int t = 1;
  while (t < n) t <<= 1;
  return t;
}

constexpr int kStage = 128;  // U-list sources staged in LDS per pass
constexpr int kLeafSlices = 16;  // parts of a target one lane adds (FP64 leaf kernel)
constexpr int kFarItems = 8;  // expansions staged in LDS per pass (FP64 leaf kernel)

// What the FP64 leaf kernel forms at a target.
enum LeafMode {
  kLeafField = 0,  // Re Psi for RB right-hand sides, then the assembled row
  kLeafPsi = 1,    // Psi, complex
  kLeafDeriv = 2   // Psi and Psi', complex
};
template <int MODE, int RB>
constexpr int leaf_values() { return MODE == kLeafField ? RB : 2 * MODE; }

// The near field of one leaf's targets [0, nt), nt <= 64, for K <= 4 targets
// per lane: lanes are (target t mod tp, slice) with tp = 2^lg <= 16, lane
// target t + tp k for k < K, and S = 64 W / tp slices, each taking every
// S-th staged source.  A source is read from LDS once for the K targets of
// a lane, whose reciprocal chains run side by side.  `fin` gets the partial
// sums, one value c of every target at a time.
template <int MODE, int RB, int K, typename Stage, typename Fin>
__device__ __forceinline__ void near_field64(int nt, int lg, int utot, int stage_n,
                                             const double *__restrict__ tx,
                                             const double *__restrict__ ty,
                                             const double2 *__restrict__ sz,
                                             const double2 *__restrict__ sp, const Stage &stage,
                                             const Fin &fin) {
  constexpr int NF = leaf_values<MODE, RB>(), UN = K >= 4 ? 1 : K >= 2 ? 2 : 4;
  const int tp = 1 << lg, S = (int)blockDim.x >> lg;
  const int tl = threadIdx.x & (tp - 1), sl = threadIdx.x >> lg;
  double zx[K], zy[K], f[K][NF];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int t = min(tl + tp * k, nt - 1);  // past the end: discarded
    zx[k] = tx[t];
    zy[k] = ty[t];
#pragma unroll
    for (int c = 0; c < NF; ++c) f[k][c] = 0.0;
  }
  for (int q0 = 0; q0 < utot; q0 += stage_n) {
    const int take = min(stage_n, utot - q0);
    // padded to a multiple of S with sources of zero strength at the
    // origin, which add 0 * rcp(|z|^2 + 1e-300) = 0
    const int tpad = (take + S - 1) & ~(S - 1);  // S: a power of two
    stage(q0, take, tpad);
    __syncthreads();
#pragma unroll UN
    for (int q = sl; q < tpad; q += S) {
      const double2 s2 = sz[q];
      double2 p2[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) p2[r] = sp[q * RB + r];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double dx = zx[k] - s2.x, dy = zy[k] - s2.y;
        // |d|^2 + 1e-300: a target's own source (d = 0) contributes
        // 0 * rcp(1e-300) = 0; any other |d|^2 above 1e-284 is unchanged
        const double inv = rcp64(fma(dx, dx, fma(dy, dy, 1e-300)));
        if constexpr (MODE == kLeafField && RB == 1) {
          f[k][0] = fma(fma(p2[0].x, dx, p2[0].y * dy), inv, f[k][0]);
        } else if constexpr (MODE == kLeafField) {
          const double ux = dx * inv, uy = dy * inv;
#pragma unroll
          for (int r = 0; r < RB; ++r) f[k][r] = fma(p2[r].x, ux, fma(p2[r].y, uy, f[k][r]));
        } else {
          const cx<double> iv{dx * inv, -dy * inv};
          const cx<double> t = cx<double>{p2[0].x, p2[0].y} * iv;
          f[k][0] += t.x;
          f[k][1] += t.y;
          if constexpr (MODE == kLeafDeriv) {
            const cx<double> d = t * iv;
            f[k][2] -= d.x;
            f[k][3] -= d.y;
          }
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < NF; ++c) {
    double v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = f[k][c];
    fin(c, sl, tl, tp, S, v, std::integral_constant<int, K>{});
  }
}

// Potential at the targets of one leaf (one work-group of W = blockDim / 64
// waves): the leaf's local expansion and M2P over its W list with one lane
// per (target, slice of the list), then the direct sum over the gathered
// sources of its U list (near_field64; the self pair excluded by d == 0),
// all parts joined in LDS by one lane per target, which writes the row:
// kLeafField the assembled operator row in API order for the RB right-hand
// sides blockIdx.y RB .. (those < nrhs), kLeafPsi / kLeafDeriv the complex
// field (and derivative) of one right-hand side.  ufp, when set, replaces
// the leaf's own U range (boxes' ranges into uf_idx).
//
// Bound by VALU issue at large node counts: 14 issue slots a pair (10 FP64
// instructions, the reciprocal estimate four slots) over 218M pairs are 90
// us at 1.02M nodes (leaf 64), where the kernel takes about 175 in the benchmark's
// applications (208 before) and 161 in repeated ones (184).  One target per
// lane, which this form replaces, read 32 bytes of LDS per pair and lane, as
// long as the arithmetic takes, and read every expansion coefficient by a
// vector load per lane; at 77k nodes it took 73 us (now 28) and at 20k 45
// (now 18), where it left most of the chip idle.  Coefficients by scalar
// loads took 212 us (a wave waits for each chunk), sources read one stage
// ahead 167.  Six waves per SIMD leave the real field of one column 80
// registers, one too few: two are spilled, 16 MB of scratch writes a launch
// beside the 9 MB of results.  The derivative's form keeps 40 bytes a lane in
// scratch.
template <int P, int MODE, int RB>
__global__ void __launch_bounds__(256, MODE == kLeafField && RB == 1 ? 6 : 3)
    k_leaf64(const LeafHdr *__restrict__ hdr,
             const double *__restrict__ cxv, const double *__restrict__ cyv,
             const double *__restrict__ rad,
             const double *__restrict__ tx, const double *__restrict__ ty,
             const int64_t *__restrict__ tperm,
             const int64_t *__restrict__ ufp,
             const int32_t *__restrict__ uf_idx,
             const int32_t *__restrict__ w_src,
             const double *__restrict__ sx, const double *__restrict__ sy,
             const cx<double> *__restrict__ p, int64_t ns,
             const cx<double> *__restrict__ M,
             const cx<double> *__restrict__ L, int nbox, int nrhs,
             double *__restrict__ out, double *__restrict__ dout, int64_t ldy, double scale,
             Assembly as) {
  constexpr int NF = leaf_values<MODE, RB>();
  // sources (kStage per wave: position, RB strengths), or the partial sums
  extern __shared__ __align__(16) double sh[];
  const LeafHdr &hd = hdr[blockIdx.x];
  const int b = hd.b;
  const int r0 = blockIdx.y * RB, nr = min(RB, nrhs - r0);
  const int tid = threadIdx.x, nth = blockDim.x, W = nth >> 6;
  const int stage_n = kStage * min(W, 2);
  double2 *sz = reinterpret_cast<double2 *>(sh), *sp = sz + stage_n;
  const int64_t tb0 = hd.t0, ntb = hd.nt;
  const int64_t uf0 = ufp ? ufp[b] : hd.uf0;
  const int utot = (int)((ufp ? ufp[b + 1] : hd.uf1) - uf0);  // U-list sources
  const int wb = hd.wb, we = hd.we;
  const bool has_local = hd.lev >= 2;
  const double ir_b = hd.ir, cx_b = hd.cx, cy_b = hd.cy;
  for (int64_t tc0 = 0; tc0 < ntb; tc0 += 64) {
    const int nt = (int)min<int64_t>(64, ntb - tc0);
    const double *txc = tx + tb0 + tc0, *tyc = ty + tb0 + tc0;
    // far part: the items (the local expansion, then the W-list boxes)
    // staged in LDS, `ni` at a time, with lanes (target, slice of items)
    const int lgf = __builtin_ctz(pow2_at_least(nt)), Sf = nth >> lgf;
    const int ft = tid & ((1 << lgf) - 1), fs = tid >> lgf;
    double far[NF];
#pragma unroll
    for (int c = 0; c < NF; ++c) far[c] = 0.0;
    const double zx = txc[min(ft, nt - 1)], zy = tyc[min(ft, nt - 1)];
    double4 *geo = reinterpret_cast<double4 *>(sh);  // centre, rad or -1 / rad
    cx<double> *co = reinterpret_cast<cx<double> *>(geo + kFarItems);
    for (int i0 = has_local ? 0 : 1; i0 < 1 + we - wb; i0 += kFarItems) {
      const int ni = min(kFarItems, 1 + we - wb - i0);
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        if (r >= nr) continue;  // uniform
        for (int x = tid; x < ni * P; x += nth) {
          const int i = i0 + x / P, k = x % P;
          co[x] = i == 0 ? L[((int64_t)(r0 + r) * nbox + b) * P + k]
                         : M[((int64_t)(r0 + r) * nbox + w_src[wb + i - 1]) * P + k];
        }
        if (r == 0 && tid < ni) {
          if (i0 + tid == 0) {
            geo[tid] = make_double4(cx_b, cy_b, -ir_b, 0.0);
          } else {
            const int cw = w_src[wb + i0 + tid - 1];
            geo[tid] = make_double4(cxv[cw], cyv[cw], rad[cw], 0.0);
          }
        }
        __syncthreads();
        for (int i = fs; i < ni; i += Sf) {
          const double4 g4 = geo[i];
          const double dx = zx - g4.x, dy = zy - g4.y;
          const bool local = g4.z < 0.0;
          // local: w = d / rad and sum_l b_l w^l; W box: rho = rad / d and
          // sum_k a_k rho^k
          const double i2 = rcp64(fma(dx, dx, dy * dy));
          const cx<double> iz{dx * i2, -dy * i2};
          const cx<double> w{local ? -g4.z * dx : g4.z * iz.x, local ? -g4.z * dy : g4.z * iz.y};
          const cx<double> *a = co + i * P;
          cx<double> acc = a[P - 1], dv{0.0, 0.0};
          const double sh1 = local ? 0.0 : 1.0;
          if constexpr (MODE == kLeafDeriv) dv = (P - 1 + sh1) * acc;
#pragma unroll
          for (int k = P - 2; k >= 0; --k) {
            const cx<double> c = a[k];
            if constexpr (MODE == kLeafDeriv) {  // (no l = 0 term when local)
              const cx<double> n = cfma(dv, w, (k + sh1) * c);
              dv = k > 0 || !local ? n : dv;
            }
            acc = cfma(acc, w, c);
          }
          const cx<double> t = local ? acc : acc * w;
          if constexpr (MODE == kLeafField) {
            far[r] += t.x;
          } else {
            far[0] += t.x;
            far[1] += t.y;
          }
          if constexpr (MODE == kLeafDeriv) {  // d w / d z = 1 / rad or -rho / d
            const cx<double> d = local ? cx<double>{g4.z * dv.x, g4.z * dv.y} : (dv * w) * iz;
            far[2] -= d.x;
            far[3] -= d.y;
          }
        }
        __syncthreads();
      }
    }
    auto stage = [&](int q0, int take, int tpad) {
      for (int q = tid; q < tpad; q += nth) {
        const bool in = q < take;
        const int64_t j = in ? uf_idx[uf0 + q0 + q] : 0;
        sz[q] = in ? make_double2(sx[j], sy[j]) : make_double2(0.0, 0.0);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          cx<double> pj{0.0, 0.0};
          if (in && r < nr) pj = p[(int64_t)(r0 + r) * ns + j];
          sp[q * RB + r] = make_double2(pj.x, pj.y);
        }
      }
    };
    // value c of every lane's targets through LDS: red[slice][target], the
    // far parts behind them; lane t < nt adds its target's parts.  Of the
    // complex fields more than kLeafSlices parts are added over the lanes of
    // their wave first: one lane's chain over them, up to 256 for a leaf of
    // one target and four waves, for each of two or four values, took longer
    // than the sums (198 leaves of 4 targets 19.7 us, now 8.4; one value's
    // chain, in kLeafField, is shorter than the shuffles)
    double tot[NF];
#pragma unroll
    for (int c = 0; c < NF; ++c) tot[c] = 0.0;
    auto fin = [&](int c, int sl, int tl, int tp, int S, const auto &v, auto kk) {
      constexpr int K = decltype(kk)::value;
      constexpr bool fold = MODE != kLeafField;
      const int row = tp * K, lane = tid & 63, wv = tid >> 6;
      const bool near = fold && S > kLeafSlices, far_ = fold && Sf > kLeafSlices;  // block-uniform
      const int ns = near ? W : S, nf = far_ ? W : Sf;
      double *fr = sh + ns * row, ff = far[c];
      if (far_)
        for (int o = 1 << lgf; o < 64; o <<= 1) ff += __shfl_xor(ff, o, 64);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        double x = v[k];
        if (near)
          for (int o = tp; o < 64; o <<= 1) x += __shfl_xor(x, o, 64);
        if (!near || lane < tp) sh[(near ? wv : sl) * row + k * tp + tl] = x;
      }
      if (!far_ || lane < 1 << lgf) fr[far_ ? (wv << lgf) + lane : tid] = ff;
      __syncthreads();
      if (tid < nt) {
        double s = 0.0;
        for (int q = 0; q < nf; ++q) s += fr[(q << lgf) + tid];
        for (int q = 0; q < ns; ++q) s += sh[q * row + tid];
        tot[c] = s;
      }
      __syncthreads();
    };
    // 16 lanes a slice above 32 targets, else 8 (fewer for fewer targets)
    const int lg = nt > 32 ? 4 : nt >= 8 ? 3 : __builtin_ctz(pow2_at_least(nt));
    switch ((nt + (1 << lg) - 1) >> lg) {  // block-uniform
      case 1: near_field64<MODE, RB, 1>(nt, lg, utot, stage_n, txc, tyc, sz, sp, stage, fin); break;
      case 2: near_field64<MODE, RB, 2>(nt, lg, utot, stage_n, txc, tyc, sz, sp, stage, fin); break;
      case 3: near_field64<MODE, RB, 3>(nt, lg, utot, stage_n, txc, tyc, sz, sp, stage, fin); break;
      default: near_field64<MODE, RB, 4>(nt, lg, utot, stage_n, txc, tyc, sz, sp, stage, fin); break;
    }
    if (tid < nt) {
      const int64_t api = tperm[tb0 + tc0 + tid];
      if constexpr (MODE == kLeafField) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          if (r < nr) {
            double val = scale * tot[r];
            if (as.sigma) {
              const double sg = as.sigma[(int64_t)(r0 + r) * as.ldx + api];
              val += (as.ident + as.tau[api]) * sg +
                     as.gamma[(r0 + r) * as.G + (as.geo ? as.geo[api] : 0)];
            }
            out[(int64_t)(r0 + r) * ldy + api] = val;
          }
        }
      } else {
        out[2 * api] = tot[0];
        out[2 * api + 1] = tot[1];
        if constexpr (MODE == kLeafDeriv) {
          dout[2 * api] = tot[2];
          dout[2 * api + 1] = tot[3];
        }
      }
    }
  }
}

// Waves per leaf of the FP64 leaf kernel: one where the leaves alone fill
// the chip (each wave then pays the staging and the joining once), two or
// four below, where a leaf's own chain of loads and sums is the time.
// Field of one right-hand side, one / two / four waves: 161 / 181 / - us at
// 31920 leaves, 62 / 58 / - at 11164, 43 / 28 / 33 at 3351, 31 / 20 / 18 at
// 822; the complex fields, with more work per pair, gain from a second wave
// only below 8192 leaves (transposed application 216 / 229 us at 11164).
// Where no leaf has more sources (max_u) than one wave stages at a time and
// there is a leaf per SIMD, more waves share only the staging: 1000 caps of 64
// nodes, application of one / two waves 47.9 / 50.6 us, transposed 26.0 / 30.2.
static int leaf64_waves(int64_t groups, bool field, int max_u) {
  if (groups >= 1024 && max_u <= kStage) return 1;
  return groups >= (field ? 16384 : 8192) ? 1 : groups >= 2048 ? 2 : 4;
}

// Launch of k_leaf64 over the plan's target leaves.
template <int P, int MODE, int RB>
static void launch_leaf64(const DevPlan &pl, const int64_t *ufp, const int32_t *uf_idx,
                          const double *sx, const double *sy, const cx<double> *p, int64_t ns,
                          const cx<double> *M, const cx<double> *L, int nrhs, double *out,
                          double *dout, int64_t ldy, double scale, const Assembly &as,
                          hipStream_t s) {
  if (pl.n_leaf_t == 0) return;
  const int ry = (nrhs + RB - 1) / RB;
  const int64_t groups = (int64_t)pl.n_leaf_t * ry;
  const int W = leaf64_waves(groups, MODE == kLeafField, ufp ? INT32_MAX : pl.max_u);
  const size_t stage = (size_t)kStage * std::min(W, 2) * (1 + RB) * sizeof(double2);
  const size_t red = (size_t)(256 + 64) * W * sizeof(double);
  const size_t fari = kFarItems * (sizeof(double4) + P * sizeof(cx<double>));
  hipLaunchKernelGGL((k_leaf64<P, MODE, RB>), dim3(pl.n_leaf_t, ry), dim3(64 * W),
                     std::max(std::max(stage, red), fari), s, pl.lt_hdr.p, pl.cx.p, pl.cy.p, pl.rad.p, pl.tx.p,
                     pl.ty.p, pl.tgt_perm.p, ufp, uf_idx, pl.w_src.p, sx, sy, p, ns, M, L,
                     pl.nbox, nrhs, out, dout, ldy, scale, as);
}

// A staged U-list source of the FP32 leaf kernel: position (FP64) and the
// FP32 strengths of RB right-hand sides, 16-byte aligned so that one
// address serves both reads.
template <int RB>
struct alignas(16) Src32 {
  double2 z;
  float2 p[RB];
};

// Direct sums of one target lane over the staged sources zq[0], zq[S],
// ..., zq[(niter - 1) S] (S compile-time, so the unrolled reads take
// immediate offsets): f[q] += Re(p_q conj(d)) / |d|^2, d = z_t - z_j formed
// in FP64 and rounded once.  |d|^2 + 1e-30: a target's own source (d = 0)
// contributes 0 * rcp(1e-30) = 0; the bias leaves any |d|^2 above 2e-23
// (node spacings above 5e-12) unchanged in FP32.
template <int S, int RB>
__device__ __forceinline__ void near_sums32(const Src32<RB> *__restrict__ zq,
                                            int niter, double ax, double ay,
                                            float (&f)[RB]) {
  if constexpr (RB == 1) {
#pragma unroll 4
    for (int it = 0; it < niter; ++it) {
      const Src32<1> &e = zq[it * S];
      const float dx = (float)(ax - e.z.x);
      const float dy = (float)(ay - e.z.y);
      const float d2 = fmaf(dx, dx, fmaf(dy, dy, 1e-30f));
      f[0] += fmaf(e.p[0].x, dx, e.p[0].y * dy) * __builtin_amdgcn_rcpf(d2);
    }
  } else {
#pragma unroll 2
    for (int it = 0; it < niter; ++it) {
      const Src32<RB> &e = zq[it * S];
      const float dx = (float)(ax - e.z.x);
      const float dy = (float)(ay - e.z.y);
      const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, fmaf(dy, dy, 1e-30f)));
      const float ux = dx * inv, uy = dy * inv;
#pragma unroll
      for (int q = 0; q < RB; ++q) f[q] = fmaf(e.p[q].x, ux, fmaf(e.p[q].y, uy, f[q]));
    }
  }
}

// FP32 variant: each pair's difference d = z_i - z_j is formed in FP64
// and rounded once to FP32 (one FP64 add and one conversion per
// coordinate, at the FP32 rate on this chip), the rest in FP32.  A block
// handles
// RB right-hand sides (blockIdx.y * RB + 0 .. RB - 1, those < nrhs): each
// pair's difference and reciprocal are formed once and applied to every
// right-hand side of the block.
template <int P, int RB>
__global__ void __launch_bounds__(64, RB == 1 ? 8 : 1)
    k_leaf32(const LeafHdr *__restrict__ hdr,
             const double *__restrict__ cxv, const double *__restrict__ cyv,
             const double *__restrict__ rad,
             const double *__restrict__ tx, const double *__restrict__ ty,
             const int64_t *__restrict__ tperm,
             const int32_t *__restrict__ uf_idx,
             const int32_t *__restrict__ w_src,
             const double *__restrict__ sx, const double *__restrict__ sy,
             const cx<float> *__restrict__ p, int64_t ns,
             const cx<float> *__restrict__ M, const cx<float> *__restrict__ L,
             int nbox, int nrhs, double *__restrict__ out, int64_t ldy,
             double scale, Assembly as) {
  __shared__ Src32<RB> sz[kStage];
  constexpr int NC = 2;  // sub-chunks of <= 32 targets per pass over U
  const LeafHdr &hd = hdr[blockIdx.x];
  const int b = hd.b;
  const int r0 = blockIdx.y * RB, nr = min(RB, nrhs - r0);
  const int lane = threadIdx.x;
  const int64_t tb0 = hd.t0, ntb = hd.nt;
  const int64_t uf0 = hd.uf0;
  const int utot = (int)(hd.uf1 - uf0);  // U-list sources of the leaf
  const int wb = hd.wb, we = hd.we;
  const bool has_local = hd.lev >= 2;
  const double ir_b = hd.ir, cx_b = hd.cx, cy_b = hd.cy;
  for (int64_t tc0 = 0; tc0 < ntb; tc0 += 32 * NC) {
    const int nt = (int)min<int64_t>(32 * NC, ntb - tc0);
    const int nch = (nt + 31) / 32;
    // sub-chunk c: targets [32 c, min(32 c + 32, nt)) on tp_c lanes times
    // S_c = 64 / tp_c source slices, tp_c = min(32, next power of two)
    int S[NC], sl[NC], ti[NC];
    bool act[NC];
    float fld[NC][RB];
    double zxd[NC], zyd[NC];
    int Smax = 1;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      S[c] = 64;
      sl[c] = 0;
      act[c] = false;
      ti[c] = 0;
      zxd[c] = zyd[c] = 0.0;
#pragma unroll
      for (int q = 0; q < RB; ++q) fld[c][q] = 0.f;
      if (c >= nch) continue;  // uniform
      const int rem = nt - 32 * c;
      const int tp = rem >= 32 ? 32 : pow2_at_least(rem);
      const int lg = __builtin_ctz(tp);  // tp is a power of two
      S[c] = 64 >> lg;
      Smax = max(Smax, S[c]);
      const int tl = lane & (tp - 1);
      sl[c] = lane >> lg;
      act[c] = 32 * c + tl < nt;
      ti[c] = (int)tc0 + 32 * c + tl;
      if (!act[c]) continue;
      const int64_t i = tb0 + ti[c];
      zxd[c] = tx[i];
      zyd[c] = ty[i];
    }
    {  // the leaf's U-list sources, kStage at a time
      const int total = utot;
      for (int q0 = 0; q0 < total; q0 += kStage) {
        const int take = min(kStage, total - q0);
        // pad to a multiple of Smax (<= 64, divides kStage) with sources of
        // zero strength at the origin: they add 0 * rcp(|z|^2 + 1e-30) = 0
        const int tpad = (take + Smax - 1) & ~(Smax - 1);  // Smax: power of two
        for (int q = lane; q < tpad; q += 64) {
          if (q < take) {
            const int64_t j = uf_idx[uf0 + q0 + q];
            sz[q].z = make_double2(sx[j], sy[j]);
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) {
              const cx<float> pj = rr < nr ? p[(int64_t)(r0 + rr) * ns + j]
                                           : cx<float>{0.f, 0.f};
              sz[q].p[rr] = make_float2(pj.x, pj.y);
            }
          } else {
            sz[q].z = make_double2(0.0, 0.0);
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) sz[q].p[rr] = make_float2(0.f, 0.f);
          }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (c >= nch) continue;  // uniform
          const int Sc = S[c], niter = tpad >> __builtin_ctz(Sc);
          const double ax = zxd[c], ay = zyd[c];
          float f[RB];
#pragma unroll
          for (int q = 0; q < RB; ++q) f[q] = fld[c][q];
          const Src32<RB> *zq = sz + sl[c];
          switch (Sc) {  // wave-uniform
            case 2: near_sums32<2, RB>(zq, niter, ax, ay, f); break;
            case 4: near_sums32<4, RB>(zq, niter, ax, ay, f); break;
            case 8: near_sums32<8, RB>(zq, niter, ax, ay, f); break;
            case 16: near_sums32<16, RB>(zq, niter, ax, ay, f); break;
            case 32: near_sums32<32, RB>(zq, niter, ax, ay, f); break;
            default: near_sums32<64, RB>(zq, niter, ax, ay, f); break;
          }
#pragma unroll
          for (int q = 0; q < RB; ++q) fld[c][q] = f[q];
        }
        __syncthreads();
      }
    }
    // per right-hand side: L2P (slice 0) and this slice's share of M2P,
    // the sum over slices, the assembled row; the accumulators of the
    // next right-hand side rotate into fld[c][0] (constant register indices)
#pragma unroll 1
    for (int q = 0; q < nr; ++q) {
      const int r = r0 + q;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (c >= nch) continue;  // uniform
        float field = fld[c][0];
        if (act[c]) {
          const double zx = zxd[c], zy = zyd[c];
          if (sl[c] == 0 && has_local) {
            const cx<float> w{float((zx - cx_b) * ir_b), float((zy - cy_b) * ir_b)};
            const cx<float> *La = L + ((int64_t)r * nbox + b) * P;
            cx<float> acc = La[P - 1];
            for (int l = P - 2; l >= 0; --l) acc = cfma(acc, w, La[l]);
            field += acc.x;
          }
          for (int e = wb + sl[c]; e < we; e += S[c]) {
            const int cw = w_src[e];
            const double dx = zx - cxv[cw], dy = zy - cyv[cw];
            const double id = rad[cw] / (dx * dx + dy * dy);
            const cx<float> rho{float(dx * id), float(-dy * id)};
            const cx<float> *a = M + ((int64_t)r * nbox + cw) * P;
            cx<float> acc = a[P - 1];
            for (int k = P - 2; k >= 0; --k) acc = cfma(acc, rho, a[k]);
            field += (acc * rho).x;
          }
        }
        for (int o = 64 >> __builtin_ctz(S[c]); o < 64; o <<= 1) field += __shfl_xor(field, o, 64);
        if (act[c] && sl[c] == 0) {
          const int64_t api = tperm[tb0 + ti[c]];
          double val = scale * (double)field;
          if (as.sigma) {
            const double sg = as.sigma[(int64_t)r * as.ldx + api];
            val += (as.ident + as.tau[api]) * sg +
                   as.gamma[r * as.G + (as.geo ? as.geo[api] : 0)];
          }
          out[(int64_t)r * ldy + api] = val;
        }
#pragma unroll
        for (int k = 0; k + 1 < RB; ++k) fld[c][k] = fld[c][k + 1];
      }
    }
  }
}

// Set-up of the FP32 leaf multipoles' inputs: w32[j] = (z_j - c) / r of
// source j's leaf, rounded once to FP32 as the multipole pass forms it, and
// perm32[j] = src_perm[j]; one wave per source leaf.
__global__ void __launch_bounds__(64)
    k_p2m_inputs32(int nleaf, const int64_t *__restrict__ ls_rng,
                   const double4 *__restrict__ ls_geo, const double *__restrict__ sx,
                   const double *__restrict__ sy, const int64_t *__restrict__ perm,
                   float2 *__restrict__ w32, int32_t *__restrict__ perm32) {
  const int e = blockIdx.x;
  if (e >= nleaf) return;
  const double4 geo = ls_geo[e];
  const int64_t e0 = ls_rng[2 * e], e1 = ls_rng[2 * e + 1];
  for (int64_t j = e0 + threadIdx.x; j < e1; j += 64) {
    w32[j] = make_float2(float((sx[j] - geo.x) * geo.z), float((sy[j] - geo.y) * geo.z));
    perm32[j] = (int32_t)perm[j];
  }
}

void build_p2m_inputs32(DevPlan &pl, hipStream_t s) {
  if (pl.ns > INT32_MAX)
    throw ApiError{LBS_ERR_UNSUPPORTED, "more than 2^31 - 1 sources in one plan"};
  pl.w32.alloc((size_t)pl.ns);
  pl.perm32.alloc((size_t)pl.ns);
  if (pl.n_leaf_s > 0)
    hipLaunchKernelGGL(k_p2m_inputs32, dim3(pl.n_leaf_s), dim3(64), 0, s, pl.n_leaf_s,
                       pl.ls_rng.p, pl.ls_geo.p, pl.sx.p, pl.sy.p, pl.src_perm.p, pl.w32.p,
                       pl.perm32.p);
  LBS_HIP(hipGetLastError());
}

// qm32[j] = (Im q_j, -Re q_j) in FP32 (so that -i q_j sigma = qm32 sigma),
// q = qfac_t interleaved complex
__global__ void k_qm32(int64_t n, const double *__restrict__ qfac_t, float2 *__restrict__ qm32) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < n) qm32[j] = make_float2(float(qfac_t[2 * j + 1]), float(-qfac_t[2 * j]));
}

void launch_qm32(int64_t n, const double *qfac_t, float2 *qm32, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_qm32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, qfac_t,
                     qm32);
  LBS_HIP(hipGetLastError());
}

// ---------------------------------------------------------------- drivers
static XBoxes x_boxes(const DevPlan &pl) {
  return XBoxes{(int)pl.x_box.n, pl.x_box.p, pl.xf_ptr.p, pl.xf_idx.p, pl.cx.p, pl.cy.p,
                pl.rad.p, pl.sx.p, pl.sy.p, pl.ns};
}

// Returns whether the correction sums of gf were formed too (by the FP32
// MFMA M2L launch).
template <typename T, int P>
static bool far_field(const DevPlan &pl, const Tables &tb, Workspace &ws,
                      cx<T> *p, cx<T> *M, cx<T> *L, int nrhs,
                      hipStream_t s, StrengthSrc ss = StrengthSrc{},
                      const GammaFused *gf = nullptr) {
  bool gamma_done = false, p2l_done = false;
  StageTimer *tm = ws.timer;
  const cx<T> *pre, *post;
  const T *H, *bc;
  if constexpr (sizeof(T) == 8) {
    H = (const T *)tb.h64.p;
    bc = (const T *)tb.bc64.p;
    pre = (const cx<T> *)tb.pre64.p;
    post = (const cx<T> *)tb.post64.p;
  } else {
    H = (const T *)tb.h32.p;
    bc = (const T *)tb.bc32.p;
    pre = (const cx<T> *)tb.pre32.p;
    post = (const cx<T> *)tb.post32.p;
  }
  {
    TimerScope ts(tm, ST_UPWARD, s);
    if (pl.n_leaf_s > 0)
    {
      if constexpr (sizeof(T) == 4 && P <= 16)  // two leaves per wave
        hipLaunchKernelGGL((k_p2m_pair<P>), dim3((pl.n_leaf_s + 1) / 2, nrhs), dim3(64), 0, s,
                           pl.leaf_s.p, pl.n_leaf_s, pl.ls_rng.p, pl.ls_geo.p, pl.sx.p,
                           pl.sy.p, pl.w32.n ? pl.w32.p : nullptr, p, pl.ns, M, pl.nbox, ss);
      else if constexpr (sizeof(T) == 8)  // two leaves per wave
        hipLaunchKernelGGL((k_p2m_pair64<P>), dim3((pl.n_leaf_s + 1) / 2, nrhs), dim3(64), 0,
                           s, pl.leaf_s.p, pl.n_leaf_s, pl.ls_rng.p, pl.ls_geo.p, pl.sx.p,
                           pl.sy.p, (cx<double> *)p, pl.ns, (cx<double> *)M, pl.nbox, ss);
      else
        hipLaunchKernelGGL((k_p2m<T, P>), dim3(pl.n_leaf_s, nrhs), dim3(64), 0,
                           s, pl.leaf_s.p, pl.ls_rng.p, pl.ls_geo.p, pl.sx.p,
                           pl.sy.p, p, pl.ns, M, pl.nbox, ss);
    }
    if constexpr (sizeof(T) == 8)
      p2l_done = run_pass<T, P, false>(pl.up[1], bc, pre, post, M, pl.nbox, nrhs, s, x_boxes(pl),
                                       p, L);
    else
      run_pass<T, P, false>(pl.up[0], bc, pre, post, M, pl.nbox, nrhs, s);
  }
  // the FP32 MFMA M2L also forms the P2L sums of its boxes: every box with
  // an X list whose local expansion is used (level >= 2, with targets) is
  // one of its boxes
  constexpr bool p2l_in_m2l = sizeof(T) == 4 && P == 16;
  if (pl.n_m2l > 0) {
    TimerScope ts(tm, ST_M2L, s);
    GammaGroups gg;  // the correction sums ride along
    if (gf && pl.n_leaf_s > 0)
      gg = GammaGroups{gf->gl_ptr, ws.gpart.p, ws.gcsum.p, ws.gcnt.p, gf->gamma,
                       pl.n_leaf_s, gf->G, gf->nchunk, 0};
    if constexpr (p2l_in_m2l) {
      const XListSrc xs{pl.xf_ptr.p, pl.xf_idx.p, pl.cx.p, pl.cy.p, pl.rad.p,
                        pl.sx.p, pl.sy.p, (const cx<float> *)p, pl.ns};
      gg.first = std::min((pl.n_m2l + 3) / 4, pl.m2l_groups);
      const int groups = gg.first + gg.nchunk * gg.G;
      gamma_done = gg.nchunk > 0;
      hipLaunchKernelGGL(k_m2l_mfma16, dim3(groups, nrhs), dim3(256), 0, s,
                         pl.n_m2l, pl.m2l_wave.p, pl.v_ptr.p, pl.v_src.p,
                         pl.v_code.p, H, (const cx<T> *)tb.itp32.p, (const cx<T> *)M, L,
                         pl.nbox, xs, gg);
    } else if constexpr (sizeof(T) == 8) {
      gamma_done = gg.nchunk > 0;
      if (pl.x_box.n > 0 && !p2l_done)  // more boxes than the pass takes, or no pass
        hipLaunchKernelGGL((k_p2l64<P>), dim3((unsigned)(pl.x_box.n + 1) / 2, nrhs), dim3(64), 0,
                           s, x_boxes(pl), p, L, pl.nbox);
      launch_m2l64<P>(pl, H, M, L, true, nrhs, gg, s);
    } else {
      hipLaunchKernelGGL((k_m2l<T, P>), dim3(pl.n_m2l, nrhs), dim3(64), 0, s,
                         pl.m2l_box.p, pl.v_ptr.p, pl.v_src.p, pl.v_code.p, H,
                         (const cx<T> *)tb.itp32.p, (const cx<T> *)M, L, pl.nbox, pl.xf_ptr.p,
                         pl.xf_idx.p,
                         pl.cx.p, pl.cy.p, pl.rad.p, pl.sx.p, pl.sy.p, (const cx<T> *)p,
                         pl.ns);
    }
  }
  TimerScope ts(tm, ST_L2L, s);
  run_pass<T, P, true>(pl.dn[sizeof(T) == 8], bc, pre, post, L, pl.nbox, nrhs, s);
  return gamma_done;
}

template <int P>
static void run64(const DevPlan &pl, const Tables &tb, Workspace &ws,
                  int nrhs, double *out, int64_t ldy, double scale,
                  const Assembly &as, hipStream_t s, const StrengthSrc &ss,
                  const GammaFused *gf) {
  auto *p = (cx<double> *)ws.pstr64.p;
  auto *M = (cx<double> *)ws.mult64.p;
  auto *L = (cx<double> *)ws.loc64.p;
  const bool gamma_done = far_field<double, P>(pl, tb, ws, p, M, L, nrhs, s, ss, gf);
  if (gf && pl.n_leaf_s > 0 && !gamma_done) {
    TimerScope ts(ws.timer, ST_GAMMA, s);
    hipLaunchKernelGGL(k_gamma_reduce, dim3(gf->nchunk, gf->G, nrhs), dim3(256), 0,
                       s, gf->gl_ptr, ws.gpart.p, pl.n_leaf_s, gf->G, ws.gcsum.p,
                       ws.gcnt.p, gf->gamma);
  }
  if (pl.n_leaf_t > 0) {
    TimerScope ts(ws.timer, ST_LEAF, s);
    // four right-hand sides per work-group share each pair's difference and
    // reciprocal (four columns at 1.02M nodes 417 us against 682 with a
    // group each, 178 against 206 at 256k) where that leaves enough groups;
    // below 8192 the groups are too few (3351: 96 us, and 70 with one each)
    const bool four = nrhs > 1 && (int64_t)pl.n_leaf_t * ((nrhs + 3) / 4) >= 8192;
    const auto launch = four ? launch_leaf64<P, kLeafField, 4> : launch_leaf64<P, kLeafField, 1>;
    launch(pl, nullptr, pl.uf_idx.p, pl.sx.p, pl.sy.p, p, pl.ns, M, L, nrhs, out, nullptr, ldy,
           scale, as, s);
  }
}

template <int P>
static void run32(const DevPlan &pl, const Tables &tb, Workspace &ws,
                  int nrhs, double *out, int64_t ldy, double scale,
                  const Assembly &as, hipStream_t s, const StrengthSrc &ss,
                  const GammaFused *gf) {
  auto *p = (cx<float> *)ws.pstr32.p;
  auto *M = (cx<float> *)ws.mult32.p;
  auto *L = (cx<float> *)ws.loc32.p;
  const bool gamma_done = far_field<float, P>(pl, tb, ws, p, M, L, nrhs, s, ss, gf);
  if (gf && pl.n_leaf_s > 0 && !gamma_done) {
    TimerScope ts(ws.timer, ST_GAMMA, s);
    hipLaunchKernelGGL(k_gamma_reduce, dim3(gf->nchunk, gf->G, nrhs), dim3(256), 0,
                       s, gf->gl_ptr, ws.gpart.p, pl.n_leaf_s, gf->G, ws.gcsum.p,
                       ws.gcnt.p, gf->gamma);
  }
  if (pl.n_leaf_t > 0) {
    TimerScope ts(ws.timer, ST_LEAF, s);
    auto launch = [&](auto kern, int rb) {
      hipLaunchKernelGGL(kern, dim3(pl.n_leaf_t, (nrhs + rb - 1) / rb), dim3(64),
                         0, s, pl.lt_hdr.p, pl.cx.p, pl.cy.p, pl.rad.p, pl.tx.p,
                         pl.ty.p,
                         pl.tgt_perm.p,
                         pl.uf_idx.p, pl.w_src.p,
                         pl.sx.p, pl.sy.p,
                         (const cx<float> *)p, pl.ns, (const cx<float> *)M,
                         (const cx<float> *)L, pl.nbox, nrhs, out, ldy, scale,
                         as);
    };
    // one right-hand side per block, or blocks of 4 sharing each pair
    if (nrhs == 1) launch(k_leaf32<P, 1>, 1);
    else launch(k_leaf32<P, 4>, 4);
  }
}

void fmm_apply64(const DevPlan &pl, const Tables &tb, Workspace &ws,
                 const double *qfac_t, const double *sigma, int64_t ldx,
                 int nrhs, double *out, int64_t ldy, double scale,
                 const Assembly &as, hipStream_t s, const GammaFused *gf) {
  // the strengths p_j = -i q_j sigma_j (and with gf the partial gamma
  // sums) are formed by the leaf multipole pass
  const StrengthSrc ss{pl.src_perm.p, qfac_t, sigma, ldx, gf ? gf->gw_t : nullptr,
                       gf ? ws.gpart.p : nullptr};
  switch (tb.P) {
    case 20: run64<20>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 24: run64<24>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 30: run64<30>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 36: run64<36>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 40: run64<40>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 48: run64<48>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    default:
      throw ApiError{LBS_ERR_UNSUPPORTED,
                     "p64 must be one of 20, 24, 30, 36, 40, 48"};
  }
  LBS_HIP(hipGetLastError());
}

void fmm_far64(const DevPlan &pl, const Tables &tb, Workspace &ws, const double *qfac_t,
               const double *sigma, int64_t ldx, int nrhs, hipStream_t s) {
  const StrengthSrc ss{pl.src_perm.p, qfac_t, sigma, ldx, nullptr, nullptr};
  auto *p = (cx<double> *)ws.pstr64.p;
  auto *M = (cx<double> *)ws.mult64.p;
  auto *L = (cx<double> *)ws.loc64.p;
  switch (tb.P) {
    case 20: far_field<double, 20>(pl, tb, ws, p, M, L, nrhs, s, ss); break;
    case 24: far_field<double, 24>(pl, tb, ws, p, M, L, nrhs, s, ss); break;
    case 30: far_field<double, 30>(pl, tb, ws, p, M, L, nrhs, s, ss); break;
    case 36: far_field<double, 36>(pl, tb, ws, p, M, L, nrhs, s, ss); break;
    case 40: far_field<double, 40>(pl, tb, ws, p, M, L, nrhs, s, ss); break;
    case 48: far_field<double, 48>(pl, tb, ws, p, M, L, nrhs, s, ss); break;
    default:
      throw ApiError{LBS_ERR_UNSUPPORTED,
                     "p64 must be one of 20, 24, 30, 36, 40, 48"};
  }
  LBS_HIP(hipGetLastError());
}

void fmm_apply32(const DevPlan &pl, const Tables &tb, Workspace &ws,
                 const double *qfac_t, const float2 *qm32, const double *sigma, int64_t ldx,
                 int nrhs, double *out, int64_t ldy, double scale,
                 const Assembly &as, hipStream_t s, const GammaFused *gf) {
  // the strengths p_j = -i q_j sigma_j (and with gf the partial gamma
  // sums) are formed by the leaf multipole pass
  const StrengthSrc ss{pl.src_perm.p, qfac_t, sigma, ldx, gf ? gf->gw_t : nullptr,
                       gf ? ws.gpart.p : nullptr,
                       qm32 && pl.perm32.n ? qm32 : nullptr,
                       qm32 && pl.perm32.n ? pl.perm32.p : nullptr};
  switch (tb.P) {
    case 12: run32<12>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 16: run32<16>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 20: run32<20>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    case 24: run32<24>(pl, tb, ws, nrhs, out, ldy, scale, as, s, ss, gf); break;
    default:
      throw ApiError{LBS_ERR_UNSUPPORTED, "p32 must be one of 12, 16, 20, 24"};
  }
  LBS_HIP(hipGetLastError());
}


// ------------------------------------------------- full complex output
// Psi(z) = sum_j p_j / (z - z_j) and Psi'(z) at the targets, complex, FP64,
// for given complex strengths (API order of the plan's sources).  Used by
// the transposed operator and the shape derivatives.
__global__ void k_strengths_given(int64_t ns, const int64_t *__restrict__ perm,
                                  const double *__restrict__ pin,
                                  cx<double> *__restrict__ p) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= ns) return;
  const int64_t a = perm[j];
  p[j] = cx<double>{pin[2 * a], pin[2 * a + 1]};
}

template <int P>
static void run64_full(const DevPlan &pl, const Tables &tb, Workspace &ws,
                       double *psi, double *dpsi, hipStream_t s) {
  auto *p = (cx<double> *)ws.pstr64.p;
  auto *M = (cx<double> *)ws.mult64.p;
  auto *L = (cx<double> *)ws.loc64.p;
  far_field<double, P>(pl, tb, ws, p, M, L, 1, s);
  const auto launch = dpsi ? launch_leaf64<P, kLeafDeriv, 1> : launch_leaf64<P, kLeafPsi, 1>;
  launch(pl, nullptr, pl.uf_idx.p, pl.sx.p, pl.sy.p, p, pl.ns, M, L, 1, psi, dpsi, 0, 1.0,
         Assembly{}, s);
}

void fmm_apply64_full(const DevPlan &pl, const Tables &tb, Workspace &ws,
                      const double *pin, double *psi, double *dpsi,
                      hipStream_t s) {
  if (pl.ns > 0)
    hipLaunchKernelGGL(k_strengths_given, dim3((unsigned)((pl.ns + 255) / 256)),
                       dim3(256), 0, s, pl.ns, pl.src_perm.p, pin,
                       (cx<double> *)ws.pstr64.p);
  switch (tb.P) {
    case 20: run64_full<20>(pl, tb, ws, psi, dpsi, s); break;
    case 24: run64_full<24>(pl, tb, ws, psi, dpsi, s); break;
    case 30: run64_full<30>(pl, tb, ws, psi, dpsi, s); break;
    case 36: run64_full<36>(pl, tb, ws, psi, dpsi, s); break;
    case 40: run64_full<40>(pl, tb, ws, psi, dpsi, s); break;
    case 48: run64_full<48>(pl, tb, ws, psi, dpsi, s); break;
    default:
      throw ApiError{LBS_ERR_UNSUPPORTED,
                     "p64 must be one of 20, 24, 30, 36, 40, 48"};
  }
  LBS_HIP(hipGetLastError());
}

// M[list[e]] = the sum of the partial multipoles of entry e's chunks
// [ptr[e], ptr[e + 1]), in chunk order; one thread per (entry, coefficient).
template <int P>
__global__ void __launch_bounds__(256)
    k_sum_chunks(int n, const int32_t *__restrict__ list, const uint32_t *__restrict__ ptr,
                 const cx<double> *__restrict__ part, cx<double> *__restrict__ M) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)n * P) return;
  const int e = (int)(id / P), k = (int)(id % P);
  cx<double> a{0.0, 0.0};
  for (uint32_t c = ptr[e]; c < ptr[e + 1]; ++c) a = a + part[(int64_t)c * P + k];
  M[(int64_t)list[e] * P + k] = a;
}

template <int P>
static void run64_sources(const DevPlan &pl, const Tables &tb, Workspace &ws,
                          PointSources &ps, const cx<double> *pin, double *psi, double *dpsi,
                          hipStream_t s) {
  auto *M = (cx<double> *)ws.mult64.p;
  auto *L = (cx<double> *)ws.loc64.p;
  const auto *H = (const double *)tb.h64.p;
  // multipoles of every box of level >= 2 from the points it holds: the
  // partial multipoles of chunks of at most kSrcChunk pairs, added per box
  // (boxes without points get zeros)
  launch_gather_cx(ps.nm, ps.m_t.p, (const double *)pin, ps.m_p.p, s);
  auto *part = (cx<double> *)ps.c_part.p;
  if (ps.n_c > 0)
    hipLaunchKernelGGL((k_p2m<double, P>), dim3(ps.n_c, 1), dim3(64), 0, s, ps.c_iota.p,
                       ps.c_rng.p, ps.c_geo.p, ps.m_x.p, ps.m_y.p, (cx<double> *)ps.m_p.p,
                       ps.nm, part, ps.n_c, StrengthSrc{});
  if (ps.n_m > 0)
    hipLaunchKernelGGL((k_sum_chunks<P>), dim3((unsigned)(((int64_t)ps.n_m * P + 255) / 256)),
                       dim3(256), 0, s, ps.n_m, ps.m_list.p, ps.c_ptr.p, part, M);
  // the tree's V lists, then the points' own local-expansion terms
  if (pl.n_m2l > 0) launch_m2l64<P>(pl, H, M, L, false, 1, GammaGroups{}, s);
  if (ps.n_m > 0)
    hipLaunchKernelGGL((k_p2l<double, P>), dim3(ps.n_m, 1), dim3(64), 0, s, ps.m_list.p,
                       ps.l_ptr.p, ps.l_t.p, pl.cx.p, pl.cy.p, pl.rad.p, ps.x, ps.y, pin, ps.n,
                       L, pl.nbox);
  run_pass<double, P, true>(pl.dn[1], (const double *)tb.bc64.p, (const cx<double> *)tb.pre64.p,
                            (const cx<double> *)tb.post64.p, L, pl.nbox, 1, s);
  // at the plan's targets: local expansions, W lists, direct sums
  const auto launch = dpsi ? launch_leaf64<P, kLeafDeriv, 1> : launch_leaf64<P, kLeafPsi, 1>;
  launch(pl, ps.d_ptr.p, ps.d_t.p, ps.x, ps.y, pin, ps.n, M, L, 1, psi, dpsi, 0, 1.0,
         Assembly{}, s);
}

void fmm_sources64_full(const DevPlan &pl, const Tables &tb, Workspace &ws, PointSources &ps,
                        const double *pin, double *psi, double *dpsi, hipStream_t s) {
  const auto *pc = (const cx<double> *)pin;
  switch (tb.P) {
    case 20: run64_sources<20>(pl, tb, ws, ps, pc, psi, dpsi, s); break;
    case 24: run64_sources<24>(pl, tb, ws, ps, pc, psi, dpsi, s); break;
    case 30: run64_sources<30>(pl, tb, ws, ps, pc, psi, dpsi, s); break;
    case 36: run64_sources<36>(pl, tb, ws, ps, pc, psi, dpsi, s); break;
    case 40: run64_sources<40>(pl, tb, ws, ps, pc, psi, dpsi, s); break;
    case 48: run64_sources<48>(pl, tb, ws, ps, pc, psi, dpsi, s); break;
    default:
      throw ApiError{LBS_ERR_UNSUPPORTED,
                     "p64 must be one of 20, 24, 30, 36, 40, 48"};
  }
  LBS_HIP(hipGetLastError());
}

// FP32 counterpart for the transposed operator (field only): strengths in
// FP32, near-field differences formed in FP64 as in k_leaf32.
__global__ void k_strengths_given32(int64_t ns, const int64_t *__restrict__ perm,
                                    const double *__restrict__ pin,
                                    cx<float> *__restrict__ p) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= ns) return;
  const int64_t a = perm[j];
  p[j] = cx<float>{float(pin[2 * a]), float(pin[2 * a + 1])};
}

template <int P>
__global__ void __launch_bounds__(64)
    k_leaf32_full(const int32_t *__restrict__ leaves,
                  const int32_t *__restrict__ lev,
                  const int64_t *__restrict__ t0, const int64_t *__restrict__ t1,
                  const int64_t *__restrict__ s0, const int64_t *__restrict__ s1,
                  const double *__restrict__ cxv, const double *__restrict__ cyv,
                  const double *__restrict__ rad,
                  const double *__restrict__ tx, const double *__restrict__ ty,
                  const int64_t *__restrict__ tperm,
                  const int64_t *__restrict__ uf_ptr,
                  const int32_t *__restrict__ uf_idx,
                  const int32_t *__restrict__ w_ptr,
                  const int32_t *__restrict__ w_src,
                  const double *__restrict__ sx, const double *__restrict__ sy,
                  const cx<float> *__restrict__ p,
                  const cx<float> *__restrict__ M,
                  const cx<float> *__restrict__ L, double *__restrict__ psi) {
  __shared__ double2 sz[kStage];
  __shared__ float2 sp[kStage];
  const int b = leaves[blockIdx.x];
  const int lane = threadIdx.x;
  const int64_t tb0 = t0[b], ntb = t1[b] - tb0;
  const int tp = ntb <= 32 ? pow2_at_least((int)ntb) : 64;
  const int S = 64 / tp, tl = lane % tp, sl = lane / tp;
  const int64_t uf0 = uf_ptr[b];
  const int utot = (int)(uf_ptr[b + 1] - uf0);  // U-list sources of the leaf
  const int wb = w_ptr[b], we = w_ptr[b + 1];
  for (int64_t tc = 0; tc < ntb; tc += tp) {
    const int64_t i = tb0 + tc + tl;
    const bool act = tc + tl < ntb;
    const double zx = act ? tx[i] : 0.0, zy = act ? ty[i] : 0.0;
    cx<float> f{0.f, 0.f};
    if (act) {
      if (sl == 0 && lev[b] >= 2) {
        const double ir = 1.0 / rad[b];
        const cx<float> w{float((zx - cxv[b]) * ir), float((zy - cyv[b]) * ir)};
        const cx<float> *La = L + (int64_t)b * P;
        cx<float> acc = La[P - 1];
        for (int l = P - 2; l >= 0; --l) acc = cfma(acc, w, La[l]);
        f = f + acc;
      }
      for (int e = wb + sl; e < we; e += S) {
        const int c = w_src[e];
        const double dx = zx - cxv[c], dy = zy - cyv[c];
        const double id = rad[c] / (dx * dx + dy * dy);
        const cx<float> rho{float(dx * id), float(-dy * id)};
        const cx<float> *a = M + (int64_t)c * P;
        cx<float> acc = a[P - 1];
        for (int k = P - 2; k >= 0; --k) acc = cfma(acc, rho, a[k]);
        f = f + acc * rho;
      }
    }
    {  // the leaf's U-list sources, kStage at a time
      const int total = utot;
      for (int q0 = 0; q0 < total; q0 += kStage) {
        const int take = min(kStage, total - q0);
        for (int q = lane; q < take; q += 64) {
          const int64_t j = uf_idx[uf0 + q0 + q];
          sz[q] = make_double2(sx[j], sy[j]);
          const cx<float> pj = p[j];
          sp[q] = make_float2(pj.x, pj.y);
        }
        __syncthreads();
        if (act) {
          for (int q = sl; q < take; q += S) {
            const double2 s2 = sz[q];
            const float2 p2 = sp[q];
            const float dx = (float)(zx - s2.x);
            const float dy = (float)(zy - s2.y);
            // p / d = p conj(d) / |d|^2; the 1e-30 bias makes a target's own
            // source (d = 0, in a self plan) contribute 0
            const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, fmaf(dy, dy, 1e-30f)));
            f.x += fmaf(p2.x, dx, p2.y * dy) * inv;
            f.y += fmaf(p2.y, dx, -p2.x * dy) * inv;
          }
        }
        __syncthreads();
      }
    }
    for (int o = tp; o < 64; o <<= 1) {
      f.x += __shfl_xor(f.x, o, 64);
      f.y += __shfl_xor(f.y, o, 64);
    }
    if (act && sl == 0) {
      const int64_t api = tperm[i];
      psi[2 * api] = f.x;
      psi[2 * api + 1] = f.y;
    }
  }
}

template <int P>
static void run32_full(const DevPlan &pl, const Tables &tb, Workspace &ws,
                       double *psi, hipStream_t s) {
  auto *p = (cx<float> *)ws.pstr32.p;
  auto *M = (cx<float> *)ws.mult32.p;
  auto *L = (cx<float> *)ws.loc32.p;
  far_field<float, P>(pl, tb, ws, p, M, L, 1, s);
  if (pl.n_leaf_t > 0)
    hipLaunchKernelGGL((k_leaf32_full<P>), dim3(pl.n_leaf_t), dim3(64), 0, s,
                       pl.leaf_t.p, pl.lev.p, pl.t0.p, pl.t1.p, pl.s0.p,
                       pl.s1.p, pl.cx.p, pl.cy.p, pl.rad.p, pl.tx.p, pl.ty.p,
                       pl.tgt_perm.p,
                       pl.uf_ptr.p, pl.uf_idx.p, pl.w_ptr.p, pl.w_src.p,
                       pl.sx.p, pl.sy.p,
                       (const cx<float> *)p, (const cx<float> *)M,
                       (const cx<float> *)L, psi);
}

void fmm_apply32_full(const DevPlan &pl, const Tables &tb, Workspace &ws,
                      const double *pin, double *psi, hipStream_t s) {
  if (pl.ns > 0)
    hipLaunchKernelGGL(k_strengths_given32, dim3((unsigned)((pl.ns + 255) / 256)),
                       dim3(256), 0, s, pl.ns, pl.src_perm.p, pin,
                       (cx<float> *)ws.pstr32.p);
  switch (tb.P) {
    case 12: run32_full<12>(pl, tb, ws, psi, s); break;
    case 16: run32_full<16>(pl, tb, ws, psi, s); break;
    case 20: run32_full<20>(pl, tb, ws, psi, s); break;
    case 24: run32_full<24>(pl, tb, ws, psi, s); break;
    default:
      throw ApiError{LBS_ERR_UNSUPPORTED, "p32 must be one of 12, 16, 20, 24"};
  }
  LBS_HIP(hipGetLastError());
}

}  // namespace lbs
