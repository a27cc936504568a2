// Near field (paper sec. 4.4, by Graf's addition theorem): at a point x of the
// propagation domain, with (r_p, theta_p) the polar coordinates of x - O_p,
//   u(x) = sum_p sum_m (i sqrt(pi / 8)) F^p_m rho^p_m H_m(k r_p) e^{i m theta_p},
// F^p_m = sqrt(a_p) J_m(k a_p) for the single-layer potential; for an operator
// set by mudiff_set_operator, F = f_L sqrt(a) J_m - f_M k sqrt(a) J'_m (its
// far-field weights: single- plus double-layer potential).  The total field
// adds the incident wave: the plane wave e^{i k beta_hat . x}, or for a point
// source s (Prop. 5) G(x, s) = (i/4) H_0(k |x - s|).  Points inside a disk get 0.
//
// One thread per point, every thread walking the same disks (so the disk data
// and the coefficients are wave-uniform loads); per (point, disk): H_0, H_1 of
// k r_p (Miller + Neumann series below 25, Hankel's expansion above), H_m by
// upward recurrence (stable for the Y part that dominates), e^{i m theta} by
// recurrence, and the mode sum for up to NF_RC right-hand sides at once.
// Bound by FP64 issue (about 390 vector instructions per point and disk of N_p = 12:
// 15 per order, 85 for the phase and amplitude, 40 for the expansion, 30 for r).
// 1e6 points around 400 disks: 10.0 ms with the series term by term, the modes +m
// and -m as two complex products and a barrier pair per disk; 7.1 with polynomials,
// combined coefficients and start orders that suit the range (four waves per SIMD:
// at two, 10.4); 5.6 with the coefficients of several disks staged at a time and no
// registers for absent right-hand sides.
#include <algorithm>

#include "bessel.h"
#include "common.h"

namespace {

constexpr int NF_THREADS = 256;
constexpr int NF_WAVES = NF_THREADS / 64;
constexpr int NF_RC = 4;
// disks whose coefficients are staged at a time: as many as fit this LDS, which
// leaves room for the workgroups that the registers allow
constexpr size_t NF_LDS = 16 * 1024;
constexpr int NF_DISKS = 16;

// Hankel's large-argument expansion of H_0, H_1 (DLMF 10.17.5) with a fixed
// number of terms by range: the k-th term is a_k(nu) (i / x)^k, a_k = prod_{j<=k}
// (4 nu^2 - (2j-1)^2) / (8 j), below 3e-17 at x = 25 for k = 18, at x = 50 for
// k = 12 and at x = 100 for k = 9 (nu = 0, 1).  The even terms are real and the
// odd ones imaginary: two polynomials in 1 / x^2 by Horner's rule, one
// multiply-add per term (term by term, with the complex factor, it was five).
// Same phase handling as the table code: e^{ix} from sincos of the exact argument.
constexpr double hankel_a(int nu, int k) {
  double a = 1.0;
  for (int j = 1; j <= k; ++j) a *= (4.0 * nu * nu - (2.0 * j - 1.0) * (2.0 * j - 1.0)) / (8.0 * j);
  return (k / 2) % 2 ? -a : a;  // with the sign of i^k, i^(k-1) for odd k
}

// sum over the k = K0, K0 + 2, .. <= K of hankel_a(NU, k) y^{(k - K0) / 2}
template <int NU, int K0, int K>
__device__ __forceinline__ double hankel_poly(double y) {
  if constexpr (K0 + 2 > K) {
    return hankel_a(NU, K0);
  } else {
    return fma(hankel_poly<NU, K0 + 2, K>(y), y, hankel_a(NU, K0));
  }
}

template <int K>
__device__ __forceinline__ void hankel01_series(double ixx, cplx* s0, cplx* s1) {
  const double y = ixx * ixx;
  *s0 = cmk(hankel_poly<0, 0, K>(y), hankel_poly<0, 1, K>(y) * ixx);
  *s1 = cmk(hankel_poly<1, 0, K>(y), hankel_poly<1, 1, K>(y) * ixx);
}

// H_0, H_1 for x < BESSEL_X_ASY: Miller's algorithm and Neumann's series as in
// bessel.h, from a start order that is the same for all lanes (the orders' factors
// and the series' coefficients then are constants): NS with (x/2)^NS / NS! below
// 1e-20 at the top of each range, NS even.
template <int NS>
__device__ __forceinline__ void hankel01_miller(double x, cplx* H0, cplx* H1) {
  const double tox = 2.0 / x;
  double jp = 0.0, j = 1.0;  // J_{n+1}, J_n (unnormalised)
  double norm = 0.0, s0 = 0.0, s1 = 0.0;
#pragma unroll 4
  for (int n = NS; n > 0; n -= 2) {  // J_n, n even, then J_{n-1}
    const int k = n / 2;
    const double ik = 1.0 / k, sg = k & 1 ? -1.0 : 1.0;  // wave-uniform
    norm += j;
    s0 = fma(sg * ik, j, s0);
    const double jm = fma(n * tox, j, -jp);  // J_{n-1}
    // coefficient of J_{2(k-1)+1} in S1 = sum (-1)^k (J_{2k-1} - J_{2k+1}) / k
    const double c = k > 1 ? sg * (1.0 / (k - 1) + ik) : -1.0;
    s1 = fma(c, jm, s1);
    jp = jm;
    j = fma((n - 1) * tox, jm, -j);  // J_{n-2}
  }
  const double inv = 1.0 / fma(2.0, norm, j);  // J_0 + 2 sum J_{2k} = 1
  double Y0, Y1;
  bessel_y01_neumann(x, j * inv, jp * inv, s0 * inv, s1 * inv, &Y0, &Y1);
  *H0 = cmk(j * inv, Y0);
  *H1 = cmk(jp * inv, Y1);
}

// H_0(x), H_1(x) given x and ixx = 1 / x.
__device__ __forceinline__ void hankel01_near(double x, double ixx, cplx* H0, cplx* H1) {
  if (x < BESSEL_X_ASY) {
    if (!(x >= 1e-18)) hankel01(x, H0, H1);  // scaled recurrences
    else if (x < 0.05) hankel01_miller<12>(x, H0, H1);
    else if (x < 5.0) hankel01_miller<30>(x, H0, H1);
    else if (x < 12.0) hankel01_miller<46>(x, H0, H1);
    else hankel01_miller<70>(x, H0, H1);
    return;
  }
  cplx s0, s1;
  if (x >= 100.0) hankel01_series<10>(ixx, &s0, &s1);
  else if (x >= 50.0) hankel01_series<13>(ixx, &s0, &s1);
  else hankel01_series<19>(ixx, &s0, &s1);
  double sn, cs;
  sincos(x, &sn, &cs);
  // sqrt(2 / (pi x)) e^{i (x - pi/4)} = amp (cos x + sin x, sin x - cos x), and -i times that
  const double amp = sqrt(0.31830988618379067154 * ixx);  // sqrt(1 / (pi x))
  const cplx u = cmk(amp * (cs + sn), amp * (sn - cs));
  *H0 = cmul(u, s0);
  *H1 = cmul(cmk(u.y, -u.x), s1);
}

__device__ __forceinline__ void hankel01_near(double x, cplx* H0, cplx* H1) {
  hankel01_near(x, 1.0 / x, H0, H1);
}

// RC right-hand sides per workgroup; the coefficients of D disks at a time in LDS:
// with c_m = (i sqrt(pi/8)) F_m rho_m, per order m >= 0 the pair
// (c_m + (-1)^m c_{-m}, i (c_m - (-1)^m c_{-m})), (c_0, 0) at m = 0.
// SPLIT: 64 points per workgroup, wave w taking every NF_WAVES-th of the staged disks,
// the waves' sums added in their order.
template <int RC, bool SPLIT>
__global__ __launch_bounds__(NF_THREADS, 4) void k_nearfield(DevView v, int R, const cplx* __restrict__ rho,
                                                             int n_pts, const double* __restrict__ pts,
                                                             const double* __restrict__ beta, int point,
                                                             cplx* __restrict__ out, int Nmax, int D) {
  extern __shared__ cplx lds[];  // [D][Nmax + 1][2][RC]; SPLIT: then the sums [RC][NF_THREADS]
  __shared__ int s_in[SPLIT ? NF_THREADS : 1];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int P = SPLIT ? blockIdx.x * 64 + (threadIdx.x & 63) : blockIdx.x * NF_THREADS + threadIdx.x;
  const int nchunk = (R + RC - 1) / RC;
  const int b = blockIdx.y / nchunk;
  const int r0 = (blockIdx.y - b * nchunk) * RC;
  const int nr = min(RC, R - r0);
  const double x1 = P < n_pts ? pts[2 * P] : 0.0, x2 = P < n_pts ? pts[2 * P + 1] : 0.0;
  const double k = v.kd[v.idisk[b]];
  const double ik = 1.0 / k;
  const double cst = 0.62665706865775012560;  // sqrt(pi / 8): (i pi a / 2) / sqrt(2 pi a) = i sqrt(pi/8) sqrt(a)
  cplx acc[RC];
#pragma unroll
  for (int c = 0; c < RC; ++c) acc[c] = cmk(0.0, 0.0);
  bool inside = false;
  const int64_t p1 = v.idisk[b + 1];
  const int per = (Nmax + 1) * RC;  // pairs of a disk
  for (int64_t pd = v.idisk[b]; pd < p1; pd += D) {
    const int nd = (int)min((int64_t)D, p1 - pd);
    __syncthreads();  // the previous disks' coefficients are no longer read
    for (int e = threadIdx.x; e < nd * per; e += NF_THREADS) {
      const int dd = e / per, q = e - dd * per, m = q / RC, c = q - m * RC;
      const int64_t p = pd + dd;
      const int Np = v.N[p];
      if (m > Np) continue;
      const int64_t i0 = v.imode[b] + v.moff[p];  // unknown of mode -N_p
      cplx tp = cmk(0.0, 0.0), tm = tp;
      if (c < nr) {
        const cplx* rc = rho + col_base(v.imode, b, R, r0 + c) + v.moff[p];
        auto coef = [&](int mi) {
          const cplx F = v.op_ff ? v.op_ff[i0 + mi] : cmk(v.sJ[i0 + mi], 0.0);
          const cplx t = cmul(F, rc[mi]);
          return cmk(-cst * t.y, cst * t.x);
        };
        tp = coef(Np + m);
        if (m > 0) tm = coef(Np - m);
        if (m & 1) tm = cmk(-tm.x, -tm.y);
      }
      const cplx df = csub(tp, tm);
      cplx* cf = lds + 2 * (dd * per + m * RC) + c;
      cf[0] = cadd(tp, tm);
      cf[RC] = cmk(-df.y, df.x);
    }
    __syncthreads();
    for (int dd = SPLIT ? wv : 0; dd < nd; dd += SPLIT ? NF_WAVES : 1) {
      const int64_t p = pd + dd;
      const int Np = v.N[p];
      const cplx* cf = lds + 2 * dd * per;
      const double dx = x1 - v.cx[p], dy = x2 - v.cy[p];
      const double r2 = dx * dx + dy * dy;
      const double ap = v.a[p];
      if (r2 < ap * ap) {
        inside = true;
        continue;
      }
      const double r = sqrt(r2);   // correctly rounded: the phase of e^{i k r} rests on it
      const double ir = rsqrt(r2);  // 1 / r, and 1 / (k r) below, with no division
      const double xx = k * r;
      const double ixx = ik * ir;
      const double tox = 2.0 * ixx;
      cplx H0, H1;
      hankel01_near(xx, ixx, &H0, &H1);
      const cplx e1 = cmk(dx * ir, dy * ir);  // e^{i theta_p}
#pragma unroll
      for (int c = 0; c < RC; ++c)
        if (RC == 1 || c < nr) cmac(acc[c], cf[c], H0);
      // H_{-m} e^{-i m theta} = (-1)^m H_m e^{-i m theta}: both modes of order m take
      // ((c_m + (-1)^m c_{-m}) cos m theta + i (c_m - (-1)^m c_{-m}) sin m theta) H_m
      auto add = [&](int m, cplx em, cplx Hm) {
        const cplx* cm = cf + 2 * m * RC;
#pragma unroll
        for (int c = 0; c < RC; ++c)
          if (RC == 1 || c < nr) {
            const cplx s = cm[c], d = cm[RC + c];
            const cplx t = cmk(fma(s.x, em.x, d.x * em.y), fma(s.y, em.x, d.y * em.y));
            cmac(acc[c], t, Hm);
          }
      };
      cplx Ha = H0, Hb = H1, em = e1;  // H_{m-1}, H_m at the top of the loop
      double f = 1.0;                  // m
      for (int m = 1; m <= Np; m += 2) {
        add(m, em, Hb);
        if (m + 1 > Np) break;
        const double fa = f * tox, fb = (f + 1.0) * tox;  // 2 m / x, 2 (m + 1) / x
        Ha = cmk(fma(Hb.x, fa, -Ha.x), fma(Hb.y, fa, -Ha.y));
        em = cmul(em, e1);
        add(m + 1, em, Ha);
        Hb = cmk(fma(Ha.x, fb, -Hb.x), fma(Ha.y, fb, -Hb.y));
        em = cmul(em, e1);
        f += 2.0;
      }
    }
  }
  if constexpr (SPLIT) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < RC; ++c) lds[c * NF_THREADS + threadIdx.x] = acc[c];
    s_in[threadIdx.x] = inside;
    __syncthreads();
    if (wv > 0) return;
    for (int w = 1; w < NF_WAVES; ++w) {
      inside |= s_in[w * 64 + threadIdx.x] != 0;
#pragma unroll
      for (int c = 0; c < RC; ++c) acc[c] = cadd(acc[c], lds[c * NF_THREADS + w * 64 + threadIdx.x]);
    }
  }
  if (P >= n_pts) return;
#pragma unroll
  for (int c = 0; c < RC; ++c) {
    if (c >= nr) continue;
    const int col = b * R + r0 + c;
    cplx u = acc[c];
    if (beta && point) {
      const double dx = x1 - beta[2 * col], dy = x2 - beta[2 * col + 1];
      cplx H0, H1;
      hankel01_near(k * sqrt(dx * dx + dy * dy), &H0, &H1);
      u = cadd(u, cmk(-0.25 * H0.y, 0.25 * H0.x));
    } else if (beta) {
      double sb, cb;
      sincos(beta[col], &sb, &cb);
      u = cadd(u, cexpi(k * (cb * x1 + sb * x2)));
    }
    out[(int64_t)col * n_pts + P] = inside ? cmk(0.0, 0.0) : u;
  }
}

}  // namespace

extern "C" int mudiff_nearfield(mudiff_t h, int R, const void* rho, int n_pts, const double* pts,
                                const double* beta, int flags, void* out, void* stream) {
  if (!h || !rho || !pts || !out) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  if (flags & ~MUDIFF_POINT_SOURCE) return fail(MUDIFF_ERR_INVALID, "unknown flags");
  if (R < 1 || n_pts < 1) return fail(MUDIFF_ERR_INVALID, "R < 1 or n_pts < 1");
  const int nchunk = (R + NF_RC - 1) / NF_RC;
  if ((int64_t)h->B * nchunk > 65535) return fail(MUDIFF_ERR_INVALID, "too many instance x RHS columns");
  const int rc = R == 1 ? 1 : (R == 2 ? 2 : NF_RC);  // right-hand sides that share a Hankel evaluation
  typedef void (*fn_t)(DevView, int, const cplx*, int, const double*, const double*, int, cplx*, int, int);
  const size_t disk = (size_t)(h->Nmax + 1) * 2 * rc * 16;  // LDS of a disk's coefficients
  // Fewer workgroups of 256 points than are resident at once (a quarter of that with few
  // disks): 64 points each, the disks split over the waves.  us without and with: 20 disks,
  // 1,000 points 107, 45; 100 disks, 1,000 points 466, 161; 300 disks, 2,000 points, 5
  // columns 1,968, 608; 100 disks, 200,000 points, 2 columns 611, 534; 400 disks, 250,000
  // points 1,728, 1,623; 4 disks, 50,000 points 35, 26, but 200,000 47, 53; 5 disks, 100,000
  // points, 2 columns 39.5, 41.0.
  const int64_t wgs = (int64_t)((n_pts + NF_THREADS - 1) / NF_THREADS) * h->B * nchunk;
  int D = (int)std::max<size_t>(1, std::min<size_t>(NF_DISKS, NF_LDS / disk));
  const int DS = (int)std::min<size_t>(NF_DISKS, 2 * NF_LDS / disk) / NF_WAVES * NF_WAVES;
  const bool split = DS > 0 && h->M_all >= 2 * h->B &&
                     wgs < (int64_t)h->n_cu * (h->M_all >= 8 * h->B ? 4 : 1);
  if (split) D = DS;
  const size_t lds = std::max(D * disk, split ? (size_t)NF_THREADS * rc * 16 : 0);
  static const fn_t kFn[2][3] = {{k_nearfield<1, false>, k_nearfield<2, false>, k_nearfield<NF_RC, false>},
                                 {k_nearfield<1, true>, k_nearfield<2, true>, k_nearfield<NF_RC, true>}};
  const int pts_wg = split ? 64 : NF_THREADS;
  dim3 grid((unsigned)((n_pts + pts_wg - 1) / pts_wg), (unsigned)(h->B * nchunk));
  hipLaunchKernelGGL(kFn[split][rc == 1 ? 0 : (rc == 2 ? 1 : 2)], grid, dim3(NF_THREADS), lds,
                     (hipStream_t)stream, h->dv, R, (const cplx*)rho, n_pts, pts, beta,
                     (flags & MUDIFF_POINT_SOURCE) ? 1 : 0, (cplx*)out, h->Nmax, D);
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}
