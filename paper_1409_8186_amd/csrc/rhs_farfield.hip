// Plane-wave right-hand side (paper Prop. 4) and far field (paper sec. 4.4).
//
//   U^p_m(beta) = sqrt(2 pi a_p) e^{i k beta_hat . O_p} e^{i m (pi/2 - beta)} J_m(k a_p)
//   f = -D^{-1} U = (2 i / pi) sqrt(2 pi) e^{i k beta_hat . O_p} e^{i m (pi/2 - beta)}
//                   / (sqrt(a_p) H_m(k a_p))             (J_m cancels)
//   a(theta) = sum_p sum_m g^p_m(theta) rho^p_m,
//   g^p_m(theta) = (e^{i pi/4} / (2 sqrt k)) e^{-i k theta_hat . O_p}
//                  sqrt(a_p) J_m(k a_p) e^{i m (theta - pi/2)}
//
// Point source s (Prop. 5): the same with the incident factor
//   e = (i/4) H_m(k r_p) e^{-i m theta_p}  (r_p, theta_p: polar coordinates of s - O_p)
// in place of e^{i k beta_hat . O_p} e^{i m (pi/2 - beta)}, so that
// U = sqrt(2 pi a) J_m e as for the plane wave.
#include <algorithm>

#include "bessel.h"
#include "common.h"

#define PI_D 3.14159265358979323846

// (i/4) H_m(k r) e^{-i m theta} of the source at src relative to disk p; NaN if
// the source is not outside the disk (the expansion needs r > a).
__device__ cplx point_factor(const DevView& v, int p, int m, const double* src) {
  const double dx = src[0] - v.cx[p], dy = src[1] - v.cy[p];
  const double r = sqrt(dx * dx + dy * dy);
  if (!(r > v.a[p])) return cmk(__builtin_nan(""), __builtin_nan(""));
  const double x = v.kd[p] * r;
  cplx Hm1, Hm;
  hankel01(x, &Hm1, &Hm);  // H_0, H_1
  const int am = m < 0 ? -m : m;
  if (am == 0) Hm = Hm1;
  for (int n = 1; n < am; ++n) {  // upward recurrence (stable: Y_n grows)
    const cplx Hn = csub(cscale(Hm, 2.0 * n / x), Hm1);
    Hm1 = Hm;
    Hm = Hn;
  }
  if (m < 0 && (am & 1)) Hm = cscale(Hm, -1.0);  // H_{-m} = (-1)^m H_m
  const cplx t = cmul(Hm, cexpi(-m * atan2(dy, dx)));
  return cmk(-0.25 * t.y, 0.25 * t.x);
}

// one thread per unknown of every (instance, rhs) column; `point`: beta holds
// source positions [B][R][2]; precond 0: U (or an operator's b), 1: the
// preconditioned b, 2: b (-U for the single layer)
__global__ void k_rhs(DevView v, int R, const double* __restrict__ beta, cplx* __restrict__ out,
                      int precond, int point) {
  const int64_t total = (int64_t)R * v.N_all;
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  // instance: R * imode[b] <= g < R * imode[b+1]
  int lo = 0, hi = v.B;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if ((int64_t)R * v.imode[mid] <= g) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int64_t Nb = v.imode[b + 1] - v.imode[b];
  const int64_t rem = g - (int64_t)R * v.imode[b];
  const int r = (int)(rem / Nb);
  const int64_t il = rem - (int64_t)r * Nb;
  const int64_t i = v.imode[b] + il;
  const int p = v.udisk[i];
  const int m = (int)(il - v.moff[p]) - v.N[p];
  cplx e;
  if (point) {
    e = point_factor(v, p, m, beta + 2 * ((int64_t)b * R + r));
  } else {
    const double be = beta[b * R + r];
    const double kk = v.kd[p];
    double sb, cb;
    sincos(be, &sb, &cb);
    const cplx e1 = cexpi(kk * (cb * v.cx[p] + sb * v.cy[p]));
    const cplx e2 = cexpi(m * (0.5 * PI_D - be));
    e = cmul(e1, e2);
  }
  const double s2pi = sqrt(2.0 * PI_D);
  if (v.op_rhs) {  // operator set by mudiff_set_operator: w_U U + w_dU dU (over its diagonal)
    out[g] = cmul(e, precond == 1 ? v.op_rhsp[i] : v.op_rhs[i]);
    return;
  }
  if (precond == 2) {  // the unpreconditioned system's right-hand side -U
    out[g] = cscale(e, -s2pi * v.sJ[i]);
    return;
  }
  if (precond) {
    const cplx w = cmul(e, v.invSH[i]);
    const double c = 2.0 / PI_D * s2pi;
    out[g] = cmk(-c * w.y, c * w.x);  // (2i/pi) sqrt(2 pi) e / (sqrt(a) H)
  } else {
    out[g] = cscale(e, s2pi * v.sJ[i]);
  }
}

int launch_rhs(mudiff_ctx* h, int R, const double* beta, cplx* out, int precond, int point,
               hipStream_t s) {
  const int64_t total = (int64_t)R * h->N_all;
  hipLaunchKernelGGL(k_rhs, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, h->dv, R, beta,
                     out, precond, point);
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}

extern "C" int mudiff_rhs(mudiff_t h, int R, const double* beta, void* out, int precond,
                          void* stream) {
  if (!h || !beta || !out) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  return launch_rhs(h, R, beta, (cplx*)out, precond ? 1 : 0, 0, (hipStream_t)stream);
}

extern "C" int mudiff_rhs_point(mudiff_t h, int R, const double* src, void* out, int precond,
                                void* stream) {
  if (!h || !src || !out) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  return launch_rhs(h, R, src, (cplx*)out, precond ? 1 : 0, 1, (hipStream_t)stream);
}

// Far field.  Workgroup = (column, tile of FF_TH angles); its FF_DG thread
// groups split the disks of the instance (thread t: angle t % FF_TH of the
// tile, disks g, g + FF_DG, ... with g = t / FF_TH), then the group sums are
// added in LDS in a fixed order.  Small tiles and many groups keep a
// one-column call (720 angles x 400 disks) spread over the chip; instances of
// few disks take wide tiles and few groups (16 x 64 or 64 x 16 threads).
template <int FF_TH, int FF_DG>
__global__ __launch_bounds__(FF_TH* FF_DG) void k_farfield(DevView v, int R,
                                                           const cplx* __restrict__ rho,
                                                           int n_theta,
                                                           const double* __restrict__ theta,
                                                           cplx* __restrict__ a_out) {
  __shared__ cplx red[FF_DG][FF_TH];
  const int col = blockIdx.y;  // b * R + r
  const int b = col / R, r = col - (col / R) * R;
  const int tj = threadIdx.x % FF_TH, dg = threadIdx.x / FF_TH;
  const int j = blockIdx.x * FF_TH + tj;
  const double th = j < n_theta ? theta[j] : 0.0;
  const double kk = v.kd[v.idisk[b]];
  const cplx* rc = rho + col_base(v.imode, b, R, r);
  double st, ct;
  sincos(th, &st, &ct);
  const cplx ephi = cexpi(th - 0.5 * PI_D);  // e^{i (theta - pi/2)}
  cplx acc = cmk(0.0, 0.0);
  for (int64_t p = v.idisk[b] + dg; p < v.idisk[b + 1]; p += FF_DG) {
    const int Np = v.N[p];
    const int64_t o = v.moff[p];
    const int64_t i0 = v.imode[b] + o;
    // sum_m sJ_m e^{i m phi} rho_m, m = -N..N, by the phase recurrence
    cplx e = cexpi(-Np * (th - 0.5 * PI_D));
    cplx sm = cmk(0.0, 0.0);
    for (int mm = 0; mm <= 2 * Np; ++mm) {
      cmac(sm, e, v.op_ff ? cmul(rc[o + mm], v.op_ff[i0 + mm]) : cscale(rc[o + mm], v.sJ[i0 + mm]));
      e = cmul(e, ephi);
    }
    const cplx ep = cexpi(-kk * (ct * v.cx[p] + st * v.cy[p]));
    cmac(acc, ep, sm);
  }
  red[dg][tj] = acc;
  __syncthreads();
  // groups 0..FF_DG-1 added in order: first eight partial runs of FF_DG / 8
  // groups, then the eight runs
  constexpr int RUN = FF_DG / 8;
  const bool summer = threadIdx.x < 8 * FF_TH;
  const int run = threadIdx.x / FF_TH;
  cplx sacc = cmk(0.0, 0.0);
  if (summer) {
    sacc = red[run * RUN][tj];
    for (int k = 1; k < RUN; ++k) sacc = cadd(sacc, red[run * RUN + k][tj]);
  }
  __syncthreads();  // every run read before any is overwritten
  if (summer) red[run][tj] = sacc;
  __syncthreads();
  if (dg == 0 && j < n_theta) {
    cplx s = red[0][tj];
    for (int k = 1; k < 8; ++k) s = cadd(s, red[k][tj]);
    // e^{i pi/4} / (2 sqrt k)
    const double c = 0.70710678118654752440 / (2.0 * sqrt(kk));
    a_out[(int64_t)col * n_theta + j] = cmul(cmk(c, c), s);
  }
}

// Far field of several columns: per instance the product
//   a[r][j] = c sum_{p, m} (s_m rho^p_m[r]) (e^{i m phi_j} e^{-i k theta_j . O_p})
// of [R x N_b] by [N_b x n_theta] on the FP64 matrix cores (v_mfma_f64_16x16x4f64:
// lane l holds A[l % 16][l / 16], B[l / 16][l % 16], D[4 v + l / 16][l % 16]).
// Workgroup: 16 columns x 16 angles, its NW waves splitting the disks; per k step
// of 4 modes a wave multiplies its densities with two panels [Re | Im] of 8 angles,
// so a complex product is two real MFMAs.  Nothing of the second factor is stored:
// e^{i m phi} of the tile's angles is a table in LDS, and e^{-i k theta . O_p} is
// evaluated once per disk (G = 4: by a lane group per disk, four disks at a time,
// handed on by lane exchange), so a phase serves 16 columns instead of one.  The
// wave sums are added in LDS in wave order.  Consecutive workgroups differ in
// their column tile, so that an XCD keeps meeting the same columns of rho in its L2.
typedef double ff_d4 __attribute__((ext_vector_type(4)));
// 256 columns of 1,000 disks at 360 angles (26 GFLOP): k_farfield, where every
// column forms its own phases, 4,810 us; 8-angle tiles 1,024 us (waiting for the
// densities, whose 16 columns are 16 separate segments per load); 16-angle tiles
// 760 us (34 TFLOP/s): 368 workgroups on 256 compute units, so the fuller ones run
// two, each busy 65% of that time.
#define FM_R 16
#define FM_T 16
#define FF_MFMA_N 127  // the table of phases fits 64 KB of LDS

template <int NW, int G, bool OPF>
__global__ __launch_bounds__(NW * 64) void k_farfield_mfma(DevView v, int R, const cplx* __restrict__ rho,
                                                           int n_theta, const double* __restrict__ theta,
                                                           cplx* __restrict__ a_out, int Nmax, int nct) {
  extern __shared__ cplx lds[];  // E [2 Nmax + 1][FM_T], then the wave sums [NW][512] (double)
  const int b = blockIdx.y;
  const int r0 = (int)(blockIdx.x % nct) * FM_R, t0 = (int)(blockIdx.x / nct) * FM_T;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int j = lane & 15, kq = lane >> 4, tj = j & 7;
  for (int e = tid; e < (2 * Nmax + 1) * FM_T; e += NW * 64) {
    const int jt = t0 + (e & (FM_T - 1));
    lds[e] = cexpi((e / FM_T - Nmax) * ((jt < n_theta ? theta[jt] : 0.0) - 0.5 * PI_D));
  }
  __syncthreads();
  const int64_t d0 = v.idisk[b], d1 = v.idisk[b + 1], i0 = v.imode[b];
  const double kk = v.kd[d0];
  double st[2], ct[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
    sincos(t0 + 8 * u + tj < n_theta ? theta[t0 + 8 * u + tj] : 0.0, &st[u], &ct[u]);
  // columns past R read column r0 (their sums are not stored)
  const cplx* __restrict__ rc = rho + col_base(v.imode, b, R, r0 + j < R ? r0 + j : r0);
  ff_d4 acc1[2], acc2[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    acc1[u] = ff_d4{0.0, 0.0, 0.0, 0.0};
    acc2[u] = ff_d4{0.0, 0.0, 0.0, 0.0};
  }
  for (int64_t p0 = d0 + G * wave; p0 < d1; p0 += G * NW) {
    cplx epg[2];  // G = 4: lane group kq evaluates disk p0 + kq
    const int64_t pe = min(p0 + (G == 4 ? kq : 0), d1 - 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) epg[u] = cexpi(-kk * (ct[u] * v.cx[pe] + st[u] * v.cy[pe]));
#pragma unroll
    for (int d = 0; d < G; ++d) {
      const int64_t p = p0 + d;
      if (p >= d1) break;
      double eu[2], ew[2];  // this lane's part of E ep: real for j < 8, imaginary else
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const cplx ep = G == 4 ? cmk(__shfl(epg[u].x, 16 * d + j, 64), __shfl(epg[u].y, 16 * d + j, 64)) : epg[u];
        eu[u] = j < 8 ? ep.x : ep.y;
        ew[u] = j < 8 ? -ep.y : ep.x;
      }
      const int Np = v.N[p], np = 2 * Np + 1;
      const int64_t o = v.moff[p] + kq;
      const cplx* __restrict__ E = lds + (Nmax - Np + kq) * FM_T + tj;
      const cplx* __restrict__ ra = rc + o;
      const double* __restrict__ sa = v.sJ + i0 + o;
      const cplx* __restrict__ fa = v.op_ff + i0 + o;
      auto step = [&](int m0, bool in) {  // modes m0 + kq; `in` false: past the disk's modes
        const int mm = in ? m0 : -kq;     // (they read mode 0 against a zero)
        cplx a = ra[mm];
        double f = in ? 1.0 : 0.0;
        if constexpr (OPF) a = cmul(a, fa[mm]);
        else f *= sa[mm];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const cplx e = E[mm * FM_T + 8 * u];
          const double bv = fma(e.x, eu[u], e.y * ew[u]) * f;
          acc1[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, bv, acc1[u], 0, 0, 0);
          acc2[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, bv, acc2[u], 0, 0, 0);
        }
      };
      int m0 = 0;
#pragma unroll 4
      for (; m0 + 4 <= np; m0 += 4) step(m0, true);
      step(m0, m0 + kq < np);  // n_p is odd: the last step is never full
    }
  }
  __syncthreads();  // E is no longer read
  double* red = reinterpret_cast<double*>(lds);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double other = __shfl_xor(acc2[u][q], 8, 64);
      // column 4 q + kq: real part of angle 8 u + j (j < 8), imaginary part of angle 8 u + j - 8
      red[wave * 512 + (4 * q + kq) * 32 + 16 * u + j] = j < 8 ? acc1[u][q] - other : acc1[u][q] + other;
    }
  __syncthreads();
  if (tid < FM_R * FM_T) {
    const int jt = tid & (FM_T - 1), r = r0 + tid / FM_T;
    const double* src = red + (tid / FM_T) * 32 + (jt & 7) + 2 * (jt & 8);
    cplx sm = cmk(0.0, 0.0);
    for (int w = 0; w < NW; ++w) sm = cadd(sm, cmk(src[w * 512], src[w * 512 + 8]));
    const double c = 0.70710678118654752440 / (2.0 * sqrt(kk));  // e^{i pi/4} / (2 sqrt k)
    if (r < R && t0 + jt < n_theta) a_out[((int64_t)b * R + r) * n_theta + t0 + jt] = cmul(cmk(c, c), sm);
  }
}

typedef void (*ff_fn)(DevView, int, const cplx*, int, const double*, cplx*, int, int);
static ff_fn ff_select(int64_t mmax, bool opf) {
  if (mmax >= 64) return opf ? k_farfield_mfma<16, 4, true> : k_farfield_mfma<16, 4, false>;
  if (mmax > 4) return opf ? k_farfield_mfma<16, 1, true> : k_farfield_mfma<16, 1, false>;
  return opf ? k_farfield_mfma<4, 1, true> : k_farfield_mfma<4, 1, false>;
}

extern "C" int mudiff_farfield(mudiff_t h, int R, const void* rho, int n_theta, const double* theta,
                               void* a_out, void* stream) {
  if (!h || !rho || !theta || !a_out) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  if (R < 1 || n_theta < 1) return fail(MUDIFF_ERR_INVALID, "R < 1 or n_theta < 1");
  if ((int64_t)h->B * R > 65535) return fail(MUDIFF_ERR_INVALID, "too many instance x RHS columns");
  int64_t mmax = 0;  // disks of the largest instance
  for (int b = 0; b < h->B; ++b) mmax = std::max<int64_t>(mmax, h->idisk[b + 1] - h->idisk[b]);
  const int64_t nct = (R + FM_R - 1) / FM_R, ntt = (n_theta + FM_T - 1) / FM_T;
  // The matrix-core kernel does the work of 16 columns however few there are, and a
  // workgroup walks all disks of its instance.  Below 4 columns the other kernel
  // does less in all; on instances of 64 disks and more it also ends earlier while
  // its workgroups (column, 16 angles) fit the chip about twice: 1,000 disks, 60
  // angles, 8 columns (32 workgroups) 158 against 389 us, 30 columns (120) 230
  // against 391, 256 columns at 360 angles (5,888) 4,810 against 760.
  bool many = R >= 4 && (mmax < 64 || (int64_t)h->B * R * ntt >= 512);
  // Instances of 5 to 63 disks with orders up to 8: a k step of 4 modes fills badly, so that
  // launches that fill the chip several times over need 5 or 6 columns (64 x 12 disks of order 2
  // at 360 angles: 4 columns 23.5 against 30.0 us, 5 columns 28, 28, 6 columns 34, 30; of order
  // 12 4 columns 44.8, 44.1; 64 x 20 of order 8 at 3,600 4 columns 1.03, of order 4 1.20 times
  // as long), and a launch of one round ends earlier on the other kernel from some 40 disks
  // and up to order 4 (50 of order 2 10.9 against 12.4; of order 5 0.96 times as long; 30 of
  // order 2 10.2, 9.4; in more rounds 0.4 to 0.7).
  if (many && mmax > 4 && mmax < 64 && h->Nmax <= 8) {
    const int64_t wgs = (int64_t)h->B * R * ((n_theta + 63) / 64);  // of the other kernel
    if (wgs >= 4 * (int64_t)h->n_cu) many = R >= (h->Nmax <= 2 ? 6 : 5);
    else if (wgs <= h->n_cu) many = mmax < 40 || h->Nmax > 4;
  }
  const int nw = mmax > 4 ? 16 : 4;
  // (a launch has fewer than 2^32 threads along x; the other kernel has its columns along y)
  if (many && h->Nmax <= FF_MFMA_N && nct * ntt * 64 * nw < ((int64_t)1 << 32)) {
    const ff_fn fn = ff_select(mmax, h->dv.op_ff != nullptr);
    const size_t lds = std::max((size_t)(2 * h->Nmax + 1) * FM_T * 16, (size_t)nw * 512 * 8);
    hipLaunchKernelGGL(fn, dim3((unsigned)(nct * ntt), (unsigned)h->B), dim3(64 * nw), lds, (hipStream_t)stream,
                       h->dv, R, (const cplx*)rho, n_theta, theta, (cplx*)a_out, h->Nmax, (int)nct);
  } else if (mmax >= 64) {
    dim3 grid((n_theta + 15) / 16, h->B * R);
    hipLaunchKernelGGL((k_farfield<16, 64>), grid, dim3(1024), 0, (hipStream_t)stream, h->dv, R,
                       (const cplx*)rho, n_theta, theta, (cplx*)a_out);
  } else {
    dim3 grid((n_theta + 63) / 64, h->B * R);
    hipLaunchKernelGGL((k_farfield<64, 16>), grid, dim3(1024), 0, (hipStream_t)stream, h->dv, R,
                       (const cplx*)rho, n_theta, theta, (cplx*)a_out);
  }
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}
