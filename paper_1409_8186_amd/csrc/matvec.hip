// Operator apply y = L x or y = D^{-1} L x (paper sec. 4.2 block formulas,
// sec. 5 single-scattering preconditioner).
//
// Off-diagonal block (p, q):  (L^{pq} x^q)_m = (i pi/2) s_m sum_n t^{pq}_{n-m} z^q_n,
//   s_m = sqrt(a_p) J_m(k a_p),  z^q_n = sqrt(a_q) J_n(k a_q) x^q_n,
// a Toeplitz product in the mode difference n - m.  The preconditioned form
// divides row m of disk p by L^{pp}_{mm}: (A x)_m = x_m + w_m / (sqrt(a_p) H_m(k a_p)),
// w_m = sum_{q != p} sum_n t^{pq}_{n-m} z^q_n (J_m(k a_p) cancels exactly).
//
// Work decomposition: an item is (row disk p, chunk of column disks).  A
// 256-thread workgroup stages, for a pass of PP column disks, the symbol rows
// t^{pq} and the scaled inputs z^q in LDS (coalesced global loads), then each
// thread accumulates BT consecutive outputs m of one pair over all n.  Chunk
// partial sums go to scratch; the last workgroup of a row (atomic counter)
// adds them in chunk order, so the result does not depend on scheduling.
#include "common.h"

#include <algorithm>
#include <cstring>
#include <mutex>


#define APPLY_THREADS 256
#define APPLY_NPASS 2

__global__ void k_fill_zero(uint32_t* p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0u;
}

int launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  size_t n = bytes / 4;
  if (n == 0) return MUDIFF_OK;
  unsigned g = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill_zero, dim3(g), dim3(256), 0, s, (uint32_t*)p, n);
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}

// acc[b] += sum_n tb[n - b] z[n],  tb = trow + (LB - 1) - m0
template <int BT, int NQ>
__device__ __forceinline__ void toeplitz_block(const cplx* __restrict__ zrow,
                                               const cplx* __restrict__ tb, int nq_pad,
                                               cplx (&acc)[BT]) {
  if constexpr (NQ > 0) {
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const cplx z = zrow[n];
#pragma unroll
      for (int b = 0; b < BT; ++b) cmac(acc[b], tb[n - b], z);
    }
  } else {
    for (int n0 = 0; n0 < nq_pad; n0 += BT) {
#pragma unroll
      for (int d = 0; d < BT; ++d) {
        const cplx z = zrow[n0 + d];
#pragma unroll
        for (int b = 0; b < BT; ++b) cmac(acc[b], tb[n0 + d - b], z);
      }
    }
  }
}

// Output of row unknown i from x_i and the off-diagonal contraction w_i.

// NSPEC >= 0: every disk of the launch has N_p = NSPEC (exact loop bounds).
template <int BT, int NSPEC>
__global__ __launch_bounds__(APPLY_THREADS) void k_apply(
    DevView v, int R, const cplx* __restrict__ x, cplx* __restrict__ y, int op,
    cplx* __restrict__ part, int64_t part_total, int32_t* __restrict__ counters,
    const int32_t* __restrict__ items, const int32_t* __restrict__ nchunk,
    const int64_t* __restrict__ partoff, const int32_t* __restrict__ active, int zs, int ts,
    int ppcap, const cplx* __restrict__ shift) {
  extern __shared__ cplx lds[];
  __shared__ int s_last;
  const int it = blockIdx.x, r = blockIdx.y;
  const int p = items[4 * it], c = items[4 * it + 1], jb = items[4 * it + 2], je = items[4 * it + 3];
  const int b = v.inst[p];
  if (active && active[b * R + r] == 0) return;
  const int Np = NSPEC >= 0 ? NSPEC : v.N[p];
  const int np = 2 * Np + 1;
  const int L = (np + BT - 1) / BT;
  const int LB = L * BT;
  const int PP = min(APPLY_THREADS / L, ppcap);
  const int64_t d0 = v.idisk[b];
  const int64_t i0 = v.imode[b];
  const int64_t cb = col_base(v.imode, b, R, r);
  const cplx* __restrict__ xc = x + cb;
  const int tid = threadIdx.x;
  const int slot = tid / L, mb = tid - (tid / L) * L;
  const int m0 = mb * BT;
  cplx* zl = lds;                 // [PP][zs]
  cplx* tl = lds + PP * zs;       // [PP][ts]

  cplx acc[BT];
#pragma unroll
  for (int k = 0; k < BT; ++k) acc[k] = cmk(0.0, 0.0);

  for (int j0 = jb; j0 < je; j0 += PP) {
    const int nslot = min(PP, je - j0);
    __syncthreads();
    // stage z^q = sqrt(a_q) J_n(k a_q) x^q_n
    for (int e = tid; e < PP * zs; e += APPLY_THREADS) {
      const int k = e / zs, n = e - (e / zs) * zs;
      cplx z = cmk(0.0, 0.0);
      if (k < nslot) {
        const int q = (int)(d0 + j0 + k + ((d0 + j0 + k) >= p ? 1 : 0));
        const int nq = 2 * (NSPEC >= 0 ? NSPEC : v.N[q]) + 1;
        if (n < nq) {
          const int64_t iq = v.moff[q] + n;
          z = col_scale(v, i0 + iq, xc[iq]);
        }
      }
      zl[e] = z;
    }
    // stage symbol rows: u = n - m + LB - 1  <->  s = u - (LB - 1) - N_q + N_p
    for (int e = tid; e < PP * ts; e += APPLY_THREADS) {
      const int k = e / ts, u = e - (e / ts) * ts;
      cplx t = cmk(0.0, 0.0);
      if (k < nslot) {
        const int q = (int)(d0 + j0 + k + ((d0 + j0 + k) >= p ? 1 : 0));
        const int Nq = NSPEC >= 0 ? NSPEC : v.N[q];
        const int S = Np + Nq;
        const int s = u - (LB - 1) - Nq + Np;
        if (s >= -S && s <= S) {
          const int64_t g = pair_index(v.idisk, v.ipair, b, p, q);
          t = v.t[v.toff[g] + S + s];
          if (p > q && (s & 1)) t = cmk(-t.x, -t.y);  // t^{qp}_s = (-1)^s t^{pq}_s
        }
      }
      tl[e] = t;
    }
    __syncthreads();
    if (slot < nslot) {
      const cplx* tb = tl + slot * ts + (LB - 1) - m0;
      if constexpr (NSPEC >= 0)
        toeplitz_block<BT, 2 * NSPEC + 1>(zl + slot * zs, tb, 0, acc);
      else
        toeplitz_block<BT, 0>(zl + slot * zs, tb, zs, acc);
    }
  }
  // reduce over pair slots
  __syncthreads();
  cplx* red = lds;  // [PP][LB]
  if (slot < PP) {
#pragma unroll
    for (int k = 0; k < BT; ++k) red[slot * LB + m0 + k] = acc[k];
  }
  __syncthreads();
  const int nch = nchunk[p];
  const int64_t ip = i0 + v.moff[p];  // unknown index (single column) of mode -N_p
  cplx* yc = y + cb + v.moff[p];
  const cplx* xp = xc + v.moff[p];
  const int nslot_max = min(PP, je - jb);
  if (nch == 1) {
    for (int m = tid; m < np; m += APPLY_THREADS) {
      cplx w = cmk(0.0, 0.0);
      for (int k = 0; k < nslot_max; ++k) w = cadd(w, red[k * LB + m]);
      cplx o = finalize(v, op, ip + m, xp[m], w);
      if (shift) o = affine(shift, b * R + r, o, xp[m]);
      yc[m] = o;
    }
    return;
  }
  cplx* pr = part + (int64_t)r * part_total + partoff[p];
  for (int m = tid; m < np; m += APPLY_THREADS) {
    cplx w = cmk(0.0, 0.0);
    for (int k = 0; k < nslot_max; ++k) w = cadd(w, red[k * LB + m]);
    pr[(int64_t)c * np + m] = w;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // publish this chunk
  __syncthreads();
  if (tid == 0) {
    int32_t* cnt = counters + (int64_t)r * v.M_all + p;
    int old = atomicAdd(cnt, 1);
    s_last = (old == nch - 1);
    if (s_last) atomicExch(cnt, 0);
  }
  __syncthreads();
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // see the other chunks
  for (int m = tid; m < np; m += APPLY_THREADS) {
    cplx w = cmk(0.0, 0.0);
    for (int k = 0; k < nch; ++k) {
      w = cadd(w, pr[(int64_t)k * np + m]);  // visible after the fence above
    }
    cplx o = finalize(v, op, ip + m, xp[m], w);
    if (shift) o = affine(shift, b * R + r, o, xp[m]);
    yc[m] = o;
  }
}

// ------------------------------------------------------------------ few disks
// Instances of up to FEW_DISKS disks, few right-hand sides: bound by latency, the chain
// of loads from the schedule to the symbols and the launch itself.  A workgroup takes 32
// outputs of a row disk and every column disk of its instance, so there are no partial
// sums.  What it needs to know of the column disks stands in its task, so that two rounds
// of loads come before the arithmetic (the LDS-staged kernel has six, through the tables).
// Wave w stages column disks w, w + 4, .. (scaled inputs z and the symbols of the 32
// outputs) and sums over them, 8 lanes over the modes n times 8 lanes of the outputs m,
// m + 8, m + 16, m + 24: a symbol read for one output serves the next one 8 modes later.
// 4 disks of 31 modes: 6.35 us as LDS-staged rows, 3.5 so.
#define FEW_THREADS 256
#define FEW_WAVES (FEW_THREADS / 64)
#define FEW_HDR 12  // instance, first output, N_p, column disks, then 64 bits: unknown of mode -N_p, imode, N_b
#define FEW_COL 4   // offset in the instance vector, 2 N_q + (1: times (-1)^s), 64 bits: symbol t^{pq}_0
#define FEW_PAD 31  // window entries before output m0's, for the outputs after it

// The tables it reads, for the operator and op of the launch: y = alpha x + beta w
// (al NULL: alpha is 1; be NULL: beta = (i pi / 2) sJ; raw: y = w).
struct FewView {
  const cplx *t, *col, *al, *be;  // col NULL: the column factors are sJ
  const double* sJ;
  bool raw;
};

__global__ __launch_bounds__(FEW_THREADS) void k_apply_few(
    FewView v, int R, const cplx* __restrict__ x, cplx* __restrict__ y,
    const int32_t* __restrict__ tasks, int stride, const int32_t* __restrict__ active,
    const cplx* __restrict__ shift, int cols, int zcap) {
  extern __shared__ cplx lds[];  // [FEW_WAVES][cols][zcap z, zcap + FEW_PAD symbols]
  __shared__ double red[FEW_WAVES][64];
  const int r = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int32_t* it = tasks + (int64_t)stride * blockIdx.x;
  const int b = it[0], m0 = it[1], Np = it[2], nc = it[3];
  const int64_t ip = *reinterpret_cast<const int64_t*>(it + 4), im = *reinterpret_cast<const int64_t*>(it + 6);
  const int64_t cb = (int64_t)R * im + (int64_t)r * *reinterpret_cast<const int64_t*>(it + 8);
  if (active && active[b * R + r] == 0) return;
  cplx xv = cmk(0.0, 0.0), al = xv, be = xv;
  const bool out = tid < 32 && m0 + tid <= 2 * Np;
  if (out) {
    const int64_t i = ip + m0 + tid;
    xv = x[cb + (i - im)];
    be = v.be ? v.be[i] : cmk(0.0, 0.5 * 3.14159265358979323846 * v.sJ[i]);
    if (v.al) al = v.al[i];
  }
  cplx* base = lds + (size_t)wv * cols * (2 * zcap + FEW_PAD);
  int k = 0;
  for (int c = wv; c < nc; c += FEW_WAVES, ++k) {
    const int32_t* rec = it + FEW_HDR + FEW_COL * c;
    const int qo = rec[0], Nq = rec[1] >> 1, neg = rec[1] & 1;
    const cplx* __restrict__ t = v.t + *reinterpret_cast<const int64_t*>(rec + 2);
    cplx* zl = base + (size_t)k * (2 * zcap + FEW_PAD);
    cplx* tl = zl + zcap;
    const int nq = 2 * Nq + 1, s0 = Np - Nq - m0 - FEW_PAD;  // window entry u holds t_{u + s0}
    for (int n = lane; n < nq; n += 64) zl[n] = v.col ? cmul(x[cb + qo + n], v.col[im + qo + n]) : cscale(x[cb + qo + n], v.sJ[im + qo + n]);
    for (int u = lane; u < nq + FEW_PAD; u += 64) {
      const int sy = u + s0;
      cplx e = sy >= -(Np + Nq) ? t[sy] : cmk(0.0, 0.0);  // below: outputs past 2 N_p
      if (neg && (sy & 1)) e = cmk(-e.x, -e.y);
      tl[u] = e;
    }
  }
  __syncthreads();
  const int part = lane & 7, mi = lane >> 3;
  cplx a[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = cmk(0.0, 0.0);
  k = 0;
  for (int c = wv; c < nc; c += FEW_WAVES, ++k) {
    const int nq = (it[FEW_HDR + FEW_COL * c + 1] | 1), full = nq >> 3;  // 2 N_q + 1
    const cplx* zq = base + (size_t)k * (2 * zcap + FEW_PAD) + part;
    const cplx* tq = zq + zcap + FEW_PAD - mi;
    cplx t1 = tq[-8], t2 = tq[-16], t3 = tq[-24];
    auto step = [&](int n) {
      const cplx t = tq[n], z = zq[n];
      cmac(a[0], t, z);
      cmac(a[1], t1, z);
      cmac(a[2], t2, z);
      cmac(a[3], t3, z);
      t3 = t2;
      t2 = t1;
      t1 = t;
    };
#pragma unroll 4
    for (int i = 0; i < full; ++i) step(8 * i);
    if (part < (nq & 7)) step(8 * full);
  }
  double val[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    val[2 * i] = a[i].x;
    val[2 * i + 1] = a[i].y;
  }
  rs_dpp_step<4, 8>(val, lane);
  rs_dpp_step<2, 4>(val, lane);
  rs_dpp_step<1, 2>(val, lane);
  red[wv][lane] = val[0];  // lane (mi, part): Re, Im of output mi + 8 (part / 2)
  __syncthreads();
  if (!out) return;
  cplx w = cmk(0.0, 0.0);
  const int l = 8 * (tid & 7) + 2 * (tid >> 3);
#pragma unroll
  for (int i = 0; i < FEW_WAVES; ++i) w = cadd(w, cmk(red[i][l], red[i][l + 1]));
  cplx o = w;
  if (!v.raw) o = cadd(v.al ? cmul(al, xv) : xv, cmul(be, w));
  if (shift) o = affine(shift, b * R + r, o, xv);
  y[cb + (ip - im) + m0 + tid] = o;
}

// ------------------------------------------------------------------ one lane per pair
// Uniform N_p = N (<= 12), few right-hand sides.  A wave takes a row disk p, one
// right-hand side and a chunk of up to 64 column disks q, one
// lane per ordered pair (p, q), with all n = 2N+1 outputs of the pair in
// registers; a workgroup is one row disk, whose lanes load their inputs, or from order
// LANE_ROWS_NMIN on four row disks on the same chunk, whose scaled inputs it loads once,
// coalesced, and hands to the lanes through LDS (loaded lane by lane, n entries apart,
// they take 25 loads of 64 cache lines each at order 12).  Each pair is read as one
// lane-interleaved record (H_0, H_1, e^{i alpha_pq}, 2 / (k b_pq)): the orders H_nu(k b_pq), nu <= 2N, follow by
// the upward recurrence H_{nu+1} = (2 nu / x) H_nu - H_{nu-1}, whose rounding
// error stays at the level of eps |H_nu| (the growing Y part dominates |H_nu|
// wherever the J part decays), and the phase e^{i nu alpha} by recurrence;
// t_{+nu} = H_nu e^{i nu alpha}, t_{-nu} = (-1)^nu H_nu e^{-i nu alpha}.  The
// product runs diagonal by diagonal (w_m += t_s z_{m+s}) with the scaled
// inputs z in registers.  The 2n real outputs are summed over the lanes by a
// reduce-scatter butterfly (lane l ends with the sum of value l >> sh) and
// stored as the chunk's partial sum; k_apply_finish adds the chunks of each
// row in order; the two launches need no counters or memory fences.
// Bound by FP64 issue: 3,000 vector instructions per wave at N = 12, 2.7 waves per
// SIMD at 400 disks, so 3 rounds of 5.6 us.  us per apply, one row per workgroup and
// four: 400 x 12 28.2, 25.9; 700 67.9, 61.4; 1,000 120, 114; 400, 7 columns 139, 133; 48
// x 50, 4 columns 73.5, 69.7.  Below LANE_FEW_WAVES waves the hop through LDS would only
// lengthen the chain (solves, one and four rows, ms: 50 disks 9.6, 10.0; 100 disks 16.5, 16.7; 150 disks,
// 450 waves, 29.2, 29.1).
template <int N, bool OPC, int ROWS = LANE_ROWS>
__global__ __launch_bounds__(64 * ROWS, ROWS > 1 ? 2 : 1) void k_apply_lane(
    DevView v, int R, const cplx* __restrict__ x, cplx* __restrict__ part, int64_t part_total,
    const int32_t* __restrict__ items, const int32_t* __restrict__ active) {
  constexpr int n = 2 * N + 1, S = 2 * N;
  constexpr int NV = 2 * n <= 8 ? 8 : (2 * n <= 16 ? 16 : (2 * n <= 32 ? 32 : 64));
  constexpr int SH = NV == 8 ? 3 : (NV == 16 ? 2 : (NV == 32 ? 1 : 0));  // 6 - log2 NV
  __shared__ cplx zl[ROWS > 1 ? (LANE_CHUNK + 1) * n : 1];
  const int r = blockIdx.y, tid = threadIdx.x;
  const int32_t* itp = items + (int64_t)LANE_ITEM_INTS * blockIdx.x;
  const int p0 = itp[0], rows = itp[1], jb = itp[2], je = itp[3], b = itp[4];
  if (active && active[b * R + r] == 0) return;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t d0 = itp[5];
  const int64_t i0 = *reinterpret_cast<const int64_t*>(itp + 6);
  const int64_t cb = (int64_t)R * i0 + (int64_t)r * *reinterpret_cast<const int64_t*>(itp + 8);
  const int p = p0 + wv, j = jb + lane;
  const int64_t recb = *reinterpret_cast<const int64_t*>(itp + 10);
  const int64_t pb = *reinterpret_cast<const int64_t*>(itp + 12);
  cplx acc[n];
  // the sums of a lane's pair: h0, H: H_0, H_1; E: e^{i alpha}; r2: 2 / (k b); z: its inputs
  auto pair = [&](cplx h0, cplx H, cplx E, double r2, const cplx (&z)[n]) {
#pragma unroll
    for (int m = 0; m < n; ++m) cmac(acc[m], h0, z[m]);
    cplx Hm = h0;
    cplx P = E;
#pragma unroll
    for (int nu = 1; nu <= S; ++nu) {
      if (nu > 1) {
        const cplx Hn = csub(cscale(H, (nu - 1) * r2), Hm);  // H_nu from H_{nu-1}, H_{nu-2}
        Hm = H;
        H = Hn;
        P = cmul(P, E);
      }
      const cplx tp = cmul(H, P);
      cplx tm = cmul(H, cconj(P));
      if (nu & 1) tm = cmk(-tm.x, -tm.y);
#pragma unroll
      for (int m = 0; m < n - nu; ++m) cmac(acc[m], tp, z[m + nu]);
#pragma unroll
      for (int m = nu; m < n; ++m) cmac(acc[m], tm, z[m - nu]);
    }
  };
  int64_t rowp = 0;  // this row's partial sums after the first row's
  if constexpr (ROWS > 1) {
    // records and partial sums of consecutive rows lie at a fixed distance, by the chunks of a row
    const int chunks = (*reinterpret_cast<const int32_t*>(itp + 8) / n - 1 + LANE_CHUNK - 1) / LANE_CHUNK;
    rowp = (int64_t)wv * chunks * n;
    // at least LANE_MIN lanes work, those past the last column on its record and zeros: waves of
    // 2 to 8 active lanes run half as fast (200 disks, whose last chunk has 7: 19 us, 11 so)
    const bool live = wv < rows && lane < max(je - jb, LANE_MIN);
    cplx h0, H, E;
    double r2 = 0.0;
    if (live) {
      const cplx* __restrict__ rec =
          v.lt + recb + (int64_t)wv * chunks * (LANE_CHUNK * LANE_REC) + min(lane, je - jb - 1);
      h0 = rec[0];
      H = rec[LANE_CHUNK];
      E = rec[2 * LANE_CHUNK];
      r2 = rec[3 * LANE_CHUNK].x;
    }
    // column disks jb .. je of the instance (those of a row skip the row itself), scaled
    const int64_t e0 = (int64_t)jb * n;
    const int ne = (je - jb + 1) * n;
    constexpr int NE = ((LANE_CHUNK + 1) * n + 64 * ROWS - 1) / (64 * ROWS);
    cplx xe[NE], fe[OPC ? NE : 1];
    double se[OPC ? 1 : NE];
#pragma unroll
    for (int u = 0; u < NE; ++u) {  // every load in flight before the first is used
      const int64_t e = e0 + min(tid + u * 64 * ROWS, ne - 1);
      xe[u] = x[cb + e];
      if constexpr (OPC) fe[u] = v.op_col[i0 + e];
      else se[u] = v.sJ[i0 + e];
    }
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int e = tid + u * 64 * ROWS;
      cplx z;
      if constexpr (OPC) z = cmul(xe[u], fe[u]);
      else z = cscale(xe[u], se[u]);
      if (e < ne) zl[e] = z;
      else if (e < (LANE_MIN + 1) * n) zl[e] = cmk(0.0, 0.0);
    }
    __syncthreads();
    if (wv >= rows) return;
#pragma unroll
    for (int m = 0; m < n; ++m) acc[m] = cmk(0.0, 0.0);
    if (live) {
      const int jl = lane + (d0 + j >= p ? 1 : 0);
      cplx z[n];
#pragma unroll
      for (int k = 0; k < n; ++k) z[k] = zl[jl * n + k];
      pair(h0, H, E, r2, z);
    }
  } else {
#pragma unroll
    for (int m = 0; m < n; ++m) acc[m] = cmk(0.0, 0.0);
    if (j < je) {
      const cplx* __restrict__ rec = v.lt + recb + lane;
      const int64_t iq = (int64_t)(j + (d0 + j >= p ? 1 : 0)) * n;
      const cplx h0 = rec[0], H = rec[LANE_CHUNK], E = rec[2 * LANE_CHUNK];
      const double r2 = rec[3 * LANE_CHUNK].x;
      cplx z[n];
#pragma unroll
      for (int k = 0; k < n; ++k)
        z[k] = OPC ? cmul(x[cb + iq + k], v.op_col[i0 + iq + k]) : cscale(x[cb + iq + k], v.sJ[i0 + iq + k]);
      pair(h0, H, E, r2, z);
    }
  }
  double val[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) val[k] = k < 2 * n ? ((k & 1) ? acc[k >> 1].y : acc[k >> 1].x) : 0.0;
  lane_reduce_scatter<NV>(val, lane);
  const int vi = lane >> SH;
  if ((lane & ((1 << SH) - 1)) == 0 && vi < 2 * n) {
    double* pr = reinterpret_cast<double*>(part + (int64_t)r * part_total + pb + rowp);
    pr[vi] = val[0];
  }
}

// ------------------------------------------------------------------ one lane per pair, any orders
// Few right-hand sides on a batch whose orders differ (or exceed LANE_NMAX), N_p
// <= PAIRS_NMAX (pairs_batch).  As in k_apply_lane a lane works on one ordered
// pair and builds its symbols from the pair's 64-byte record by the recurrences
// of H_nu and e^{i nu alpha}, so no symbol row is read; but a wave takes a block
// of consecutive outputs m of its row disk, so that outputs and inputs fit the
// registers at any order: step nu moves a window z_{m+-nu} of the block's inputs
// by one mode (one new entry from the panel [n][column disk] of the workgroup's
// 64 column disks in LDS) and adds t_{+-nu} times the window.  The column disks
// are ordered by decreasing N, so that the lanes of a wave walk about the same
// number of modes.  A workgroup scales and stages its panel once, then its waves
// take (row disk, block) tasks from a counter in LDS until none is left: no
// barrier, no fence and no uneven rows inside.
// Bound by FP64 issue: a step costs 4 multiply-adds per output plus 12 for the
// recurrences and the symbol, and the window's ends add BT - 1 idle columns, so
// blocks are as wide as the registers allow: up to 14 outputs at two waves per
// SIMD, or 8 at three where the launch has too few tasks to fill the chip.
// 1,000 disks of N_p 13..20, one right-hand side (9.9 GFLOP): 3,480 us with the
// LDS-staged kernel (each multiply-add read 1.25 LDS values, rows ended in
// agent-scope fences), 368 us with 8 outputs, 352 us with 14 (28 TFLOP/s, vector
// units busy 77% at the 2.0 GHz that this load runs at).
#define PAIRS_ITEM_INTS 8
#define PAIRS_THREADS 256
#define PAIRS_BT_NARROW 8
#define PAIRS_BT_WIDE 14
#define PAIRS_LD 65  // LDS row stride (complex): consecutive modes of a disk in different banks

// One direction of the block's sums: steps nu = 1..top of acc_i += t_{+-nu}
// z_{m0+i+-nu}, t_{+-nu} = H_nu E^nu with E = e^{i alpha} upward and -e^{-i alpha}
// downward.  The window w is a ring: after step nu entry i sits in slot
// (i + nu) mod BT (upward) or (i - nu) mod BT.
template <int BT, bool UP, class Z>
__device__ __forceinline__ void pairs_walk(cplx (&acc)[BT], cplx (&w)[BT], const Z& zat, int m0, int top,
                                           cplx Hm, cplx H, cplx E, double r2) {
  cplx P = E;
  double nf = 1.0;
  for (int nb = 0; nb < top; nb += BT) {
#pragma unroll
    for (int k = 1; k <= BT; ++k) {
      const int nu = nb + k;
      if (nu > top) return;
      w[UP ? (k - 1) % BT : (BT - k) % BT] = zat(UP ? m0 + BT - 1 + nu : m0 - nu);
      const cplx t = cmul(H, P);
#pragma unroll
      for (int i = 0; i < BT; ++i) cmac(acc[i], t, w[(UP ? i + k : i + BT - k) % BT]);
      const double c = nf * r2;
      const cplx Hn = cmk(fma(H.x, c, -Hm.x), fma(H.y, c, -Hm.y));
      Hm = H;
      H = Hn;
      P = cmul(P, E);
      nf += 1.0;
    }
  }
}

// One task: outputs m0 .. m0 + nval - 1 of a row disk, summed over the wave's
// pairs, into pr (real and imaginary parts in turn), added to it unless `first`.
template <int BT>
__device__ __forceinline__ void pairs_block(const cplx* zl, int Nm, int lane, bool ok, int m0, int nval,
                                            const cplx* __restrict__ rec, double* pr, bool first) {
  constexpr int NV = 2 * BT <= 16 ? 16 : 32;
  constexpr int SH = NV == 16 ? 2 : 1;  // 6 - log2 NV
  cplx acc[BT];
#pragma unroll
  for (int i = 0; i < BT; ++i) acc[i] = cmk(0.0, 0.0);
  if (ok) {
    // z_n of this lane's disk; modes beyond the panel read its last row, zeros (n is wave-uniform)
    const unsigned last = 2 * Nm + 1;
    auto zat = [&](int n) { return zl[min((unsigned)(n + Nm), last) * PAIRS_LD + lane]; };
    const cplx h0 = rec[0], h1 = rec[LANE_CHUNK], e = rec[2 * LANE_CHUNK];
    const double r2 = rec[3 * LANE_CHUNK].x;
    cplx w[BT];
#pragma unroll
    for (int i = 0; i < BT; ++i) {
      w[i] = zat(m0 + i);
      cmac(acc[i], h0, w[i]);
    }
    pairs_walk<BT, true>(acc, w, zat, m0, Nm - m0, h0, h1, e, r2);
#pragma unroll
    for (int i = 0; i < BT; ++i) w[i] = zat(m0 + i);
    pairs_walk<BT, false>(acc, w, zat, m0, m0 + nval - 1 + Nm, h0, h1, cmk(-e.x, e.y), r2);
  }
  double val[NV];
#pragma unroll
  for (int i = 0; i < NV / 2; ++i) {
    val[2 * i] = i < BT ? acc[i < BT ? i : 0].x : 0.0;
    val[2 * i + 1] = i < BT ? acc[i < BT ? i : 0].y : 0.0;
  }
  lane_reduce_scatter<NV>(val, lane);
  const int vi = lane >> SH;
  if ((lane & ((1 << SH) - 1)) == 0 && vi < 2 * nval) pr[vi] = first ? val[0] : pr[vi] + val[0];
}

// Item: instance, first chunk of 64 column disks, chunks, tasks [t0, t1), first
// disk, partial-sum segment, disks of the instance.
template <bool WIDE>
__global__ __launch_bounds__(PAIRS_THREADS, WIDE ? 2 : 3) void k_apply_pairs(
    DevView v, int R, const cplx* __restrict__ x, cplx* __restrict__ part, int64_t part_total,
    const int32_t* __restrict__ items, const int32_t* __restrict__ tasks,
    const int64_t* __restrict__ partoff, const int32_t* __restrict__ active) {
  extern __shared__ cplx lds[];  // [2 Nm + 2][PAIRS_LD], the last row zeros
  __shared__ int s_next;
  const int r = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int32_t* it = items + (int64_t)PAIRS_ITEM_INTS * blockIdx.x;
  const int b = it[0], c0 = it[1], nc = it[2], t0 = it[3], t1 = it[4], seg = it[6], Mb = it[7];
  const int64_t d0 = it[5];
  if (active && active[b * R + r] == 0) return;
  const int64_t i0 = v.imode[b];
  const cplx* __restrict__ xc = x + col_base(v.imode, b, R, r);
  for (int c = c0; c < c0 + nc; ++c) {
    const int cnt = min(LANE_CHUNK, Mb - LANE_CHUNK * c);
    const int32_t* __restrict__ ord = v.lord + d0 + (int64_t)LANE_CHUNK * c;
    const int Nm = v.N[ord[0]], rows = 2 * Nm + 1;
    __syncthreads();  // the previous chunk's panel is no longer read
    if (tid == 0) s_next = t0;
    for (int e = tid; e < cnt * rows; e += PAIRS_THREADS) {
      const int k = e / rows, n = e - (e / rows) * rows;  // modes of a disk: coalesced
      const int q = ord[k];
      const int Nq = v.N[q], u = n - Nm + Nq;
      cplx z = cmk(0.0, 0.0);
      if (u >= 0 && u <= 2 * Nq) {
        const int64_t iq = v.moff[q] + u;
        z = col_scale(v, i0 + iq, xc[iq]);
      }
      lds[n * PAIRS_LD + k] = z;
    }
    if (tid < LANE_CHUNK) lds[rows * PAIRS_LD + tid] = cmk(0.0, 0.0);
    __syncthreads();
    const int q = lane < cnt ? ord[lane] : -1;
    for (;;) {
      int t = 0;
      if (lane == 0) t = atomicAdd(&s_next, 1);
      t = __builtin_amdgcn_readfirstlane(t);
      if (t >= t1) break;
      const int p = tasks[2 * t], ms = tasks[2 * t + 1] >> 8, bt = tasks[2 * t + 1] & 255;
      const int Np = v.N[p], np = 2 * Np + 1;
      const int nval = min(bt, np - ms);
      const bool ok = q >= 0 && q != p;
      const cplx* __restrict__ rec = v.lt + v.ltoff[p] + (int64_t)c * (LANE_CHUNK * LANE_REC) + lane;
      double* pr = reinterpret_cast<double*>(part + (int64_t)r * part_total + partoff[p] +
                                             (int64_t)seg * np + ms);
      const int m0 = ms - Np;
      const bool first = c == c0;
      // widths of pairs_width
#define PAIRS_CASE(W) case W: pairs_block<W>(lds, Nm, lane, ok, m0, nval, rec, pr, first); break;
      if constexpr (WIDE) {
        switch (bt) {
          PAIRS_CASE(7) PAIRS_CASE(8) PAIRS_CASE(9) PAIRS_CASE(10) PAIRS_CASE(11) PAIRS_CASE(12) PAIRS_CASE(13)
          default: pairs_block<PAIRS_BT_WIDE>(lds, Nm, lane, ok, m0, nval, rec, pr, first); break;
        }
      } else {
        switch (bt) {
          PAIRS_CASE(5) PAIRS_CASE(6) PAIRS_CASE(7)
          default: pairs_block<PAIRS_BT_NARROW>(lds, Nm, lane, ok, m0, nval, rec, pr, first); break;
        }
      }
#undef PAIRS_CASE
    }
  }
}

// y = finalize(sum over the chunks of row p of the partial sums), one thread
// per output row, chunks added in order.
__global__ void k_apply_finish(DevView v, int R, const cplx* __restrict__ x, cplx* __restrict__ y,
                               int op, const cplx* __restrict__ part, int64_t part_total,
                               const int32_t* __restrict__ nchunk,
                               const int64_t* __restrict__ partoff,
                               const int32_t* __restrict__ active,
                               const cplx* __restrict__ shift) {
  const int64_t total = (int64_t)R * v.N_all;
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  // column (b, r) and unknown i of the packed row g
  int lo = 0, hi = v.B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)R * v.imode[mid] <= g) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int64_t Nb = v.imode[b + 1] - v.imode[b];
  const int64_t rem = g - (int64_t)R * v.imode[b];
  const int r = (int)(rem / Nb);
  if (active && active[b * R + r] == 0) return;
  const int64_t i = v.imode[b] + (rem - (int64_t)r * Nb);
  const cplx w = lane_chunk_sum(v, part + (int64_t)r * part_total, nchunk, partoff, b, i);
  cplx o = finalize(v, op, i, x[g], w);
  if (shift) o = affine(shift, b * R + r, o, x[g]);
  y[g] = o;
}

// ------------------------------------------------------------------ multi-RHS (MFMA)
// For R right-hand sides the block product T^{pq} Z^q (n_p x n_q times n_q x R)
// is a dense contraction: it runs on FP64 MFMA (v_mfma_f64_16x16x4f64,
// D[16x16] += A[16x4] B[4x16]).  A complex product is two real MFMAs: the B
// panel holds [Re Z | Im Z] for 8 right-hand sides side by side, so
//   acc1 = Re(T) [Re Z | Im Z],  acc2 = Im(T) [Re Z | Im Z],
//   Re W = acc1[:, :8] - acc2[:, 8:],  Im W = acc1[:, 8:] + acc2[:, :8].
// Lane layout (checked on the device): lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and D[4 v + l / 16][l % 16], v < 4.
//
// Work item: a group of rp <= RP row disks of one instance (disks of equal row
// tile count grouped together, so that the waves of a workgroup issue equal
// numbers of MFMAs between barriers), a tile of 8 CT right-hand sides and a
// segment [q0, q1) of its column disks.  Wave w of the workgroup computes row
// w / CT and right-hand-side sub-tile w % CT.  The input panel
// Z^q = sqrt(a_q) J_n(k a_q) x^q_n is formed once per apply for all columns
// (k_apply_mfma_scale); per column disk q its panel and the symbol rows of the
// item's row disks are staged in LDS once for all waves, and the next disk's
// values are gathered into registers while the current one is on the matrix
// cores.  The workgroups are persistent: each takes items from a queue
// (one atomic counter, items sorted by decreasing cost), so instances of very
// different sizes share one launch and the launch ends evenly.  Each item's
// sums go to its own partial block; k_apply_mfma_finish adds the segments of
// every row in order (no inter-workgroup synchronisation).  The tile shape
// (RP, CT), the segment length and the workgroup size are chosen per handle
// and R by timing the candidates on the real data (mfma_autotune).
typedef double mf_d4 __attribute__((ext_vector_type(4)));

#define MF_REC 7       // item record: row group, rp, tile, q0, q1, partial block, list flag

// Column of element (n, c) of the staged input panel [4 ktmax][RC] in LDS:
// c XOR a function of the row n, so that a staging store (consecutive rows, one
// column) spreads over 16 bank groups and an MFMA B read (rows n..n+3, eight
// columns) puts even and odd rows in different halves of the banks.
__device__ __forceinline__ int mf_zcol(int n, int c, int RC) {
  const int f = ((n & 1) << 3) | ((n >> 1) & 7);
  return c ^ (f & (RC >= 16 ? 15 : RC - 1));
}

// K row tiles of one wave against one staged column disk: KT k-steps of 4,
// two real MFMAs per tile and step (Re T, Im T against [Re Z | Im Z]); zl is
// the staged panel and zc this lane's panel column.
template <int K, int MT>
__device__ __forceinline__ void mf_tiles(const cplx* trow, const cplx* zl, int zc, int RC, int j,
                                         int kq, int KT, mf_d4* acc1, mf_d4* acc2) {
  for (int kk = 0; kk < KT; ++kk) {
    const int n = 4 * kk + kq;
    const cplx zz = zl[n * RC + mf_zcol(n, zc, RC)];
    const double bv = j < 8 ? zz.x : zz.y;
#pragma unroll
    for (int mt = 0; mt < K; ++mt) {
      const cplx t = trow[n - (16 * mt + j) + 16 * MT - 1];  // A[i = lane % 16][k = kq]
      acc1[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.x, bv, acc1[mt], 0, 0, 0);
      acc2[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.y, bv, acc2[mt], 0, 0, 0);
    }
  }
}

// MT row tiles of 16 (n_p <= 16 MT); ZK / TK staged input / symbol values per
// thread, sized on the host for the batch (4 ktmax RC <= ZK THREADS and
// RP TL <= TK THREADS), which keeps the register footprint of the staging to
// what the batch needs.
// An item with its list flag set takes its column disks from qlist[q0..q1):
// entry (q << 8) | mask, mask bit r set when row r of the item's group is a
// close pair with q (the circulant form covers the other pairs).
template <int MT, int THREADS, int ZK, int TK>
__global__ __launch_bounds__(THREADS) void k_apply_mfma(
    DevView v, int R, const cplx* __restrict__ x, const int32_t* __restrict__ active,
    const int32_t* __restrict__ items, int n_items, int32_t* __restrict__ head,
    cplx* __restrict__ part, int64_t blk, int npad, int ktmax, int RP, int CT,
    const int32_t* __restrict__ grow, const int32_t* __restrict__ qlist) {
  extern __shared__ cplx lds[];
  __shared__ int s_item;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int j = lane & 15, kq = lane >> 4;
  const int RC = 8 * CT;
  const int row = wave / CT, ctile = wave - (wave / CT) * CT;
  const int TL = 4 * ktmax + 16 * MT - 1;  // symbol row length in LDS
  const int zrows = 4 * ktmax;
  cplx* zl = lds;                          // [4 ktmax][RC]
  cplx* tl = lds + zrows * RC;             // [RP][TL]
  // this thread's staging slots: input panel element (column zc, row zn),
  // symbol element (row trr, position tru)
  int zc[ZK], zn[ZK], trr[TK], tru[TK];
#pragma unroll
  for (int k = 0; k < ZK; ++k) {
    const int e = tid + k * THREADS;
    zc[k] = e / zrows;
    zn[k] = e - zc[k] * zrows;
  }
#pragma unroll
  for (int k = 0; k < TK; ++k) {
    const int e = tid + k * THREADS;
    trr[k] = e / TL;
    tru[k] = e - trr[k] * TL;
  }
  for (;;) {
    __syncthreads();  // the previous item is done with s_item and LDS
    if (tid == 0) s_item = atomicAdd(head, 1);
    __syncthreads();
    const int it = s_item;
    if (it >= n_items) break;
    const int32_t* rec = items + (int64_t)MF_REC * it;
    const int rp = rec[1], tile = rec[2], qb = rec[3], qe = rec[4];
    const int32_t* __restrict__ ql = rec[6] ? qlist : nullptr;
    // column disk and row mask of list position i (qb <= i < qe)
    auto qat = [&](int i) { return ql ? (ql[i] >> 8) : i; };
    auto mat = [&](int i) { return ql ? (ql[i] & 0xff) : 0xff; };
    const int32_t* grp = grow + (int64_t)rec[0] * RP;  // the item's row disks
    const int64_t pb = rec[5];
    const int c0 = tile * RC;
    const int b = v.inst[grp[0]];
    bool any = false;  // converged columns: the whole tile may be skipped
    for (int r = c0; r < min(R, c0 + RC); ++r)
      if (!active || active[b * R + r]) any = true;
    if (!any) continue;
    const int64_t i0 = v.imode[b];
    const bool row_ok = row < rp;
    const int p = row_ok ? grp[row] : -1;
    const int mtp = row_ok ? (2 * v.N[p] + 1 + 15) >> 4 : 0;  // row tiles of this row disk
    bool wave_active = row_ok;
    if (wave_active) {
      wave_active = false;
      for (int c = 0; c < 8; ++c) {
        const int r = c0 + ctile * 8 + c;
        if (r < R && (!active || active[b * R + r])) wave_active = true;
      }
    }
    mf_d4 acc1[MT], acc2[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      acc1[t] = mf_d4{0.0, 0.0, 0.0, 0.0};
      acc2[t] = mf_d4{0.0, 0.0, 0.0, 0.0};
    }
    // Gathered values of the next column disk, loaded while the current one is
    // on the matrix cores: nothing in the gather consumes a load (the input
    // arrives scaled by its column factor, the symbol sign is applied when
    // staging), so the gather does not hold up the MFMAs behind it.  N and the
    // mode offset of the disks are read one disk ahead of their gather, N of
    // the item's row disks once.
    cplx zr[ZK], tr[TK];
    double tsg[TK];
    int32_t tof[TK];  // symbol offsets (the MFMA path requires T_all < 2^31)
    int npr[TK], prw[TK];  // N and index of this thread's symbol-row disks
#pragma unroll
    for (int k = 0; k < TK; ++k) {
      prw[k] = trr[k] < rp ? grp[trr[k]] : -1;
      npr[k] = prw[k] >= 0 ? v.N[prw[k]] : 0;
    }
    auto gather = [&](int q, int qmask, int Nq, int64_t mq) {
      const int nq = 2 * Nq + 1;
#pragma unroll
      for (int k = 0; k < ZK; ++k) {
        const int c = zc[k], n = zn[k];
        cplx z = cmk(0.0, 0.0);
        if (c < RC && n < nq && c0 + c < R) z = x[col_base(v.imode, b, R, c0 + c) + mq + n];
        zr[k] = z;
      }
#pragma unroll
      for (int k = 0; k < TK; ++k) {
        const int rr = trr[k], u = tru[k];
        cplx t = cmk(0.0, 0.0);
        double sg = 1.0;
        const int pr = prw[k];
        if (rr < rp && pr != q && ((qmask >> rr) & 1)) {
          const int Npr = npr[k];
          const int S = Npr + Nq;
          const int s = u - (16 * MT - 1) - Nq + Npr;
          if (s >= -S && s <= S) {
            t = v.t[tof[k] + S + s];
            if (pr > q && (s & 1)) sg = -1.0;
          }
        }
        tr[k] = t;
        tsg[k] = sg;
      }
    };
    // symbol-row offsets of column disk q, loaded one disk ahead of gather(q)
    // so that gathering the symbols is a single dependent load
    auto load_toff = [&](int q, int qmask) {
#pragma unroll
      for (int k = 0; k < TK; ++k) {
        const int pr = prw[k];
        tof[k] = (q >= 0 && trr[k] < rp && pr != q && ((qmask >> trr[k]) & 1))
                     ? (int32_t)v.toff[pair_index(v.idisk, v.ipair, b, pr, q)] : 0;
      }
    };
    // disk, row mask, N and mode offset of list positions i (0), i + 1 (1)
    // and i + 2 (2)
    int qd0 = -1, qd1 = -1, qd2 = -1, qm0 = 0, qm1 = 0, qm2 = 0;
    int Nq0 = 0, Nq1 = 0, Nq2 = 0;
    int64_t mq0 = 0, mq1 = 0, mq2 = 0;
    if (qb < qe) {
      qd0 = qat(qb);
      qm0 = mat(qb);
      Nq0 = v.N[qd0];
      mq0 = v.moff[qd0];
    }
    if (qb + 1 < qe) {
      qd1 = qat(qb + 1);
      qm1 = mat(qb + 1);
      Nq1 = v.N[qd1];
      mq1 = v.moff[qd1];
    }
    if (qb < qe) {
      load_toff(qd0, qm0);
      gather(qd0, qm0, Nq0, mq0);
      load_toff(qd1, qm1);
    }
    for (int qi = qb; qi < qe; ++qi) {
      const int q = qd0;
      const int nq = 2 * Nq0 + 1, KT = (nq + 3) >> 2;
      __syncthreads();  // previous column disk done with LDS
#pragma unroll
      for (int k = 0; k < ZK; ++k)
        if (zc[k] < RC) zl[zn[k] * RC + mf_zcol(zn[k], zc[k], RC)] = zr[k];
#pragma unroll
      for (int k = 0; k < TK; ++k)
        if (trr[k] < RP) tl[trr[k] * TL + tru[k]] = cscale(tr[k], tsg[k]);
      __syncthreads();
      qd2 = -1;
      qm2 = 0;
      if (qi + 2 < qe) {  // used by the next iteration's gather
        qd2 = qat(qi + 2);
        qm2 = mat(qi + 2);
        Nq2 = v.N[qd2];
        mq2 = v.moff[qd2];
      }
      if (qi + 1 < qe) {  // in flight during the MFMAs
        gather(qd1, qm1, Nq1, mq1);
        load_toff(qd2, qm2);
      }
      if (wave_active && q != p && ((qm0 >> row) & 1)) {
        const cplx* trow = tl + row * TL;
        const int zcl = ctile * 8 + (j & 7);
        // only the row tiles of this row disk (wave-uniform count)
        if (mtp >= MT) mf_tiles<MT, MT>(trow, zl, zcl, RC, j, kq, KT, acc1, acc2);
        else if constexpr (MT >= 2) {
          if (mtp == MT - 1) mf_tiles<MT - 1, MT>(trow, zl, zcl, RC, j, kq, KT, acc1, acc2);
          else if constexpr (MT >= 3) {
            if (mtp == MT - 2) mf_tiles<MT - 2, MT>(trow, zl, zcl, RC, j, kq, KT, acc1, acc2);
            else if constexpr (MT >= 4) mf_tiles<MT - 3, MT>(trow, zl, zcl, RC, j, kq, KT, acc1, acc2);
          }
        }
      }
      qd0 = qd1;
      qm0 = qm1;
      Nq0 = Nq1;
      mq0 = mq1;
      qd1 = qd2;
      qm1 = qm2;
      Nq1 = Nq2;
      mq1 = mq2;
    }
    if (!wave_active) continue;
    // partial block [RP][npad][RC]: row r of the item, mode row m, RHS column
    cplx* pbk = part + pb * blk + (int64_t)row * npad * RC + ctile * 8 + (j & 7);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int vv = 0; vv < 4; ++vv) {
        const double a1 = acc1[mt][vv], a2 = acc2[mt][vv];
        const double other = __shfl_xor(a2, 8, 64);
        const double val = j < 8 ? a1 - other : a1 + other;  // Re W (j < 8), Im W (j >= 8)
        const double im = __shfl_xor(val, 8, 64);
        const int m = 16 * mt + 4 * vv + kq;  // D row 4 v + lane / 16
        if (j < 8) pbk[(int64_t)m * RC] = cmk(val, im);
      }
    }
  }
}

#define CLOSE_LONG 8
// The close pairs e0, e0 + step, .. < e1 of one row disk: NT row tiles (of MTW
// accumulators), no branch between the loads of a step.
template <int NT, int MTW, bool OPC>
__device__ __forceinline__ void close_walk(const DevView& v, const cplx* __restrict__ xc, int64_t i0,
                                           const int4* __restrict__ crec, int e0, int e1, int step, int Np,
                                           int top, int j, int kq, mf_d4 (&acc1)[MTW], mf_d4 (&acc2)[MTW]) {
  int4 rec = crec[min(e0, e1 - 1)];
  for (int e = e0; e < e1; e += step) {
    const int4 cur = rec;
    rec = crec[min(e + step, e1 - 1)];
    const int Nq = cur.y, nq_ = 2 * Nq + 1, S = Np + Nq, KT = (nq_ + 3) >> 2;
    const cplx* __restrict__ trow = v.t + cur.z + S;
    const cplx* __restrict__ zq = xc + cur.x;
    const double* __restrict__ sq = v.sJ + i0 + cur.x;
    const cplx* __restrict__ oq = v.op_col + i0 + cur.x;
#pragma unroll 4
    for (int kt = 0; kt < KT; ++kt) {
      const int n = 4 * kt + kq, nc = min(n, nq_ - 1);
      const cplx zz = OPC ? cmul(zq[nc], oq[nc]) : cscale(zq[nc], sq[nc]);
      const double bv = n < nq_ ? (j < 8 ? zz.x : zz.y) : 0.0;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        // rows past n_p read some symbol of the row (their sums are never read)
        const int sv = max(-S, (nc - Nq) - (top + 16 * i));
        cplx a = trow[sv];
        if (cur.w & sv & 1) a = cmk(-a.x, -a.y);  // t^{pq}_s = (-1)^s t^{qp}_s
        acc1[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, bv, acc1[i], 0, 0, 0);
        acc2[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, bv, acc2[i], 0, 0, 0);
      }
    }
  }
}

// Close pairs of the instances in the circulant form with 8-column tiles: a wave
// takes (row disk p, tile of 8 columns, MTW row tiles) and walks p's close pairs;
// per column disk q and k step it loads the input panel element of its lane
// (B[k][j]: Re or Im of column j & 7 at mode 4 kt + k, times its column factor) and
// per row tile the symbol value of its lane (A[i][k]: t_{(n - N_q) - (m - N_p)},
// m = 16 mt + i), straight into the operand layout of v_mfma_f64_16x16x4f64 (two
// MFMAs per complex product, as k_apply_mfma), no LDS.  The row's sums stay in
// registers and go to segment 0 of its group, which the output pass adds; rows
// without close pairs are not launched (ROW_EMPTY).
// Bound by load latency: a record per pair (read one ahead) names everything its
// loads need, four k steps of loads are issued together, and lists longer than
// CLOSE_LONG are split over the four waves of a workgroup, whose sums meet in LDS,
// so that one long list does not outlast the launch.  Registers for the loads in
// flight count for more than waves: four waves per SIMD and four steps, against
// eight waves and one step 78 and 91 us on 48 unequal instances of up to 200 disks
// with 8 columns, 179 and 207 us on 1,000 disks with 256 (one wave per list, loads
// behind branches, offsets looked up per pair: 293 and 183 us); a branch on the kind
// of column factor between the loads costs as much again (121 and 248).
template <int MT, int MTW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_apply_close(
    DevView v, int R, const cplx* __restrict__ x, cplx* __restrict__ part, int64_t blk, int npad,
    const int32_t* __restrict__ dgrp, const int32_t* __restrict__ drow,
    const int64_t* __restrict__ gbase, const int4* __restrict__ crow, const int4* __restrict__ crec,
    int n_rows, int n_long, int ntile, const int32_t* __restrict__ active) {
  constexpr int ZG = (MT + MTW - 1) / MTW;  // waves per (row disk, tile): groups of row tiles
  __shared__ double sums[3][MTW * 8][64];
  const int wave = (int)threadIdx.x >> 6, lane = threadIdx.x & 63;
  // Block -> rows and waves (t, zi) of them.  Consecutive blocks are different rows
  // and the row counts are padded to a multiple of 8, so that all tiles of a row run
  // on one XCD and meet its symbols in that L2.  Long lists: one (t, zi) a block;
  // short ones: a block takes wpr = 1, 2 or 4 consecutive (t, zi) of 4 / wpr rows.
  const int per = ntile * ZG, nlp = (n_long + 7) & ~7;
  const bool split = (int)blockIdx.x < nlp * per;  // block-uniform
  int i, tz;
  if (split) {
    i = (int)blockIdx.x % nlp;
    tz = (int)blockIdx.x / nlp;
    if (i >= n_long) return;
  } else {
    const int wpr = per >= 4 ? 4 : per, rpb = 4 / wpr;
    const int nrb = ((n_rows - n_long + rpb - 1) / rpb + 7) & ~7;
    const int k = (int)blockIdx.x - nlp * per;
    i = n_long + (k % nrb) * rpb + wave / wpr;
    tz = (k / nrb) * wpr + wave % wpr;
    if (i >= n_rows || tz >= per || wave >= rpb * wpr) return;
  }
  const int zi = tz % ZG, t = tz / ZG;
  const int4 rw = crow[i];
  const int p = rw.x, mt0 = MTW * zi, c0 = 8 * t;
  const int b = v.inst[p];
  const int Np = v.N[p], np_ = 2 * Np + 1, mtp = (np_ + 15) >> 4;
  if (mt0 >= mtp) return;  // no mode of p in these row tiles
  if (active) {
    bool any = false;
    for (int r = c0; r < min(R, c0 + 8); ++r) any |= active[b * R + r] != 0;
    if (!any) return;
  }
  const int j = lane & 15, kq = lane >> 4;
  mf_d4 acc1[MTW], acc2[MTW];
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
    acc1[i] = mf_d4{0.0, 0.0, 0.0, 0.0};
    acc2[i] = mf_d4{0.0, 0.0, 0.0, 0.0};
  }
  // columns past R read column c0 (their sums are never read)
  const int col = c0 + (j & 7) < R ? c0 + (j & 7) : c0;
  const cplx* __restrict__ xc = x + col_base(v.imode, b, R, col);
  const int e0 = rw.y + (split ? wave : 0), step = split ? 4 : 1;
  const int top = 16 * mt0 + j - Np;  // first mode of this lane's rows
  if (MTW == 1 || mt0 + 1 >= mtp) {
    if (v.op_col) close_walk<1, MTW, true>(v, xc, v.imode[b], crec, e0, rw.z, step, Np, top, j, kq, acc1, acc2);
    else close_walk<1, MTW, false>(v, xc, v.imode[b], crec, e0, rw.z, step, Np, top, j, kq, acc1, acc2);
  } else {
    if (v.op_col) close_walk<MTW, MTW, true>(v, xc, v.imode[b], crec, e0, rw.z, step, Np, top, j, kq, acc1, acc2);
    else close_walk<MTW, MTW, false>(v, xc, v.imode[b], crec, e0, rw.z, step, Np, top, j, kq, acc1, acc2);
  }
  if (split) {
    if (wave > 0) {
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          sums[wave - 1][8 * i + q][lane] = acc1[i][q];
          sums[wave - 1][8 * i + 4 + q][lane] = acc2[i][q];
        }
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc1[i][q] += sums[w][8 * i + q][lane];
          acc2[i][q] += sums[w][8 * i + 4 + q][lane];
        }
  }
  // segment 0 of the group's tile t: [RP][npad][8]
  cplx* pbk = part + (gbase[dgrp[p]] + t) * blk + (int64_t)drow[p] * npad * 8 + (j & 7);
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
#pragma unroll
    for (int vv = 0; vv < 4; ++vv) {
      const double a1 = acc1[i][vv], a2 = acc2[i][vv];
      const double other = __shfl_xor(a2, 8, 64);
      const double val = j < 8 ? a1 - other : a1 + other;  // Re W (j < 8), Im W (j >= 8)
      const double im = __shfl_xor(val, 8, 64);
      const int m = 16 * (mt0 + i) + 4 * vv + kq;
      if (j < 8 && m < np_) pbk[(int64_t)m * 8] = cmk(val, im);
    }
  }
}

// z = x scaled by the column factor of its unknown (sqrt(a) J_n, or the
// operator's column table), once per apply: the MFMA gathers then load one
// value per panel element.  With `skip`, only the instances not marked in it (the
// others have no work-queue items).
__global__ void k_apply_mfma_scale(DevView v, int R, const cplx* __restrict__ x, cplx* __restrict__ z,
                                   const int32_t* __restrict__ active, const int32_t* __restrict__ skip) {
  // blockIdx.x: column (b, r); blockIdx.y: 256-unknown slice of that column
  const int col = blockIdx.x, b = col / R;
  if (active && active[col] == 0) return;  // columns that no longer iterate
  if (skip && skip[b]) return;
  const int64_t Nb = v.imode[b + 1] - v.imode[b];
  const int64_t k = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (k >= Nb) return;
  const int64_t g = (int64_t)R * v.imode[b] + (int64_t)(col - b * R) * Nb + k;
  z[g] = col_scale(v, v.imode[b] + k, x[g]);
}

// y = finalize(sum over the segments of the MFMA partial blocks), one thread
// per output row, segments added in order.
__global__ void k_apply_mfma_finish(DevView v, int R, const cplx* __restrict__ x,
                                    cplx* __restrict__ y, int op, const cplx* __restrict__ part,
                                    int64_t blk, int npad, int RC, const int32_t* __restrict__ dgrp,
                                    const int32_t* __restrict__ drow,
                                    const int32_t* __restrict__ gnseg,
                                    const int64_t* __restrict__ gbase,
                                    const int32_t* __restrict__ active,
                                    const cplx* __restrict__ wh,
                                    const int32_t* __restrict__ con,
                                    const cplx* __restrict__ shift) {
  const int64_t total = (int64_t)R * v.N_all;
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  int lo = 0, hi = v.B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)R * v.imode[mid] <= g) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int64_t Nb = v.imode[b + 1] - v.imode[b];
  const int64_t rem = g - (int64_t)R * v.imode[b];
  const int r = (int)(rem / Nb);
  if (active && active[b * R + r] == 0) return;
  const int64_t i = v.imode[b] + (rem - (int64_t)r * Nb);
  const int p = v.udisk[i];
  const int64_t m = i - v.imode[b] - v.moff[p];
  const int gr = dgrp[p];
  const int t = r / RC, rc = r - (r / RC) * RC;
  const int ns = gnseg[gr], nsr = drow[p] & ROW_EMPTY ? 0 : ns;
  const cplx* pr = part + (gbase[gr] + (int64_t)t * ns) * blk +
                   ((int64_t)(drow[p] & (ROW_EMPTY - 1)) * npad + m) * RC + rc;
  cplx w = cmk(0.0, 0.0);
  for (int s = 0; s < nsr; ++s) w = cadd(w, pr[(int64_t)s * blk]);
  if (wh && con[b]) {  // well-separated pairs: w_j += sum_f w^{f j} W_f[p][r]
    const int Lb = v.cL[b];
    const int64_t d0 = v.idisk[b], Mb = v.idisk[b + 1] - d0;
    const cplx* __restrict__ wf = wh + (int64_t)R * v.cZo[b] + (p - d0) * R + r;
    const cplx* __restrict__ tw = v.ctw + v.cWo[b];
    const int jm = (int)m;
    int idx = 0;
    cplx acc = cmk(0.0, 0.0);
    for (int f = 0; f < Lb; ++f) {
      cmac(acc, tw[idx], wf[(int64_t)f * Mb * R]);
      idx += jm;
      if (idx >= Lb) idx -= Lb;
    }
    w = cadd(w, acc);
  }
  cplx o = finalize(v, op, i, x[g], w);
  if (shift) o = affine(shift, b * R + r, o, x[g]);
  y[g] = o;
}

// R at and above which the MFMA kernel applies the operator (N_p <= 31).
#define MFMA_MIN_R 8
// Column-disk segment length once few columns are still iterating: short
// segments spread a large straggler instance over many workgroups.
#define MFMA_TAIL_QS 16

static bool use_mfma(const mudiff_ctx* h, int R) {
  return R >= MFMA_MIN_R && h->Nmax <= 31 && h->mfma_enabled && h->T_all < ((int64_t)1 << 31);
}

int circ_variant(int R);
std::vector<int> circ_variants(int R);
std::vector<int> circ_timed(int R);
void circ_tile(int var, int* bm, int* bn);
void circ_var_dims(int var, int* bm, int* bn, int* bk, int* db, int* nt, int* mult);
int circ_finish(mudiff_ctx* h, int R, const cplx* x, cplx* y, int op, const cplx* part, int64_t blk,
                int npad, int RC, const int32_t* dgrp, const int32_t* drow, const int32_t* gnseg,
                const int64_t* gbase, const int32_t* active, const cplx* wh, const int32_t* con,
                const int32_t* con_h, const cplx* shift, hipStream_t s);
int circ_launch(mudiff_ctx* h, int R, const cplx* x, cplx* zh, cplx* wh, const int32_t* citems,
                int n_citems, int var, const int32_t* con, const int32_t* con_h,
                const int32_t* active, hipStream_t s);

static int segment(const mudiff_ctx* h, int R, const MfmaChoice& c);

// Host schedule of the MFMA apply for one tile choice.  With c.circ, the
// instances marked circ_on keep only their close pairs in the MFMA items
// (column lists) and get per-frequency product items instead.
static void mfma_build(const mudiff_ctx* h, int R, const MfmaChoice& c, MfmaSched& S,
                       const std::vector<int32_t>& cols = {}) {
  S.R = R;
  S.c = c;
  S.dev = nullptr;
  S.resident = false;
  const int RC = 8 * c.CT, QS = segment(h, R, c);
  S.ntile = (R + RC - 1) / RC;
  const int mt = (2 * h->Nmax + 1 + 15) / 16;
  S.npad = 16 * mt;
  S.blk = (int64_t)c.RP * S.npad * RC;
  S.items.clear();
  S.grow.clear();
  S.gnseg.clear();
  S.gbase.clear();
  S.qlist.clear();
  S.citems.clear();
  S.crow.clear();
  S.crec.clear();
  S.n_long = 0;
  S.close_rows = c.circ && h->circ && c.CT == 1;
  S.con.assign(h->B, 0);
  S.dgrp.assign(h->M_all, 0);
  S.drow.assign(h->M_all, 0);
  S.cvar = c.cvar >= 0 ? c.cvar : circ_variant(R);
  int cbm = 0, cbn = 0;
  circ_tile(S.cvar, &cbm, &cbn);
  struct It {
    double cost;
    int32_t r[MF_REC];
  };
  std::vector<It> its;
  auto tile_runs = [&](int b, int r0, int r1) {  // straggler schedule: a running column in [r0, r1)
    if (cols.empty()) return true;
    for (int r = r0; r < std::min(R, r1); ++r)
      if (cols[(size_t)b * R + r] != 0) return true;
    return false;
  };
  int64_t pb = 0;
  for (int b = 0; b < h->B; ++b) {
    const int64_t d0 = h->idisk[b], d1 = h->idisk[b + 1], Mb = d1 - d0;
    const bool circ = c.circ && h->circ && h->circ_on[b];
    S.con[b] = circ ? 1 : 0;
    const int64_t qs = QS > 0 ? QS : Mb;
    // row disks ordered by their number of 16-row tiles (stable), in groups of
    // RP; for the column lists of the circulant form, by a Z-order (Morton)
    // code of their centers within each tile class, so that a group's rows are
    // neighbours and share most of their close column disks
    std::vector<int32_t> ord((size_t)Mb);
    for (int64_t k = 0; k < Mb; ++k) ord[(size_t)k] = (int32_t)(d0 + k);
    std::vector<uint32_t> zc;
    if (circ) {
      double x0 = h->cx[d0], x1 = x0, y0 = h->cy[d0], y1 = y0;
      for (int64_t q = d0; q < d1; ++q) {
        x0 = std::min(x0, h->cx[q]);
        x1 = std::max(x1, h->cx[q]);
        y0 = std::min(y0, h->cy[q]);
        y1 = std::max(y1, h->cy[q]);
      }
      const double sc = 65535.0 / std::max(std::max(x1 - x0, y1 - y0), 1e-300);
      zc.resize((size_t)Mb);
      for (int64_t k = 0; k < Mb; ++k) {
        const uint32_t ix = (uint32_t)((h->cx[d0 + k] - x0) * sc), iy = (uint32_t)((h->cy[d0 + k] - y0) * sc);
        uint32_t z = 0;
        for (int bit = 0; bit < 16; ++bit)
          z |= (((ix >> bit) & 1u) << (2 * bit)) | (((iy >> bit) & 1u) << (2 * bit + 1));
        zc[(size_t)k] = z;
      }
    }
    std::stable_sort(ord.begin(), ord.end(), [&](int32_t u, int32_t w) {
      const int tu = (2 * h->N[u] + 16) / 16, tw = (2 * h->N[w] + 16) / 16;
      if (tu != tw) return tu > tw;
      return circ && zc[(size_t)(u - d0)] < zc[(size_t)(w - d0)];
    });
    for (int64_t o = 0; o < Mb; o += c.RP) {
      const int rp = (int)std::min<int64_t>(c.RP, Mb - o);
      const int gi = (int)S.gnseg.size();
      for (int k = 0; k < c.RP; ++k) {
        const int32_t pk = k < rp ? ord[(size_t)(o + k)] : -1;
        S.grow.push_back(pk);
        if (pk >= 0) {
          S.dgrp[pk] = gi;
          S.drow[pk] = k;
        }
      }
      double rows = 0.0;
      for (int k = 0; k < rp; ++k) rows += 2 * h->N[ord[(size_t)(o + k)]] + 1;
      // column disks of the group: a contiguous range, or the list of the
      // close pairs of its rows (with the mask of the rows close to each)
      int64_t ncol = Mb, lbase = 0;
      std::vector<double> lw;  // column widths of the list entries
      if (circ && S.close_rows) {
        ncol = 0;  // k_apply_close writes segment 0 of every tile
      } else if (circ) {
        std::map<int32_t, int> mask;
        for (int k = 0; k < rp; ++k) {
          const int32_t pk = ord[(size_t)(o + k)];
          for (int64_t e = h->near_off[pk]; e < h->near_off[pk + 1]; ++e) mask[h->near[(size_t)e]] |= 1 << k;
        }
        lbase = (int64_t)S.qlist.size();
        for (const auto& kv : mask) {
          S.qlist.push_back((kv.first << 8) | kv.second);
          lw.push_back(2.0 * h->N[kv.first] + 1);
        }
        ncol = (int64_t)mask.size();
      }
      const int64_t qsg = circ ? (QS > 0 ? QS : std::max<int64_t>(ncol, 1)) : qs;
      const int nseg = (circ && S.close_rows) ? 1 : (int)((ncol + qsg - 1) / qsg);
      S.gnseg.push_back(nseg);
      S.gbase.push_back(pb);
      for (int t = 0; t < S.ntile; ++t) {
        if (!tile_runs(b, t * RC, (t + 1) * RC)) continue;
        for (int sg = 0; sg < (circ && S.close_rows ? 0 : nseg); ++sg) {
          const int64_t i0 = sg * qsg, i1 = std::min<int64_t>(ncol, i0 + qsg);
          double cw = 0.0;
          for (int64_t i = i0; i < i1; ++i) cw += circ ? lw[(size_t)i] : 2.0 * h->N[d0 + i] + 1;
          It e;
          e.cost = rows * cw + 64.0 * (double)(i1 - i0);  // MACs + per-disk staging
          e.r[0] = gi;
          e.r[1] = rp;
          e.r[2] = t;
          e.r[3] = (int32_t)((circ ? lbase : d0) + i0);
          e.r[4] = (int32_t)((circ ? lbase : d0) + i1);
          e.r[5] = (int32_t)(pb + (int64_t)t * nseg + sg);
          e.r[6] = circ ? 1 : 0;
          its.push_back(e);
        }
      }
      pb += (int64_t)S.ntile * nseg;
    }
    if (circ) {  // per-frequency products: (instance, frequency, row tile, column tile)
      const int Lb = h->cL[b];
      const int nrt = (int)((Mb + cbm - 1) / cbm), nct = (R + cbn - 1) / cbn;
      for (int f = 0; f < Lb; ++f)
        for (int rt = 0; rt < nrt; ++rt)
          for (int ct = 0; ct < nct; ++ct) {
            if (!tile_runs(b, ct * cbn, (ct + 1) * cbn)) continue;
            S.citems.push_back(b);
            S.citems.push_back(f);
            S.citems.push_back(rt);
            S.citems.push_back(ct);
          }
    }
  }
  S.n_pb = pb;
  if (S.close_rows) {
    std::vector<std::pair<int64_t, int32_t>> rows;  // (work: k steps x row tiles, row disk)
    for (int p = 0; p < h->M_all; ++p) {
      if (!S.con[(size_t)h->inst[p]]) continue;
      int64_t work = 0;
      for (int64_t e = h->near_off[p]; e < h->near_off[p + 1]; ++e)
        work += (int64_t)((2 * h->N[h->near[(size_t)e]] + 4) / 4) * ((2 * h->N[p] + 16) / 16);
      if (work > 0) rows.push_back({work, p});
      else S.drow[p] |= ROW_EMPTY;
    }
    std::stable_sort(rows.begin(), rows.end(), [&](const auto& u, const auto& w) {
      const bool lu = h->near_off[u.second + 1] - h->near_off[u.second] > CLOSE_LONG;
      const bool lw = h->near_off[w.second + 1] - h->near_off[w.second] > CLOSE_LONG;
      return lu != lw ? lu : u.first > w.first;
    });
    for (const auto& rw : rows) {
      const int p = rw.second, b = h->inst[p];
      const int e0 = (int)(S.crec.size() / 4);
      for (int64_t e = h->near_off[p]; e < h->near_off[p + 1]; ++e) {
        const int q = h->near[(size_t)e];
        S.crec.push_back((int32_t)h->moff[q]);
        S.crec.push_back(h->N[q]);
        S.crec.push_back((int32_t)h->toff[(size_t)pair_index(h->idisk.data(), h->ipair.data(), b, p, q)]);
        S.crec.push_back(p > q ? 1 : 0);
      }
      const int e1 = (int)(S.crec.size() / 4);
      S.n_long += e1 - e0 > CLOSE_LONG;
      for (int32_t w : {p, e0, e1, 0}) S.crow.push_back(w);
    }
  }
  std::stable_sort(its.begin(), its.end(), [](const It& a, const It& b) { return a.cost > b.cost; });
  S.items.resize(its.size() * MF_REC);
  for (size_t k = 0; k < its.size(); ++k)
    for (int f = 0; f < MF_REC; ++f) S.items[k * MF_REC + f] = its[k].r[f];
  S.n_items = (int)its.size();
  S.n_citems = (int)(S.citems.size() / 4);
  // Close pairs beside the transforms and products (a fork and a join between two
  // streams): worth it while the rest lasts long enough to cover the host's 50 us for
  // six launches and four event calls, and before it fills the chip so well that the
  // close pairs take as much from the products as they gain.  In between, by a score fitted to
  // the measurements: the product's operations and symbol bytes at the rates they reach,
  // added up though they overlap, and 2.2 ns per disk and column for the transforms (score
  // in brackets; us in turn, beside): 200 x 16 (24) 53.2, 57.4; 150 x 32 (23) 52.0, 54.6; 200 x
  // 32 (36) 61.5, 55.7; 100 x 128 (42) 70.8, 64.8; 400 x 32 (115) 121, 107; 1,000 x 8 (370) 282,
  // 271; 500 x 128 (472) 473, 450; 700 x 64 (494) 413, 414; 400 x 256 (602) 607, 617; 1,000 x 64
  // (947) 772, 792.
  double score = 2.2e-3 * R * h->M_all;
  if (c.circ)
    for (int b = 0; b < h->B; ++b)
      if (S.con[(size_t)b]) {
        const double M = (double)(h->idisk[b + 1] - h->idisk[b]), t = h->cL[(size_t)b] * M * M;
        score += t * (6.0 * R / 60e6 + 16.0 / 4.5e6);
      }
  S.close_beside = S.close_rows && !S.crow.empty() && score >= 30.0 && score <= 500.0;
}

// Device view of a schedule's arrays.
struct SchedDev {
  const int32_t *items, *dgrp, *grow, *gnseg, *drow, *qlist, *citems, *con, *crow, *crec;
  const int64_t* gbase;
};
template <class F>
static void sched_arrays(const MfmaSched& S, F&& f) {  // f(vector, pointer of the device view)
  f(S.items, &SchedDev::items);
  f(S.dgrp, &SchedDev::dgrp);
  f(S.grow, &SchedDev::grow);
  f(S.gnseg, &SchedDev::gnseg);
  f(S.drow, &SchedDev::drow);
  f(S.qlist, &SchedDev::qlist);
  f(S.citems, &SchedDev::citems);
  f(S.con, &SchedDev::con);
  f(S.crow, &SchedDev::crow);
  f(S.crec, &SchedDev::crec);
}
static size_t sched_blob_bytes(const MfmaSched& S) {
  size_t n = align256(S.gbase.size() * 8);
  sched_arrays(S, [&](const std::vector<int32_t>& v, auto) { n += align256(v.size() * 4); });
  return n;
}
static void sched_pack(MfmaSched& S) {
  S.blob.assign(sched_blob_bytes(S), 0);
  size_t o = align256(S.gbase.size() * 8);
  if (!S.gbase.empty()) memcpy(S.blob.data(), S.gbase.data(), S.gbase.size() * 8);
  sched_arrays(S, [&](const std::vector<int32_t>& v, auto) {
    if (!v.empty()) memcpy(S.blob.data() + o, v.data(), v.size() * 4);
    o += align256(v.size() * 4);
  });
}
static SchedDev sched_view(const MfmaSched& S) {
  SchedDev d{};
  d.gbase = (const int64_t*)S.dev;
  size_t o = align256(S.gbase.size() * 8);
  sched_arrays(S, [&](const std::vector<int32_t>& v, auto m) {
    d.*m = (const int32_t*)(S.dev + o);
    o += align256(v.size() * 4);
  });
  return d;
}

// Byte layout of the apply scratch on the MFMA path: queue counter, partial
// blocks, scaled input, transformed inputs and outputs (circulant form), and the
// schedule when it is not resident.
struct MfmaScratch {
  size_t head, part, z, zh, wh, sched, total;
};
static MfmaScratch mfma_scratch_layout(const mudiff_ctx* h, const MfmaSched& S) {
  MfmaScratch L{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t r = o;
    o = align256(o + bytes);
    return r;
  };
  L.head = take(4);
  L.part = take((size_t)S.n_pb * S.blk * 16);
  L.z = take((size_t)S.R * h->N_all * 16);  // the input with its column scale applied
  const size_t zw = S.c.circ ? (size_t)S.R * h->cZ_all * 16 : 0;
  L.zh = take(zw);
  L.wh = take(zw);
  L.sched = take(sched_blob_bytes(S));
  L.total = o;
  return L;
}

// Room for schedules in the tables workspace: a few of the sizes that
// multi-right-hand-side applies of this batch have (1,000 disks, 256 columns in
// the circulant form: 0.15 MB; what does not fit is uploaded at every call).
size_t resident_bytes(int B, const int64_t* disk_off) {
  return ((size_t)256 << 10) + (size_t)B * 1024 + (size_t)disk_off[B] * 256;
}

// Candidate tile choices for R right-hand sides (RP * CT waves of 64 lanes).
static std::vector<MfmaChoice> mfma_candidates(int R) {
  std::vector<MfmaChoice> out;
  const int ctmax = std::max(1, std::min(4, (R + 7) / 8));
  for (int waves : {4, 8})
    for (int ct : {1, 2, 4}) {
      if (ct > ctmax && ct > 1) continue;
      const int rp = waves / ct;
      if (rp < 1 || rp > 8) continue;
      for (int qs : {0, 32}) out.push_back(MfmaChoice{ct, rp, qs, 64 * waves, false});
    }
  return out;
}

// Column-disk segment of a tile: the longest of 64, 32, .. 4 that cuts the
// instances in the work queue (all of them, or with the circulant form those
// outside it) into at least four items per compute unit; 4 when none does, 0 (whole
// instances) when that already gives as many.  A workgroup spends 4 to 5 us on each
// column disk of an item whatever the tile (two barriers and a gather that has one
// disk's time to arrive), so few items leave the chip idle for as long as the
// longest takes (30 disks, 8 columns: 148 us with whole instances, 34 with segments
// of 4; 100 disks, 16 columns 190 with segments of 32, 92 of 4), while at two items
// a compute unit a launch still ends unevenly (200 disks, 64 columns: 847 us with
// segments of 64, 796 of 32) and ever shorter ones add partial sums.
static int auto_segment(const mudiff_ctx* h, int R, int CT, int RP, bool circ) {
  const int64_t tiles = (R + 8 * CT - 1) / (8 * CT), want = 4 * (int64_t)h->n_cu;
  int64_t mmax = 0;
  auto items = [&](int64_t qs) {
    int64_t n = 0;
    for (int b = 0; b < h->B; ++b) {
      if (circ && h->circ_on[(size_t)b]) continue;
      const int64_t M = h->idisk[b + 1] - h->idisk[b];
      mmax = std::max(mmax, M);
      n += (M + RP - 1) / RP * tiles * (qs > 0 ? (M + qs - 1) / qs : 1);
    }
    return n;
  };
  if (items(0) >= want || mmax <= 4) return 0;
  for (int qs = 64; qs > 4; qs /= 2)
    if (qs < mmax && items(qs) >= want) return qs;
  return 4;
}

// Segment length of a choice.  A timed one holds no length but the rule, so that the
// length follows the form when set_circulant or set_circulant_tile changes it: that of
// the circulant form counts only the instances outside it, and its short segments over
// whole instances would make more partial sums than the scratch is sized for.  With
// tiles of more than 8 columns the form's close pairs are in the queue too, as lists no
// longer than their instance, and take the direct form's length.
static int segment(const mudiff_ctx* h, int R, const MfmaChoice& c) {
  return c.QS == QS_RULE ? auto_segment(h, R, c.CT, c.RP, c.circ && c.CT == 1) : c.QS;
}

// The tiles that are timed on first use of R (mfma_candidates are those that a
// caller may fix): eight waves, the segment by rule.  Four waves were slower by
// half wherever the queue was timed (100 disks x 4, 64 columns: 684-739 against
// 367-458 us).  In the circulant form the queue holds the instances outside it and
// the close pairs run on k_apply_close, which takes 8-column tiles.
static std::vector<MfmaChoice> mfma_timed(int R, bool circ) {
  std::vector<MfmaChoice> out;
  for (int ct : {1, 2, 4}) {
    if (ct > 1 && (circ || 8 * (ct / 2) >= R)) continue;
    out.push_back(MfmaChoice{ct, 8 / ct, QS_RULE, 512, circ});
  }
  return out;
}

// The circulant form is a candidate when the tables hold it and some
// instance is worth it (and the caller has not switched it off for R).
static bool circ_usable(const mudiff_ctx* h, int R) {
  if (!h->circ || h->M_all >= (1 << 23)) return false;  // column lists hold q << 8
  auto f = h->circ_modes.find(R);
  if (f != h->circ_modes.end() && f->second == 0) return false;
  for (uint8_t c : h->circ_on)
    if (c) return true;
  return false;
}

static MfmaChoice mfma_default(int R) {
  const int ct0 = std::min(4, (R + 7) / 8);
  const int ct = ct0 == 3 ? 4 : ct0;
  return MfmaChoice{ct, 4 / ct, 0, 256, false};
}

void sched_wait(mudiff_ctx* h) {
  if (h->sched_pending) {
    (void)hipEventSynchronize(h->sched_ev);
    h->sched_pending = false;
  }
}

// Upload schedule S into the apply scratch at `scratch`, asynchronously: its blob
// stays untouched until sched_wait (a schedule of the handle) or a synchronisation
// of the stream (a local S).  Not for use under graph capture.
static int mfma_upload(mudiff_ctx* h, MfmaSched& S, char* scratch, hipStream_t s) {
  char* dst = scratch + mfma_scratch_layout(h, S).sched;
  HIP_TRY(hipMemcpyAsync(dst, S.blob.data(), S.blob.size(), hipMemcpyHostToDevice, s));
  if (!h->sched_ev) HIP_TRY(hipEventCreateWithFlags(&h->sched_ev, hipEventDisableTiming));
  HIP_TRY(hipEventRecord(h->sched_ev, s));
  h->sched_pending = true;
  S.dev = dst;
  return MUDIFF_OK;
}

// Put schedule S of the handle on the device: into the resident part of the
// tables workspace if it fits (once: this waits for the copy, so that applies on
// any stream find it), else into the apply scratch.  A capturing stream cannot
// wait: there the scratch takes it.
static int sched_place(mudiff_ctx* h, MfmaSched& S, char* scratch, hipStream_t s) {
  if (S.dev && (S.resident || S.dev == scratch + mfma_scratch_layout(h, S).sched)) return MUDIFF_OK;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess) cs = hipStreamCaptureStatusActive;
  if (cs == hipStreamCaptureStatusNone && &S != &h->mfma_tail_sched &&
      h->res_used + S.blob.size() <= h->res_bytes) {
    char* dst = h->res_base + h->res_used;
    HIP_TRY(hipMemcpyAsync(dst, S.blob.data(), S.blob.size(), hipMemcpyHostToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
    h->res_used += S.blob.size();
    S.dev = dst;
    S.resident = true;
    return MUDIFF_OK;
  }
  return mfma_upload(h, S, scratch, s);
}

// Second stream of the handle (straggler phase, medium sizes, short queues) and its events.
static int aux_stream(mudiff_ctx* h) {
  if (h->aux) return MUDIFF_OK;
  HIP_TRY(hipStreamCreateWithFlags(&h->aux, hipStreamNonBlocking));
  HIP_TRY(hipEventCreateWithFlags(&h->fork_ev, hipEventDisableTiming));
  HIP_TRY(hipEventCreateWithFlags(&h->join_ev, hipEventDisableTiming));
  return MUDIFF_OK;
}

// Enqueue one MFMA apply with schedule S already on the device (S.dev).
typedef void (*mf_fn)(DevView, int, const cplx*, const int32_t*, const int32_t*, int, int32_t*,
                      cplx*, int64_t, int, int, int, int, const int32_t*, const int32_t*);

#define MF_TK3(MT, TH, ZK)                                 \
  if (zk == ZK) {                                          \
    if (tk == 1) return k_apply_mfma<MT, TH, ZK, 1>;       \
    if (tk == 2) return k_apply_mfma<MT, TH, ZK, 2>;       \
    if (TH == 256 && tk == 4) return k_apply_mfma<MT, TH, ZK, 4>; \
  }
#define MF_MT(MT)                                                                   \
  if (mt == MT) {                                                                   \
    if (th == 512) { MF_TK3(MT, 512, 1) MF_TK3(MT, 512, 2) MF_TK3(MT, 512, 4) }     \
    if (th == 256) { MF_TK3(MT, 256, 1) MF_TK3(MT, 256, 2) MF_TK3(MT, 256, 4)       \
                     MF_TK3(MT, 256, 8) }                                           \
  }

// Kernel variant for MT row tiles, workgroup size th and staging sizes zk, tk
// (powers of two; at 512 threads zk <= 4, tk <= 2, at 256 zk <= 8, tk <= 4).
static mf_fn mf_select(int mt, int th, int zk, int tk) {
  MF_MT(1) MF_MT(2) MF_MT(3) MF_MT(4)
  return nullptr;
}
#undef MF_MT
#undef MF_TK3

static int mfma_launch(mudiff_ctx* h, const MfmaSched& S, char* base, const cplx* x, cplx* y, int op,
                       const int32_t* active, hipStream_t s, const cplx* shift = nullptr) {
  const MfmaScratch L = mfma_scratch_layout(h, S);
  const SchedDev d = sched_view(S);
  int32_t* head = (int32_t*)(base + L.head);
  cplx* part = (cplx*)(base + L.part);
  const int mt = S.npad / 16;
  const int kt = (2 * h->Nmax + 1 + 3) / 4;
  const int RC = 8 * S.c.CT;
  const size_t lds = ((size_t)4 * kt * RC + (size_t)S.c.RP * (4 * kt + 16 * mt - 1)) * 16;
  prof_open(h, s);
  int rc = MUDIFF_OK;
  if (S.n_items > 0 && (rc = launch_fill_zero(head, 4, s)) != MUDIFF_OK) return rc;
  cplx* z = (cplx*)(base + L.z);
  if (S.n_items > 0) {  // the work queue's input; the circulant form's kernels scale as they read
    int64_t nbmax = 0;  // longest instance vector
    for (int b = 0; b < h->B; ++b) nbmax = std::max(nbmax, h->imode[b + 1] - h->imode[b]);
    if ((nbmax + 255) / 256 > 65535) return fail(MUDIFF_ERR_INVALID, "instance too large for the input scaling grid");
    hipLaunchKernelGGL(k_apply_mfma_scale, dim3((unsigned)(h->B * S.R), (unsigned)((nbmax + 255) / 256)),
                       dim3(256), 0, s, h->dv, S.R, x, z, active, S.close_rows ? d.con : nullptr);
    HIP_TRY(hipGetLastError());
  }
  prof_mark(h, s, 1);
  cplx* wh = nullptr;
  const int32_t* con = d.con;
  // direct-form work: in the straggler phase of a solve with the circulant form the
  // work queue and the close-pair rows run on the second stream, beside the
  // transforms and products, which share none of their outputs (there every launch
  // is small and latency-bound), the close pairs also at medium sizes (close_beside).
  // A short queue, that of a few instances outside the form, runs there at all sizes: it
  // leaves most of the chip idle for as long as its items take.
  mf_fn fn = nullptr;  // checked before the fork, so that every error leaves the streams joined
  if (S.n_items > 0) {
    const int TL = 4 * kt + 16 * mt - 1;
    auto pow2 = [](int v) { int r = 1; while (r < v) r <<= 1; return r; };
    const int zk = pow2((4 * kt * RC + S.c.threads - 1) / S.c.threads);
    const int tk = pow2((S.c.RP * TL + S.c.threads - 1) / S.c.threads);
    fn = mf_select(mt, S.c.threads, zk, tk);
    if (!fn) return fail(MUDIFF_ERR_INVALID, "no MFMA apply variant for this tile");
  }
  if (S.close_rows && (mt < 1 || mt > 4)) return fail(MUDIFF_ERR_INVALID, "close pairs: orders out of range");
  hipStream_t cs = s;
  // the block -> row mapping of the close-pair kernel
  const int n_close = (int)(S.crow.size() / 4);
  const int64_t per = (int64_t)S.ntile * (mt > 2 ? 2 : 1);  // waves per row
  const int64_t wpr = std::min<int64_t>(per, 4), rpb = 4 / wpr, n_short = n_close - S.n_long;
  const int64_t close_blocks = ((S.n_long + 7) & ~7) * per +
                               (((n_short + rpb - 1) / rpb + 7) & ~(int64_t)7) * ((per + wpr - 1) / wpr);
  if (n_close > 0 && close_blocks >= ((int64_t)1 << 31)) return fail(MUDIFF_ERR_INVALID, "close pairs: too many tiles");
  // (a caller's capture keeps to the caller's stream; a profiled apply keeps its phases apart)
  bool beside = h->mfma_tail, fork = S.c.circ && beside && (S.n_items > 0 || S.close_rows);
  const bool short_queue = S.c.circ && S.close_rows && S.n_items > 0 && S.n_items <= 4 * h->n_cu;
  if (!beside && (S.close_beside || short_queue) && h->prof_cur < 0) {
    hipStreamCaptureStatus cst = hipStreamCaptureStatusNone;
    fork = h->own_capture || (hipStreamIsCapturing(s, &cst) == hipSuccess && cst == hipStreamCaptureStatusNone);
    beside = fork && S.close_beside;
  }
  if (fork) {
    if ((rc = aux_stream(h)) != MUDIFF_OK) return rc;
    HIP_TRY(hipEventRecord(h->fork_ev, s));
    HIP_TRY(hipStreamWaitEvent(h->aux, h->fork_ev, 0));
    cs = h->aux;
  }
  auto launch_queue = [&](hipStream_t cs) -> int {
    if (S.n_items > 0) {
      // persistent grid: as many workgroups as are resident at once
      int per_cu = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)fn, S.c.threads, lds) !=
              hipSuccess || per_cu < 1)
        per_cu = 1;
      const int grid = std::max(1, std::min(S.n_items, per_cu * h->n_cu));
      hipLaunchKernelGGL(fn, dim3(grid), dim3(S.c.threads), lds, cs, h->dv, S.R, (const cplx*)z, active, d.items,
                         S.n_items, head, part, S.blk, S.npad, kt, S.c.RP, S.c.CT, d.grow, d.qlist);
      HIP_TRY(hipGetLastError());
    }
    return MUDIFF_OK;
  };
  auto launch_close = [&](hipStream_t cs) -> int {
    if (n_close == 0) return MUDIFF_OK;
    typedef void (*close_fn)(DevView, int, const cplx*, cplx*, int64_t, int, const int32_t*, const int32_t*,
                             const int64_t*, const int4*, const int4*, int, int, int, const int32_t*);
    static const close_fn kClose[5] = {nullptr, k_apply_close<1, 1>, k_apply_close<2, 2>,
                                       k_apply_close<3, 2>, k_apply_close<4, 2>};
    hipLaunchKernelGGL(kClose[mt], dim3((unsigned)close_blocks), dim3(256), 0, cs, h->dv, S.R, x, part, S.blk, S.npad,
                       d.dgrp, d.drow, d.gbase, (const int4*)d.crow, (const int4*)d.crec, n_close, S.n_long,
                       S.ntile, active);
    HIP_TRY(hipGetLastError());
    return MUDIFF_OK;
  };
  if (fork) {
    if ((rc = launch_queue(cs)) != MUDIFF_OK) return rc;
    if (beside && (rc = launch_close(cs)) != MUDIFF_OK) return rc;
    HIP_TRY(hipEventRecord(h->join_ev, cs));
  }
  if (S.c.circ) {  // well-separated pairs of the marked instances
    cplx* zh = (cplx*)(base + L.zh);
    wh = (cplx*)(base + L.wh);
    rc = circ_launch(h, S.R, x, zh, wh, d.citems, S.n_citems, S.cvar, con, S.con.data(), active, s);
    if (rc != MUDIFF_OK) return rc;
  } else {
    prof_mark(h, s, 2);
    prof_mark(h, s, 3);
  }
  if (!(fork && beside) && (rc = launch_close(s)) != MUDIFF_OK) return rc;
  if (fork) HIP_TRY(hipStreamWaitEvent(s, h->join_ev, 0));
  else if ((rc = launch_queue(s)) != MUDIFF_OK) return rc;
  prof_mark(h, s, 4);
  if (S.c.circ) {
    rc = circ_finish(h, S.R, x, y, op, (const cplx*)part, S.blk, S.npad, RC,
                     d.dgrp, d.drow, d.gnseg, d.gbase, active, (const cplx*)wh, con, S.con.data(), shift, s);
    prof_mark(h, s, 5);
    return rc;
  }
  const int64_t total = (int64_t)S.R * h->N_all;
  hipLaunchKernelGGL(k_apply_mfma_finish, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                     h->dv, S.R, x, y, op, (const cplx*)part, S.blk, S.npad, RC,
                     d.dgrp, d.drow, d.gnseg, d.gbase, active, (const cplx*)wh, con, shift);
  HIP_TRY(hipGetLastError());
  prof_mark(h, s, 5);
  return MUDIFF_OK;
}

// Apply scratch that covers every choice for R: the tiles that a caller may fix,
// the timed ones and the straggler schedule, in both forms.  The partial blocks
// are those of the direct form with its shortest segments (a close-pair item never
// has more column disks than its instance), the schedule's arrays are bounded.
static size_t mfma_scratch_bytes(mudiff_ctx* h, int R) {
  auto f = h->mfma_bytes.find(R);
  if (f != h->mfma_bytes.end()) return f->second;
  const int64_t npad = 16 * ((2 * h->Nmax + 1 + 15) / 16), n_near = (int64_t)h->near.size();
  int64_t part = 0, items = 0, groups = 0, rows = 0;
  std::vector<MfmaChoice> cs = mfma_candidates(R);
  for (MfmaChoice& c : cs) c.QS = MFMA_TAIL_QS;
  cs.push_back(mfma_default(R));
  for (const MfmaChoice& c : mfma_timed(R, false)) cs.push_back(c);
  if (h->circ)
    for (const MfmaChoice& c : mfma_timed(R, true)) cs.push_back(c);
  for (const MfmaChoice& c : cs) {
    const int64_t tiles = (R + 8 * c.CT - 1) / (8 * c.CT), QS = segment(h, R, c);
    int64_t n_pb = 0, g = 0;
    for (int b = 0; b < h->B; ++b) {
      const int64_t M = h->idisk[b + 1] - h->idisk[b], gb = (M + c.RP - 1) / c.RP;
      // a timed choice of the circulant form has its short segments outside the form only
      const bool whole = c.circ && h->circ_on[(size_t)b];
      n_pb += gb * tiles * (QS > 0 && !whole ? (M + QS - 1) / QS : 1);
      g += gb;
    }
    part = std::max(part, n_pb * c.RP * npad * 8 * c.CT);
    items = std::max(items, n_pb);
    groups = std::max(groups, g);
    rows = std::max(rows, g * c.RP);
  }
  int64_t citems = 0;
  if (h->circ) {
    std::vector<int> vars = circ_variants(R);
    vars.push_back(circ_variant(R));
    for (int v : circ_timed(R)) vars.push_back(v);
    for (int v : vars) {
      int bm = 0, bn = 0;
      circ_tile(v, &bm, &bn);
      int64_t n = 0;
      for (int b = 0; b < h->B; ++b)
        n += (int64_t)h->cL[b] * ((h->idisk[b + 1] - h->idisk[b] + bm - 1) / bm) * ((R + bn - 1) / bn);
      citems = std::max(citems, n);
    }
  }
  const size_t zw = h->circ ? (size_t)R * h->cZ_all * 16 : 0;
  const size_t sched = (size_t)items * MF_REC * 4 + (size_t)groups * 12 + (size_t)rows * 4 +
                       (size_t)h->M_all * 8 + (size_t)h->B * 4 + (size_t)n_near * 4 + (size_t)citems * 16 +
                       (h->circ ? (size_t)h->M_all * 16 + (size_t)n_near * 16 : 0) + 16 * 256;
  const size_t mx = align256(4) + align256((size_t)part * 16) + align256((size_t)R * h->N_all * 16) +
                    2 * align256(zw) + align256(sched);
  h->mfma_bytes[R] = mx;
  return mx;
}

// Whether schedule S keeps to the scratch that was asked for (mfma_scratch_bytes covers
// every choice; this is what stands between a choice it misses and memory that is not ours).
static int scratch_check(mudiff_ctx* h, const MfmaSched& S) {
  const size_t need = mfma_scratch_layout(h, S).total, have = mfma_scratch_bytes(h, S.R);
  if (need <= have) return MUDIFF_OK;
  return fail(MUDIFF_ERR_NOMEM, "this apply's schedule needs " + std::to_string(need) + " bytes of scratch, more than the " +
                                    std::to_string(have) + " of its workspace");
}

// Pick the tile choice for R by timing the mfma_timed tiles and the product
// variants worth it on x -> y (outputs are overwritten; the inputs only need to be
// finite).
static int mfma_autotune(mudiff_ctx* h, int R, const cplx* x, cplx* y, char* scratch,
                         hipStream_t s) {
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  float best = 0.0f;
  MfmaChoice bc = mfma_default(R);
  int rc = MUDIFF_OK;
  std::vector<MfmaChoice> cands;
  auto fc = h->circ_modes.find(R);
  const int cmode = fc != h->circ_modes.end() ? fc->second : -1;
  const bool cu = circ_usable(h, R);
  // the circulant form first: it usually sets the bar the direct tiles then fail
  if (cu) cands = mfma_timed(R, true);
  if (cmode != 1 || !cu)
    for (const MfmaChoice& c : mfma_timed(R, false)) cands.push_back(c);
  // The direct form's work (8 flops per complex multiply-add over every
  // ordered pair) at the FP64 matrix-core peak, 78.6 TFLOP/s: no direct tile
  // beats it, so once a candidate's pair of applies is faster than twice that,
  // the direct tiles are not timed.
  double dflops = 0.0;
  for (int b = 0; b < h->B; ++b) {
    double sn = 0.0, sn2 = 0.0;
    for (int64_t p = h->idisk[b]; p < h->idisk[b + 1]; ++p) {
      const double n = 2.0 * h->N[(size_t)p] + 1.0;
      sn += n;
      sn2 += n * n;
    }
    dflops += 8.0 * R * (sn * sn - sn2);
  }
  int64_t mmax = 0;  // disks of the largest instance
  for (int b = 0; b < h->B; ++b) mmax = std::max(mmax, h->idisk[b + 1] - h->idisk[b]);
  const float direct_floor_ms = (float)(2.0 * dflops / 78.6e12 * 1e3);
  // one warm-up and two timed applies of candidate c; keeps the fastest (and
  // returns the time, 0 when skipped or failed)
  auto time_one = [&](const MfmaChoice& c) -> float {
    MfmaSched S;
    mfma_build(h, R, c, S);
    if ((rc = scratch_check(h, S)) != MUDIFF_OK) return 0.0f;
    struct Drain {  // the local schedule's copies finish before it is released
      hipStream_t st;
      ~Drain() { (void)hipStreamSynchronize(st); }
    } drain{s};
    sched_pack(S);
    if ((rc = mfma_upload(h, S, scratch, s)) != MUDIFF_OK) return 0.0f;
    (void)hipEventRecord(e0, s);
    if ((rc = mfma_launch(h, S, scratch, x, y, MUDIFF_OP_A, nullptr, s)) != MUDIFF_OK) return 0.0f;  // warm-up
    (void)hipEventRecord(e1, s);
    if (best > 0.0f) {  // a warm-up already twice as slow as the best pair of applies: no contender
      float w = 0.0f;
      if (hipEventSynchronize(e1) == hipSuccess && hipEventElapsedTime(&w, e0, e1) == hipSuccess &&
          w > best)
        return 0.0f;
    }
    (void)hipEventRecord(e0, s);
    for (int k = 0; k < 2 && rc == MUDIFF_OK; ++k) rc = mfma_launch(h, S, scratch, x, y, MUDIFF_OP_A, nullptr, s);
    (void)hipEventRecord(e1, s);
    if (rc != MUDIFF_OK) return 0.0f;
    if (hipEventSynchronize(e1) != hipSuccess) {
      rc = fail(MUDIFF_ERR_DEVICE, "autotune: event synchronisation failed");
      return 0.0f;
    }
    float ms = 0.0f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    if (best == 0.0f || ms < best) {
      best = ms;
      bc = c;
    }
    return ms;
  };
  const std::vector<int> cvars = circ_timed(R);
  for (MfmaChoice c : cands) {
    if (!c.circ && best > 0.0f && direct_floor_ms > best) continue;
    if (c.circ) c.cvar = cvars[0];
    const float ms = time_one(c);
    if (rc != MUDIFF_OK) break;
    // A tile of the direct form that is no more than 1.3 times as slow as the best is also timed
    // with whole instances and segments of 32: the rule counts items, but short segments of
    // small instances or of many row tiles cost more in partial sums than the evener end saves
    // (us of an apply by rule, and by these: 64 x 12 disks of order 3, 20 columns 46, 38; 200 of
    // order 31, 20 columns 746, 680; 300 x 6 of orders 5..18, 12 columns 90, 81; 200 of orders
    // 5..18, 20 columns 268, 223).
    const int rule = segment(h, R, c);
    for (int qs : {0, 32}) {
      if (c.circ || ms == 0.0f || ms > 1.3f * best || qs == rule || qs >= mmax || rc != MUDIFF_OK) continue;
      MfmaChoice q = c;
      q.QS = qs;
      time_one(q);
    }
  }
  if (rc == MUDIFF_OK && bc.circ) {  // then the other per-frequency product variants
    MfmaChoice c = bc;
    for (size_t k = 1; k < cvars.size() && rc == MUDIFF_OK; ++k) {
      c.cvar = cvars[k];
      time_one(c);
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != MUDIFF_OK) return rc;
  h->mfma_choice[R] = bc;
  h->mfma_time_ms[R] = best / 2.0f;
  return MUDIFF_OK;
}

// Drop the schedule of R (its choice changed): no upload still reads it.
static void sched_drop(mudiff_ctx* h, int R) {
  sched_wait(h);
  h->mfma_scheds.erase(R);
}

// Make the schedule for R current and place it on the device (autotuning on
// first use of R when x, y are given, else the default choice).
static int mfma_prepare(mudiff_ctx* h, int R, const cplx* x, cplx* y, char* scratch,
                        hipStream_t s) {
  int rc = MUDIFF_OK;
  auto f = h->mfma_choice.find(R);
  if (f == h->mfma_choice.end()) {
    if (x && y && h->mfma_tune) {
      if ((rc = mfma_autotune(h, R, x, y, scratch, s)) != MUDIFF_OK) return rc;
    } else {
      MfmaChoice d = mfma_default(R);
      d.circ = circ_usable(h, R);
      h->mfma_choice[R] = d;
    }
    f = h->mfma_choice.find(R);
  }
  MfmaChoice c = f->second;
  if (h->mfma_tail) c.QS = MFMA_TAIL_QS;
  MfmaSched& S = h->mfma_tail ? h->mfma_tail_sched : h->mfma_scheds[R];
  if (S.R != R || !(S.c == c)) {
    sched_wait(h);
    mfma_build(h, R, c, S, h->mfma_tail ? h->mfma_tail_cols : std::vector<int32_t>{});
    if ((rc = scratch_check(h, S)) != MUDIFF_OK) {
      S.R = 0;  // not a schedule that a later call may run
      return rc;
    }
    sched_pack(S);
  }
  return sched_place(h, S, scratch, s);
}

// The schedule that mfma_prepare made current.
static const MfmaSched& mfma_current(const mudiff_ctx* h, int R) {
  return h->mfma_tail ? h->mfma_tail_sched : h->mfma_scheds.at(R);
}

int apply_set_tail(mudiff_ctx* h, int R, bool tail, cplx* scratch, hipStream_t s,
                   const int32_t* cols) {
  if (!use_mfma(h, R)) return MUDIFF_OK;
  if (!tail && !h->mfma_tail) return MUDIFF_OK;
  h->mfma_tail = tail;
  if (tail && cols) h->mfma_tail_cols.assign(cols, cols + (size_t)h->B * R);
  else h->mfma_tail_cols.clear();
  sched_wait(h);
  h->mfma_tail_sched.R = 0;  // rebuild
  apply_forget_upload(h);    // the two forms lay out the scratch differently
  return mfma_prepare(h, R, nullptr, nullptr, (char*)scratch, s);
}

// ------------------------------------------------------------------ planning
namespace {
typedef void (*apply_fn)(DevView, int, const cplx*, cplx*, int, cplx*, int64_t, int32_t*,
                         const int32_t*, const int32_t*, const int64_t*, const int32_t*, int, int, int,
                         const cplx*);
typedef void (*lane_fn)(DevView, int, const cplx*, cplx*, int64_t, const int32_t*,
                        const int32_t*);

struct Variant {
  int bt, nspec;
  apply_fn fn;
};

// LDS-staged kernels: generic (nspec = -1) and uniform-N specialisations (batches of N = 15 with
// instances of 17 to some 65 disks, us, generic and exact loop bounds: one of 20 10.3, 8.2, 40
// of 22 25.9, 17.9, 8 of 50, 4 columns 67.8, 44.7, 40 of 65 142.8, 94.9)
const Variant kVariants[] = {
    {4, -1, k_apply<4, -1>}, {4, 15, k_apply<4, 15>},
};

const Variant* find_variant(int bt, int nspec) {
  for (const Variant& v : kVariants)
    if (v.bt == bt && v.nspec == nspec) return &v;
  return nullptr;
}

struct LaneVariant {
  int n;
  lane_fn fn[2];     // single-layer column factors (real): LANE_ROWS rows per workgroup, one row
  lane_fn fn_op[2];  // column factors of an operator set by mudiff_set_operator
};

// one-lane-per-pair kernels (uniform N); LANE_ROWS rows from order LANE_ROWS_NMIN on
template <int N>
constexpr LaneVariant lane_variant() {
  if constexpr (N >= LANE_ROWS_NMIN)
    return {N, {k_apply_lane<N, false>, k_apply_lane<N, false, 1>}, {k_apply_lane<N, true>, k_apply_lane<N, true, 1>}};
  else
    return {N, {nullptr, k_apply_lane<N, false, 1>}, {nullptr, k_apply_lane<N, true, 1>}};
}
const LaneVariant kLane[] = {lane_variant<1>(), lane_variant<2>(),  lane_variant<3>(),  lane_variant<4>(),
                             lane_variant<5>(), lane_variant<6>(),  lane_variant<7>(),  lane_variant<8>(),
                             lane_variant<9>(), lane_variant<10>(), lane_variant<11>(), lane_variant<12>()};

const LaneVariant* find_lane(int n) {
  for (const LaneVariant& v : kLane)
    if (v.n == n) return &v;
  return nullptr;
}
}  // namespace

// Host plan of the operator apply: kernel variant, work items and partial-sum
// layout, from the batch description alone (also used to size workspaces).
struct PlanHost {
  int lane = 0;  // LANE_UNIFORM (N = nspec), LANE_PAIRS, or 0: LDS-staged kernel
  int item_ints = 4;
  bool wide = false;  // k_apply_pairs<true>
  int bt = 4, nspec = -1, zs = 0, ts = 0, ppcap = 1;
  size_t lds = 0;
  int64_t part = 0;
  int few = 0, few_cols = 0, few_z = 0, lane_rows = 1;  // few: ints per task
  int64_t row_part = 0;  // partial sums of the LDS-staged kernel (bounds mudiff_matvec_noalloc)
  double few_us = 0.0, lane_us = 0.0;
  bool count = false;  // only the sizes: nothing goes into items and tasks
  size_t item_total = 0, task_total = 0;  // ints of items and tasks
  std::vector<int32_t> items, nch, tasks, few_tasks;
  std::vector<int64_t> poff;
};

// The uniform-N specialisation when every disk has the same N and one is
// compiled, else the generic kernel with BT = 4.
static void choose_variant(int M, const int32_t* N, int* bt, int* nspec) {
  bool uniform = true;
  for (int p = 1; p < M; ++p)
    if (N[p] != N[0]) uniform = false;
  if (uniform) {
    for (const Variant& v : kVariants)
      if (v.nspec == N[0]) {
        *bt = v.bt;
        *nspec = v.nspec;
        return;
      }
  }
  *bt = 4;
  *nspec = -1;
}

#define APPLY_LDS_BUDGET (64 * 1024)

// Column disks that the LDS-staged kernel passes over at a time, for a row of np modes
// in a batch whose largest order is nmax.
static int lds_cols(int np, int nmax, int bt) {
  const int zs = (2 * nmax + 1 + bt - 1) / bt * bt;
  const int cap = std::max(1, (int)(APPLY_LDS_BUDGET / ((size_t)(3 * zs - 1) * 16)));
  return std::max(1, std::min(APPLY_THREADS / ((np + bt - 1) / bt), cap));
}

// The same for the rows of a batch, with the passes and work items of a row in an instance of
// M disks.  Kept by the order: set-up counts every row several times over, and the divisions
// were most of it (set-up of 64 instances of 30 disks of orders 2 to 9, with an apply, 568 us
// with them, 433 without; orders 13 to 20 615, 482).
struct LdsRows {
  struct Row {
    int cols = 0;
    int64_t M = 0, passes = 0, items = 0;
  };
  int nmax, bt;
  std::vector<Row> rows;
  LdsRows(int nmax_, int bt_) : nmax(nmax_), bt(bt_), rows((size_t)nmax_ + 1) {}
  const Row& at(int N, int64_t M) {
    Row& r = rows[(size_t)N];
    if (r.M != M) {
      if (r.cols == 0) r.cols = lds_cols(2 * N + 1, nmax, bt);
      const int64_t qc = (int64_t)APPLY_NPASS * r.cols;
      r.M = M;
      r.passes = (M - 1 + r.cols - 1) / r.cols;
      r.items = (M - 1 + qc - 1) / qc;
    }
    return r;
  }
};

// Batches of k_apply_pairs: every N_p <= PAIRS_NMAX, and the faster one of the two by an
// estimate.  A wave of k_apply_pairs fills its 64 lanes with the disks of one instance and
// issues the same instructions however few they are; the LDS-staged kernel spreads one
// pair over many threads, but pays for every pass over its rows' columns, for every
// workgroup, and for the fences of rows that span several.  One column, us (fitted to 124
// batches of 18 to 8,700 disks, orders 1..4, 13..20 and 24..31, within 12% and 8% in the
// mean):
//   LDS-staged   5.9 + 0.096 passes (2N+1) + 9.5 (some row spans workgroups) + 0.010 a
//                workgroup + 0.92 (1.16 in rows that span) per 10^6 multiply-adds
//   k_apply_pairs   6.8 + 0.144 (2N+1) + 2.33 per 10^6 wave instructions + 0.00107 a task
// Measured, LDS-staged against k_apply_pairs: orders 13..20, 100 instances of 5 to 12 disks
// and one of 24 24.5, 31.7, and one of 200 143, 52; 1,000 and one of 24 188, 235; 300 of 2
// to 4 and one of 24 22.4, 36.4; one instance of 26 19.1, 14.7, 8 of 64 148, 27; orders
// 24..31, 1,000 of 5 to 12 and one of 24 297, 483; orders 1..4, one of 26 7.9, 9.4.
#define PAIRS_MARGIN 1.05
bool pairs_batch(int B, const int64_t* idisk, const int32_t* N) {
  int64_t mmax = 0;
  int nmax = 0;
  for (int b = 0; b < B; ++b) mmax = std::max(mmax, idisk[b + 1] - idisk[b]);
  for (int64_t p = 0; p < idisk[B]; ++p) nmax = std::max(nmax, (int)N[p]);
  if (nmax > PAIRS_NMAX || !(mmax >= 24 || (mmax > FEW_DISKS && idisk[B] >= 2048))) return false;
  double passes = 0.0, wgs = 0.0, macs = 0.0, macs_span = 0.0, instr = 0.0, tasks = 0.0;
  LdsRows rows(nmax, 4);
  int nblk[PAIRS_NMAX + 1], wid[PAIRS_NMAX + 1];  // blocks of a row and their width, by the order
  for (int n = 0; n <= nmax; ++n) {
    nblk[n] = (2 * n + PAIRS_BT_WIDE) / PAIRS_BT_WIDE;
    wid[n] = std::max((2 * n + nblk[n]) / nblk[n], 7);
  }
  for (int b = 0; b < B; ++b) {
    const int64_t d0 = idisk[b], d1 = idisk[b + 1], M = d1 - d0;
    if (M < 2) continue;
    double sum = 0.0;
    int nb = 0;  // largest order of the instance
    for (int64_t p = d0; p < d1; ++p) {
      sum += 2 * N[p] + 1;
      nb = std::max(nb, (int)N[p]);
    }
    const double chunks = (double)((M + LANE_CHUNK - 1) / LANE_CHUNK);
    for (int64_t p = d0; p < d1; ++p) {
      const int np = 2 * N[p] + 1, blocks = nblk[N[p]], w = wid[N[p]];
      const LdsRows::Row& r = rows.at(N[p], M);
      passes = std::max(passes, (double)r.passes);
      wgs += (double)r.items;
      macs += np * (sum - np);
      if (r.items > 1) macs_span += np * (sum - np);
      tasks += chunks * blocks;
      instr += chunks * blocks * (2 * nb + w) * (4 * w + 12);
    }
  }
  const double n = 2.0 * nmax + 1.0;
  double lds = 5.9 + 0.096 * passes * n + (macs_span > 0.0 ? 9.5 : 0.0) + 0.010 * wgs + 0.92e-6 * macs + 0.24e-6 * macs_span;
  int bt = 0, nspec = -1;
  choose_variant((int)idisk[B], N, &bt, &nspec);
  // the variant for one order (the factors fit the choices at 71 batches; k_apply_pairs in turn,
  // us): 40 instances of 24 disks 20.4, 25.2, 120 of 28 62.7, 77.2, 40 of 50 63.6, 51.5, 40 of 65
  // 94.9, 122.6, one of 100 27.6, 15.6
  if (nspec >= 0) lds *= macs_span > 0.0 ? 0.9 : 0.57;
  const double pairs = 6.8 + 0.144 * n + 2.33e-6 * instr + 0.00107 * tasks;
  return PAIRS_MARGIN * pairs < lds;
}

// Schedule of k_apply_pairs.  Tasks: the rows of an instance by decreasing N, each
// cut into blocks of equal width, at most PAIRS_BT_WIDE outputs, or
// PAIRS_BT_NARROW where wide blocks make fewer tasks than the 3,072 waves that
// narrow blocks keep resident (1,000 disks: 368 us narrow, 352 wide; 400: 96 and
// 90; at 200, too few tasks, 40 narrow).  Items: 64 column disks x a run of tasks,
// four tasks (one per wave) up to the point where the launch is PAIRS_WGS
// workgroups, longer runs beyond (1,000 disks: 371 us with 3,000, 373 with 1,500,
// 468 against 427 with 740, a single round of resident workgroups).  A row keeps
// one partial sum per 64 column disks; where those would exceed PAIRS_PART_MAX per
// right-hand side an item walks several chunks, at least `qc` column disks, the
// widest item of the LDS-staged kernel (so the scratch never exceeds that kernel's,
// nor the bound that mudiff_matvec_noalloc works under).
#define PAIRS_WGS 3000
#define PAIRS_PART_MAX ((int64_t)1 << 18)  // complex values: 4 MiB
#define PAIRS_WIDE_TASKS 3072
// Block width that k_apply_pairs is compiled for, at least w.
static int pairs_width(int w, bool wide) { return std::max(w, wide ? 7 : 5); }

static void make_pairs_plan(int B, const int64_t* idisk, const int32_t* N, int64_t qc, PlanHost& P) {
  P.lane = LANE_PAIRS;
  P.item_ints = PAIRS_ITEM_INTS;
  int lane_N = -1, nmax = 0;
  std::vector<int32_t> ord;
  if (!P.count) lane_layout(B, idisk, N, &lane_N, nullptr, &ord);
  int64_t part1 = 0;  // partial sums at one chunk per segment
  for (int b = 0; b < B; ++b) {
    const int64_t d0 = idisk[b], Mb = idisk[b + 1] - d0;
    const int64_t nch = Mb > 1 ? (Mb + LANE_CHUNK - 1) / LANE_CHUNK : 0;
    for (int64_t p = d0; p < d0 + Mb; ++p) {
      const int np = 2 * N[p] + 1;
      part1 += std::max<int64_t>(nch, 1) * np;
      nmax = std::max(nmax, (int)N[p]);
    }
  }
  const int64_t K = part1 <= PAIRS_PART_MAX ? 1 : qc / LANE_CHUNK + 1;  // chunks per segment
  auto count = [&](int bt) {  // tasks of all segments with blocks of at most bt outputs
    int blocks[PAIRS_NMAX + 1];
    for (int o = 0; o <= nmax; ++o) blocks[o] = (2 * o + bt) / bt;
    int64_t n = 0;
    for (int b = 0; b < B; ++b) {
      const int64_t d0 = idisk[b], Mb = idisk[b + 1] - d0;
      const int64_t nch = Mb > 1 ? (Mb + LANE_CHUNK - 1) / LANE_CHUNK : 0, nseg = (nch + K - 1) / K;
      for (int64_t p = d0; p < d0 + Mb; ++p) n += nseg * blocks[N[p]];
    }
    return n;
  };
  P.wide = count(PAIRS_BT_WIDE) >= PAIRS_WIDE_TASKS;
  const int btmax = P.wide ? PAIRS_BT_WIDE : PAIRS_BT_NARROW;
  const int64_t run = std::max<int64_t>(4, (count(btmax) + PAIRS_WGS - 1) / PAIRS_WGS);
  P.lds = (size_t)(2 * nmax + 2) * PAIRS_LD * 16;  // 66,560 bytes at PAIRS_NMAX
  int wid[PAIRS_NMAX + 1], ntask[PAIRS_NMAX + 1];  // width and number of a row's blocks, by the order
  for (int o = 0; o <= nmax; ++o) {
    const int np = 2 * o + 1, nblk = (np + btmax - 1) / btmax;
    wid[o] = pairs_width((np + nblk - 1) / nblk, P.wide);
    ntask[o] = (np + wid[o] - 1) / wid[o];
  }
  for (int b = 0; b < B; ++b) {
    const int64_t d0 = idisk[b], Mb = idisk[b + 1] - d0;
    const int64_t nch = Mb > 1 ? (Mb + LANE_CHUNK - 1) / LANE_CHUNK : 0, nseg = (nch + K - 1) / K;
    const int64_t tb = (int64_t)P.task_total / 2;
    for (int64_t k = d0; k < d0 + Mb; ++k) {
      const int p = P.count ? (int)k : ord[(size_t)k], np = 2 * N[p] + 1;
      P.nch[p] = (int32_t)nseg;
      P.poff[p] = P.part;
      P.part += std::max<int64_t>(nseg, 1) * np;
      const int w = wid[N[p]];
      if (nch > 0) P.task_total += 2 * (size_t)ntask[N[p]];
      for (int ms = 0; ms < np && nch > 0 && !P.count; ms += w) {
        P.tasks.push_back(p);
        P.tasks.push_back((ms << 8) | w);
      }
    }
    const int64_t te = (int64_t)P.task_total / 2;
    P.item_total += (size_t)(nseg * ((te - tb + run - 1) / run)) * PAIRS_ITEM_INTS;
    for (int64_t sg = 0; sg < nseg && !P.count; ++sg)
      for (int64_t t = tb; t < te; t += run) {
        const int64_t rec[PAIRS_ITEM_INTS] = {b, sg * K, std::min(K, nch - sg * K), t, std::min(te, t + run),
                                              d0, sg, Mb};
        for (int64_t w : rec) P.items.push_back((int32_t)w);
      }
  }
}

void make_plan(int B, const int64_t* idisk, const int32_t* N, bool pairs, PlanHost& P) {
  const int M = (int)idisk[B];
  P.items.clear();
  P.tasks.clear();
  P.item_total = P.task_total = 0;
  P.nch.assign(M, 0);
  P.poff.assign(M, 0);
  P.part = 0;
  P.lds = 0;
  bool uniform = true;
  for (int p = 1; p < M; ++p)
    if (N[p] != N[0]) uniform = false;
  if (uniform && N[0] <= LANE_NMAX && find_lane(N[0])) {
    P.lane = LANE_UNIFORM;
    P.item_ints = LANE_ITEM_INTS;
    P.nspec = N[0];
    const int np = 2 * N[0] + 1;
    int lane_N = -1;
    std::vector<int64_t> ltoff;
    lane_layout(B, idisk, N, &lane_N, &ltoff);
    auto push64 = [&](int64_t v) {
      P.items.push_back((int32_t)(v & 0xffffffff));
      P.items.push_back((int32_t)(v >> 32));
    };
    // Four rows of a workgroup share the scaled inputs of their chunk (k_apply_lane) where the
    // inputs are many and the waves that a last group of an instance leaves idle are few.  Time
    // with four rows over that with one, launches of 6,000 waves and more: order 9 0.92 to
    // 0.97, 12 0.93 to 1.00, but 1.00 to 1.05 for orders 8 and less (7: 1.01 to 1.12); in
    // instances of 13 disks (16 waves for 13) 1.17, of 17 1.10, of 22 1.06, of 50 1.00.
    int64_t waves = 0, padded = 0;
    for (int b = 0; b < B; ++b) {
      const int64_t Mb = idisk[b + 1] - idisk[b], n = (Mb - 1 + LANE_CHUNK - 1) / LANE_CHUNK;
      waves += Mb * n;
      padded += (Mb + LANE_ROWS - 1) / LANE_ROWS * LANE_ROWS * n;
    }
    P.lane_rows = N[0] >= LANE_ROWS_NMIN && waves >= LANE_FEW_WAVES && 20 * padded <= 21 * waves ? LANE_ROWS : 1;
    P.lane_us = (double)waves * np * (0.037e-3 + 9.4e-6 * np);
    int64_t i0 = 0;  // first unknown of instance b
    for (int b = 0; b < B; ++b) {
      const int64_t d0 = idisk[b], Mb = idisk[b + 1] - d0;
      const int64_t n = (Mb - 1 + LANE_CHUNK - 1) / LANE_CHUNK;  // 0 for M = 1
      for (int64_t p = d0; p < d0 + Mb; ++p) {
        P.nch[p] = (int32_t)n;
        P.poff[p] = P.part;
        P.part += std::max<int64_t>(n, 1) * np;
      }
      P.item_total += (size_t)((Mb + P.lane_rows - 1) / P.lane_rows * n) * LANE_ITEM_INTS;
      for (int64_t p = d0; p < d0 + Mb && !P.count; p += P.lane_rows)
        for (int64_t c = 0; c < n; ++c) {
          const int64_t jb = c * LANE_CHUNK, je = std::min<int64_t>(jb + LANE_CHUNK, Mb - 1);
          P.items.push_back((int32_t)p);
          P.items.push_back((int32_t)std::min<int64_t>(P.lane_rows, d0 + Mb - p));
          P.items.push_back((int32_t)jb);
          P.items.push_back((int32_t)je);
          P.items.push_back(b);
          P.items.push_back((int32_t)d0);
          push64(i0);
          push64(Mb * np);
          push64(ltoff[p] + c * (int64_t)(LANE_CHUNK * LANE_REC));
          push64(P.poff[p] + c * np);
          push64(0);
        }
      i0 += Mb * np;
    }
    return;
  }
  P.lane = 0;
  choose_variant(M, N, &P.bt, &P.nspec);
  const int bt = P.bt;
  int nmax = 0;
  for (int p = 0; p < M; ++p) nmax = std::max(nmax, (int)N[p]);
  // LDS rows: z stride zs (padded to BT), symbol rows ts = zs + LB_max - 1
  P.zs = ((2 * nmax + 1) + bt - 1) / bt * bt;
  P.ts = P.zs + P.zs - 1;
  P.ppcap = std::max(1, (int)(APPLY_LDS_BUDGET / ((size_t)(P.zs + P.ts) * 16)));
  LdsRows rows(nmax, bt);
  if (pairs && pairs_batch(B, idisk, N)) {
    make_pairs_plan(B, idisk, N, (int64_t)lds_cols(1, nmax, bt) * APPLY_NPASS, P);
    P.row_part = 0;
    for (int b = 0; b < B; ++b) {
      const int64_t Mb = idisk[b + 1] - idisk[b];
      for (int64_t p = idisk[b]; p < idisk[b + 1]; ++p) {
        P.row_part += std::max<int64_t>(1, rows.at(N[p], Mb).items) * (2 * N[p] + 1);
      }
    }
    return;
  }
  for (int b = 0; b < B; ++b) {
    const int64_t d0 = idisk[b], Mb = idisk[b + 1] - d0;
    for (int64_t p = d0; p < d0 + Mb; ++p) {
      const int np = 2 * N[p] + 1;
      const int L = (np + bt - 1) / bt;
      const LdsRows::Row& r = rows.at(N[p], Mb);
      const int64_t qc = (int64_t)APPLY_NPASS * r.cols, n = std::max<int64_t>(1, r.items);
      P.nch[p] = (int32_t)n;
      P.poff[p] = P.part;
      P.part += n * np;
      P.item_total += (size_t)n * 4;
      for (int64_t c = 0; c < n && !P.count; ++c) {
        int64_t jb = c * qc, je = std::min<int64_t>(jb + qc, Mb - 1);
        P.items.push_back((int32_t)p);
        P.items.push_back((int32_t)c);
        P.items.push_back((int32_t)jb);
        P.items.push_back((int32_t)je);
      }
      const int64_t pp = r.cols;
      P.lds = std::max(P.lds, (size_t)pp * (P.zs + P.ts) * 16);
      P.lds = std::max(P.lds, (size_t)pp * L * bt * 16);
    }
  }
}

// Tasks of k_apply_few, for batches of small instances whose panels fit its LDS: in place
// of the plan's items, but for uniform orders, where few_applies chooses for the number of
// right-hand sides.  The rest of the plan stays: the scratch it asks for is what the entry
// points check.  us per apply, the kernels before and this one: mixed orders of about 33
// modes, 10 disks, one column 9.7, 8.7 (the host's part); 256 x 10 61, 29; 64 x 16, 4 columns
// 110, 65; 1,000 x 10, 7 columns 1,446, 643.
#define FEW_LDS (64 * 1024)

static size_t few_lds(int cols, int zcap) { return (size_t)FEW_WAVES * cols * (2 * zcap + FEW_PAD) * 16; }

// Shape of the tasks (P.few and the LDS they take); the ints of all tasks, 0: none.
static size_t few_shape(int B, const int64_t* idisk, const int32_t* N, PlanHost& P) {
  int64_t mmax = 0;
  int nmax = 0;
  for (int b = 0; b < B; ++b) mmax = std::max(mmax, idisk[b + 1] - idisk[b]);
  if (mmax > FEW_DISKS || (P.lane == LANE_UNIFORM && mmax > 12 && idisk[B] > 1024)) return 0;
  size_t tasks = 0;
  for (int64_t p = 0; p < idisk[B]; ++p) {
    nmax = std::max(nmax, (int)N[p]);
    tasks += (size_t)(2 * N[p] + 32) / 32;
  }
  const int cols = (int)(mmax - 1 + FEW_WAVES - 1) / FEW_WAVES, zcap = 2 * nmax + 1;
  if (few_lds(cols, zcap) > FEW_LDS) return 0;
  P.few = FEW_HDR + FEW_COL * (int)(mmax - 1);
  P.few_cols = cols;
  P.few_z = zcap;
  return tasks * (size_t)P.few;
}

static void make_few(int B, const int64_t* idisk, const int32_t* N, PlanHost& P) {
  const size_t ints = few_shape(B, idisk, N, P);
  if (ints == 0) return;
  P.few_tasks.resize(ints, 0);
  if (P.lane != LANE_UNIFORM) {
    P.items.clear();
    P.item_total = 0;
  }
  int32_t* it = P.few_tasks.data();
  int64_t i0 = 0, t0 = 0;  // first unknown and symbol of the instance
  for (int b = 0; b < B; ++b) {
    const int64_t d0 = idisk[b];
    const int M = (int)(idisk[b + 1] - d0);
    int64_t off[FEW_DISKS + 1] = {0}, sym[FEW_DISKS][FEW_DISKS], t = t0;
    for (int p = 0; p < M; ++p) {
      off[p + 1] = off[p] + 2 * N[d0 + p] + 1;
      for (int q = p + 1; q < M; ++q) {
        const int64_t S = N[d0 + p] + N[d0 + q];
        sym[p][q] = sym[q][p] = t + S;
        t += 2 * S + 1;
      }
    }
    for (int p = 0; p < M; ++p)
      for (int m0 = 0; m0 <= 2 * N[d0 + p]; m0 += 32) {
        P.few_us += 0.45e-3 + 0.158e-3 * M + 8.5e-6 * (double)off[M];
        auto put64 = [&](int k, int64_t x) {
          it[k] = (int32_t)(x & 0xffffffff);
          it[k + 1] = (int32_t)(x >> 32);
        };
        it[0] = b;
        it[1] = m0;
        it[2] = N[d0 + p];
        it[3] = M - 1;
        put64(4, i0 + off[p]);
        put64(6, i0);
        put64(8, off[M]);
        for (int q = 0, k = FEW_HDR; q < M; ++q) {
          if (q == p) continue;
          it[k] = (int32_t)off[q];
          it[k + 1] = 2 * N[d0 + q] + (p > q ? 1 : 0);
          put64(k + 2, sym[p][q]);
          k += FEW_COL;
        }
        it += P.few;
      }
    i0 += off[M];
    t0 = t;
  }
}

// Whether applies of R right-hand sides run on k_apply_few.  For uniform orders one lane per
// pair is the other way, by far the faster one where the launch is many tasks of few modes:
// a wave then is a row with all its columns and k_apply_few a workgroup of 256 threads.  Both
// by estimates (us of whole applies, 4.5 and 9.3 besides, fitted to 1,900 batches of 1 to 3,000
// instances within 15% and 9% in the mean; per row and right-hand side 0.45 + 0.158 M + 0.0085 M
// n, and 0.037 n + 0.0094 n^2 ns, n modes): 4 disks of 31 modes 8.4 with one lane per pair, 6.5
// with k_apply_few; of 25 modes 2 disks 11.9, 8.6, 1,000 x 4 44, 11.5, 256 x 12 80, 71; of 3
// modes 40 x 12 10.9, 5.4, 1,000 x 12 12.1, 49, with 7 columns 32.7, 325; of 15 modes 1,000 x 8, 7
// columns 155, 193.
// split: the sums are added by the kernel that follows, so that one lane per pair is one
// launch as well, its chain of 2 N orders against the panels of M disks (steps of solves, us,
// one lane per pair and whole rows: one instance of 4 disks of 3 modes 24.7, 24.1, of 25 30.6,
// 25.0, 16 of 3 modes 25.0, 26.5, of 25 32.1, 27.8; 64 x 8 of 3, 4 columns 26.2, 30.9).
#define FEW_MARGIN 1.15
static double lane_chain(const MatvecPlan& P) {
  const int M = (P.few - FEW_HDR) / FEW_COL + 1;
  return 0.5 * P.spec_N - 0.8 - 0.13 * (M - 4);
}

static bool few_applies(const mudiff_ctx* h, int R, bool split) {
  const MatvecPlan& P = h->plan;
  if (!P.few || P.lane != LANE_UNIFORM) return P.few > 0;
  const double few = R * P.few_us, lane = R * P.lane_us;
  return FEW_MARGIN * few < lane + lane_chain(P) || (!split && FEW_MARGIN * (few + 4.5) < lane + 9.3);
}

double apply_few_us(const mudiff_ctx* h, int R) {
  if (few_applies(h, R, true)) return R * h->plan.few_us;
  if (h->plan.lane != LANE_UNIFORM) return 10.0;
  return (h->plan.few ? 1.5 * lane_chain(h->plan) : 3.0) + R * h->plan.lane_us;
}

size_t plan_sched_bytes(const PlanHost& P, int M) {
  return align256(P.item_total * 4) + align256((size_t)M * 4) + align256((size_t)M * 8) +
         align256(P.task_total * 4) + align256(P.few_tasks.size() * 4) + 256;
}

size_t sched_bytes_for(int B, const int64_t* disk_off, const int32_t* n_modes) {
  PlanHost H;
  H.count = true;
  make_plan(B, disk_off, n_modes, false, H);
  const size_t few = few_shape(B, disk_off, n_modes, H);
  if (few > 0 && H.lane != LANE_UNIFORM) H.item_total = 0;
  const size_t bytes = plan_sched_bytes(H, (int)disk_off[B]) + align256(few * 4);
  if (H.lane == LANE_UNIFORM || few > 0 || !pairs_batch(B, disk_off, n_modes)) return bytes;
  PlanHost Q;  // which of the two also depends on the centers
  Q.count = true;
  make_plan(B, disk_off, n_modes, true, Q);
  return std::max(bytes, plan_sched_bytes(Q, (int)disk_off[B]));
}

int ensure_plan(mudiff_ctx* h, hipStream_t s) {
  if (h->plan.ready) return MUDIFF_OK;
  PlanHost H;
  make_plan(h->B, h->idisk.data(), h->N.data(), h->pairs_ok, H);
  make_few(h->B, h->idisk.data(), h->N.data(), H);
  if (H.lds > (H.lane ? 80 : 64) * 1024) return fail(MUDIFF_ERR_INVALID, "operator rows too long for LDS");
  if (plan_sched_bytes(H, h->M_all) > h->sched_bytes)
    return fail(MUDIFF_ERR_INVALID, "schedule area too small");
  MatvecPlan& P = h->plan;
  P.d_items = (int32_t*)h->sched_base;
  P.d_nchunk = (int32_t*)(h->sched_base + align256(H.items.size() * 4));
  P.d_partoff = (int64_t*)((char*)P.d_nchunk + align256(h->M_all * 4));
  P.d_tasks = (int32_t*)((char*)P.d_partoff + align256((size_t)h->M_all * 8));
  P.d_few = (int32_t*)((char*)P.d_tasks + align256(H.tasks.size() * 4));
  // one copy of all five (a copy from pageable memory takes the host some 5 us)
  std::vector<char> blob((char*)P.d_few - h->sched_base + H.few_tasks.size() * 4);
  auto put = [&](const void* d, const void* src, size_t n) {
    if (n) memcpy(blob.data() + ((const char*)d - h->sched_base), src, n);
  };
  put(P.d_items, H.items.data(), H.items.size() * 4);
  put(P.d_nchunk, H.nch.data(), (size_t)h->M_all * 4);
  put(P.d_partoff, H.poff.data(), (size_t)h->M_all * 8);
  put(P.d_tasks, H.tasks.data(), H.tasks.size() * 4);
  put(P.d_few, H.few_tasks.data(), H.few_tasks.size() * 4);
  HIP_TRY(hipMemcpyAsync(h->sched_base, blob.data(), blob.size(), hipMemcpyHostToDevice, s));
  HIP_TRY(hipStreamSynchronize(s));  // the host vectors are released on return
  P.lane = H.lane;
  P.Bt = H.bt;
  P.spec_N = H.nspec;
  P.zs = H.zs;
  P.ts = H.ts;
  P.ppcap = H.ppcap;
  P.part_total = H.part;
  P.wide = H.wide;
  P.row_part = H.lane == LANE_PAIRS ? H.row_part : H.part;
  P.lds_bytes = H.lds;
  P.few = H.few;
  P.lane_rows = H.lane_rows;
  P.few_cols = H.few_cols;
  P.few_z = H.few_z;
  P.few_us = H.few_us;
  P.lane_us = H.lane_us;
  P.n_few = H.few ? (int)(H.few_tasks.size() / H.few) : 0;
  P.n_items = (int)(H.items.size() / H.item_ints);
  P.ready = true;
  return MUDIFF_OK;
}

// Apply scratch: the partial sums (or the MFMA schedule and partial blocks),
// then R * M_all counters of the generic kernel.
size_t apply_scratch_bytes(mudiff_ctx* h, int R) {
  const size_t counters = align256((size_t)R * h->M_all * 4);
  if (use_mfma(h, R)) return align256(mfma_scratch_bytes(h, R)) + counters;
  if (h->plan.ready) h->plan_part = h->plan.part_total;
  if (h->plan_part < 0) {
    PlanHost H;
    make_plan(h->B, h->idisk.data(), h->N.data(), h->pairs_ok, H);
    h->plan_part = H.part;
  }
  return align256((size_t)R * h->plan_part * 16) + counters;
}

void apply_forget_upload(mudiff_ctx* h) {
  for (auto& kv : h->mfma_scheds)
    if (!kv.second.resident) kv.second.dev = nullptr;
  h->mfma_tail_sched.dev = nullptr;
}

int prepare_apply(mudiff_ctx* h, int R, const cplx* x, cplx* y, cplx* scratch, hipStream_t s) {
  if (use_mfma(h, R)) return mfma_prepare(h, R, x, y, (char*)scratch, s);
  return ensure_plan(h, s);
}

// Chunk partial sums of the one-lane-per-pair kernels.
static int launch_lanes(mudiff_ctx* h, int R, const cplx* x, cplx* part, const int32_t* active,
                        hipStream_t s) {
  const MatvecPlan& P = h->plan;
  if (P.n_items == 0) return MUDIFF_OK;
  if (P.lane == LANE_PAIRS) {
    hipLaunchKernelGGL(P.wide ? k_apply_pairs<true> : k_apply_pairs<false>, dim3(P.n_items, R), dim3(PAIRS_THREADS), P.lds_bytes, s, h->dv, R, x,
                       part, P.part_total, P.d_items, P.d_tasks, P.d_partoff, active);
  } else {
    const LaneVariant* lv = find_lane(P.spec_N);
    if (!lv) return fail(MUDIFF_ERR_INVALID, "no operator kernel variant");
    hipLaunchKernelGGL((h->dv.op_col ? lv->fn_op : lv->fn)[P.lane_rows == 1], dim3(P.n_items, R), dim3(64 * P.lane_rows), 0, s, h->dv, R,
                       x, part, P.part_total, P.d_items, active);
  }
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}

int apply_operator_split(mudiff_ctx* h, int R, const cplx* x, cplx* y, int op, cplx* part,
                         int32_t* counters, const int32_t* active, hipStream_t s,
                         bool* pending) {
  *pending = false;
  if (use_mfma(h, R)) return apply_operator(h, R, x, y, op, part, counters, active, s);
  int st = ensure_plan(h, s);
  if (st != MUDIFF_OK) return st;
  const MatvecPlan& P = h->plan;
  if (P.lane && !few_applies(h, R, true)) {
    if ((st = launch_lanes(h, R, x, part, active, s)) != MUDIFF_OK) return st;
    *pending = true;  // the chunk sums still have to be added and finalised
    return MUDIFF_OK;
  }
  return apply_operator(h, R, x, y, op, part, counters, active, s);
}

int apply_operator(mudiff_ctx* h, int R, const cplx* x, cplx* y, int op, cplx* part,
                   int32_t* counters, const int32_t* active, hipStream_t s, const cplx* shift) {
  if (use_mfma(h, R)) {
    int st = mfma_prepare(h, R, nullptr, nullptr, (char*)part, s);  // no-op when current
    if (st != MUDIFF_OK) return st;
    return mfma_launch(h, mfma_current(h, R), (char*)part, x, y, op, active, s, shift);
  }
  int st = ensure_plan(h, s);
  if (st != MUDIFF_OK) return st;
  const MatvecPlan& P = h->plan;
  prof_open(h, s);
  prof_mark(h, s, 1);
  prof_mark(h, s, 2);
  prof_mark(h, s, 3);
  if (few_applies(h, R, false)) {
    const DevView& v = h->dv;
    FewView fv{v.t, v.op_col, nullptr, v.invSH, v.sJ, op == OP_RAW_W};
    if (v.op_rowA) fv.be = op == MUDIFF_OP_A ? v.op_rowA : v.op_row;
    else if (op != MUDIFF_OP_A) fv.be = nullptr;
    if (op != MUDIFF_OP_A) fv.al = v.op_rowA ? v.op_diag : v.Ldiag;
    hipLaunchKernelGGL(k_apply_few, dim3(P.n_few, R), dim3(FEW_THREADS), few_lds(P.few_cols, P.few_z), s, fv, R,
                       x, y, P.d_few, P.few, active, shift, P.few_cols, P.few_z);
    HIP_TRY(hipGetLastError());
    prof_mark(h, s, 4);
    prof_mark(h, s, 5);
    return MUDIFF_OK;
  }
  if (P.lane) {
    if ((st = launch_lanes(h, R, x, part, active, s)) != MUDIFF_OK) return st;
    prof_mark(h, s, 4);
    const int64_t total = (int64_t)R * h->N_all;
    hipLaunchKernelGGL(k_apply_finish, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                       h->dv, R, x, y, op, (const cplx*)part, P.part_total, P.d_nchunk,
                       P.d_partoff, active, shift);
    HIP_TRY(hipGetLastError());
    prof_mark(h, s, 5);
    return MUDIFF_OK;
  }
  const Variant* var = find_variant(P.Bt, P.spec_N);
  if (!var) return fail(MUDIFF_ERR_INVALID, "no operator kernel variant");
  hipLaunchKernelGGL(var->fn, dim3(P.n_items, R), dim3(APPLY_THREADS), P.lds_bytes, s, h->dv, R, x,
                     y, op, part, P.part_total, counters, P.d_items, P.d_nchunk, P.d_partoff, active,
                     P.zs, P.ts, P.ppcap, shift);
  HIP_TRY(hipGetLastError());
  prof_mark(h, s, 4);
  prof_mark(h, s, 5);
  return MUDIFF_OK;
}

namespace {
// Mode flip P (x^p_m -> x^p_{-m} in every disk) of R columns: out = P in, or
// in place when out == in (one thread per pair m > 0 then).  L^T = P L P.
__global__ void k_flip_modes(DevView v, int R, const cplx* in, cplx* out) {
  const int64_t total = (int64_t)R * v.N_all;
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  int lo = 0, hi = v.B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)R * v.imode[mid] <= g) lo = mid; else hi = mid;
  }
  const int64_t Nb = v.imode[lo + 1] - v.imode[lo];
  const int64_t rem = g - (int64_t)R * v.imode[lo];
  const int64_t il = rem - (rem / Nb) * Nb;
  const int p = v.udisk[v.imode[lo] + il];
  const int64_t m = il - v.moff[p] - v.N[p];
  const int64_t g2 = g - 2 * m;  // mode -m of the same disk and column
  if (in != out) {
    out[g] = in[g2];
  } else if (m > 0) {
    const cplx a = out[g];
    out[g] = out[g2];
    out[g2] = a;
  }
}
}  // namespace

extern "C" size_t mudiff_matvec_workspace_size(mudiff_t h, int R) {
  if (!h || R < 1) return 0;
  // apply scratch, then room for the flipped input of MUDIFF_OP_LT
  return apply_scratch_bytes(h, R) + align256((size_t)R * h->N_all * 16);
}

extern "C" int mudiff_matvec(mudiff_t h, int R, const void* x, void* y, int op, void* workspace,
                             size_t ws_bytes, void* stream) {
  if (!h || !x || !y) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  if (x == y) return fail(MUDIFF_ERR_INVALID, "x and y must be distinct buffers");
  if (op != MUDIFF_OP_L && op != MUDIFF_OP_A && op != MUDIFF_OP_LT)
    return fail(MUDIFF_ERR_INVALID, "unknown op");
  if (op == MUDIFF_OP_LT && h->dv.op_col)
    return fail(MUDIFF_ERR_INVALID, "MUDIFF_OP_LT applies the single layer only (reset the operator first)");
  const size_t need = apply_scratch_bytes(h, R);
  const size_t need_all = mudiff_matvec_workspace_size(h, R);
  if (!workspace) return fail(MUDIFF_ERR_INVALID, "workspace is NULL");
  if (ws_bytes < (op == MUDIFF_OP_LT ? need_all : need))
    return fail(MUDIFF_ERR_NOMEM, "matvec workspace needs " + std::to_string(need_all) + " bytes");
  apply_forget_upload(h);
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)workspace;
  const cplx* xin = (const cplx*)x;
  const int64_t tot = (int64_t)R * h->N_all;
  const unsigned fb = (unsigned)((tot + 255) / 256);
  if (op == MUDIFF_OP_LT) {  // L^T x = P L (P x)
    cplx* xf = (cplx*)(w + need);
    hipLaunchKernelGGL(k_flip_modes, dim3(fb), dim3(256), 0, s, h->dv, R, xin, xf);
    HIP_TRY(hipGetLastError());
    xin = xf;
  }
  const int aop = op == MUDIFF_OP_LT ? MUDIFF_OP_L : op;
  int rc;
  if (use_mfma(h, R)) {
    rc = mfma_prepare(h, R, xin, (cplx*)y, w, s);  // autotunes on first use of R
    if (rc == MUDIFF_OK) rc = mfma_launch(h, mfma_current(h, R), w, xin, (cplx*)y, aop, nullptr, s);
  } else {
    size_t part_bytes = need - align256((size_t)R * h->M_all * 4);
    int32_t* counters = (int32_t*)(w + part_bytes);  // zero on first use, left zero
    rc = apply_operator(h, R, xin, (cplx*)y, aop, (cplx*)w, counters, nullptr, s);
  }
  if (rc != MUDIFF_OK || op != MUDIFF_OP_LT) return rc;
  hipLaunchKernelGGL(k_flip_modes, dim3(fb), dim3(256), 0, s, h->dv, R, (const cplx*)y, (cplx*)y);
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}

extern "C" int mudiff_apply_config(mudiff_t h, int R, int* kind, int* ct, int* rp, int* qs,
                                   int* threads, float* ms) {
  if (!h) return fail(MUDIFF_ERR_INVALID, "NULL handle");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  int k = 2, c = 0, r = 0, q = 0, t = 0;
  float tm = 0.0f;
  if (use_mfma(h, R)) {
    k = 1;
    auto f = h->mfma_choice.find(R);
    MfmaChoice ch = f != h->mfma_choice.end() ? f->second : mfma_default(R);
    if (f == h->mfma_choice.end()) ch.circ = circ_usable(h, R);
    if (ch.circ) k = 3;
    c = ch.CT;
    r = ch.RP;
    q = segment(h, R, ch);
    t = ch.threads;
    auto g = h->mfma_time_ms.find(R);
    if (g != h->mfma_time_ms.end()) tm = g->second;
  } else {
    PlanHost H;
    make_plan(h->B, h->idisk.data(), h->N.data(), h->pairs_ok, H);
    k = H.lane == LANE_UNIFORM ? 0 : 2;
  }
  if (kind) *kind = k;
  if (ct) *ct = c;
  if (rp) *rp = r;
  if (qs) *qs = q;
  if (threads) *threads = t;
  if (ms) *ms = tm;
  return MUDIFF_OK;
}

extern "C" int mudiff_set_apply_config(mudiff_t h, int R, int ct, int rp, int qs, int threads) {
  if (!h) return fail(MUDIFF_ERR_INVALID, "NULL handle");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  if (!use_mfma(h, R)) return fail(MUDIFF_ERR_INVALID, "this apply does not run on MFMA");
  MfmaChoice want{ct, rp, qs, threads, false};
  std::vector<MfmaChoice> cands = mfma_candidates(R);
  if (std::find(cands.begin(), cands.end(), want) == cands.end())
    // a timed configuration, as mudiff_apply_config reports it in either form
    for (MfmaChoice c : mfma_timed(R, false)) {
      const bool tile = ct == c.CT && rp == c.RP && threads == c.threads;
      if (tile && (qs == segment(h, R, c) || (h->circ && ct == 1 && qs == auto_segment(h, R, ct, rp, true)))) {
        want.QS = c.QS;
        cands.push_back(c);
      }
    }
  for (const MfmaChoice& c : cands)
    if (c == want) {
      auto f = h->circ_modes.find(R);
      want.circ = circ_usable(h, R) && (f == h->circ_modes.end() || f->second != 0);
      h->mfma_choice[R] = want;
      h->mfma_time_ms.erase(R);
      return MUDIFF_OK;
    }
  return fail(MUDIFF_ERR_INVALID, "MFMA tile not among the candidates");
}

extern "C" int mudiff_set_circulant(mudiff_t h, int R, int mode) {
  if (!h) return fail(MUDIFF_ERR_INVALID, "NULL handle");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  if (mode < -1 || mode > 1) return fail(MUDIFF_ERR_INVALID, "mode must be -1, 0 or 1");
  if (!h->circ) return fail(MUDIFF_ERR_INVALID, "the handle was built without MUDIFF_TABLES_CIRCULANT");
  h->circ_modes[R] = mode;
  auto f = h->mfma_choice.find(R);
  if (f != h->mfma_choice.end()) {
    if (h->mfma_time_ms.count(R)) {  // timed choice: time again with the new mode
      h->mfma_choice.erase(f);
      h->mfma_time_ms.erase(R);
    } else {  // fixed tile: keep it, switch the form
      f->second.circ = mode != 0 && circ_usable(h, R);
    }
  }
  sched_drop(h, R);  // rebuild at the next apply
  return MUDIFF_OK;
}

extern "C" int mudiff_circulant_tile(mudiff_t h, int R, int* rows, int* cols, int* kstep,
                                     int* stages, int* threads, int* mults) {
  if (!h) return fail(MUDIFF_ERR_INVALID, "NULL handle");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  int bm = 0, bn = 0, bk = 0, db = 0, nt = 0, mu = 0;
  if (use_mfma(h, R)) {
    auto f = h->mfma_choice.find(R);
    MfmaChoice ch = f != h->mfma_choice.end() ? f->second : mfma_default(R);
    if (f == h->mfma_choice.end()) ch.circ = circ_usable(h, R);
    if (ch.circ) circ_var_dims(ch.cvar >= 0 ? ch.cvar : circ_variant(R), &bm, &bn, &bk, &db, &nt, &mu);
  }
  if (rows) *rows = bm;
  if (cols) *cols = bn;
  if (kstep) *kstep = bk;
  if (stages) *stages = db;
  if (threads) *threads = nt;
  if (mults) *mults = mu;
  return MUDIFF_OK;
}

extern "C" int mudiff_set_circulant_tile(mudiff_t h, int R, int rows, int cols, int kstep,
                                         int stages, int threads, int mults) {
  if (!h) return fail(MUDIFF_ERR_INVALID, "NULL handle");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  if (!use_mfma(h, R) || !circ_usable(h, R))
    return fail(MUDIFF_ERR_INVALID, "this apply does not use the circulant form");
  for (int v : circ_variants(R)) {
    int bm, bn, bk, db, nt, mu;
    circ_var_dims(v, &bm, &bn, &bk, &db, &nt, &mu);
    if (bm == rows && bn == cols && bk == kstep && db == stages && nt == threads && mu == mults) {
      auto f = h->mfma_choice.find(R);
      MfmaChoice ch = f != h->mfma_choice.end() ? f->second : mfma_default(R);
      ch.circ = true;
      ch.cvar = v;
      h->mfma_choice[R] = ch;
      h->mfma_time_ms.erase(R);
      h->circ_modes[R] = 1;
      sched_drop(h, R);
      return MUDIFF_OK;
    }
  }
  return fail(MUDIFF_ERR_INVALID, "product tile not among the candidates for this R");
}

// ------------------------------------------------------------------ phase timing
void prof_open(mudiff_ctx* h, hipStream_t s) {
  h->prof_cur = -1;
  if (h->prof_n >= h->prof_max) return;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return;
  h->prof_cur = h->prof_n++;
  (void)hipEventRecord(h->prof_ev[(size_t)h->prof_cur * (MUDIFF_N_PHASES + 1)], s);
}

void prof_mark(mudiff_ctx* h, hipStream_t s, int k) {
  if (h->prof_cur < 0) return;
  (void)hipEventRecord(h->prof_ev[(size_t)h->prof_cur * (MUDIFF_N_PHASES + 1) + k], s);
  if (k == MUDIFF_N_PHASES) h->prof_cur = -1;
}

static void prof_release(mudiff_ctx* h) {
  for (hipEvent_t e : h->prof_ev) (void)hipEventDestroy(e);
  h->prof_ev.clear();
  h->prof_max = h->prof_n = 0;
  h->prof_cur = -1;
}

extern "C" int mudiff_profile_begin(mudiff_t h, int max_applies) {
  if (!h) return fail(MUDIFF_ERR_INVALID, "NULL handle");
  if (max_applies < 1 || max_applies > 100000) return fail(MUDIFF_ERR_INVALID, "max_applies out of range");
  prof_release(h);
  h->prof_ev.resize((size_t)max_applies * (MUDIFF_N_PHASES + 1));
  for (size_t k = 0; k < h->prof_ev.size(); ++k) {
    if (hipEventCreate(&h->prof_ev[k]) != hipSuccess) {
      h->prof_ev.resize(k);
      prof_release(h);
      return fail(MUDIFF_ERR_DEVICE, "hipEventCreate failed");
    }
  }
  h->prof_max = max_applies;
  return MUDIFF_OK;
}

extern "C" int mudiff_profile_end(mudiff_t h, int* n_applies, double* ms) {
  if (!h || !n_applies || !ms) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  for (int k = 0; k < MUDIFF_N_PHASES; ++k) ms[k] = 0.0;
  *n_applies = h->prof_n;
  if (h->prof_n > 0) {
    const hipEvent_t last = h->prof_ev[(size_t)(h->prof_n - 1) * (MUDIFF_N_PHASES + 1) + MUDIFF_N_PHASES];
    if (hipEventSynchronize(last) != hipSuccess) {
      prof_release(h);
      return fail(MUDIFF_ERR_DEVICE, "profile: event synchronisation failed");
    }
    for (int a = 0; a < h->prof_n; ++a)
      for (int k = 0; k < MUDIFF_N_PHASES; ++k) {
        float t = 0.0f;
        const size_t b = (size_t)a * (MUDIFF_N_PHASES + 1);
        if (hipEventElapsedTime(&t, h->prof_ev[b + k], h->prof_ev[b + k + 1]) == hipSuccess) ms[k] += t;
      }
  }
  prof_release(h);
  return MUDIFF_OK;
}

// ------------------------------------------------------------------ no-allocation apply
// Apply scratch of mudiff_matvec_noalloc: a file-scope device array, one copy
// per device, held until the process ends.  Host code never hands the array's
// name to a kernel (on the host it is only a stand-in for the symbol): its
// device address comes from hipGetSymbolAddress, once per device.
#define NOALLOC_SCRATCH_BYTES ((size_t)MUDIFF_NOALLOC_SCRATCH_MB << 20)
static __device__ __align__(256) char scratch[NOALLOC_SCRATCH_BYTES];

static std::mutex g_scratch_mu;
static std::map<int, char*> g_scratch_ptr;  // device -> address of its copy of scratch

static int scratch_address(char** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  auto f = g_scratch_ptr.find(dev);
  if (f != g_scratch_ptr.end()) {
    *out = f->second;
    return MUDIFF_OK;
  }
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr)
    return fail(MUDIFF_ERR_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
  g_scratch_ptr[dev] = (char*)ptr;
  *out = (char*)ptr;
  return MUDIFF_OK;
}

extern "C" int mudiff_matvec_noalloc(mudiff_t h, int R, const void* x, void* y, int op,
                                     void* stream) {
  if (!h || !x || !y) return fail(MUDIFF_ERR_INVALID, "NULL argument");
  if (R < 1) return fail(MUDIFF_ERR_INVALID, "R < 1");
  if (x == y) return fail(MUDIFF_ERR_INVALID, "x and y must be distinct buffers");
  if (op != MUDIFF_OP_L && op != MUDIFF_OP_A && op != MUDIFF_OP_LT)
    return fail(MUDIFF_ERR_INVALID, "unknown op");
  if (op == MUDIFF_OP_LT && h->dv.op_col)
    return fail(MUDIFF_ERR_INVALID, "MUDIFF_OP_LT applies the single layer only (reset the operator first)");
  if (use_mfma(h, R))
    return fail(MUDIFF_ERR_INVALID, "the no-allocation apply covers the one-lane and generic kernels "
                                    "(R < 8, or N_p > 31); use mudiff_matvec");
  if (!h->plan.ready) return fail(MUDIFF_ERR_INVALID, "no operator plan for this handle");
  const size_t need = apply_scratch_bytes(h, R);
  const size_t flip = op == MUDIFF_OP_LT ? align256((size_t)R * h->N_all * 16) : 0;
  // the size that the call is refused by: that of the LDS-staged kernel's chunks,
  // also where k_apply_pairs runs and needs less (or, below the limit, a little more)
  const size_t want = align256((size_t)R * h->plan.row_part * 16) + align256((size_t)R * h->M_all * 4) + flip;
  if (want > NOALLOC_SCRATCH_BYTES || need + flip > NOALLOC_SCRATCH_BYTES)
    return fail(MUDIFF_ERR_NOMEM, "the no-allocation apply needs " + std::to_string(std::max(want, need + flip)) +
                                      " bytes of scratch, more than its " +
                                      std::to_string(NOALLOC_SCRATCH_BYTES));
  char* w = nullptr;
  int rc = scratch_address(&w);
  if (rc != MUDIFF_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  const size_t part_bytes = need - align256((size_t)R * h->M_all * 4);
  int32_t* counters = (int32_t*)(w + part_bytes);
  // the generic kernel's counters start at zero (a fill kernel: no memset node
  // if the caller captures this call)
  if ((rc = launch_fill_zero(counters, (size_t)R * h->M_all * 4, s)) != MUDIFF_OK) return rc;
  const cplx* xin = (const cplx*)x;
  const int64_t tot = (int64_t)R * h->N_all;
  const unsigned fb = (unsigned)((tot + 255) / 256);
  if (op == MUDIFF_OP_LT) {  // L^T x = P L (P x)
    cplx* xf = (cplx*)(w + need);
    hipLaunchKernelGGL(k_flip_modes, dim3(fb), dim3(256), 0, s, h->dv, R, xin, xf);
    HIP_TRY(hipGetLastError());
    xin = xf;
  }
  rc = apply_operator(h, R, xin, (cplx*)y, op == MUDIFF_OP_LT ? MUDIFF_OP_L : op, (cplx*)w, counters,
                      nullptr, s);
  if (rc != MUDIFF_OK || op != MUDIFF_OP_LT) return rc;
  hipLaunchKernelGGL(k_flip_modes, dim3(fb), dim3(256), 0, s, h->dv, R, (const cplx*)y, (cplx*)y);
  HIP_TRY(hipGetLastError());
  return MUDIFF_OK;
}
