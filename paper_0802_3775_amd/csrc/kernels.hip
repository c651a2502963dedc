// gfx950 kernels of libfdtd beside the fused step (step.hip): the passes of the
// density-matrix gain medium (a ground level and three degenerate upper levels,
// held at the cell centre), the running-DFT flux update, the integer voxelizer,
// the sums of reads and small helpers.
//
// Method: C. Conti and A. Fratalocchi, arXiv:0802.3775 — Yee FDTD with absorbing
// walls in a disordered inverted opal, pumped gain medium seeded by a stochastic
// source, transmitted power T(t) (sections "Sample and numerical approach" and
// "Dynamical diffusion and localization").
//
#include "fd_device.h"

#include <hip/hip_ext.h>

#include <mutex>

using namespace fdk;

namespace {

// ------------------------------------------------- density-matrix gain cells
// State of one cell in registers: upper-level populations rho_kk as (hi, lo)
// pairs, the ground-upper coherences rho_0k = cr + i ci and the upper-upper
// coherences rho_12, rho_13, rho_23 = xr + i xi.  The trace is fixed at 1, so
// rho_00 = 1 - sum rho_kk (the real su(4) coordinates of the paper's model,
// with the diagonal held as level populations).
struct Cz {
  float r, i;
};
__device__ __forceinline__ Cz zm(Cz a, Cz b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__device__ __forceinline__ Cz zc(Cz a) { return {a.r, -a.i}; }
__device__ __forceinline__ Cz za(Cz a, Cz b) { return {a.r + b.r, a.i + b.i}; }
__device__ __forceinline__ Cz zs(Cz a, float s) { return {a.r * s, a.i * s}; }

// Half-step relaxation R(dt/2): exact flow of T1 decay, pump and T2 dephasing.
// p: populations (updated), inc: their accumulated increments.
__device__ __forceinline__ void dm_relax(const fd_mat& mt, float p[3], float inc[3], Cz c[3], Cz x[3]) {
  const float e = (p[0] + p[1]) + p[2];
  const float de3 = (mt.beinf - e) * mt.bg1m * (1.0f / 3.0f);
  const float e3 = e * (1.0f / 3.0f);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float d = de3 - (p[k] - e3) * mt.bh1m;
    inc[k] += d;
    p[k] += d;
    c[k] = zs(c[k], mt.bf2);
    x[k] = zs(x[k], mt.bf2);
  }
}

// Cayley step C(E): rho -> V rho V^+, V = (I + i tau H')^{-1}(I - i tau H'),
// tau = dt/2.  In closed form (D = 1 + tau^2 |E|^2 + i w' tau):
//   V_00 = (1 + i w' tau - tau^2 |E|^2) / D,  V_0k = V_k0 = 2 i tau E_k / D,
//   V_kl = r delta_kl + g E_k E_l,  r = (1 - i w' tau)/(1 + i w' tau),
//   g = -2 tau^2 / (D (1 + i w' tau)).
// With w_k = rho_k0, y = X^T E (X the upper block), s = E.w, q = E.X.E:
//   T_k0 = E_k (b p00 + g s) + r w_k,  z_k = E_k (b s* + g q) + r y_k*,
//   rho'_k0 = a* T_k0 + b* z_k,
//   rho'_kl = X_kl + r* E_k (b w_l* + g y_l) + E_l (b* T_k0 + g* z_k)
// (a = V_00, b = V_0k / E_k).  FULL = false stops after rho'_k0 (the predictor).
template <bool FULL>
__device__ __forceinline__ void dm_cayley(const fd_mat& mt, const float E[3], float p[3], float inc[3], Cz c[3],
                                          Cz x[3]) {
  const float tau = mt.btau;
  const float t2e = tau * tau * fmaf(E[0], E[0], fmaf(E[1], E[1], E[2] * E[2]));
  const float dr = 1.0f + t2e, di = mt.bwt;
  const float inv = 1.0f / fmaf(dr, dr, di * di);
  const Cz iD = {dr * inv, -di * inv};
  const Cz al = zm({1.0f - t2e, di}, iD);
  const Cz be = {-2.0f * tau * iD.i, 2.0f * tau * iD.r};
  const Cz ga = zs(zm(iD, {mt.bc1r, mt.bc1i}), -2.0f * tau * tau);
  const Cz rr = {mt.brr, mt.bri};
  const float p00 = 1.0f - ((p[0] + p[1]) + p[2]);
  Cz w[3], y[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) w[k] = zc(c[k]);
  // upper block: X_kk = p_k, X_01 = x0, X_02 = x1, X_12 = x2, X_lk = X_kl*
  y[0] = za(za({E[0] * p[0], 0.0f}, zs(zc(x[0]), E[1])), zs(zc(x[1]), E[2]));
  y[1] = za(za(zs(x[0], E[0]), {E[1] * p[1], 0.0f}), zs(zc(x[2]), E[2]));
  y[2] = za(za(zs(x[1], E[0]), zs(x[2], E[1])), {E[2] * p[2], 0.0f});
  const Cz sv = za(za(zs(w[0], E[0]), zs(w[1], E[1])), zs(w[2], E[2]));
  const float qv = fmaf(E[0], y[0].r, fmaf(E[1], y[1].r, E[2] * y[2].r));
  const Cz u0 = za(zs(be, p00), zm(ga, sv));
  const Cz u1 = za(zm(be, zc(sv)), zs(ga, qv));
  Cz T[3], z[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T[k] = za(zs(u0, E[k]), zm(rr, w[k]));
    z[k] = za(zs(u1, E[k]), zm(rr, zc(y[k])));
    c[k] = zc(za(zm(zc(al), T[k]), zm(zc(be), z[k])));  // rho'_0k = (rho'_k0)*
  }
  if (!FULL) return;
  Cz a[3], b[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    a[k] = zm(zc(rr), za(zm(be, zc(w[k])), zm(ga, y[k])));  // r* (b w_k* + g y_k)
    b[k] = za(zm(zc(be), T[k]), zm(zc(ga), z[k]));
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float d = E[k] * (a[k].r + b[k].r);
    inc[k] += d;
    p[k] += d;
  }
  x[0] = za(x[0], za(zs(a[1], E[0]), zs(b[0], E[1])));
  x[1] = za(x[1], za(zs(a[2], E[0]), zs(b[0], E[2])));
  x[2] = za(x[2], za(zs(a[2], E[1]), zs(b[1], E[2])));
}

// ------------------------------------------------------------- flux DFT
// Running DFT of the flux-plane fields (E^n at the plane, H^{n+1/2} averaged
// onto it), sampled every decim steps.  The step kernels store the samples in a
// ring of FD_DFT_RING planes; a launch after the step that fills it adds the whole
// ring to the FP64 accumulators, so each accumulator (16 bytes per point, component and
// frequency) is read and written once per ring rather than once per sample.
// The flush is a small dense product (samples x weights e^{i 2 pi f t_m});
// the weights of one frequency block are tabulated in LDS.

// complex product and integer power (square and multiply)
__device__ __forceinline__ void cmul(double ar, double ai, double br, double bi, double& cr, double& ci) {
  cr = ar * br - ai * bi;
  ci = ar * bi + ai * br;
}
__device__ __forceinline__ void cpow(double br, double bi, long long e, double& rr, double& ri) {
  rr = 1.0;
  ri = 0.0;
  while (e > 0) {
    if (e & 1) cmul(rr, ri, br, bi, rr, ri);
    cmul(br, bi, br, bi, br, bi);
    e >>= 1;
  }
}

// out = in + sum over the samples m < count (sample index first + m, step
// (first + m) decim) of v_m e^{i 2 pi f t_m} decim dt, for the work unit's
// FD_DFT_PTS points (one per lane), 4 components (one per wave) and FD_DFT_QB
// frequencies.  first is a multiple of FD_DFT_RING; the weights are
// built from three unit phasors per frequency set up on the host (a ring, one
// sample and half a step of rotation): e^{i 2 pi f t_m} = R^(first/RING) S^m,
// and H samples carry the extra half step.
__device__ void dft_flush(const cdesc* d, int fl, int q0, int p0, long long first, int count, const gd* in, gd* out,
                          double (*tab)[FD_DFT_RING][4], double (*base)[4], float (*samp)[FD_DFT_RING][64]) {
  const int nf = d->flux_nf[fl], plane = d->plane, decim = d->flux_decim[fl];
  const double dt = d->dt;
  const gd* rot = G((const double*)d->flux_rot[fl]);  // [nf][6]: R, S, half step
  if (threadIdx.x < FD_DFT_QB) {
    const int q = q0 + (int)threadIdx.x;
    double br = 1.0, bi = 0.0, hr = 1.0, hi = 0.0;
    if (q < nf) {
      cpow(rot[6 * q], rot[6 * q + 1], first / FD_DFT_RING, br, bi);
      hr = rot[6 * q + 4];
      hi = rot[6 * q + 5];
    }
    base[threadIdx.x][0] = br;
    base[threadIdx.x][1] = bi;
    base[threadIdx.x][2] = hr;
    base[threadIdx.x][3] = hi;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < FD_DFT_QB * FD_DFT_RING; idx += blockDim.x) {
    const int qq = idx / FD_DFT_RING, m = idx % FD_DFT_RING;
    const int q = q0 + qq;
    double ce = 0.0, se = 0.0, chh = 0.0, shh = 0.0;
    if (q < nf && m < count) {
      double sr, si;
      cpow(rot[6 * q + 2], rot[6 * q + 3], m, sr, si);
      const double* b0 = base[qq];
      cmul(b0[0], b0[1], sr, si, ce, se);
      cmul(ce, se, b0[2], b0[3], chh, shh);
    }
    tab[qq][m][0] = ce;
    tab[qq][m][1] = se;
    tab[qq][m][2] = chh;
    tab[qq][m][3] = shh;
  }
  __syncthreads();
  const gf* ring = G((const float*)d->flux_ring[fl]);
  const double w = (double)decim * dt;
  const int lane = threadIdx.x & 63;
  const int p = p0 + lane;
  if (p >= plane) return;
  const int wv = threadIdx.x >> 6;
  for (int c = wv; c < 4; c += blockDim.x >> 6) {  // one component per wave
    // the wave's samples go to LDS (8 loads in flight at a time); samples
    // m >= count have zero weight but must be finite
    float* sm = samp[wv][0];
    for (int m0 = 0; m0 < FD_DFT_RING; m0 += 8) {
      float v8[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int m = m0 + u;
        v8[u] = ring[((size_t)(m < count ? m : 0) * 4 + c) * plane + p];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) sm[(m0 + u) * 64 + lane] = v8[u];
    }
    // the block's sums, loaded ahead of the products
    const int nq = min(FD_DFT_QB, nf - q0);
    double ar[FD_DFT_QB], ai[FD_DFT_QB], re[FD_DFT_QB], im[FD_DFT_QB];
#pragma unroll
    for (int qq = 0; qq < FD_DFT_QB; ++qq) {
      const size_t at = 2 * (((size_t)c * nf + q0 + (qq < nq ? qq : 0)) * plane + p);
      ar[qq] = in[at];
      ai[qq] = in[at + 1];
      re[qq] = im[qq] = 0.0;
    }
    const int ph = c < 2 ? 0 : 2;
#pragma unroll 2
    for (int m = 0; m < FD_DFT_RING; ++m) {
      const double v = (double)sm[m * 64 + lane];
#pragma unroll
      for (int qq = 0; qq < FD_DFT_QB; ++qq) {
        re[qq] = fma(v, tab[qq][m][ph], re[qq]);
        im[qq] = fma(v, tab[qq][m][ph + 1], im[qq]);
      }
    }
#pragma unroll
    for (int qq = 0; qq < FD_DFT_QB; ++qq) {
      if (qq < nq) {
        const size_t at = 2 * (((size_t)c * nf + q0 + qq) * plane + p);
        out[at] = ar[qq] + re[qq] * w;
        out[at + 1] = ai[qq] + im[qq] * w;
      }
    }
  }
}

// In the step sequence, after the step whose sample fills a realization's ring:
// add the ring to the sums (units of planes whose ring is not full return).
__global__ __launch_bounds__(256) void dft_kernel(const fd_dft_tile* __restrict__ tiles, int s) {
  __shared__ double tab[FD_DFT_QB][FD_DFT_RING][4];
  __shared__ double base[FD_DFT_QB][4];
  __shared__ float samp[4][FD_DFT_RING][64];
  const fd_dft_tile t = tiles[blockIdx.x];
  const cdesc* d = (const cdesc*)t.d;
  const int fl = t.flux;
  if (d->flux_nf[fl] == 0) return;
  const long long n = d->step + s;
  const int decim = d->flux_decim[fl];
  const long long si = n / decim;
  if (si * decim != n || si % FD_DFT_RING != FD_DFT_RING - 1) return;
  gd* acc = G(d->flux_acc[fl]);
  dft_flush(d, fl, t.q0, t.p0, si - (FD_DFT_RING - 1), FD_DFT_RING, acc, acc, tab, base, samp);
}

// For reads: flux_prev = flux_acc + the count samples waiting in the ring
// (sample indices first ...), for flux plane fl; the sums themselves are kept.
__global__ __launch_bounds__(256) void dft_preview_kernel(const fd_dft_tile* __restrict__ tiles, int fl,
                                                          long long first, int count) {
  __shared__ double tab[FD_DFT_QB][FD_DFT_RING][4];
  const fd_dft_tile t = tiles[blockIdx.x];
  if (t.flux != fl) return;
  const cdesc* d = (const cdesc*)t.d;
  if (d->flux_nf[fl] == 0) return;
  __shared__ double base[FD_DFT_QB][4];
  __shared__ float samp[4][FD_DFT_RING][64];
  dft_flush(d, fl, t.q0, t.p0, first, count, G((const double*)d->flux_acc[fl]), G(d->flux_prev[fl]), tab, base, samp);
}

// For reads: the flux spectrum's sums over a plane, on the device: a plane's
// complex sums (655 MB for 320^2 points and 100 frequencies) are read once at the
// HBM rate instead of being copied to the host and summed there (169 -> 0.6 ms;
// 80^2 points 10.4 -> 0.13 ms).  One workgroup per frequency and FD_SPEC_PTS
// points, enough of them to fill the chip on a plane of a few thousand points.
__global__ __launch_bounds__(256) void spectrum_kernel(const double* __restrict__ acc, int nf, int plane,
                                                       double* __restrict__ parts) {
  __shared__ double red[4];
  const int q = (int)blockIdx.y, p0 = (int)blockIdx.x * FD_SPEC_PTS, p1 = min(plane, p0 + FD_SPEC_PTS);
  const size_t cs = (size_t)nf * plane;  // points from one component to the next
  const double2* e = reinterpret_cast<const double2*>(acc) + (size_t)q * plane;
  double v = 0.0;
  for (int p = p0 + (int)threadIdx.x; p < p1; p += 256) {
    const double2 ex = e[p], ey = e[cs + p], hx = e[2 * cs + p], hy = e[3 * cs + p];
    v += (ex.x * hy.x + ex.y * hy.y) - (ey.x * hx.x + ey.y * hx.y);
  }
  const double tot = block_sum(v, red);
  if (threadIdx.x == 0) parts[(size_t)q * gridDim.x + blockIdx.x] = tot;
}

// For reads: the partial sums of each T(t) or energy sample (a row of m) added in
// order, as a host loop would, so that only one number per sample leaves the
// device.  A workgroup stages kRowCols columns of kRows rows at a time in LDS
// (coalesced loads), then a thread per row adds them up.  At most kRowGroups
// workgroups go over the rows in turn: they fill the chip, and a group for each of
// the 2^31 samples that a plan may have would exceed a launch's 2^32 threads.
constexpr int kRows = 16, kRowCols = 128, kRowGroups = 4096;
__global__ __launch_bounds__(256) void row_sums_kernel(const double* __restrict__ part, long long n, int m,
                                                       double* __restrict__ out) {
  __shared__ double buf[kRows][kRowCols + 1];
  for (long long r0 = (long long)blockIdx.x * kRows; r0 < n; r0 += (long long)gridDim.x * kRows) {
    double acc = 0.0;
    for (int c0 = 0; c0 < m; c0 += kRowCols) {
      const int w = min(kRowCols, m - c0);
      for (int t = (int)threadIdx.x; t < kRows * kRowCols; t += 256) {
        const int r = t / kRowCols, c = t % kRowCols;
        if (r0 + r < n && c < w) buf[r][c] = part[(size_t)(r0 + r) * m + c0 + c];
      }
      __syncthreads();
      if (threadIdx.x < kRows && r0 + threadIdx.x < n) {
#pragma unroll 16
        for (int c = 0; c < w; ++c) acc += buf[threadIdx.x][c];  // LDS reads ahead of the sums
      }
      __syncthreads();
    }
    if (threadIdx.x < kRows && r0 + threadIdx.x < n) out[r0 + threadIdx.x] = acc;
  }
}

__global__ void advance_kernel(fd_desc* const* descs, int n, long long k) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) descs[t]->step += k;
}

__global__ void advance_one_kernel(fd_desc* d, long long k) {
  if (threadIdx.x == 0 && blockIdx.x == 0) d->step += k;
}

__global__ void fill_kernel(uint4* p, size_t n16, uint8_t* tail, size_t ntail) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n16; q += stride)
    p[q] = make_uint4(0u, 0u, 0u, 0u);
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < ntail) tail[t] = 0;
}

// Integer-exact voxelization: voxel centre X = (2 (i - origin) + 1) 2^16 quanta,
// inside sphere (C, rho) iff |X - C|^2 < rho^2 (minimum image on periodic axes).
// Candidate sites: those whose nominal position (h res 2^16 quanta along each axis)
// lies within `reach` of the voxel centre.
__device__ __forceinline__ long long floordiv_ll(long long a, long long b) {
  long long q = a / b;
  if ((a % b != 0) && (a < 0)) --q;
  return q;
}

__global__ void voxelize_kernel(const int64_t* __restrict__ sites, int ex, int ey, int ez, int3 per,
                                int3 ncr, int3 org, longlong3 reach, int res, int mat_bg, int mat_void,
                                int mat_out, int nx, int ny, int nz, int px, uint8_t* __restrict__ map) {
  const long long ncell = (long long)nx * ny * nz;
  const long long stride = (long long)gridDim.x * blockDim.x;
  const long long H16 = 65536;
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < ncell; v += stride) {
    const int i = (int)(v % nx);
    const int j = (int)((v / nx) % ny);
    const int k = (int)(v / ((long long)nx * ny));
    const int rel[3] = {i - org.x, j - org.y, k - org.z};
    const int nc[3] = {ncr.x, ncr.y, ncr.z};
    bool in_crystal = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) in_crystal = in_crystal && rel[a] >= 0 && rel[a] < nc[a];
    const long long vo = ((long long)k * ny + j) * px + i;  // padded rows
    if (!in_crystal) {
      map[vo] = (uint8_t)mat_out;
      continue;
    }
    const int pr[3] = {per.x, per.y, per.z};
    const long long rc[3] = {reach.x, reach.y, reach.z};
    const int ext[3] = {ex, ey, ez};
    const long long X[3] = {(2LL * rel[0] + 1) * H16, (2LL * rel[1] + 1) * H16, (2LL * rel[2] + 1) * H16};
    // res * 2^16 quanta between consecutive half-lattice sites; the period of a
    // periodic axis is the crystal length, ncr * 2^17 quanta
    long long hlo[3], hhi[3], sstep[3], period[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      sstep[a] = (long long)res * H16;
      period[a] = (long long)nc[a] * 2 * H16;
      hlo[a] = -floordiv_ll(-(X[a] - rc[a]), sstep[a]);  // ceil
      hhi[a] = floordiv_ll(X[a] + rc[a], sstep[a]);
      if (!pr[a]) {
        if (hlo[a] < 0) hlo[a] = 0;
        if (hhi[a] > ext[a] - 1) hhi[a] = ext[a] - 1;
      }
    }
    bool hit = false;
    for (long long l = hlo[2]; l <= hhi[2] && !hit; ++l) {
      long long lw = l;
      if (pr[2]) { lw %= ext[2]; if (lw < 0) lw += ext[2]; }
      for (long long kk = hlo[1]; kk <= hhi[1] && !hit; ++kk) {
        long long kw = kk;
        if (pr[1]) { kw %= ext[1]; if (kw < 0) kw += ext[1]; }
        for (long long h = hlo[0]; h <= hhi[0] && !hit; ++h) {
          long long hw = h;
          if (pr[0]) { hw %= ext[0]; if (hw < 0) hw += ext[0]; }
          if (((hw + kw + lw) & 1) != 0) continue;
          const int64_t* S = sites + 4 * ((lw * ey + kw) * ex + hw);
          const long long rho = S[3];
          if (rho <= 0) continue;
          long long r2 = 0;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            long long dd = X[a] - S[a];
            if (pr[a]) {
              dd %= period[a];
              if (dd < 0) dd += period[a];
              if (2 * dd > period[a]) dd -= period[a];
            }
            r2 += dd * dd;
          }
          if (r2 < rho * rho) hit = true;
        }
      }
    }
    map[vo] = (uint8_t)(hit ? mat_void : mat_bg);
  }
}

// Initial upper-level populations of the gain cells at their gain ordinals, as
// (hi, lo) pairs whose sum is n_init to about 48 bits (every other state
// variable starts at zero with the arena).
__global__ void init_pop_kernel(const uint8_t* __restrict__ map, const float* __restrict__ ninit,
                                const uint32_t* __restrict__ gidx, unsigned gainmask, float* pop, int ncell,
                                int nx, int px) {
  const int stride = gridDim.x * blockDim.x;
  for (int o = blockIdx.x * blockDim.x + threadIdx.x; o < ncell; o += stride) {
    if (o % px >= nx) continue;  // row padding
    const int m = map[o];
    if (!((gainmask >> m) & 1u)) continue;
    const uint32_t g = gidx[o];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      pop[(size_t)q * ncell + g] = ninit[8 * m + 1 + q];        // hi
      pop[(size_t)(3 + q) * ncell + g] = ninit[8 * m + 5 + q];  // lo
    }
  }
}

// ------------------------------------- density matrix at the cell centres
// A density-matrix gain cell holds rho at its centre (i+1/2, j+1/2, k+1/2), where
// the paper solves the density-matrix equations.  The step kernels leave on
// every edge A = E^n + dt/(eps dx) (curl H - dx J_src), the field before the
// polarization change.  With <F> the average of the four edges of a component
// around a centre and [Q] on an edge a quarter of the sum of Q over the (up to
// four) gain cells sharing it -- the adjoint of <.>, so the field gives the
// matter exactly the energy the matter takes -- the matter then makes one
// predictor-corrector pass of the implicit midpoint coupling:
//   predictor  rho* = S(rho^n; <(E^n + A)/2>),   Q* = P(rho*) - P(rho^n) + dt J
//   corrector  E* = A - [Q*]/eps,  rho^{n+1} = S(rho^n; <(E^n + E*)/2>),
//              Q = P(rho^{n+1}) - P(rho^n) + dt J
//   edges      E^{n+1} = A - [Q]/eps
// with S = R(dt/2) C(E) R(dt/2), P_c = 2 kappa Re rho_0c, J the
// spontaneous-emission noise current at the centre and eps that of the edge's
// own voxel.  Each pass reads what the previous one wrote for neighbouring
// cells, so the passes are separate launches; a cell's rho is read and written
// only by its own thread.
// Memory bounds the passes: on the 168^3 box, 2.09 M gain cells, they count 271 MB in
// 55 us, 508 MB in 106 us and 139 MB in 32 us, 4.4-4.9 TB/s beside the 5.1 TB/s of a
// large copy.  Numbering the gain cells and edges in blocks of 8 x 8 rows with
// neighbouring units on one XCD took the corrector's traffic from 636 MB to 508, and
// neighbour offsets without wall tests and divisions its instructions from 1,200 to
// 930 a wave and its registers from 135 to 112, four waves per SIMD instead of three:
// 124 -> 112 us, the rest by the order of the passes (dm_unit).

// The plan's material table in LDS (a gain cell's own medium, an edge's
// permittivity), staged once per workgroup: a work unit's cells belong to one
// plan, so every coefficient read of the passes is an LDS read.
struct DmMats {
  fd_mat m[FD_MAXMAT];
};
// loads(): issues the thread's loads that need only its list position; they are in
// flight with the table's (the memory counter retires in order, so only the
// table's are waited for) and across the barrier, which waits for LDS alone.
template <class F>
__device__ __forceinline__ void dm_stage_mats(const cdesc* d, DmMats& sm, F&& loads) {
  const int words = d->nmat * (int)(sizeof(fd_mat) / 4), t = (int)threadIdx.x;
  const gf* src = G((const float*)d->mats);
  float* dst = reinterpret_cast<float*>(sm.m);
  const float w = src[t < words ? t : 0];
  loads();
  if (t < words) dst[t] = w;
  for (int q = t + (int)blockDim.x; q < words; q += (int)blockDim.x) dst[q] = src[q];
  lds_barrier();
}

// Work unit of this workgroup.  Workgroups go to the 8 XCDs in turn; runs of
// kDmRun consecutive units are kept on one XCD, so that the fields and increments
// a unit gathers from the rows and planes beside its own cells are in that XCD's
// L2 from the units next to it (gain cells are numbered in blocks of 8 x 8 rows).
// REV: from the last unit to the first.  The step kernel goes up through the grid,
// the predictor down, the corrector up and the edge pass down, so that each starts
// with what the one before it has just read and written and the Infinity Cache
// still holds: 168^3 box 301.6 -> 287.7 us per step (predictor 61.6 -> 58, corrector
// 112 -> 103), the paper's 200^3 lasing box 301 -> 298.
constexpr int kDmRun = 32;
template <bool REV>
__device__ __forceinline__ int dm_unit(int w, int n) {
  const int full = n / (8 * kDmRun) * (8 * kDmRun);
  if (w >= full) return w;  // the rest, in order
  const int x = w % 8, q = REV ? full / 8 - 1 - w / 8 : w / 8;  // a unit is on the same XCD in every pass
  return (q / kDmRun * 8 + x) * kDmRun + q % kDmRun;
}

struct Ijk {
  int i, j, k;
};
// Coordinates of cell o, the divisions as a product and a shift (fd_desc)
__device__ __forceinline__ Ijk ijk_of(const cdesc* d, uint32_t o) {
  const uint32_t k = (uint32_t)(((uint64_t)o * d->div_plane[0]) >> d->div_plane[1]);
  const uint32_t r = o - k * (uint32_t)d->plane;
  const uint32_t j = (uint32_t)(((uint64_t)r * d->div_px[0]) >> d->div_px[1]);
  return {(int)(r - j * (uint32_t)d->px), (int)j, (int)k};
}

// Cell p's neighbourhood: element offsets to its neighbours at -1, 0, +1 along
// each axis (periodic wrap; 0 beyond a PEC wall, where ok is false), so that a
// neighbour's index is the cell's plus one offset per axis.  wall: the cell lies
// on or next to a PEC wall, where values beyond it and held edges have to be
// looked at; waves without such a cell run without those tests.
struct Nbr {
  int d[3][3];  // [axis][offset + 1]
  bool ok[3][3], low[3];
  bool wall;
};
__device__ __forceinline__ Nbr neighbours(const cdesc* d, Ijk p) {
  Nbr b;
  const int q[3] = {p.i, p.j, p.k}, n[3] = {d->nx, d->ny, d->nz}, s[3] = {1, d->px, d->plane};
  b.wall = false;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const bool lo = q[a] == 0, hi = q[a] == n[a] - 1, pec = !d->per[a];
    const int span = (n[a] - 1) * s[a];
    b.d[a][0] = lo ? (pec ? 0 : span) : -s[a];
    b.d[a][1] = 0;
    b.d[a][2] = hi ? (pec ? 0 : -span) : s[a];
    b.ok[a][0] = !(lo & pec);
    b.ok[a][1] = true;
    b.ok[a][2] = !(hi & pec);
    b.low[a] = lo & pec;
    b.wall = b.wall | ((lo | hi) & pec);
  }
  return b;
}
// The cell at offsets u, v in {-1, 0, 1} along the two axes transverse to
// component c ((c+1) mod 3, (c+2) mod 3): its offset, and whether it exists.
__device__ __forceinline__ int nb_off(const Nbr& b, int c, int u, int v) {
  return b.d[(c + 1) % 3][u + 1] + b.d[(c + 2) % 3][v + 1];
}
__device__ __forceinline__ bool nb_ok(const Nbr& b, int c, int u, int v) {
  return b.ok[(c + 1) % 3][u + 1] & b.ok[(c + 2) % 3][v + 1];
}
// That cell's component-c edge lies on a PEC wall (index 0 of a non-periodic
// transverse axis) and is held at zero; u, v in {0, 1}: only the cell itself can
// have index 0 along an axis it is not stepped along (or that it wraps around,
// which a PEC axis does not).
__device__ __forceinline__ bool nb_held(const Nbr& b, int c, int u, int v) {
  return (u == 0 && b.low[(c + 1) % 3]) | (v == 0 && b.low[(c + 2) % 3]);
}

// A gain cell's state (populations as (hi, lo) FP32 pairs, coherences), its
// medium, its noise term dt J and P(rho^n).
struct DmCell {
  uint32_t g, o;
  Ijk p;
  const fd_mat* mt;
  float nh[3], nl[3], pp[3], inc[3];
  Cz c[3], x[3];
  float Pn[3], dJ[3];
};

// The cell and state of gain ordinal g (issued before the material table is
// waited for), then what needs the table.  LO: with the populations' low parts.
// The predictor leaves them out (12 of 113 bytes): a pair is stored with hi the
// rounded sum of both (two_sum, and n_init at bind), so hi is the population.
template <bool LO>
__device__ __forceinline__ void dm_load_state(const cdesc* d, uint32_t g, DmCell& z) {
  const size_t ncs = (size_t)d->ncell;
  const gf* pop = G((const float*)d->pop);
  auto state = [&](int q) { return R32<const float>{pop + (size_t)q * ncs}[g]; };
  z.g = g;
  z.o = R32<const uint32_t>{(const __attribute__((address_space(1))) uint32_t*)d->glist}[g];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    z.nh[q] = state(q);
    z.nl[q] = LO ? state(3 + q) : 0.0f;
    z.c[q] = {state(6 + q), state(9 + q)};
    z.x[q] = {state(12 + q), state(15 + q)};
  }
}
__device__ __forceinline__ void dm_load_medium(const cdesc* d, const DmMats& sm, long long n, DmCell& z) {
  z.p = ijk_of(d, z.o);
  z.mt = &sm.m[R32<const uint8_t>{(const gu8*)d->mat}[z.o]];
  const fd_mat& mt = *z.mt;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    z.pp[q] = z.nh[q] + z.nl[q];
    z.inc[q] = 0.0f;
    z.Pn[q] = mt.bk2 * z.c[q].r;
    z.dJ[q] = 0.0f;
  }
  if (mt.noise != 0.0f) {
    float gg[3];
    // the counter takes the dense cell index (k ny + j) nx + i
    normals3((uint32_t)n, ((uint32_t)z.p.k * (uint32_t)d->ny + (uint32_t)z.p.j) * (uint32_t)d->nx + (uint32_t)z.p.i,
             d->key0, d->key1, gg);
#pragma unroll
    for (int q = 0; q < 3; ++q) z.dJ[q] = mt.noise * sqrtf(fmaxf(z.pp[q], 0.0f)) * gg[q];
  }
}

// Gathers are branch-free within a wave: a neighbour beyond a PEC wall has offset
// 0 and its value is replaced by 0 where it is used, so a thread's loads go out
// together and are waited for once (a load under a lane's branch is waited for on
// its own).  Waves without a cell at a wall (WALL = false) leave those tests out.
__device__ __forceinline__ R32<const float> comp(const float* p) { return R32<const float>{G(p)}; }

template <bool WALL>
__device__ __forceinline__ void dm_centre_pred(const cdesc* d, const Nbr& b, uint32_t o, int par, float em[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    // <(E^n + A)/2>: the cell's four component-q edges sit at offsets {0, 1}
    const R32<const float> En = comp(d->E[par][q]), A = comp(d->E[par ^ 1][q]);
    float acc = 0.0f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint32_t e = o + nb_off(b, q, a, c);
        const float v = En[e] + A[e];
        acc += !WALL || nb_ok(b, q, a, c) ? v : 0.0f;
      }
    em[q] = 0.125f * acc;
  }
}

__global__ __launch_bounds__(FD_DM_CELLS) void dm_predict_kernel(const fd_dm_unit* __restrict__ units, int s) {
  __shared__ DmMats sm;
  const fd_dm_unit u = units[dm_unit<true>((int)blockIdx.x, (int)gridDim.x)];
  const cdesc* d = (const cdesc*)u.d;
  const long long n = d->step + s;
  const int par = (int)(n & 1), t = (int)threadIdx.x;
  DmCell z;
  dm_stage_mats(d, sm, [&] { dm_load_state<false>(d, (uint32_t)(u.first + (t < u.count ? t : 0)), z); });
  if (t >= u.count) return;
  dm_load_medium(d, sm, n, z);
  const Nbr b = neighbours(d, z.p);
  float em[3];
  if (__any(b.wall)) dm_centre_pred<true>(d, b, z.o, par, em);
  else dm_centre_pred<false>(d, b, z.o, par, em);
  dm_relax(*z.mt, z.pp, z.inc, z.c, z.x);
  dm_cayley<false>(*z.mt, em, z.pp, z.inc, z.c, z.x);
  gf* Q = G(d->dmq[0]);
  const size_t ncs = (size_t)d->ncell;
#pragma unroll
  for (int q = 0; q < 3; ++q)
    R32<float>{Q + (size_t)q * ncs}[z.o] = z.mt->bk2 * (z.c[q].r * z.mt->bf2) - z.Pn[q] + z.dJ[q];
}

template <bool WALL>
__device__ __forceinline__ void dm_centre_corr(const cdesc* d, const DmMats& sm, const Nbr& b, uint32_t o, int par,
                                               float em[3]) {
  const R32<const uint8_t> map{(const gu8*)d->mat};
  const size_t ncs = (size_t)d->ncell;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    // Q* of the 3 x 3 cells around the centre across component q (0 off the
    // grid; cells without gain hold 0)
    const R32<const float> Qs = comp(d->dmq[0] + (size_t)q * ncs);
    float qn[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float v = Qs[o + nb_off(b, q, a - 1, c - 1)];
        qn[a][c] = !WALL || nb_ok(b, q, a - 1, c - 1) ? v : 0.0f;
      }
    // <E^n + E*> with E* = A - [Q*]/eps on the edges (0 beyond or on a PEC wall);
    // the edge at offsets (a, c) is shared by the cells at (a - 1 .. a, c - 1 .. c)
    const R32<const float> En = comp(d->E[par][q]), A = comp(d->E[par ^ 1][q]);
    float acc = 0.0f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint32_t e = o + nb_off(b, q, a, c);
        const float en = En[e], av = A[e];
        const float sh = 0.25f * ((qn[a][c] + qn[a + 1][c]) + (qn[a][c + 1] + qn[a + 1][c + 1]));
        const float es = av - sh * sm.m[map[e]].inv_eps;
        const bool ok = !WALL || nb_ok(b, q, a, c);
        acc += ok ? en : 0.0f;
        acc += !WALL || (ok & !nb_held(b, q, a, c)) ? es : 0.0f;
      }
    em[q] = 0.125f * acc;
  }
}

__global__ __launch_bounds__(FD_DM_CELLS) void dm_correct_kernel(const fd_dm_unit* __restrict__ units, int s) {
  __shared__ DmMats sm;
  const fd_dm_unit u = units[dm_unit<false>((int)blockIdx.x, (int)gridDim.x)];
  const cdesc* d = (const cdesc*)u.d;
  const long long n = d->step + s;
  const int par = (int)(n & 1), t = (int)threadIdx.x;
  DmCell z;
  dm_stage_mats(d, sm, [&] { dm_load_state<true>(d, (uint32_t)(u.first + (t < u.count ? t : 0)), z); });
  if (t >= u.count) return;
  dm_load_medium(d, sm, n, z);
  const Nbr b = neighbours(d, z.p);
  const size_t ncs = (size_t)d->ncell;
  float em[3];
  if (__any(b.wall)) dm_centre_corr<true>(d, sm, b, z.o, par, em);
  else dm_centre_corr<false>(d, sm, b, z.o, par, em);
  dm_relax(*z.mt, z.pp, z.inc, z.c, z.x);
  dm_cayley<true>(*z.mt, em, z.pp, z.inc, z.c, z.x);
  dm_relax(*z.mt, z.pp, z.inc, z.c, z.x);
  gf* pop = G(d->pop);
  gf* Q = G(d->dmq[1]);
  auto put = [&](int q, float v) { R32<float>{pop + (size_t)q * ncs}[z.g] = v; };
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    R32<float>{Q + (size_t)r * ncs}[z.o] = z.mt->bk2 * z.c[r].r - z.Pn[r] + z.dJ[r];
    two_sum(z.nh[r], z.nl[r], z.inc[r]);
    put(r, z.nh[r]);
    put(3 + r, z.nl[r]);
    put(6 + r, z.c[r].r);
    put(9 + r, z.c[r].i);
    put(12 + r, z.x[r].r);
    put(15 + r, z.x[r].i);
  }
}

// E^{n+1} = A - [Q]/eps on the edges next to gain cells, one listed cell per
// thread (the cells whose edges a gain cell shares): the twelve Q values first
// (cells without gain hold Q = 0), then, for a cell with a changed edge, its A
// and the new E; and the samples of the E probes in listed cells (u.probes), which
// the step kernel recorded from A.
template <bool WALL>
__device__ __forceinline__ void dm_edge_sums(const cdesc* d, const Nbr& b, uint32_t o, float acc[3]) {
  const size_t ncs = (size_t)d->ncell;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    // the cells sharing the edge: offsets {0, -1} along the transverse axes
    const R32<const float> Q = comp(d->dmq[1] + (size_t)c * ncs);
    acc[c] = 0.0f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const float qv = Q[o + nb_off(b, c, -a, -v)];
        acc[c] += !WALL || nb_ok(b, c, -a, -v) ? qv : 0.0f;
      }
    if (WALL && nb_held(b, c, 0, 0)) acc[c] = 0.0f;
  }
}

__global__ __launch_bounds__(FD_DM_EDGES) void dm_edges_kernel(const fd_dm_unit* __restrict__ units, int s) {
  __shared__ DmMats sm;
  const fd_dm_unit u = units[dm_unit<true>((int)blockIdx.x, (int)gridDim.x)];
  const cdesc* d = (const cdesc*)u.d;
  const int t = (int)threadIdx.x;
  const long long n = d->step + s;
  const int par = (int)(n & 1);
  uint32_t o;
  dm_stage_mats(d, sm, [&] {
    o = R32<const uint32_t>{(const __attribute__((address_space(1))) uint32_t*)d->elist}[u.first + (t < u.count ? t : 0)];
  });
  if (t >= u.count) return;
  const Nbr b = neighbours(d, ijk_of(d, o));
  // the cell's A and material go out with the sharers' Q (one round trip)
  float ev[3], acc[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) ev[c] = comp(d->E[par ^ 1][c])[o];
  const uint32_t mo = R32<const uint8_t>{(const gu8*)d->mat}[o];
  if (__any(b.wall)) dm_edge_sums<true>(d, b, o, acc);
  else dm_edge_sums<false>(d, b, o, acc);
  const float ie = sm.m[mo].inv_eps;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (acc[c] != 0.0f) {
      ev[c] = ev[c] - 0.25f * acc[c] * ie;
      R32<float>{G(d->E[par ^ 1][c])}[o] = ev[c];
    }
  for (unsigned mm = u.probes; mm; mm &= mm - 1u) {  // uniform
    const int p = __builtin_ctz(mm), cp = d->probe_comp[p];
    if ((uint32_t)(d->probe_k[p] * d->plane + d->probe_cell[p]) != o) continue;
    float v = ev[2];
    v = cp == 1 ? ev[1] : v;
    v = cp == 0 ? ev[0] : v;
    G(d->probe_ring)[(long long)p * d->max_steps + n] = v;
  }
}

// After the edge pass: the T(t) partial of every xy tile of a flux plane,
// recomputed from the final E^{n+1} (the step kernels recorded it from A).  Unit:
// first = flux plane, count = xy tile; the block has the plan's tile shape.
__global__ __launch_bounds__(FD_MAXBLOCK) void dm_diag_kernel(const fd_dm_unit* __restrict__ units, int s) {
  __shared__ double red[FD_MAXBLOCK / 64];
  const fd_dm_unit u = units[blockIdx.x];
  const cdesc* d = (const cdesc*)u.d;
  const long long n = d->step + s;
  const int par = (int)(n & 1);
  const int t = (int)threadIdx.x;
  const int f = u.first, blk = u.count;
  const int TX = d->tile_x, TY = (int)blockDim.x / TX;
  const int ntx = (d->nx + TX - 1) / TX;
  const int i = (blk % ntx) * TX + t % TX, j = (blk / ntx) * TY + t / TX;
  double v = 0.0;
  if (i < d->nx && j < d->ny) {
    const int kf = d->flux_k[f], km = kf > 0 ? kf - 1 : d->nz - 1;
    const size_t off = (size_t)j * d->px + i;
    const size_t o = (size_t)kf * d->plane + off, om = (size_t)km * d->plane + off;
    const float sx = 0.5f * (G((const float*)d->E[par][0])[o] + G((const float*)d->E[par ^ 1][0])[o]);
    const float sy = 0.5f * (G((const float*)d->E[par][1])[o] + G((const float*)d->E[par ^ 1][1])[o]);
    const gf* hx = G((const float*)d->H[par ^ 1][0]);
    const gf* hy = G((const float*)d->H[par ^ 1][1]);
    const float hyc = 0.5f * (hy[om] + hy[o]), hxc = 0.5f * (hx[om] + hx[o]);
    v = (double)(sx * hyc) - (double)(sy * hxc);
  }
  const double tot = block_sum(v, red);
  if (t == 0) G(d->flux_T[f])[n * d->nblk + blk] = tot;
}

}  // namespace

hipError_t fd_launch_step(int cls, const fd_tile* tiles, int ntiles, int tile_x, int block, int grid, int s,
                          const fd_xcd* part, int nt, int nflux, int rev, hipStream_t st, hipEvent_t start,
                          hipEvent_t stop) {
  if (ntiles <= 0) return hipSuccess;
  if (nflux < 0 || nflux > FD_MAXFLUX) return hipErrorInvalidValue;
  if (block < 64 || block > FD_MAXBLOCK || (block & 63) != 0 || grid <= 0 || block % tile_x != 0 ||
      2 * (tile_x + 2) + 2 * (block / tile_x) > block)
    return hipErrorInvalidValue;
  const unsigned lds = fd_sample_spare(tile_x, block, nflux) ? 0u : (unsigned)(nflux * 4 * FD_MAXBLOCK * (int)sizeof(float));
  fd_xcd pz{};
  int use = 0;
  if (part) {
    // every part must lie inside the list and the grid must cover the longest one
    int longest = 0;
    for (int x = 0; x < 8; ++x) {
      if (part->start[x] < 0 || part->count[x] < 0 || part->start[x] + part->count[x] > ntiles)
        return hipErrorInvalidValue;
      longest = part->count[x] > longest ? part->count[x] : longest;
    }
    if (grid < 8 * longest) return hipErrorInvalidValue;
    pz = *part;
    use = 1;
    use |= rev ? 2 : 0;
  }
  switch (tile_x) {
    case 16: return fd_launch_step_16(cls, tiles, ntiles, block, grid, s, pz, use, nt, lds, st, start, stop);
    case 32: return fd_launch_step_32(cls, tiles, ntiles, block, grid, s, pz, use, nt, lds, st, start, stop);
    case 64: return fd_launch_step_64(cls, tiles, ntiles, block, grid, s, pz, use, nt, lds, st, start, stop);
    default: return hipErrorInvalidValue;
  }
}

hipError_t fd_launch_dft(const fd_dft_tile* tiles, int ntiles, int s, hipStream_t st, hipEvent_t start,
                         hipEvent_t stop) {
  if (ntiles <= 0) return hipSuccess;
  hipExtLaunchKernelGGL(dft_kernel, dim3(ntiles), dim3(256), 0, st, start, stop, 0, tiles, s);
  return hipGetLastError();
}

hipError_t fd_launch_dft_preview(const fd_dft_tile* tiles, int ntiles, int flux, long long first, int count,
                                 hipStream_t st) {
  if (ntiles <= 0 || count <= 0) return hipSuccess;
  if (count > FD_DFT_RING || first < 0) return hipErrorInvalidValue;
  dft_preview_kernel<<<ntiles, 256, 0, st>>>(tiles, flux, first, count);
  return hipGetLastError();
}

hipError_t fd_launch_spectrum(const double* acc, int nf, int plane, double* parts, hipStream_t st) {
  if (nf <= 0 || plane <= 0) return hipSuccess;
  if (nf > 65535) return hipErrorInvalidValue;
  spectrum_kernel<<<dim3((plane + FD_SPEC_PTS - 1) / FD_SPEC_PTS, nf), 256, 0, st>>>(acc, nf, plane, parts);
  return hipGetLastError();
}

hipError_t fd_launch_row_sums(const double* part, long long n, int m, double* out, hipStream_t st) {
  if (n <= 0 || m <= 0) return hipSuccess;
  const long long groups = (n + kRows - 1) / kRows;
  row_sums_kernel<<<(unsigned)(groups < kRowGroups ? groups : kRowGroups), 256, 0, st>>>(part, n, m, out);
  return hipGetLastError();
}

hipError_t fd_launch_advance(fd_desc* const* descs, int n, long long k, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  advance_kernel<<<(n + 255) / 256, 256, 0, st>>>(descs, n, k);
  return hipGetLastError();
}

hipError_t fd_launch_advance_one(fd_desc* d, long long k, hipStream_t st) {
  advance_one_kernel<<<1, 64, 0, st>>>(d, k);
  return hipGetLastError();
}

hipError_t fd_launch_fill(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  const size_t n16 = bytes / 16;
  const size_t ntail = bytes - n16 * 16;
  size_t blocks = (n16 + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 4096) blocks = 4096;
  fill_kernel<<<(unsigned)blocks, 256, 0, st>>>(reinterpret_cast<uint4*>(p), n16,
                                                reinterpret_cast<uint8_t*>(p) + n16 * 16, ntail);
  return hipGetLastError();
}

hipError_t fd_launch_voxelize(const int64_t* sites, int ex, int ey, int ez, const int* per, const int* ncr,
                              const int* origin, const int64_t* reach, int res, int mat_bg,
                              int mat_void, int mat_out, int nx, int ny, int nz, int px, uint8_t* map,
                              hipStream_t st) {
  const long long ncell = (long long)nx * ny * nz;
  long long blocks = (ncell + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  voxelize_kernel<<<(unsigned)blocks, 256, 0, st>>>(
      sites, ex, ey, ez, make_int3(per[0], per[1], per[2]), make_int3(ncr[0], ncr[1], ncr[2]),
      make_int3(origin[0], origin[1], origin[2]), make_longlong3(reach[0], reach[1], reach[2]), res, mat_bg,
      mat_void, mat_out, nx, ny, nz, px, map);
  return hipGetLastError();
}

hipError_t fd_launch_init_pop(const uint8_t* map, const float* n_init_by_mat, const uint32_t* gidx, unsigned gainmask,
                              float* pop, int ncell, int nx, int px, hipStream_t st) {
  int blocks = (ncell + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  init_pop_kernel<<<blocks, 256, 0, st>>>(map, n_init_by_mat, gidx, gainmask, pop, ncell, nx, px);
  return hipGetLastError();
}

// ------------------------------------------------------------ static tables
// The launch tables (tile lists, DFT work units, descriptor pointers) of batches
// made by fdtd_batch_create_static live here instead of in a hipMalloc'd block:
// one array per GPU, held until the process ends.  In host code the name is
// only a handle: kernels get the address hipGetSymbolAddress returns for the
// current device.
static __device__ __align__(256) unsigned char scratch[FD_STATIC_TABLE_BYTES];

hipError_t fd_static_tables(void** ptr, int* device) {
  static std::mutex mu;
  static void* addr[FD_MAX_DEVICES] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= FD_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = a;
  }
  *ptr = addr[dev];
  *device = dev;
  return hipSuccess;
}

hipError_t fd_launch_dm(const fd_dm_unit* cells, int ncells, const fd_dm_unit* edges, int nedges,
                        const fd_dm_unit* diag, int ndiag, int block, int s, hipStream_t st, hipEvent_t* ev) {
  if (ncells <= 0) return hipSuccess;
  if (block < 64 || block > FD_MAXBLOCK || (block & 63) != 0) return hipErrorInvalidValue;
  auto E = [&](int q) -> hipEvent_t { return ev ? ev[q] : nullptr; };
  hipExtLaunchKernelGGL(dm_predict_kernel, dim3(ncells), dim3(FD_DM_CELLS), 0, st, E(0), E(1), 0, cells, s);
  hipExtLaunchKernelGGL(dm_correct_kernel, dim3(ncells), dim3(FD_DM_CELLS), 0, st, E(2), E(3), 0, cells, s);
  if (nedges > 0)
    hipExtLaunchKernelGGL(dm_edges_kernel, dim3(nedges), dim3(FD_DM_EDGES), 0, st, E(4), E(5), 0, edges, s);
  if (ndiag > 0) hipExtLaunchKernelGGL(dm_diag_kernel, dim3(ndiag), dim3(block), 0, st, E(6), E(7), 0, diag, s);
  return hipGetLastError();
}
