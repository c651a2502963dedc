// gfx950 step kernels of libfdtd for tiles FD_STEP_TX columns wide (this file is
// compiled once for each width): one fused Yee step -- H then E, CPML, the Lorentz
// gain medium (ADE with four-level populations and noise), soft sources, probes,
// transmitted power, DFT samples, energy.
//
// Method: C. Conti and A. Fratalocchi, arXiv:0802.3775 — Yee FDTD with absorbing
// walls in a disordered inverted opal, pumped gain medium seeded by a stochastic
// source, transmitted power T(t) (sections "Sample and numerical approach" and
// "Dynamical diffusion and localization").
//
// Stepping scheme.  E, H, the H-side CPML memory and the Lorentz polarization
// are double-buffered by step parity, so one step reads only buffer n&1 and
// writes only the other one (the E-side CPML memory and the populations are read
// and written only by their own cell's thread).  Every tile is therefore
// independent within a step, and a
// workgroup can recompute the H^{n+1/2} values its E update needs at x-1, y-1 and
// z-1 from the read-only inputs instead of waiting for the owner: one pass over
// HBM per step (E, H, material index in; E, H out).
//
// Work mapping.  A tile is TX x block/TX (i,j) columns (x fastest: a wavefront reads
// one run of 64 floats per array in tiles 64 wide, two of 32 or four of 16 in the
// others) and a z range [k0, k1) that the workgroup marches upward, carrying the
// H^{n+1/2} of plane k-1 in registers.  Tiles whose columns touch no CPML slab and no gain cell
// run a specialised kernel without that code.
#include "fd_device.h"

#include <hip/hip_ext.h>

using namespace fdk;

namespace {

// ------------------------------------------------------------------ context
struct Ctx {
  int nx, ny, nz, plane;
  int rx;  // row pitch of the per-cell arrays
  int px, py, pz;
  float ch;
  R32<const float> Ein[3];
  R32<float> Eout[3];
  R32<const float> Hin[3];
  R32<float> Hout[3];
  // CPML (used by the kernels specialised with PML)
  int lo[3], hi[3], t[3], n[3];
  int wx, xhi;  // x slabs' psi: row length, start of the high slab's
  const cfloat* prof[3];  // read-only for the kernel: scalar loads where uniform
  R32<float> psiE[3][2];
  R32<const float> psiHin[3][2];
  R32<float> psiHout[3][2];
};

__device__ __forceinline__ void make_ctx(Ctx& x, const cdesc* d, int par, bool pml) {
  x.nx = d->nx; x.ny = d->ny; x.nz = d->nz; x.plane = d->plane; x.rx = d->px;
  x.px = d->per[0]; x.py = d->per[1]; x.pz = d->per[2];
  x.ch = d->ch;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    x.Ein[c].p = G((const float*)d->E[par][c]);
    x.Eout[c].p = G(d->E[par ^ 1][c]);
    x.Hin[c].p = G((const float*)d->H[par][c]);
    x.Hout[c].p = G(d->H[par ^ 1][c]);
  }
  x.n[0] = d->nx; x.n[1] = d->ny; x.n[2] = d->nz;
  if (!pml) return;
  // equal x slabs: an array each; else rows of both
  const bool apart = d->pml_lo[0] == d->pml_hi[0];
  x.wx = apart ? d->pml_lo[0] : d->pml_t[0];
  x.xhi = apart ? d->pml_lo[0] * x.ny * x.nz : d->pml_lo[0];
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    x.lo[w] = d->pml_lo[w]; x.hi[w] = d->pml_hi[w]; x.t[w] = d->pml_t[w];
    x.prof[w] = (const cfloat*)d->prof[w];
    // an axis without CPML has no psi arrays: its pointers are set to E so
    // that the unconditional reads of the all-axes march stay in bounds (their
    // values are never used; stores happen only inside slabs)
    float* const spare = d->E[par][0];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      x.psiE[w][f].p = G(d->psiE[w][f] ? d->psiE[w][f] : spare);
      x.psiHin[w][f].p = G((const float*)(d->psiH[par][w][f] ? d->psiH[par][w][f] : spare));
      x.psiHout[w][f].p = G(d->psiH[par ^ 1][w][f] ? d->psiH[par ^ 1][w][f] : spare);
    }
  }
}

// slab-local index along axis w, or -1 outside the slabs
__device__ __forceinline__ int slab(const Ctx& x, int w, int p) {
  if (x.t[w] == 0) return -1;
  if (p < x.lo[w]) return p;
  if (p >= x.n[w] - x.hi[w]) return p - (x.n[w] - x.hi[w]) + x.lo[w];
  return -1;
}

// psi array offset for axis w, slab index sp, at (i, j, k).  z slabs are whole
// planes.  The rows of y slabs have the fields' pitch, and x slabs of equal width are an
// array each: a tile's rows of one x slab follow each other, where rows that held both
// slabs left most 128-byte lines to two tiles at the grid's two ends (200x200x200
// box 138.1 -> 135.5 us; while interior tiles took the all-axes march too, 139.9 and
// 140.3).
__device__ __forceinline__ int psi_off(const Ctx& x, int w, int sp, int i, int j, int k) {
  if (w == 2) return sp * x.plane + j * x.rx + i;
  if (w == 1) return (k * x.t[1] + sp) * x.rx + i;
  return (k * x.ny + j) * x.wx + (sp < x.lo[0] ? sp : sp - x.lo[0] + x.xhi);
}
// The same for the x slabs by xslab(), which finds the high slab's place once per
// lane: a product and a sum per plane remain.  A choice of the row length and the
// start in every plane cost tiles in x slabs that work from the cache 2-7% (94x94x94
// box, 64 wide, 26.7 us, rows of both slabs 26.1, this 26.0).
__device__ __forceinline__ int xslab(const Ctx& x, int i) {
  const int sp = slab(x, 0, i);
  return sp < x.lo[0] ? sp : sp - x.lo[0] + x.xhi;
}
__device__ __forceinline__ int xpsi_off(const Ctx& x, int sx, int j, int k) { return (k * x.ny + j) * x.wx + sx; }

// CPML stretch of one difference d along axis w at index p (E position when
// HSIDE = false, H position when HSIDE = true): returns d/kappa + psi with the
// psi recursion psi = b psi + c d; the owner of the cell stores psi.
template <bool HSIDE, int PM>
__device__ __forceinline__ float stretch(const Ctx& x, int c, int w, int p, int i, int j, int k, float d,
                                         bool own) {
  if (!((PM >> w) & 1)) return d;  // no slab on this axis in this tile class
  const int sp = slab(x, w, p);
  if (sp < 0) return d;
  const cfloat* pr = x.prof[w] + (HSIDE ? 3 : 0) * x.n[w];
  const float kinv = pr[p], b = pr[x.n[w] + p], cc = pr[2 * x.n[w] + p];
  const int off = psi_off(x, w, sp, i, j, k);
  const int f = fam(c, w);
  float psi;
  if (HSIDE) {
    psi = fmaf(b, x.psiHin[w][f][off], cc * d);
    if (own) x.psiHout[w][f][off] = psi;
  } else {
    psi = fmaf(b, x.psiE[w][f][off], cc * d);
    if (own) x.psiE[w][f][off] = psi;
  }
  return fmaf(d, kinv, psi);
}

// The same for a z difference when the old psi and the plane's grading
// (pz = 1/kappa, b, c) have already been loaded: z slabs are whole planes, so
// the slab index sz of plane k is uniform over a tile.  off2d: j*px + i of the
// cell.  Bit-identical to stretch<HSIDE, PM>(.., 2, k, ..).
template <bool HSIDE>
__device__ __forceinline__ float stretch_z(const Ctx& x, int c, const float* pz, int sz, int off2d, float d,
                                           bool own, float psi_old) {
  if (sz < 0) return d;
  const float kinv = pz[0], b = pz[1], cc = pz[2];
  const float psi = fmaf(b, psi_old, cc * d);
  if (own) {
    const int off = sz * x.plane + off2d;
    if (HSIDE) x.psiHout[2][fam(c, 2)][off] = psi;
    else x.psiE[2][fam(c, 2)][off] = psi;
  }
  return fmaf(d, kinv, psi);
}

// A CPML difference whose old psi and grading are already in registers (sp: slab
// index, -1 outside): returns d/kappa + psi with psi = b psi_old + c d and stores
// psi at dst[off] when own.  Bit-identical to stretch<HSIDE, PM>.
__device__ __forceinline__ float stretch_v(float d, int sp, float kinv, float b, float cc, float psi_old, bool own,
                                           const R32<float>& dst, uint32_t off) {
  if (sp < 0) return d;
  const float psi = fmaf(b, psi_old, cc * d);
  if (own) dst[off] = psi;
  return fmaf(d, kinv, psi);
}

// One H component from its two differences: H^{n+1/2} = H^{n-1/2} - (dt/dx)(d1 - d2),
// each difference stretched by the CPML where the position lies in a slab.  The
// owner and every workgroup that recomputes the value as a halo call this with
// identical operands, so all copies agree bit for bit.
// c: component; (w1, p1) / (w2, p2): axis and index of the two differences.
// ZPRE: a z difference takes its old psi from zpsi (slab index sz, cell off2d).
template <int PM, bool ZPRE = false>
__device__ __forceinline__ float h_from(const Ctx& x, int c, int w1, int p1, int w2, int p2, int i, int j, int k,
                                        float a1, float a0, float b1, float b0, float hold, bool own, int sz = -1,
                                        int off2d = 0, float zpsi = 0.0f, const float* pz = nullptr) {
  float d1 = a1 - a0, d2 = b1 - b0;
  if (PM) {
    d1 = (ZPRE && w1 == 2) ? stretch_z<true>(x, c, pz, sz, off2d, d1, own, zpsi)
                           : stretch<true, PM>(x, c, w1, p1, i, j, k, d1, own);
    d2 = (ZPRE && w2 == 2) ? stretch_z<true>(x, c, pz, sz, off2d, d2, own, zpsi)
                           : stretch<true, PM>(x, c, w2, p2, i, j, k, d2, own);
  }
  return fmaf(-x.ch, d1 - d2, hold);
}

// The H-side stretch of a difference of the plane below a tile (the prologue
// of the all-axes march; no psi store), in two parts so that the loads go out
// with the prologue's other loads, whatever the lane's slab membership (index 0
// outside a slab; the result is selected): pre_load issues them, pre_apply is
// stretch<true, PM>(.., own = false) bit for bit.
struct PreStretch {
  float kinv, b, cc, po;
  bool in;
};
template <int PM>
__device__ __forceinline__ PreStretch pre_load(const Ctx& x, int c, int w, int p, int i, int j, int k, bool live) {
  PreStretch r{1.0f, 0.0f, 0.0f, 0.0f, false};
  if (!((PM >> w) & 1) || x.t[w] == 0) return r;  // uniform: no slab code on this axis
  const int sp = slab(x, w, p);
  r.in = live && sp >= 0;
  const cfloat* pr = x.prof[w] + 3 * x.n[w];
  const int pc = r.in ? p : 0;
  r.kinv = pr[pc];
  r.b = pr[x.n[w] + pc];
  r.cc = pr[2 * x.n[w] + pc];
  r.po = x.psiHin[w][fam(c, w)][r.in ? psi_off(x, w, sp, i, j, k) : 0];
  return r;
}
__device__ __forceinline__ float pre_apply(const PreStretch& r, float d) {
  const float psi = fmaf(r.b, r.po, r.cc * d);
  return r.in ? fmaf(d, r.kinv, psi) : d;
}

template <int TX>
struct Lds {
  static constexpr int TYM = FD_MAXBLOCK / TX;
  static constexpr int W = TX + 2, N = (TYM + 2) * W;
  float E[2][3][N];  // E^n, planes k and k+1, over [i0-1, i0+TX] x [j0-1, j0+TY]
  float H[3][(TYM + 1) * (TX + 1)];     // H^{n+1/2} of plane k over [i0-1, i0+TX-1] x [j0-1, j0+TY-1]
  fd_mat mat[FD_MAXMAT];
  double red[FD_MAXBLOCK / 64];
  double ftot[FD_MAXFLUX];  // T(t) partial of the tile per flux plane, stored after the z march
  float probe[FD_MAXPROBE];  // probe samples of the tile, stored after the z march
  // all-axes CPML tiles: x and y grading (1/kappa, b, c at E then H positions) of
  // columns i0-1 .. i0+TX-1 and rows j0-1 .. j0+TYM-1 (0 outside the slabs)
  float gx[6][TX + 1];
  float gy[6][TYM + 1];
};

// Whether step n records the energy (n / ke as a product and a shift: steps stay
// below 2^31).
__device__ __forceinline__ bool energy_due(const cdesc* d, long long n) {
  const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)n * d->div_ke[0]) >> d->div_ke[1]);
  return q * (uint32_t)d->ke == (uint32_t)n;
}

// ZT: the tile's z range holds z-slab planes.  Without them the z march drops
// every z-CPML test (PMM), so interior tiles of a CPML launch run the same
// code as tiles of a plain launch; the plane below the range still takes the
// general path.
// SP: the tile has sources, probes or flux planes, or the step records the energy;
// the other tiles' march has none of that code (nor its uniform values).
template <int TX, int PM, int GAIN, bool ZT, bool NT, bool SP>
__device__ __forceinline__ void run_tile(const fd_tile& tl, int s_rel, Lds<TX>& s) {
  extern __shared__ float smp[];  // DFT samples that do not fit into s.E (fd_sample_spare)
  const cdesc* d = (const cdesc*)tl.d;
  constexpr int W = Lds<TX>::W;
  const int TY = (int)blockDim.x / TX;
  const int t = (int)threadIdx.x;
  const int tx = t % TX, ty = t / TX;
  lds_barrier();  // LDS reuse across tiles of the persistent loop
  // material table: the load is issued here and stored to LDS just before the
  // z march, so its latency overlaps the set-up loads
  const int mwords = d->nmat * (int)(sizeof(fd_mat) / 4);
  const gf* msrc = G((const float*)d->mats);
  const float mword = t < mwords ? msrc[t] : 0.0f;
  const long long n = d->step + s_rel;
  const int par = (int)(n & 1);
  Ctx x;
  make_ctx(x, d, par, PM != 0);
  const int i0 = tl.i0, j0 = tl.j0, k0 = tl.k0, k1 = tl.k1;
  const unsigned gmask = GAIN ? d->gainmask : 0u;
  const size_t ncs = (size_t)d->ncell;
  // field stores: non-temporal (NT) when the launch's working set exceeds the
  // Infinity Cache, so they stream to HBM without displacing lines that are
  // still to be read; a compile-time choice (a runtime branch between the two
  // forms of the same store is merged into the plain one by the compiler)
  auto put = [&](const R32<float>& a, int idx, float v) {
    if constexpr (NT) __builtin_nontemporal_store(v, &a[idx]);
    else a[idx] = v;
  };
  const int i = i0 + tx, j = j0 + ty;
  const bool act = i < x.nx && j < x.ny;
  const int c = j * x.rx + i;
  // the cell's column / row lies on the PEC wall x = 0 / y = 0 (its tangential
  // E components are held at zero there)
  const bool pec_i = !x.px && i == 0, pec_j = !x.py && j == 0;

  // ---- per-tile gather offsets (plane-relative), outside the z loop
  int own_off;
  {
    const int gi = wrap(i, x.nx, x.px), gj = wrap(j, x.ny, x.py);
    own_off = (gi >= 0 && gj >= 0) ? gj * x.rx + gi : -1;
  }
  const int own_slot = (ty + 1) * W + tx + 1;
  // The E staging area has a one-cell ring around the TX x TY tile: ring cell q
  // (bottom row, top row, left column, right column) maps to an LDS slot and a
  // plane offset (-1 beyond a PEC wall).  Thread t stages ring cell t; the
  // launch guarantees 2 (TX + 2) + 2 TY <= blockDim.
  const int nring = 2 * (TX + 2) + 2 * TY;
  auto ring_cell = [&](int q, int& slot, int& off) {
    int lx, ly;
    if (q < TX + 2) { lx = q; ly = 0; }
    else if (q < 2 * (TX + 2)) { lx = q - (TX + 2); ly = TY + 1; }
    else if (q < 2 * (TX + 2) + TY) { lx = 0; ly = 1 + q - 2 * (TX + 2); }
    else { lx = TX + 1; ly = 1 + q - 2 * (TX + 2) - TY; }
    const int gi = wrap(i0 - 1 + lx, x.nx, x.px), gj = wrap(j0 - 1 + ly, x.ny, x.py);
    slot = ly * W + lx;
    off = (gi >= 0 && gj >= 0) ? gj * x.rx + gi : -1;
  };
  int r_slot = -1, r_off = -1;
  if (t < nring) ring_cell(t, r_slot, r_off);
  // halo duty: threads [0, TX) own the row j0-1, threads [TX, TX+TY) the column
  // i0-1; hr: column of the row cell / row of the column cell
  const bool bh = t < TX;
  const bool lh = !bh && t < TX + TY;
  const int hr = lh ? t - TX : t;
  const int hgi = wrap(lh ? i0 - 1 : i0 + hr, x.nx, x.px);
  const int hgj = wrap(lh ? j0 + hr : j0 - 1, x.ny, x.py);
  const bool hact = (lh || bh) && hgi >= 0 && hgj >= 0 && (lh ? (j0 + hr < x.ny) : (i0 + hr < x.nx));
  const int h_off = hact ? hgj * x.rx + hgi : 0;

  // ---- sources, probes and flux planes that touch the tile (set on the host);
  // srcmine: the sources that drive this thread's column
  const unsigned srcmask = SP ? tl.srcmask : 0u, pmask = SP ? tl.pmask : 0u, fmask = SP ? tl.fmask : 0u;
  unsigned srcmine = 0u;
  for (unsigned mm = srcmask; mm; mm &= mm - 1u) {
    const int q = __builtin_ctz(mm);
    if (d->src_kind[q] != 0 || d->src_cell[q] == c) srcmine |= 1u << q;  // sheets drive every column
  }
  const bool edue = SP && (tl.flags & FD_TILE_KE) && energy_due(d, n);
  double eacc = 0.0;

  // ---- staging.  Iteration k of the z march consumes a Stage holding E^n of
  // plane k+1 (own cell and one ring cell; stored to LDS at the top of the
  // iteration) and the own inputs of plane k (H^{n-1/2}, the halo-duty H, the
  // material index).  Two Stages alternate, so the loads for plane k+3 (E) and
  // k+2 (own inputs) are in flight while plane k is computed: the global-load
  // latency is spread over two iterations.  Slots outside the grid hold the
  // periodic image or 0.
  // A Stage holds raw load results; validity selects are applied where the
  // values are used, so no instruction touches a load result before it is due.
  struct Stage {
    float own[3];
    float ring[3];
    bool zok;     // plane inside the grid (or its periodic image)
    float ho[3];  // H^{n-1/2} of the own cell
    float hsel;   // halo-duty cell: Hy (column cell) or Hx (row cell)
    float hh2;    // halo-duty cell: Hz
    int m;
    float ph[2];  // z-slab planes: old psi_H of Hx, Hy (own)
    float phz;    // z-slab planes: old psi_H of hsel's z difference at the halo-duty cell
    float pe[2];  // z-slab planes: old psi_E of Ex, Ey (own)
    float gh[3];  // z-slab planes: H-side grading 1/kappa, b, c (uniform)
    float ge[3];  // z-slab planes: E-side grading (uniform)
    uint32_t gi;  // gain cells: the cell's gain ordinal (index of its gain state)
  };
  // Every global load of the z march is issued whatever the lane's own cell (a
  // lane with nothing to load reads element 0 and discards it; only uniform
  // conditions -- the all-axes tile's slabs -- skip loads), and the march stores to
  // global memory only the fields and CPML memory: the loads in flight per
  // iteration are then the same on every path, so the compiler waits for
  // exactly the Stage it consumes and leaves the other one in flight.
  // live = false: the plane is past the tile; the loads are still issued (at
  // element 0) so that every path through the march issues the same loads.
  // Linear tiles without x / y CPML (EREG) keep the own cell's E^n of planes k
  // and k+1 in registers and form each load address with one select: in-plane
  // offsets are clamped to cell 0 once where the lane has nothing to load (its
  // values are discarded at use).  The other classes, near their register caps,
  // read those E values from LDS and select per load.  Either way a plane the
  // march does not need (past the tile, or outside the CPML slabs for psi) is
  // read at element 0 by every lane: one cache line, not a row of another plane.
  constexpr bool EREG = GAIN == 0 && !(ZT && PM == 7);
  const uint32_t own_l = own_off >= 0 ? own_off : 0, ring_l = r_off >= 0 ? r_off : 0;
  const uint32_t c_l = act ? c : 0;  // h_off is already 0 without halo duty
  auto load_e = [&](int kk, Stage& S, bool live) {
    const int kz = kk < x.nz ? kk : (x.pz ? kk - x.nz : -1);
    S.zok = kz >= 0;
    const uint32_t zo = S.zok ? kz * x.plane : 0;
    const uint32_t io = EREG ? (live ? zo + own_l : 0u) : ((live && own_off >= 0) ? zo + own_off : 0u);
    const uint32_t ir = EREG ? (live ? zo + ring_l : 0u) : ((live && r_off >= 0) ? zo + r_off : 0u);
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) S.own[cc] = x.Ein[cc][io];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) S.ring[cc] = x.Ein[cc][ir];
  };
  // stages E^n of the Stage's plane into LDS buffer b; eown receives the own
  // cell's values (0 beyond a PEC wall), which the march keeps in registers
  auto store_e = [&](int b, const Stage& S, float eown[3]) {
    const bool oko = S.zok && own_off >= 0, okr = S.zok && r_off >= 0;
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      eown[cc] = oko ? S.own[cc] : 0.0f;
      s.E[b][cc][own_slot] = eown[cc];
    }
    if (r_slot >= 0) {
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) s.E[b][cc][r_slot] = okr ? S.ring[cc] : 0.0f;
    }
  };
  const R32<const uint8_t> matp{(const gu8*)d->mat};
  const R32<const uint32_t> gidxp{(const __attribute__((address_space(1))) uint32_t*)d->gidx};
  constexpr int PMM = ZT ? PM : (PM & 3);  // CPML axes the march handles
  constexpr bool ZP = ZT && PM == 4;       // z-slab psi prefetched with the plane (z-only CPML tiles)
  constexpr bool AX = PMM == 7;            // all-axes CPML tiles: psi of the plane issued up front
  static_assert(PMM == 0 || PMM == 4 || PMM == 7, "tile classes: no CPML, z slabs, all axes");
  auto load_h = [&](int kk, Stage& S, bool live) {
    kk = live ? kk : 0;
    const uint32_t zo = kk * x.plane;
    const uint32_t io = EREG ? (live ? zo + c_l : 0u) : ((live && act) ? zo + c : 0u);
    const uint32_t ih = EREG ? (live ? zo + h_off : 0u) : ((live && hact) ? zo + h_off : 0u);
#pragma unroll
    for (int q = 0; q < 3; ++q) S.ho[q] = x.Hin[q][io];
    S.m = matp[io];  // lanes outside the grid read cell 0: a valid material
    if (GAIN) S.gi = gidxp[io];
    // the column i0-1 needs Hy, Hz; the row j0-1 needs Hx, Hz.  The lane picks
    // the array (a choice between two loaded values would wait for both loads
    // at once, and a choice between two Stage fields becomes an indexed, spilled
    // access)
    S.hsel = R32<const float>{lh ? x.Hin[1].p : x.Hin[0].p}[ih];
    S.hh2 = x.Hin[2][ih];
    if (ZP) {
      // the z differences of Hx, Hy, Ex, Ey in a z slab carry psi: load the
      // old values with the plane's other inputs (psi_E is touched only by the
      // owner of the cell, so reading it early is safe); the grading is uniform
      const int sz = slab(x, 2, kk);
      const int nz = x.n[2];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        S.ge[q] = x.prof[2][q * nz + kk];
        S.gh[q] = x.prof[2][(3 + q) * nz + kk];
      }
      const bool in = live && sz >= 0;
      const uint32_t base = in ? sz * x.plane : 0;
      const uint32_t jo = EREG ? (in ? base + c_l : 0u) : ((in && act) ? base + c : 0u);
      const uint32_t jh = EREG ? (in ? base + h_off : 0u) : ((in && hact) ? base + h_off : 0u);
      S.ph[0] = x.psiHin[2][fam(0, 2)][jo];
      S.ph[1] = x.psiHin[2][fam(1, 2)][jo];
      S.pe[0] = x.psiE[2][fam(0, 2)][jo];
      S.pe[1] = x.psiE[2][fam(1, 2)][jo];
      S.phz = R32<const float>{lh ? x.psiHin[2][fam(1, 2)].p : x.psiHin[2][fam(0, 2)].p}[jh];
    }
  };

  // Loads are issued in the order their values are consumed (the memory
  // counter retires in order): plane k0, the inputs of H^{n+1/2} at plane
  // k0-1 (the march carries H of the plane below), then the two Stages.
  Stage SA, SB;
  load_e(k0, SA, true);
  const int km = prv(k0, x.nz, x.pz);
  const bool pro = act && km >= 0;
  const int jp = nxt(j, x.ny, x.py), ip = nxt(i, x.nx, x.px);
  float pEz, pEzj, pEzi, pEy, pEx, pHx, pHy;
  {
    const int zm = pro ? km * x.plane : 0;
    const uint32_t om = pro ? zm + c : 0;
    const uint32_t ojp = (pro && jp >= 0) ? zm + jp * x.rx + i : 0;
    const uint32_t oip = (pro && ip >= 0) ? zm + j * x.rx + ip : 0;
    pEz = x.Ein[2][om];
    pEzj = x.Ein[2][ojp];
    pEzi = x.Ein[2][oip];
    pEy = x.Ein[1][om];
    pEx = x.Ein[0][om];
    pHx = x.Hin[0][om];
    pHy = x.Hin[1][om];
  }
  // all-axes tiles: the CPML inputs of H at plane k0-1 and this thread's first
  // entry of the x / y grading tables, issued now so that their latency
  // overlaps the loads above instead of following them
  PreStretch px1{}, px2{}, py1{}, py2{};
  float gxv = 0.0f, gyv = 0.0f;
  if (AX) {
    px1 = pre_load<PM>(x, 0, 1, j, i, j, km, pro);
    px2 = pre_load<PM>(x, 0, 2, km, i, j, km, pro);
    py1 = pre_load<PM>(x, 1, 2, km, i, j, km, pro);
    py2 = pre_load<PM>(x, 1, 0, i, i, j, km, pro);
    if (x.t[0] > 0) {
      const int r = t / (TX + 1), ii = i0 - 1 + t % (TX + 1);
      const bool ok = t < 6 * (TX + 1) && ii >= 0 && ii < x.nx && slab(x, 0, ii) >= 0;
      const float v = x.prof[0][ok ? r * x.nx + ii : 0];
      gxv = ok ? v : 0.0f;
    }
    if (x.t[1] > 0) {
      constexpr int GY = Lds<TX>::TYM + 1;
      const int r = t / GY, jj = j0 - 1 + t % GY;
      const bool ok = t < 6 * GY && jj >= 0 && jj < x.ny && slab(x, 1, jj) >= 0;
      const float v = x.prof[1][ok ? r * x.ny + jj : 0];
      gyv = ok ? v : 0.0f;
    }
  }
  float ecur[3];  // E^n of the own cell at the plane being marched
  store_e(0, SA, ecur);
  load_e(k0 + 1, SA, true);
  load_h(k0, SA, true);
  load_e(k0 + 2, SB, k0 + 1 < k1);
  load_h(k0 + 1, SB, k0 + 1 < k1);
  // next plane of the march that holds a flux plane: looked up here, while the loads
  // above are in flight, and after each of them.  A look at flux_k in every plane was a
  // load that the plane waited for, and a launch waits for its slowest tile (80x80x224
  // slab 19.3 -> 18.1 us, 160x160x224, 64 x 48 planes, 78.1 -> 74.6).  Not in the class
  // without CPML, whose shortest steps pay for the registers (32^3 periodic cell 4.05,
  // with it 4.16), nor with Lorentz gain, whose boxes have no flux planes (84^3, 32
  // wide, 28.6 and 28.9); with the place in the tile's record that cell takes 4.03, but
  // the 64x64x120 slab 9.85 instead of 9.76.
  constexpr bool FNEXT = PM != 0 && GAIN == 0;
  auto flux_from = [&](int from) {
    int best = 0x7fffffff;
    for (unsigned mm = fmask; mm; mm &= mm - 1u) {  // uniform
      const int fk = d->flux_k[__builtin_ctz(mm)];
      best = fk >= from && fk < best ? fk : best;
    }
    return best;
  };
  int nextf = FNEXT ? flux_from(k0) : 0;
  // H^{n+1/2} at (i, j, k0-1); E^n at (i, j, k0) is already in LDS buffer 0
  float hxm = 0.0f, hym = 0.0f;
  if (AX) {
    const float ey1 = ecur[1], ex1 = ecur[0];
    const float ezj = jp >= 0 ? pEzj : 0.0f, ezi = ip >= 0 ? pEzi : 0.0f;
    const float hx = fmaf(-x.ch, pre_apply(px1, ezj - pEz) - pre_apply(px2, ey1 - pEy), pHx);
    const float hy = fmaf(-x.ch, pre_apply(py1, ex1 - pEx) - pre_apply(py2, ezi - pEz), pHy);
    hxm = pro ? hx : 0.0f;
    hym = pro ? hy : 0.0f;
  } else if (pro) {
    const float ey1 = ecur[1], ex1 = ecur[0];
    const float ezj = jp >= 0 ? pEzj : 0.0f, ezi = ip >= 0 ? pEzi : 0.0f;
    hxm = h_from<PM>(x, 0, 1, j, 2, km, i, j, km, ezj, pEz, ey1, pEy, pHx, false);
    hym = h_from<PM>(x, 1, 2, km, 0, i, i, j, km, ex1, pEx, ezi, pEz, pHy, false);
  }

  // plane k uses LDS E buffer cb = (k - k0) & 1, a compile-time constant in
  // each of the two unrolled copies, so every LDS address is a fixed offset
  {
    float* mdst = reinterpret_cast<float*>(s.mat);
    if (t < mwords) mdst[t] = mword;
    for (int q = t + (int)blockDim.x; q < mwords; q += (int)blockDim.x) mdst[q] = msrc[q];
  }
  // all-axes CPML: slab indices of the own column and of the halo-duty cell along
  // x and y (fixed over the march), and the tile's x / y grading tables in LDS
  int sxo = -1, syo = -1, sxh = -1, syh = -1;
  // uniform: the tile's columns (with the halo column i0-1) reach an x slab,
  // its rows (with the halo row j0-1) a y slab
  const bool uxs = AX && x.t[0] > 0 && (i0 - 1 < x.lo[0] || i0 + TX > x.nx - x.hi[0]);
  const bool uys = AX && x.t[1] > 0 && (j0 - 1 < x.lo[1] || j0 + TY > x.ny - x.hi[1]);
  if (AX) {
    sxo = xslab(x, i);
    syo = slab(x, 1, j);
    if (hact) {
      sxh = xslab(x, hgi);
      syh = slab(x, 1, hgj);
    }
    if (t < 6 * (TX + 1)) s.gx[t / (TX + 1)][t % (TX + 1)] = gxv;
    for (int q = t + (int)blockDim.x; q < 6 * (TX + 1); q += (int)blockDim.x) {
      const int r = q / (TX + 1), ii = i0 - 1 + q % (TX + 1);
      s.gx[r][q % (TX + 1)] = (ii >= 0 && ii < x.nx && slab(x, 0, ii) >= 0) ? x.prof[0][r * x.nx + ii] : 0.0f;
    }
    if (t < 6 * (Lds<TX>::TYM + 1)) s.gy[t / (Lds<TX>::TYM + 1)][t % (Lds<TX>::TYM + 1)] = gyv;
    for (int q = t + (int)blockDim.x; q < 6 * (Lds<TX>::TYM + 1); q += (int)blockDim.x) {
      const int r = q / (Lds<TX>::TYM + 1), jj = j0 - 1 + q % (Lds<TX>::TYM + 1);
      s.gy[r][q % (Lds<TX>::TYM + 1)] = (jj >= 0 && jj < x.ny && slab(x, 1, jj) >= 0) ? x.prof[1][r * x.ny + jj] : 0.0f;
    }
  }

  // Where thread `at` has the DFT sample of flux plane f, and the stride of its four
  // values: at the ends of four E arrays, or in the launch's own LDS
  auto sample_at = [&](int f, int at, int& stride) __attribute__((always_inline)) -> float* {
    const int r = __builtin_popcount(fmask & ((1u << f) - 1u));
    if constexpr (TX == 16) {
      const int bd = (int)blockDim.x;
      if (fd_sample_spare(TX, bd, __builtin_popcount(fmask))) {
        stride = Lds<TX>::N;
        return &s.E[0][0][0] + Lds<TX>::N - (r + 1) * bd + at;
      }
    }
    stride = FD_MAXBLOCK;
    return smp + r * 4 * FD_MAXBLOCK + at;
  };

  auto plane_step = [&](auto cbc, const int k, Stage& S) __attribute__((always_inline)) {
    constexpr int cb = decltype(cbc)::value;
    constexpr int nb = cb ^ 1;
    // plane k+1 into LDS; the loads two planes ahead reuse the same Stage
    float enx[3];  // E^n of the own cell at plane k+1
    store_e(nb, S, enx);
    const int zo = k * x.plane;
    const int o = zo + c;
    const int sz = (ZP || AX) ? slab(x, 2, k) : -1;
    // all-axes CPML: the old psi the plane needs, issued before the barriers
    // (lanes outside a slab read element 0); z grading is uniform over the plane
    float aH[6] = {}, aE[6] = {}, aHh[4] = {}, gzE[3] = {}, gzH[3] = {};
    uint32_t ox = 0, oy = 0, oz = 0, ohx = 0, ohy = 0, ohz = 0;
    if (AX) {
      ox = (act && sxo >= 0) ? (uint32_t)xpsi_off(x, sxo, j, k) : 0u;
      oy = (act && syo >= 0) ? (uint32_t)psi_off(x, 1, syo, i, j, k) : 0u;
      oz = (act && sz >= 0) ? (uint32_t)(sz * x.plane + c) : 0u;
      ohx = (hact && sxh >= 0) ? (uint32_t)xpsi_off(x, sxh, hgj, k) : 0u;
      ohy = (hact && syh >= 0) ? (uint32_t)psi_off(x, 1, syh, hgi, hgj, k) : 0u;
      ohz = (hact && sz >= 0) ? (uint32_t)(sz * x.plane + h_off) : 0u;
      // own H: Hx(y, z), Hy(z, x), Hz(x, y); own E in the same order.  The
      // reads of an axis whose slabs neither the tile (x, y) nor the plane (z)
      // touches are skipped (uniform branches; the values stay 0 and unused)
      // halo: column cells (lh) need Hy(z, x), row cells Hx(y, z); both need Hz(x, y)
      if (uxs) {
        aH[3] = x.psiHin[0][0][ox];
        aH[4] = x.psiHin[0][1][ox];
        aE[3] = x.psiE[0][0][ox];
        aE[4] = x.psiE[0][1][ox];
        aHh[2] = x.psiHin[0][1][ohx];
      }
      if (uys) {
        aH[0] = x.psiHin[1][1][oy];
        aH[5] = x.psiHin[1][0][oy];
        aE[0] = x.psiE[1][1][oy];
        aE[5] = x.psiE[1][0][oy];
        aHh[3] = x.psiHin[1][0][ohy];
      }
      if (uxs | uys) {
        const gf* pc1o = lh ? x.psiHin[0][0].p : x.psiHin[1][1].p;
        aHh[1] = pc1o[lh ? ohx : ohy];
      }
      if (sz >= 0) {
        aH[1] = x.psiHin[2][0][oz];
        aH[2] = x.psiHin[2][1][oz];
        aE[1] = x.psiE[2][0][oz];
        aE[2] = x.psiE[2][1][oz];
        const gf* pc1z = lh ? x.psiHin[2][1].p : x.psiHin[2][0].p;
        aHh[0] = pc1z[ohz];
      }
      if (sz >= 0) {  // uniform: the z grading exists only with z slabs
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          gzE[q] = x.prof[2][q * x.nz + k];
          gzH[q] = x.prof[2][(3 + q) * x.nz + k];
        }
      }
    }
    // gain-cell inputs of plane k (populations, P^n, P^{n-1}), consumed in the E
    // update; other lanes read element 0
    float gnh[3], gnl[3], gPn[3], gPm[3];
    bool gk = false;
    if (GAIN) {
      gk = act && ((gmask >> S.m) & 1u);
      const uint32_t ig = gk ? S.gi : 0u;
      const gf* pop = G(d->pop);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        gnh[q] = pop[(size_t)q * ncs + ig];
        gnl[q] = pop[(size_t)(3 + q) * ncs + ig];
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        gPn[q] = G((const float*)d->P[par][q])[ig];
        gPm[q] = G((const float*)d->P[par ^ 1][q])[ig];
      }
    }
    // the loads two planes ahead go out after this plane's psi and gain inputs:
    // the memory counter retires in order, so waiting for those does not wait
    // for them
    load_e(k + 3, S, k + 2 < k1);
    // E^n of the own cell at plane k, from registers or read from LDS before the
    // second barrier (after it a faster wave may already be staging plane k+2
    // into this buffer)
    float eo[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) eo[q] = EREG ? ecur[q] : s.E[cb][q][own_slot];
    lds_barrier();
    // ---- H^{n+1/2} of plane k: own cell and halo duty
    float hx = 0.0f, hy = 0.0f, hz = 0.0f;
    {
      const float* Ex = s.E[cb][0];
      const float* Ey = s.E[cb][1];
      const float* Ez = s.E[cb][2];
      const float* Ex1 = s.E[nb][0];
      const float* Ey1 = s.E[nb][1];
      const int a = own_slot;
      // own-cell E^n at planes k and k+1: registers in the classes that carry
      // them, else the LDS copies (equal values; the capped classes are short
      // of registers)
      const float e0x = EREG ? eo[0] : Ex[a], e0y = EREG ? eo[1] : Ey[a], e0z = EREG ? eo[2] : Ez[a];
      const float e1x = EREG ? enx[0] : Ex1[a], e1y = EREG ? enx[1] : Ey1[a];
      if (act && AX) {
        const int xi = tx + 1, yj = ty + 1;
        const float* gxh[3] = {s.gx[3], s.gx[4], s.gx[5]};
        const float* gyh[3] = {s.gy[3], s.gy[4], s.gy[5]};
        float d1 = Ez[a + W] - e0z, d2 = e1y - e0y;
        d1 = stretch_v(d1, syo, gyh[0][yj], gyh[1][yj], gyh[2][yj], aH[0], true, x.psiHout[1][1], oy);
        d2 = stretch_v(d2, sz, gzH[0], gzH[1], gzH[2], aH[1], true, x.psiHout[2][0], oz);
        hx = fmaf(-x.ch, d1 - d2, S.ho[0]);
        d1 = e1x - e0x;
        d2 = Ez[a + 1] - e0z;
        d1 = stretch_v(d1, sz, gzH[0], gzH[1], gzH[2], aH[2], true, x.psiHout[2][1], oz);
        d2 = stretch_v(d2, sxo, gxh[0][xi], gxh[1][xi], gxh[2][xi], aH[3], true, x.psiHout[0][0], ox);
        hy = fmaf(-x.ch, d1 - d2, S.ho[1]);
        d1 = Ey[a + 1] - e0y;
        d2 = Ex[a + W] - e0x;
        d1 = stretch_v(d1, sxo, gxh[0][xi], gxh[1][xi], gxh[2][xi], aH[4], true, x.psiHout[0][1], ox);
        d2 = stretch_v(d2, syo, gyh[0][yj], gyh[1][yj], gyh[2][yj], aH[5], true, x.psiHout[1][0], oy);
        hz = fmaf(-x.ch, d1 - d2, S.ho[2]);
        put(x.Hout[0], o, hx);
        put(x.Hout[1], o, hy);
        put(x.Hout[2], o, hz);
      } else if (PMM == 0) {
        // no CPML memory: every lane computes (lanes outside the grid read
        // in-bounds LDS slots and element 0 of H) and only the stores are masked
        hx = h_from<0>(x, 0, 1, j, 2, k, i, j, k, Ez[a + W], e0z, e1y, e0y, S.ho[0], true);
        hy = h_from<0>(x, 1, 2, k, 0, i, i, j, k, e1x, e0x, Ez[a + 1], e0z, S.ho[1], true);
        hz = h_from<0>(x, 2, 0, i, 1, j, i, j, k, Ey[a + 1], e0y, Ex[a + W], e0x, S.ho[2], true);
        hx = act ? hx : 0.0f;
        hy = act ? hy : 0.0f;
        hz = act ? hz : 0.0f;
        if (act) {
          put(x.Hout[0], o, hx);
          put(x.Hout[1], o, hy);
          put(x.Hout[2], o, hz);
        }
      } else if (act) {
        hx = h_from<PMM, ZP>(x, 0, 1, j, 2, k, i, j, k, Ez[a + W], e0z, e1y, e0y, S.ho[0], true, sz, c, S.ph[0], S.gh);
        hy = h_from<PMM, ZP>(x, 1, 2, k, 0, i, i, j, k, e1x, e0x, Ez[a + 1], e0z, S.ho[1], true, sz, c, S.ph[1], S.gh);
        hz = h_from<PMM, ZP>(x, 2, 0, i, 1, j, i, j, k, Ey[a + 1], e0y, Ex[a + W], e0x, S.ho[2], true, sz, c, 0.0f, S.gh);
        put(x.Hout[0], o, hx);
        put(x.Hout[1], o, hy);
        put(x.Hout[2], o, hz);
      }
      const int hs = (ty + 1) * (TX + 1) + tx + 1;
      s.H[0][hs] = hx;
      s.H[1][hs] = hy;
      s.H[2][hs] = hz;
      if (hact && AX) {
        // column cell (i0-1, j0+hr): Hy(z, x) and Hz(x, y); row cell (i0+hr, j0-1):
        // Hx(y, z) and Hz(x, y).  One path, operands selected per lane (the
        // column's x-table entry is 0 and its y-table entry hr+1, the row's the
        // reverse); bit-identical to separate column and row paths
        const int b = lh ? (hr + 1) * W : hr + 1;  // E slot of the halo cell
        const int xe = lh ? 0 : hr + 1, ye = lh ? hr + 1 : 0;
        const float* z1 = lh ? Ex1 : Ey1;
        const float* z0 = lh ? Ex : Ey;
        float zd = z1[b] - z0[b];
        zd = stretch_v(zd, sz, gzH[0], gzH[1], gzH[2], aHh[0], false, x.psiHout[2][0], 0u);
        // the transverse difference of Ez: along x for the column, along y for the row
        float td = Ez[b + (lh ? 1 : W)] - Ez[b];
        td = stretch_v(td, lh ? sxh : syh, lh ? s.gx[3][0] : s.gy[3][0], lh ? s.gx[4][0] : s.gy[4][0],
                       lh ? s.gx[5][0] : s.gy[5][0], aHh[1], false, x.psiHout[0][0], 0u);
        const float v1 = fmaf(-x.ch, lh ? zd - td : td - zd, S.hsel);
        float d1 = Ey[b + 1] - Ey[b];
        float d2 = Ex[b + W] - Ex[b];
        d1 = stretch_v(d1, sxh, s.gx[3][xe], s.gx[4][xe], s.gx[5][xe], aHh[2], false, x.psiHout[0][1], 0u);
        d2 = stretch_v(d2, syh, s.gy[3][ye], s.gy[4][ye], s.gy[5][ye], aHh[3], false, x.psiHout[1][0], 0u);
        const float hzv = fmaf(-x.ch, d1 - d2, S.hh2);
        const int hb = lh ? (hr + 1) * (TX + 1) : hr + 1;  // H slot of the halo cell
        (lh ? s.H[1] : s.H[0])[hb] = v1;
        s.H[2][hb] = hzv;
      } else if (hact) {
        // the column cell (i0-1, j0+hr) takes Hy and Hz, the row cell (i0+hr, j0-1)
        // Hx and Hz: one path for both, operands selected per lane.  The first
        // component is -(dt/dx)(z difference - transverse difference of Ez) for
        // the column and -(dt/dx)(y difference of Ez - z difference) for the row;
        // bit-identical to the two h_from calls it replaces
        const int b = lh ? (hr + 1) * W : hr + 1;  // E slot of the halo cell
        const float* z1 = lh ? Ex1 : Ey1;
        const float* z0 = lh ? Ex : Ey;
        float zd = z1[b] - z0[b];
        if (ZP) zd = stretch_z<true>(x, 0, S.gh, sz, h_off, zd, false, S.phz);
        const float td = Ez[b + (lh ? 1 : W)] - Ez[b];
        const float v1 = fmaf(-x.ch, lh ? zd - td : td - zd, S.hsel);
        const float hzv = fmaf(-x.ch, (Ey[b + 1] - Ey[b]) - (Ex[b + W] - Ex[b]), S.hh2);
        const int hb = lh ? (hr + 1) * (TX + 1) : hr + 1;  // H slot of the halo cell
        (lh ? s.H[1] : s.H[0])[hb] = v1;
        s.H[2][hb] = hzv;
      }
    }
    lds_barrier();
    // ---- E^{n+1} of plane k (own cell)
    float ex_n = 0.0f, ey_n = 0.0f, ez_n = 0.0f;
    if (act) {
      const int hs = (ty + 1) * (TX + 1) + tx + 1;
      const float hz_im = s.H[2][hs - 1], hy_im = s.H[1][hs - 1];
      const float hx_jm = s.H[0][hs - (TX + 1)], hz_jm = s.H[2][hs - (TX + 1)];
      const fd_mat& mt = s.mat[S.m];
      float dP[3] = {0.0f, 0.0f, 0.0f};
      float Pnew[3] = {0.0f, 0.0f, 0.0f};
      const bool g = GAIN && gk;
      float nh[3] = {0.0f, 0.0f, 0.0f}, nl[3] = {0.0f, 0.0f, 0.0f};
      if (g) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          nh[q] = gnh[q];
          nl[q] = gnl[q];
        }
      }
      if (GAIN == 1 && g) {
        const float n1 = nh[0] + nl[0], n2 = nh[1] + nl[1];
        float F[3] = {0.0f, 0.0f, 0.0f};
        if (mt.noise != 0.0f) {
          float gg[3];
          // the counter takes the dense cell index (k ny + j) nx + i
          normals3((uint32_t)n, ((uint32_t)k * (uint32_t)x.ny + (uint32_t)j) * (uint32_t)x.nx + (uint32_t)i,
                   d->key0, d->key1, gg);
          const float amp = mt.noise * sqrtf(fmaxf(n2, 0.0f));
#pragma unroll
          for (int q = 0; q < 3; ++q) F[q] = amp * gg[q];
        }
        const float dn = n1 - n2;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const float Pn = gPn[q];
          const float Pm = gPm[q];
          Pnew[q] = fmaf(mt.C1, Pn, fmaf(mt.C2, Pm, fmaf(mt.C3k * dn, eo[q], mt.C3 * F[q])));
          dP[q] = Pnew[q] - Pn;
        }
      }
      float cx = 0.0f, cy = 0.0f, cz = 0.0f;  // source terms dx*J of this cell
      for (unsigned mm = srcmask; mm; mm &= mm - 1u) {  // uniform; scalar loads only
        const int q = __builtin_ctz(mm);
        if (d->src_k[q] != k) continue;
        float v = n < d->src_len[q] ? ((const cfloat*)d->src_tab[q])[n] : 0.0f;
        if (!((srcmine >> q) & 1u)) continue;
        if (d->src_kind[q] == 2) v *= G(d->src_prof[q])[c];  // beam: transverse waist profile
        const int sc = d->src_comp[q];
        if (sc == 0) cx += v;
        else if (sc == 1) cy += v;
        else cz += v;
      }
      // av: E^{n+1} without the polarization current; on: not a PEC-held component
      float av[3] = {0.0f, 0.0f, 0.0f};
      bool on[3] = {false, false, false};
      if (PMM == 0) {
        // no CPML memory: plain selects for the components held by a PEC wall
        const bool pec_k = !x.pz && k == 0;  // uniform over the plane
        on[0] = !(pec_j | pec_k);
        on[1] = !(pec_k | pec_i);
        on[2] = !(pec_i | pec_j);
        const float v0 = fmaf(mt.cb, ((hz - hz_jm) - (hy - hym)) - cx, eo[0]);
        const float v1 = fmaf(mt.cb, ((hx - hxm) - (hz - hz_im)) - cy, eo[1]);
        const float v2 = fmaf(mt.cb, ((hy - hy_im) - (hx - hx_jm)) - cz, eo[2]);
        av[0] = on[0] ? v0 : 0.0f;
        av[1] = on[1] ? v1 : 0.0f;
        av[2] = on[2] ? v2 : 0.0f;
      } else {
      if (!(pec_j || (!x.pz && k == 0))) {  // Ex: d/dy Hz - d/dz Hy
        float d1 = hz - hz_jm, d2 = hy - hym;
        if (AX) {
          d1 = stretch_v(d1, syo, s.gy[0][ty + 1], s.gy[1][ty + 1], s.gy[2][ty + 1], aE[0], true, x.psiE[1][1], oy);
          d2 = stretch_v(d2, sz, gzE[0], gzE[1], gzE[2], aE[1], true, x.psiE[2][0], oz);
        } else if (PMM) {
          d1 = stretch<false, PMM>(x, 0, 1, j, i, j, k, d1, true);
          d2 = ZP ? stretch_z<false>(x, 0, S.ge, sz, c, d2, true, S.pe[0]) : stretch<false, PMM>(x, 0, 2, k, i, j, k, d2, true);
        }
        av[0] = fmaf(mt.cb, (d1 - d2) - cx, eo[0]);
        on[0] = true;
      }
      if (!((!x.pz && k == 0) || pec_i)) {  // Ey: d/dz Hx - d/dx Hz
        float d1 = hx - hxm, d2 = hz - hz_im;
        if (AX) {
          d1 = stretch_v(d1, sz, gzE[0], gzE[1], gzE[2], aE[2], true, x.psiE[2][1], oz);
          d2 = stretch_v(d2, sxo, s.gx[0][tx + 1], s.gx[1][tx + 1], s.gx[2][tx + 1], aE[3], true, x.psiE[0][0], ox);
        } else if (PMM) {
          d1 = ZP ? stretch_z<false>(x, 1, S.ge, sz, c, d1, true, S.pe[1]) : stretch<false, PMM>(x, 1, 2, k, i, j, k, d1, true);
          d2 = stretch<false, PMM>(x, 1, 0, i, i, j, k, d2, true);
        }
        av[1] = fmaf(mt.cb, (d1 - d2) - cy, eo[1]);
        on[1] = true;
      }
      if (!(pec_i || pec_j)) {  // Ez: d/dx Hy - d/dy Hx
        float d1 = hy - hy_im, d2 = hx - hx_jm;
        if (AX) {
          d1 = stretch_v(d1, sxo, s.gx[0][tx + 1], s.gx[1][tx + 1], s.gx[2][tx + 1], aE[4], true, x.psiE[0][1], ox);
          d2 = stretch_v(d2, syo, s.gy[0][ty + 1], s.gy[1][ty + 1], s.gy[2][ty + 1], aE[5], true, x.psiE[1][0], oy);
        } else if (PMM) {
          d1 = stretch<false, PMM>(x, 2, 0, i, i, j, k, d1, true);
          d2 = stretch<false, PMM>(x, 2, 1, j, i, j, k, d2, true);
        }
        av[2] = fmaf(mt.cb, (d1 - d2) - cz, eo[2]);
        on[2] = true;
      }
      }
      if (GAIN == 0) {
        // no polarization current: av is E^{n+1} (0 where a PEC wall holds it),
        // bit for bit what av - 0 / eps gives
        ex_n = av[0];
        ey_n = av[1];
        ez_n = av[2];
      } else {
        if (on[0]) ex_n = av[0] - dP[0] * mt.inv_eps;
        if (on[1]) ey_n = av[1] - dP[1] * mt.inv_eps;
        if (on[2]) ez_n = av[2] - dP[2] * mt.inv_eps;
      }
      put(x.Eout[0], o, ex_n);
      put(x.Eout[1], o, ey_n);
      put(x.Eout[2], o, ez_n);
      if (GAIN == 1 && g) {
        const float en[3] = {ex_n, ey_n, ez_n};
        float u = 0.0f;
#pragma unroll
        for (int q = 0; q < 3; ++q) u = fmaf(0.5f * (eo[q] + en[q]), dP[q] * mt.inv_dt, u);
        const float nn[4] = {1.0f - ((nh[0] + nh[1]) + nh[2]) - ((nl[0] + nl[1]) + nl[2]),
                             nh[0] + nl[0], nh[1] + nl[1], nh[2] + nl[2]};
        const int nc = d->ncell;
        gf* pop = G(d->pop);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          float inc = mt.Bu[r] * u;
#pragma unroll
          for (int q = 0; q < 4; ++q) inc = fmaf(mt.MI[r][q], nn[q], inc);
          two_sum(nh[r], nl[r], inc);
          pop[(size_t)r * nc + S.gi] = nh[r];
          pop[(size_t)(3 + r) * nc + S.gi] = nl[r];
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) G(d->P[par ^ 1][q])[S.gi] = Pnew[q];
      }
      for (unsigned mm = pmask; mm; mm &= mm - 1u) {  // uniform
        const int p = __builtin_ctz(mm);
        if (d->probe_k[p] != k || d->probe_cell[p] != c) continue;
        const int cp = d->probe_comp[p];
        s.probe[p] = cp == 0 ? ex_n : cp == 1 ? ey_n : cp == 2 ? ez_n : cp == 3 ? hx : cp == 4 ? hy : hz;
      }
      if (edue) {
        const float e2 = fmaf(eo[0], eo[0], fmaf(eo[1], eo[1], eo[2] * eo[2]));
        const float hh = fmaf(S.ho[0], hx, fmaf(S.ho[1], hy, S.ho[2] * hz));
        eacc += (double)(mt.eps * e2) + (double)hh;
      }
    }
    // own inputs two planes ahead into the Stage just consumed
    load_h(k + 2, S, k + 2 < k1);
    // transmitted power through flux planes at this k (uniform branch)
    if (FNEXT ? SP && k == nextf : fmask != 0u) {
      if (FNEXT) nextf = flux_from(k + 1);
#pragma unroll 1
      for (int f = 0; f < FD_MAXFLUX; ++f) {
        if (!((fmask >> f) & 1u) || d->flux_k[f] != k) continue;
        double v = 0.0;
        if (act) {
          const float sx = 0.5f * (eo[0] + ex_n), sy = 0.5f * (eo[1] + ey_n);
          const float hyc = 0.5f * (hym + hy), hxc = 0.5f * (hxm + hx);
          v = (double)(sx * hyc) - (double)(sy * hxc);
        }
        const double tot = block_sum(v, s.red);
        if (t == 0) s.ftot[f] = tot;
        // the plane's sample for the running DFT (E^n, H^{n+1/2} averaged onto the
        // plane), where all four values are at hand; it goes to its ring after the
        // march, so that the march's loads and stores are the same on every path
        int at = t;
        __asm__("" : "+v"(at));  // formed here: hoisted out of the march it would take a register per plane
        int st;
        float* sv = sample_at(f, at, st);
        sv[0] = eo[0];
        sv[st] = eo[1];
        sv[2 * st] = 0.5f * (hxm + hx);
        sv[3 * st] = 0.5f * (hym + hy);
      }
    }
    hxm = hx;
#pragma unroll
    for (int q = 0; q < 3; ++q) ecur[q] = enx[q];
    hym = hy;
  };

  // the loop body is both copies unconditionally (a path that skips the second
  // copy would make the compiler wait for every load at the loop head)
  int k = k0;
  for (; k + 1 < k1; k += 2) {
    plane_step(std::integral_constant<int, 0>(), k, SA);
    plane_step(std::integral_constant<int, 1>(), k + 1, SB);
  }
  if (k < k1) plane_step(std::integral_constant<int, 0>(), k, SA);
  // probe samples and T(t) partials gathered during the march
  if (pmask | fmask) {
    lds_barrier();
    if (t < FD_MAXPROBE && ((pmask >> t) & 1u)) G(d->probe_ring)[(long long)t * d->max_steps + n] = s.probe[t];
    if (t < FD_MAXFLUX && ((fmask >> t) & 1u)) G(d->flux_T[t])[n * d->nblk + tl.blk] = s.ftot[t];
  }
  // the DFT samples: a launch of its own for them took 4-6 us every decim steps (31
  // of 32 of the DFT's launches)
  for (unsigned mm = fmask; mm; mm &= mm - 1u) {  // uniform
    const int f = __builtin_ctz(mm);
    const uint32_t si = (uint32_t)(((uint64_t)(uint32_t)n * d->div_decim[f][0]) >> d->div_decim[f][1]);  // n / decim
    if (d->flux_nf[f] == 0 || si * (uint32_t)d->flux_decim[f] != (uint32_t)n || !act) continue;
    gf* ring = G(d->flux_ring[f]) + (size_t)(si % FD_DFT_RING) * 4 * (size_t)x.plane + c;
    int st;
    const float* sv = sample_at(f, t, st);
#pragma unroll
    for (int q = 0; q < 4; ++q) ring[(size_t)q * (size_t)x.plane] = sv[q * st];
  }
  if (edue) {
    const double tot = block_sum(eacc, s.red);
    if (t == 0) G(d->energy)[(n / d->ke) * d->ntiles + tl.tidx] = tot;
  }
}

// Workgroups are dealt to the 8 XCDs round-robin (workgroup w runs on XCD
// w mod 8), and each XCD has its own L2.  Renumber so that XCD x walks one
// contiguous eighth of the tile list: tiles adjacent in the list (x, y and z
// neighbours, whose halos overlap) then share an L2.  A bijection on [0, n).
__device__ __forceinline__ int xcd_tile(int w, int n) {
  constexpr int kXcd = 8;
  const int q = n / kXcd, r = n % kXcd;
  const int x = w % kXcd, s = w / kXcd;
  return x * q + (x < r ? x : r) + s;
}

// With a cost-balanced partition (use_part), workgroup w takes tile
// part.start[x] + w/8 of XCD x = w mod 8, or nothing if that part is shorter; with
// bit 1 of use_part set, each part from its end.  Steps of grids beyond the
// Infinity Cache alternate: a step then starts with the tiles whose fields the
// step before wrote last and the Infinity Cache still holds (200x200x200 slab with
// ordinary stores 128 -> 115 us, 176x176x176 78.6 -> 74.8; with non-temporal ones
// 110.0 -> 109.4 and 72.6 -> 72.3; in the cache 16 batched realizations took 228.4
// -> 229.8).
// Without a partition the workgroups loop over the renumbered tile list.
// FORM: 0 the partition, 1 the loop, 2 either.  The plain and all-axes classes with
// Lorentz gain have the loop in kernels of their own: what it keeps in registers cost
// the partition's form 17 VGPRs (32 wide: plain 142 -> 125 and four waves per SIMD,
// all-axes 168 -> 151; 128x128x96 with gain 36.2 -> 33.4 us per step, the 168^3 box
// 150.9 -> 148.6).  The z-CPML class with gain lost 1% apart (160^3 84.3 -> 85.1), the
// classes without gain nothing or up to 0.7%; one call of the march for both forms
// made every class slower (the 200^3 box 135.5 -> 149.3 us).
constexpr bool loop_apart(int pm, int gain) { return gain != 0 && pm != 4; }
template <int TX, int PM, int GAIN, bool NT, int FORM>
__device__ __forceinline__ void step_body(const fd_tile* __restrict__ tiles, int ntiles, int s, const fd_xcd& part,
                                          int use_part, Lds<TX>& lds) {
  // A march without the code of sources, probes, flux planes and energy for the
  // tiles that have none; z-only CPML launches specialise their interior tiles, and
  // all-axes launches without gain their lean tiles off the x and y slabs, which lose
  // the psi registers and tests of those axes (a folded or merged launch holds them:
  // 200x200x200 box 139.5 -> 138.0 us, with the x slabs apart 139.9 -> 135.4).  With gain
  // they cost more than they save: a gain cell's state sets the registers of every
  // march (168^3 Lorentz box 148.9 -> 151.8 us, 84^3, 32 wide, 29.3 -> 31.6).
  // Inlined by hand: as a call, which the compiler chose for the z-CPML class with
  // gain, the marches took 264 VGPRs instead of 146 (160x160x160, 111 us and 84).
  auto run = [&](const fd_tile& tl) __attribute__((always_inline)) {
    // (the look at the step only in plans that record the energy: it is a round trip
    // before the tile's first loads)
    bool edue = false;
    if (tl.flags & FD_TILE_KE) {
      const cdesc* d = (const cdesc*)tl.d;
      edue = energy_due(d, d->step + s);
      // a plan's two tile sets take turns by whether the step records the energy
      // (never in the looped form)
      if (tl.flags & (edue ? FD_TILE_NOENERGY : FD_TILE_ENERGY)) return;
    }
    const bool sp = edue | ((tl.srcmask | tl.pmask | tl.fmask) != 0u);
    if constexpr (PM == 4) {
      if (!(tl.flags & FD_TILE_ZSLAB)) {
        if (sp) run_tile<TX, PM, GAIN, false, NT, true>(tl, s, lds);
        else run_tile<TX, PM, GAIN, false, NT, false>(tl, s, lds);
        return;
      }
    }
    if constexpr (PM == 7 && GAIN == 0) {
      if (!sp && !(tl.flags & FD_TILE_XYSLAB)) {
        if (tl.flags & FD_TILE_ZSLAB) run_tile<TX, 4, GAIN, true, NT, false>(tl, s, lds);
        else run_tile<TX, 4, GAIN, false, NT, false>(tl, s, lds);
        return;
      }
    }
    if (sp) run_tile<TX, PM, GAIN, (PM & 4) != 0, NT, true>(tl, s, lds);
    else run_tile<TX, PM, GAIN, (PM & 4) != 0, NT, false>(tl, s, lds);
  };
  if (FORM == 0 || (FORM == 2 && use_part)) {
    const int x = (int)blockIdx.x % 8, q = (int)blockIdx.x / 8;
    if (q < part.count[x]) {
      const fd_tile tl = tiles[part.start[x] + (use_part & 2 ? part.count[x] - 1 - q : q)];
      run(tl);
    }
    return;
  }
  if constexpr (FORM != 0) {
    for (int w = blockIdx.x; w < ntiles; w += gridDim.x) {
      const fd_tile tl = tiles[xcd_tile(w, ntiles)];
      run(tl);
    }
  }
}

// All-axes CPML with Lorentz gain: held at three waves per SIMD (151 VGPRs; with 180,
// two waves, the 168^3 box took 191 us per step instead of 150).
template <int TX, int PM, int GAIN, bool NT>
__global__ __launch_bounds__(FD_MAXBLOCK) __attribute__((amdgpu_waves_per_eu(PM == 7 && GAIN ? 3 : 1))) void step_kernel(
    const fd_tile* __restrict__ tiles, int ntiles, int s, fd_xcd part, int use_part) {
  __shared__ Lds<TX> lds;
  step_body<TX, PM, GAIN, NT, loop_apart(PM, GAIN) ? 0 : 2>(tiles, ntiles, s, part, use_part, lds);
}

// All-axes CPML without gain: capped at four waves per SIMD (128 VGPRs; the
// compiler alone takes 134 and three waves), 7% faster on the beam box.
template <int TX, bool NT>
__global__ __launch_bounds__(FD_MAXBLOCK) __attribute__((amdgpu_waves_per_eu(4))) void step_kernel_ax(
    const fd_tile* __restrict__ tiles, int ntiles, int s, fd_xcd part, int use_part) {
  __shared__ Lds<TX> lds;
  step_body<TX, 7, 0, NT, 2>(tiles, ntiles, s, part, use_part, lds);
}

template <int TX, int PM, bool NT>
__global__ __launch_bounds__(FD_MAXBLOCK) __attribute__((amdgpu_waves_per_eu(3))) void step_kernel_gain_loop(
    const fd_tile* __restrict__ tiles, int ntiles, int s, fd_xcd part) {
  __shared__ Lds<TX> lds;
  step_body<TX, PM, 1, NT, 1>(tiles, ntiles, s, part, 0, lds);
}

}  // namespace

// start/stop (optional) take the kernel's own begin and end timestamps
template <int TX, int PM, int GAIN>
static void launch_one(const fd_tile* tiles, int ntiles, int block, int grid, int s, const fd_xcd& part, int use,
                       int nt, unsigned lds, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  if constexpr (loop_apart(PM, GAIN)) {
    if (!use) {
      if (nt)
        hipExtLaunchKernelGGL(step_kernel_gain_loop<TX, PM, true>, dim3(grid), dim3(block), lds, st, start, stop, 0,
                              tiles, ntiles, s, part);
      else
        hipExtLaunchKernelGGL(step_kernel_gain_loop<TX, PM, false>, dim3(grid), dim3(block), lds, st, start, stop, 0,
                              tiles, ntiles, s, part);
      return;
    }
  }
  if constexpr (PM == 7 && GAIN == 0) {
    if (nt)
      hipExtLaunchKernelGGL(step_kernel_ax<TX, true>, dim3(grid), dim3(block), lds, st, start, stop, 0, tiles, ntiles,
                            s, part, use);
    else
      hipExtLaunchKernelGGL(step_kernel_ax<TX, false>, dim3(grid), dim3(block), lds, st, start, stop, 0, tiles, ntiles,
                            s, part, use);
  } else if (nt) {
    hipExtLaunchKernelGGL(step_kernel<TX, PM, GAIN, true>, dim3(grid), dim3(block), lds, st, start, stop, 0, tiles,
                          ntiles, s, part, use);
  } else {
    hipExtLaunchKernelGGL(step_kernel<TX, PM, GAIN, false>, dim3(grid), dim3(block), lds, st, start, stop, 0, tiles,
                          ntiles, s, part, use);
  }
}

#define FD_CAT(a, b) a##b
#define FD_STEP_NAME(tx) FD_CAT(fd_launch_step_, tx)
hipError_t FD_STEP_NAME(FD_STEP_TX)(int cls, const fd_tile* tiles, int ntiles, int block, int grid, int s,
                            const fd_xcd& part, int use, int nt, unsigned lds, hipStream_t st, hipEvent_t start,
                            hipEvent_t stop) {
  switch (cls) {
    case FD_CLASS_PLAIN: launch_one<FD_STEP_TX, 0, 0>(tiles, ntiles, block, grid, s, part, use, nt, lds, st, start, stop); break;
    case FD_CLASS_PMLZ: launch_one<FD_STEP_TX, 4, 0>(tiles, ntiles, block, grid, s, part, use, nt, lds, st, start, stop); break;
    case FD_CLASS_PML: launch_one<FD_STEP_TX, 7, 0>(tiles, ntiles, block, grid, s, part, use, nt, lds, st, start, stop); break;
    case FD_CLASS_GAIN: launch_one<FD_STEP_TX, 0, 1>(tiles, ntiles, block, grid, s, part, use, nt, lds, st, start, stop); break;
    case FD_CLASS_PMLZ_GAIN: launch_one<FD_STEP_TX, 4, 1>(tiles, ntiles, block, grid, s, part, use, nt, lds, st, start, stop); break;
    case FD_CLASS_PML_GAIN: launch_one<FD_STEP_TX, 7, 1>(tiles, ntiles, block, grid, s, part, use, nt, lds, st, start, stop); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

