// The fused Yee step without a march, for gfx950: small grids.
//
// Same operation and the same per-sample arithmetic as step_tile in
// yee_kernels.hpp, so the bits are the same.
//
// What bounds a small grid is the chain of dependent waits inside one launch,
// not bandwidth: step_tile fills tables, waits, loads a plane, waits, and then
// walks its planes one after another, each waiting for loads issued a plane
// earlier.  Here a workgroup owns ty rows of one plane and that chain is as
// short as it gets: one sample per lane, every load (the planes below and
// above, the row above, auxiliaries, profiles) is issued at the start straight
// into registers, H^{n+1/2} of the plane below is recomputed instead of
// carried, and one barrier, between the H and the E half step, hands H of the
// row below to each row.  The price is about 1.6 times the arithmetic and
// twice the cache reads per cell, which a small grid has room for.
//
// Measured per step against the march (us): 32^3 FP64 without CPML 8.8 -> 4.0,
// 12 x 12 x 140 FP32 8.5 -> 4.1, 32^3 FP32 with CPML 8 11.1 -> 4.0, 64^3 FP32
// 12.9 -> 8.5, 80^3 20.3 -> 17.2, 96^3 22.8 -> 23.5, 128^3 33 -> 41 (direct_rows
// in yee_runtime.hip draws the line).
#pragma once

#include "yee_kernels.hpp"

namespace yee {

// LDS of a workgroup, in compute-type elements:
//   H rows j0-1 .. j0+ty-1        [ty+1][2][RL]   (Hx, Hz; RL = 64 wpr)
//   the last Hy sample of a wave  [ty+1][wpr]
//   source values                 [kMaxSources]
//   int32: tile row (0: not here) and 4 i + component of each source  [2][kMaxSources]
__host__ __device__ inline size_t direct_lds_bytes_for(int ty, int wpr, size_t csize) {
  return (((size_t)(ty + 1) * (2 * (size_t)wpr * kWave + wpr) + kMaxSources) * csize + 2 * kMaxSources * 4 + 15) &
         ~size_t(15);
}

// CPML profile of one sample
template <class C>
struct Prof {
  C omb, a, kinv;   // 1 - b, a, 1/kappa
};

// lane i gets lane i+1's value (0 into lane 63); lane i-1's (0 into lane 0)
template <class C, int CTRL>
__device__ __forceinline__ C lane_shift(C v) {
  if constexpr (sizeof(C) == 8) {
    const u32x2 w = __builtin_bit_cast(u32x2, v);
    const unsigned int a = w.x, b = w.y;
    u32x2 o;
    o.x = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)a, CTRL, 0xF, 0xF, true);
    o.y = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(C, o);
  } else {
    return __builtin_bit_cast(C, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
  }
}
template <class C>
__device__ __forceinline__ C lane_next(C v) { return lane_shift<C, 0x130>(v); }
template <class C>
__device__ __forceinline__ C lane_prev(C v) { return lane_shift<C, 0x138>(v); }

// SEAM: rows of several waves (nx > 64).
template <class T, class C, bool SEAM, int EXTRA = kPlain>
__device__ __forceinline__ void direct_tile(const StepArgs<T, C>& a, const int ytile, const int k,
                                            unsigned char* smem_raw) {
  constexpr bool nt = EXTRA == kStream;
  constexpr uint32_t TB = sizeof(T), CB = sizeof(C);
  const int wpr = SEAM ? a.wpr : 1;
  const int ty = a.ty;
  const int RL = wpr * kWave;
  C* ldsH = reinterpret_cast<C*>(smem_raw);
  C* ldsY = ldsH + (ty + 1) * 2 * RL;
  C* ldsS = ldsY + (ty + 1) * wpr;
  int32_t* ldsK = reinterpret_cast<int32_t*>(ldsS + kMaxSources);
  const int nx = a.nx, ny = a.ny, nz = a.nz, px = a.px;
  const int Lx = a.L[0], Ly = a.L[1], Lz = a.L[2];
  const int j0 = ytile * ty;
  const int tid = threadIdx.x;

  // ---- the wave's row (uniform) ----
  const int wid = uniform(tid >> 6);
  const int lane = tid & 63;
  if (wid >= (ty + 1) * wpr) {
    // one wave more where there are sources: it evaluates the waveforms of
    // those the tile holds while the rows' loads are in flight
    if (lane < a.nsrc) {
      const SrcDev sd = a.src[lane];
      const bool here = sd.k == k && sd.j >= j0 && sd.j < j0 + ty;
      ldsK[lane] = here ? sd.j - j0 + 1 : 0;
      if (here) {
        ldsK[kMaxSources + lane] = 4 * sd.i + sd.comp;
        ldsS[lane] = static_cast<C>(sd.amp * waveform(sd, (double)(a.n + 1) * a.dt));
      }
    }
    __syncthreads();
    return;
  }
  const int r = SEAM ? wid / wpr : wid;              // tile row: 0 = halo row j0-1
  const int xs = SEAM ? wid - r * wpr : 0;           // x segment of the row
  const int j = j0 - 1 + r;
  const bool row_ok = j >= 0 && j < ny;
  const bool own = row_ok && r > 0;
  const int jc = min(max(j, 0), ny - 1);
  const int km = max(k - 1, 0);                      // (plane -1: nothing is loaded)
  const bool below = own && k > 0;                   // H of the plane below: Hx, Hy of the own rows
  const bool iny = row_ok && (j < Ly || j >= ny - Ly);
  const bool inz = row_ok && (k < Lz || k >= nz - Lz);
  const bool inzm = below && (km < Lz || km >= nz - Lz);
  const int i = xs * kWave + lane;
  const bool lane_ok = i < nx;
  const bool wave_inx = row_ok && Lx > 0 && (xs * kWave < Lx || xs * kWave + kWave > nx - Lx);
  const bool inx = wave_inx && lane_ok && (i < Lx || i >= nx - Lx);

  // ---- per-lane byte offsets (kOut: nothing there) ----
  const uint32_t plane_b = (uint32_t)ny * (uint32_t)px * TB;
  const uint32_t o = ((uint32_t)jc * (uint32_t)px + (uint32_t)i) * TB;
  const uint32_t vr = (row_ok && lane_ok) ? o : kOut;
  const uint32_t vm = below ? vr : kOut;
  const uint32_t vu = j + 1 < ny ? vr + (uint32_t)px * TB : kOut;      // row above (kOut stays out of range)
  const uint32_t vum = below ? vu : kOut;
  const uint32_t vn = (SEAM && lane == kWave - 1 && row_ok && i + 1 < nx) ? o + TB : kOut;   // x+1 in the next wave
  const uint32_t vc = (row_ok && lane_ok) ? (uint32_t)i * 2 * CB : kOut;                     // y and z pairs
  const uint32_t vx = (uint32_t)(i < Lx ? i : i - nx + 2 * Lx) * 2 * CB;                     // x pairs (inx lanes)
  const uint32_t cs_b = (uint32_t)(a.cstride * TB);
  const rsrc_t rin = make_rsrc(a.fin, 6 * cs_b);
  const rsrc_t rout = make_rsrc(a.fout, 6 * cs_b);
  const char* psb = reinterpret_cast<const char*>(a.pse);
  const uint32_t phin = (uint32_t)(reinterpret_cast<const char*>(a.psh_in) - psb);
  const uint32_t phout = (uint32_t)(reinterpret_cast<const char*>(a.psh_out) - psb);
  const rsrc_t rpsi = make_rsrc(a.pse, max(phin, phout) + a.psi_bytes);
  const rsrc_t rcoef = make_rsrc(a.coef, a.coef_bytes);
  const C idx_ = a.inv_d[0], idy = a.inv_d[1], idz = a.inv_d[2];
  const C dtm = a.dt_mu;
  const int sy = j < Ly ? j : j - ny + 2 * Ly;
  auto yso = [&](int kk) { return (a.psoff[PEXY] + ((uint32_t)kk * (2 * Ly) + sy) * (uint32_t)px * 2) * CB; };
  auto zso = [&](int kk) {
    const int sz = kk < Lz ? kk : kk - nz + 2 * Lz;
    return (a.psoff[PEXZ] + ((uint32_t)sz * ny + jc) * (uint32_t)px * 2) * CB;
  };
  auto xso = [&](int kk) { return (a.psoff[PEYX] + ((uint32_t)kk * ny + jc) * (uint32_t)(2 * Lx) * 2) * CB; };

  // ---- loads ----
  // (the material block first: the coefficients wait for it; vector loads
  // without branches throughout, so that nothing waits in between)
  const rsrc_t rseg = make_rsrc(a.seg, (uint32_t)(px + ny + nz) * 4);
  const rsrc_t rflag = make_rsrc(a.rowflag, (uint32_t)nz * (uint32_t)ny);
  const uint32_t v0 = own ? 0u : kOut;
  const uint32_t bx = buf_ld<uint32_t>(rseg, (own && lane_ok) ? (uint32_t)i * 4 : kOut, 0);
  const uint32_t by = buf_ld<uint32_t>(rseg, v0, (uint32_t)(px + jc) * 4);
  const uint32_t bz = buf_ld<uint32_t>(rseg, v0, (uint32_t)(px + ny + k) * 4);
  const uint32_t vflags = __builtin_amdgcn_raw_buffer_load_b8(rflag, v0, (uint32_t)k * (uint32_t)ny + (uint32_t)jc, 0);
  auto ldE = [&](uint32_t vo, int kk, int c) __attribute__((always_inline)) {
    return buf_ld<VecT<T, 1>>(rin, vo, (uint32_t)kk * plane_b + (uint32_t)c * cs_b).v[0];
  };
  const T qx0 = ldE(vr, k, 0), qy0 = ldE(vr, k, 1), qz0 = ldE(vr, k, 2);        // E^n(k)
  const T qxp = ldE(vr, k + 1, 0), qyp = ldE(vr, k + 1, 1);                      // E^n(k+1) (plane nz: zero)
  const T qxu = ldE(vu, k, 0), qzu = ldE(vu, k, 2);                              // row j+1
  const T qhx = ldE(vr, k, 3), qhy = ldE(own ? vr : kOut, k, 4), qhz = ldE(vr, k, 5);
  const T qxm = ldE(vm, km, 0), qym = ldE(vm, km, 1), qzm = ldE(vm, km, 2);      // E^n(k-1)
  const T qzum = ldE(vum, km, 2);
  const T qhxm = ldE(vm, km, 3), qhym = ldE(vm, km, 4);
  T qyn = T(0), qzn = T(0), qznm = T(0);
  if constexpr (SEAM) {
    qyn = ldE(vn, k, 1);
    qzn = ldE(vn, k, 2);
    qznm = ldE(below ? vn : kOut, km, 2);
  }
  const int pln = a.pec_plane[k];
  // Auxiliaries (H side of planes k and k-1, E side of plane k) and profiles
  // of the layers the wave is in
  auto profile = [&](int side, int axis, int q) __attribute__((always_inline)) {
    return reinterpret_cast<const Prof<C>*>(a.prof)[(side * 3 + axis) * a.plen + q];   // one load
  };
  Pair<C> yh{}, yhm{}, ye{}, zh{}, zhm{}, ze{}, xh{}, xhm{}, xe{};
  Prof<C> yph{}, ype{}, zph{}, zpe{}, zpm{}, xph{C(0), C(0), C(1)}, xpe = xph;
  if (iny) {
    yh = buf_ld<Pair<C>>(rpsi, vc, phin + yso(k));
    yhm = buf_ld<Pair<C>>(rpsi, below ? vc : kOut, phin + yso(km));
    ye = buf_ld<Pair<C>>(rpsi, own ? vc : kOut, yso(k));
    yph = profile(1, 1, jc);
    ype = profile(0, 1, jc);
  }
  if (inz) {
    zh = buf_ld<Pair<C>>(rpsi, vc, phin + zso(k));
    ze = buf_ld<Pair<C>>(rpsi, own ? vc : kOut, zso(k));
    zph = profile(1, 2, k);
    zpe = profile(0, 2, k);
  }
  if (inzm) {
    zhm = buf_ld<Pair<C>>(rpsi, vc, phin + zso(km));
    zpm = profile(1, 2, km);
  }
  if (inx) {
    xh = buf_ld<Pair<C>>(rpsi, vx, phin + xso(k));
    xhm = buf_ld<Pair<C>>(rpsi, below ? vx : kOut, phin + xso(km));
    xe = buf_ld<Pair<C>>(rpsi, own ? vx : kOut, xso(k));
    xph = profile(1, 0, i);
    xpe = profile(0, 0, i);
  }
  const Coef2<C> cf = buf_ld<Coef2<C>>(rcoef, (own && lane_ok) ? (bx + by * (uint32_t)a.nsx + bz * (uint32_t)a.nsxy) * (uint32_t)sizeof(Coef2<C>) : kOut, 0);
  uint32_t pm = 0u;
  if (pln >= 0 && own && lane_ok) pm = a.pec_mask[((size_t)pln * ny + jc) * px + i];

  // ---- H half step at plane k, and Hx, Hy of the plane below ----
  auto dec = [&](T v, int c) __attribute__((always_inline)) { return Conv<T, C>::ld(v, a.dec[c]); };
  const C ex = dec(qx0, 0), ey = dec(qy0, 1), ez = dec(qz0, 2);
  C hx = C(0), hy = C(0), hz = C(0), hxm = C(0), hym = C(0);
  T bhx = T(0), bhy = T(0), bhz = T(0);
  {
    C eyr = lane_next<C>(ey), ezr = lane_next<C>(ez);
    if constexpr (SEAM) {
      eyr = lane == kWave - 1 ? dec(qyn, 1) : eyr;
      ezr = lane == kWave - 1 ? dec(qzn, 2) : ezr;
    }
    C dEz_dy = fdiff(dec(qzu, 2), ez, idy), dEy_dz = fdiff(dec(qyp, 1), ey, idz);
    C dEx_dz = fdiff(dec(qxp, 0), ex, idz), dEz_dx = fdiff(ezr, ez, idx_);
    C dEy_dx = fdiff(eyr, ey, idx_), dEx_dy = fdiff(dec(qxu, 0), ex, idy);
    if (iny) {
      dEz_dy = cpml_term(yh.a, dEz_dy, yph.omb, yph.a, yph.kinv);
      dEx_dy = cpml_term(yh.b, dEx_dy, yph.omb, yph.a, yph.kinv);
    }
    if (inz) {
      dEy_dz = cpml_term(zh.a, dEy_dz, zph.omb, zph.a, zph.kinv);
      dEx_dz = cpml_term(zh.b, dEx_dz, zph.omb, zph.a, zph.kinv);
    }
    if (wave_inx) {   // lanes outside the layer: (1 - b, a, 1/kappa) = (0, 0, 1), psi 0
      dEz_dx = cpml_term(xh.a, dEz_dx, xph.omb, xph.a, xph.kinv);
      dEy_dx = cpml_term(xh.b, dEy_dx, xph.omb, xph.a, xph.kinv);
    }
    // lanes and rows beyond the grid publish zeros
    if (row_ok && lane_ok) {
      hx = to_storage<T, C>(h_new(dec(qhx, 3), dEz_dy, dEy_dz, dtm), a.enc[3], a.dec[3], bhx);
      hy = to_storage<T, C>(h_new(dec(qhy, 4), dEx_dz, dEz_dx, dtm), a.enc[4], a.dec[4], bhy);
      hz = to_storage<T, C>(h_new(dec(qhz, 5), dEy_dx, dEx_dy, dtm), a.enc[5], a.dec[5], bhz);
    }
  }
  if (below) {
    const C exm = dec(qxm, 0), eym = dec(qym, 1), ezm = dec(qzm, 2);
    C ezr = lane_next<C>(ezm);
    if constexpr (SEAM) ezr = lane == kWave - 1 ? dec(qznm, 2) : ezr;
    C dEz_dy = fdiff(dec(qzum, 2), ezm, idy), dEy_dz = fdiff(ey, eym, idz);
    C dEx_dz = fdiff(ex, exm, idz), dEz_dx = fdiff(ezr, ezm, idx_);
    if (iny) dEz_dy = cpml_term(yhm.a, dEz_dy, yph.omb, yph.a, yph.kinv);
    if (inzm) {
      dEy_dz = cpml_term(zhm.a, dEy_dz, zpm.omb, zpm.a, zpm.kinv);
      dEx_dz = cpml_term(zhm.b, dEx_dz, zpm.omb, zpm.a, zpm.kinv);
    }
    if (wave_inx) dEz_dx = cpml_term(xhm.a, dEz_dx, xph.omb, xph.a, xph.kinv);
    if (lane_ok) {
      hxm = to_storage<T, C>(h_new(dec(qhxm, 3), dEz_dy, dEy_dz, dtm), a.enc[3], a.dec[3]);
      hym = to_storage<T, C>(h_new(dec(qhym, 4), dEx_dz, dEz_dx, dtm), a.enc[4], a.dec[4]);
    }
  }
  C* myH = ldsH + r * 2 * RL + i;
  myH[0] = hx;
  myH[RL] = hz;
  if constexpr (SEAM) {
    if (lane == kWave - 1) ldsY[r * wpr + xs] = hy;
  }
  __syncthreads();
  if (!own) return;

  // ---- E half step of the own rows, stores ----
  const int flags = uniform((int)vflags);
  int4 probe0 = make_int4(0, 0, -1, -1);
  if ((flags & 2) && lane < a.nprobe) probe0 = a.probe[lane];
  const C hxd = myH[-2 * RL], hzd = myH[-RL];        // row j-1
  C hyl = lane_prev<C>(hy), hzl = lane_prev<C>(hz);
  if constexpr (SEAM) {
    if (lane == 0 && xs > 0) {
      hyl = ldsY[r * wpr + xs - 1];
      hzl = myH[RL - 1];
    }
  }
  C dHz_dy = fdiff(hz, hzd, idy), dHy_dz = fdiff(hy, hym, idz), dHx_dz = fdiff(hx, hxm, idz);
  C dHz_dx = fdiff(hz, hzl, idx_), dHy_dx = fdiff(hy, hyl, idx_), dHx_dy = fdiff(hx, hxd, idy);
  if (iny) {
    dHz_dy = cpml_term(ye.a, dHz_dy, ype.omb, ype.a, ype.kinv);
    dHx_dy = cpml_term(ye.b, dHx_dy, ype.omb, ype.a, ype.kinv);
  }
  if (inz) {
    dHy_dz = cpml_term(ze.a, dHy_dz, zpe.omb, zpe.a, zpe.kinv);
    dHx_dz = cpml_term(ze.b, dHx_dz, zpe.omb, zpe.a, zpe.kinv);
  }
  if (wave_inx) {
    dHz_dx = cpml_term(xe.a, dHz_dx, xpe.omb, xpe.a, xpe.kinv);
    dHy_dx = cpml_term(xe.b, dHy_dx, xpe.omb, xpe.a, xpe.kinv);
  }
  C eo[3];
  eo[0] = e_new(ex, dHz_dy, dHy_dz, pm & 1 ? C(0) : cf.ca, pm & 1 ? C(0) : cf.cb);
  eo[1] = e_new(ey, dHx_dz, dHz_dx, pm & 2 ? C(0) : cf.ca, pm & 2 ? C(0) : cf.cb);
  eo[2] = e_new(ez, dHy_dx, dHx_dy, pm & 4 ? C(0) : cf.ca, pm & 4 ? C(0) : cf.cb);
  // E samples on the outer faces are never updated; their auxiliaries stay 0
  // (pairs: y (XY, ZY), z (XZ, YZ), x (YX, ZX))
  const bool wx = j == 0 || k == 0, wy = i == 0 || k == 0, wz = i == 0 || j == 0;
  eo[0] = wx ? ex : eo[0];
  eo[1] = wy ? ey : eo[1];
  eo[2] = wz ? ez : eo[2];
  if (iny) {
    buf_st<Pair<C>>(yh, rpsi, vc, phout + yso(k), nt);
    buf_st<Pair<C>>(Pair<C>{wx ? C(0) : ye.a, wz ? C(0) : ye.b}, rpsi, vc, yso(k), nt);
  }
  if (inz) {
    buf_st<Pair<C>>(zh, rpsi, vc, phout + zso(k), nt);
    buf_st<Pair<C>>(Pair<C>{wx ? C(0) : ze.a, wy ? C(0) : ze.b}, rpsi, vc, zso(k), nt);
  }
  if (inx) {
    buf_st<Pair<C>>(xh, rpsi, vx, phout + xso(k), nt);
    buf_st<Pair<C>>(Pair<C>{wy ? C(0) : xe.a, wz ? C(0) : xe.b}, rpsi, vx, xso(k), nt);
  }
  if (flags & 1) {
    for (int s = 0; s < a.nsrc; ++s) {
      if (ldsK[s] == r && ldsK[kMaxSources + s] >> 2 == i) {
        const C v = ldsS[s];
        const int sc = ldsK[kMaxSources + s] & 3;
        eo[0] = sc == 0 ? eo[0] + v : eo[0];
        eo[1] = sc == 1 ? eo[1] + v : eo[1];
        eo[2] = sc == 2 ? eo[2] + v : eo[2];
      }
    }
  }
  T be[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) eo[c] = to_storage<T, C>(eo[c], a.enc[c], a.dec[c], be[c]);
  const uint32_t so = (uint32_t)k * plane_b;
  if constexpr (std::is_same<T, C>::value) {
    be[0] = eo[0]; be[1] = eo[1]; be[2] = eo[2];
    bhx = hx; bhy = hy; bhz = hz;
  }
  const T bh[3] = {bhx, bhy, bhz};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    buf_st<VecT<T, 1>>(VecT<T, 1>{{be[c]}}, rout, vr, so + (uint32_t)c * cs_b, nt);
    buf_st<VecT<T, 1>>(VecT<T, 1>{{bh[c]}}, rout, vr, so + (uint32_t)(3 + c) * cs_b, nt);
  }
  if constexpr (EXTRA == kWriteCount) {
    if (vr != kOut) {
#pragma unroll
      for (int c = 0; c < 6; ++c) atomicAdd(a.wcount + (size_t)c * a.cstride + (so + vr) / TB, 1u);
    }
  }
  if constexpr (EXTRA == kHistory) {
    // E^{n+1} of the box cells of this row and plane (adjoint history)
    if (k >= a.hbox[4] && k < a.hbox[5] && j >= a.hbox[2] && j < a.hbox[3] && i >= a.hbox[0] && i < a.hbox[1]) {
      const int hbx = a.hbox[1] - a.hbox[0], hby = a.hbox[3] - a.hbox[2];
      T* hp = a.hist + ((size_t)(k - a.hbox[4]) * hby + (j - a.hbox[2])) * hbx + (i - a.hbox[0]);
#pragma unroll
      for (int c = 0; c < 3; ++c) hp[c * a.hstride] = be[c];
    }
  }
  if (flags & 2) {
    // lanes look at the probes side by side; the row's own ones are few
    for (int p0 = 0; p0 < a.nprobe; p0 += kWave) {
      int4 pr = probe0;
      if (p0 > 0) pr = p0 + lane < a.nprobe ? a.probe[p0 + lane] : make_int4(0, 0, -1, -1);
      uint64_t m = __ballot(pr.z == j && pr.w == k);
      while (m) {
        const int b = (int)__builtin_ctzll(m);
        m &= m - 1;
        const int pc = __builtin_amdgcn_readlane(pr.x, b), pi = __builtin_amdgcn_readlane(pr.y, b);
        if (i == pi) {
          const C v = pc == 0 ? eo[0] : pc == 1 ? eo[1] : pc == 2 ? eo[2] : pc == 3 ? hx : pc == 4 ? hy : hz;
          a.series[(size_t)a.series_slot * a.nprobe + p0 + b] = static_cast<double>(v);
        }
      }
    }
  }
}

template <class T, class C, bool SEAM, int EXTRA = kPlain>
__global__ void __launch_bounds__(kWave * kMaxBlockWaves)
direct_kernel(const StepArgs<T, C> a) {
  extern __shared__ unsigned char smem_raw[];
  direct_tile<T, C, SEAM, EXTRA>(a, blockIdx.x, blockIdx.y, smem_raw);
}

}  // namespace yee
