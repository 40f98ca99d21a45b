// Sixth-order AT step (gfx950): the (1,6) first derivative of Appendix B (Table atschemes, (1,6)
// rows) in the flux form of the fourth-order path, with three ghost layers per face and ghost
// values extrapolated from four published levels (cubic in time; the Appendix B weights at c_s = 0).
//
// Work decomposition.  A workgroup owns a column tile of at most 256 points that lies inside one PE
// along x and y (tile6_of: the PE's face is cut into equal tiles, the last of a row or column may
// be narrower) and marches through a z chunk of one PE.  Every point outside the workgroup's box
// that a stencil reaches is therefore across exactly one face of the workgroup's own PE, or inside
// that PE: a point across a face whose delay k is >= 1 takes the extrapolated value
// w_0 v^{n-k} + w_1 v^{n-k-1} + w_2 v^{n-k-2} + w_3 v^{n-k-3} (kappa = k + c_s), any other point its
// current value.  Each stage is two launches:
//
//  k6_gradflux: primitives, the 12 velocity and temperature gradients at the tile's points (x, y
//    from an LDS plane with a 3-point halo, z from a 7-plane register window of the column), the
//    total fluxes F_x, F_y, F_z (written to the flux buffer), and at stage 1 the publication of the
//    three layers next to each PE face (u, v, w, T and the face-normal flux) into ring slot n mod R;
//  k6_divupdate: the flux divergence (F_x, F_y through LDS planes with a 3-point halo, F_z through a
//    7-plane register window) with ghost fluxes from the ring across delayed faces, then the
//    low-storage RK3 (or Adams-Bashforth) update and the FP64 block totals, or the RHS output.
//
// The fluxes make one round trip through HBM (15 words written, then read), which the fused
// fourth-order kernel avoids; in exchange every point's flux is computed once.
#include <algorithm>

#include "atns_internal.h"

namespace atns {
namespace {

constexpr int kM6 = 3;  // layers per face

template <typename T>
struct A6 {
  const T* q;
  T* q_out;
  T* dq;
  T* flux;           // [3][5][N]: F_d of conserved component c at [(d 5 + c) N + i]
  T* ring;
  T* gv;             // extrapolated values behind the faces, ring-slot layout: this stage's (stage
                     // kernels), or the first of nst consecutive ones (k6_ghosts)
  T* rhs_out;
  const int8_t* delays;  // [ntiles][6] for this step
  double* tot_part;
  uint32_t N, plane;
  uint32_t slab0, slab1, slab2, rdir1, rdir2, rslot;
  int nx, ny, nz, px, py, pz, ex, ey, ez;
  int bx, by;        // largest tile (columns in x and y)
  int tpx, tpy, tpz; // tiles of one PE along x and y, z chunks of one PE
  int zc;            // planes of a z chunk (the last of a PE may hold fewer)
  int gbx, gby;      // workgroups along x and y
  int R, step_mod_r, publish, store_dq, mode;
  T cs;              // c_s of this stage
  T cs3[3];          // k6_ghosts: c_s of each stage it forms
  int nst;
  T i60x, i60y, i60z, gas_r, inv_cv, cp_over_pr, mu_ref, inv_tref, mu_exp;
  T rk_a, rk_b, dt, c_prev;
  double vol;
};

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

template <typename T>
__device__ __forceinline__ T rcp6(T x) { return T(1) / x; }
template <>
__device__ __forceinline__ float rcp6<float>(float x) { return __builtin_amdgcn_rcpf(x); }

template <typename T>
__device__ __forceinline__ T visc6(const A6<T>& a, T t) { return a.mu_ref * pow(t * a.inv_tref, a.mu_exp); }
template <>
__device__ __forceinline__ float visc6<float>(const A6<float>& a, float t) {
  return a.mu_ref * __builtin_amdgcn_exp2f(a.mu_exp * __builtin_amdgcn_logf(t * a.inv_tref));
}

// u, v, w, T of conserved values q (rho, m, E).
template <typename T>
__device__ __forceinline__ void prims(const T q[5], T inv_cv, T& u, T& v, T& w, T& t) {
  const T ri = rcp6<T>(q[0]);
  u = q[1] * ri;
  v = q[2] * ri;
  w = q[3] * ri;
  t = (q[4] * ri - T(0.5) * (u * u + v * v + w * w)) * inv_cv;
}

// The (1,6) central numerator: -v(-3) + 9 v(-2) - 45 v(-1) + 45 v(+1) - 9 v(+2) + v(+3).
template <typename T>
__device__ __forceinline__ T c6(T m3, T m2, T m1, T p1, T p2, T p3) {
  return (T(9) * m2 - m3) + T(45) * (p1 - m1) + (p3 - T(9) * p2);
}

// Cubic extrapolation weights to kappa = k + c_s from levels n-k .. n-k-3.
template <typename T>
__device__ __forceinline__ void weights6(T kap, T w[4]) {
  w[0] = (kap + T(1)) * (kap + T(2)) * (kap + T(3)) * T(1.0 / 6.0);
  w[1] = -kap * (kap + T(2)) * (kap + T(3)) * T(0.5);
  w[2] = kap * (kap + T(1)) * (kap + T(3)) * T(0.5);
  w[3] = -kap * (kap + T(1)) * (kap + T(2)) * T(1.0 / 6.0);
}

// Ring element offset (slot 0, component 0) of direction d at global point (x, y, z) on one of the
// six published layers of its PE along d: layer jp = 6 t + (l < 3 ? l : l - e + 6).
template <typename T>
__device__ __forceinline__ uint32_t ring_off6(const A6<T>& a, int d, int x, int y, int z) {
  if (d == 0) {
    const int t = x / a.ex, l = x - t * a.ex;
    const int jp = 6 * t + (l < kM6 ? l : l - a.ex + 2 * kM6);
    return ((uint32_t)z * a.ny + y) * (uint32_t)(6 * a.px) + jp;
  }
  if (d == 1) {
    const int t = y / a.ey, l = y - t * a.ey;
    const int jp = 6 * t + (l < kM6 ? l : l - a.ey + 2 * kM6);
    return a.rdir1 + ((uint32_t)z * (6 * a.py) + jp) * (uint32_t)a.nx + x;
  }
  const int t = z / a.ez, l = z - t * a.ez;
  const int jp = 6 * t + (l < kM6 ? l : l - a.ez + 2 * kM6);
  return a.rdir2 + ((uint32_t)jp * a.ny + y) * (uint32_t)a.nx + x;
}

template <typename T>
__device__ __forceinline__ uint32_t slab6(const A6<T>& a, int d) {
  return d == 0 ? a.slab0 : (d == 1 ? a.slab1 : a.slab2);
}

// Extrapolated value of ring component `comp` (0..3 u, v, w, T; 4..8 face-normal flux) at ring
// offset `off` of direction d, as the PE reading it across its delayed face sees it at this stage
// (formed by k6_ghosts for that reader's delay).
template <typename T>
__device__ __forceinline__ T ghost6(const A6<T>& a, int d, int comp, uint32_t off) {
  return a.gv[off + (uint32_t)comp * slab6(a, d)];
}

// Extrapolated values behind the PE faces for the stages of one step (Sec. 2.1, Eq. at; Appendix
// B, (1,6) rows), one thread per element e of a ring slot.  Element e (direction d, component c,
// layer jp = 6 t + j of PE t along d) is read across a face by one PE only, its neighbour on the
// layer's side: PE t - 1 across its upper face for the lower layers (j < 3), PE t + 1 across its
// lower face for the upper ones.  With that reader's delay k >= 1, stage s gets the cubic
// extrapolation to kappa = k + c_s of levels n - k .. n - k - 3, written at e of its slot-sized
// buffer; elements whose reader is not delayed are left alone (no stage reads them).  The four
// levels are read once for all the stages, coalesced.
template <typename T>
__global__ __launch_bounds__(256) void k6_ghosts(A6<T> a) {
  const uint32_t e = blockIdx.x * 256u + threadIdx.x;
  if (e >= a.rslot) return;
  const int d = e < a.rdir1 ? 0 : (e < a.rdir2 ? 1 : 2);
  const uint32_t pos = (e - (d == 0 ? 0u : (d == 1 ? a.rdir1 : a.rdir2))) % slab6(a, d);
  int jp, tx, ty, tz;
  if (d == 0) {  // pos = (z ny + y) 6 px + jp
    const uint32_t w6 = 6u * (uint32_t)a.px, zy = pos / w6;
    jp = (int)(pos - zy * w6);
    ty = (int)(zy % (uint32_t)a.ny) / a.ey;
    tz = (int)(zy / (uint32_t)a.ny) / a.ez;
    tx = jp / 6;
  } else if (d == 1) {  // pos = (z 6 py + jp) nx + x
    const uint32_t r = pos / (uint32_t)a.nx, h6 = 6u * (uint32_t)a.py;
    tx = (int)(pos - r * (uint32_t)a.nx) / a.ex;
    jp = (int)(r % h6);
    tz = (int)(r / h6) / a.ez;
    ty = jp / 6;
  } else {  // pos = (jp ny + y) nx + x
    const uint32_t r = pos / (uint32_t)a.nx;
    tx = (int)(pos - r * (uint32_t)a.nx) / a.ex;
    ty = (int)(r % (uint32_t)a.ny) / a.ey;
    jp = (int)(r / (uint32_t)a.ny);
    tz = jp / 6;
  }
  const bool low = jp - 6 * (jp / 6) < kM6;
  const int np = d == 0 ? a.px : (d == 1 ? a.py : a.pz);
  int t = jp / 6;
  t = low ? (t == 0 ? np - 1 : t - 1) : (t == np - 1 ? 0 : t + 1);
  tx = d == 0 ? t : tx;
  ty = d == 1 ? t : ty;
  tz = d == 2 ? t : tz;
  const int k = a.delays[((tz * a.py + ty) * a.px + tx) * 6 + 2 * d + (low ? 1 : 0)];
  if (k <= 0) return;
  T lev[4];
  int s = a.step_mod_r - k;
  s += s < 0 ? a.R : 0;
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    lev[l] = a.ring[(uint32_t)s * a.rslot + e];
    s = s == 0 ? a.R - 1 : s - 1;
  }
  for (int st = 0; st < a.nst; ++st) {
    T w[4];
    weights6<T>(T(k) + a.cs3[st], w);
    T v = T(0);
#pragma unroll
    for (int l = 0; l < 4; ++l) v += w[l] * lev[l];
    __builtin_nontemporal_store(v, a.gv + (uint32_t)st * a.rslot + e);
  }
}

// Workgroups are dealt to the 8 XCDs in turn (dispatch index w to XCD w mod 8), each with its own
// L2.  Logical workgroup xcd_major(w, nb) gives each XCD a contiguous range of tiles, so the tiles
// whose 3-point halos overlap run on the same L2 (a bijection of [0, nb)).
constexpr uint32_t kNumXcd = 8;
__device__ __forceinline__ uint32_t xcd_major(uint32_t w, uint32_t nb) {
  const uint32_t c = w % kNumXcd, i = w / kNumXcd, q = nb / kNumXcd, r = nb % kNumXcd;
  return c * q + min(c, r) + i;
}

// A workgroup's box: its column tile [x0, x0 + w) x [y0, y0 + h), its planes [z0, z1), the PE it
// lies in (x, y, z ranges [pxl, pxh) etc.) and that PE's six face delays; L numbers the workgroups.
struct Box6 {
  int x0, y0, z0, z1, w, h;
  int pxl, pxh, pyl, pyh, pzl, pzh;
  int kf[6];
  uint32_t L;
};

template <typename T>
__device__ __forceinline__ Box6 box6(const A6<T>& a) {
  Box6 b;
  b.L = xcd_major(blockIdx.x, gridDim.x);
  const int L = (int)b.L, gxy = a.gbx * a.gby;
  const int bkz = L / gxy, r = L - bkz * gxy, bky = r / a.gbx, bkx = r - bky * a.gbx;
  const int tx = bkx / a.tpx, ty = bky / a.tpy, tz = bkz / a.tpz;
  b.pxl = tx * a.ex;
  b.pxh = b.pxl + a.ex;
  b.pyl = ty * a.ey;
  b.pyh = b.pyl + a.ey;
  b.pzl = tz * a.ez;
  b.pzh = b.pzl + a.ez;
  b.x0 = b.pxl + (bkx - tx * a.tpx) * a.bx;
  b.y0 = b.pyl + (bky - ty * a.tpy) * a.by;
  b.z0 = b.pzl + (bkz - tz * a.tpz) * a.zc;
  b.w = min(a.bx, b.pxh - b.x0);
  b.h = min(a.by, b.pyh - b.y0);
  b.z1 = min(b.z0 + a.zc, b.pzh);
  const int8_t* k = a.delays + ((tz * a.py + ty) * a.px + tx) * 6;
#pragma unroll
  for (int f = 0; f < 6; ++f) b.kf[f] = k[f];
  return b;
}

// One halo point of a thread, fixed for the whole march: component c of plane z is src[c cs + z zs],
// `li` its place in the LDS plane.  Across a delayed face of the box's PE (ghost) src is the
// extrapolated value, elsewhere the field (cs, zs accordingly).
template <typename T>
struct Halo6 {
  const T* src;
  uint32_t cs, zs;
  int li;
  bool on, ghost;
};

// Halo point at (hx, hy), dx (dy) layers outside the tile along d; field = the array of the values
// the PE has itself, comp0 the first ring component that stands for them behind a delayed face.
template <typename T>
__device__ __forceinline__ Halo6<T> halo6(const A6<T>& a, const Box6& b, int d, int hx, int hy, const T* field,
                                          int comp0) {
  Halo6<T> o;
  o.on = true;
  const int face = d == 0 ? (hx < b.pxl ? 0 : hx >= b.pxh ? 1 : -1) : (hy < b.pyl ? 2 : hy >= b.pyh ? 3 : -1);
  const int k = face < 0 ? 0 : face == 0 ? b.kf[0] : face == 1 ? b.kf[1] : face == 2 ? b.kf[2] : b.kf[3];
  hx = wrapi(hx, a.nx);
  hy = wrapi(hy, a.ny);
  o.ghost = k > 0;
  if (o.ghost) {
    o.cs = d == 0 ? a.slab0 : a.slab1;
    o.zs = d == 0 ? (uint32_t)a.ny * (uint32_t)(6 * a.px) : (uint32_t)(6 * a.py) * (uint32_t)a.nx;
    o.src = a.gv + ring_off6(a, d, hx, hy, 0) + (uint32_t)comp0 * o.cs;
  } else {
    o.cs = a.N;
    o.zs = a.plane;
    o.src = field + ((uint32_t)hy * (uint32_t)a.nx + hx);
  }
  return o;
}

// Gradients and fluxes.  HBM and issue bound (5 words read, 15 written per point, about 250 vector
// instructions): the halo points of a thread are located once (their integer divisions were a
// fifth of the instructions of a plane), the loads of the next plane are issued before the barrier
// of the current one, and two LDS planes leave one barrier per plane.  NH: halo points per thread.
template <typename T, int NH>
__global__ __launch_bounds__(256) void k6_gradflux(A6<T> a) {
  extern __shared__ unsigned char s_raw[];
  const int BX = a.bx, BY = a.by, LW = BX + 2 * kM6, NT = BX * BY;
  const int plane_lds = LW * (BY + 2 * kM6);
  T* s_p = reinterpret_cast<T*>(s_raw);  // [2][4][BY + 6][LW]
  const Box6 b = box6(a);
  const int tid = threadIdx.x, ly = tid / BX, lx = tid - ly * BX;
  const bool act = lx < b.w && ly < b.h;
  const int X = min(b.x0 + lx, b.pxh - 1), Y = min(b.y0 + ly, b.pyh - 1);
  const uint32_t col = (uint32_t)Y * (uint32_t)a.nx + X;
  const int own = (ly + kM6) * LW + lx + kM6;
  Halo6<T> hp[NH];
#pragma unroll
  for (int j = 0; j < NH; ++j) {
    const int i = tid + j * NT, nx6 = 2 * kM6 * b.h;
    hp[j].on = false;
    if (i < nx6) {  // x halo
      const int hr = i / (2 * kM6), c = i - hr * (2 * kM6);
      const int hx = c < kM6 ? b.x0 - kM6 + c : b.x0 + b.w + c - kM6, hy = b.y0 + hr;
      hp[j] = halo6<T>(a, b, 0, hx, hy, a.q, 0);
      hp[j].li = (hr + kM6) * LW + hx - b.x0 + kM6;
    } else if (i < nx6 + 2 * kM6 * b.w) {
      const int r = (i - nx6) / b.w, c = i - nx6 - r * b.w;
      const int hy = r < kM6 ? b.y0 - kM6 + r : b.y0 + b.h + r - kM6, hx = b.x0 + c;
      hp[j] = halo6<T>(a, b, 1, hx, hy, a.q, 0);
      hp[j].li = (hy - b.y0 + kM6) * LW + c + kM6;
    }
  }
  // the column's plane z: its conserved variables, or (across a delayed z face) u, v, w, T
  auto zghost = [&](int z) { return (z < b.pzl && b.kf[4] > 0) || (z >= b.pzh && b.kf[5] > 0); };
  auto fetch_col = [&](int z, T v[5]) {
    const int zw = wrapi(z, a.nz);
    if (zghost(z)) {
      const uint32_t o = ring_off6(a, 2, X, Y, zw);
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = ghost6(a, 2, c, o);
      v[4] = T(0);
    } else {
      const uint32_t o = (uint32_t)zw * a.plane + col;
#pragma unroll
      for (int c = 0; c < 5; ++c) v[c] = a.q[(uint32_t)c * a.N + o];
    }
  };
  auto finish = [&](bool ghost, const T v[5], T& u, T& vv, T& w, T& t) {
    if (ghost) {
      u = v[0];
      vv = v[1];
      w = v[2];
      t = v[3];
    } else {
      prims<T>(v, a.inv_cv, u, vv, w, t);
    }
  };
  // z window: u, v, w, T at planes zc-3 .. zc+3 (slot j = 0 .. 6)
  T win[4][7];
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    T v[5];
    fetch_col(b.z0 - kM6 + j, v);
    finish(zghost(b.z0 - kM6 + j), v, win[0][j], win[1][j], win[2][j], win[3][j]);
  }
  T nq[5], hq[NH][5], rho, E;
  auto fetch_plane = [&](int z) {
    fetch_col(z + kM6, nq);
#pragma unroll
    for (int j = 0; j < NH; ++j)
      if (hp[j].on) {
#pragma unroll
        for (int c = 0; c < 5; ++c) hq[j][c] = hp[j].src[(uint32_t)c * hp[j].cs + (uint32_t)z * hp[j].zs];
      }
    const uint32_t o = (uint32_t)z * a.plane + col;
    rho = a.q[o];
    E = a.q[4 * a.N + o];
  };
  fetch_plane(b.z0);
  T* rb = a.ring + (uint32_t)a.step_mod_r * a.rslot;
  for (int zc = b.z0; zc < b.z1; ++zc) {
    T* sp = s_p + ((zc - b.z0) & 1) * 4 * plane_lds;
    finish(zghost(zc + kM6), nq, win[0][6], win[1][6], win[2][6], win[3][6]);
    const T r0 = rho, E0 = E;
    if (act) {
#pragma unroll
      for (int c = 0; c < 4; ++c) sp[c * plane_lds + own] = win[c][3];
    }
#pragma unroll
    for (int j = 0; j < NH; ++j)
      if (hp[j].on) {
        T u, v, w, t;
        finish(hp[j].ghost, hq[j], u, v, w, t);
        sp[0 * plane_lds + hp[j].li] = u;
        sp[1 * plane_lds + hp[j].li] = v;
        sp[2 * plane_lds + hp[j].li] = w;
        sp[3 * plane_lds + hp[j].li] = t;
      }
    if (zc + 1 < b.z1) fetch_plane(zc + 1);
    __syncthreads();
    if (act) {
      const uint32_t i = (uint32_t)zc * a.plane + col;
      T G[kNGrad];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T* p = sp + c * plane_lds + own;
        const T gx = c6(p[-3], p[-2], p[-1], p[1], p[2], p[3]) * a.i60x;
        const T gy = c6(p[-3 * LW], p[-2 * LW], p[-LW], p[LW], p[2 * LW], p[3 * LW]) * a.i60y;
        const T gz = c6(win[c][0], win[c][1], win[c][2], win[c][4], win[c][5], win[c][6]) * a.i60z;
        const int base = c < 3 ? 3 * c : 9;
        G[base + 0] = gx;
        G[base + 1] = gy;
        G[base + 2] = gz;
      }
      const T u = win[0][3], v = win[1][3], w = win[2][3], t = win[3][3];
      const T mu = visc6<T>(a, t);
      const T kt = mu * a.cp_over_pr;
      const T th = G[0] + G[4] + G[8];
      const T s00 = mu * (G[0] + G[0]) - T(2.0 / 3.0) * mu * th;
      const T s11 = mu * (G[4] + G[4]) - T(2.0 / 3.0) * mu * th;
      const T s22 = mu * (G[8] + G[8]) - T(2.0 / 3.0) * mu * th;
      const T s01 = mu * (G[1] + G[3]);
      const T s02 = mu * (G[2] + G[6]);
      const T s12 = mu * (G[5] + G[7]);
      const T p = r0 * a.gas_r * t;
      const T mx = r0 * u, my = r0 * v, mz = r0 * w, Ep = E0 + p;
      T F[3][5];
      F[0][0] = mx;
      F[0][1] = mx * u + p - s00;
      F[0][2] = my * u - s01;
      F[0][3] = mz * u - s02;
      F[0][4] = Ep * u - (u * s00 + v * s01 + w * s02) - kt * G[9];
      F[1][0] = my;
      F[1][1] = mx * v - s01;
      F[1][2] = my * v + p - s11;
      F[1][3] = mz * v - s12;
      F[1][4] = Ep * v - (u * s01 + v * s11 + w * s12) - kt * G[10];
      F[2][0] = mz;
      F[2][1] = mx * w - s02;
      F[2][2] = my * w - s12;
      F[2][3] = mz * w + p - s22;
      F[2][4] = Ep * w - (u * s02 + v * s12 + w * s22) - kt * G[11];
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int c = 0; c < 5; ++c)  // streamed out: read by the next launch, far beyond the caches
          __builtin_nontemporal_store(F[d][c], a.flux + (uint32_t)(d * 5 + c) * a.N + i);
      if (a.publish) {
        const int lxe = X - b.pxl, lye = Y - b.pyl, lze = zc - b.pzl;
        const bool on[3] = {lxe < kM6 || lxe >= a.ex - kM6, lye < kM6 || lye >= a.ey - kM6,
                            lze < kM6 || lze >= a.ez - kM6};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          if (!on[d]) continue;
          const uint32_t o = ring_off6(a, d, X, Y, zc), sl = slab6(a, d);
          T* r = rb + o;
          r[0] = u;
          r[sl] = v;
          r[2 * sl] = w;
          r[3 * sl] = t;
#pragma unroll
          for (int c = 0; c < 5; ++c) r[(4 + c) * sl] = F[d][c];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 6; ++j) win[c][j] = win[c][j + 1];
  }
}

// Divergence and update.  HBM bound (15 flux words, the state and the register in, 10 words out).
// The F_x, F_y planes and their halos are fetched a plane ahead.  FP32 holds two LDS planes (one
// barrier per plane); FP64 one (two barriers), which leaves room for twice the workgroups.
template <typename T, int NH>
__global__ __launch_bounds__(256) void k6_divupdate(A6<T> a) {
  constexpr int NB = sizeof(T) == 4 ? 2 : 1;
  extern __shared__ unsigned char s_raw[];
  const int BX = a.bx, BY = a.by, LWX = BX + 2 * kM6, LHY = BY + 2 * kM6, NT = BX * BY;
  const int nel = 5 * BY * LWX + 5 * LHY * BX;
  T* s_f = reinterpret_cast<T*>(s_raw);  // [NB]: F_x [5][BY][LWX], then F_y [5][LHY][BX]
  double* s_red = reinterpret_cast<double*>(s_f + NB * (nel + (nel & 1)));
  const Box6 b = box6(a);
  const int tid = threadIdx.x, ly = tid / BX, lx = tid - ly * BX;
  const bool act = lx < b.w && ly < b.h;
  const int X = min(b.x0 + lx, b.pxh - 1), Y = min(b.y0 + ly, b.pyh - 1);
  const uint32_t col = (uint32_t)Y * (uint32_t)a.nx + X;
  const int sx = BY * LWX, sy = LHY * BX;  // LDS component strides
  const int ownx = ly * LWX + lx + kM6, owny = 5 * sx + (ly + kM6) * BX + lx;
  Halo6<T> hp[NH];
  int hst[NH];
#pragma unroll
  for (int j = 0; j < NH; ++j) {
    const int i = tid + j * NT, nx6 = 2 * kM6 * b.h;
    hp[j].on = false;
    hst[j] = 0;
    if (i < nx6) {  // F_x beyond the tile's x sides
      const int hr = i / (2 * kM6), c = i - hr * (2 * kM6);
      const int hx = c < kM6 ? b.x0 - kM6 + c : b.x0 + b.w + c - kM6, hy = b.y0 + hr;
      hp[j] = halo6<T>(a, b, 0, hx, hy, a.flux, 4);
      hp[j].li = hr * LWX + hx - b.x0 + kM6;
      hst[j] = sx;
    } else if (i < nx6 + 2 * kM6 * b.w) {  // F_y beyond its y sides
      const int r = (i - nx6) / b.w, c = i - nx6 - r * b.w;
      const int hy = r < kM6 ? b.y0 - kM6 + r : b.y0 + b.h + r - kM6, hx = b.x0 + c;
      hp[j] = halo6<T>(a, b, 1, hx, hy, a.flux + (size_t)5 * a.N, 4);
      hp[j].li = 5 * sx + (hy - b.y0 + kM6) * BX + c;
      hst[j] = sy;
    }
  }
  auto fetch_fz = [&](int z, T& f0, T& f1, T& f2, T& f3, T& f4) {
    const int zw = wrapi(z, a.nz);
    const bool ghost = (z < b.pzl && b.kf[4] > 0) || (z >= b.pzh && b.kf[5] > 0);  // uniform
    const T* p = ghost ? a.gv + ring_off6(a, 2, X, Y, zw) + 4 * a.slab2
                       : a.flux + (size_t)10 * a.N + ((uint32_t)zw * a.plane + col);
    const uint32_t cs = ghost ? a.slab2 : a.N;
    f0 = p[0];
    f1 = p[cs];
    f2 = p[2 * cs];
    f3 = p[3 * cs];
    f4 = p[4 * cs];
  };
  T fz[5][7];
#pragma unroll
  for (int j = 0; j < 6; ++j)
    fetch_fz(b.z0 - kM6 + j, fz[0][j], fz[1][j], fz[2][j], fz[3][j], fz[4][j]);
  T fxy[10], hq[NH][5];
  auto fetch_plane = [&](int z) {
    const uint32_t o = (uint32_t)z * a.plane + col;
#pragma unroll
    for (int c = 0; c < 10; ++c) fxy[c] = a.flux[(uint32_t)c * a.N + o];
#pragma unroll
    for (int j = 0; j < NH; ++j)
      if (hp[j].on) {
#pragma unroll
        for (int c = 0; c < 5; ++c) hq[j][c] = hp[j].src[(uint32_t)c * hp[j].cs + (uint32_t)z * hp[j].zs];
      }
  };
  fetch_plane(b.z0);
  double tsum[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const bool upd = a.mode != kModeRhsH, keep = a.rk_a != T(0) || a.c_prev != T(0);
  for (int zc = b.z0; zc < b.z1; ++zc) {
    const uint32_t i = (uint32_t)zc * a.plane + col;
    T* sf = s_f + (NB == 2 ? ((zc - b.z0) & 1) * (nel + (nel & 1)) : 0);
    if (act) {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        sf[c * sx + ownx] = fxy[c];
        sf[c * sy + owny] = fxy[5 + c];
      }
    }
#pragma unroll
    for (int j = 0; j < NH; ++j)
      if (hp[j].on) {
#pragma unroll
        for (int c = 0; c < 5; ++c) sf[hp[j].li + c * hst[j]] = hq[j][c];
      }
    // this plane's state and RK register and the newest plane of the z window, then the next
    // plane's x / y fluxes (a wave's loads complete in order, so these stay in flight longest)
    T qv[5], prev[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      qv[c] = upd ? a.q[(uint32_t)c * a.N + i] : T(0);
      prev[c] = upd && keep ? __builtin_nontemporal_load(a.dq + (uint32_t)c * a.N + i) : T(0);
    }
    fetch_fz(zc + kM6, fz[0][6], fz[1][6], fz[2][6], fz[3][6], fz[4][6]);
    if (zc + 1 < b.z1) fetch_plane(zc + 1);
    __syncthreads();
    if (act) {
      T rhs[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        const T* px_ = sf + c * sx + ownx;
        const T* py_ = sf + c * sy + owny;
        const T dfx = c6(px_[-3], px_[-2], px_[-1], px_[1], px_[2], px_[3]) * a.i60x;
        const T dfy = c6(py_[-3 * BX], py_[-2 * BX], py_[-BX], py_[BX], py_[2 * BX], py_[3 * BX]) * a.i60y;
        const T dfz = c6(fz[c][0], fz[c][1], fz[c][2], fz[c][4], fz[c][5], fz[c][6]) * a.i60z;
        rhs[c] = -((dfx + dfy) + dfz);
      }
      if (a.mode == kModeRhsH) {
#pragma unroll
        for (int c = 0; c < 5; ++c) __builtin_nontemporal_store(rhs[c], a.rhs_out + (uint32_t)c * a.N + i);
      } else {
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const T d = a.rk_a * prev[c] + a.dt * rhs[c];
          const T inc = a.rk_b * d + a.c_prev * prev[c];
          if (a.store_dq) __builtin_nontemporal_store(d, a.dq + (uint32_t)c * a.N + i);
          __builtin_nontemporal_store(qv[c] + inc, a.q_out + (uint32_t)c * a.N + i);
          tsum[c] += a.c_prev != T(0) ? (double)inc : (double)d;
        }
      }
    }
    if (NB == 1) __syncthreads();
#pragma unroll
    for (int c = 0; c < 5; ++c)
#pragma unroll
      for (int j = 0; j < 6; ++j) fz[c][j] = fz[c][j + 1];
  }
  if (a.mode != kModeStepH) return;  // uniform across the grid
  // FP64 block sums in a fixed order: B_s * sum(dQ) * h^3 (or the Adams-Bashforth increment)
  for (int c = 0; c < 5; ++c) {
    s_red[tid] = tsum[c];
    __syncthreads();
    for (int len = 128; len > 0; len >>= 1) {
      if (tid < len && tid + len < NT) s_red[tid] += s_red[tid + len];
      __syncthreads();
    }
    if (tid == 0) {
      const double scale = a.c_prev != T(0) ? 1.0 : (double)a.rk_b;
      a.tot_part[b.L * kNQ + c] += scale * s_red[0] * a.vol;
    }
    __syncthreads();
  }
}

template <typename T>
A6<T> pack6(const Stage6Args<T>& s) {
  A6<T> a{};
  const Geom& g = s.g;
  a.q = s.q;
  a.q_out = s.q_out;
  a.dq = s.dq;
  a.flux = s.flux;
  a.ring = s.ring;
  a.gv = s.gv;
  a.rhs_out = s.rhs_out;
  a.delays = s.delays;
  a.tot_part = s.tot_part;
  a.N = (uint32_t)g.npts;
  a.plane = (uint32_t)g.n[0] * (uint32_t)g.n[1];
  a.slab0 = (uint32_t)g.slab[0];
  a.slab1 = (uint32_t)g.slab[1];
  a.slab2 = (uint32_t)g.slab[2];
  a.rdir1 = (uint32_t)g.ring_dir_off[1];
  a.rdir2 = (uint32_t)g.ring_dir_off[2];
  a.rslot = (uint32_t)g.ring_slot;
  a.nx = g.n[0];
  a.ny = g.n[1];
  a.nz = g.n[2];
  a.px = g.p[0];
  a.py = g.p[1];
  a.pz = g.p[2];
  a.ex = g.e[0];
  a.ey = g.e[1];
  a.ez = g.e[2];
  const Tile6& t = s.tile;
  a.bx = t.bx;
  a.by = t.by;
  a.zc = t.zc;
  a.tpx = (g.e[0] + t.bx - 1) / t.bx;
  a.tpy = (g.e[1] + t.by - 1) / t.by;
  a.tpz = (g.e[2] + t.zc - 1) / t.zc;
  a.gbx = g.p[0] * a.tpx;
  a.gby = g.p[1] * a.tpy;
  a.R = g.R;
  a.step_mod_r = s.step_mod_r;
  a.publish = s.publish;
  a.store_dq = s.store_dq;
  a.mode = s.mode;
  a.cs = s.cs;
  for (int st = 0; st < 3; ++st) a.cs3[st] = s.cs3[st];
  a.nst = s.nst;
  for (int d = 0; d < 3; ++d) (d == 0 ? a.i60x : d == 1 ? a.i60y : a.i60z) = s.i60h[d];
  a.gas_r = s.cf.gas_r;
  a.inv_cv = s.cf.inv_cv;
  a.cp_over_pr = s.cf.cp_over_pr;
  a.mu_ref = s.cf.mu_ref;
  a.inv_tref = s.cf.inv_tref;
  a.mu_exp = s.cf.mu_exp;
  a.rk_a = s.rk_a;
  a.rk_b = s.rk_b;
  a.dt = s.dt;
  a.c_prev = s.c_prev;
  a.vol = s.vol;
  return a;
}

}  // namespace

namespace {
int cdiv(int a, int b) { return (a + b - 1) / b; }
int halos6(int bx, int by) { return 2 * kM6 * (bx + by); }
}  // namespace

// Tile of a PE: its x-y face is cut into equal tiles of at most 256 points.  Of a few widths the one
// of least cost per PE is taken, the cost of a tile being its waves, half a point for each of its
// halo points and a few for each row (a row of a tile is a run of memory of its own).  Tiles of
// powers of two that divide the edges, the first rule here, were 4 x 1 on edges of 44 x 25: of 140 grids
// timed, of 2,000 to 17 million points, none is slower than with them.
// The two weights are rough.  Without the row term 256^3 FP32 on PEs of 64^3 takes 4.21 ms a step instead
// of 3.06, and 130 x 90 x 60 on 2 x 2 x 2 PEs 386 us instead of 256.  Without the halo term most grids keep
// their tiles; 200^3 on PEs of 50^3 takes 2.16 ms instead of 2.87 and 225 x 56 x 183 FP64 on 5 x 4 x 3 PEs
// 1.19 instead of 1.65, but 288 x 148 x 204 FP64 on 4 x 4 x 6 PEs 3.80 instead of 3.32.
// z chunks: PEs with fewer than 1024 tiles in all (4 workgroups per CU) are cut along z, into chunks
// of at least 8 planes (a chunk reads 6 planes more than it owns).
Tile6 tile6_of(const Geom& g) {
  Tile6 best{};
  double least = 1e300;
  for (int want : {64, 48, 32, 24, 16, 12, 8}) {
    const int bx = cdiv(g.e[0], cdiv(g.e[0], want));
    const int by = cdiv(g.e[1], cdiv(g.e[1], 256 / bx));
    if (halos6(bx, by) > 2 * bx * by) continue;  // a thread holds at most two halo points
    const double cost = (double)cdiv(g.e[0], bx) * cdiv(g.e[1], by) *
                        (64.0 * cdiv(bx * by, 64) + 0.5 * halos6(bx, by) + 6.0 * by);
    if (cost < least) {
      least = cost;
      best.bx = bx;
      best.by = by;
    }
  }
  const int64_t nt = (int64_t)g.p[0] * cdiv(g.e[0], best.bx) * g.p[1] * cdiv(g.e[1], best.by) * g.p[2];
  const int64_t want = (1024 + nt - 1) / nt;
  const int nc = (int)std::max<int64_t>(1, std::min<int64_t>(want, g.e[2] / 8));
  best.zc = cdiv(g.e[2], nc);
  return best;
}

int64_t blocks6(const Geom& g) {
  const Tile6 t = tile6_of(g);
  return (int64_t)g.p[0] * cdiv(g.e[0], t.bx) * g.p[1] * cdiv(g.e[1], t.by) * g.p[2] * cdiv(g.e[2], t.zc);
}

namespace {
template <typename T, int NH>
void launch6(const A6<T>& a, bool gradflux, hipStream_t stream) {
  const dim3 grid((unsigned)(a.gbx * a.gby) * (unsigned)(a.pz * a.tpz)), block((unsigned)(a.bx * a.by));
  if (gradflux) {
    const size_t lds = sizeof(T) * 2 * 4 * (a.bx + 2 * kM6) * (a.by + 2 * kM6);
    hipLaunchKernelGGL((k6_gradflux<T, NH>), grid, block, lds, stream, a);
  } else {
    const size_t nel = (size_t)5 * a.by * (a.bx + 2 * kM6) + (size_t)5 * (a.by + 2 * kM6) * a.bx;
    const size_t lds = sizeof(T) * (sizeof(T) == 4 ? 2 : 1) * (nel + (nel & 1)) + sizeof(double) * 256;
    hipLaunchKernelGGL((k6_divupdate<T, NH>), grid, block, lds, stream, a);
  }
}
}  // namespace

template <typename T>
hipError_t launch_stage6(const Stage6Args<T>& s, bool gradflux, hipStream_t stream) {
  const A6<T> a = pack6<T>(s);
  const int nt = a.bx * a.by, nh = halos6(a.bx, a.by);
  if (nt < 1 || nt > 256 || nh > 2 * nt || a.zc < 1) return hipErrorInvalidConfiguration;
  if (nh <= nt) launch6<T, 1>(a, gradflux, stream);
  else launch6<T, 2>(a, gradflux, stream);
  return hipGetLastError();
}

template hipError_t launch_stage6<float>(const Stage6Args<float>&, bool, hipStream_t);
template hipError_t launch_stage6<double>(const Stage6Args<double>&, bool, hipStream_t);

template <typename T>
hipError_t launch_ghosts6(const Stage6Args<T>& s, hipStream_t stream) {
  if (s.nst < 1 || s.nst > 3 || !s.gv) return hipErrorInvalidValue;
  const A6<T> a = pack6<T>(s);
  const dim3 grid((unsigned)((a.rslot + 255u) / 256u)), block(256);
  hipLaunchKernelGGL(k6_ghosts<T>, grid, block, 0, stream, a);
  return hipGetLastError();
}

template hipError_t launch_ghosts6<float>(const Stage6Args<float>&, hipStream_t);
template hipError_t launch_ghosts6<double>(const Stage6Args<double>&, hipStream_t);

}  // namespace atns
