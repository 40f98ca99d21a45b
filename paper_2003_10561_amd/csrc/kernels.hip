// gfx950 support kernels of the AT compressible Navier-Stokes library: FP64 statistics with
// synchronous 4th-order central derivatives (the k = 0 rows of the (1,4) schemes, Appendix B) and
// fixed-order reductions, precision conversion, and the separable forcing table.
#include <algorithm>

#include "atns_internal.h"

namespace atns {
namespace {

constexpr int kBX = 64;  // one wavefront along x
constexpr int kBY = 4;

__device__ __forceinline__ int wrap1(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// rho, u, v, w, T from the fifth variable E (form 0) or rho e (form 1, the paper's own form).
template <typename T>
__device__ __forceinline__ void primitives(const T* q, int64_t N, int64_t i, T inv_cv, int form, T pr[5]) {
  const T rho = q[i];
  const T rinv = T(1) / rho;
  const T u = q[N + i] * rinv, v = q[2 * N + i] * rinv, w = q[3 * N + i] * rinv;
  pr[0] = rho;
  pr[1] = u;
  pr[2] = v;
  pr[3] = w;
  pr[4] = form == 1 ? q[4 * N + i] * rinv * inv_cv : (q[4 * N + i] * rinv - T(0.5) * (u * u + v * v + w * w)) * inv_cv;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Statistics partials per block with synchronous periodic derivatives (no PE faces) of the run's
// order: the (1,4) central stencil (M = 2) or the (1,6) one (M = 3).  A workgroup marches a 64 x 8
// column tile through zc planes: each point's primitives are formed once (1.6 times with the halo; 13
// times, a division each, when every point formed its neighbours' own), x and y neighbours come from
// an LDS plane (two of them, one barrier a plane), z neighbours from a register window, and the loads
// of the next plane are issued before the barrier.  Bound by FP64 arithmetic (a division and a power
// per point).  256^3 FP64: 0.67 ms with a point per thread, 0.33 now; 32^3: 11 us and 17, but the
// reductions' lane exchanges take the call from 69 to 47 us.
constexpr int kSX = 64, kSY = 8;
template <typename T, int M>
__global__ __launch_bounds__(kSX* kSY) void k_stats(Geom g, Coef<T> cf, const T* __restrict__ q,
                                                    double* __restrict__ part, int zc) {
  constexpr int LW = kSX + 2 * M, LH = kSY + 2 * M;
  __shared__ T s_u[2][3][LH][LW];
  __shared__ double red[kSY][kNStat];
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int gx = (nx + kSX - 1) / kSX, gy = (ny + kSY - 1) / kSY;
  const int blk = (int)blockIdx.x, bz = blk / (gx * gy), br = blk - bz * gx * gy, by = br / gx, bx = br - by * gx;
  const int x0 = bx * kSX, y0 = by * kSY, z0 = bz * zc, z1 = min(z0 + zc, nz);
  const int w = min(kSX, nx - x0), h = min(kSY, ny - y0);
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * kSX + tx;
  const bool act = tx < w && ty < h;
  const int64_t N = g.npts, plane = (int64_t)nx * ny;
  const int64_t col = (int64_t)(y0 + min(ty, h - 1)) * nx + x0 + min(tx, w - 1);
  // this thread's halo point of every plane
  int hl = -1;  // its place in the LDS plane
  int64_t hcol = col;
  {
    int hx = 0, hy = 0;
    if (tid < 2 * M * h) {
      const int r = tid / (2 * M), c = tid - r * (2 * M);
      hx = c < M ? c - M : w + c - M;
      hy = r;
    } else if (tid < 2 * M * (h + w)) {
      const int i = tid - 2 * M * h, r = i / w;
      hx = i - r * w;
      hy = r < M ? r - M : h + r - M;
    }
    if (tid < 2 * M * (h + w)) {
      hl = (hy + M) * LW + hx + M;
      hcol = (int64_t)wrap1(y0 + hy, ny) * nx + wrap1(x0 + hx, nx);
    }
  }
  double s[kNStat];
#pragma unroll
  for (int c = 0; c < kNStat; ++c) s[c] = 0.0;
  T win[3][2 * M + 1], tw[M + 1];  // u, v, w of planes z - M .. z + M; T of planes z .. z + M
  auto fetch = [&](int64_t c0, int z, T v[5]) {
    const int64_t i = (int64_t)wrap1(z, nz) * plane + c0;
#pragma unroll
    for (int c = 0; c < kNQ; ++c) v[c] = q[c * N + i];
  };
  // u, v, w, T of a column's plane; own planes of the chunk add their pointwise sums here
  auto absorb = [&](const T v[5], bool mine, T pr[5]) {
    primitives<T>(v, 1, 0, cf.inv_cv, cf.form, pr);
    if (mine) {
      const double u = pr[1], vv = pr[2], ww = pr[3];
      const double uu = u * u + vv * vv + ww * ww;
      int nonfin = 0;
#pragma unroll
      for (int c = 0; c < kNQ; ++c) {
        const double qv = (double)v[c];
        s[c] += qv;
        if (!isfinite(qv)) nonfin = 1;
      }
      s[5] += 0.5 * (double)pr[0] * uu;
      s[8] += uu;
      s[9] += (double)pr[4];
      s[10] = fmax(s[10], uu);
      if (nonfin) s[11] = 1.0;
    }
  };
#pragma unroll
  for (int j = 0; j < 2 * M; ++j) {
    const int z = z0 - M + j;
    T v[5], pr[5];
    fetch(col, z, v);
    absorb(v, act && j >= M && z < z1, pr);
#pragma unroll
    for (int c = 0; c < 3; ++c) win[c][j] = pr[1 + c];
    if (j >= M) tw[j - M] = pr[4];
  }
  T nq[5], hq[5];
  fetch(col, z0 + M, nq);
  fetch(hcol, z0, hq);
  for (int z = z0; z < z1; ++z) {
    T* sp = &s_u[(z - z0) & 1][0][0][0];
    {
      T pr[5];
      absorb(nq, act && z + M < z1, pr);
#pragma unroll
      for (int c = 0; c < 3; ++c) win[c][2 * M] = pr[1 + c];
      tw[M] = pr[4];
    }
    if (act) {
#pragma unroll
      for (int c = 0; c < 3; ++c) sp[(c * LH + ty + M) * LW + tx + M] = win[c][M];
    }
    if (hl >= 0) {
      T pr[5];
      absorb(hq, false, pr);
#pragma unroll
      for (int c = 0; c < 3; ++c) sp[c * LH * LW + hl] = pr[1 + c];
    }
    if (z + 1 < z1) {
      fetch(col, z + 1 + M, nq);
      fetch(hcol, z + 1, hq);
    }
    __syncthreads();
    if (act) {
      T G[9];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const T* p = sp + (c * LH + ty + M) * LW + tx + M;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          T v[2 * M];
#pragma unroll
          for (int mi = 0; mi < 2 * M; ++mi) {
            const int m = mi < M ? mi - M : mi - M + 1;
            v[mi] = d == 0 ? p[m] : (d == 1 ? p[m * LW] : win[c][M + m]);
          }
          const T num = M == 2 ? (v[0] - T(8) * v[1] + T(8) * v[2] - v[3])
                               : (T(9) * v[1] - v[0]) + T(45) * (v[3] - v[2]) + (v[5] - T(9) * v[4]);
          G[3 * c + d] = num * (M == 2 ? cf.inv12h[d] : cf.inv60h[d]);
        }
      }
      const double temp = (double)tw[0], tt = temp * (double)cf.inv_tref;
      const double mu = cf.visc == 1 ? (double)cf.mu_ref * tt * sqrt(tt) * (1.0 / (double)cf.inv_tref + (double)cf.suth_s) /
                                           (temp + (double)cf.suth_s)
                                     : (double)cf.mu_ref * pow(tt, (double)cf.mu_exp);
      const double th = (double)G[0] + (double)G[4] + (double)G[8];
      double eps = 0.0;
#pragma unroll
      for (int ii = 0; ii < 3; ++ii)
#pragma unroll
        for (int jj = 0; jj < 3; ++jj) {
          double sg = mu * ((double)G[3 * ii + jj] + (double)G[3 * jj + ii]);
          if (ii == jj) sg -= (2.0 / 3.0) * mu * th;
          eps += sg * (double)G[3 * ii + jj];
        }
      const double ox = (double)G[7] - (double)G[5];
      const double oy = (double)G[2] - (double)G[6];
      const double oz = (double)G[3] - (double)G[1];
      s[6] += eps;
      s[7] += ox * ox + oy * oy + oz * oz;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int j = 0; j < 2 * M; ++j) win[c][j] = win[c][j + 1];
#pragma unroll
    for (int j = 0; j < M; ++j) tw[j] = tw[j + 1];
  }
  s[10] = sqrt(s[10]);
#pragma unroll
  for (int c = 0; c < kNStat; ++c) {
    double v = s[c];
    if (c == 10 || c == 11) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    } else {
      v = wave_sum(v);
    }
    if (tx == 0) red[ty][c] = v;
  }
  __syncthreads();
  if (tid < kNStat) {
    double v = red[0][tid];
    for (int r = 1; r < kSY; ++r) v = tid == 10 || tid == 11 ? fmax(v, red[r][tid]) : v + red[r][tid];
    part[(int64_t)blk * kNStat + tid] = v;
  }
}

// Planes of a workgroup of k_stats, and its workgroups: 64 planes, or as many fewer as leave 1024
// workgroups (a march reads 2 M planes more than it owns).
int stats_zc(const Geom& g) {
  const int64_t tiles = (int64_t)((g.n[0] + kSX - 1) / kSX) * ((g.n[1] + kSY - 1) / kSY);
  return (int)std::max<int64_t>(4, std::min<int64_t>(64, tiles * g.n[2] / 1024));
}
int64_t stats_workgroups(const Geom& g) {
  const int zc = stats_zc(g);
  return (int64_t)((g.n[0] + kSX - 1) / kSX) * ((g.n[1] + kSY - 1) / kSY) * ((g.n[2] + zc - 1) / zc);
}

// Fixed-order two-level reduction of the per-block partials (deterministic: the order depends only
// on the partial counts).  Level 1: workgroup j reduces its contiguous share of the statistic
// partials [nblk][13] and of the FP64 RK-total slots [ntot][5] into mid[j][18]; level 2 reduces
// the kStatRed rows of mid into out[18].  Components 10 (max |u|) and 11 (non-finite flag) take
// the maximum, the others the sum.  A wave takes a component: its lanes stride over the entries and
// are added by lane exchanges (a tree of 8 barriers for each of the 18 components took 17 us a level).
constexpr int kStatOut = kNStat + kNQ;
static_assert(kStatRed == 256, "level 2 gives four level-1 rows to a lane");

__device__ __forceinline__ double wave_reduce(double v, bool is_max) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(v, off, 64);
    v = is_max ? fmax(v, o) : v + o;
  }
  return v;
}

__global__ __launch_bounds__(256) void k_stats_reduce(const double* __restrict__ part, int64_t nblk,
                                                      const double* __restrict__ tot_part, int64_t ntot,
                                                      double* __restrict__ mid) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j = blockIdx.x;
  const int64_t lp = (nblk + kStatRed - 1) / kStatRed, lt = (ntot + kStatRed - 1) / kStatRed;
  const int64_t p0 = j * lp, p1 = min(p0 + lp, nblk), t0 = j * lt, t1 = min(t0 + lt, ntot);
  for (int c = wave; c < kStatOut; c += 4) {
    const bool is_max = (c == 10 || c == 11);
    double v = 0.0;
    if (c < kNStat) {
      for (int64_t b = p0 + lane; b < p1; b += 64) {
        const double pv = part[b * kNStat + c];
        v = is_max ? fmax(v, pv) : v + pv;
      }
    } else if (tot_part) {
      for (int64_t b = t0 + lane; b < t1; b += 64) v += tot_part[b * kNQ + (c - kNStat)];
    }
    v = wave_reduce(v, is_max);
    if (lane == 0) mid[j * kStatOut + c] = v;
  }
}

__global__ __launch_bounds__(1024) void k_stats_final(const double* __restrict__ mid, double* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c = wave; c < kStatOut; c += 16) {
    const bool is_max = (c == 10 || c == 11);
    double v = mid[lane * kStatOut + c];
#pragma unroll
    for (int r = 1; r < kStatRed / 64; ++r) {
      const double o = mid[(r * 64 + lane) * kStatOut + c];
      v = is_max ? fmax(v, o) : v + o;
    }
    v = wave_reduce(v, is_max);
    if (lane == 0) out[c] = v;
  }
}

// The statistics record of a field from the reduced sums (the conversions at_stats makes on the
// host), for a caller without a handle: no step count and no RK history, so step and time are 0
// and the RK-accumulated totals repeat the direct sums.
__global__ void k_stats_record(const double* __restrict__ st, at_stats_t* __restrict__ o, double npts, double vol,
                               double gamma, double gas_r) {
  if (threadIdx.x != 0) return;
  o->step = 0;
  o->time = 0.0;
  o->mass = st[0] * vol;
  for (int a = 0; a < 3; ++a) o->mom[a] = st[1 + a] * vol;
  o->energy = st[4] * vol;
  o->mass_rk = o->mass;
  for (int a = 0; a < 3; ++a) o->mom_rk[a] = o->mom[a];
  o->energy_rk = o->energy;
  o->K = st[5] / npts;
  o->eps = st[6] / npts;
  o->enstrophy = st[7] / npts;
  o->Mt = sqrt(st[8] / npts) / sqrt(gamma * gas_r * (st[9] / npts));
  o->umax = st[10];
  o->nonfinite = st[11] != 0.0 ? 1 : 0;
  o->reserved = 0;
}

template <typename T>
__global__ void k_convert(const double* __restrict__ src, T* __restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (T)src[i];
}

template <typename T>
__global__ void k_to_double(const T* __restrict__ src, double* __restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (double)src[i];
}

// A[pair][x][c] = sum over wavevectors of that (ky, kz) pair of fhat(c) e^{i kx x}.
template <typename T>
__global__ void k_force_table(int nx, const double* __restrict__ fhat, const int* __restrict__ wv_kx,
                              const int* __restrict__ wv_pair, int npair, T* __restrict__ table,
                              const T* __restrict__ phase_x) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= npair * nx) return;
  const int pidx = tid / nx, x = tid - pidx * nx;
  double acc[3][2] = {{0, 0}, {0, 0}, {0, 0}};
  for (int w = 0; w < kNForce; ++w) {
    if (wv_pair[w] != pidx) continue;
    const T* ph = phase_x + ((int64_t)(wv_kx[w] + 2) * nx + x) * 2;
    const double ec = (double)ph[0], es = (double)ph[1];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double fr = fhat[(w * 3 + c) * 2], fi = fhat[(w * 3 + c) * 2 + 1];
      acc[c][0] += fr * ec - fi * es;
      acc[c][1] += fr * es + fi * ec;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    table[(int64_t)tid * 6 + 2 * c] = (T)acc[c][0];
    table[(int64_t)tid * 6 + 2 * c + 1] = (T)acc[c][1];
  }
}

dim3 grid_of(const Geom& g) {
  return dim3((g.n[0] + kBX - 1) / kBX, (g.n[1] + kBY - 1) / kBY, g.n[2]);
}

}  // namespace

int64_t update_blocks(const Geom& g) {
  const dim3 gr = grid_of(g);
  return (int64_t)gr.x * gr.y * gr.z;
}
// Room for the statistics partials, counted in blocks of 64 x 4 points of one plane: a measure of the grid
// that stays when the march is cut otherwise (k_stats leaves fewer partials, one per stats_workgroups).
int64_t stats_blocks(const Geom& g) { return update_blocks(g); }

const char* kernel_name(int id) {
  static const char* names[kKCount] = {"k_stage", "k_stage(rhs)", "k_stage(publish)", "k_force_table",
                                       "k_stats", "k_at_sums", "k6_gradflux", "k6_divupdate",
                                       "kp_publish", "kp_grad", "kp_rhs", "k6_ghosts"};
  return (id >= 0 && id < kKCount) ? names[id] : "";
}

#define HOOKED(id, launch)              \
  do {                                  \
    if (hook) hook->before(id, stream); \
    launch;                             \
    if (hook) hook->after(id, stream);  \
  } while (0)

template <typename T>
hipError_t launch_convert(const double* src, T* dst, int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(k_convert<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, src, dst, n);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_to_double(const T* src, double* dst, int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(k_to_double<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, src, dst, n);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_stats(const Geom& g, const Coef<T>& cf, const T* q, double* part, double* out,
                        const double* tot_part, int64_t ntot_blocks, double gamma, hipStream_t stream,
                        LaunchHook* hook) {
  (void)gamma;
  const dim3 blk(kSX, kSY, 1);
  const int64_t nblk = stats_workgroups(g);  // at most stats_blocks(g), the partials there is room for
  const int zc = stats_zc(g);
  if (g.order == 6)
    HOOKED(kKStats, hipLaunchKernelGGL((k_stats<T, 3>), dim3((unsigned)nblk), blk, 0, stream, g, cf, q, part, zc));
  else
    HOOKED(kKStats, hipLaunchKernelGGL((k_stats<T, 2>), dim3((unsigned)nblk), blk, 0, stream, g, cf, q, part, zc));
  double* mid = out + kStatOutSlots;
  hipLaunchKernelGGL(k_stats_reduce, dim3(kStatRed), dim3(256), 0, stream, part, nblk, tot_part,
                     ntot_blocks, mid);
  hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(1024), 0, stream, (const double*)mid, out);
  return hipGetLastError();
}

hipError_t launch_stats_record(const double* raw, at_stats_t* dst, double npts, double vol, double gamma,
                               double gas_r, hipStream_t stream) {
  hipLaunchKernelGGL(k_stats_record, dim3(1), dim3(64), 0, stream, raw, dst, npts, vol, gamma, gas_r);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_force_table(const Geom& g, const double* fhat_step, const int* wv_kx,
                              const int* wv_pair, int npair, T* table, const T* phase_x,
                              hipStream_t stream, LaunchHook* hook) {
  const int n = npair * g.n[0];
  HOOKED(kKForce, hipLaunchKernelGGL(k_force_table<T>, dim3((n + 255) / 256), dim3(256), 0, stream,
                                     g.n[0], fhat_step, wv_kx, wv_pair, npair, table, phase_x));
  return hipGetLastError();
}

#define ATNS_INSTANTIATE(T)                                                                          \
  template hipError_t launch_convert<T>(const double*, T*, int64_t, hipStream_t);                    \
  template hipError_t launch_to_double<T>(const T*, double*, int64_t, hipStream_t);                  \
  template hipError_t launch_stats<T>(const Geom&, const Coef<T>&, const T*, double*, double*,       \
                                      const double*, int64_t, double, hipStream_t, LaunchHook*);     \
  template hipError_t launch_force_table<T>(const Geom&, const double*, const int*, const int*, int, \
                                            T*, const T*, hipStream_t, LaunchHook*);
ATNS_INSTANTIATE(double)
ATNS_INSTANTIATE(float)

}  // namespace atns
