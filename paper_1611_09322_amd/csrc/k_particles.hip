// Particle-side kernels: wrapping and linked-cell binning, the sorted order,
// the near-field neighbour list, the real-space product w = M_r v
// (eq. Mreal, Appendix A) and the Lanczos square-root iteration (Sec. II B.1).
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <unordered_set>

#include "launch.hpp"
#include "philox.hpp"

namespace pse {

template <typename T> __device__ __forceinline__ T wrap_coord(T x, T L, T invL) {
  x = x - L * floor(x * invL);
  if (x >= L || x < T(0)) x = T(0);  // x == L (or rounding just past it) maps to 0
  return x;
}

template <typename T> __device__ __forceinline__ T min_image(T d, T L, T invL) { return d - L * rint(d * invL); }

// --------------------------------------------------------------- binning
template <typename T>
__device__ __forceinline__ void wrap_bin_at(const T *__restrict__ pos, int n, T L, T invL, T inv_cs, int nc,
                                            typename vec4<T>::type *__restrict__ pos_w, int *__restrict__ cell_of,
                                            int *__restrict__ slot, int *__restrict__ cell_count,
                                            int *__restrict__ flags, int i) {
  if (i >= n) return;
  T x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
  if (!isfinite(x) || !isfinite(y) || !isfinite(z)) {
    atomicOr(&flags[0], 1);
    x = y = z = T(0);
  }
  x = wrap_coord(x, L, invL);
  y = wrap_coord(y, L, invL);
  z = wrap_coord(z, L, invL);
  const int cx = min((int)(x * inv_cs), nc - 1);
  const int cy = min((int)(y * inv_cs), nc - 1);
  const int cz = min((int)(z * inv_cs), nc - 1);
  const int c = (cx * nc + cy) * nc + cz;
  cell_of[i] = c;
  // The particle's slot in its cell (arrival order; k_cell_sort fixes the
  // final order).  Lanes holding the same cell as the lane before them join
  // its run, and the first lane of each run reserves the run's slots with
  // one atomic: all runs of the wavefront in a single instruction, one per
  // particle for shuffled callers, a few for spatially ordered ones.  The
  // active lanes are 0 .. k-1 (only the last wavefront is partial).
  const int lane = threadIdx.x & 63;
  const unsigned long long act = __ballot(1);
  const int prev = __shfl_up(c, 1, 64);
  const bool head = lane == 0 || prev != c;
  const unsigned long long H = __ballot(head);
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);  // lanes 0 .. lane
  const int hl = 63 - __clzll((long long)(H & upto));                             // first lane of my run
  const unsigned long long later = H & ~upto;
  const int next = later ? __ffsll((long long)later) - 1 : 64 - __clzll((long long)act);
  int b = 0;
  if (head) b = atomicAdd(&cell_count[c], next - lane);
  slot[i] = __shfl(b, hl, 64) + (lane - hl);
  typename vec4<T>::type q;
  q.x = x; q.y = y; q.z = z; q.w = T(0);
  pos_w[i] = q;
}

template <typename T>
__global__ void k_wrap_bin(const T *__restrict__ pos, int n, T L, T invL, T inv_cs, int nc,
                           typename vec4<T>::type *__restrict__ pos_w, int *__restrict__ cell_of,
                           int *__restrict__ slot, int *__restrict__ cell_count, int *__restrict__ flags) {
  wrap_bin_at<T>(pos, n, L, invL, inv_cs, nc, pos_w, cell_of, slot, cell_count, flags,
                 blockIdx.x * blockDim.x + threadIdx.x);
}

// Exclusive scan of the cell counts in tiles of 4096 cells: k_scan_tiles
// sums each tile, k_scan_apply adds the sums of the tiles before its own
// (a few thousand at most) and scans its tile (16 consecutive cells per
// thread through LDS, the 256 thread sums scanned across wavefronts).
__device__ __forceinline__ int block_sum_i32(int v, int *sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  int t = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  return t;
}

__device__ __forceinline__ void scan_tiles_at(const int *__restrict__ count, int ncell, int *__restrict__ tile_sum,
                                              int tile) {
  __shared__ int sh[kScanNT / 64];
  const int base = tile * kScanTile;
  int v = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    const int i = base + k * kScanNT + (int)threadIdx.x;
    if (i < ncell) v += count[i];
  }
  v = block_sum_i32(v, sh);
  if (threadIdx.x == 0) tile_sum[tile] = v;
}

__global__ __launch_bounds__(kScanNT) void k_scan_tiles(const int *__restrict__ count, int ncell,
                                                        int *__restrict__ tile_sum) {
  scan_tiles_at(count, ncell, tile_sum, blockIdx.x);
}

__device__ __forceinline__ void scan_apply_at(const int *__restrict__ count, const int *__restrict__ tile_sum,
                                              int ncell, int *__restrict__ start, int tb) {
  __shared__ int tile[kScanTile];
  __shared__ int sh[kScanNT / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int base = tb * kScanTile;
  int off = 0;
  for (int k = t; k < tb; k += kScanNT) off += tile_sum[k];
  off = block_sum_i32(off, sh);
  for (int k = t; k < kScanTile; k += kScanNT) {
    const int i = base + k;
    tile[k] = i < ncell ? count[i] : 0;
  }
  __syncthreads();
  int loc = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) loc += tile[t * kScanPer + k];
  int v = loc;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  __syncthreads();  // sh is reused
  if (lane == 63) sh[wave] = v;
  __syncthreads();
  int wpre = 0;
  for (int w = 0; w < wave; ++w) wpre += sh[w];
  int run = off + wpre + v - loc;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    const int cnt = tile[t * kScanPer + k];
    tile[t * kScanPer + k] = run;
    run += cnt;
  }
  __syncthreads();
  for (int k = t; k < kScanTile; k += kScanNT) {
    const int i = base + k;
    if (i < ncell) start[i] = tile[k];
  }
  if (t == kScanNT - 1 && base + kScanTile >= ncell) start[ncell] = run;
}

__global__ __launch_bounds__(kScanNT) void k_scan_apply(const int *__restrict__ count, const int *__restrict__ tile_sum,
                                                        int ncell, int *__restrict__ start) {
  scan_apply_at(count, tile_sum, ncell, start, blockIdx.x);
}

__global__ void k_scatter(const int *__restrict__ cell_of, const int *__restrict__ slot, const int *__restrict__ start,
                          int *__restrict__ perm, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) perm[start[cell_of[i]] + slot[i]] = i;
}

// Order each cell's members by caller index: the sorted order (and with it
// every summation order downstream) is then deterministic.  One wavefront
// per cell: with at most 64 members each lane holds one and its rank is the
// number of smaller indices (the indices are distinct); larger cells fall
// back to an insertion sort by lane 0.  The sorted positions are gathered in
// the same pass.
template <typename T4>
__device__ __forceinline__ void cell_sort_at(const int *__restrict__ start, int *__restrict__ perm, int ncell,
                                             const T4 *__restrict__ pos_w, T4 *__restrict__ pos_s, int c) {
  const int lane = threadIdx.x & 63;
  if (c >= ncell) return;
  const int b = start[c], e = start[c + 1], m = e - b;
  if (m <= 64) {
    const int v = lane < m ? perm[b + lane] : 0x7FFFFFFF;
    int rank = 0;
    for (int j = 0; j < m; ++j) rank += __shfl(v, j, 64) < v ? 1 : 0;
    if (lane < m) {
      perm[b + rank] = v;
      pos_s[b + rank] = pos_w[v];
    }
    return;
  }
  if (lane != 0) return;
  for (int i = b + 1; i < e; ++i) {
    const int v = perm[i];
    int j = i - 1;
    while (j >= b && perm[j] > v) {
      perm[j + 1] = perm[j];
      --j;
    }
    perm[j + 1] = v;
  }
  for (int i = b; i < e; ++i) pos_s[i] = pos_w[perm[i]];
}

template <typename T4>
__global__ __launch_bounds__(256) void k_cell_sort(const int *__restrict__ start, int *__restrict__ perm, int ncell,
                                                   const T4 *__restrict__ pos_w, T4 *__restrict__ pos_s) {
  cell_sort_at<T4>(start, perm, ncell, pos_w, pos_s, (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
}

// ------------------------------------------------------- F, G evaluation
// FP32 modes: linear interpolation in an LDS table of (mu0 F, mu0 (G-F)).
struct FGTable {
  const float2 *tab;  // nodes, LDS or global
  float inv_dr;
  __device__ __forceinline__ void eval(float r2, float rinv, float &Fm, float &Dm) const {
    const float u = r2 * rinv * inv_dr;
    int k = (int)u;
    k = min(k, kTableK);
    const float f = u - (float)k;
    const float2 e0 = tab[k], e1 = tab[k + 1];
    Fm = fmaf(f, e1.x - e0.x, e0.x);
    Dm = fmaf(f, e1.y - e0.y, e0.y);
  }
};

// FP64 mode: Appendix A closed forms on the fly (Case 1 / Case 2), with the
// series of the wave complement below the small-r threshold.
struct FGExact {
  const double *ser;  // [2 * kSeriesTerms]: F then G series coefficients
  double xi, a, mu0, small_r2;
  __device__ __forceinline__ void eval(double r2, double rinv, double &Fm, double &Dm) const {
    const double r = r2 * rinv;
    double F, G;
    if (r2 < small_r2) {
      double Ff, Gf;
      if (r > 2.0 * a) {
        const double ci = 0.75 * a / r + 0.5 * a * a * a / (r * r2);
        F = ci;
        G = ci + 0.75 * a / r - 1.5 * a * a * a / (r * r2);
      } else {
        F = 1.0 - 9.0 * r / (32.0 * a);
        G = 1.0 - 3.0 * r / (16.0 * a);
      }
      Ff = 0.0;
      Gf = 0.0;
      for (int n = kSeriesTerms - 1; n >= 0; --n) {
        Ff = Ff * r2 + ser[n];
        Gf = Gf * r2 + ser[kSeriesTerms + n];
      }
      F -= Ff;
      G -= Gf;
    } else {
      const double sp = 1.7724538509055160273;
      const double x = xi, x2 = x * x, x3 = x2 * x, x4 = x2 * x2;
      const double r3 = r2 * r, r4 = r2 * r2, a2 = a * a;
      const double rm = r - 2.0 * a, rp = r + 2.0 * a;
      const double qp = 4.0 * a2 + 4.0 * a * r + 9.0 * r2, qm = 4.0 * a2 - 4.0 * a * r + 9.0 * r2;
      const double e1 = exp(-r2 * x2), e2 = exp(-rm * rm * x2), e3 = exp(-rp * rp * x2);
      const double c1 = erfc(r * x), c2 = erfc(rm * x), c3 = erfc(rp * x);
      const double i64 = 1.0 / (64.0 * sp * a * r3 * x3), i128 = 0.5 * i64;
      const double f1 = (18.0 * r2 * x2 + 3.0) / (64.0 * sp * a * r2 * x3);
      const double f2 = (2.0 * x2 * (2.0 * a - r) * qp - 2.0 * a - 3.0 * r) * i128;
      const double f3 = (-2.0 * x2 * rp * qm + 2.0 * a - 3.0 * r) * i128;
      const double f4 = (3.0 - 36.0 * r4 * x4) / (128.0 * a * r3 * x4);
      const double f5 = (4.0 * x4 * rm * rm * qp - 3.0) / (256.0 * a * r3 * x4);
      const double f6 = (4.0 * x4 * rp * rp * qm - 3.0) / (256.0 * a * r3 * x4);
      const double g1 = (6.0 * r2 * x2 - 3.0) / (32.0 * sp * a * r2 * x3);
      const double g2 = (-2.0 * x2 * rm * rm * (2.0 * a + 3.0 * r) + 2.0 * a + 3.0 * r) * i64;
      const double g3 = (2.0 * x2 * rp * rp * (2.0 * a - 3.0 * r) - 2.0 * a + 3.0 * r) * i64;
      const double g4 = -(3.0 * (4.0 * r4 * x4 + 1.0)) / (64.0 * a * r3 * x4);
      const double tm = 2.0 * a - r;
      const double g5 = (3.0 - 4.0 * x4 * tm * tm * tm * (2.0 * a + 3.0 * r)) / (128.0 * a * r3 * x4);
      const double g6 = (3.0 - 4.0 * x4 * (2.0 * a - 3.0 * r) * rp * rp * rp) / (128.0 * a * r3 * x4);
      double f0 = 0.0, g0 = 0.0;
      if (r <= 2.0 * a) {
        f0 = -rm * rm * qp / (32.0 * a * r3);
        g0 = tm * tm * tm * (2.0 * a + 3.0 * r) / (16.0 * a * r3);
      }
      F = f0 + f1 * e1 + f2 * e2 + f3 * e3 + f4 * c1 + f5 * c2 + f6 * c3;
      G = g0 + g1 * e1 + g2 * e2 + g3 * e3 + g4 * c1 + g5 * c2 + g6 * c3;
    }
    Fm = F * mu0;
    Dm = (G - F) * mu0;
  }
};

// ------------------------------------------ learned-preconditioner features
// 24 geometry features of one particle, accumulated over its near
// neighbours (minimum image, r < 4.5a; d = x_i - x_j, dh = d / r, dh = 0 at
// r = 0) with the dimensionless F, G of Appendix A; f3 alone counts every
// neighbour within rc:
//   0..3   #{r < 2.2a}/4, #{r < 3a}/8, #{r < 4.5a}/16, #{r <= rc}/128
//   4      sum F / 8
//   5..10  sum (G - F) dh dh^T (xx, yy, zz, xy, xz, yz)
//   11..16 sum_{r < 3a} dh dh^T / 4
//   17..19 sum_{r < 3a} dh / 4
//   20     sum (G - F)
//   21     min r / 4.5a (1 without near neighbours)
//   22     sum_{r < 3a} (3a - r) / a / 4
//   23     F_self (eq. self)
template <typename T> struct FeatAcc {
  T f[kNFeat];
  __device__ __forceinline__ void init(T fself) {
#pragma unroll
    for (int k = 0; k < kNFeat; ++k) f[k] = T(0);
    f[21] = T(1);
    f[23] = fself;
  }
  // one near neighbour (r < 4.5a): separation d, r and 1/r (0 at r = 0),
  // dimensionless F and G - F.  The 1/8 of f4 is applied in store(), f3
  // comes from the neighbour count there.
  __device__ __forceinline__ void add(T dx, T dy, T dz, T r, T ir, T Fd, T Dd, T a, T inv_near) {
    const T hx = dx * ir, hy = dy * ir, hz = dz * ir;
    f[0] += r < T(2.2) * a ? T(0.25) : T(0);
    f[2] += T(0.0625);
    f[4] += Fd;
    const T ex = Dd * hx, ey = Dd * hy, ez = Dd * hz;
    f[5] += ex * hx;
    f[6] += ey * hy;
    f[7] += ez * hz;
    f[8] += ex * hy;
    f[9] += ex * hz;
    f[10] += ey * hz;
    f[20] += Dd;
    f[21] = min(f[21], r * inv_near);
    if (r < T(3) * a) {  // close neighbours (a small fraction of the hits)
      f[1] += T(0.125);
      const T qx = T(0.25) * hx, qy = T(0.25) * hy, qz = T(0.25) * hz;
      f[11] += qx * hx;
      f[12] += qy * hy;
      f[13] += qz * hz;
      f[14] += qx * hy;
      f[15] += qx * hz;
      f[16] += qy * hz;
      f[17] += qx;
      f[18] += qy;
      f[19] += qz;
      f[22] += (T(3) * a - r) / a * T(0.25);
    }
  }
  __device__ __forceinline__ void store(uint16_t *__restrict__ out, int count) {
    f[3] = T(count) * T(1.0 / 128);
    f[4] *= T(0.125);
    uint32_t w[kNFeat / 2];
#pragma unroll
    for (int k = 0; k < kNFeat / 2; ++k)
      w[k] = (uint32_t)f32_to_bf16((float)f[2 * k]) | ((uint32_t)f32_to_bf16((float)f[2 * k + 1]) << 16);
    uint4 *o = (uint4 *)out;  // 48 bytes per particle: three 16-byte stores
    o[0] = make_uint4(w[0], w[1], w[2], w[3]);
    o[1] = make_uint4(w[4], w[5], w[6], w[7]);
    o[2] = make_uint4(w[8], w[9], w[10], w[11]);
  }
};

// Global near-field list (FP64, and FP32 boxes without an LDS block): row s
// holds the sorted indices nbr[s cap + k], k < cnt[s], of every t != s with
// minimum-image distance <= rc, in the order of the adjacent cells (fewer
// than 27 when a side has < 3 cells, so no cell is visited twice).
// With REP the overlap repulsion f_s = sum_{t: r < 2a} krep (2a - r) d / r
// (d = x_s - x_t) goes to frep[s].
//
// The adjacent cells of one (x, y) column: a run of consecutive z cells,
// split in two where it wraps.
struct CellRun {
  int a1, n1, a2, n;  // first particle and length of the first part, first of the second, total
  __device__ __forceinline__ int at(int i) const { return i < n1 ? a1 + i : a2 + (i - n1); }
};
__device__ __forceinline__ CellRun cell_run(const int *__restrict__ start, int nc, int ax, int ay, int z0, int nz) {
  const int base = (ax * nc + ay) * nc, zl = (z0 + nc) % nc, z1 = zl + nz - 1;
  CellRun r;
  r.a1 = start[base + zl];
  r.n1 = start[base + min(z1, nc - 1) + 1] - r.a1;
  r.a2 = start[base];
  r.n = r.n1 + (z1 >= nc ? start[base + z1 - nc + 1] - r.a2 : 0);
  return r;
}

// flags[1], flags[5]: largest count; flags[2..3]: total.  One set of atomics
// per workgroup: every wavefront hitting the same words serialises at the L2
// (about 12 ns each; testing the maxima with a load first is slower still, the
// loads queue behind the atomics: 212 -> 470 us with 4096 workgroups).
__device__ __forceinline__ void nbr_stats(unsigned long long mine, int mx, int *__restrict__ flags) {
  __shared__ unsigned long long wtot[16];
  __shared__ int wmx[16];
  const unsigned long long tot = wave_sum(mine);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off, 64));
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    wtot[wave] = tot;
    wmx[wave] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    int m = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      t += wtot[w];
      m = max(m, wmx[w]);
    }
    if (t) atomicAdd((unsigned long long *)(flags + 2), t);
    atomicMax(&flags[1], m);
    atomicMax(&flags[5], m);
  }
}

// 16 lanes per target scan its candidates, 16 at a time; the hits are
// compacted with a ballot into consecutive entries of the row.  (One lane per
// target took 150 us for 1000 particles, a serial scan on 16 wavefronts.)
constexpr int kRowLanes = 16;
template <typename T, bool REP>
__global__ __launch_bounds__(256) void k_nbr_rows(const typename vec4<T>::type *__restrict__ pos,
                                                  const int *__restrict__ start, int n, int nc, T L, T invL, T inv_cs,
                                                  T rc2, int *__restrict__ nbr, int *__restrict__ cnt_out, int cap,
                                                  int *__restrict__ flags, T a, T krep,
                                                  typename vec4<T>::type *__restrict__ frep) {
  constexpr int RL = kRowLanes;
  const int sub = threadIdx.x % RL, grp0 = ((threadIdx.x & 63) / RL) * RL;  // first lane of the group
  const int lo = nc >= 3 ? -1 : 0, nz = nc >= 3 ? 3 : (nc >= 2 ? 2 : 1);
  const int rows = gridDim.x * (256 / RL);
  unsigned long long mine = 0;
  int mx = 0;
  // a wavefront's groups leave the loop together (ballots below)
  for (int s0 = (blockIdx.x * 256 + (threadIdx.x & ~63)) / RL; s0 < n; s0 += rows) {
    const int s = s0 + grp0 / RL;
    const bool act = s < n;
    const auto p = pos[act ? s : n - 1];
    const int cx = min((int)(p.x * inv_cs), nc - 1), cy = min((int)(p.y * inv_cs), nc - 1),
              cz = min((int)(p.z * inv_cs), nc - 1);
    int cnt = 0;
    T fx = T(0), fy = T(0), fz = T(0);
    for (int dx = 0; dx < nz; ++dx)
      for (int dy = 0; dy < nz; ++dy) {
        const CellRun r = cell_run(start, nc, (cx + lo + dx + nc) % nc, (cy + lo + dy + nc) % nc, cz + lo, nz);
        const int tot = act ? r.n : 0;
        for (int c0 = 0; __any(c0 < tot); c0 += RL) {
          const int ci = c0 + sub, t = ci < tot ? r.at(ci) : s;
          const bool cand = ci < tot && t != s;
          const auto q = pos[cand ? t : (act ? s : n - 1)];
          const T ddx = min_image(p.x - q.x, L, invL);
          const T ddy = min_image(p.y - q.y, L, invL);
          const T ddz = min_image(p.z - q.z, L, invL);
          const T r2 = ddx * ddx + ddy * ddy + ddz * ddz;
          if (REP && cand && r2 < T(4) * a * a && r2 > T(0)) {
            const T rr = sqrt(r2), m = krep * (T(2) * a - rr) / rr;
            fx += m * ddx;
            fy += m * ddy;
            fz += m * ddz;
          }
          const bool hit = cand && r2 <= rc2;
          const unsigned gm = (unsigned)(__ballot(hit) >> grp0) & ((1u << RL) - 1u);
          const int slot = cnt + __popc(gm & ((1u << sub) - 1u));
          if (hit && slot < cap) nbr[(size_t)s * cap + slot] = t;
          cnt += __popc(gm);
        }
      }
    if (REP) {
#pragma unroll
      for (int off = RL / 2; off > 0; off >>= 1) {
        fx += __shfl_xor(fx, off, 64);
        fy += __shfl_xor(fy, off, 64);
        fz += __shfl_xor(fz, off, 64);
      }
    }
    if (act && sub == 0) {
      if (REP) {
        typename vec4<T>::type f;
        f.x = fx;
        f.y = fy;
        f.z = fz;
        f.w = T(0);
        frep[s] = f;
      }
      cnt_out[s] = min(cnt, cap);  // entries stored; flags[1] carries the capacity needed
      mine += (unsigned long long)cnt;
      mx = max(mx, cnt);
    }
  }
  nbr_stats(mine, mx, flags);
}

// The same list with the learned-preconditioner features of s accumulated
// from its hits (fg gives mu0 F and mu0 (G - F); FeatAcc): one lane per
// target, which holds the 24 sums.
template <typename T, typename FG, bool REP>
__global__ void k_nbr_feat(const typename vec4<T>::type *__restrict__ pos, const int *__restrict__ start, int n,
                           int nc, T L, T invL, T inv_cs, T rc2, int *__restrict__ nbr, int *__restrict__ cnt_out,
                           int cap, int *__restrict__ flags, FG fg, T inv_mu0, T fself, T a,
                           uint16_t *__restrict__ feat, T krep, typename vec4<T>::type *__restrict__ frep) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  int cnt = 0;
  if (s < n) {
    FeatAcc<T> acc;
    acc.init(fself);
    T fx = T(0), fy = T(0), fz = T(0);
    const auto p = pos[s];
    const int cx = min((int)(p.x * inv_cs), nc - 1), cy = min((int)(p.y * inv_cs), nc - 1),
              cz = min((int)(p.z * inv_cs), nc - 1);
    const int lo = nc >= 3 ? -1 : 0, nz = nc >= 3 ? 3 : (nc >= 2 ? 2 : 1);
    for (int dx = 0; dx < nz; ++dx)
      for (int dy = 0; dy < nz; ++dy) {
        const CellRun run = cell_run(start, nc, (cx + lo + dx + nc) % nc, (cy + lo + dy + nc) % nc, cz + lo, nz);
        for (int k = 0; k < run.n; ++k) {
          const int t = run.at(k);
          if (t == s) continue;
          const auto q = pos[t];
          const T ddx = min_image(p.x - q.x, L, invL);
          const T ddy = min_image(p.y - q.y, L, invL);
          const T ddz = min_image(p.z - q.z, L, invL);
          const T r2 = ddx * ddx + ddy * ddy + ddz * ddz;
          if (REP && r2 < T(4) * a * a && r2 > T(0)) {
            const T r = sqrt(r2), m = krep * (T(2) * a - r) / r;
            fx += m * ddx;
            fy += m * ddy;
            fz += m * ddz;
          }
          if (r2 <= rc2) {
            if (cnt < cap) nbr[(size_t)s * cap + cnt] = t;
            ++cnt;
            if (r2 < T(20.25) * a * a) {  // near shell r < 4.5a
              T Fm = fself / inv_mu0, Dm = T(0), r = T(0), ir = T(0);
              if (r2 > T(1e-24)) {
                r = sqrt(r2);
                ir = T(1) / r;
                fg.eval(r2, ir, Fm, Dm);
              }
              acc.add(ddx, ddy, ddz, r, ir, Fm * inv_mu0, Dm * inv_mu0, a, T(1) / (T(4.5) * a));
            }
          }
        }
      }
    acc.store(feat + (size_t)s * kNFeat, cnt);
    if (REP) {
      typename vec4<T>::type f;
      f.x = fx;
      f.y = fy;
      f.z = fz;
      f.w = T(0);
      frep[s] = f;
    }
    cnt_out[s] = min(cnt, cap);  // entries stored; flags[1] carries the capacity needed
  }
  nbr_stats((unsigned long long)cnt, cnt, flags);
}

// --------------------------------------------------- near-field product
// mu0 F and mu0 (G - F) / r^2 of one pair (the coincident limit is isotropic).
template <typename T, typename FG>
__device__ __forceinline__ void pair_coef(T r2, const FG &fg, T self_r, T &Fm, T &Dr) {
  if (r2 > T(1e-24)) {
    const T rinv = T(1) / sqrt(r2);
    T Dm;
    fg.eval(r2, rinv, Fm, Dm);
    Dr = Dm * rinv * rinv;
  } else {
    Fm = self_r;
    Dr = T(0);
  }
}

// FP64: both coefficients of every list entry, evaluated once per
// configuration.  The closed forms take six transcendental functions a pair;
// evaluated inside every product they were 112 us of the 116 us a product of
// 1000 particles took, 7 products a sample.  Positions without a product pay
// them too (300000 particles: list 435 -> 275 us, coefficients 460 us, so
// set_positions 506 -> 772 us, with one product 1100 -> 961 us).
__global__ __launch_bounds__(256) void k_pair_coef(const double4 *__restrict__ pos, const int *__restrict__ nbr,
                                                   const int *__restrict__ cnt, int n, int cap, double L, double invL,
                                                   FGExact fg, double self_r, double2 *__restrict__ coef) {
  // consecutive lanes take consecutive entries of a row; grid.y splits long rows
  const int sub = threadIdx.x % kRowLanes, s = (blockIdx.x * 256 + threadIdx.x) / kRowLanes;
  if (s >= n) return;
  const int c = cnt[s];
  const double4 p = pos[s];
  for (int k = blockIdx.y * kRowLanes + sub; k < c; k += gridDim.y * kRowLanes) {
    const size_t e = (size_t)s * cap + k;
    const double4 q = pos[nbr[e]];
    const double dx = min_image(p.x - q.x, L, invL), dy = min_image(p.y - q.y, L, invL),
                 dz = min_image(p.z - q.z, L, invL);
    double2 o;
    pair_coef(dx * dx + dy * dy + dz * dz, fg, self_r, o.x, o.y);
    coef[e] = o;
  }
}

// out_s = self * v_s + sum_{t in nbr(s)} mu0 [F v_t + (G-F)(d.v_t) d / r^2]
// with v = src: kRowLanes lanes per row, partial sums combined by lane
// shuffles.  A Lanczos iteration passes `done`, the flag of its state: once
// set the product is skipped (null: always formed).  The pair coefficients come
// from coef(entry, r^2, F, D).
template <typename T, typename Coef>
__device__ __forceinline__ void spmv_rows(const typename vec4<T>::type *__restrict__ pos, const int *__restrict__ nbr,
                                          const int *__restrict__ cnt, int n, int cap, T L, T invL, T self_r,
                                          const typename vec4<T>::type *__restrict__ src,
                                          typename vec4<T>::type *__restrict__ out, Coef coef) {
  using T4 = typename vec4<T>::type;
  constexpr int RL = kRowLanes;
  const int sub = threadIdx.x % RL, rows = gridDim.x * (blockDim.x / RL);
  for (int s0 = (blockIdx.x * blockDim.x + (threadIdx.x & ~63)) / RL; s0 < n; s0 += rows) {
    const int s = s0 + (threadIdx.x & 63) / RL;
    T ax = T(0), ay = T(0), az = T(0);
    if (s < n) {
      const T4 p = pos[s];
      const int c = cnt[s];
#pragma unroll 2
      for (int k = sub; k < c; k += RL) {
        const size_t e = (size_t)s * cap + k;
        const int t = nbr[e];
        const T4 q = pos[t];
        const T4 w = src[t];
        const T dx = min_image(p.x - q.x, L, invL);
        const T dy = min_image(p.y - q.y, L, invL);
        const T dz = min_image(p.z - q.z, L, invL);
        T F, Dr;
        coef(e, dx * dx + dy * dy + dz * dz, F, Dr);
        const T pr = Dr * (dx * w.x + dy * w.y + dz * w.z);
        ax += F * w.x + pr * dx;
        ay += F * w.y + pr * dy;
        az += F * w.z + pr * dz;
      }
    }
#pragma unroll
    for (int off = RL / 2; off > 0; off >>= 1) {
      ax += __shfl_xor(ax, off, 64);
      ay += __shfl_xor(ay, off, 64);
      az += __shfl_xor(az, off, 64);
    }
    if (s < n && sub == 0) {
      const T4 v = src[s];
      T4 o;
      o.x = ax + self_r * v.x;
      o.y = ay + self_r * v.y;
      o.z = az + self_r * v.z;
      o.w = T(0);
      out[s] = o;
    }
  }
}

__global__ __launch_bounds__(256) void k_spmv_table(const float4 *__restrict__ pos, const int *__restrict__ nbr,
                                                    const int *__restrict__ cnt, int n, int cap, float L, float invL,
                                                    const float2 *__restrict__ tab_g, float inv_dr, float self_r,
                                                    const float4 *__restrict__ src, float4 *__restrict__ out,
                                                    const int *__restrict__ done) {
  __shared__ float2 tab[kTableN];
  if (done && *done) return;
  for (int i = threadIdx.x; i < kTableN; i += blockDim.x) tab[i] = tab_g[i];
  __syncthreads();
  const FGTable fg{tab, inv_dr};
  spmv_rows<float>(pos, nbr, cnt, n, cap, L, invL, self_r, src, out,
                   [&](size_t, float r2, float &F, float &Dr) { pair_coef(r2, fg, self_r, F, Dr); });
}

__global__ __launch_bounds__(256) void k_spmv_coef(const double4 *__restrict__ pos, const int *__restrict__ nbr,
                                                   const int *__restrict__ cnt, int n, int cap, double L, double invL,
                                                   const double2 *__restrict__ coef, double self_r,
                                                   const double4 *__restrict__ src, double4 *__restrict__ out,
                                                   const int *__restrict__ done) {
  if (done && *done) return;
  spmv_rows<double>(pos, nbr, cnt, n, cap, L, invL, self_r, src, out, [&](size_t e, double, double &F, double &Dr) {
    const double2 c = coef[e];
    F = c.x;
    Dr = c.y;
  });
}

// where the coefficients found no memory (16 bytes per list slot)
__global__ __launch_bounds__(256) void k_spmv_exact(const double4 *__restrict__ pos, const int *__restrict__ nbr,
                                                    const int *__restrict__ cnt, int n, int cap, double L, double invL,
                                                    FGExact fg, double self_r, const double4 *__restrict__ src,
                                                    double4 *__restrict__ out, const int *__restrict__ done) {
  if (done && *done) return;
  spmv_rows<double>(pos, nbr, cnt, n, cap, L, invL, self_r, src, out,
                    [&](size_t, double r2, double &F, double &Dr) { pair_coef(r2, fg, self_r, F, Dr); });
}

// ------------------------------------------- LDS-staged near-field kernels
// Target blocks of B x B x B linked cells.  The block's halo, the (B+2)^3
// cells within one cell of its own, is staged in LDS once; the neighbour
// list then holds 16-bit LDS indices, so the product reads neighbours from
// LDS instead of gathering 16-byte records from global memory per pair.
// List layout: chunks of 8 indices, chunk q of sorted particle s at 16-byte
// slot (q * n + s): one coalesced 16-byte load per lane per 8 neighbours.
// The last chunk is padded with the index one past the halo (the product's
// zero source).
// Needs nc >= B + 2 (no halo cell appears twice).  B = 1 ... 4: blocks of
// more cells keep enough targets per workgroup when cells hold few
// particles (small rc).
//
// The halo is handled as (B+2)^2 columns of B + 2 consecutive z cells: the
// particles of a column are one contiguous run of the sorted order, or two
// where the column wraps around the box.  Every column is staged at the
// periodic image that continues the block's own coordinates across the box
// face, relative to the block centre.  Pairs then need no minimum-image
// correction: both particles sit in cells that touch, at the images in which
// they touch, and with at least 3 cells of side >= rc the other images of the
// pair are more than rc apart.  The staged coordinates are small (a few
// cells), so their differences keep the precision of the relative position
// rather than of the box size, except in the columns taken across a box face:
// there the distance to the block centre, of size L, is rounded first (at most
// L 2^-25).
template <int B> struct Halo {
  static constexpr int HB = B + 2;
  static constexpr int NH = HB * HB * HB;  // 27, 64, 125 or 216 halo cells
  static constexpr int NC = HB * HB;       // halo columns
  static constexpr int NT = B * B;         // target columns
};

template <int B> struct HaloTab {
  int g1[Halo<B>::NC], n1[Halo<B>::NC];  // first run: sorted index, length
  int g2[Halo<B>::NC];                   // second run (after the z face)
  int base[Halo<B>::NC + 1];             // LDS index of each column's first particle; the halo size
  int tl[Halo<B>::NT];                   // LDS index of each target column's first target
  int tpre[Halo<B>::NT + 1];             // exclusive prefix of the target counts
};

// blk: the block of B^3 cells this workgroup serves.  Columns past the box
// in the partial last blocks are staged like the others; their cells are no
// targets.  One wavefront, one lane per column: the column's cell starts are
// read together and the prefix sums taken across lanes.
template <int B>
__device__ __forceinline__ void halo_setup(const int *__restrict__ cell_start, int nc, HaloTab<B> &ht, int blk) {
  constexpr int HB = Halo<B>::HB, NC = Halo<B>::NC, NT = Halo<B>::NT;
  const int nb = (nc + B - 1) / B;
  const int bz = blk % nb, by = (blk / nb) % nb, bx = blk / (nb * nb);
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const int hx = lane / HB, hy = lane % HB;
    int len = 0, tlen = 0, toff = 0;
    if (lane < NC) {
      const int row = (((bx * B - 1 + hx + nc) % nc) * nc + (by * B - 1 + hy + nc) % nc) * nc;
      const int zl = bz * B - 1, z0 = zl < 0 ? nc - 1 : zl;  // first cell of the column
      const int split = min(HB, nc - z0);                    // cells before the face
      const int a1 = cell_start[row + z0], e1 = cell_start[row + z0 + split];
      const int a2 = cell_start[row], e2 = cell_start[row + HB - split];
      // targets: cells bz B ... of this column, as far as the box goes
      const int zt = bz * B, zn = min(B, nc - zt);
      const int t0 = cell_start[row + zt], t1 = cell_start[row + zt + zn];
      const bool targ = hx >= 1 && hx <= B && hy >= 1 && hy <= B && bx * B + hx - 1 < nc && by * B + hy - 1 < nc;
      ht.g1[lane] = a1;
      ht.n1[lane] = e1 - a1;
      ht.g2[lane] = a2;
      len = (e1 - a1) + (e2 - a2);
      tlen = targ ? t1 - t0 : 0;
      toff = zl < 0 ? (e1 - a1) + (t0 - a2) : t0 - a1;
    }
    int v = len;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int u = __shfl_up(v, off, 64);
      if (lane >= off) v += u;
    }
    if (lane < NC) ht.base[lane + 1] = v;
    if (lane == 0) ht.base[0] = 0;
    // lane t < B^2 takes target column t = (ox, oy)
    const int from = (lane / B + 1) * HB + lane % B + 1;
    const int tl = __shfl(v - len + toff, from & 63, 64);
    int w = __shfl(tlen, from & 63, 64);
    if (lane >= NT) w = 0;
    const int own = w;
#pragma unroll
    for (int off = 1; off < NT; off <<= 1) {
      const int u = __shfl_up(w, off, 64);
      if (lane >= off) w += u;
    }
    if (lane < NT) {
      ht.tl[lane] = tl;
      ht.tpre[lane] = w - own;
    }
    if (lane == NT - 1) ht.tpre[NT] = w;
  }
  __syncthreads();
}

// Sorted index of particle k of a halo column.
template <int B> __device__ __forceinline__ int column_at(const HaloTab<B> &ht, int col, int k) {
  const int n1 = ht.n1[col];
  return k < n1 ? ht.g1[col] + k : ht.g2[col] + (k - n1);
}

// The staged halo plus the zero-source slot fit the `hcap` records the
// launch reserved.  A launch whose capacity was fixed in advance (a
// captured graph replayed on new positions) may meet a larger halo: the
// workgroup then stages nothing, raises *ovf and returns, and the caller
// redoes that system with capacities sized for it.  Uniform per workgroup.
template <int B> __device__ __forceinline__ bool halo_fits(const HaloTab<B> &ht, int hcap, int *ovf) {
  const bool ok = ht.base[Halo<B>::NC] + 1 <= hcap;
  if (!ok && threadIdx.x == 0) atomicOr(ovf, 1);
  return ok;
}

// put(LDS index, sorted index, position relative to the block centre) for
// every halo particle: one wavefront per column.
template <int B, typename Put>
__device__ __forceinline__ void halo_stage(const float4 *__restrict__ pos, const HaloTab<B> &ht, int nc, float cs,
                                           float L, int blk, Put put) {
  constexpr int HB = Halo<B>::HB, NC = Halo<B>::NC;
  const int nb = (nc + B - 1) / B;
  const int bz = blk % nb, by = (blk / nb) % nb, bx = blk / (nb * nb);
  const float c0 = 0.5f * B * cs;
  const float cx = bx * B * cs + c0, cy = by * B * cs + c0, cz = bz * B * cs + c0;
  auto image = [&](int g) { return g < 0 ? -L : (g >= nc ? L : 0.0f); };
  const float zs1 = image(bz * B - 1), zs2 = bz == 0 ? 0.0f : L;  // of the two runs
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  for (int col = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); col < NC; col += nw) {
    const float xs = image(bx * B - 1 + col / HB), ys = image(by * B - 1 + col % HB);
    const int b0 = ht.base[col], len = ht.base[col + 1] - b0, n1 = ht.n1[col], g1 = ht.g1[col], g2 = ht.g2[col];
#pragma unroll 2
    for (int k = lane; k < len; k += 64) {
      const bool first = k < n1;
      const int g = first ? g1 + k : g2 + (k - n1);
      float4 q = pos[g];
      q.x = (q.x - cx) + xs;
      q.y = (q.y - cy) + ys;
      q.z = (q.z - cz) + (first ? zs1 : zs2);
      put(b0 + k, g, q);
    }
  }
}

// target i of the block -> (target column, LDS index, sorted index)
template <int B>
__device__ __forceinline__ void target_of(const HaloTab<B> &ht, int i, int &t, int &li, int &s) {
  // largest target column t with tpre[t] <= i
  t = 0;
  int hi = Halo<B>::NT;
  while (hi - t > 1) {
    const int mid = (t + hi) >> 1;
    if (ht.tpre[mid] <= i) t = mid;
    else hi = mid;
  }
  li = ht.tl[t] + (i - ht.tpre[t]);
  const int col = (t / B + 1) * Halo<B>::HB + t % B + 1;
  s = column_at<B>(ht, col, li - ht.base[col]);
}

// Per-block halo sizes (largest goes to flags[4]) for sizing the LDS: one
// wavefront per block, lane (hx, hy) takes its column of HB halo cells, one or
// two runs of consecutive cells.  At most kHaloWG workgroups walk the blocks and
// add one maximum each: one atomic per block (about 8 ns each, all on one
// word) took 33 us at 10^6 and 93 us at 4 10^6 particles, this 5 and 7 us.
constexpr int kHaloWG = 256, kHaloNT = 512;
template <int B>
__global__ __launch_bounds__(kHaloNT) void k_halo_size(const int *__restrict__ cell_start, int nc,
                                                       int *__restrict__ flags) {
  constexpr int HB = Halo<B>::HB, NW = kHaloNT / 64;
  static_assert(HB * HB <= 64, "one lane per halo column");
  __shared__ int sh[NW];
  const int nb = (nc + B - 1) / B, nblocks = nb * nb * nb;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int hx = lane / HB, hy = lane % HB;
  int mx = 0;
  for (int blk = (int)blockIdx.x * NW + wave; blk < nblocks; blk += (int)gridDim.x * NW) {
    const int bz = blk % nb, by = (blk / nb) % nb, bx = blk / (nb * nb);
    int tot = 0;
    if (lane < HB * HB) {
      const int row = (((bx * B - 1 + hx + nc) % nc) * nc + (by * B - 1 + hy + nc) % nc) * nc;
      const int zl = bz * B - 1, z0 = zl < 0 ? nc - 1 : zl, split = min(HB, nc - z0);
      tot = cell_start[row + z0 + split] - cell_start[row + z0] + cell_start[row + HB - split] - cell_start[row];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    mx = max(mx, tot);
  }
  if (lane == 0) sh[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < NW; ++w) mx = max(mx, sh[w]);
    atomicMax(&flags[4], mx);
  }
}

// Neighbour list of a target block on the matrix cores.  The squared
// distances of 16 targets to 16 candidates, less rc^2, are one
// v_mfma_f32_16x16x4_f32:
//   D[c][t] = sum_k A[c][k] B[k][t] + (|p_t|^2 - rc^2),
//   A[c] = (x, y, z, |q|^2) of candidate c,  B[.][t] = (-2x, -2y, -2z, 1) of target t,
// whose sign is the hit: lane l holds the results of target l % 16 and four
// candidates, and shifts their sign bits into its hit word (one v_alignbit
// each).  A tile is 16 consecutive targets of a z column of the block; its
// candidates are the 9 columns around it, from the cell below its first
// target to the cell above its last, in segments of at most 8 x 16.  Lane
// quarter q = l / 16 takes the q-th quarter of a segment, so its bits are
// consecutive candidates and a row lists its neighbours in candidate order.
// The bit counts give each lane its place in the target's row; the hits
// are then taken out one by one into a stage in LDS and written to the list 8
// at a time.
// D carries a rounding error of at most 10 u (|p| + |q|)^2, u = 2^-24, the
// directly computed (x_p - x_q)^2 + ... one of 4 u rc^2.  A segment in which
// any |D| lies within their sum, for |q| <= |p| + rc, is evaluated directly
// instead (about one in 200), so the list holds exactly the pairs of the direct
// test.
// One lane per target with direct distances (19 VALU instructions a candidate)
// took 33 us at 10^3 spheres, 99 us at 8000 with rc = 6.3a and the repulsion,
// 65 us at 64000, 267 us at 10^6 (rc = 5.9a: 390 candidates and 60 hits a
// target); this takes 14, 36, 34 and 270 us.  Small systems gain from the 16 x 4
// split of a target's candidates; large ones are bound by taking out the hits,
// where the lane with most hits of a word sets the pace.  Interleaving the
// quarters evens that out (231 us at 10^6) but reorders the list, and with it
// the rounding of the learned features.
// flags[1]: list capacity needed; flags[5]: largest count.  With REP the
// overlap repulsion of each target,
//   f_s = sum_{t: r < 2a} krep (2a - r) d / r,  d = x_s - x_t,
// is accumulated into frep[s]: from its hits (kRepHits) where rc >= 2a, as in
// every chosen parameter set; else (kRepAll) from all candidates in the cells
// around its own, as in the global list.
enum Rep { kRepNone, kRepHits, kRepAll };
constexpr int kNbrNT = 768, kNbrWaves = kNbrNT / 64;
constexpr int kNbrPad = 16;    // halo records read past the last one
constexpr int kNbrRound = 48;  // hits of one word a target may stage
constexpr int kNbrStage = 7 + kNbrRound + 1;  // entries per target: with the rest of a chunk
static_assert(kNbrStage % 8 == 0, "rows of whole chunks");
__device__ __forceinline__ void lds_order() {
  // a wavefront's own LDS accesses stay in program order across lanes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// part of `parts`: workgroups that share the block's tiles (small systems)
template <int B, Rep REP>
__device__ __forceinline__ void nbr_lds_block(const float4 *__restrict__ pos, const int *__restrict__ cell_start,
                                              int nc, float cs, int n, float L, float rc, float rc2,
                                              uint16_t *__restrict__ nbr, int *__restrict__ cnt_out, int cap,
                                              int *__restrict__ flags, float contact, float krep,
                                              float4 *__restrict__ frep, int hcap, int blk, int part, int parts) {
  constexpr int HB = Halo<B>::HB, NC = Halo<B>::NC, NT = Halo<B>::NT;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  extern __shared__ float hal[];  // planes x, y, z, |q|^2, hs floats each
  __shared__ HaloTab<B> ht;
  __shared__ int cbase[NC * HB + 1];  // LDS index of each halo cell's first particle (z fastest)
  __shared__ int tp[NT + 1];          // exclusive prefix of the target columns' tiles
  __shared__ __attribute__((aligned(16))) uint16_t stage_all[kNbrWaves][16][kNbrStage];
  const int hs = hcap + kNbrPad;
  halo_setup<B>(cell_start, nc, ht, blk);
  if (!halo_fits<B>(ht, hcap, flags + 7)) return;
  {
    const int nb = (nc + B - 1) / B;
    const int bz = blk % nb, by = (blk / nb) % nb, bx = blk / (nb * nb);
    for (int h = threadIdx.x; h < NC * HB; h += blockDim.x) {
      const int col = h / HB, hz = h % HB, gz = bz * B - 1 + hz;
      const int row = (((bx * B - 1 + col / HB + nc) % nc) * nc + (by * B - 1 + col % HB + nc) % nc) * nc;
      const int c = cell_start[row + (gz + nc) % nc];
      const bool second = bz == 0 ? gz >= 0 : gz >= nc;
      cbase[h] = ht.base[col] + (second ? ht.n1[col] + c - ht.g2[col] : c - ht.g1[col]);
    }
    if (threadIdx.x == 0) {
      cbase[NC * HB] = ht.base[NC];
      int k = 0;
      for (int t = 0; t < NT; ++t) {
        tp[t] = k;
        k += (ht.tpre[t + 1] - ht.tpre[t] + 15) / 16;
      }
      tp[NT] = k;
    }
  }
  halo_stage<B>(pos, ht, nc, cs, L, blk, [&](int e, int, const float4 &q) {
    hal[e] = q.x;
    hal[hs + e] = q.y;
    hal[2 * hs + e] = q.z;
    hal[3 * hs + e] = q.x * q.x + q.y * q.y + q.z * q.z;
  });
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane >> 4, col = lane & 15;
  const int ntile = tp[NT], tpl = tp[min(lane, NT)];
  uint16_t *stage = stage_all[wave][col];
  uint4 *row = (uint4 *)nbr;
  unsigned long long mine = 0;
  int mx = 0;
  for (int tile = wave * parts + part; tile < ntile; tile += parts * kNbrWaves) {
    // the tile's target column: the last whose first tile is not past it
    const int tc = __popcll(__ballot(lane <= NT && tpl <= tile)) - 1;
    const int ox = tc / B, oy = tc % B, t0 = 16 * (tile - tp[tc]);
    const int nt16 = min(16, ht.tpre[tc + 1] - ht.tpre[tc] - t0);  // targets of the tile
    const bool targ = col < nt16;
    const int li = ht.tl[tc] + t0 + min(col, nt16 - 1);
    const int hcol = (ox + 1) * HB + oy + 1;
    const int s = column_at<B>(ht, hcol, li - ht.base[hcol]);
    int oz = 0;  // the target's cell in its column
    while (oz < B - 1 && cbase[hcol * HB + 2 + oz] <= li) ++oz;
    const int z0 = __builtin_amdgcn_readlane(oz, 0), z1 = __builtin_amdgcn_readlane(oz, 15);
    const float px = hal[li], py = hal[hs + li], pz = hal[2 * hs + li], p2 = hal[3 * hs + li];
    const float bop = q == 0 ? -2.0f * px : (q == 1 ? -2.0f * py : (q == 2 ? -2.0f * pz : 1.0f));
    const float c0 = p2 - rc2;
    const float far = 2.0f * sqrtf(p2) + rc, margin = 8.5e-7f * far * far;  // 14 u (2 |p| + rc)^2
    float fx = 0.f, fy = 0.f, fz = 0.f;  // overlap repulsion (REP)
    int have = 0, chunks = 0;            // staged entries, chunks written (of the lane's target)
    auto repel = [&](int j) {
      const float dx = px - hal[j], dy = py - hal[hs + j], dz = pz - hal[2 * hs + j];
      const float r2 = dx * dx + dy * dy + dz * dz;
      if (r2 < contact * contact && r2 > 0.f) {
        const float r = sqrtf(r2), f = krep * (contact - r) / r;
        fx += f * dx;
        fy += f * dy;
        fz += f * dz;
      }
    };
    // the hits of a word, whose bit b is candidate jl + b, to the stage
    auto extract = [&](uint32_t w, int jl, uint16_t *at) {
      while (w) {
        const int j = jl + __builtin_ctz(w);
        w &= w - 1u;
        *at++ = (uint16_t)j;
        if (REP == kRepHits) repel(j);
      }
    };
    // this lane's place in the stage for its m hits; the target's total
    auto place = [&](int m, int &total) {
      const int s1 = __shfl_xor(m, 16, 64), s2 = __shfl_xor(m, 32, 64), s3 = __shfl_xor(m, 48, 64);
      total = m + s1 + s2 + s3;
      return (q & 1 ? s1 : 0) + (q & 2 ? s2 + s3 : 0);
    };
    // whole chunks of the stage to the list, the rest to its front
    auto flush = [&]() {
      lds_order();
      const int full = have >> 3;
      for (int c = q; c < full; c += 4) {
        const uint4 v = *(const uint4 *)(stage + 8 * c);
        if (chunks + c < (cap >> 3)) row[(size_t)(chunks + c) * n + s] = v;
      }
      lds_order();
      if (q == 0 && full) *(uint4 *)stage = *(const uint4 *)(stage + 8 * full);
      lds_order();
      chunks += full;
      have &= 7;
    };
    for (int d = 0; d < 9; ++d) {
      const int cc = (hcol + (d / 3 - 1) * HB + d % 3 - 1) * HB;
      const int j0 = __builtin_amdgcn_readfirstlane(cbase[cc + z0]), je = __builtin_amdgcn_readfirstlane(cbase[cc + z1 + 3]);
      for (int jb = j0; jb < je; jb += 128) {
        const int nt = min(8, (je - jb + 15) >> 4);  // tiles of 16 candidates
        // operand row col, plane q of candidate col / 4 * 4 nt + 4 t + col % 4
        // of the segment
        const float *ap = hal + q * hs + jb + (col >> 2) * 4 * nt + (col & 3);
        uint32_t w = 0u;
        float mn = 1e30f;
        auto take = [&](const f32x4 &D4) {
#pragma unroll
          for (int v = 3; v >= 0; --v) w = __builtin_amdgcn_alignbit(w, __float_as_uint(D4[v]), 31);
          mn = fminf(fminf(mn, fabsf(D4[0])), fabsf(D4[1]));
          mn = fminf(fminf(mn, fabsf(D4[2])), fabsf(D4[3]));
        };
        const f32x4 C4 = {c0, c0, c0, c0};
        int t = nt - 1;
        for (; t > 0; t -= 2) {  // two in flight
          const float a1 = ap[4 * t], a0 = ap[4 * t - 4];
          const f32x4 D1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, bop, C4, 0, 0, 0);
          const f32x4 D0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, bop, C4, 0, 0, 0);
          take(D1);
          take(D0);
        }
        if (t == 0) take(__builtin_amdgcn_mfma_f32_16x16x4f32(ap[0], bop, C4, 0, 0, 0));
        const int jl = jb + q * 4 * nt;  // this lane's first candidate
        const int valid = targ ? min(max(je - jl, 0), 4 * nt) : 0;
        if (__any(mn < margin)) {
          w = 0u;
          for (int b = 0; b < valid; ++b) {
            const float dx = px - hal[jl + b], dy = py - hal[hs + jl + b], dz = pz - hal[2 * hs + jl + b];
            const float r2 = dx * dx + dy * dy + dz * dz;
            w |= r2 <= rc2 ? 1u << b : 0u;
          }
        }
        w &= valid >= 32 ? 0xffffffffu : (1u << valid) - 1u;
        if (d == 4 && (unsigned)(li - jl) < 32u) w &= ~(1u << (li - jl));  // not itself
        if (REP == kRepAll) {
          const int jhi = min(jl + valid, cbase[cc + oz + 3]);
          for (int j = max(jl, cbase[cc + oz]); j < jhi; ++j) repel(j);
        }
        int total;
        const int off = place(__popc(w), total);
        if (__any(have + total > kNbrStage - 1)) flush();  // leaves at most 7
        if (!__any(total > kNbrRound)) {
          extract(w, jl, stage + have + off);
          have += total;
        } else {
          // more than the stage takes: a quarter of the word (at most 32 hits a target) at a time
          for (int sh = 0; sh < 32; sh += 8) {
            const uint32_t wq = w & (0xffu << sh);
            const int offq = place(__popc(wq), total);
            extract(wq, jl, stage + have + offq);
            have += total;
            flush();
          }
        }
      }
    }
    flush();
    const int cnt = 8 * chunks + have;
    if (have) {
      // the rest of the last chunk points at the zero-source slot the product
      // stages after the halo (index = halo size)
      const uint16_t none = (uint16_t)ht.base[NC];
      if (2 * q >= have) stage[2 * q] = none;
      if (2 * q + 1 >= have) stage[2 * q + 1] = none;
      lds_order();
      if (q == 0 && targ && chunks < (cap >> 3)) row[(size_t)chunks * n + s] = *(const uint4 *)stage;
      lds_order();
    }
    if (REP) {
      fx += __shfl_xor(fx, 16, 64);
      fy += __shfl_xor(fy, 16, 64);
      fz += __shfl_xor(fz, 16, 64);
      fx += __shfl_xor(fx, 32, 64);
      fy += __shfl_xor(fy, 32, 64);
      fz += __shfl_xor(fz, 32, 64);
    }
    if (q == 0 && targ) {
      cnt_out[s] = min(cnt, cap);  // entries stored; flags[1] carries the capacity needed
      if (REP) frep[s] = make_float4(fx, fy, fz, 0.f);
      mine += (unsigned long long)cnt;
      mx = max(mx, cnt);
    }
  }
  nbr_stats(mine, mx, flags);
}

template <int B, Rep REP>
__global__ __launch_bounds__(kNbrNT) __attribute__((amdgpu_waves_per_eu(REP ? 4 : 6))) void k_nbr_lds(const float4 *__restrict__ pos, const int *__restrict__ cell_start,
                                                    int nc, float cs, int n, float L, float rc, float rc2,
                                                    uint16_t *__restrict__ nbr, int *__restrict__ cnt_out, int cap,
                                                    int *__restrict__ flags, float contact, float krep,
                                                    float4 *__restrict__ frep, int hcap, int parts) {
  const int b = xcd_block(blockIdx.x, gridDim.x);
  nbr_lds_block<B, REP>(pos, cell_start, nc, cs, n, L, rc, rc2, nbr, cnt_out, cap, flags, contact, krep, frep, hcap,
                        b / parts, b % parts, parts);
}

// The neighbour build of many systems (a batch of replicas) in one launch:
// pmap lists (system, block of that system) per workgroup.
template <int B>
__global__ __launch_bounds__(kNbrNT) __attribute__((amdgpu_waves_per_eu(6))) void k_nbr_lds_batch(const NbrRep *__restrict__ reps,
                                                          const int2 *__restrict__ pmap) {
  const int2 rb = pmap[blockIdx.x];
  const NbrRep &r = reps[rb.x];
  nbr_lds_block<B, kRepNone>(r.pos, r.cell_start, r.nc, r.cs, r.n, r.L, r.rc, r.rc2, r.nbr, r.cnt, r.cap, r.flags, 0.0f,
                          0.0f, nullptr, r.hcap, rb.y, 0, 1);
}

// Preconditioner features (FeatAcc; F, G from the LDS table).  Three lanes
// per target, as in the product:
// lane q of a group scans neighbour chunks q, q + 3, ... against the staged
// halo and queues every entry closer than 4.5a in its column of an LDS
// queue.  The queue is drained (one FeatAcc.add per entry) when some lane of
// the wavefront could overflow it, and at the end, so a wavefront spends on
// the features about its largest near count rather than the largest per
// chunk summed over chunks.  The three partial sums are then combined with
// lane shuffles (the minimum for f21).
constexpr int kFeatQ = 16;    // queue entries per lane
constexpr int kFeatNT = 512;  // lanes per workgroup (two workgroups per CU)
template <int B>
__global__ __launch_bounds__(kFeatNT) void k_feat_lds(const float4 *__restrict__ pos, const int *__restrict__ cell_start,
                                                   int nc, float cs, int n, float L,
                                                   const uint16_t *__restrict__ nbr, const int *__restrict__ cnt,
                                                   const float2 *__restrict__ tab, float inv_dr, float inv_mu0,
                                                   float fself, float a, float near2, uint16_t *__restrict__ feat,
                                                   int hcap, int *__restrict__ ovf) {
  constexpr int G = 3, GPW = 64 / G;
  extern __shared__ float4 hpos[];
  __shared__ HaloTab<B> ht;
  __shared__ uint16_t queue[kFeatQ * kFeatNT];
  __shared__ float2 ftab[kTableN];
  for (int k = threadIdx.x; k < kTableN; k += blockDim.x) ftab[k] = tab[k];
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  halo_setup<B>(cell_start, nc, ht, blk);
  if (!halo_fits<B>(ht, hcap, ovf)) return;
  halo_stage<B>(pos, ht, nc, cs, L, blk, [&](int e, int, const float4 &q) { hpos[e] = q; });
  __syncthreads();
  const FGTable fg{ftab, inv_dr};
  const int ntarg = ht.tpre[Halo<B>::NT];
  const uint4 *row = (const uint4 *)nbr;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / G, g = lane - grp * G;
  const bool ingrp = grp < GPW;
  uint16_t *myq = queue + threadIdx.x;  // entry t at myq[kFeatNT t]
  for (int i0 = 0; i0 < ntarg; i0 += (int)(blockDim.x >> 6) * GPW) {
    const int i = i0 + wave * GPW + grp;
    const bool act = ingrp && i < ntarg;
    int h = 0, li = 0, s = 0;
    if (act) target_of<B>(ht, i, h, li, s);
    const float4 p = hpos[li];
    FeatAcc<float> acc;
    acc.init(0.0f);
    int nq = 0;
    // one near pair into the sums (F, G - F from the LDS table)
    auto add = [&](const float4 &q) {
      const float ddx = p.x - q.x, ddy = p.y - q.y, ddz = p.z - q.z;
      const float r2 = ddx * ddx + ddy * ddy + ddz * ddz;
      const bool nz = r2 > 1e-24f;
      const float ir = nz ? __frsqrt_rn(r2) : 0.0f;
      float Fm = fself / inv_mu0, Dm = 0.0f;
      if (nz) fg.eval(r2, ir, Fm, Dm);
      acc.add(ddx, ddy, ddz, r2 * ir, ir, Fm * inv_mu0, Dm * inv_mu0, a, 1.0f / (4.5f * a));
    };
    // two queue entries per pass: their LDS reads are in flight together
    auto drain = [&]() {
      for (int t = 0; t < nq; t += 2) {
        const bool two = t + 1 < nq;
        const int j0 = myq[kFeatNT * t], j1 = myq[kFeatNT * (two ? t + 1 : t)];
        const float4 q0 = hpos[j0], q1 = hpos[j1];
        add(q0);
        if (two) add(q1);
      }
      nq = 0;
    };
    const int c = act ? cnt[s] : 0;
    uint4 nxt = 8 * g < c ? row[(size_t)g * n + s] : make_uint4(0, 0, 0, 0);
    for (int kb = 8 * g; kb < c; kb += 8 * G) {
      const uint4 pk = nxt;
      if (kb + 8 * G < c) nxt = row[(size_t)((kb >> 3) + G) * n + s];
      const uint32_t wd[4] = {pk.x, pk.y, pk.z, pk.w};
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = (wd[u >> 1] >> (16 * (u & 1))) & 0xFFFF;
        const float4 q = hpos[kb + u < c ? j : li];
        const float ddx = p.x - q.x, ddy = p.y - q.y, ddz = p.z - q.z;
        const float r2 = ddx * ddx + ddy * ddy + ddz * ddz;
        if (kb + u < c && r2 < near2) {
          myq[kFeatNT * nq] = (uint16_t)j;
          ++nq;
        }
      }
      // the next chunk adds at most 8 entries
      if (__any(nq > kFeatQ - 8)) drain();
    }
    drain();
    // combine the G lanes of the target (lanes G grp .. G grp + G - 1)
    const int base_lane = (lane / G) * G;
#pragma unroll
    for (int k = 0; k < kNFeat; ++k) {
      if (k == 3 || k == 23) continue;  // set by store() / the self value
      float v = acc.f[k];
#pragma unroll
      for (int o = 1; o < G; ++o) {
        const int srcl = base_lane + o < 64 ? base_lane + o : lane;
        const float t = __shfl(acc.f[k], srcl, 64);
        v = k == 21 ? fminf(v, t) : v + t;
      }
      acc.f[k] = v;
    }
    acc.f[23] = fself;
    if (act && g == 0) acc.store(feat + (size_t)s * kNFeat, c);
  }
}

// Near-field product from the staged halo.  The halo is packed as
// (x, y, z, v_x) + (v_y, v_z) (24 bytes per particle) together with the F/G
// table (mu0 F, mu0 (G - F) at nodes rc / 2048 apart; two 8-byte reads per
// pair for the linear interpolation).  G lanes per target (lane q of the group takes neighbour chunks
// q, q + G, ...; 64 / G groups per wavefront; 3 unless pse_autotune picks 2
// or 4) are combined with lane shuffles; each chunk of 8 neighbours is processed branch-free in two
// halves of 4 (padding entries read the zero source), the LDS reads of a half
// in flight together.  Registers are held to 64 so that two 1024-lane
// workgroups share a compute unit: one stages its halo while the other
// computes.
// A Lanczos iteration passes `done`, the flag of its state: once set the
// product is skipped (null: always formed).  With PC (Lanczos on
// A = P M_r P^T): src holds P^T u and the epilogue forms out = P M_r src;
// Pm holds the rows of P_i as (x, y, z, 0).
template <int B, bool PC, int G>
__device__ __forceinline__ void spmv_lds_block(const float4 *__restrict__ pos, const float4 *__restrict__ src,
                                               const int *__restrict__ cell_start, int nc, float cs, int n, int hcap,
                                               float L, const uint16_t *__restrict__ nbr,
                                               const int *__restrict__ cnt, const float2 *__restrict__ tab,
                                               float inv_dr, float self_r, float4 *__restrict__ out,
                                               const int *__restrict__ done, int *__restrict__ ovf,
                                               const float4 *__restrict__ Pm, int blk) {
  static_assert(G >= 2 && G <= 4, "lanes per target");
  constexpr int GPW = 64 / G;               // groups per wavefront (lane 63 idle at G = 3)
  extern __shared__ float4 smem[];
  float4 *hA = smem;                        // (x, y, z, v_x)
  float2 *hB = (float2 *)(smem + hcap);     // (v_y, v_z)
  __shared__ float2 tabs[kTableN];
  __shared__ HaloTab<B> ht;
  if (done && *done) return;
  for (int k = threadIdx.x; k < kTableN; k += blockDim.x) tabs[k] = tab[k];
  halo_setup<B>(cell_start, nc, ht, blk);
  // a halo past the capacity stages nothing and computes no target
  const bool fits = halo_fits<B>(ht, hcap, ovf);
  if (fits) {
    // slot `total`: a source with zero vector at the block centre, read by
    // the padding entries of the neighbour chunks (contributes exactly 0)
    // coordinates are staged in units of the table spacing rc / kTableK:
    // r is then the table coordinate itself (the (G - F) term is invariant)
    if (threadIdx.x == 0) {
      const int total = ht.base[Halo<B>::NC];
      hA[total] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      hB[total] = make_float2(0.0f, 0.0f);
    }
    halo_stage<B>(pos, ht, nc, cs, L, blk, [&](int e, int gi, const float4 &q) {
      const float4 v = src[gi];
      hA[e] = make_float4(q.x * inv_dr, q.y * inv_dr, q.z * inv_dr, v.x);
      hB[e] = make_float2(v.y, v.z);
    });
  }
  __syncthreads();
  const int ntarg = fits ? ht.tpre[Halo<B>::NT] : 0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / G, g = lane - grp * G;
  const bool ingrp = grp < GPW;
  for (int i0 = 0; i0 < ntarg; i0 += (int)(blockDim.x >> 6) * GPW) {
    const int i = i0 + wave * GPW + grp;
    const bool act = ingrp && i < ntarg;
    int h = 0, li = 0, s = 0;
    if (act) target_of<B>(ht, i, h, li, s);
    const float4 pa = hA[li];
    const float2 pb = hB[li];
    float ax = 0.f, ay = 0.f, az = 0.f;
    const int c = act ? cnt[s] : 0;
    const uint4 *row = (const uint4 *)nbr + s;
    // the next chunk of indices is loaded while the current one is used
    uint4 nxt = 8 * g < c ? row[(size_t)g * n] : make_uint4(0, 0, 0, 0);
    for (int kb = 8 * g; kb < c; kb += 8 * G) {
      const uint4 pk = nxt;
      if (kb + 8 * G < c) nxt = row[(size_t)((kb >> 3) + G) * n];
      const uint32_t wd[4] = {pk.x, pk.y, pk.z, pk.w};
      // entries past the count in the last chunk hold the zero-source slot;
      // two halves of 4: all halo reads of a half first, then its table reads
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        int jj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) jj[u] = (wd[2 * hf + (u >> 1)] >> (16 * (u & 1))) & 0xFFFF;
        float4 q[4];
        float2 wb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          q[u] = hA[jj[u]];
          wb[u] = hB[jj[u]];
        }
        float dx[4], dy[4], dz[4], rinv[4], fr[4];
        int kk[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          dx[u] = pa.x - q[u].x;
          dy[u] = pa.y - q[u].y;
          dz[u] = pa.z - q[u].z;
          const float r2 = fmaxf(dx[u] * dx[u] + dy[u] * dy[u] + dz[u] * dz[u], 1e-20f);
          rinv[u] = __frsqrt_rn(r2);
          const float uu = r2 * rinv[u];
          kk[u] = min((int)uu, kTableK);
          fr[u] = __builtin_amdgcn_fractf(uu);
        }
        float2 e0[4], e1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          e0[u] = tabs[kk[u]];
          e1[u] = tabs[kk[u] + 1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float wx = q[u].w, wy = wb[u].x, wz = wb[u].y;
          const float Fm = fmaf(fr[u], e1[u].x - e0[u].x, e0[u].x);
          const float Dm = fmaf(fr[u], e1[u].y - e0[u].y, e0[u].y);
          const float pr = Dm * rinv[u] * rinv[u] * (dx[u] * wx + dy[u] * wy + dz[u] * wz);
          ax = fmaf(pr, dx[u], fmaf(Fm, wx, ax));
          ay = fmaf(pr, dy[u], fmaf(Fm, wy, ay));
          az = fmaf(pr, dz[u], fmaf(Fm, wz, az));
        }
      }
    }
    // combine the G lanes of the target (lanes G grp .. G grp + G - 1)
    const int base_lane = (lane / G) * G;
    float sx = ax, sy = ay, sz = az;
#pragma unroll
    for (int o = 1; o < G; ++o) {
      const int srcl = base_lane + o < 64 ? base_lane + o : lane;
      const float tx = __shfl(ax, srcl, 64), ty = __shfl(ay, srcl, 64), tz = __shfl(az, srcl, 64);
      sx += tx;
      sy += ty;
      sz += tz;
    }
    if (act && g == 0) {
      sx += self_r * pa.w;
      sy += self_r * pb.x;
      sz += self_r * pb.y;
      if (PC) {
        const float tx = sx, ty = sy, tz = sz;
        const float4 p0 = Pm[3 * (size_t)s], p1 = Pm[3 * (size_t)s + 1], p2 = Pm[3 * (size_t)s + 2];
        sx = p0.x * tx + p0.y * ty + p0.z * tz;
        sy = p1.x * tx + p1.y * ty + p1.z * tz;
        sz = p2.x * tx + p2.y * ty + p2.z * tz;
      }
      out[s] = make_float4(sx, sy, sz, 0.0f);
    }
  }
}

template <int B, bool PC = false, int G = 3>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_spmv_lds(
    const float4 *__restrict__ pos, const float4 *__restrict__ src, const int *__restrict__ cell_start, int nc, float cs,
    int n, int hcap, float L, const uint16_t *__restrict__ nbr, const int *__restrict__ cnt,
    const float2 *__restrict__ tab, float inv_dr, float self_r, float4 *__restrict__ out,
    const int *__restrict__ done, int *__restrict__ ovf, const float4 *__restrict__ Pm = nullptr) {
  spmv_lds_block<B, PC, G>(pos, src, cell_start, nc, cs, n, hcap, L, nbr, cnt, tab, inv_dr, self_r, out,
                                   done, ovf, Pm, xcd_block(blockIdx.x, gridDim.x));
}

// ------------------------------------------------------------- Lanczos
// Iteration m on the basis of unnormalised vectors (LzState):
//   t = M_r u_m                                       (the product)
//   alpha_m = <v_m, M_r v_m> = rs_m^2 <u_m, t>
//   u_{m+1} = 2^-e (rs_m t - alpha_m v_m - beta_m v_{m-1}),  beta_{m+1} = 2^e |u_{m+1}|
// and the check of iteration m: the square root of T_{m+1} and the stopping
// rule.  Systems of at most kLzStepMax particles take one launch of one
// workgroup for all of it (k_lz_step); larger ones the pair k_lz_alpha,
// k_lz_update.  The next product needs none of the scalars, and the next
// vector work only beta, so there the check of iteration m is queued as one
// more workgroup of iteration m + 1's k_lz_alpha, and only the last
// iteration's is a launch of its own.  Iteration m + 1 is then speculative:
// what it writes (the next basis slot, alpha, beta) is not read once the
// state is done.  A sample that needs fewer iterations than the one before pays
// one product more for it (115 us at 10^6 spheres), any other saves a launch of
// about 5 us an iteration.  A captured step, which queues more iterations than it
// needs, checks before the next product instead (no speculation).
__device__ __forceinline__ float dot3(float acc, const float4 &a, const float4 &b) {
  return acc + (a.x * b.x + a.y * b.y + a.z * b.z);
}
__device__ __forceinline__ double dot3(double acc, const float4 &a, const float4 &b) {
  return acc + ((double)a.x * (double)b.x + (double)a.y * (double)b.y + (double)a.z * (double)b.z);
}
__device__ __forceinline__ double dot3(double acc, const double4 &a, const double4 &b) {
  return acc + (a.x * b.x + a.y * b.y + a.z * b.z);
}

// The even exponent e of alpha (0 where alpha is no positive number).
template <typename A> __device__ __forceinline__ int lz_exponent(A alpha) {
  const int e = alpha > A(0) && isfinite(alpha) ? ilogb(alpha) : 0;
  return e - (e & 1);
}

// FP32 sums of iteration 0 take <z, t> as 2^-k <z, t>, k the exponent of |z| = b0
// (the later vectors are of order 1): |z|^2 mu0 may leave the range where
// |z|^2 and mu0 are well inside.  Powers of two change no digit.
template <typename A> __device__ __forceinline__ int lz_start_exponent(A b0) {
  return sizeof(A) == 4 && b0 > A(0) && isfinite(b0) ? ilogb(b0) : 0;
}
template <typename T4, typename T> __device__ __forceinline__ T4 scaled3(T4 a, T c) {
  a.x *= c;
  a.y *= c;
  a.z *= c;
  return a;
}

// State before iteration 0 from z2 = |z|^2 (one thread).
template <typename A> __device__ __forceinline__ void lz_begin(LzState<A> *st, A z2) {
  const A b0 = sqrt(z2);
  st->beta[0] = b0;
  st->rs[0] = b0 > A(0) ? A(1) / b0 : A(0);
  st->m = 0;
  st->rel_change = A(1);
  st->converged = b0 == A(0);
  st->nonfinite = !isfinite(b0);
  st->done = b0 == A(0) || !isfinite(b0);
}

// beta_{m+1} and rs_{m+1} from x2 = |u_{m+1}|^2 (one thread).
template <typename A> __device__ __forceinline__ void lz_set_beta(LzState<A> *st, int m, A x2) {
  const A nrm = sqrt(x2);
  st->beta[m + 1] = ldexp(nrm, lz_exponent(st->alpha[m]));
  st->rs[m + 1] = nrm > A(0) ? A(1) / nrm : A(0);
}

// u_{m+1} at one particle: c1 t - c2 u_m - c3 u_{m-1}, (x, y, z, 0).
template <typename T4, typename T>
__device__ __forceinline__ T4 lz_next(const T4 &t, const T4 &u, const T4 *__restrict__ uprev, int i, T c1, T c2, T c3) {
  T4 x;
  x.x = c1 * t.x - c2 * u.x;
  x.y = c1 * t.y - c2 * u.y;
  x.z = c1 * t.z - c2 * u.z;
  if (uprev) {
    const T4 q = uprev[i];
    x.x -= c3 * q.x;
    x.y -= c3 * q.y;
    x.z -= c3 * q.z;
  }
  x.w = T(0);
  return x;
}

// c1, c2, c3 of iteration m for alpha_m = al.
template <typename T, typename A>
__device__ __forceinline__ void lz_coef(const LzState<A> *st, int m, A al, T &c1, T &c2, T &c3) {
  const int e = -lz_exponent(al);
  c1 = (T)ldexp(st->rs[m], e);
  c2 = (T)ldexp(al * st->rs[m], e);
  c3 = m > 0 ? (T)ldexp(st->beta[m] * st->rs[m - 1], e) : T(0);
}

// Value of v in lane i (wave-uniform i) as a scalar.
__device__ __forceinline__ double lane_value(double v, int i) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i),
                          __builtin_amdgcn_readlane(__double2loint(v), i));
}

// r = sqrt(x) and ri = 1 / sqrt(x) for normal x > 0: the hardware estimate
// of 1 / sqrt(x), refined by the coupled Newton iteration g -> sqrt(x),
// h -> 1 / (2 sqrt(x)) to within about an ulp.
__device__ __forceinline__ void sqrt_pair(double x, double &r, double &ri) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double d = fma(-h, g, 0.5);
    g = fma(g, d, g);
    h = fma(h, d, h);
  }
  r = g;
  ri = 2.0 * h;
}

// 1 / x by the hardware estimate and two Newton steps (about an ulp).
__device__ __forceinline__ double rcp_newton(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// s = T^{1/2} e_1 for the n x n tridiagonal T (lane j holds the diagonal d[j]
// and e[j], which couples j and j + 1), Gershgorin bound in (1/4, 1], by the
// quadrature
//   lambda^{1/2} = sum_j w_j lambda / (lambda + t_j),   lambda in [1e-13, 1]
// (lz_quadrature; relative error 2e-15 there): lane j solves
// (T + t_j) x_j = T e_1 and s = sum_j w_j x_j.  Eliminating from the last
// row up leaves one stored factor per row: with pivots D_i, r_i = 1 / D_i,
//   x_0 = (D_0 - t) r_0,  x_1 = e_0 t r_0 r_1,  x_i = -e_{i-1} r_i x_{i-1}.
// A step of the elimination is one reciprocal and two FMAs for all nodes at
// once: about a microsecond at five rows, where the eigen-decomposition's
// chain of rotations took 10 (22 at eight rows).  False when some eigenvalue
// is below the range (T nearly singular or indefinite; between -t_j and 0 the
// sum has poles), or T is not finite: the caller then takes the
// eigen-decomposition, which clamps.  The test is on the trailing minors p of
// T - 1e-13, two FMAs a row beside the elimination; a minor that underflows
// counts as not positive.  X: 64 n values.
__device__ __forceinline__ bool tridiag_root_quadrature(int n, double d, double e, const double2 *__restrict__ nodes,
                                                        double *X, double &s) {
  const int lane = threadIdx.x & 63;
  const double2 tw = nodes[lane];
  double D = lane_value(d, n - 1), r = 0.0;
  double p = D - kRootLow, p1 = 1.0;  // minors of the rows from i on and from i + 1 on
  bool pos = p > 0.0;
  for (int i = n - 1; i > 0; --i) {
    const double ei = lane_value(e, i - 1), di = lane_value(d, i - 1), e2 = ei * ei;
    r = rcp_newton(D + tw.x);
    X[i * 64 + lane] = r;
    D = fma(-e2, r, di);
    const double p0 = fma(di - kRootLow, p, -e2 * p1);
    p1 = p;
    p = p0;
    pos = pos && p > 0.0;
  }
  if (!pos) return false;  // (the same in every lane)
  const double r0 = rcp_newton(D + tw.x);
  X[lane] = tw.y * D * r0;
  double x = lane_value(e, 0) * (tw.y * tw.x * r0) * r;  // r = r_1 here
  for (int i = 1; i < n; ++i) {
    if (i > 1) x *= -lane_value(e, i - 1) * X[i * 64 + lane];
    X[i * 64 + lane] = x;
  }
  // lane k sums row k over the nodes (rotated columns: no bank conflicts); the
  // columns are the other lanes'
  lds_order();
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  if (lane < n) {
    for (int j = 0; j < 64; j += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) a[u] += X[lane * 64 + ((j + u + lane) & 63)];
  }
  s = (a[0] + a[1]) + (a[2] + a[3]);
  return true;
}

// The same by implicit QL with Wilkinson-type shifts (A. Dubrulle, R. S. Martin
// and J. H. Wilkinson, "The implicit QL algorithm", Numer. Math. 12, 1968),
// negative eigenvalues taken as 0.  Lane k owns row k of the eigenvector
// matrix Q (stored column-major in LDS).  Returns s_k in lane k.
// A serial chain of rotations bounds it, so each rotation is kept short:
// uniform values are read from their lane as scalars instead of through LDS
// permutes, one reciprocal square root gives r, 1/r and with them the sine
// and cosine (no hypot, no divisions), the deflation test looks at every
// lane at once, and the updated column of Q stays in a register for the
// next rotation.  Entries of order 1 keep f^2 + g^2 in range.
__device__ double tridiag_root_ql(int n, double d, double e, double *Q, int &ok) {
  const int lane = threadIdx.x & 63;
  const double eps = 2.2e-16, tiny = 1e-290;
  for (int j = 0; j < n; ++j) Q[j * 64 + lane] = (lane == j) ? 1.0 : 0.0;
  ok = 1;
  for (int l = 0; l < n; ++l) {
    int iter = 0;
    while (true) {
      // the first negligible off-diagonal entry at or after l
      const double ad = fabs(d), an = __shfl_down(ad, 1, 64);
      const bool cut = lane >= n - 1 || fabs(e) <= eps * (ad + an);
      const unsigned long long cuts = __ballot(cut) >> l;
      const int mm = l + (cuts ? __ffsll((long long)cuts) - 1 : 0);
      if (mm == l) break;
      if (++iter > 60) {
        ok = 0;
        break;
      }
      const double dl = lane_value(d, l), el = lane_value(e, l);
      double g = (lane_value(d, l + 1) - dl) / (2.0 * el);
      double r = sqrt(g * g + 1.0);
      g = lane_value(d, mm) - dl + el / (g + copysign(r, g));
      double s = 1, c = 1, p = 0;
      bool early = false;
      double q1 = Q[mm * 64 + lane], dn = lane_value(d, mm);
      for (int i = mm - 1; i >= l; --i) {
        const double qi = Q[i * 64 + lane];
        const double ei = lane_value(e, i), di = lane_value(d, i);
        const double f = s * ei, b = c * ei;
        const double h2 = f * f + g * g;
        if (h2 < tiny) {
          if (lane == i + 1) {
            e = 0.0;
            d = dn - p;
          }
          if (lane == mm) e = 0.0;
          early = true;
          Q[(i + 1) * 64 + lane] = q1;
          break;
        }
        double ri;
        sqrt_pair(h2, r, ri);
        if (lane == i + 1) e = r;
        s = f * ri;
        c = g * ri;
        g = dn - p;
        r = (di - g) * s + 2.0 * c * b;
        p = s * r;
        if (lane == i + 1) d = g + p;
        g = c * r - b;
        Q[(i + 1) * 64 + lane] = s * qi + c * q1;
        q1 = c * qi - s * q1;
        dn = di;
      }
      if (early) continue;
      Q[l * 64 + lane] = q1;
      if (lane == l) {
        d = dn - p;
        e = g;
      }
      if (lane == mm) e = 0.0;
    }
    if (!ok) break;
  }
  lds_order();  // row 0 is lane 0's
  const double root = sqrt(d < 0.0 ? 0.0 : d);  // (NaN stays)
  double acc = 0;
  for (int j = 0; j < n; ++j) acc += Q[j * 64 + lane] * lane_value(root, j) * Q[j * 64];
  return acc;
}

// s = T^{1/2} e_1 by the quadrature, or by QL outside its range, at n = 1
// (where QL is one square root) and with force_ql, on T scaled by an even power of two, so that the root's scale is
// a power of two too.  True if by the quadrature; ok = 0 if neither.
__device__ __forceinline__ bool tridiag_root(int n, double d, double e, const double2 *__restrict__ nodes, double *X,
                                             bool force_ql, double &s, int &ok) {
  const int lane = threadIdx.x & 63;
  const double el = __shfl_up(e, 1, 64), g = fabs(d) + fabs(e) + (lane ? fabs(el) : 0.0);
  double bound = 0.0;  // Gershgorin
  for (int j = 0; j < n; ++j) bound = fmax(bound, lane_value(g, j));
  const bool scaled = bound > 0.0 && isfinite(bound);
  int ex = scaled ? ilogb(bound) + 1 : 0;
  ex += ex & 1;
  d = ldexp(d, -ex);
  e = ldexp(e, -ex);
  ok = 1;
  const bool quad = scaled && n > 1 && !force_ql && tridiag_root_quadrature(n, d, e, nodes, X, s);
  if (!quad) s = tridiag_root_ql(n, d, e, X, ok);
  s = ldexp(s, ex / 2);
  return quad;
}

// After iteration m: beta_{m+1} (from the partial sums of |u_{m+1}|^2, or set
// already by k_lz_step when nparts is 0), s = T_{m+1}^{1/2} e_1, and the
// convergence test |s_{m+1} - s_m| <= tol |s_{m+1}| (successive iterates; V
// orthonormal), in FP64 for every Lanczos scalar type.  The first wavefront
// of a workgroup, all of whose threads call it.
template <typename A>
__device__ __forceinline__ void lz_check_body(const A *__restrict__ partials, int nparts, LzState<A> *st, int m, A tol,
                                              int max_iter, const double2 *__restrict__ nodes) {
  __shared__ double Q[kMaxIter * 64];
  if (threadIdx.x >= 64 || st->done) return;
  const int lane = threadIdx.x;
  A bb;
  if (nparts > 0) {
    // eight interleaved sums keep eight loads in flight (fixed order)
    A vs[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int i = lane;
    for (; i + 7 * 64 < nparts; i += 8 * 64) {
#pragma unroll
      for (int u = 0; u < 8; ++u) vs[u] += partials[i + u * 64];
    }
    for (; i < nparts; i += 64) vs[0] += partials[i];
    A v = ((vs[0] + vs[1]) + (vs[2] + vs[3])) + ((vs[4] + vs[5]) + (vs[6] + vs[7]));
    v = wave_sum(v);
    if (lane == 0) lz_set_beta(st, m, v);
    bb = ldexp(sqrt(v), lz_exponent(st->alpha[m]));
  } else {
    bb = st->beta[m + 1];
  }
  const int nn = m + 1;
  const double d = lane < nn ? (double)st->alpha[lane] : 0.0;
  const double e = lane < nn - 1 ? (double)st->beta[lane + 1] : 0.0;
  int ok;
  double sk;
  tridiag_root(nn, d, e, nodes, Q, false, sk, ok);
  const double sold = lane < m ? (double)st->s[lane] : 0.0;
  const double dif = lane < nn ? sk - sold : 0.0;
  double num = 0.0, den = 0.0, scale2 = 0.0;
  for (int j = 0; j < nn; ++j) {
    const double dj = lane_value(dif, j), sj = lane_value(sk, j), aj = lane_value(d, j);
    num += dj * dj;
    den += sj * sj;
    scale2 += aj * aj;
  }
  const double rel = den > 0.0 ? sqrt(num / den) : 0.0;
  const double bdn = (sizeof(A) == 8 ? 1e-11 : 1e-6) * sqrt(scale2 + (double)bb * (double)bb);
  const bool finite = isfinite(bb) && isfinite(den) && ok;
  if (lane < nn) st->s[lane] = (A)sk;
  if (lane == 0) {
    st->rel_change = m > 0 ? (A)rel : A(1);
    st->m = nn;
    const bool conv = (m > 0 && rel <= (double)tol) || ((double)bb <= bdn);
    st->converged = conv && finite;
    st->nonfinite = !finite;
    st->done = conv || !finite || nn >= max_iter;
  }
}

template <typename A>
__global__ __launch_bounds__(64) void k_lz_check(const A *__restrict__ partials, int nparts, LzState<A> *st, int m,
                                                 A tol, int max_iter, const double2 *__restrict__ nodes) {
  lz_check_body<A>(partials, nparts, st, m, tol, max_iter, nodes);
}

// The check's root alone, for pse_internal_tridiag_root: path 1 by the
// quadrature, 0 by QL, -1 if it found none.
__global__ __launch_bounds__(64) void k_tridiag_root(int n, const double *__restrict__ d, const double *__restrict__ e,
                                                     const double2 *__restrict__ nodes, bool force_ql,
                                                     double *__restrict__ s, int *__restrict__ path) {
  __shared__ double X[kMaxIter * 64];
  const int lane = threadIdx.x;
  double sk;
  int ok;
  const bool quad = tridiag_root(n, lane < n ? d[lane] : 0.0, lane < n - 1 ? e[lane] : 0.0, nodes, X, force_ql, sk, ok);
  if (lane < n) s[lane] = sk;
  if (lane == 0) *path = !ok ? -1 : (quad ? 1 : 0);
}

// Sum of nparts partial sums in a fixed order, valid in every thread of
// the workgroup.
template <typename A> __device__ A lz_parts_sum(const A *parts, int nparts, A *sh) {
  __shared__ A all;
  A v = 0;
  for (int i = threadIdx.x; i < nparts; i += blockDim.x) v += parts[i];
  v = block_sum(v, sh);
  if (threadIdx.x == 0) all = v;
  __syncthreads();
  return all;
}

// Block partial sums of |z|^2 (sorted order).
template <typename T, typename A>
__global__ __launch_bounds__(256) void k_lz_norm(const typename vec4<T>::type *__restrict__ z, int n,
                                                 A *__restrict__ partials) {
  __shared__ A sh[16];
  A v = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const auto a = z[i];
    v = dot3(v, a, a);
  }
  v = block_sum(v, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = v;
}

// Block partial sums of <u_m, t>, in iteration 0 (z2parts: the partial sums of
// |z|^2) scaled by 2^-k.  Computed here rather than in the LDS
// product's epilogue: without the reduction the product needs no register
// spills (64 VGPRs), which costs far more than this extra pass over two
// vectors.  The workgroup past the nparts partial sums, if launched, starts
// the state (m = 0, from the partial sums of |z|^2) or checks iteration m - 1.
template <typename T, typename A>
__device__ __forceinline__ void lz_alpha_block(const typename vec4<T>::type *__restrict__ t,
                                               const typename vec4<T>::type *__restrict__ u, int n, LzState<A> *st,
                                               bool test, const A *z2parts, A *__restrict__ apart, int blk,
                                               int nparts) {
  __shared__ A sh[16];
  if (test && st->done) return;
  T sc = T(1);
  if (sizeof(A) == 4 && z2parts) sc = ldexp(T(1), -lz_start_exponent(sqrt(lz_parts_sum(z2parts, nparts, sh))));
  A v = 0;
#pragma unroll 4
  for (int i = blk * blockDim.x + threadIdx.x; i < n; i += nparts * blockDim.x)
    v = dot3(v, t[i], sizeof(A) == 4 ? scaled3(u[i], sc) : u[i]);
  v = block_sum(v, sh);
  if (threadIdx.x == 0) apart[blk] = v;
}
template <typename A>
__device__ __forceinline__ void lz_side_block(const A *__restrict__ partials, int nparts, LzState<A> *st, int m, A tol,
                                              int max_iter, const double2 *__restrict__ nodes) {
  __shared__ A sh[16];
  if (m == 0) {
    const A z2 = lz_parts_sum(partials, nparts, sh);
    if (threadIdx.x == 0) lz_begin(st, z2);
  } else {
    lz_check_body<A>(partials, nparts, st, m - 1, tol, max_iter, nodes);
  }
}

template <typename T, typename A>
__global__ __launch_bounds__(256) void k_lz_alpha(const typename vec4<T>::type *__restrict__ t,
                                                  const typename vec4<T>::type *__restrict__ u, int n, LzState<A> *st,
                                                  int m, A *__restrict__ partials, int nparts, A tol, int max_iter,
                                                  const double2 *__restrict__ nodes) {
  // (beside a check, which may set `done` meanwhile, the flag is not tested:
  // the sums of a finished process are not used)
  if ((int)blockIdx.x < nparts)
    lz_alpha_block<T, A>(t, u, n, st, (int)gridDim.x == nparts, m == 0 ? partials : nullptr, partials + kRedBlock,
                         blockIdx.x, nparts);
  else
    lz_side_block<A>(partials, nparts, st, m, tol, max_iter, nodes);
}

// alpha_m from its partial sums (every workgroup; block 0 stores it),
// u_{m+1} into the next basis slot and the block partial sums of its square.
// With P (rows as (x, y, z, 0), 12 values each) also up = P^T u_{m+1}, the
// source of the next preconditioned product.
template <typename T, typename A>
__device__ __forceinline__ void lz_update_block(const typename vec4<T>::type *__restrict__ t,
                                                typename vec4<T>::type *__restrict__ V, int n, LzState<A> *st, int m,
                                                A *__restrict__ partials, int blk, int nparts,
                                                const T *__restrict__ P, typename vec4<T>::type *__restrict__ up) {
  using T4 = typename vec4<T>::type;
  __shared__ A sh[16];
  if (st->done) return;
  const A rs = st->rs[m];
  const A al = lz_parts_sum(partials + kRedBlock, nparts, sh) * rs *
               (m == 0 ? ldexp(rs, lz_start_exponent(st->beta[0])) : rs);
  if (blk == 0 && threadIdx.x == 0) st->alpha[m] = al;
  T c1, c2, c3;
  lz_coef<T, A>(st, m, al, c1, c2, c3);
  const T4 *u = V + (size_t)m * n, *uprev = m > 0 ? u - n : nullptr;
  T4 *un = V + (size_t)(m + 1) * n;
  A v = 0;
#pragma unroll 2
  for (int i = blk * blockDim.x + threadIdx.x; i < n; i += nparts * blockDim.x) {
    const T4 x = lz_next<T4, T>(t[i], u[i], uprev, i, c1, c2, c3);
    un[i] = x;
    v = dot3(v, x, x);
    if (P) {
      const T4 *pr = (const T4 *)(P + (size_t)i * 12);  // rows of P_i
      const T4 r0 = pr[0], r1 = pr[1], r2 = pr[2];
      T4 o;
      o.x = r0.x * x.x + r1.x * x.y + r2.x * x.z;
      o.y = r0.y * x.x + r1.y * x.y + r2.y * x.z;
      o.z = r0.z * x.x + r1.z * x.y + r2.z * x.z;
      o.w = T(0);
      up[i] = o;
    }
  }
  v = block_sum(v, sh);
  if (threadIdx.x == 0) partials[blk] = v;
}

template <typename T, typename A>
__global__ __launch_bounds__(256) void k_lz_update(const typename vec4<T>::type *__restrict__ t,
                                                   typename vec4<T>::type *__restrict__ V, int n, LzState<A> *st, int m,
                                                   A *__restrict__ partials, int nparts, const T *__restrict__ P,
                                                   typename vec4<T>::type *__restrict__ up) {
  lz_update_block<T, A>(t, V, n, st, m, partials, blockIdx.x, nparts, P, up);
}

// Vector work and check of iteration m in one workgroup of 1024 lanes: 64 n
// bytes (FP32 storage) through one compute unit against two or three launches
// whose time is launch and reduction latency (4 to 5 us each).  The bound
// kLzStepMax is where the two meet: 7 us at 1000 particles, 12.7 at 8000,
// against 10 to 14.
template <typename T, typename A>
__device__ __forceinline__ void lz_step_block(const typename vec4<T>::type *__restrict__ t,
                                              typename vec4<T>::type *__restrict__ V, int n, LzState<A> *st, int m,
                                              A tol, int max_iter, const double2 *__restrict__ nodes) {
  using T4 = typename vec4<T>::type;
  __shared__ A sh[16];
  __shared__ A al_s;
  __shared__ int stop, k_s;
  if (threadIdx.x == 0) stop = 0;
  if (m > 0 && st->done) return;
  const T4 *u = V + (size_t)m * n, *uprev = m > 0 ? u - n : nullptr;
  T4 *un = V + (size_t)(m + 1) * n;
  if (m == 0) {
    A z2 = 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += 1024) z2 = dot3(z2, u[i], u[i]);
    z2 = block_sum(z2, sh);
    if (threadIdx.x == 0) {
      lz_begin(st, z2);
      stop = st->done;
      k_s = lz_start_exponent(st->beta[0]);
    }
    if (sizeof(A) == 4) __syncthreads();
  }
  const int k = sizeof(A) == 4 && m == 0 ? k_s : 0;
  const T sc = ldexp(T(1), -k);
  A v = 0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) v = dot3(v, t[i], sizeof(A) == 4 ? scaled3(u[i], sc) : u[i]);
  v = block_sum(v, sh);
  if (threadIdx.x == 0) {
    const A al = v * st->rs[m] * ldexp(st->rs[m], k);
    st->alpha[m] = al;
    al_s = al;
  }
  __syncthreads();
  if (stop) return;
  T c1, c2, c3;
  lz_coef<T, A>(st, m, al_s, c1, c2, c3);
  v = 0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) {
    const T4 x = lz_next<T4, T>(t[i], u[i], uprev, i, c1, c2, c3);
    un[i] = x;
    v = dot3(v, x, x);
  }
  v = block_sum(v, sh);
  if (threadIdx.x == 0) lz_set_beta(st, m, v);
  __syncthreads();
  lz_check_body<A>(nullptr, 0, st, m, tol, max_iter, nodes);
}

template <typename T, typename A>
__global__ __launch_bounds__(1024) void k_lz_step(const typename vec4<T>::type *__restrict__ t,
                                                  typename vec4<T>::type *__restrict__ V, int n, LzState<A> *st, int m,
                                                  A tol, int max_iter, const double2 *__restrict__ nodes) {
  lz_step_block<T, A>(t, V, n, st, m, tol, max_iter, nodes);
}

// ------------------------------------------------- batched Krylov loop
// Iteration m of the Lanczos process on many systems at once (a batch of
// replicas): the same arithmetic, in the same order, as the single-system
// kernels above, so that every system's iterate is bit-identical to its own
// run.  pmap / vmap list (system, block of that system) per workgroup: the
// product's blocks of B^3 cells, and the vector kernels' blocks of 256
// particles (n <= kRedBlock 256 per system, so that each thread owns at most
// one particle, as in the single-system kernels).
__device__ __forceinline__ int lz_parts(int n) { return min(kRedBlock, (n + 255) / 256); }

template <int B, typename A, int G>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_spmv_lds_batch(
    const LzRep<A> *__restrict__ reps, const int2 *__restrict__ pmap, int m) {
  const int2 rb = pmap[blockIdx.x];
  const LzRep<A> &r = reps[rb.x];
  spmv_lds_block<B, false, G>(r.pos, r.V + (size_t)m * r.n, r.cell_start, r.nc, r.cs, r.n, r.hcap, r.L,
                                      r.nbr, r.cnt, r.tab, r.inv_dr, r.self_r, r.t, m > 0 ? &r.st->done : nullptr,
                                      r.ovf, nullptr, rb.y);
}

// M_r F of the systems whose record carries forces (the others' blocks exit)
template <int B, typename A, int G>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_spmv_lds_batch_plain(
    const LzRep<A> *__restrict__ reps, const int2 *__restrict__ pmap) {
  const int2 rb = pmap[blockIdx.x];
  const LzRep<A> &r = reps[rb.x];
  if (!r.fs) return;
  spmv_lds_block<B, false, G>(r.pos, r.fs, r.cell_start, r.nc, r.cs, r.n, r.hcap, r.L, r.nbr, r.cnt,
                                      r.tab, r.inv_dr, r.self_r, r.ur, nullptr, r.ovf, nullptr, rb.y);
}

template <typename A>
__global__ __launch_bounds__(256) void k_lz_alpha_batch(const LzRep<A> *__restrict__ reps, LzVecMaps vm, int m) {
  if ((int)blockIdx.x < vm.nv) {
    const int2 rb = vm.vmap[blockIdx.x];
    const LzRep<A> &r = reps[rb.x];
    lz_alpha_block<float, A>(r.t, r.V + (size_t)m * r.n, r.n, r.st, m > 0, m == 0 ? r.partials : nullptr,
                             r.partials + kRedBlock, rb.y, lz_parts(r.n));
  } else {
    const LzRep<A> &r = reps[vm.big[blockIdx.x - vm.nv]];
    lz_side_block<A>(r.partials, lz_parts(r.n), r.st, 0, r.tol, r.maxit, r.nodes);
  }
}

template <typename A>
__global__ __launch_bounds__(256) void k_lz_update_batch(const LzRep<A> *__restrict__ reps, LzVecMaps vm, int m) {
  const int2 rb = vm.vmap[blockIdx.x];
  const LzRep<A> &r = reps[rb.x];
  lz_update_block<float, A>(r.t, r.V, r.n, r.st, m, r.partials, rb.y, lz_parts(r.n), nullptr, nullptr);
}

// the systems of at most kLzStepMax particles
template <typename A>
__global__ __launch_bounds__(1024) void k_lz_step_batch(const LzRep<A> *__restrict__ reps, LzVecMaps vm, int m) {
  const LzRep<A> &r = reps[vm.small[blockIdx.x]];
  lz_step_block<float, A>(r.t, r.V, r.n, r.st, m, r.tol, r.maxit, r.nodes);
}

// the checks of the larger systems: one wavefront each
template <typename A>
__global__ __launch_bounds__(64) void k_lz_check_batch(const LzRep<A> *__restrict__ reps, LzVecMaps vm, int m) {
  const LzRep<A> &r = reps[vm.big[blockIdx.x]];
  lz_check_body<A>(r.partials, lz_parts(r.n), r.st, m, r.tol, r.maxit, r.nodes);
}

// y = beta_0 sum_{j < m} s_j v_j: the coefficients beta_0 s_j rs_j of the basis
// vectors into sc (all threads), and one particle of y (sorted order).
template <typename A> __device__ __forceinline__ int lz_combine_coef(const LzState<A> *st, A *sc) {
  const int m = st->m;
  if (threadIdx.x < (unsigned)m) sc[threadIdx.x] = st->beta[0] * st->s[threadIdx.x] * st->rs[threadIdx.x];
  __syncthreads();
  return m;
}
template <typename T, typename A>
__device__ __forceinline__ typename vec4<T>::type lz_combine_at(const typename vec4<T>::type *__restrict__ V, int n,
                                                                const A *sc, int m, int i) {
  A x = 0, y = 0, z = 0;
#pragma unroll 4
  for (int j = 0; j < m; ++j) {
    const auto v = V[(size_t)j * n + i];
    x += sc[j] * (A)v.x;
    y += sc[j] * (A)v.y;
    z += sc[j] * (A)v.z;
  }
  typename vec4<T>::type o;
  o.x = (T)x;
  o.y = (T)y;
  o.z = (T)z;
  o.w = T(0);
  return o;
}

template <typename T, typename A>
__global__ __launch_bounds__(256) void k_lz_combine(const typename vec4<T>::type *__restrict__ V, int n,
                                                    const LzState<A> *st, typename vec4<T>::type *__restrict__ y) {
  __shared__ A sc[kMaxIter];
  const int m = lz_combine_coef<A>(st, sc);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = lz_combine_at<T, A>(V, n, sc, m, i);
}

// ------------------------------------------------------------- vectors
// Caller-order n x 3 -> sorted (x, y, z, 0).
template <typename T>
__global__ void k_gather3(const T *__restrict__ in, const int *__restrict__ perm, typename vec4<T>::type *__restrict__ out,
                          int n) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int i = perm[s];
  typename vec4<T>::type v;
  v.x = in[3 * i];
  v.y = in[3 * i + 1];
  v.z = in[3 * i + 2];
  v.w = T(0);
  out[s] = v;
}

// Caller-order n x 3 (or none) -> sorted (x, y, z, 0), plus a sorted
// vector `add` (or none).
template <typename T>
__global__ void k_gather3_add(const T *__restrict__ in, const int *__restrict__ perm,
                              const typename vec4<T>::type *__restrict__ add, typename vec4<T>::type *__restrict__ out,
                              int n) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  typename vec4<T>::type v;
  v.x = v.y = v.z = v.w = T(0);
  if (in) {
    const int i = perm[s];
    v.x = in[3 * i];
    v.y = in[3 * i + 1];
    v.z = in[3 * i + 2];
  }
  if (add) {
    const auto a = add[s];
    v.x += a.x;
    v.y += a.y;
    v.z += a.z;
  }
  out[s] = v;
}

// x += dx over len scalars (caller order, the Euler-Maruyama update).
template <typename T> __global__ void k_advance(T *__restrict__ x, const T *__restrict__ dx, int len) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < len) x[i] += dx[i];
}

// out[perm[s]] = cr * y + dt * ur[s] + wv[s]   (y the particle's Krylov
// sample; null terms omitted; sorted inputs are (x, y, z, 0), the output is
// caller-order n x 3)
template <typename T>
__device__ __forceinline__ void finalize_at(const int *__restrict__ perm, const typename vec4<T>::type *yr, T cr,
                                            const typename vec4<T>::type *__restrict__ ur, T dt,
                                            const typename vec4<T>::type *__restrict__ wv, T *__restrict__ out, int s) {
  const int i = perm[s];
  T x = 0, y = 0, z = 0;
  if (yr) {
    x += cr * yr->x;
    y += cr * yr->y;
    z += cr * yr->z;
  }
  if (ur) {
    const auto a = ur[s];
    x += dt * a.x;
    y += dt * a.y;
    z += dt * a.z;
  }
  if (wv) {
    const auto a = wv[s];
    x += a.x;
    y += a.y;
    z += a.z;
  }
  out[3 * i] = x;
  out[3 * i + 1] = y;
  out[3 * i + 2] = z;
}

template <typename T>
__global__ __launch_bounds__(256) void k_finalize(const int *__restrict__ perm,
                                                  const typename vec4<T>::type *__restrict__ yr, T cr,
                                                  const typename vec4<T>::type *__restrict__ ur, T dt,
                                                  const typename vec4<T>::type *__restrict__ wv, T *__restrict__ out,
                                                  int n) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) finalize_at<T>(perm, yr ? yr + s : nullptr, cr, ur, dt, wv, out, s);
}

// the same with y formed here from the basis: one pass less over a vector
// than a combination of its own (write and read 32 n bytes)
template <typename T, typename A>
__global__ __launch_bounds__(256) void k_finalize_krylov(const int *__restrict__ perm,
                                                         const typename vec4<T>::type *__restrict__ V,
                                                         const LzState<A> *st, T cr,
                                                         const typename vec4<T>::type *__restrict__ ur, T dt,
                                                         const typename vec4<T>::type *__restrict__ wv,
                                                         T *__restrict__ out, int n) {
  __shared__ A sc[kMaxIter];
  const int m = lz_combine_coef<A>(st, sc);
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const auto y = lz_combine_at<T, A>(V, n, sc, m, s);
  finalize_at<T>(perm, &y, cr, ur, dt, wv, out, s);
}

// ------------------------------------------------ Philox noise for z1
template <typename T> __device__ __forceinline__ void box_muller(uint64_t wa, uint64_t wb, T &na, T &nb);
template <> __device__ __forceinline__ void box_muller<double>(uint64_t wa, uint64_t wb, double &na, double &nb) {
  const double ua = ((double)(wa >> 11) + 0.5) * 0x1.0p-53;
  const double ub = ((double)(wb >> 11) + 0.5) * 0x1.0p-53;
  const double rho = sqrt(-2.0 * log(ua));
  double sn, cs;
  sincospi(2.0 * ub, &sn, &cs);
  na = rho * cs;
  nb = rho * sn;
}
template <> __device__ __forceinline__ void box_muller<float>(uint64_t wa, uint64_t wb, float &na, float &nb) {
  const float ua = ((float)(uint32_t)(wa >> 40) + 0.5f) * 0x1.0p-24f;
  const float ub = ((float)(uint32_t)(wb >> 40) + 0.5f) * 0x1.0p-24f;
  const float rho = sqrtf(-2.0f * logf(ua));
  float sn, cs;
  sincospif(2.0f * ub, &sn, &cs);
  na = rho * cs;
  nb = rho * sn;
}

// z1 is defined in caller order: Philox block b (key (seed, 0), counter
// (b, sample)) gives elements 4b .. 4b+3 of the 3n vector.  It is written
// straight into sorted order: sorted particle s (caller index i = perm[s])
// takes elements 3i .. 3i+2, i.e. the normals of block (3i) >> 2 and, when
// they straddle, of the next.
template <typename T>
__device__ __forceinline__ void real_noise_at(const int *__restrict__ perm, int n, uint64_t seed, uint64_t sample,
                                              typename vec4<T>::type *__restrict__ z, const uint64_t *__restrict__ rng,
                                              int s) {
  if (s >= n) return;
  if (rng) {
    // key and counter from device memory (a graph replayed per step)
    seed = rng[0];
    sample = rng[1];
  }
  const uint64_t e0 = 3ull * (uint64_t)perm[s];
  const uint64_t b0 = e0 >> 2;
  const int off = (int)(e0 & 3);
  T v[8];
  {
    uint64_t c[4] = {b0, sample, 0ull, 0ull};
    philox4x64_10(c, seed, 0ull);
    box_muller<T>(c[0], c[1], v[0], v[1]);
    box_muller<T>(c[2], c[3], v[2], v[3]);
  }
  if (off >= 2) {
    uint64_t c[4] = {b0 + 1, sample, 0ull, 0ull};
    philox4x64_10(c, seed, 0ull);
    box_muller<T>(c[0], c[1], v[4], v[5]);
    box_muller<T>(c[2], c[3], v[6], v[7]);
  }
  typename vec4<T>::type o;
  o.x = off == 0 ? v[0] : (off == 1 ? v[1] : (off == 2 ? v[2] : v[3]));
  o.y = off == 0 ? v[1] : (off == 1 ? v[2] : (off == 2 ? v[3] : v[4]));
  o.z = off == 0 ? v[2] : (off == 1 ? v[3] : (off == 2 ? v[4] : v[5]));
  o.w = T(0);
  z[s] = o;
}

template <typename T>
__global__ void k_real_noise_sorted(const int *__restrict__ perm, int n, uint64_t seed, uint64_t sample,
                                    typename vec4<T>::type *__restrict__ z, const uint64_t *__restrict__ rng) {
  real_noise_at<T>(perm, n, seed, sample, z, rng, blockIdx.x * blockDim.x + threadIdx.x);
}

// ----------------------------------------------------------- launchers
static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

__global__ void k_zero_words(uint32_t *__restrict__ p, size_t nw) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nw; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

void launch_zero_words(hipStream_t s, void *p, size_t nwords) {
  if (!nwords) return;
  const size_t b = (nwords + 255) / 256;
  k_zero_words<<<(int)(b < 4096 ? b : 4096), 256, 0, s>>>((uint32_t *)p, nwords);
}

// a[0 .. na) = 0 and b[0 .. nb) = 0.
__global__ void k_zero_i32(int *__restrict__ a, int na, int *__restrict__ b, int nb) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < na) a[i] = 0;
  else if (i - na < nb) b[i - na] = 0;
}

template <typename T>
void launch_bin(pse_ctx *c, const void *pos) {
  using T4 = typename vec4<T>::type;
  const int n = c->n;
  const T L = (T)c->d.L, invL = (T)(1.0 / c->d.L), inv_cs = (T)(1.0 / c->d.cs);
  ProfScope ps(c, PSE_STAGE_BIN);
  // a fill kernel rather than a memset: the same code runs under graph capture
  k_zero_i32<<<nblk(c->ncell + 8, 256), 256, 0, c->stream>>>(c->cell_count, c->ncell, c->flags, 8);
  // cell_of holds the cells [0, n) and the slots [n, 2n); cell_count the
  // counts [0, ncell) and the tile sums of the scan after them
  k_wrap_bin<T><<<nblk(n, 256), 256, 0, c->stream>>>((const T *)pos, n, L, invL, inv_cs, c->d.nc, (T4 *)c->pos_w,
                                                     c->cell_of, c->cell_of + n, c->cell_count, c->flags);
  const int ntiles = nblk(c->ncell, kScanTile);
  k_scan_tiles<<<ntiles, kScanNT, 0, c->stream>>>(c->cell_count, c->ncell, c->cell_count + c->ncell);
  k_scan_apply<<<ntiles, kScanNT, 0, c->stream>>>(c->cell_count, c->cell_count + c->ncell, c->ncell, c->cell_start);
  k_scatter<<<nblk(n, 256), 256, 0, c->stream>>>(c->cell_of, c->cell_of + n, c->cell_start, c->perm, n);
  k_cell_sort<T4><<<nblk(c->ncell, 4), 256, 0, c->stream>>>(c->cell_start, c->perm, c->ncell, (const T4 *)c->pos_w,
                                                           (T4 *)c->pos_s);
}

static FGExact fg_exact(const pse_ctx *c) { return FGExact{c->series, c->p.xi, c->p.a, c->d.mu0, c->small_r2}; }
// workgroups of 256 lanes, kRowLanes per row, at most 8 per compute unit
static int row_blocks(int n) { return std::min(nblk(n, 256 / kRowLanes), 2048); }

template <typename T>
void launch_nbr(pse_ctx *c) {
  using T4 = typename vec4<T>::type;
  const int n = c->n;
  const T L = (T)c->d.L, invL = (T)(1.0 / c->d.L), inv_cs = (T)(1.0 / c->d.cs);
  const T rc2 = (T)(c->p.rcut * c->p.rcut);
  ProfScope ps(c, PSE_STAGE_NBR);
  const T inv_mu0 = (T)(1.0 / c->d.mu0), fself = (T)(c->d.self_r / c->d.mu0), a = (T)c->p.a;
  const bool rep = c->rep_k > 0;
  if (c->pc_on) {
    auto go = [&](auto kern, auto fg) {
      kern<<<nblk(n, 128), 128, 0, c->stream>>>((const T4 *)c->pos_s, c->cell_start, n, c->d.nc, L, invL, inv_cs, rc2,
                                                c->nbr, c->nbr_cnt, c->nbr_cap, c->flags, fg, inv_mu0, fself, a,
                                                c->pc_feat, (T)c->rep_k, (T4 *)c->vbuf[kRepBuf]);
    };
    auto both = [&](auto fg) {
      using FG = decltype(fg);
      rep ? go(k_nbr_feat<T, FG, true>, fg) : go(k_nbr_feat<T, FG, false>, fg);
    };
    if constexpr (sizeof(T) == 8) both(fg_exact(c));
    else both(FGTable{c->table, (float)(kTableK / c->p.rcut)});
  } else {
    auto go = [&](auto kern) {
      kern<<<row_blocks(n), 256, 0, c->stream>>>((const T4 *)c->pos_s, c->cell_start, n, c->d.nc, L, invL, inv_cs, rc2,
                                                 c->nbr, c->nbr_cnt, c->nbr_cap, c->flags, a, (T)c->rep_k,
                                                 (T4 *)c->vbuf[kRepBuf]);
    };
    rep ? go(k_nbr_rows<T, true>) : go(k_nbr_rows<T, false>);
  }
  if constexpr (sizeof(T) == 8) {
    // small systems: rows split so that the evaluations fill the GPU
    if (c->nbr_coef)
      k_pair_coef<<<dim3(nblk(n, 256 / kRowLanes), n < 32768 ? 8 : 1), 256, 0, c->stream>>>(
          (const double4 *)c->pos_s, c->nbr, c->nbr_cnt, n, c->nbr_cap, L, invL, fg_exact(c), c->d.self_r, c->nbr_coef);
  }
}

static int lds_nblocks(int nc, int B) {
  const int nb = (nc + B - 1) / B;
  return nb * nb * nb;
}

// f(std::integral_constant<int, B>) for the block edge B = 1 ... 4.
template <typename F> static void with_block_edge(int B, F f) {
  switch (B) {
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    default: f(std::integral_constant<int, 1>{}); break;
  }
}

void launch_halo_size(pse_ctx *c, int B) {
  ProfScope ps(c, PSE_STAGE_NBR);
  const int nblocks = lds_nblocks(c->d.nc, B);
  with_block_edge(B, [&](auto b) {
    constexpr int BE = decltype(b)::value;
    k_halo_size<BE><<<std::min(kHaloWG, nblk(64L * nblocks, kHaloNT)), kHaloNT, 0, c->stream>>>(c->cell_start, c->d.nc,
                                                                                             c->flags);
  });
}

// Dynamic LDS above 64 KB needs a per-kernel attribute.  It is set once per
// kernel, to everything the CU's LDS leaves beside the kernel's static LDS,
// so that launches from several host threads (batches) with different halo
// sizes never lower it under one another.
template <typename K> static void allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return;
  static std::mutex mu;
  static std::unordered_set<const void *> done;
  const void *k = reinterpret_cast<const void *>(kernel);
  std::lock_guard<std::mutex> lock(mu);
  if (!done.insert(k).second) return;
  hipFuncAttributes fa{};
  const size_t stat = hipFuncGetAttributes(&fa, k) == hipSuccess ? fa.sharedSizeBytes : 32 * 1024;
  (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsPerCU - stat));
}

size_t nbr_lds_bytes(int hcap) { return 4 * sizeof(float) * (size_t)(hcap + kNbrPad); }

void launch_nbr_lds(pse_ctx *c) {
  ProfScope ps(c, PSE_STAGE_NBR);
  const size_t smem = nbr_lds_bytes(c->hcap);
  const float L = (float)c->d.L, rc2 = (float)(c->p.rcut * c->p.rcut);
  // small systems: a block's tiles shared by up to 8 workgroups, about two
  // for each of the 256 compute units
  const int parts = std::min(8, std::max(1, 512 / c->lds_blocks));
  auto *nb = (uint16_t *)c->nbr;
  auto go = [&](auto kern) {
    allow_lds(kern, smem);
    kern<<<c->lds_blocks * parts, kNbrNT, smem, c->stream>>>(
        (const float4 *)c->pos_s, c->cell_start, c->d.nc, (float)c->d.cs, c->n, L, (float)c->p.rcut, rc2, nb, c->nbr_cnt,
        c->nbr_cap, c->flags, (float)(2.0 * c->p.a), (float)c->rep_k, (float4 *)c->vbuf[kRepBuf], c->hcap, parts);
  };
  with_block_edge(c->lds_B, [&](auto b) {
    constexpr int BE = decltype(b)::value;
    if (!(c->rep_k > 0)) go(k_nbr_lds<BE, kRepNone>);
    else if (c->p.rcut >= 2.0 * c->p.a) go(k_nbr_lds<BE, kRepHits>);
    else go(k_nbr_lds<BE, kRepAll>);
  });
}

void launch_nbr_batch(hipStream_t s, const NbrRep *reps, const NbrGroup *groups, int ngroups) {
  for (int g = 0; g < ngroups; ++g) {
    const NbrGroup &gr = groups[g];
    with_block_edge(gr.B, [&](auto b) {
      constexpr int BE = decltype(b)::value;
      allow_lds(k_nbr_lds_batch<BE>, gr.smem);
      k_nbr_lds_batch<BE><<<gr.nblk, kNbrNT, gr.smem, s>>>(reps, gr.pmap);
    });
  }
}

// Preconditioner features on the LDS path, from the list and the staged halo.
void launch_feat_lds(pse_ctx *c) {
  ProfScope ps(c, PSE_STAGE_PRECOND);
  const size_t smem = sizeof(float4) * (size_t)c->hcap;
  const float L = (float)c->d.L;
  const float inv_mu0 = (float)(1.0 / c->d.mu0), fself = (float)(c->d.self_r / c->d.mu0);
  const float near2 = (float)(20.25 * c->p.a * c->p.a);  // r < 4.5a
  with_block_edge(c->lds_B, [&](auto b) {
    constexpr int BE = decltype(b)::value;
    allow_lds(k_feat_lds<BE>, smem);
    k_feat_lds<BE><<<c->lds_blocks, kFeatNT, smem, c->stream>>>(
        (const float4 *)c->pos_s, c->cell_start, c->d.nc, (float)c->d.cs, c->n, L, (const uint16_t *)c->nbr, c->nbr_cnt,
        (const float2 *)c->table, (float)(kTableK / c->p.rcut), inv_mu0, fself, (float)c->p.a, near2, c->pc_feat,
        c->hcap, c->flags + 7);
  });
}

template <bool PC = false>
static void spmv_lds(pse_ctx *c, const float4 *src, float4 *out, const int *done = nullptr) {
  const size_t smem = (sizeof(float4) + sizeof(float2)) * (size_t)c->hcap;
  const float L = (float)c->d.L;
  const auto *nb = (const uint16_t *)c->nbr;
  const float inv_dr = (float)(kTableK / c->p.rcut), self_r = (float)c->d.self_r;
  auto go = [&](auto kernel) {
    allow_lds(kernel, smem);
    kernel<<<c->lds_blocks, 1024, smem, c->stream>>>((const float4 *)c->pos_s, src, c->cell_start, c->d.nc,
                                                      (float)c->d.cs, c->n, c->hcap, L, nb, c->nbr_cnt,
                                                      c->table, inv_dr, self_r, out, done, c->flags + 7,
                                                      (const float4 *)c->pc_P);
  };
  auto pick = [&](auto g) {
    constexpr int G = decltype(g)::value;
    with_block_edge(c->lds_B, [&](auto b) {
      go(k_spmv_lds<decltype(b)::value, PC, G>);
    });
  };
  // lanes per target: 3 built in (the best measured at phi = 0.3 with
  // r_c = 8a), 2 or 4 when pse_autotune found them faster
  if (c->tune_spmv_lanes == 2) pick(std::integral_constant<int, 2>{});
  else if (c->tune_spmv_lanes == 4) pick(std::integral_constant<int, 4>{});
  else pick(std::integral_constant<int, 3>{});
}

// The product is timed on the sorted positions as its source (finite) into
// vbuf[5], scratch that every sample rewrites.
static pse_status autotune_spmv_impl(pse_ctx *c) {
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return PSE_ERR_HIP;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return PSE_ERR_HIP;
  }
  const int keep = c->tune_spmv_lanes;
  int best = 0;
  float tbest = 1e30f, t3 = 1e30f;
  for (int g : {3, 2, 4}) {
    c->tune_spmv_lanes = g;
    auto launch = [&] { spmv_lds(c, (const float4 *)c->pos_s, (float4 *)c->vbuf[5]); };
    launch();  // warm-up
    float t = 1e30f;
    for (int rep = 0; rep < 3; ++rep) {
      float ms = 1e30f;
      if (hipEventRecord(e0, c->stream) != hipSuccess) break;
      launch();
      if (hipEventRecord(e1, c->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
          hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
        break;
      t = ms < t ? ms : t;
    }
    if (g == 3) t3 = t;
    // another lane count replaces the built-in 3 only when it is faster by
    // more than the timing noise (3 %), so that the choice is stable
    if (g == 3 ? t < tbest : t < tbest && t < 0.97f * t3) {
      tbest = t;
      best = g;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  const pse_status st_ = hipGetLastError() == hipSuccess ? PSE_OK : PSE_ERR_HIP;
  c->tune_spmv_lanes = st_ == PSE_OK && best ? best : keep;
  return st_;
}

pse_status autotune_spmv(pse_ctx *c, int32_t *lanes) {
  if (lanes) *lanes = 0;
  if (c->dbl || !c->lds_B) return PSE_OK;
  const uint32_t mask = c->prof_mask;
  c->prof_mask = 0;  // the trial launches are not stage time
  const pse_status st = autotune_spmv_impl(c);
  c->prof_mask = mask;
  if (lanes) *lanes = c->tune_spmv_lanes ? c->tune_spmv_lanes : 3;
  return st;
}

template <typename T> static void spmv(pse_ctx *c, const void *src, void *out, const int *done) {
  const int n = c->n, nb = row_blocks(n), cap = c->nbr_cap;
  ProfScope ps(c, PSE_STAGE_SPMV);
  if constexpr (sizeof(T) == 8) {
    const double L = c->d.L, invL = 1.0 / L, self_r = c->d.self_r;
    if (c->nbr_coef)
      k_spmv_coef<<<nb, 256, 0, c->stream>>>((const double4 *)c->pos_s, c->nbr, c->nbr_cnt, n, cap, L, invL,
                                             c->nbr_coef, self_r, (const double4 *)src, (double4 *)out, done);
    else
      k_spmv_exact<<<nb, 256, 0, c->stream>>>((const double4 *)c->pos_s, c->nbr, c->nbr_cnt, n, cap, L, invL,
                                              fg_exact(c), self_r, (const double4 *)src, (double4 *)out, done);
  } else if (c->lds_B) {
    spmv_lds(c, (const float4 *)src, (float4 *)out, done);
  } else {
    k_spmv_table<<<nb, 256, 0, c->stream>>>((const float4 *)c->pos_s, c->nbr, c->nbr_cnt, n, cap, (float)c->d.L,
                                            (float)(1.0 / c->d.L), c->table, (float)(kTableK / c->p.rcut),
                                            (float)c->d.self_r, (const float4 *)src, (float4 *)out, done);
  }
}
template <typename T> void launch_spmv(pse_ctx *c, const void *src, void *out) { spmv<T>(c, src, out, nullptr); }

// Iteration m; with `check` that of iteration m - 1 goes with it (the systems
// above kLzStepMax and the preconditioned ones; k_lz_step holds its own).
template <typename T, typename A> static void lz_iter(pse_ctx *c, int m, bool pc, bool check) {
  using T4 = typename vec4<T>::type;
  const int n = c->n, nparts = std::min(kRedBlock, nblk(n, 256));
  T4 *V = (T4 *)c->V, *t = (T4 *)c->vbuf[2];
  auto *st = (LzState<A> *)c->lz;
  const A tol = (A)c->p.lanczos_tol;
  const int *done = m > 0 ? &st->done : nullptr;
  if (pc) {
    // t = P M_r P^T u_m; P^T u_m comes from the previous update (m > 0)
    T4 *up = (T4 *)c->vbuf[8], *tp = (T4 *)c->vbuf[9];
    if (m == 0) {
      ProfScope ps(c, PSE_STAGE_PRECOND);
      launch_pc_pre<T>(c, V, up);
    }
    bool fused = false;
    if constexpr (sizeof(T) == 4) {
      if (c->lds_B) {
        ProfScope ps(c, PSE_STAGE_SPMV);
        spmv_lds<true>(c, (const float4 *)up, (float4 *)t, done);
        fused = true;
      }
    }
    if (!fused) {
      spmv<T>(c, up, tp, done);
      ProfScope ps(c, PSE_STAGE_PRECOND);
      launch_pc_post<T>(c, tp, t);
    }
  } else {
    spmv<T>(c, V + (size_t)m * n, t, done);
  }
  ProfScope ps(c, PSE_STAGE_LANCZOS);
  A *part = (A *)c->partials;
  if (!pc && n <= kLzStepMax) {
    k_lz_step<T, A><<<1, 1024, 0, c->stream>>>(t, V, n, st, m, tol, c->lz_maxit, c->lz_nodes);
    return;
  }
  k_lz_alpha<T, A><<<nparts + (m == 0 || check ? 1 : 0), 256, 0, c->stream>>>(t, V + (size_t)m * n, n, st, m, part,
                                                                             nparts, tol, c->lz_maxit, c->lz_nodes);
  k_lz_update<T, A><<<nparts, 256, 0, c->stream>>>(t, V, n, st, m, part, nparts, pc ? (const T *)c->pc_P : nullptr,
                                                   pc ? (T4 *)c->vbuf[8] : nullptr);
}

template <typename T, typename A> void launch_lz_norm(pse_ctx *c, bool pc) {
  if (!pc && c->n <= kLzStepMax) return;
  ProfScope ps(c, PSE_STAGE_LANCZOS);
  k_lz_norm<T, A><<<std::min(kRedBlock, nblk(c->n, 256)), 256, 0, c->stream>>>((const typename vec4<T>::type *)c->V,
                                                                              c->n, (A *)c->partials);
}

template <typename T, typename A> void launch_lz_iters(pse_ctx *c, int m0, int k, bool pc) {
  const int nparts = std::min(kRedBlock, nblk(c->n, 256));
  const bool step = !pc && c->n <= kLzStepMax;
  if (m0 == 0) launch_lz_norm<T, A>(c, pc);
  for (int m = m0; m < m0 + k; ++m) {
    lz_iter<T, A>(c, m, pc, m > m0 && !c->graph);
    if (step || (!c->graph && m + 1 < m0 + k)) continue;
    ProfScope ps(c, PSE_STAGE_LANCZOS);
    k_lz_check<A><<<1, 64, 0, c->stream>>>((const A *)c->partials, nparts, (LzState<A> *)c->lz, m,
                                           (A)c->p.lanczos_tol, c->lz_maxit, c->lz_nodes);
  }
}

// The batched Krylov loop: per iteration the product of every group of
// systems sharing a block edge and lanes per target, then the
// vector work and the checks of all systems.
template <typename A>
void launch_lz_batch(hipStream_t s, const LzRep<A> *reps, const LzGroup *groups, int ngroups,
                     const LzVecMaps &vm, int iters) {
  for (int m = 0; m < iters; ++m) {
    for (int g = 0; g < ngroups; ++g) {
      const LzGroup &gr = groups[g];
      with_block_edge(gr.B, [&](auto b) {
        constexpr int BE = decltype(b)::value;
        auto go = [&](auto kernel) {
          allow_lds(kernel, gr.smem);
          kernel<<<gr.nblk, 1024, gr.smem, s>>>(reps, gr.pmap, m);
        };
        auto pick = [&](auto gl) {
          constexpr int GL = decltype(gl)::value;
          go(k_spmv_lds_batch<BE, A, GL>);
        };
        if (gr.G == 2) pick(std::integral_constant<int, 2>{});
        else if (gr.G == 4) pick(std::integral_constant<int, 4>{});
        else pick(std::integral_constant<int, 3>{});
      });
    }
    if (vm.nsmall) k_lz_step_batch<A><<<vm.nsmall, 1024, 0, s>>>(reps, vm, m);
    if (vm.nbig) {
      k_lz_alpha_batch<A><<<vm.nv + (m == 0 ? vm.nbig : 0), 256, 0, s>>>(reps, vm, m);
      k_lz_update_batch<A><<<vm.nv, 256, 0, s>>>(reps, vm, m);
      k_lz_check_batch<A><<<vm.nbig, 64, 0, s>>>(reps, vm, m);
    }
  }
}
__global__ void k_batch_status(const RepStatusSrc *__restrict__ src, int nrep, RepStatus *__restrict__ out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrep) return;
  const RepStatusSrc q = src[r];
  RepStatus o;
  for (int k = 0; k < 8; ++k) o.flags[k] = q.flags[k];
  if (q.acc_dbl) {
    const auto *st = (const LzState<double> *)q.lz;
    o.m = st->m;
    o.done = st->done;
    o.converged = st->converged;
    o.nonfinite = st->nonfinite;
    o.rel_change = st->rel_change;
  } else {
    const auto *st = (const LzState<float> *)q.lz;
    o.m = st->m;
    o.done = st->done;
    o.converged = st->converged;
    o.nonfinite = st->nonfinite;
    o.rel_change = (double)st->rel_change;
  }
  out[r] = o;
}

void launch_batch_status(hipStream_t s, const RepStatusSrc *src, int nrep, RepStatus *out) {
  k_batch_status<<<(nrep + 63) / 64, 64, 0, s>>>(src, nrep, out);
}

// ------------------------------------------ fully batched systems
// The per-system kernels of a captured step (binning, noise, Krylov start,
// combination, final sum) for many systems in one launch each: the same
// bodies as the single-system kernels, the system and block from a map.
__global__ __launch_bounds__(256) void k_zero_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  const int i = rb.y * 256 + (int)threadIdx.x;
  if (i < r.ncell) r.cell_count[i] = 0;
  else if (i - r.ncell < 8) r.flags[i - r.ncell] = 0;
}
__global__ __launch_bounds__(256) void k_wrap_bin_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  wrap_bin_at<float>(r.pos_in, r.n, r.L, r.invL, r.inv_cs, r.nc, r.pos_w, r.cell_of, r.slot, r.cell_count, r.flags,
                     rb.y * 256 + (int)threadIdx.x);
}
__global__ __launch_bounds__(kScanNT) void k_scan_tiles_batch(const SampRep *__restrict__ reps,
                                                              const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  scan_tiles_at(r.cell_count, r.ncell, r.tile_sum, rb.y);
}
__global__ __launch_bounds__(kScanNT) void k_scan_apply_batch(const SampRep *__restrict__ reps,
                                                              const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  scan_apply_at(r.cell_count, r.tile_sum, r.ncell, r.cell_start, rb.y);
}
__global__ __launch_bounds__(256) void k_scatter_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  const int i = rb.y * 256 + (int)threadIdx.x;
  if (i < r.n) r.perm[r.cell_start[r.cell_of[i]] + r.slot[i]] = i;
}
__global__ __launch_bounds__(256) void k_cell_sort_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  cell_sort_at<float4>(r.cell_start, r.perm, r.ncell, r.pos_w, r.pos_s, rb.y * 4 + (int)(threadIdx.x >> 6));
}
__global__ __launch_bounds__(256) void k_noise_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  real_noise_at<float>(r.perm, r.n, 0ull, 0ull, r.V, r.rng, rb.y * 256 + (int)threadIdx.x);
}
// partial sums of |z|^2 (the systems whose vector work is one workgroup sum
// it themselves)
template <typename A>
__global__ __launch_bounds__(256) void k_lz_norm_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  __shared__ A sh[16];
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  if (r.n <= kLzStepMax) return;
  const int i = rb.y * 256 + (int)threadIdx.x;
  A v = 0;
  if (i < r.n) {
    const float4 a = r.V[i];
    v = dot3(v, a, a);
  }
  v = block_sum(v, sh);
  if (threadIdx.x == 0) ((A *)r.partials)[rb.y] = v;
}
template <typename A>
__global__ __launch_bounds__(256) void k_finalize_batch(const SampRep *__restrict__ reps, const int2 *__restrict__ map) {
  __shared__ A sc[kMaxIter];
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  const int m = lz_combine_coef<A>((const LzState<A> *)r.st, sc);
  const int s = rb.y * 256 + (int)threadIdx.x;
  if (s >= r.n) return;
  const float4 y = lz_combine_at<float, A>(r.V, r.n, sc, m, s);
  finalize_at<float>(r.perm, &y, r.cr, r.f_in ? r.ur : nullptr, r.dt, r.wave, r.out, s);
}
__global__ __launch_bounds__(256) void k_gather_forces_batch(const SampRep *__restrict__ reps,
                                                             const int2 *__restrict__ map) {
  const int2 rb = map[blockIdx.x];
  const SampRep &r = reps[rb.x];
  const int s = rb.y * 256 + (int)threadIdx.x;
  if (!r.f_in || s >= r.n) return;
  const int i = r.perm[s];
  float4 v;
  v.x = r.f_in[3 * i];
  v.y = r.f_in[3 * i + 1];
  v.z = r.f_in[3 * i + 2];
  v.w = 0.0f;
  r.f_s[s] = v;
}

void launch_samp_batch_bin(hipStream_t s, const SampRep *reps, const SampMaps &m) {
  k_zero_batch<<<m.nzero, 256, 0, s>>>(reps, m.zero);
  k_wrap_bin_batch<<<m.npart, 256, 0, s>>>(reps, m.part);
  k_scan_tiles_batch<<<m.ntile, kScanNT, 0, s>>>(reps, m.tile);
  k_scan_apply_batch<<<m.ntile, kScanNT, 0, s>>>(reps, m.tile);
  k_scatter_batch<<<m.npart, 256, 0, s>>>(reps, m.part);
  k_cell_sort_batch<<<m.ncell, 256, 0, s>>>(reps, m.cell);
}
void launch_samp_batch_forces(hipStream_t s, const SampRep *reps, const SampMaps &m) {
  k_gather_forces_batch<<<m.npart, 256, 0, s>>>(reps, m.part);
}
template <typename A> void launch_samp_batch_start(hipStream_t s, const SampRep *reps, const SampMaps &m) {
  k_noise_batch<<<m.npart, 256, 0, s>>>(reps, m.part);
  k_lz_norm_batch<A><<<m.npart, 256, 0, s>>>(reps, m.part);
}
template <typename A> void launch_samp_batch_end(hipStream_t s, const SampRep *reps, const SampMaps &m) {
  k_finalize_batch<A><<<m.npart, 256, 0, s>>>(reps, m.part);
}
template void launch_samp_batch_start<float>(hipStream_t, const SampRep *, const SampMaps &);
template void launch_samp_batch_start<double>(hipStream_t, const SampRep *, const SampMaps &);
template void launch_samp_batch_end<float>(hipStream_t, const SampRep *, const SampMaps &);
template void launch_samp_batch_end<double>(hipStream_t, const SampRep *, const SampMaps &);

template <typename A>
void launch_lz_batch_plain(hipStream_t s, const LzRep<A> *reps, const LzGroup *groups, int ngroups) {
  for (int g = 0; g < ngroups; ++g) {
    const LzGroup &gr = groups[g];
    with_block_edge(gr.B, [&](auto b) {
      constexpr int BE = decltype(b)::value;
      auto go = [&](auto kernel) {
        allow_lds(kernel, gr.smem);
        kernel<<<gr.nblk, 1024, gr.smem, s>>>(reps, gr.pmap);
      };
      auto pick = [&](auto gl) {
        constexpr int GL = decltype(gl)::value;
        go(k_spmv_lds_batch_plain<BE, A, GL>);
      };
      if (gr.G == 2) pick(std::integral_constant<int, 2>{});
      else if (gr.G == 4) pick(std::integral_constant<int, 4>{});
      else pick(std::integral_constant<int, 3>{});
    });
  }
}
template void launch_lz_batch_plain<float>(hipStream_t, const LzRep<float> *, const LzGroup *, int);
template void launch_lz_batch_plain<double>(hipStream_t, const LzRep<double> *, const LzGroup *, int);

template void launch_lz_batch<float>(hipStream_t, const LzRep<float> *, const LzGroup *, int, const LzVecMaps &, int);
template void launch_lz_batch<double>(hipStream_t, const LzRep<double> *, const LzGroup *, int, const LzVecMaps &,
                                      int);

template <typename T, typename A>
void launch_lz_combine(pse_ctx *c, void *y) {
  using T4 = typename vec4<T>::type;
  ProfScope ps(c, PSE_STAGE_LANCZOS);
  k_lz_combine<T, A><<<nblk(c->n, 256), 256, 0, c->stream>>>((const T4 *)c->V, c->n, (const LzState<A> *)c->lz, (T4 *)y);
}

template <typename T>
void launch_gather3(pse_ctx *c, const void *in, void *out) {
  ProfScope ps(c, PSE_STAGE_OTHER);
  k_gather3<T><<<nblk(c->n, 256), 256, 0, c->stream>>>((const T *)in, c->perm, (typename vec4<T>::type *)out, c->n);
}

template <typename T> void launch_gather3_add(pse_ctx *c, const void *in, const void *add, void *out) {
  ProfScope ps(c, PSE_STAGE_OTHER);
  using T4 = typename vec4<T>::type;
  k_gather3_add<T><<<nblk(c->n, 256), 256, 0, c->stream>>>((const T *)in, c->perm, (const T4 *)add, (T4 *)out, c->n);
}

template <typename T> void launch_advance(pse_ctx *c, void *x, const void *dx) {
  ProfScope ps(c, PSE_STAGE_OTHER);
  k_advance<T><<<nblk(3 * (long)c->n, 256), 256, 0, c->stream>>>((T *)x, (const T *)dx, 3 * c->n);
}

template <typename T>
void launch_finalize(pse_ctx *c, const void *yr, double cr, const void *ur, double dt, const void *wv, void *out) {
  using T4 = typename vec4<T>::type;
  ProfScope ps(c, PSE_STAGE_OTHER);
  k_finalize<T><<<nblk(c->n, 256), 256, 0, c->stream>>>(c->perm, (const T4 *)yr, (T)cr, (const T4 *)ur, (T)dt,
                                                        (const T4 *)wv, (T *)out, c->n);
}

template <typename T, typename A>
void launch_finalize_krylov(pse_ctx *c, double cr, const void *ur, double dt, const void *wv, void *out) {
  using T4 = typename vec4<T>::type;
  ProfScope ps(c, PSE_STAGE_OTHER);
  k_finalize_krylov<T, A><<<nblk(c->n, 256), 256, 0, c->stream>>>(c->perm, (const T4 *)c->V, (const LzState<A> *)c->lz,
                                                                  (T)cr, (const T4 *)ur, (T)dt, (const T4 *)wv,
                                                                  (T *)out, c->n);
}

template <typename T>
void launch_real_noise(pse_ctx *c, void *z_sorted, uint64_t seed, uint64_t sample) {
  ProfScope ps(c, PSE_STAGE_NOISE);
  k_real_noise_sorted<T><<<nblk(c->n, 256), 256, 0, c->stream>>>(c->perm, c->n, seed, sample,
                                                                  (typename vec4<T>::type *)z_sorted, c->rng_dev);
}

#define INST_T(T)                                                                                  \
  template void launch_bin<T>(pse_ctx *, const void *);                                            \
  template void launch_nbr<T>(pse_ctx *);                                                          \
  template void launch_spmv<T>(pse_ctx *, const void *, void *);                                   \
  template void launch_gather3<T>(pse_ctx *, const void *, void *);                                \
  template void launch_gather3_add<T>(pse_ctx *, const void *, const void *, void *);              \
  template void launch_advance<T>(pse_ctx *, void *, const void *);                                \
  template void launch_finalize<T>(pse_ctx *, const void *, double, const void *, double, const void *, void *); \
  template void launch_real_noise<T>(pse_ctx *, void *, uint64_t, uint64_t);
INST_T(float)
INST_T(double)
#define INST_TA(T, A)                                                           \
  template void launch_lz_norm<T, A>(pse_ctx *, bool);                          \
  template void launch_lz_iters<T, A>(pse_ctx *, int, int, bool);                \
  template void launch_lz_combine<T, A>(pse_ctx *, void *);                     \
  template void launch_finalize_krylov<T, A>(pse_ctx *, double, const void *, double, const void *, void *);
INST_TA(float, float)
INST_TA(float, double)
INST_TA(double, double)

}  // namespace pse

// The square root of the Krylov check on a given matrix (host arrays d[n],
// e[n - 1], s[n]; no part of the API): 1 by the quadrature, 0 by QL, -1 not
// found, -2 invalid n or no device.
extern "C" int pse_internal_tridiag_root(int force_ql, int n, const double *d, const double *e, double *s) {
  using namespace pse;
  if (n < 1 || n > kMaxIter) return -2;
  struct Bufs {
    double2 nodes[kRootNodes];
    double d[kMaxIter], e[kMaxIter], s[kMaxIter];
    int path;
  } h{}, *dev = nullptr;
  lz_quadrature(h.nodes);
  for (int i = 0; i < n; ++i) h.d[i] = d[i];
  for (int i = 0; i + 1 < n; ++i) h.e[i] = e[i];
  if (hipMalloc((void **)&dev, sizeof h) != hipSuccess) return -2;
  int path = -2;
  if (hipMemcpy(dev, &h, sizeof h, hipMemcpyHostToDevice) == hipSuccess) {
    k_tridiag_root<<<1, 64>>>(n, dev->d, dev->e, dev->nodes, force_ql != 0, dev->s, &dev->path);
    if (hipMemcpy(&h, dev, sizeof h, hipMemcpyDeviceToHost) == hipSuccess) {
      path = h.path;
      for (int i = 0; i < n; ++i) s[i] = h.s[i];
    }
  }
  (void)hipFree(dev);
  return path;
}
