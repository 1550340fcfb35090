// Auxiliary kernels around the solver:
//  * preparation step (paper Sec. 4.2): periodic ghost fill of patch groups
//    from a resident box, and trilinear fill of AMR-shaped groups from a
//    coarse field (spatial interpolation at coarse-fine boundaries);
//  * FP64 CFL time step, dt = cfl * dh / max (max is order-free, so the result
//    is deterministic and equals a serial evaluation bit for bit), and FP64
//    conserved sums with a fixed reduction order, in one launch; the time steps
//    of a segment table in two.

#include <algorithm>
#include <type_traits>

#include "fill_order.hpp"
#include "hydro_internal.h"

namespace hy {

// Stores the q-th 16 bytes of an LDS array to the q-th of a 16-byte aligned
// global one, around the caches (for outputs that are larger than they are).
template <typename T> __device__ __forceinline__ void store16(T* dst, int q, const T* lds) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(reinterpret_cast<const f4*>(lds)[q], reinterpret_cast<f4*>(dst) + q);
}

// ---------------------------------------------------------------------------
// Periodic ghost fill.  Output groups [G][5][N][N][N], G = (gz*ngy+gy)*ngx+gx.
// Source either a plain box [5][nz][ny][nx] or the grouped interior layout
// [G][5][16][16][16] (grouped != 0).  One thread per output cell, x fastest.
// ---------------------------------------------------------------------------
// GC > 0: the ghost width fixed at compile time (no run-time integer
// division per cell); GC == 0: g taken at run time.
//
// Bound by memory: 20 B written per ghosted FP32 cell and 20 B read, the reads
// of ghost layers from L2, which fill_order.hpp's order by XCD keeps local.
// WIDE (out 16-byte aligned; an N x N plane is a multiple of that): the planes
// are passed through LDS and stored 16 bytes a lane, around the caches, which
// the output would sweep of the input.  Both together, g = 3, FP32, plain box:
// 128^3 cells 49 -> 25 us, 192^3 198 -> 79 (148 through the caches), 256^3 480
// -> 322 (396).  Below 64 groups (4 us) neither pays.
template <typename T, int GC, bool WIDE>
__global__ void __launch_bounds__(512) fill_periodic_kernel(const T* __restrict__ box, int nx, int ny, int nz, int g_rt,
                                                            int grouped, T* __restrict__ out, long long g_off, int cnt,
                                                            bool by_xcd) {
  // A workgroup fills planes k and k + 1 of a padded group (N = 16 + 2g is
  // even; k even), all ten loads of a thread issued before its stores; threads
  // cover the N x N plane, x fastest.  Group counts stay below 2^31 (the caller
  // checks), so the group coordinates use 32-bit division.
  __shared__ __align__(16) T sm[WIDE ? 10 * (16 + 2 * GC) * (16 + 2 * GC) : 1];
  const int g = GC > 0 ? GC : g_rt;
  const int N = 16 + 2 * g;
  const long long nc = (long long)N * N * N;
  const FillItem it = fill_item(blockIdx.x, cnt, N / 2, by_xcd);
  const unsigned gl = it.group;
  const int k = 2 * (int)it.pair;
  if (gl >= (unsigned)cnt) return;  // uniform
  const unsigned G = (unsigned)(g_off + gl);
  const unsigned ngx = (unsigned)nx >> 4, ngy = (unsigned)ny >> 4;
  const long long boxc = (long long)nx * ny * nz;
  const int gx = (int)(G % ngx), gy = (int)((G / ngx) % ngy), gz = (int)(G / ngx / ngy);
  int sz0 = gz * 16 + k - g, sz1 = sz0 + 1;
  sz0 += (sz0 < 0) ? nz : 0;
  sz0 -= (sz0 >= nz) ? nz : 0;
  sz1 += (sz1 < 0) ? nz : 0;
  sz1 -= (sz1 >= nz) ? nz : 0;
  T* o = out + (long long)G * 5 * nc + (long long)k * N * N;
  for (int r = threadIdx.x; r < N * N; r += blockDim.x) {
    const int i = r % N, j = r / N;
    int sx = gx * 16 + i - g, sy = gy * 16 + j - g;
    sx += (sx < 0) ? nx : 0; sx -= (sx >= nx) ? nx : 0;
    sy += (sy < 0) ? ny : 0; sy -= (sy >= ny) ? ny : 0;
    const T *s0, *s1;
    long long vs;  // between variables
    if (grouped) {
      const long long base = ((long long)(sy >> 4) * ngx + (sx >> 4));
      const long long sg0 = (long long)(sz0 >> 4) * ngy * ngx + base, sg1 = (long long)(sz1 >> 4) * ngy * ngx + base;
      const int in = ((sy & 15) * 16 + (sx & 15));
      s0 = box + sg0 * 5 * 4096 + (sz0 & 15) * 256 + in;
      s1 = box + sg1 * 5 * 4096 + (sz1 & 15) * 256 + in;
      vs = 4096;
    } else {
      s0 = box + ((long long)sz0 * ny + sy) * nx + sx;
      s1 = box + ((long long)sz1 * ny + sy) * nx + sx;
      vs = boxc;
    }
    T v0[5], v1[5];
#pragma unroll
    for (int n = 0; n < 5; ++n) { v0[n] = s0[n * vs]; v1[n] = s1[n * vs]; }
#pragma unroll
    for (int n = 0; n < 5; ++n) {
      if constexpr (WIDE) {
        sm[2 * n * N * N + r] = v0[n];
        sm[(2 * n + 1) * N * N + r] = v1[n];
      } else {
        o[n * nc + r] = v0[n];
        o[n * nc + N * N + r] = v1[n];
      }
    }
  }
  if constexpr (WIDE) {
    __syncthreads();
    const int Q = 2 * N * N * (int)sizeof(T) / 16;  // 16-byte pieces of two planes
    for (int q = threadIdx.x; q < 5 * Q; q += blockDim.x) store16(o + (q / Q) * nc, q % Q, sm + (q / Q) * 2 * N * N);
  }
}

template <typename T, int GC>
static void go_fill_periodic(const T* box, int nx, int ny, int nz, int g, int grouped, T* out, long long g0, int cnt,
                             hipStream_t st) {
  const bool many = cnt >= 64, by_xcd = fill_by_xcd(cnt, sizeof(T), g, nx / 16, grouped != 0);
  const dim3 grid(fill_grid(cnt, 8 + g, by_xcd));
  if constexpr (GC > 0) {
    if (many && (uintptr_t)out % 16 == 0) {
      fill_periodic_kernel<T, GC, true><<<grid, dim3(512), 0, st>>>(box, nx, ny, nz, g, grouped, out, g0, cnt, by_xcd);
      return;
    }
  }
  fill_periodic_kernel<T, GC, false><<<grid, dim3(512), 0, st>>>(box, nx, ny, nz, g, grouped, out, g0, cnt, by_xcd);
}

template <typename T>
hipError_t launch_fill_periodic(const T* box, int nx, int ny, int nz, int g, int grouped, T* out, hipStream_t st) {
  const long long groups = (long long)(nx / 16) * (ny / 16) * (nz / 16);
  // at most 2^20 groups per launch: the grid stays below 2^31
  for (long long g0 = 0; g0 < groups; g0 += 1 << 20) {
    const int cnt = (int)(groups - g0 < (1 << 20) ? groups - g0 : (1 << 20));
    switch (g) {
      case 2: go_fill_periodic<T, 2>(box, nx, ny, nz, g, grouped, out, g0, cnt, st); break;
      case 3: go_fill_periodic<T, 3>(box, nx, ny, nz, g, grouped, out, g0, cnt, st); break;
      case 4: go_fill_periodic<T, 4>(box, nx, ny, nz, g, grouped, out, g0, cnt, st); break;
      default: go_fill_periodic<T, 0>(box, nx, ny, nz, g, grouped, out, g0, cnt, st); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template hipError_t launch_fill_periodic<float>(const float*, int, int, int, int, int, float*, hipStream_t);
template hipError_t launch_fill_periodic<double>(const double*, int, int, int, int, int, double*, hipStream_t);

// ---------------------------------------------------------------------------
// AMR-shaped preparation: every cell of every padded group is the trilinear
// interpolation, at its centre, of a periodic coarse field [5][cn][cn][cn]
// on the unit box.  layout[G] = (level, ox, oy, oz): the group's first
// interior cell on the level-l grid of spacing base_dh / 2^l.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) fill_interp_kernel(const T* __restrict__ coarse, int cn,
                                                          const int4* __restrict__ layout, int g, double base_dh,
                                                          T* __restrict__ out, long long total) {
  const int N = 16 + 2 * g;
  const long long nc = (long long)N * N * N;
  const long long cc = (long long)cn * cn * cn;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const long long G = t / nc;
    const int r = (int)(t - G * nc);
    const int i = r % N, j = (r / N) % N, k = r / (N * N);
    const int4 L = layout[G];
    const double dh = base_dh / (double)(1 << L.x);
    // Coarse-index coordinates of the fine cell centre.
    const double X = ((double)(L.y + i - g) + 0.5) * dh * cn - 0.5;
    const double Y = ((double)(L.z + j - g) + 0.5) * dh * cn - 0.5;
    const double Z = ((double)(L.w + k - g) + 0.5) * dh * cn - 0.5;
    const double fx0 = floor(X), fy0 = floor(Y), fz0 = floor(Z);
    const double ax = X - fx0, ay = Y - fy0, az = Z - fz0;
    int x0 = (int)fx0, y0 = (int)fy0, z0 = (int)fz0;
    x0 = ((x0 % cn) + cn) % cn; y0 = ((y0 % cn) + cn) % cn; z0 = ((z0 % cn) + cn) % cn;
    const int x1 = (x0 + 1) % cn, y1 = (y0 + 1) % cn, z1 = (z0 + 1) % cn;
    const long long c000 = ((long long)z0 * cn + y0) * cn + x0, c001 = ((long long)z0 * cn + y0) * cn + x1;
    const long long c010 = ((long long)z0 * cn + y1) * cn + x0, c011 = ((long long)z0 * cn + y1) * cn + x1;
    const long long c100 = ((long long)z1 * cn + y0) * cn + x0, c101 = ((long long)z1 * cn + y0) * cn + x1;
    const long long c110 = ((long long)z1 * cn + y1) * cn + x0, c111 = ((long long)z1 * cn + y1) * cn + x1;
    T* o = out + G * 5 * nc + r;
#pragma unroll
    for (int n = 0; n < 5; ++n) {
      const T* f = coarse + n * cc;
      const double v00 = (1.0 - ax) * (double)f[c000] + ax * (double)f[c001];
      const double v01 = (1.0 - ax) * (double)f[c010] + ax * (double)f[c011];
      const double v10 = (1.0 - ax) * (double)f[c100] + ax * (double)f[c101];
      const double v11 = (1.0 - ax) * (double)f[c110] + ax * (double)f[c111];
      const double v0 = (1.0 - ay) * v00 + ay * v01;
      const double v1 = (1.0 - ay) * v10 + ay * v11;
      o[n * nc] = (T)((1.0 - az) * v0 + az * v1);
    }
  }
}

// The same interpolation with one workgroup per group and one thread per
// (x, y) column of its padded region, the ghost width fixed at compile time.
// A column's x and y weights and coarse indices are formed once.  Along z,
// the value of a fine cell is the z blend of the x-y interpolations at the
// two coarse layers that bracket it.  Where the fine level is finer than the
// coarse field, the pair stays the same over several consecutive fine planes
// and moves by one layer at a time, so each thread keeps both layers' x-y
// values in registers and reads the coarse field only for a new layer.
// Every value is formed by the expressions of fill_interp_kernel, in the
// same order and without contraction, so the results are those of a plain
// FP64 evaluation.
__device__ __forceinline__ int wrap_index(long long v, int n) {
  if (v < 0 || v >= n) {  // ghost cells across the periodic boundary
    v %= n;
    if (v < 0) v += n;
  }
  return (int)v;
}
template <int G> constexpr int interp_threads() { return ((16 + 2 * G) * (16 + 2 * G) + 63) / 64 * 64; }

template <typename T, int G>
__global__ void __launch_bounds__(interp_threads<G>()) fill_interp_group_kernel(const T* __restrict__ coarse, int cn,
                                                                               const int4* __restrict__ layout,
                                                                               double base_dh, T* __restrict__ out) {
#pragma clang fp contract(off)
  constexpr int N = 16 + 2 * G;
  constexpr long long nc = (long long)N * N * N;
  const long long cc = (long long)cn * cn * cn;
  const long long grp = blockIdx.x;
  const int4 L = layout[grp];
  const double dh = base_dh / (double)(1 << L.x);
  const int r = threadIdx.x;
  if (r >= N * N) return;  // no barrier below
  const int i = r % N, j = r / N;
  const double X = ((double)(L.y + i - G) + 0.5) * dh * cn - 0.5;
  const double Y = ((double)(L.z + j - G) + 0.5) * dh * cn - 0.5;
  const double fx0 = floor(X), fy0 = floor(Y);
  const double ax = X - fx0, ay = Y - fy0;
  const int x0 = wrap_index((long long)fx0, cn), y0 = wrap_index((long long)fy0, cn);
  const int x1 = x0 + 1 == cn ? 0 : x0 + 1, y1 = y0 + 1 == cn ? 0 : y0 + 1;
  // x-y interpolation of layer z of variable n at this column.
  auto layer = [&](int z, int n) -> double {
    const T* f = coarse + n * cc + (long long)z * cn * cn;
    const double v00 = (1.0 - ax) * (double)f[y0 * cn + x0] + ax * (double)f[y0 * cn + x1];
    const double v01 = (1.0 - ax) * (double)f[y1 * cn + x0] + ax * (double)f[y1 * cn + x1];
    return (1.0 - ay) * v00 + ay * v01;
  };
  T* o = out + grp * 5 * nc + r;
  double v0[5], v1[5];
  int zc = -1;  // coarse layer of v0 (none yet)
  for (int k = 0; k < N; ++k) {
    const double Z = ((double)(L.w + k - G) + 0.5) * dh * cn - 0.5;
    const double fz0 = floor(Z);
    const double az = Z - fz0;
    const int z0 = wrap_index((long long)fz0, cn), z1 = z0 + 1 == cn ? 0 : z0 + 1;
    if (z0 != zc) {  // uniform over the workgroup
      const bool shift = zc >= 0 && z0 == (zc + 1 == cn ? 0 : zc + 1);
#pragma unroll
      for (int n = 0; n < 5; ++n) {
        v0[n] = shift ? v1[n] : layer(z0, n);
        v1[n] = layer(z1, n);
      }
      zc = z0;
    }
#pragma unroll
    for (int n = 0; n < 5; ++n) o[n * nc + (long long)k * N * N] = (T)((1.0 - az) * v0[n] + az * v1[n]);
  }
}

template <typename T, int G>
static hipError_t launch_interp_groups(const T* coarse, int cn, const int* layout, long long n_groups, double base_dh,
                                       T* out, hipStream_t st) {
  fill_interp_group_kernel<T, G><<<dim3((unsigned)n_groups), dim3(interp_threads<G>()), 0, st>>>(
      coarse, cn, (const int4*)layout, base_dh, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// AMR preparation step for groups next to coarse-fine boundaries (Sec. 4.2:
// ghost data by spatial and temporal interpolation).  Level l spans the
// periodic unit box with ng_l = ng0 << l groups (16 ng_l cells) per side;
// the group map holds, per level, the index of the group at each group
// position or -1: map[off_l + (gz ng_l + gy) ng_l + gx], off_l = sum over
// m < l of ng_m^3.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) fill_int_kernel(int* __restrict__ p, long long n, int v) {
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
    p[t] = v;
}
// Group origins off the level's 16-cell grid or outside it, and levels out of
// range, are left out; where two groups share a position the higher index
// wins (atomicMax), so the map does not depend on scheduling.
__global__ void __launch_bounds__(256) group_map_kernel(const int4* __restrict__ layout, int n_groups, int ng0,
                                                        int n_levels, int* __restrict__ map) {
  const int G = blockIdx.x * blockDim.x + threadIdx.x;
  if (G >= n_groups) return;
  const int4 L = layout[G];
  if (L.x < 0 || L.x >= n_levels) return;
  const long long ng = (long long)ng0 << L.x, nl = 16 * ng;
  if (L.y < 0 || L.z < 0 || L.w < 0 || L.y >= nl || L.z >= nl || L.w >= nl || ((L.y | L.z | L.w) & 15)) return;
  long long off = 0;
  for (int m = 0; m < L.x; ++m) {
    const long long q = (long long)ng0 << m;
    off += q * q * q;
  }
  atomicMax(&map[off + ((long long)(L.w >> 4) * ng + (L.z >> 4)) * ng + (L.y >> 4)], G);
}

hipError_t launch_group_map(const int* layout, int n_groups, int ng0, int n_levels, long long map_len, int* map,
                            hipStream_t st) {
  long long blocks = (map_len + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  fill_int_kernel<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(map, map_len, -1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || n_groups == 0) return e;
  group_map_kernel<<<dim3((unsigned)((n_groups + 255) / 256)), dim3(256), 0, st>>>((const int4*)layout, n_groups, ng0,
                                                                                  n_levels, map);
  return hipGetLastError();
}

// One workgroup per group, one thread per (x, y) column of its padded
// region, marching along z.  A cell is the group's own interior value, else
// the value of the same-level group that the map places at its (periodic)
// position, else the coarse state blended in time, (1 - alpha_l) coarse0 +
// alpha_l coarse1 at the four coarse points of a layer, interpolated in x
// and y and then in z between the two layers that bracket the cell; a
// thread keeps both layers' values and recomputes them only when the pair
// moves.  When the coarse points that the group's padded region touches fit
// in kFoot^3 (levels at least about 4x finer than the coarse field), the
// workgroup first blends them once into LDS and the columns interpolate
// from there; when one layer of them fits in kSide^2 (levels as fine as the
// coarse field), it blends a layer at a time; otherwise every column blends
// from global memory.  All give the same values.  No contraction: a plain FP64 evaluation of that
// expression.  Map entries outside [0, n_groups) count as empty, and levels
// are clamped into range, so every access stays inside the arrays whatever
// the layout holds.
//
// The floor is memory (FP32, g = 3: 213 KB written and 82 KB read a group,
// 1.16 ms for 20,480 groups at 5.2 TB/s).  It took 2.0 ms, bound by its
// instructions (every cell formed its plane's coarse coordinate in FP64 and
// tested three sources) and by stores of 4 bytes a lane.  A column meets three
// z ranges (below the group, its own planes, above), each a copy from one
// group or an interpolation throughout, so the sources are chosen once per
// range, and the planes' coarse layers and weights come from a table: 1.56 ms.
// Two planes at a time then pass through LDS and are stored 16 bytes a lane
// around the caches: 1.36 ms.  (Such stores of 4 bytes a lane were slower, 1.9
// ms: they split the 128-byte lines of a 22 x 22 plane.)  Small launches split
// a group's planes over gridDim.y workgroups.
template <typename T>
struct AmrArgs {
  const T* fine;       // [n][5][16][16][16]
  const int4* layout;  // [n] (level, ox, oy, oz)
  const int* map;
  const T* c0;         // [5][cn][cn][cn]
  const T* c1;
  T* out;              // [n][5][N][N][N]
  int n_groups, ng0, n_levels, cn;
  double alpha[8];
};

constexpr int kFoot = 8;   // coarse points per axis staged in LDS as a whole
constexpr int kSide = 25;  // coarse points per axis of a layer staged in LDS
static_assert(kSide * kSide >= kFoot * kFoot * kFoot, "one buffer serves both");

template <typename T, int G>
__global__ void __launch_bounds__(interp_threads<G>()) fill_amr_group_kernel(AmrArgs<T> a) {
#pragma clang fp contract(off)
  constexpr int N = 16 + 2 * G;
  constexpr long long nc = (long long)N * N * N;
  __shared__ double sB[5][kSide * kSide];  // blended coarse points: the footprint [z][y][x] or a layer [y][x]
  __shared__ double sAz[N];                // z weight of each plane
  __shared__ int sZ[N];                    // its lower coarse layer (unwrapped)
  __shared__ __align__(16) T sm[10 * N * N];  // two finished planes of the five variables
  // The workgroup's planes, an even number.
  const int kb = 2 * ((int)blockIdx.y * (N / 2) / (int)gridDim.y);
  const int ke = 2 * (((int)blockIdx.y + 1) * (N / 2) / (int)gridDim.y);
  const int cn = a.cn;
  const long long cc = (long long)cn * cn * cn;
  const long long grp = blockIdx.x;
  const int4 L = a.layout[grp];
  const int r = threadIdx.x;
  const int lev = L.x < 0 ? 0 : (L.x >= a.n_levels ? a.n_levels - 1 : L.x);
  const long long ng = (long long)a.ng0 << lev;
  const int nl = (int)(16 * ng);
  long long moff = 0;
  for (int m = 0; m < lev; ++m) {
    const long long q = (long long)a.ng0 << m;
    moff += q * q * q;
  }
  const double dh = 1.0 / (double)nl;
  const double al = a.alpha[lev];
  // Coarse-index coordinate of the centre of padded-region cell c (-G .. 15+G)
  // along an axis whose group origin is o.
  auto coord = [&](int o, int c) -> double { return (((double)o + c) + 0.5) * dh * cn - 0.5; };
  // Footprint: unwrapped coarse indices lo .. lo + W - 1 per axis.
  const int lox = (int)floor(coord(L.y, -G)), loy = (int)floor(coord(L.z, -G)), loz = (int)floor(coord(L.w, kb - G));
  const int wx = (int)floor(coord(L.y, 15 + G)) + 2 - lox, wy = (int)floor(coord(L.z, 15 + G)) + 2 - loy,
            wz = (int)floor(coord(L.w, ke - 1 - G)) + 2 - loz;
  // Uniform over the workgroup.  Origins outside the level take the direct
  // path, whose indices all wrap.
  const bool inside = L.y >= 0 && L.y < nl && L.z >= 0 && L.z < nl && L.w >= 0 && L.w < nl;
  const bool staged = inside && wx <= kFoot && wy <= kFoot && wz <= kFoot;
  const bool layered = inside && !staged && wx <= kSide && wy <= kSide;
  // Blended coarse values of point (ix, iy) of the footprint in layer zu.
  auto blend = [&](int ix, int iy, int zu, int p) {
    const long long g = ((long long)wrap_index((long long)zu, cn) * cn + wrap_index((long long)loy + iy, cn)) * cn +
                        wrap_index((long long)lox + ix, cn);
    T u0[5], u1[5];
#pragma unroll
    for (int n = 0; n < 5; ++n) { u0[n] = a.c0[n * cc + g]; u1[n] = a.c1[n * cc + g]; }
#pragma unroll
    for (int n = 0; n < 5; ++n) sB[n][p] = (1.0 - al) * (double)u0[n] + al * (double)u1[n];
  };
  if (staged) {
    for (int p = r; p < kFoot * kFoot * kFoot; p += blockDim.x) {
      const int ix = p % kFoot, iy = (p / kFoot) % kFoot, iz = p / (kFoot * kFoot);
      if (ix < wx && iy < wy && iz < wz) blend(ix, iy, loz + iz, p);
    }
  }
  if (r < N) {
    const double Z = coord(L.w, r - G), fz0 = floor(Z);
    sAz[r] = Z - fz0;
    sZ[r] = (int)fz0;
  }
  __syncthreads();
  const bool column = r < N * N;  // the others help at the barriers
  const int rc = column ? r : 0;
  const int ci = rc % N - G, cj = rc / N - G;
  const bool in_xy = ci >= 0 && ci < 16 && cj >= 0 && cj < 16;
  const int px = wrap_index((long long)L.y + ci, nl), py = wrap_index((long long)L.z + cj, nl);
  const int pz0 = wrap_index((long long)L.w, nl) & 15;  // 0 for origins on the 16-cell grid
  const double X = coord(L.y, ci), Y = coord(L.z, cj);
  const double fx0 = floor(X), fy0 = floor(Y);
  const double ax = X - fx0, ay = Y - fy0;
  const int x0 = wrap_index((long long)fx0, cn), y0 = wrap_index((long long)fy0, cn);
  const int x1 = x0 + 1 == cn ? 0 : x0 + 1, y1 = y0 + 1 == cn ? 0 : y0 + 1;
  const int sx = (int)fx0 - lox, sy = (int)fy0 - loy;  // staged footprint indices
  // x-y interpolation of layer z (unwrapped coarse index) of variable n; with
  // layered, of the layer that sB holds.
  auto layer = [&](int zu, int n) -> double {
    if (staged || layered) {
      const int w = staged ? kFoot : kSide;
      const double* f = sB[n] + (staged ? (zu - loz) * kFoot * kFoot : 0) + sy * w + sx;
      const double v00 = (1.0 - ax) * f[0] + ax * f[1];
      const double v01 = (1.0 - ax) * f[w] + ax * f[w + 1];
      return (1.0 - ay) * v00 + ay * v01;
    }
    const long long base = (long long)n * cc + (long long)wrap_index(zu, cn) * cn * cn;
    const T* f0 = a.c0 + base;
    const T* f1 = a.c1 + base;
    auto b = [&](int q) -> double { return (1.0 - al) * (double)f0[q] + al * (double)f1[q]; };
    const double v00 = (1.0 - ax) * b(y0 * cn + x0) + ax * b(y0 * cn + x1);
    const double v01 = (1.0 - ax) * b(y1 * cn + x0) + ax * b(y1 * cn + x1);
    return (1.0 - ay) * v00 + ay * v01;
  };
  // The column meets three group positions along z (below, its own, above;
  // G < 16): the cells it copies there (null: it interpolates).
  const T* src[3];
  {
    const long long gzc = wrap_index((long long)L.w, nl) >> 4;
    const int in = (py & 15) * 16 + (px & 15);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      long long gz = gzc + t - 1;
      gz += gz < 0 ? ng : 0;
      gz -= gz >= ng ? ng : 0;
      const int ow = a.map[moff + (gz * ng + (py >> 4)) * ng + (px >> 4)];
      src[t] = ow >= 0 && ow < a.n_groups ? a.fine + (long long)ow * 5 * 4096 + in : nullptr;
    }
    if (in_xy) src[1] = a.fine + grp * 5 * 4096 + cj * 16 + ci;
  }
  double v0[5], v1[5];
  bool have = false;
  int zc = 0;  // unwrapped coarse layer of v0 (if any), the same for all columns of the wavefront
  // A layer at a time, by all threads (the caller is uniform).
  auto load_layer = [&](int zu, double (&v)[5]) {
    __syncthreads();  // the previous layer has been read
    for (int p = r; p < wx * wy; p += blockDim.x) blend(p % wx, p / wx, zu, p / wx * kSide + p % wx);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 5; ++n) v[n] = layer(zu, n);
  };
  // Where plane k of the column comes from.
  auto source = [&](int k) -> const T* {
    const int t = k < G ? 0 : (k < G + 16 ? 1 : 2);
    const T* s = src[t];
    return s ? s + (((t == 1 && in_xy ? 0 : pz0) + k - G) & 15) * 256 : nullptr;
  };
  // The copied cells of two planes are requested while the two before them are
  // stored.
  T next[2][5];
  auto request = [&](int k) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const T* q = source(k + p);
      if (q) {
#pragma unroll
        for (int n = 0; n < 5; ++n) next[p][n] = q[n * 4096];
      }
    }
  };
  T* og = a.out + grp * 5 * nc;
  const bool wide = (uintptr_t)a.out % 16 == 0;  // uniform
  request(kb);
  for (int k = kb; k < ke; k += 2) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const bool copied = source(k + p) != nullptr;
      T val[5];
#pragma unroll
      for (int n = 0; n < 5; ++n) val[n] = next[p][n];
      if (layered || __any(!copied)) {
        const int z = __builtin_amdgcn_readfirstlane(sZ[k + p]);
        const double az = sAz[k + p], bz = 1.0 - az;
        if (!have || z != zc) {
          const bool shift = have && z == zc + 1;
          if (layered) {
            if (shift) {
#pragma unroll
              for (int n = 0; n < 5; ++n) v0[n] = v1[n];
            } else {
              load_layer(z, v0);
            }
            load_layer(z + 1, v1);
          } else {
#pragma unroll
            for (int n = 0; n < 5; ++n) {
              v0[n] = shift ? v1[n] : layer(z, n);
              v1[n] = layer(z + 1, n);
            }
          }
          zc = z;
          have = true;
        }
        if (!copied) {
#pragma unroll
          for (int n = 0; n < 5; ++n) val[n] = (T)(bz * v0[n] + az * v1[n]);
        }
      }
      if (column) {
#pragma unroll
        for (int n = 0; n < 5; ++n) sm[(2 * n + p) * N * N + r] = val[n];
      }
    }
    if (k + 2 < ke) request(k + 2);
    __syncthreads();
    constexpr int C = 2 * N * N, Q = C * (int)sizeof(T) / 16;
    T* o = og + (long long)k * N * N;
    if (wide) {
      for (int q = r; q < 5 * Q; q += blockDim.x) store16(o + (q / Q) * nc, q % Q, sm + (q / Q) * C);
    } else {
      for (int q = r; q < 5 * C; q += blockDim.x) o[(q / C) * nc + q % C] = sm[q];
    }
    __syncthreads();
  }
}

template <typename T, int G>
static hipError_t launch_amr_g(const AmrArgs<T>& a, hipStream_t st) {
  // Workgroups per group: 60 groups (FP32, g = 3) 23.5 us with one, 11.5 with
  // four; 600 groups 45.8 / 43.7 / 49.6 us with 1 / 2 / 4; 2,600 groups 178 /
  // 193 with 1 / 2 (each stages its coarse points anew).
  const int ns = a.n_groups <= 128 ? 4 : (a.n_groups <= 1000 ? 2 : 1);
  fill_amr_group_kernel<T, G><<<dim3((unsigned)a.n_groups, (unsigned)ns), dim3(interp_threads<G>()), 0, st>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fill_amr(const T* fine, const int* layout, int n_groups, const int* map, int ng0, int n_levels,
                           const T* c0, const T* c1, int cn, const double* alpha, int g, T* out, hipStream_t st) {
  if (n_groups == 0) return hipSuccess;
  AmrArgs<T> a;
  a.fine = fine;
  a.layout = (const int4*)layout;
  a.map = map;
  a.c0 = c0;
  a.c1 = c1;
  a.out = out;
  a.n_groups = n_groups;
  a.ng0 = ng0;
  a.n_levels = n_levels;
  a.cn = cn;
  for (int l = 0; l < 8; ++l) a.alpha[l] = l < n_levels ? alpha[l] : 0.0;
  switch (g) {
    case 0: return launch_amr_g<T, 0>(a, st);
    case 1: return launch_amr_g<T, 1>(a, st);
    case 2: return launch_amr_g<T, 2>(a, st);
    case 3: return launch_amr_g<T, 3>(a, st);
    case 4: return launch_amr_g<T, 4>(a, st);
    default: return hipErrorInvalidValue;
  }
}
template hipError_t launch_fill_amr<float>(const float*, const int*, int, const int*, int, int, const float*,
                                           const float*, int, const double*, int, float*, hipStream_t);
template hipError_t launch_fill_amr<double>(const double*, const int*, int, const int*, int, int, const double*,
                                            const double*, int, const double*, int, double*, hipStream_t);

// ---------------------------------------------------------------------------
// Coarse-grid correction after a coarse step (Sec. 2 step 5, Sec. 4.3): the
// coarse level is a periodic n^3 box in patch-group order, the fine level
// has ratio 2 and its groups (fine-grid origins on the 16-cell grid) each
// cover one 8^3 coarse patch; fmap is the fine level's group map (n / 8
// groups per side).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int fine_owner(const int* fmap, int nf, int ngf, int cx, int cy, int cz) {
  const int o = fmap[((long long)(cz >> 3) * ngf + (cy >> 3)) * ngf + (cx >> 3)];
  return (o >= 0 && o < nf) ? o : -1;
}

// Refluxing.  An uncovered coarse cell next to a covered one across a face
// replaces the coarse flux of that face (stored by the coarse step on the
// patch faces: group faces -, + and the mid plane) by the mean of the four
// fine fluxes on it: U -= dt/dh (Ff - Fc) when the fine cell lies on its +
// side, += on its - side, in the order x, y, z and -, +.  No contraction:
// the same FP64 expression as a plain evaluation.
//
// Restriction.  A covered coarse cell becomes the mean of its 8 children.
//
// One 512-thread workgroup per fine group: a thread per covered cell (8^3)
// for the restriction, and waves 0 to 5 a face each, a thread per coarse cell
// just outside it (8 x 8).  The two write disjoint cells (covered, uncovered).
// A cell next to several refined patches is visited from several faces; only
// the face of its first covered neighbour in the order above processes it,
// applying all of its corrections in that order, so every cell is written by
// one thread.  Only the group that the map names at its position writes.
//
// A face's cells lie in one coarse patch, so all that is looked up in the map
// is uniform: the patch itself and its four neighbours beside the face.  Both
// parts wait for memory (a chain of layout, map, fluxes against a stream of
// fine cells), so they share a launch and the fine cells are requested before
// the chain is followed.  6144 groups in a 256^3 box, FP32: 330 us in two
// launches (refluxing 153, restriction 177), 290 in one, which moves 1.2 GB
// (counted; rows of 8 cells of 16, single cells beside x faces): 4.2 TB/s.
template <typename T> struct Reflux {
  const T* cflux;
  const T* fflux;
  double dtdh;
};
// Adds the correction of face q = 2 d + (fine side > 0) of cell c (in group
// G) from fine group F with layout entry o.
template <typename T>
__device__ __forceinline__ void reflux_face(double (&u)[5], const Reflux<T>& R, long long G, const int (&c)[3], int d,
                                            int side, int F, const int4 o) {
#pragma clang fp contract(off)
  // transverse coordinates (slow, fast) of a d-face: x (z, y), y (z, x), z (y, x)
  const int cd = d == 0 ? c[0] : (d == 1 ? c[1] : c[2]);
  const int cs = d == 2 ? c[1] : c[2], cf = d == 0 ? c[1] : c[0];
  const int os = d == 2 ? o.z : o.w, of = d == 0 ? o.z : o.y;
  const int ld = cd & 15;
  const int slot = side > 0 ? (ld == 15 ? 1 : (ld == 7 ? 2 : -1)) : (ld == 0 ? 0 : (ld == 8 ? 2 : -1));
  if (slot < 0) return;  // cannot happen: fine groups cover whole coarse patches
  const int fs0 = 2 * (cs - (os >> 1)), ff0 = 2 * (cf - (of >> 1));
  if (fs0 < 0 || fs0 > 14 || ff0 < 0 || ff0 > 14) return;  // layout disagrees with the map
  const int fslot = side > 0 ? 0 : 1;  // F's face towards this cell
  const double sg = side > 0 ? -1.0 : 1.0;
  const T* cp = R.cflux + ((G * 3 + d) * 3 + slot) * 1280 + (cs & 15) * 16 + (cf & 15);
  const T* fp = R.fflux + (((long long)F * 3 + d) * 2 + fslot) * 1280 + fs0 * 16 + ff0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double Fc = (double)cp[v * 256];
    double Ff = 0.0;
    Ff += (double)fp[v * 256];
    Ff += (double)fp[v * 256 + 1];
    Ff += (double)fp[v * 256 + 16];
    Ff += (double)fp[v * 256 + 17];
    Ff *= 0.25;
    u[v] += sg * R.dtdh * (Ff - Fc);
  }
}

template <typename T>
__global__ void __launch_bounds__(512) amr_correct_kernel(T* __restrict__ U, int n, const T* __restrict__ cflux,
                                                          const T* __restrict__ fine, const int4* __restrict__ flayout,
                                                          const int* __restrict__ fmap, int nf,
                                                          const T* __restrict__ fflux, double dtdh) {
#pragma clang fp contract(off)
  const int F0 = blockIdx.x, tid = threadIdx.x;
  T r[5][8];
  {
    const int i = tid & 7, j = (tid >> 3) & 7, k = tid >> 6;
    const T* f = fine + (long long)F0 * 5 * 4096 + (2 * k * 16 + 2 * j) * 16 + 2 * i;
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int q = 0; q < 8; ++q) r[v][q] = f[v * 4096 + (q >> 2) * 256 + ((q >> 1) & 1) * 16 + (q & 1)];
  }
  asm volatile("" ::: "memory");  // the loads stay ahead of the chain below
  const int4 o0 = flayout[F0];
  const int nfine = 2 * n, ng = n >> 4, ngf = n >> 3;
  if (o0.y < 0 || o0.z < 0 || o0.w < 0 || o0.y >= nfine || o0.z >= nfine || o0.w >= nfine ||
      ((o0.y | o0.z | o0.w) & 15))
    return;
  const int p0[3] = {o0.y >> 4, o0.z >> 4, o0.w >> 4};  // coarse patch of 8^3 cells
  if (fine_owner(fmap, nf, ngf, 8 * p0[0], 8 * p0[1], 8 * p0[2]) != F0) return;

  const int face = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (face < 6) {
    const int dF = face >> 1, sF = (face & 1) ? 1 : -1;  // the fine group's face: axis and side
    // the patch outside this face, and a lane's cell in it
    int p[3] = {p0[0] + (dF == 0 ? sF : 0), p0[1] + (dF == 1 ? sF : 0), p0[2] + (dF == 2 ? sF : 0)};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      p[d] += p[d] < 0 ? ngf : 0;
      p[d] -= p[d] >= ngf ? ngf : 0;
    }
    auto owner = [&](int a, int b, int e) {
      const int o = fmap[((long long)e * ngf + b) * ngf + a];
      return (o >= 0 && o < nf) ? o : -1;
    };
    // Transverse neighbours of the patch, axes e1 < e2, sides -, +.
    const int e1 = dF == 0 ? 1 : 0, e2 = dF == 2 ? 1 : 2;
    int nb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = k < 2 ? e1 : e2, sd = (k & 1) ? 1 : -1;
      int b[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        b[d] = p[d] + (d == e ? sd : 0);
        b[d] += b[d] < 0 ? ngf : 0;
        b[d] -= b[d] >= ngf ? ngf : 0;
      }
      nb[k] = owner(b[0], b[1], b[2]);
    }
    if (owner(p[0], p[1], p[2]) < 0) {  // else covered: restriction sets it
      const int l1 = tid & 7, l2 = (tid >> 3) & 7;
      const int ln = sF < 0 ? 7 : 0;  // along dF, next to the refined patch
      const int c[3] = {8 * p[0] + (dF == 0 ? ln : l1), 8 * p[1] + (dF == 1 ? ln : (dF == 0 ? l1 : l2)),
                        8 * p[2] + (dF == 2 ? ln : l2)};
      // Covered neighbours beside the face, per lane: e1 -, +, e2 -, +.
      const int own[4] = {l1 == 0 ? nb[0] : -1, l1 == 7 ? nb[1] : -1, l2 == 0 ? nb[2] : -1, l2 == 7 ? nb[3] : -1};
      // An axis before dF: that face processes the cell.
      const bool mine = !((e1 < dF && (own[0] >= 0 || own[1] >= 0)) || (e2 < dF && (own[2] >= 0 || own[3] >= 0)));
      if (mine) {
        const Reflux<T> R{cflux, fflux, dtdh};
        const long long G = ((long long)(c[2] >> 4) * ng + (c[1] >> 4)) * ng + (c[0] >> 4);
        T* up = U + G * 5 * 4096 + ((c[2] & 15) * 16 + (c[1] & 15)) * 16 + (c[0] & 15);
        double u[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) u[v] = (double)up[v * 4096];
        reflux_face(u, R, G, c, dF, -sF, F0, o0);  // from the cell, the patch lies on side -sF
        // and the faces after it in the order
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int e = k < 2 ? e1 : e2;
          if (e > dF && nb[k] >= 0 && own[k] >= 0) reflux_face(u, R, G, c, e, (k & 1) ? 1 : -1, nb[k], flayout[nb[k]]);
        }
#pragma unroll
        for (int v = 0; v < 5; ++v) up[v * 4096] = (T)u[v];
      }
    }
  }

  const int cx = 8 * p0[0] + (tid & 7), cy = 8 * p0[1] + ((tid >> 3) & 7), cz = 8 * p0[2] + (tid >> 6);
  T* up = U + (((long long)(cz >> 4) * ng + (cy >> 4)) * ng + (cx >> 4)) * 5 * 4096 +
          ((cz & 15) * 16 + (cy & 15)) * 16 + (cx & 15);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s += (double)r[v][q];
    up[v * 4096] = (T)(0.125 * s);
  }
}

template <typename T>
hipError_t launch_amr_correct(T* U, int n, const T* cflux, const T* fine, const int* flayout, int nf,
                              const int* fmap, const T* fflux, double dtdh, hipStream_t st) {
  if (nf == 0) return hipSuccess;
  amr_correct_kernel<T><<<dim3((unsigned)nf), dim3(512), 0, st>>>(U, n, cflux, fine, (const int4*)flayout, fmap, nf,
                                                                 fflux, dtdh);
  return hipGetLastError();
}
template hipError_t launch_amr_correct<float>(float*, int, const float*, const float*, const int*, int, const int*,
                                              const float*, double, hipStream_t);
template hipError_t launch_amr_correct<double>(double*, int, const double*, const double*, const int*, int,
                                               const int*, const double*, double, hipStream_t);

// acc += w * x, elementwise (the weighted sum of fine fluxes over sub-steps).
template <typename T>
__global__ void __launch_bounds__(256) axpy_kernel(T* __restrict__ acc, const T* __restrict__ x, double w, long long n) {
#pragma clang fp contract(off)
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
    acc[t] = (T)((double)acc[t] + w * (double)x[t]);
}
template <typename T>
hipError_t launch_axpy(T* acc, const T* x, double w, long long n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  long long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  axpy_kernel<T><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(acc, x, w, n);
  return hipGetLastError();
}
template hipError_t launch_axpy<float>(float*, const float*, double, long long, hipStream_t);
template hipError_t launch_axpy<double>(double*, const double*, double, long long, hipStream_t);

template <typename T>
hipError_t launch_fill_interp(const T* coarse, int cn, const int* layout, long long n_groups, int g, double base_dh,
                              T* out, hipStream_t st) {
  const int N = 16 + 2 * g;
  const long long total = n_groups * N * N * N;
  if (total == 0) return hipSuccess;
  switch (g) {
    case 2: return launch_interp_groups<T, 2>(coarse, cn, layout, n_groups, base_dh, out, st);
    case 3: return launch_interp_groups<T, 3>(coarse, cn, layout, n_groups, base_dh, out, st);
    case 4: return launch_interp_groups<T, 4>(coarse, cn, layout, n_groups, base_dh, out, st);
    default: break;
  }
  long long blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  fill_interp_kernel<T><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(coarse, cn, (const int4*)layout, g, base_dh,
                                                                      out, total);
  return hipGetLastError();
}
template hipError_t launch_fill_interp<float>(const float*, int, const int*, long long, int, double, float*,
                                              hipStream_t);
template hipError_t launch_fill_interp<double>(const double*, int, const int*, long long, int, double, double*,
                                               hipStream_t);

// ---------------------------------------------------------------------------
// FP64 signal speed and time step.  The per-cell expression is evaluated in
// double without contraction, in a fixed order, so that the maximum (and
// hence dt) is bit-identical to a serial FP64 evaluation on the same data.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Four consecutive cells of one variable.  WIDE: 16-byte loads (the array is
// 16-byte aligned; groups and variables are whole multiples of that).
template <typename T, bool WIDE> __device__ __forceinline__ void load4(const T* p, T (&v)[4]) {
  if constexpr (WIDE && sizeof(T) == 4) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else if constexpr (WIDE) {
    const double2 a = reinterpret_cast<const double2*>(p)[0], b = reinterpret_cast<const double2*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = p[k];
  }
}

// Quotients by one divisor b, correctly rounded like the compiler's division:
// the same reciprocal refinement and residual step, the refinement done once
// and without the exponent scaling, which is the identity for operands in the
// range of values upcast from float (and their products and differences).
struct SharedDiv {
  double b, r;
  __device__ __forceinline__ explicit SharedDiv(double d) : b(d), r(__builtin_amdgcn_rcp(d)) {
    r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
  }
  __device__ __forceinline__ double operator()(double a) const {
    const double q = a * r;
    return __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-b, q, a), r, q), b, a);  // zero, inf and NaN
  }
};
struct IeeeDiv {
  double b;
  __device__ __forceinline__ explicit IeeeDiv(double d) : b(d) {}
  __device__ __forceinline__ double operator()(double a) const { return a / b; }
};

// max_d |v_d| + c of a conserved cell of type T, in the order and rounding of
// a serial IEEE evaluation.
template <typename T> __device__ __forceinline__ double signal_speed(const double c[5], double gamma) {
#pragma clang fp contract(off)
  using Div = typename std::conditional<sizeof(T) == 4, SharedDiv, IeeeDiv>::type;
  const Div over_rho(c[0]);
  const double mx = c[1], my = c[2], mz = c[3];
  const double vx = over_rho(mx), vy = over_rho(my), vz = over_rho(mz);
  const double ke = 0.5 * (mx * vx + my * vy + mz * vz);
  const double p = (gamma - 1.0) * (c[4] - ke);
  const double cs = __builtin_sqrt(over_rho(gamma * p));
  double av = __builtin_fabs(vx);
  if (__builtin_fabs(vy) > av) av = __builtin_fabs(vy);
  if (__builtin_fabs(vz) > av) av = __builtin_fabs(vz);
  return av + cs;
}

// Batched time step: one workgroup per group of a segment table computes the
// group's maximum signal speed (same expression as above), four cells a
// thread: the launch is short and bound by latency, so all of a group's loads
// are in flight at once (520 FP32 groups, finish included: 13.6 us, 18.0 with
// 256 threads that took 16 cells one after another).  One workgroup per segment then
// writes dt = cfl * dh / max to the segment's dt pointer.
template <typename T>
__global__ void __launch_bounds__(1024) seg_maxspeed_kernel(const Seg* __restrict__ segs, int n_segs, double gamma,
                                                            double* __restrict__ partial) {
  __shared__ double red[16];
  const long long gidx = blockIdx.x;
  int lo = 0, hi = n_segs - 1;  // last segment with first <= gidx
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (segs[mid].first <= gidx) lo = mid;
    else hi = mid - 1;
  }
  const Seg& S = segs[lo];
  const T* u = reinterpret_cast<const T*>(S.out) + (gidx - S.first) * 5 * 4096 + threadIdx.x * 4;
  T v[5][4];
  if ((uintptr_t)S.out % 16 == 0) {  // uniform
#pragma unroll
    for (int n = 0; n < 5; ++n) load4<T, true>(u + n * 4096, v[n]);
  } else {
#pragma unroll
    for (int n = 0; n < 5; ++n) load4<T, false>(u + n * 4096, v[n]);
  }
  double m = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double c[5] = {(double)v[0][k], (double)v[1][k], (double)v[2][k], (double)v[3][k], (double)v[4][k]};
    const double sp = signal_speed<T>(c, gamma);
    m = sp > m ? sp : m;
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x < 64) {
    m = wave_max(threadIdx.x < 16 ? red[threadIdx.x] : 0.0);
    if (threadIdx.x == 0) partial[gidx] = m;
  }
}

__global__ void __launch_bounds__(256) seg_dt_finish_kernel(const Seg* __restrict__ segs,
                                                            const double* __restrict__ partial, double cfl) {
#pragma clang fp contract(off)
  __shared__ double red[4];
  const Seg& S = segs[blockIdx.x];
  double m = 0.0;
  for (long long q = threadIdx.x; q < S.count; q += blockDim.x) m = fmax(m, partial[S.first + q]);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    *const_cast<double*>(S.dt) = cfl * S.dh / mx;
  }
}

hipError_t launch_seg_dt(const Seg* segs, int n_segs, long long n_groups, double gamma, double cfl, int f64,
                         double* partial, hipStream_t st) {
  if (n_groups > 2147483647LL) return hipErrorInvalidValue;
  if (f64) seg_maxspeed_kernel<double><<<dim3((unsigned)n_groups), dim3(1024), 0, st>>>(segs, n_segs, gamma, partial);
  else seg_maxspeed_kernel<float><<<dim3((unsigned)n_groups), dim3(1024), 0, st>>>(segs, n_segs, gamma, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  seg_dt_finish_kernel<<<dim3(n_segs), dim3(256), 0, st>>>(segs, partial, cfl);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Time step and conserved sums of a whole state, one launch.  A workgroup
// takes a contiguous slice of 1,024-cell chunks (four consecutive cells a
// thread and chunk, lane order, then fixed shuffle trees) and stores its
// partial results; the workgroup that finishes last reduces the partials, in a
// fixed order, and writes the results.  The slices depend on the number of
// groups alone, so repeated calls are bitwise identical, and the time step and
// the sums are the same whether they are asked for together or apart.
//
// Small states are bound by launches (12.2 us with a second launch for the
// finish and scalar loads, 6.7 us now, at 8 groups), large ones by reading the
// state once (4,096 FP32 groups: 81 -> 63 us, 5.4 TB/s; 512: 18.4 -> 13.4).
// In between, the workgroups' arrivals count: up to 512 of them are as fast as
// 1,024 below 2,048 groups (512 groups 13.4 against 14.2 us) and slower from
// there (4,096 groups 66 against 63 us).
//
// The partials pass between workgroups on different XCDs, whose L2 caches are
// not coherent for plain accesses: they are stored and loaded as device-scope
// atomics, and a workgroup counts itself as done only after its stores have
// been acknowledged.
// ---------------------------------------------------------------------------
enum { kRedDt = 1, kRedSums = 2 };

template <typename T, int MODE, bool WIDE>
__global__ void __launch_bounds__(256) reduce_kernel(const T* __restrict__ U, long long n_chunks, long long per,
                                                     double gamma, double cdh, double vol, double* partial,
                                                     unsigned* done, double* __restrict__ dt_out,
                                                     double* __restrict__ sums_out) {
#pragma clang fp contract(off)
  __shared__ double red[6][4];
  __shared__ int last;
  const int tid = threadIdx.x, wave = tid >> 6;
  const long long lo = blockIdx.x * per, hi = lo + per < n_chunks ? lo + per : n_chunks;
  double s[5] = {0, 0, 0, 0, 0}, m = 0.0;
#pragma unroll 2
  for (long long c = lo; c < hi; ++c) {
    const T* u = U + (c >> 2) * (5 * 4096) + (c & 3) * 1024 + tid * 4;
    T v[5][4];
#pragma unroll
    for (int n = 0; n < 5; ++n) load4<T, WIDE>(u + n * 4096, v[n]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double q[5] = {(double)v[0][k], (double)v[1][k], (double)v[2][k], (double)v[3][k], (double)v[4][k]};
      if constexpr (MODE & kRedSums) {
#pragma unroll
        for (int n = 0; n < 5; ++n) s[n] += q[n];
      }
      if constexpr (MODE & kRedDt) {
        const double sp = signal_speed<T>(q, gamma);
        m = sp > m ? sp : m;
      }
    }
  }
  // Per-workgroup results: partial[n * P + b], n = 0..4 the sums, 5 the maximum.
  const int P = gridDim.x;
  auto block_reduce = [&]() {
    if constexpr (MODE & kRedSums) {
#pragma unroll
      for (int n = 0; n < 5; ++n) {
        const double v = wave_sum(s[n]);
        if ((tid & 63) == 0) red[n][wave] = v;
      }
    }
    if constexpr (MODE & kRedDt) {
      m = wave_max(m);
      if ((tid & 63) == 0) red[5][wave] = m;
    }
    __syncthreads();
  };
  constexpr int n0 = MODE & kRedSums ? 0 : 5, n1 = MODE & kRedDt ? 6 : 5;
  auto block_value = [&](int n) -> double {
    return n < 5 ? (red[n][0] + red[n][1]) + (red[n][2] + red[n][3])
                 : fmax(fmax(red[n][0], red[n][1]), fmax(red[n][2], red[n][3]));
  };
  block_reduce();
  if (wave == 0) {
    if (tid >= n0 && tid < n1)
      __hip_atomic_store(&partial[(long long)tid * P + blockIdx.x], block_value(tid), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's stores have reached the device's memory
    if (tid == 0) {
      const unsigned w = arrival_weight(blockIdx.x, P);
      last = arrival_completes(atomicAdd(done + arrival_leaf(blockIdx.x), w), w, kLeafSum) &&
             arrival_completes(atomicAdd(done, 1u), 1u, kDoneLeaves);
    }
  }
  __syncthreads();
  if (!last) return;
  m = 0.0;
#pragma unroll
  for (int n = 0; n < 5; ++n) s[n] = 0.0;
  for (int b = tid; b < P; b += 256) {
    double v[6];
#pragma unroll
    for (int n = n0; n < n1; ++n)
      v[n] = __hip_atomic_load(&partial[(long long)n * P + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (MODE & kRedSums) {
#pragma unroll
      for (int n = 0; n < 5; ++n) s[n] += v[n];
    }
    if constexpr (MODE & kRedDt) m = fmax(m, v[5]);
  }
  block_reduce();
  if (tid >= n0 && tid < n1) {
    const double v = block_value(tid);
    if (tid < 5) sums_out[tid] = v * vol;
    else dt_out[0] = cdh / v;
  }
}

template <typename T, int MODE>
static hipError_t launch_reduce_mode(const T* U, long long n_groups, double dh, double gamma, double cfl,
                                     double* partial, unsigned* done, double* dt_out, double* sums_out,
                                     hipStream_t st) {
  const long long n_chunks = 4 * n_groups, max_partial = n_groups < 2048 ? kReduceMax / 2 : kReduceMax;
  const long long per = (n_chunks + max_partial - 1) / max_partial > 0 ? (n_chunks + max_partial - 1) / max_partial : 1;
  const long long P = std::max((n_chunks + per - 1) / per, (long long)kDoneLeaves);
  auto k = (uintptr_t)U % 16 == 0 ? reduce_kernel<T, MODE, true> : reduce_kernel<T, MODE, false>;
  k<<<dim3((unsigned)P), dim3(256), 0, st>>>(U, n_chunks, per, gamma, cfl * dh, dh * dh * dh, partial, done, dt_out,
                                            sums_out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_reduce(const T* U, long long n_groups, double dh, double gamma, double cfl, double* partial,
                         unsigned* done, double* dt_out, double* sums_out, hipStream_t st) {
  if (dt_out && sums_out)
    return launch_reduce_mode<T, kRedDt | kRedSums>(U, n_groups, dh, gamma, cfl, partial, done, dt_out, sums_out, st);
  if (dt_out)
    return launch_reduce_mode<T, kRedDt>(U, n_groups, dh, gamma, cfl, partial, done, dt_out, sums_out, st);
  return launch_reduce_mode<T, kRedSums>(U, n_groups, dh, gamma, cfl, partial, done, dt_out, sums_out, st);
}
template hipError_t launch_reduce<float>(const float*, long long, double, double, double, double*, unsigned*,
                                         double*, double*, hipStream_t);
template hipError_t launch_reduce<double>(const double*, long long, double, double, double, double*, unsigned*,
                                          double*, double*, hipStream_t);

}  // namespace hy
