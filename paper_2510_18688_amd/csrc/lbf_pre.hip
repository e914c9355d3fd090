// Cahn-Hilliard smoothing of a binary solid image (contract in
// include/lbf_pre.h).  Wavefronts march along the image with the windows of the
// stencils in registers: four Euler steps a pass in 2D, one in 3D.  The first
// pass reads the image itself and the last one writes phi0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "lbf_pre.h"
#include "lbf_sim.hpp"
#include "lbf_step.hpp"

using lbfi::fail;

// Scratch of the allocation-free entry point (lbf_ch_smooth_noalloc): the two
// planes of c for images of up to kStaticNodesCH nodes.  Every device the
// library runs on holds its own copy (32 MiB) from the module's load until
// the process ends.  In host code the array's name is not a device address:
// kernels and copies use the per-device address that hipGetSymbolAddress
// returns.
constexpr long long kStaticNodesCH = 1LL << 22;
static __device__ __align__(256) float scratch[2 * kStaticNodesCH];

namespace {

constexpr long long kMaxNodesCH = 0x7FFFFFFFLL;

// 2D pass: Euler steps, columns per lane, rows in flight per lane, wavefronts
// wanted; 3D pass: rows per lane, wavefronts wanted.
//
// Both passes are bound by vector instructions once enough wavefronts are in
// flight, and the strips' overlaps are recomputed: longer strips waste less and
// leave fewer wavefronts to hide the latencies.  Microseconds per Euler step,
// 4096 x 2048: 4 steps a pass, 1 column a lane, 2048 / 3072 / 4096 / 5500
// wavefronts 13.4 / 10.5 / 10.2 / 10.9; 3 steps 14.1 / 10.7 / 11.3 / 10.3; 2 steps
// 15.3 / 12.2 / 11.1 / 11.0; 1 step (4096) 16.3; 6 steps 14.8 / 11.4 / 13.2 / 12.2; 2
// columns a lane, 4 steps 11.6 / 12.2 / 12.5 / 13.4; 8 rows in flight instead of 4
// within 2 %.  256^3: 4 rows a lane, 2280 / 3040 / 4180 / 6080 wavefronts 58.5 / 41.7
// / 46.1 / 40.5; 6 rows 51.6 / 45.5 / 45.8 / 44.3; 8 rows 55.2 / 52.5 / 45.1 / 47.1; every
// wavefront with its own overlap along y (no LDS) 45 at best.  One step a pass
// through a tile of c and of mu in LDS took 25.2 (2D) and 98 (3D).  Other sizes, 2048 /
// 3072 / 4096 / 5500 wavefronts: 1024^2 3.5 / 3.8 / 3.8 / 3.8, 2000^2 7.1 / 6.7 / 7.3 /
// 7.9, 3333 x 1111 6.6 / 6.7 / 6.6 / 6.9; 3D, 3072 / 4096 / 6144 / 8192: 160^3 16.4 / 16.6 /
// 18.2 / 18.2, 250 x 170 x 90 19.0 / 16.7 / 18.1 / 18.1, 200^3 29.0 / 24.4 / 25.6 / 26.7.  The
// same lines serve all of them within a tenth.  At least four slabs a strip (1 / 2 / 4:
// 20^3 6.0 / 6.7 / 8.1, 64^3 8.0 / 7.7 / 8.2, 128^3 16.0 / 16.2 / 14.1).
constexpr int kT2 = 4, kV2 = 1, kPF2 = 4, kWaves2 = 4096;
constexpr int kR3 = 4, kWaves3 = 6144;

struct ChGeo {
  int n[3];
  int per[3];
};

// Source node of index v along an axis of n nodes: wrapped, or reflected at
// the walls (-1 -> 0, -2 -> 1, n -> n - 1, ...).  The model's ghost repeats the
// first node beyond a wall at every step, and the stencil below treats both
// directions of an axis alike to the last bit, so the reflected continuation
// of the data stays the reflected continuation of the result and the ghost of
// c and of mu needs no step of its own.
__device__ __forceinline__ int source_node(int v, int n, int periodic) {
  while (v < 0 || v >= n) {   // once at most, unless the image is narrower than a strip's overlap
    if (v < 0) v = periodic ? v + n : -1 - v;
    else v = periodic ? v - n : n - 1 - (v - n);
  }
  return v;
}

// The wavefront's place in its workgroup, as a scalar: what a strip derives
// from it (rows, bounds, addresses) then costs no vector instruction.
__device__ __forceinline__ int wave_of_block() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// The value of the next or previous lane of the wavefront (zero beyond its ends).
__device__ __forceinline__ float next_lane(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float prev_lane(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}

// Both lattices' Laplacians 6 sum_i w_i (X(x + c_i) - X(x)) are sums of second
// differences d_x, d_y, d_z (d_x X = (X(x + 1) - X) - (X - X(x - 1))) and their
// products: D2Q9 d_x + d_y + d_x d_y / 6, D3Q19 d_x + d_y + d_z + (d_x d_y +
// d_y d_z + d_x d_z) / 6.  Marching along an axis, a second difference costs two
// subtractions (the first difference is carried), so a Laplacian takes 8 (2D) or
// 13 (3D) operations instead of 19 or 37, every one on differences of
// neighbours: nothing of order X is added up.
//
// No contraction but the written ones: each step rounds alike however many
// steps a launch makes.

__device__ __forceinline__ float ch_mu(float c, float lap, float A, float kappa) {
#pragma clang fp contract(off)
  return __builtin_fmaf(A, __builtin_fmaf(c * c, c, -c), -(kappa * lap));
}

__device__ __forceinline__ float ch_out(float c, bool final) {
  return final ? fminf(fmaxf(0.5f * (1.0f + c), 0.0f), 1.0f) : c;
}

// Element x of the row at `row`: of the image at its first step (img set), else
// of the plane of c.
__device__ __forceinline__ float ch_in(const float* __restrict__ c, const uint8_t* __restrict__ img,
                                       long long row, int x) {
  if (img) return (img + row)[x] ? 1.0f : -1.0f;
  return (c + row)[x];
}

// ---- 2D: T Euler steps in one pass.  A wavefront owns 64 V adjacent columns
// (V per lane) and marches up the rows with every step's window in registers,
// step t two rows behind step t - 1: neighbours along x come from the lane
// next door, along y from the carried differences.  Nothing passes through
// LDS and no wavefront waits for another.  Each step uses up two columns on
// either side and two rows at either end, which a strip recomputes.

// Window of one step: the value at the last row seen (c, mu), its d_x (a) and
// the first differences along y of both; c of the row before.
template <int V>
struct ChWin2 {
  float c[V], c1[V], ec[V], a[V], ea[V], mu[V], em[V], am[V], eam[V];
};

template <int V>
__device__ __forceinline__ void second_diff_x(const float* c, float* a) {
#pragma clang fp contract(off)
  float e[V];
#pragma unroll
  for (int v = 0; v + 1 < V; ++v) e[v] = c[v + 1] - c[v];
  e[V - 1] = next_lane(c[0]) - c[V - 1];
  a[0] = e[0] - prev_lane(e[V - 1]);
#pragma unroll
  for (int v = 1; v < V; ++v) a[v] = e[v] - e[v - 1];
}

// A row of a step's input enters its window (row); the step's result two rows
// before it takes its place.
template <int V>
__device__ __forceinline__ void ch_advance2(ChWin2<V>& w, float* row, float A, float kappa,
                                            float dtM) {
#pragma clang fp contract(off)
  constexpr float sixth = 1.0f / 6.0f;
  float a[V], mu[V], am[V];
  second_diff_x<V>(row, a);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const float ec = row[v] - w.c[v], ea = a[v] - w.a[v];
    const float lap = __builtin_fmaf(sixth, ea - w.ea[v], w.a[v] + (ec - w.ec[v]));
    mu[v] = ch_mu(w.c[v], lap, A, kappa);
    w.ec[v] = ec;
    w.ea[v] = ea;
    w.a[v] = a[v];
  }
  second_diff_x<V>(mu, am);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const float em = mu[v] - w.mu[v], eam = am[v] - w.am[v];
    const float lap = __builtin_fmaf(sixth, eam - w.eam[v], w.am[v] + (em - w.em[v]));
    const float next = __builtin_fmaf(dtM, lap, w.c1[v]);
    w.em[v] = em;
    w.eam[v] = eam;
    w.mu[v] = mu[v];
    w.am[v] = am[v];
    w.c1[v] = w.c[v];
    w.c[v] = row[v];
    row[v] = next;
  }
}

template <int T, int V, int PF>
__global__ __launch_bounds__(256) void k_ch_step2(ChGeo G, const float* __restrict__ c,
                                                  const uint8_t* __restrict__ img,
                                                  float* __restrict__ cn, float A, float kappa,
                                                  float dtM, int rows, int nsx, int nstrips,
                                                  int final) {
  constexpr int W = 64 * V - 4 * T;   // columns a strip delivers
  const int t = lbf::xcd_tile(blockIdx.x, gridDim.x) * 4 + wave_of_block();
  if (t >= nstrips) return;
  const int nx = G.n[0], ny = G.n[1];
  const int xs = (t % nsx) * W, ys = (t / nsx) * rows, ye = ys + min(rows, ny - ys);
  const int lane = threadIdx.x & 63;
  int gx[V], ox[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int col = lane * V + v - 2 * T;   // column of the strip
    gx[v] = source_node(xs + col, nx, G.per[0]);
    ox[v] = col >= 0 && col < W && xs + col < nx ? xs + col : -1;
  }
  const int r0 = ys - 2 * T, r1 = ye + 2 * T;
  auto load = [&](int r, float* b) {
    const long long row = (long long)source_node(r, ny, G.per[1]) * nx;
#pragma unroll
    for (int v = 0; v < V; ++v) b[v] = ch_in(c, img, row, gx[v]);
  };
  float buf[PF][V];
#pragma unroll
  for (int k = 0; k < PF; ++k) load(r0 + k, buf[k]);
  ChWin2<V> w[T] = {};
  for (int r = r0; r < r1; r += PF) {
#pragma unroll
    for (int k = 0; k < PF; ++k) {
      float q[V];
#pragma unroll
      for (int v = 0; v < V; ++v) q[v] = buf[k][v];
      load(r + k + PF, buf[k]);
#pragma unroll
      for (int s = 0; s < T; ++s) ch_advance2<V>(w[s], q, A, kappa, dtM);
      const int ro = r + k - 2 * T;
      if (ro >= ys && ro < ye) {
        float* o = cn + (long long)ro * nx;
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (ox[v] >= 0) o[ox[v]] = ch_out(q[v], final != 0);
      }
    }
  }
}

// ---- 3D: one Euler step per pass, marching along z.  A workgroup's four
// wavefronts own 60 columns and 4 R - 2 rows, R rows of one column per lane;
// neighbours along x come from the lanes next door, along y from the lane's own
// rows, along z from the carried differences.  c is loaded with one row more on
// either side; only mu of a wavefront's outer rows passes through LDS, to the
// wavefronts above and below (one barrier per slab, two buffers), so the rows
// between wavefronts are not computed twice.
template <int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_ch_step3(
    ChGeo G, const float* __restrict__ c, const uint8_t* __restrict__ img, float* __restrict__ cn,
    float A, float kappa, float dtM, int slabs, int nsx, int nsy, int final) {
#pragma clang fp contract(off)
  constexpr int W = 60, H = 4 * R - 2;
  constexpr float sixth = 1.0f / 6.0f;
  __shared__ float edge[2][4][2][64];   // [slab parity][wavefront][first, last row][lane]
  const int t = lbf::xcd_tile(blockIdx.x, gridDim.x);
  const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
  const int wv = wave_of_block(), lane = threadIdx.x & 63;
  const int xs = (t % nsx) * W, yb = ((t / nsx) % nsy) * H, zs = (t / (nsx * nsy)) * slabs;
  const int ys = yb - 1 + wv * R;   // the lane's first row
  const int ze = zs + min(slabs, nz - zs);
  const int gx = source_node(xs + lane - 2, nx, G.per[0]);
  const bool mine = lane >= 2 && lane < 62 && xs + lane - 2 < nx;
  const int below = max(wv - 1, 0), above = min(wv + 1, 3);
  // A wavefront whose rows lie beyond the first one past the image only keeps the
  // barriers: what it would pass on, nobody delivers (us a step with its work and
  // without, and of the former tiles: 4 x 4 x 4000 14.7, 10.5, 10.8; 2 x 2 x 30000 49,
  // 36, 42; 8 x 8 x 8000 21.4, 19.7, 17.3; 256^3 41.5, 41.1, 95).
  if (ys > ny) {
    for (int z = zs - 2; z < ze + 2; ++z) __syncthreads();
    return;
  }
  int gy[R + 2];
#pragma unroll
  for (int r = 0; r < R + 2; ++r) gy[r] = source_node(ys + r - 1, ny, G.per[1]) * nx;
  const long long slab = (long long)nx * ny;
  auto load = [&](int z, float* b) {
    const long long base = source_node(z, nz, G.per[2]) * slab;
    if (img) {
#pragma unroll
      for (int r = 0; r < R + 2; ++r) b[r] = (img + base + gy[r])[gx] ? 1.0f : -1.0f;
    } else {
#pragma unroll
      for (int r = 0; r < R + 2; ++r) b[r] = (c + base + gy[r])[gx];
    }
  };
  // windows along z of c and of mu: the value at the last slab (and c of the
  // one before), d_x + d_y (s), d_x d_y (q) and the first differences along z of
  // the value and of s
  float cz[R] = {}, c2[R] = {}, ez[R] = {}, s[R] = {}, es[R] = {}, q[R] = {};
  float mz[R] = {}, em[R] = {}, sm[R] = {}, esm[R] = {}, qm[R] = {};
  float nxt[R + 2];
  load(zs - 2, nxt);
  for (int z = zs - 2; z < ze + 2; ++z) {
    float in[R + 2], a[R + 2], mu[R + 2];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) in[r] = nxt[r];
    if (z + 1 < ze + 2) load(z + 1, nxt);
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
      const float e = next_lane(in[r]) - in[r];
      a[r] = e - prev_lane(e);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float sn = a[r + 1] + ((in[r + 2] - in[r + 1]) - (in[r + 1] - in[r]));
      const float qn = (a[r + 2] - a[r + 1]) - (a[r + 1] - a[r]);
      const float e = in[r + 1] - cz[r], f = sn - s[r];
      const float lap = __builtin_fmaf(sixth, q[r] + (f - es[r]), s[r] + (e - ez[r]));
      mu[r + 1] = ch_mu(cz[r], lap, A, kappa);
      ez[r] = e;
      es[r] = f;
      s[r] = sn;
      q[r] = qn;
    }
    float(*ed)[2][64] = edge[z & 1];
    ed[wv][0][lane] = mu[1];
    ed[wv][1][lane] = mu[R];
    __syncthreads();
    mu[0] = ed[below][1][lane];
    mu[R + 1] = ed[above][0][lane];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
      const float e = next_lane(mu[r]) - mu[r];
      a[r] = e - prev_lane(e);
    }
    const int zo = z - 2;
    float* o = cn + zo * slab + xs + lane - 2;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float sn = a[r + 1] + ((mu[r + 2] - mu[r + 1]) - (mu[r + 1] - mu[r]));
      const float qn = (a[r + 2] - a[r + 1]) - (a[r + 1] - a[r]);
      const float e = mu[r + 1] - mz[r], f = sn - sm[r];
      const float lap = __builtin_fmaf(sixth, qm[r] + (f - esm[r]), sm[r] + (e - em[r]));
      const float v = __builtin_fmaf(dtM, lap, c2[r]);
      // (the workgroup's outer rows lack their neighbours' mu)
      const int row = ys + r;
      if (zo >= zs && row >= yb && row < yb + H && row < ny && mine)
        o[(long long)row * nx] = ch_out(v, final != 0);
      em[r] = e;
      esm[r] = f;
      sm[r] = sn;
      qm[r] = qn;
      mz[r] = mu[r + 1];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      c2[r] = cz[r];
      cz[r] = in[r + 1];
    }
  }
}

__global__ __launch_bounds__(256) void k_ch_init(const uint8_t* __restrict__ s,
                                                 float* __restrict__ c, int N) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < N) c[k] = s[k] ? 1.0f : -1.0f;
}

__global__ __launch_bounds__(256) void k_ch_final(const float* __restrict__ c,
                                                  float* __restrict__ phi0, int N) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < N) phi0[k] = fminf(fmaxf(0.5f * (1.0f + c[k]), 0.0f), 1.0f);
}

size_t plane_bytes(long long n) { return ((size_t)n * 4 + 255) / 256 * 256; }

int ceil_div(int a, int b) { return (int)(((long long)a + b - 1) / b); }

// Longest sides the passes take: the coordinates of a strip and its overlap stay ints.
constexpr int kMaxSide[3] = {0x7FFFFFFF - 63, 0x7FFFFFFF - 15, 0x7FFFFFFF - 3};

// Checks shared by both entry points.
int ch_validate(const lbf_ch_params* p, int32_t iterations) {
  if (!p) return fail(LBF_EINVAL, "NULL argument");
  if (p->nx < 1 || p->ny < 1 || p->nz < 1)
    return fail(LBF_EINVAL, "image size %d x %d x %d", p->nx, p->ny, p->nz);
  const long long n = (long long)p->nx * p->ny * p->nz;
  if (n > kMaxNodesCH) return fail(LBF_EINVAL, "image of %lld nodes exceeds 2^31 - 1", n);
  if (iterations < 0) return fail(LBF_EINVAL, "iterations %d", iterations);
  if (!(p->A >= 0.0) || !(p->kappa >= 0.0) || !(p->mobility >= 0.0) || !(p->dt > 0.0) ||
      !std::isfinite(p->A) || !std::isfinite(p->kappa) || !std::isfinite(p->mobility) ||
      !std::isfinite(p->dt))
    return fail(LBF_EINVAL, "A, kappa, mobility must be >= 0 and dt > 0, all finite");
  const double lmax = 16.0 / 3.0;
  const double amp = p->dt * p->mobility * lmax * (2.0 * p->A + p->kappa * lmax);
  if (amp > 2.0)
    return fail(LBF_EINVAL, "dt = %g is outside the explicit scheme's stability bound "
                            "(dt M 16/3 (2 A + kappa 16/3) = %g > 2)", p->dt, amp);
  return LBF_OK;
}

bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

// One pass of T steps over a 2D plane.
template <int T>
int ch_pass2(const ChGeo& G, const float* c, const uint8_t* img, float* cn, float A, float kappa,
             float dtM, bool final, hipStream_t st) {
  constexpr int W = 64 * kV2 - 4 * T;
  const int nsx = ceil_div(G.n[0], W);
  const long long want = ((long long)G.n[1] * nsx + kWaves2 - 1) / kWaves2;
  const int rows = (int)std::max(8LL, (want + 3) / 4 * 4);
  const int nstrips = nsx * ceil_div(G.n[1], rows);
  hipLaunchKernelGGL((k_ch_step2<T, kV2, kPF2>), dim3(ceil_div(nstrips, 4)), dim3(256), 0, st, G, c, img,
                     cn, A, kappa, dtM, rows, nsx, nstrips, final ? 1 : 0);
  HIP_TRY(hipGetLastError());
  return LBF_OK;
}

int ch_pass3(const ChGeo& G, const float* c, const uint8_t* img, float* cn, float A, float kappa,
             float dtM, bool final, hipStream_t st) {
  const int nsx = ceil_div(G.n[0], 60), nsy = ceil_div(G.n[1], 4 * kR3 - 2);
  const long long cols = 4LL * nsx * nsy;   // wavefronts side by side
  const int slabs = (int)std::max(4LL, ((long long)G.n[2] * cols + kWaves3 - 1) / kWaves3);
  const int nblk = nsx * nsy * ceil_div(G.n[2], slabs);
  hipLaunchKernelGGL((k_ch_step3<kR3>), dim3(nblk), dim3(256), 0, st, G, c, img, cn, A, kappa, dtM,
                     slabs, nsx, nsy, final ? 1 : 0);
  HIP_TRY(hipGetLastError());
  return LBF_OK;
}

// The smoothing itself on two planes c0, c1 of at least plane_bytes(n) each
// (c1 also stages a host image and, when phi0 is host memory, the result).
// Stream-ordered; synchronises only when host memory is read or written.
int ch_run(const lbf_ch_params* p, const uint8_t* solid, bool solid_on_device, float* phi0,
           bool phi0_on_device, int32_t iterations, hipStream_t st, float* c0, float* c1) {
  if (iterations > 0 && (p->nx > kMaxSide[0] || p->ny > kMaxSide[1] || p->nz > kMaxSide[2]))
    return fail(LBF_EINVAL, "image of %d x %d x %d nodes: sides up to %d, %d, %d", p->nx, p->ny,
                p->nz, kMaxSide[0], kMaxSide[1], kMaxSide[2]);
  const int N = p->nx * p->ny * p->nz;
  float* c[2] = {c0, c1};
  const int nb = (int)(((long long)N + 255) / 256);
  const ChGeo G{{p->nx, p->ny, p->nz},
                {p->periodic[0] ? 1 : 0, p->periodic[1] ? 1 : 0, p->periodic[2] ? 1 : 0}};
  const bool is3d = p->nz > 1;
  const float A = (float)p->A, kap = (float)p->kappa, dtM = (float)(p->dt * p->mobility);
  const uint8_t* s = solid;
  if (!solid_on_device) {
    HIP_TRY(hipMemcpyAsync(c[1], solid, (size_t)N, hipMemcpyHostToDevice, st));
    s = (const uint8_t*)c[1];
  }
  // The first pass reads the image and the last one writes phi0, unless the
  // caller's buffers overlap each other or the planes (then c is copied in
  // and out, as for no steps at all).
  const size_t pb = (size_t)N * 4;
  const bool apart = !overlap(s, (size_t)N, phi0, pb) && !overlap(s, (size_t)N, c0, pb) &&
                     !overlap(phi0, pb, c0, pb) && !overlap(phi0, pb, c1, pb);
  const bool fused = iterations > 0 && (apart || !phi0_on_device);
  int cur = 0;   // the plane that holds c (fused: after the first pass)
  if (!fused) {
    hipLaunchKernelGGL(k_ch_init, dim3(nb), dim3(256), 0, st, s, c[0], N);
    HIP_TRY(hipGetLastError());
  }
  for (int it = 0; it < iterations;) {
    const bool first = fused && it == 0;
    const int T = is3d ? 1 : std::min(kT2, iterations - it);
    it += T;
    const bool last = fused && it == iterations;
    const int nxt = first ? 0 : 1 - cur;
    float* out = last && phi0_on_device ? phi0 : c[nxt];
    const uint8_t* img = first ? s : nullptr;
    int rc;
    if (is3d) rc = ch_pass3(G, c[cur], img, out, A, kap, dtM, last, st);
    else if (T == 1) rc = ch_pass2<1>(G, c[cur], img, out, A, kap, dtM, last, st);
    else if (T == 2) rc = ch_pass2<2>(G, c[cur], img, out, A, kap, dtM, last, st);
    else if (T == 3) rc = ch_pass2<3>(G, c[cur], img, out, A, kap, dtM, last, st);
    else rc = ch_pass2<4>(G, c[cur], img, out, A, kap, dtM, last, st);
    if (rc) return rc;
    cur = nxt;
  }
  const float* res = c[cur];
  if (!fused) {
    float* dst = phi0_on_device ? phi0 : c[1 - cur];
    hipLaunchKernelGGL(k_ch_final, dim3(nb), dim3(256), 0, st, (const float*)c[cur], dst, N);
    HIP_TRY(hipGetLastError());
    res = dst;
  }
  if (!phi0_on_device) HIP_TRY(hipMemcpyAsync(phi0, res, pb, hipMemcpyDeviceToHost, st));
  if (!phi0_on_device || !solid_on_device) HIP_TRY(hipStreamSynchronize(st));
  return LBF_OK;
}

// Address of `scratch` per device, looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch[kMaxDevices];

int scratch_on_current_device(float** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(LBF_EINVAL, "device %d: the scratch table holds devices 0..%d", dev,
                kMaxDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(LBF_EHIP, "hipGetSymbolAddress(scratch) on device %d failed: %s", dev,
                  hipGetErrorString(e));
    g_scratch[dev] = (float*)p;
  }
  *out = g_scratch[dev];
  return LBF_OK;
}

}  // namespace

extern "C" {

size_t lbf_ch_workspace_bytes(int32_t nx, int32_t ny, int32_t nz) {
  if (nx < 1 || ny < 1 || nz < 1) return 0;
  const long long n = (long long)nx * ny * nz;
  if (n > kMaxNodesCH) return 0;
  // c, two ping-pong planes; a host image is staged in the second one
  return 2 * plane_bytes(n);
}

int lbf_ch_smooth(const lbf_ch_params* p, const uint8_t* solid, int32_t solid_on_device,
                  float* phi0, int32_t phi0_on_device, int32_t iterations, void* stream,
                  void* workspace, size_t workspace_bytes) {
  if (!solid || !phi0) return fail(LBF_EINVAL, "NULL argument");
  int rc = ch_validate(p, iterations);
  if (rc != LBF_OK) return rc;
  const long long n = (long long)p->nx * p->ny * p->nz;
  const size_t need = lbf_ch_workspace_bytes(p->nx, p->ny, p->nz);
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  bool owns = false;
  if (ws) {
    if (workspace_bytes < need || (uintptr_t)ws % 256)
      return fail(LBF_ENOMEM, "workspace too small or not 256-byte aligned");
  } else {
    if (hipMalloc((void**)&ws, need) != hipSuccess) return fail(LBF_ENOMEM, "hipMalloc failed");
    owns = true;
  }
  const size_t pb = plane_bytes(n);
  rc = ch_run(p, solid, solid_on_device != 0, phi0, phi0_on_device != 0, iterations, st,
              (float*)ws, (float*)(ws + pb));
  if (owns) {
    (void)hipStreamSynchronize(st);
    (void)hipFree(ws);
  }
  return rc;
}

size_t lbf_ch_noalloc_max_nodes(void) { return (size_t)kStaticNodesCH; }

int lbf_ch_smooth_noalloc(const lbf_ch_params* p, const uint8_t* solid_dev, float* phi0_dev,
                          int32_t iterations, void* stream) {
  if (!solid_dev || !phi0_dev) return fail(LBF_EINVAL, "NULL argument");
  int rc = ch_validate(p, iterations);
  if (rc != LBF_OK) return rc;
  const long long n = (long long)p->nx * p->ny * p->nz;
  if (n > kStaticNodesCH)
    return fail(LBF_EINVAL, "image of %lld nodes exceeds the allocation-free limit of %lld "
                            "nodes (use lbf_ch_smooth with a workspace)", n, kStaticNodesCH);
  float* c = nullptr;
  rc = scratch_on_current_device(&c);
  if (rc != LBF_OK) return rc;
  // every node of both planes that the smoothing reads is written first
  // (k_ch_init fills c0 from the image), so nothing needs clearing
  return ch_run(p, solid_dev, true, phi0_dev, true, iterations, (hipStream_t)stream, c,
                c + plane_bytes(n) / sizeof(float));
}

}  // extern "C"
