// Coupled steps on patches: one to three steps of a patch of the lattice per
// workgroup, one node per lane, the state in registers and LDS between them.
//
// A strip (step_strip) forms the moments of a row from three rows of loads, waits for
// memory once per row, and writes and reads the whole state once per step; below about
// a million nodes it has too few rows to march for the waits to be hidden, and on a
// lattice whose rows are not a multiple of the memory's lines each access is split.
// A patch loads the post-collision state of its TX x TY nodes once, every lane its own
// node (no shifted loads), and from then on streams through LDS: the moving
// populations are exchanged there, then the moments the stencils take.  Each step uses
// up two rings of nodes (the pull reaches one node, the stencil of pulled moments
// another), so K steps deliver the inner (TX - 4 K) x (TY - 4 K) nodes; the rings are
// computed by the neighbouring patches as well.
//
// What bounds it is the vector instructions (76 % busy at 2048^2, 1410 per node and step;
// under MRT 83 %, 1860), of the nodes computed twice too: at 32 x 16 and two steps 1.67
// collisions and 2.33 pulls per node and step delivered, rows of wholly outer nodes
// skipped.  A pair moves 299 + 136 bytes a node (the rings are half found in L2; 148 +
// 136 without them), 4.5 TB/s.  2048^2: 201 us a step against 233 of strips, which move
// 301 bytes in each.
// Patches of 32 x 32 and 64 x 16 compute less twice, but one fills a compute unit and
// nothing runs beside its barriers and loads (1400 x 1000: 99 and 95 us against 75).
//
// The same functions give the same bits as step_strip.
#pragma once
#include "lbf_step.hpp"

namespace lbf {

// Plain stores, not the strips' policy: a patch's rows are 24 nodes, so that the
// cache puts the lines of neighbouring patches together, and a small state is found
// there by the next launch (plain, non-temporal, SC1, both; us a step: 455 x 318 11.4,
// 11.8, 11.1, 12.6; 1000 x 700 36.3, 40.3, 37.4, 45.3; 1400 x 1000 76, 76, 88, 89; a
// recorded pair at 1024^2 145, 218, 171, 263).
constexpr int kPatchPolicy = 0;

template <int TX, int TY>
struct PatchShared {
  static constexpr int N = TX * TY;
  float f[8][N], g[8][N], h[8][N];   // moving populations of the lane's node
  float m[3][N];                     // phi, f_s, rho
  float p[N];                        // p of the step before
  float u[2][N];                     // velocity of the step before
};

// A lane's links: which cross a wall, and what the node on the other side gives.
struct PatchWalls {
  bool wl, wr, wb, wt, any;
};

__device__ __forceinline__ bool patch_wall(const PatchWalls& w, int i) {
  const bool y = cy(i) > 0 ? w.wb : (cy(i) < 0 ? w.wt : false);
  const bool x = cx(i) > 0 ? w.wl : (cx(i) < 0 ? w.wr : false);
  return y || x;
}

// Pulled moving populations of lane t: the neighbours', or the node's own in the
// opposite direction across a wall (half-way bounce-back).
template <int TX, int N>
__device__ __forceinline__ void patch_pull(const float (*pop)[N], int t, const PatchWalls& w,
                                           float* v) {
#pragma unroll
  for (int i = 1; i < 9; ++i) v[i] = pop[i - 1][t - cx(i) - cy(i) * TX];
  if (w.any) {
#pragma unroll
    for (int i = 1; i < 9; ++i)
      if (patch_wall(w, i)) v[i] = pop[opp(i) - 1][t];
  }
}

// The enthalpy's, with anti-bounce-back at the temperature of a Dirichlet wall
// (a link through a bottom/top wall takes that wall even at a corner).
template <int TX, int N>
__device__ __forceinline__ void patch_pull_h(const Geo& G, const Phys& ph, const Bufs& B,
                                             const float (*pop)[N], int t, int x, int y,
                                             const PatchWalls& w, float* v) {
#pragma unroll
  for (int i = 1; i < 9; ++i) v[i] = pop[i - 1][t - cx(i) - cy(i) * TX];
  if (w.any) {
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      if (patch_wall(w, i)) {
        const float hb = pop[opp(i) - 1][t];
        const bool wy = cy(i) > 0 ? w.wb : (cy(i) < 0 ? w.wt : false);
        const int wall = wy ? (cy(i) > 0 ? 0 : 1) : (cx(i) > 0 ? 2 : 3);
        if ((G.tmask >> wall) & 1) {
          const float Tw = B.wallT[wall * B.wstride + (wall < 2 ? x : y)];
          v[i] = -hb + 2.0f * wgt(i) * ph.Eref * Tw;
        } else {
          v[i] = hb;
        }
      }
    }
  }
}

// Pulls the phase-field and enthalpy populations from LDS again when the collision
// comes to them: held from the moments on, they and the flow's would not fit 128
// registers, and two patches share a compute unit (1000 x 700: 66 -> 46 us a step).
template <int TX, int N>
struct PatchLate {
  const Geo& G;
  const Phys& ph;
  const Bufs& B;
  const float (*g)[N];
  const float (*h)[N];
  const PatchWalls& w;
  int t, x, y;
  __device__ __forceinline__ void phase(float* v) const {
    __builtin_amdgcn_sched_barrier(0);
    patch_pull<TX, N>(g, t, w, v);
  }
  __device__ __forceinline__ void enthalpy(float* v) const {
    __builtin_amdgcn_sched_barrier(0);
    patch_pull_h<TX, N>(G, ph, B, h, t, x, y, w, v);
  }
};

// Where a recorded run's states and moments lie: the state of step s and the phi,
// f_s, rho it was stepped from, `state` and `mom` floats apart (0: not recorded).
struct PatchRecord {
  size_t state, mom;
};

// Patch (bx, by) of the lattice, K steps of the state in A.  Stores the last step's
// state, or with RECORD every step's, and the moments each was stepped from.
template <int TX, int TY, bool MRT, bool RECORD>
__device__ __forceinline__ void patch_steps(const Geo& G, const Phys& ph, BufArgs A,
                                            PatchRecord rec, int bx, int by, int K,
                                            PatchShared<TX, TY>& sh) {
  const Bufs B = make_bufs(A, G);
  constexpr int N = TX * TY;
  const int t = threadIdx.x;
  const int lx = t % TX, ly = t / TX;
  const int ix = TX - 4 * K, iy = TY - 4 * K;
  int x = bx * ix - 2 * K + lx, y = by * iy - 2 * K + ly;
  // nodes beyond a wall do not exist; across a periodic side they are the
  // wrapped ones (a small lattice may appear more than once in a patch)
  const bool act = (G.px || (x >= 0 && x < G.nx)) && (G.py || (y >= 0 && y < G.ny));
  const bool own = x < G.nx && y < G.ny;   // with its ring: delivered by this patch
  if (G.px) {
    x %= G.nx;
    if (x < 0) x += G.nx;
  }
  if (G.py) {
    y %= G.ny;
    if (y < 0) y += G.ny;
  }
  const int ring = min(min(lx, TX - 1 - lx), min(ly, TY - 1 - ly));
  const bool flow = ph.phi_src_flow != 0;
  const int P = G.P;
  const int k = act ? nidx(G, x, y) : 0;

  // (a lane outside the ring of a step keeps nothing of it: left unset there, so
  // that old values do not occupy registers beside the new ones)
  float fv[9], gv[9], hv[9];
  float fsp, Qp, jxp, jyp, pp, ghi, hhi, uxp, uyp;
  float phi0 = 0.0f, cth = 0.0f, lap0 = 0.0f, thold = 0.0f;
  if (act) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      fv[i] = ldp(B.fin, i, P, k);
      gv[i] = ldp(B.gin, i, P, k);
      hv[i] = ldp(B.hin, i, P, k);
    }
    fsp = ldp(B.lin, LAG_FS, P, k);
    Qp = ldp(B.lin, LAG_Q, P, k);
    jxp = ldp(B.lin, LAG_JX, P, k);
    if (!flow) jyp = ldp(B.lin, LAG_JY, P, k);
    pp = ldp(B.lin, LAG_P, P, k);
    const uint32_t hp = __builtin_bit_cast(uint32_t, ldp(B.lin, LAG_GHI, P, k));
    ghi = unpack_ghi(hp);
    hhi = unpack_hhi(hp);
    if (flow) {
      uxp = ldp(B.lin, LAG_UX, P, k);
      uyp = ldp(B.lin, LAG_UY, P, k);
    }
    phi0 = ldp(B.stat, ST_PHI0, P, k);
    cth = ldp(B.stat, ST_CTH, P, k);
    lap0 = ldp(B.stat, ST_LAP0, P, k);
    if (ph.subfix == 2) thold = ldp(B.stat, ST_THOLD, P, k);
  }
  // the lane's populations, p and velocity, for its neighbours
  auto publish = [&]() {
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      sh.f[i - 1][t] = fv[i];
      sh.g[i - 1][t] = gv[i];
      sh.h[i - 1][t] = hv[i];
    }
    sh.p[t] = pp;
    if (flow) {
      sh.u[0][t] = uxp;
      sh.u[1][t] = uyp;
    }
  };
  // the nodes this patch delivers
  const bool inner = act && own && ring >= 2 * K;
  auto store = [&](const Bufs& B) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      stp<kPatchPolicy>(B.fout, i, P, k, fv[i]);
      stp<kPatchPolicy>(B.gout, i, P, k, gv[i]);
      stp<kPatchPolicy>(B.hout, i, P, k, hv[i]);
    }
    stp<kPatchPolicy>(B.lout, LAG_FS, P, k, fsp);
    stp<kPatchPolicy>(B.lout, LAG_Q, P, k, Qp);
    stp<kPatchPolicy>(B.lout, LAG_JX, P, k, jxp);
    if (!flow) stp<kPatchPolicy>(B.lout, LAG_JY, P, k, jyp);
    stp<kPatchPolicy>(B.lout, LAG_P, P, k, pp);
    stp<kPatchPolicy>(B.lout, LAG_GHI, P, k, __builtin_bit_cast(float, pack_hi(ghi, hhi)));
    if (flow) {
      stp<kPatchPolicy>(B.lout, LAG_UX, P, k, uxp);
      stp<kPatchPolicy>(B.lout, LAG_UY, P, k, uyp);
    }
  };
  if (act) publish();
  __syncthreads();
  for (int s = 0; s < K; ++s) {
    // opaque to the compiler in every step: a product of them formed once, ahead
    // of the loop, would not be fused with the sum it belongs to, and the walls'
    // addresses, kept over the loop, would spill (1000 x 700: 57 -> 46 us a step)
    asm volatile("" : "+v"(phi0), "+v"(cth), "+v"(lap0), "+v"(x), "+v"(y), "+v"(thold));
    // links across walls, and the stencil's neighbours (the node's own row or
    // column beyond a wall: the mirror ghost)
    PatchWalls w;
    w.wl = !G.px && x == 0;
    w.wr = !G.px && x == G.nx - 1;
    w.wb = !G.py && y == 0;
    w.wt = !G.py && y == G.ny - 1;
    w.any = w.wl || w.wr || w.wb || w.wt;
    const int nb_x[3] = {w.wl ? 0 : -1, 0, w.wr ? 0 : 1};
    const int nb_y[3] = {w.wb ? 0 : -TX, 0, w.wt ? 0 : TX};
    const bool pulls = act && ring >= 2 * s + 1, collides = act && ring >= 2 * s + 2;
    Mom m;
    if (pulls) {
      NodeIn in;
      in.g[0] = gv[0];
      in.h[0] = hv[0];
      patch_pull<TX, N>(sh.g, t, w, in.g);
      patch_pull_h<TX, N>(G, ph, B, sh.h, t, x, y, w, in.h);
      in.fsp = fsp;
      in.Qp = Qp;
      in.phi0 = phi0;
      in.ghi = ghi;
      in.hhi = hhi;
      in.pprev = pp;
      in.dlag = 0.0f;
      if (flow) {
        float ux[9], uy[9];
#pragma unroll
        for (int i = 1; i < 9; ++i) {
          const int q = t + nb_x[cx(i) + 1] + nb_y[cy(i) + 1];
          ux[i] = cx(i) ? sh.u[0][q] : 0.0f;
          uy[i] = cy(i) ? sh.u[1][q] : 0.0f;
        }
        in.dlag = div9(ux, uy);
      }
      float st[4];
      node_finish(ph, in, m, st);
      sh.m[0][t] = st[0];
      sh.m[1][t] = st[1];
      sh.m[2][t] = st[2];
    }
    __syncthreads();
    if (collides) {
      Stencil S;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        const int q = t + nb_x[cx(i) + 1] + nb_y[cy(i) + 1];
        S.phi[i] = sh.m[0][q];
        S.fs[i] = sh.m[1][q];
        S.rho[i] = sh.m[2][q];
        S.p[i] = sh.p[q];
      }
      patch_pull<TX, N>(sh.f, t, w, fv);
      const float jx0 = flow ? jxp * uxp : jxp, jy0 = flow ? jxp * uyp : jyp;
      Post o;
      const PatchLate<TX, N> late{G, ph, B, sh.g, sh.h, w, t, x, y};
      collide_node<true, MRT>(ph, m, S, phi0, cth, lap0, Qp, jx0, jy0, hhi, thold, fv, gv, hv, o,
                              late);
      fsp = m.fs;
      Qp = o.Q;
      pp = o.p;
      ghi = o.ghi;
      hhi = o.hhi;
      if (flow) {
        jxp = m.phi;
        uxp = o.ux;
        uyp = o.uy;
      } else {
        jxp = o.jx;
        jyp = o.jy;
      }
    }
    if (RECORD && inner) {
      BufArgs C = A;
      C.dout += s * rec.state;
      C.lout += s * rec.state;
      C.fields += s * rec.mom;
      const Bufs D = make_bufs(C, G);
      stp<kPatchPolicy>(D.fields, 0, P, k, m.phi);
      stp<kPatchPolicy>(D.fields, 1, P, k, m.fs);
      stp<kPatchPolicy>(D.fields, 2, P, k, m.rho);
      store(D);
    }
    if (s + 1 < K) {
      __syncthreads();
      if (collides) publish();
      __syncthreads();
    }
  }
  if (!RECORD && inner) store(B);
}

constexpr int kPatchX = 32, kPatchY = 16, kPatchSteps = 2;

// 1D grid of nbx * nby patches; four wavefronts per SIMD (two patches per compute
// unit) hold the registers to 128.
template <bool MRT, bool RECORD = false>
__global__ __launch_bounds__(kPatchX* kPatchY) __attribute__((amdgpu_waves_per_eu(4, 8))) void
patch_kernel(Geo G, Phys ph, BufArgs A, PatchRecord rec, int K, int nbx) {
  __shared__ PatchShared<kPatchX, kPatchY> sh;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  patch_steps<kPatchX, kPatchY, MRT, RECORD>(G, ph, A, rec, t % nbx, t / nbx, K, sh);
}

// The same on the lattices of a batch: one workgroup per (instance, patch) of the work
// list, two steps.
template <bool MRT>
__global__ __launch_bounds__(kPatchX* kPatchY) __attribute__((amdgpu_waves_per_eu(4, 8))) void
batch_patch_kernel(const InstDesc* __restrict__ D, const int2* __restrict__ items, int parity) {
  __shared__ PatchShared<kPatchX, kPatchY> sh;
  const int2 item = items[xcd_tile(blockIdx.x, gridDim.x)];
  const Geo G = D[item.x].G;
  const Phys ph = D[item.x].ph;
  const BufArgs A = D[item.x].A[parity];
  const int nbx = D[item.x].npx;
  patch_steps<kPatchX, kPatchY, MRT, false>(G, ph, A, PatchRecord{0, 0}, item.y % nbx,
                                            item.y / nbx, kPatchSteps, sh);
}

}  // namespace lbf
