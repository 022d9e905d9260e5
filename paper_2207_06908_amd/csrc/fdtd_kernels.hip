// fdtd_kernels.hip -- HIP kernels of the Yee FDTD step for gfx950.
//
// Layout (all device memory lives in the caller's workspace): each field
// component is an nx*ny*nz array, x fastest, holding the component owned by
// node (i, j, k).  Values on the upper walls (index n along an axis) are not
// stored: they are the zero tangential E of a perfect conductor or the zero
// normal H next to it, so reads past the last node return 0.  Each node
// carries a 1- or 2-byte coefficient class id; the class table holds the 9
// coefficients of the node's six components.
//
// Variants:
//   split  two passes (H over the grid, then E), in place;
//   fused  one pass per step over x-y tiles marching up z; each block
//          recomputes the H it needs on a one-node low-side halo; reads one
//          field set and writes the other;
//   tb2    one pass per two steps (temporal blocking) in one launch: 60 x TY
//          output tiles in 64 x (TY+4) regions, four stages per plane, each
//          tile by the code of the CPML slabs it reaches, probes included.
// fused and tb2 also run batched over many grids, and fused as tile lists
// grouped by those slabs.  All evaluate every component through h_core /
// e_core of fdtd_tile.h (with the arithmetic of yee_update.h) and are compiled with FP
// contraction off, so they agree bit for bit.
#include <hip/hip_runtime.h>

#include "fdtd_dev.h"
#include "fdtd_march.h"
#include "fdtd_tile.h"
#include "yee_update.h"

namespace mi355fdtd {

// ---------------------------------------------------------------------------
// split variant: two in-place passes
// ---------------------------------------------------------------------------

template <typename T, typename CI, bool PML, int NB>
__global__ __launch_bounds__(NB) void k_h_split(GridView<T> g) {
  // node of the xy plane, x fastest.  On small planes (NB 256) each XCD takes
  // a contiguous band of the plane, so a block's neighbour row was just read
  // into the same L2 (5% faster on a 100 x 100 plane, 5.5% slower on a
  // 512 x 512 one, where the blocks keep their dealt order).
  const unsigned t =
      (unsigned)(NB == 256 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x) * (unsigned)NB + threadIdx.x;
  if (t >= (unsigned)g.sxy) return;
  const int i = (int)(t % (unsigned)g.nx), j = (int)(t / (unsigned)g.nx);
  const int k = blockIdx.y;
  const unsigned n = (unsigned)i + (unsigned)g.nx * ((unsigned)j + (unsigned)g.ny * (unsigned)k);
  const T* cf = g.ctab + (int)ldg((const CI*)g.cls, n) * K_STRIDE;
  const T ex = ldg(g.fi[0], n), ey = ldg(g.fi[1], n), ez = ldg(g.fi[2], n);
  const T ex_j = (j + 1 < g.ny) ? ldg(g.fi[0], n + (unsigned)g.nx) : T(0);
  const T ex_k = (k + 1 < g.nz) ? ldg(g.fi[0], n + (unsigned)g.sxy) : T(0);
  const T ey_i = (i + 1 < g.nx) ? ldg(g.fi[1], n + 1) : T(0);
  const T ey_k = (k + 1 < g.nz) ? ldg(g.fi[1], n + (unsigned)g.sxy) : T(0);
  const T ez_i = (i + 1 < g.nx) ? ldg(g.fi[2], n + 1) : T(0);
  const T ez_j = (j + 1 < g.ny) ? ldg(g.fi[2], n + (unsigned)g.nx) : T(0);
  const T hold[3] = {ldg(g.fi[3], n), ldg(g.fi[4], n), ldg(g.fi[5], n)};
  T h[3];
  h_point<T, PML>(g, i, j, k, cf, ex, ey, ez, ex_j, ex_k, ey_i, ey_k, ez_i, ez_j, hold, true, h);
  stg(g.fo[3], n, h[0]);
  stg(g.fo[4], n, h[1]);
  stg(g.fo[5], n, h[2]);
}

template <typename T, typename CI, bool PML, int NB>
__global__ __launch_bounds__(NB) void k_e_split(GridView<T> g, int step) {
  step = gstep(g, step);
  // node of the xy plane, x fastest.  On small planes (NB 256) each XCD takes
  // a contiguous band of the plane, so a block's neighbour row was just read
  // into the same L2 (5% faster on a 100 x 100 plane, 5.5% slower on a
  // 512 x 512 one, where the blocks keep their dealt order).
  const unsigned t =
      (unsigned)(NB == 256 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x) * (unsigned)NB + threadIdx.x;
  if (t >= (unsigned)g.sxy) return;
  const int i = (int)(t % (unsigned)g.nx), j = (int)(t / (unsigned)g.nx);
  const int k = blockIdx.y;
  const unsigned n = (unsigned)i + (unsigned)g.nx * ((unsigned)j + (unsigned)g.ny * (unsigned)k);
  const T* cf = g.ctab + (int)ldg((const CI*)g.cls, n) * K_STRIDE;
  const T hx = ldg(g.fi[3], n), hy = ldg(g.fi[4], n), hz = ldg(g.fi[5], n);
  const T hx_j = (j > 0) ? ldg(g.fi[3], n - (unsigned)g.nx) : T(0);
  const T hx_k = (k > 0) ? ldg(g.fi[3], n - (unsigned)g.sxy) : T(0);
  const T hy_i = (i > 0) ? ldg(g.fi[4], n - 1) : T(0);
  const T hy_k = (k > 0) ? ldg(g.fi[4], n - (unsigned)g.sxy) : T(0);
  const T hz_i = (i > 0) ? ldg(g.fi[5], n - 1) : T(0);
  const T hz_j = (j > 0) ? ldg(g.fi[5], n - (unsigned)g.nx) : T(0);
  const T eold[3] = {ldg(g.fi[0], n), ldg(g.fi[1], n), ldg(g.fi[2], n)};
  T e[3];
  const SrcRange sr = src_node(g, i, j, k);
  e_point<T, PML>(g, i, j, k, n, cf, hx, hy, hz, hx_j, hx_k, hy_i, hy_k, hz_i, hz_j, eold, step, e, sr.lo, sr.hi);
  stg(g.fo[0], n, e[0]);
  stg(g.fo[1], n, e[1]);
  stg(g.fo[2], n, e[2]);
}

// Split E update in Debye media: the plain update, then the pole currents.
// Nodes whose class has no pole term (air, walls, wire edges) skip them, so
// their J stays 0 without traffic.
template <typename T, typename CI, bool PML, int NB>
__global__ __launch_bounds__(NB) void k_e_split_debye(GridView<T> g, DebyeView<T> d, int step) {
  step = gstep(g, step);
  // node of the xy plane, x fastest.  On small planes (NB 256) each XCD takes
  // a contiguous band of the plane, so a block's neighbour row was just read
  // into the same L2 (5% faster on a 100 x 100 plane, 5.5% slower on a
  // 512 x 512 one, where the blocks keep their dealt order).
  const unsigned t =
      (unsigned)(NB == 256 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x) * (unsigned)NB + threadIdx.x;
  if (t >= (unsigned)g.sxy) return;
  const int i = (int)(t % (unsigned)g.nx), j = (int)(t / (unsigned)g.nx);
  const int k = blockIdx.y;
  const unsigned n = (unsigned)i + (unsigned)g.nx * ((unsigned)j + (unsigned)g.ny * (unsigned)k);
  const int cid = (int)ldg((const CI*)g.cls, n);
  const T* cf = g.ctab + cid * K_STRIDE;
  const T hx = ldg(g.fi[3], n), hy = ldg(g.fi[4], n), hz = ldg(g.fi[5], n);
  const T hx_j = (j > 0) ? ldg(g.fi[3], n - (unsigned)g.nx) : T(0);
  const T hx_k = (k > 0) ? ldg(g.fi[3], n - (unsigned)g.sxy) : T(0);
  const T hy_i = (i > 0) ? ldg(g.fi[4], n - 1) : T(0);
  const T hy_k = (k > 0) ? ldg(g.fi[4], n - (unsigned)g.sxy) : T(0);
  const T hz_i = (i > 0) ? ldg(g.fi[5], n - 1) : T(0);
  const T hz_j = (j > 0) ? ldg(g.fi[5], n - (unsigned)g.nx) : T(0);
  const T eold[3] = {ldg(g.fi[0], n), ldg(g.fi[1], n), ldg(g.fi[2], n)};
  T e[3];
  const SrcRange sr = src_node(g, i, j, k);
  e_point<T, PML>(g, i, j, k, n, cf, hx, hy, hz, hx_j, hx_k, hy_i, hy_k, hz_i, hz_j, eold, step, e, sr.lo, sr.hi);
  debye_point(d, cid, n, eold, e);
  stg(g.fo[0], n, e[0]);
  stg(g.fo[1], n, e[1]);
  stg(g.fo[2], n, e[2]);
}


template <typename T, typename CI, bool PML, int TX, int TY>
__global__ __launch_bounds__(TX * TY) void k_fused(GridView<T> g, int step, int kz, int ntx, int nty) {
  step = gstep(g, step);
  __shared__ FusedSmem<T, TX, TY> sm;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tile_x = tile % ntx, rest = tile / ntx;
  const int k0 = (rest / nty) * kz;
  fused_tile<T, CI, PML, TX, TY>(g, sm, tile_x * TX, (rest % nty) * TY, k0, min(k0 + kz, g.nz), step);
}

// One grid, tile list: block b takes tile (i0, j0, k0, k1).  The host splits
// a grid with a CPML into tiles clear of every slab (including the recomputed
// halo and the prologue plane), which run the lean instantiation, and the
// rest, which runs the CPML one.
template <typename T, typename CI, bool PML, int TX, int TY, int AX>
__global__ __launch_bounds__(TX * TY) void k_fused_list(GridView<T> g, const int4* __restrict__ tiles, int step) {
  step = gstep(g, step);
  __shared__ FusedSmem<T, TX, TY> sm;
  const int4 t = tiles[xcd_tile(blockIdx.x, gridDim.x)];
  fused_tile<T, CI, PML, TX, TY, AX>(g, sm, t.x, t.y, t.z, t.w, step);
}

// Batched: one block per entry of a tile list spanning many grids; each
// grid's view is read from a device table (one table per field-set parity).
// The step index is a device counter (plus a per-launch offset) so that a
// captured graph of several steps can be replayed unchanged.
template <typename T, typename CI, bool PML, int TX, int TY>
__global__ __launch_bounds__(TX * TY) void k_fused_batch(const GridView<T>* __restrict__ views,
                                                        const int4* __restrict__ tiles,
                                                        const int* __restrict__ d_step, int offset) {
  __shared__ FusedSmem<T, TX, TY> sm;
  const int4 t = tiles[xcd_tile(blockIdx.x, gridDim.x)];  // (grid, i0, j0, k0 | kz << 16)
  const GridView<T>& g = views[t.x];
  const int k0 = t.w & 0xffff, kz = t.w >> 16;
  fused_tile<T, CI, PML, TX, TY>(g, sm, t.y, t.z, k0, min(k0 + kz, g.nz), *d_step + offset);
}

// ---------------------------------------------------------------------------
// temporally blocked variant: two steps per pass.  Most tiles are those of
// fdtd_march.h; this one (tb2_tile), a plane of every stage at a time, is that
// of FP64 grids in the CPML slabs and of grids whose classes do not fit March's
// table in LDS.
//
// Block = TY + 4 waves; wave v, lane u own the point x = i0 - 2 + u,
// y = j0 - 2 + v of a 64 x (TY + 4) region around the 60 x TY output tile
// [i0, i0+60) x [j0, j0+TY).  Each point is updated by the same thread in
// every stage it belongs to (the dependency cone shrinks by one node per
// half step on the high or low side):
//   A  H^{n+1/2} on u <= 62, v <= TY+2            (from E^n, H^{n-1/2})
//   B  E^{n+1}   on 1 <= u <= 62, 1 <= v <= TY+2  (sources of step n)
//   C  H^{n+3/2} on 1 <= u <= 61, 1 <= v <= TY+1
//   D  E^{n+2}   on 2 <= u <= 61, 2 <= v <= TY+1  (the tile; sources n+1)
// Marching up z, iteration k does A and B of plane k and C and D of plane
// k-1; the chunk [k0, k1) starts its pipeline at k0-2.  Neighbours are read
// from LDS planes; a point's own values of earlier planes stay in
// registers, as does its CPML state between the two steps.  Only E^{n+2},
// H^{n+3/2} and the CPML state after two steps reach memory (output set).
// ---------------------------------------------------------------------------

template <typename T, int TY>
struct TB2Smem {
  static constexpr int R = TY + 4;
  static constexpr int PZ = 512 / sizeof(T);  // longest z profile row held here (2 npml)
  T se0[3][R][64];      // E^n, plane k
  T sh1[3][R][64];      // H^{n+1/2}, plane k
  T se1[2][3][R][64];   // E^{n+1}, planes k and k-1
  T sh2[3][R][64];      // H^{n+3/2}, plane k-1
  T stab[256 * K_STRIDE];
  T px[P_NROW][64];     // CPML profile at each lane's x
  T py[P_NROW][R];      // ... at each wave's y
  T pz[P_NROW * PZ];    // the z table
};

// CPML profile values of a two-step tile from the LDS copies made at the
// tile start.  Reading them from global memory in every plane would make the
// wave wait for its whole prefetch at each CPML term.  (The host runs the
// two-step pass only on grids whose z table fits its copy: 2 npml <= PZ.)
template <typename T, int TY>
struct ProfTB2 {
  const GridView<T>& g;
  const TB2Smem<T, TY>& sm;
  int u, v;
  template <int U>
  __device__ __forceinline__ Prof3<T> at(int row, int l) const {
    if (U == 0) return {sm.px[row][u], sm.px[row + 1][u], sm.px[row + 2][u]};
    if (U == 1) return {sm.py[row][v], sm.py[row + 1][v], sm.py[row + 2][v]};
    const int tn = 2 * g.npml, q = row * tn + l;
    return {sm.pz[q], sm.pz[q + tn], sm.pz[q + 2 * tn]};
  }
};

// One two-step tile: outputs [i0, i0+iw) x [j0, j0+jh) x [k0, k1) with iw <= 60,
// jh <= TY, a plane of every stage at a time (tb2_any); AX masks the axes whose
// CPML slabs the tile's region reaches.
template <typename T, typename CI, int TY, int AX, bool TABV>
__device__ __forceinline__ void tb2_tile(const GridView<T>& g, TB2Smem<T, TY>& sm, int i0, int j0, int iw, int jh,
                                         int k0, int k1, int step) {
  constexpr int TX = 60, NT = 64 * (TY + 4);
  constexpr bool LDS_TAB = sizeof(CI) == 1, WIDE = sizeof(T) == 4;
  const int tid = threadIdx.x, u = tid & 63, v = tid >> 6;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const unsigned sxy = (unsigned)g.sxy;
  const CI* cls = (const CI*)g.cls;
  if (LDS_TAB) {
    for (int q = tid; q < g.ncls * K_STRIDE; q += NT) sm.stab[q] = ldg(g.ctab, (unsigned)q);
  }
  // TABV: the view comes from a table of views, so that the compiler does not
  // know its pointers for global memory's, and would use FLAT loads
  T cf[K_STRIDE];
  auto coef = [&](int c) -> const T* {
    if constexpr (LDS_TAB) {
      return sm.stab + c * K_STRIDE;
    } else if constexpr (!TABV) {
      return g.ctab + c * K_STRIDE;
    } else {
      const auto* row = (const __attribute__((address_space(1))) T*)g.ctab + c * K_STRIDE;
      for (int q = 0; q < K_NCOEF; ++q) cf[q] = row[q];  // (what a stage does not use is not loaded)
      return cf;
    }
  };

  const int x = i0 - 2 + u, y = j0 - 2 + v;
  const bool dom = x >= 0 && x < nx && y >= 0 && y < ny;
  const bool inA = dom && u <= TX + 2 && v <= TY + 2;
  const bool inB = inA && u >= 1 && v >= 1;
  const bool inC = inB && u <= TX + 1 && v <= TY + 1;
  const bool inD = inC && u >= 2 && v >= 2 && u < 2 + iw && v < 2 + jh;
  const unsigned n0 = dom ? (unsigned)x + (unsigned)nx * (unsigned)y : 0u;
  const int lx = (AX & 1) && dom ? slab_pos(x, nx, g.npml) : -1;
  const int ly = (AX & 2) && dom ? slab_pos(y, ny, g.npml) : -1;
  // (E is updated on planes k0 - 1 .. k1: the first step's cone, then the outputs)
  const SrcRange srcr = src_wave(g, n0, inB, k0 - 1, k1);
  const int tn = 2 * g.npml;
  if ((AX & 1) && v == 0) {
    const int xl = x >= 0 && x < nx ? slab_pos(x, nx, g.npml) : -1;
    for (int r = 0; r < P_NROW; ++r) sm.px[r][u] = xl >= 0 ? ldg(g.prof[0], (unsigned)(r * tn + xl)) : T(0);
  }
  if ((AX & 2) && u == 0) {
    const int yl = y >= 0 && y < ny ? slab_pos(y, ny, g.npml) : -1;
    for (int r = 0; r < P_NROW; ++r) sm.py[r][v] = yl >= 0 ? ldg(g.prof[1], (unsigned)(r * tn + yl)) : T(0);
  }
  if (AX & 4)
    for (int q = tid; q < P_NROW * tn; q += NT) sm.pz[q] = ldg(g.prof[2], (unsigned)q);
  const ProfTB2<T, TY> pf{g, sm, u, v};

  auto ld_e = [&](int k, T e[3]) {
    const bool in = k >= 0 && k < nz;
    const bool ok = dom && in;
    const unsigned n = n0 + sxy * (unsigned)(ok ? k : 0);
    e[0] = ok ? ldg(g.fi[0], n) : T(0);
    e[1] = ok ? ldg(g.fi[1], n) : T(0);
    e[2] = ok ? ldg(g.fi[2], n) : T(0);
  };
  auto ld_h = [&](int k, T h[3]) {
    const bool ok = inA && k >= 0 && k < nz;
    const unsigned n = n0 + sxy * (unsigned)(ok ? k : 0);
    h[0] = ok ? ldg(g.fi[3], n) : T(0);
    h[1] = ok ? ldg(g.fi[4], n) : T(0);
    h[2] = ok ? ldg(g.fi[5], n) : T(0);
  };
  auto ld_c = [&](int k) -> int {
    return (inA && k >= 0 && k < nz) ? (int)ldg(cls, n0 + sxy * (unsigned)k) : 0;
  };

  // E's sources in plane k (every lane of the wave; `on`: this lane's point
  // takes them), many of them as in March.  FP32 only: an oblique wire, a
  // source at every edge it touches, in 42 x 36 x 61 nodes of 17,000 classes
  // 61 us a step, 100 with all of a column's sources read in every plane; FP64
  // tiles, of which few meet a source, are 6% slower with it.
  auto sources = [&](int k, bool on, int st, T e[3]) {
    if (k < srcr.klo || k > srcr.khi) return;  // uniform
    const unsigned n = on ? n0 + sxy * (unsigned)k : 0xFFFFFFFFu;
    if (srcr.hi - srcr.lo <= 4) {
      e_sources(&g, srcr.lo, srcr.hi, n, st, e);
      return;
    }
    for (int s0 = srcr.lo; s0 < srcr.hi; s0 += 64) {
      const int s = s0 + u;
      const bool here = s < srcr.hi && (unsigned)ldg(g.src_idx, (unsigned)s) - sxy * (unsigned)k < sxy;
      for (unsigned long long m = __ballot(here); m; m &= m - 1) {
        const int q = s0 + __builtin_ctzll(m);
        e_sources(&g, q, q + 1, n, st, e);
      }
    }
  };

  // pipeline registers of this thread's point
  T e0c[3], e0n[3], h0c[3];
  T h1p[3] = {T(0), T(0), T(0)};   // H^{n+1/2}, plane k-1
  T e1p[3] = {T(0), T(0), T(0)};   // E^{n+1},   plane k-1
  T h2p[2] = {T(0), T(0)};         // H^{n+3/2}, plane k-2 (x, y)
  T psh[3][2], pse[3][2];          // CPML state after step n+1, plane k-1
  for (int a = 0; a < 3; ++a) psh[a][0] = psh[a][1] = pse[a][0] = pse[a][1] = T(0);
  const int kb = k0 - 2;
  ld_e(kb, e0c);
  ld_e(kb + 1, e0n);
  ld_h(kb, h0c);
  int cc = ld_c(kb), cp = 0;

  // Let the prologue's loads land before the loop.  Otherwise the compiler,
  // which merges the loop entry with the back edge, places the wait for them
  // after the stores at the top of every iteration and so waits for those
  // stores as well.  (vmcnt 0, expcnt and lgkmcnt unconstrained)
  __builtin_amdgcn_s_waitcnt(0x0F70);
  for (int k = kb; k <= k1; ++k) {
    // prefetch: classes and H^{n-1/2} of plane k+1, E^n of plane k+2 (the
    // classes first: the end of the iteration then waits for all of it)
    T e0f[3], h0f[3];
    const int cf1 = ld_c(k + 1);
    ld_e(k + 2, e0f);
    ld_h(k + 1, h0f);
    const bool kin = k >= 0 && k < nz;
    for (int c = 0; c < 3; ++c) sm.se0[c][v][u] = dom ? e0c[c] : T(0);
    __syncthreads();
    // A: H^{n+1/2}, plane k
    T h1c[3] = {T(0), T(0), T(0)};
    T pshn[3][2];
    // The z-slab planes take their own branch (lz is uniform), so that the
    // CPML state loaded there is consumed inside it and no wait for it is
    // left at the end of the iteration, where it would also wait for the
    // prefetch and the stores.
    const int lz = AX & 4 ? slab_pos(k, nz, g.npml) : -1;
    if (inA && kin) {
      auto stage_a = [&](const int l[3]) {
        psi_load(g, 1, l, x, y, k, pshn);
        h_core_pf<T, true>(pf, l, coef(cc), e0c[0], e0c[1], e0c[2], sm.se0[0][v + 1][u], e0n[0], sm.se0[1][v][u + 1],
                       e0n[1], sm.se0[2][v][u + 1], sm.se0[2][v + 1][u], h0c, pshn[0], pshn[1], pshn[2], h1c);
      };
      if (lz >= 0) {
        const int l[3] = {lx, ly, lz};
        stage_a(l);
      } else {
        const int l[3] = {lx, ly, -1};
        stage_a(l);
      }
    }
    for (int c = 0; c < 3; ++c) sm.sh1[c][v][u] = h1c[c];
    __syncthreads();
    // B: E^{n+1}, plane k (needs H^{n+1/2} of plane k-1: valid from k0-1 on)
    T e1c[3] = {T(0), T(0), T(0)};
    T psen[3][2];
    if (inB && kin && k >= k0 - 1) {
      auto stage_b = [&](const int l[3]) {
        psi_load(g, 0, l, x, y, k, psen);
        e_core_pf<T, true>(pf, l, coef(cc), h1c[0], h1c[1], h1c[2], sm.sh1[0][v - 1][u], h1p[0], sm.sh1[1][v][u - 1],
                          h1p[1], sm.sh1[2][v][u - 1], sm.sh1[2][v - 1][u], e0c, psen[0], psen[1], psen[2], e1c);
        if constexpr (!WIDE) e_sources(&g, srcr.first(k), srcr.last(k), n0 + sxy * (unsigned)k, step, e1c);
      };
      if (lz >= 0) {
        const int l[3] = {lx, ly, lz};
        stage_b(l);
      } else {
        const int l[3] = {lx, ly, -1};
        stage_b(l);
      }
    }
    if (WIDE && k >= k0 - 1) sources(k, inB && kin, step, e1c);
    const int s1 = (k + 2) & 1, s1m = s1 ^ 1;
    for (int c = 0; c < 3; ++c) sm.se1[s1][c][v][u] = e1c[c];
    // No barrier here: C reads the neighbours' E^{n+1} of plane k-1 (slot
    // s1m, written in the previous iteration, before its two barriers) and
    // this thread's own E^{n+1} of plane k (a register).  Slot s1, written
    // just now, is read by the next iteration's C, after that iteration's
    // first two barriers; it last held plane k-2, whose readers finished
    // before this iteration's barriers.
    // C: H^{n+3/2}, plane k-1
    const int km = k - 1;
    T h2c[3] = {T(0), T(0), T(0)};
    if (inC && k >= k0 && km >= 0 && km < nz) {
      int l[3] = {lx, ly, AX & 4 ? slab_pos(km, nz, g.npml) : -1};
      h_core_pf<T, true>(pf, l, coef(cp), e1p[0], e1p[1], e1p[2], sm.se1[s1m][0][v + 1][u], e1c[0],
                     sm.se1[s1m][1][v][u + 1], e1c[1], sm.se1[s1m][2][v][u + 1], sm.se1[s1m][2][v + 1][u], h1p, psh[0],
                     psh[1], psh[2], h2c);
      if (inD && km >= k0) {
        const unsigned n = n0 + sxy * (unsigned)km;
        stg(g.fo[3], n, h2c[0]);
        stg(g.fo[4], n, h2c[1]);
        stg(g.fo[5], n, h2c[2]);
        psi_store(g, 1, l, x, y, km, psh);
      }
    }
    for (int c = 0; c < 3; ++c) sm.sh2[c][v][u] = h2c[c];
    __syncthreads();
    // D: E^{n+2}, plane k-1 (the output tile; km < k1 always holds)
    T e2[3];
    auto stage_d = [&](const int l[3]) {
      e_core_pf<T, true>(pf, l, coef(cp), h2c[0], h2c[1], h2c[2], sm.sh2[0][v - 1][u], h2p[0], sm.sh2[1][v][u - 1],
                        h2p[1], sm.sh2[2][v][u - 1], sm.sh2[2][v - 1][u], e1p, pse[0], pse[1], pse[2], e2);
    };
    if constexpr (WIDE) {
      if (inD && km >= k0) {
        const int l[3] = {lx, ly, AX & 4 ? slab_pos(km, nz, g.npml) : -1};
        stage_d(l);
      }
      if (km >= k0) sources(km, inD, step + 1, e2);
    }
    if (inD && km >= k0) {
      const unsigned nst = n0 + sxy * (unsigned)km;
      int l[3] = {lx, ly, AX & 4 ? slab_pos(km, nz, g.npml) : -1};
      if constexpr (!WIDE) {
        stage_d(l);
        e_sources(&g, srcr.first(km), srcr.last(km), nst, step + 1, e2);
      }
      stg(g.fo[0], nst, e2[0]);
      stg(g.fo[1], nst, e2[1]);
      stg(g.fo[2], nst, e2[2]);
      psi_store(g, 0, l, x, y, km, pse);
    }
    // rotate the pipeline
    h2p[0] = h2c[0];
    h2p[1] = h2c[1];
    for (int c = 0; c < 3; ++c) {
      h1p[c] = h1c[c];
      e1p[c] = e1c[c];
      e0c[c] = e0n[c];
      e0n[c] = e0f[c];
      h0c[c] = h0f[c];
    }
    for (int a = 0; a < 3; ++a) {
      psh[a][0] = pshn[a][0];
      psh[a][1] = pshn[a][1];
      pse[a][0] = psen[a][0];
      pse[a][1] = psen[a][1];
    }
    cp = cc;
    cc = cf1;
  }
}

// One tile of a two-step pass by the code its CPML needs: tiles whose region
// (halo and pipeline planes included) is clear of some slabs leave their code
// out.  FP64 tiles in the CPML would spill in March's registers; they take
// the one-plane-at-a-time tile.  So do all tiles with the classes' table in
// memory (NC 0): March, which loads three planes ahead, waits for all of it at
// each coefficient, four times a plane (us a step, March / tb2_tile / split
// pass, FP32, 17,000 classes: 203 x 157 x 131 with a CPML 155 / 78 / 86, 384 x
// 384 x 288 1,500 / 741 / 1,137, without one 1,366 / 723 / 1,101; FP64 320 x
// 300 x 256 896 / 748 / 1,130).
template <typename T, int TY, int NC>
union TileSmem {
  MarchSmem<T, TY, NC> m;
  TB2Smem<T, TY> t;
};
template <int TY, int NC>
union TileSmem<float, TY, NC> {
  MarchSmem<float, TY, NC> m;
};
template <int TY>
union TileSmem<float, TY, 0> {
  MarchSmem<float, TY, 0> m;
  TB2Smem<float, TY> t;
};
template <typename T, typename CI, bool PML, int TY, int NC, bool TABV>
__device__ __forceinline__ void tb2_any(const GridView<T>& g, ColdView<T> cold, TileSmem<T, TY, NC>& sm, int i0, int j0,
                                        int iw, int jh, int k0, int k1, int step) {
  if constexpr (!PML && NC == 0) {
    tb2_tile<T, CI, TY, 0, TABV>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
  } else if constexpr (!PML) {
    March<T, CI, TY, 0, 0, NC>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
  } else {
    const int n = g.npml;
    const bool cx = i0 - 2 >= n && i0 + 62 <= g.nx - n, cy = j0 - 2 >= n && j0 + TY + 2 <= g.ny - n,
               cz = k0 - 2 >= n && k1 < g.nz - n;
    if constexpr (NC == 0) {
      if (cx && cy) tb2_tile<T, CI, TY, 4, TABV>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
      else if (cy) tb2_tile<T, CI, TY, 5, TABV>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
      else if (cx) tb2_tile<T, CI, TY, 6, TABV>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
      else tb2_tile<T, CI, TY, 7, TABV>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
    } else if (cx && cy && cz) {
      March<T, CI, TY, 0, 0, NC>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
    } else if constexpr (sizeof(T) == 8) {
      tb2_tile<T, CI, TY, 7, TABV>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
    } else {
      if (cx && cy) March<T, CI, TY, 4, 0, NC>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
      else if (cy) March<T, CI, TY, 5, 0, NC>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
      else if (cx) March<T, CI, TY, 6, 0, NC>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
      else March<T, CI, TY, 7, 0, NC>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
    }
  }
}

// Registers a lane may use: FP32 tiles with CPML code take what one block per
// CU leaves them; tiles without it, and 8-row ones with their table in memory
// (64 KB of LDS), stay below 80 so that two 12-wave blocks share a CU.
constexpr int tb2_waves(int size, bool pml, int ty, int nc) {
  return size == 8 ? 1 : (nc == 0 && ty == 8) ? 6 : pml || ty == 12 || nc > TB2_NC2 ? (ty + 4) / 4 : 6;
}

// A whole two-step pass in one launch: blocks 0 .. npb - 1 each record a few
// probes (sample `step` recomputed from the input set and, with `prev`, the
// previous pass's second sample, step - 1, which is the input set itself),
// the others march one 60 x TY tile over kz planes.  The probes of a pass's
// last step are left to the next pass or to k_probes after the last one; more
// than PR_MANY probes are k_probes_tb2's, npb 0.
// `run`: tiles that an XCD takes in a row (xcd_runs).
template <typename T, typename CI, bool PML, int TY, int NC>
__global__ __launch_bounds__(64 * (TY + 4), tb2_waves(sizeof(T), PML, TY, NC)) void k_tb2(GridView<T> g, int step,
                                                                                       int kz, int ntx, int nty,
                                                                                       int npb, int prev, int run) {
  step = gstep(g, step);
  __shared__ TileSmem<T, TY, NC> sm;
  constexpr int GRP = 64 * (TY + 4) / PR_NT;  // probes per block
  __shared__ double red[12 * GRP];
  if ((int)blockIdx.x < npb) {  // uniform per block
    const int grp = (int)threadIdx.x / PR_NT, t = (int)threadIdx.x % PR_NT, q = (int)blockIdx.x * GRP + grp;
    const int p = q < g.n_probe ? q : -1;
    probe_tb2<T, CI, PML>(g, p, step, t, red + 12 * grp);
    if (prev) probe_one(g, p, step - 1, t, red + 12 * grp + 8);
    return;
  }
  const int tile = xcd_runs((int)blockIdx.x - npb, (int)gridDim.x - npb, run);
  const int tile_x = tile % ntx, rest = tile / ntx, k0 = (rest / nty) * kz;
  // the view is the kernel's first argument: read again where it is needed
  const ColdView<T> cold{(typename ColdView<T>::P)__builtin_amdgcn_kernarg_segment_ptr()};
  tb2_any<T, CI, PML, TY, NC, false>(g, cold, sm, tile_x * 60, (rest % nty) * TY, 60, TY, k0, min(k0 + kz, g.nz), step);
}

// Batched two-step pass: as k_tb2 over a tile list that spans every grid
// (grid, i0 | iw << 16, j0 | jh << 16, k0 | kz << 16) and a list of (grid,
// probe) pairs; step index *d_step + offset.  Nearly every tile of a small
// grid is in the CPML and marches at 1.7 us a plane, instruction bound.  256
// grids of 32 to 96 cells a side with an 8-cell CPML: 1179 us a step (1473
// with one work-queue launch per CPML group and a probe launch); 64 of them
// 296, 8 of them 47 (80).
template <typename T, typename CI, int NC>
__global__ __launch_bounds__(768, tb2_waves(sizeof(T), true, 8, NC)) void k_tb2_batch(
    const GridView<T>* __restrict__ views, const int4* __restrict__ tiles, const int2* __restrict__ plist, int n_probes,
    int npb, const int* __restrict__ d_step, int offset, int prev, int run) {
  const int step = *d_step + offset;
  __shared__ TileSmem<T, 8, NC> sm;
  constexpr int GRP = 768 / PR_NT;
  __shared__ double red[12 * GRP];
  if ((int)blockIdx.x < npb) {  // uniform per block
    const int grp = (int)threadIdx.x / PR_NT, t = (int)threadIdx.x % PR_NT, q = (int)blockIdx.x * GRP + grp;
    const int2 e = plist[min(q, n_probes - 1)];
    const int p = q < n_probes ? e.y : -1;
    probe_tb2<T, CI, true>(views[e.x], p, step, t, red + 12 * grp);
    if (prev) probe_one(views[e.x], p, step - 1, t, red + 12 * grp + 8);
    return;
  }
  const int4 t = tiles[xcd_runs((int)blockIdx.x - npb, (int)gridDim.x - npb, run)];
  const int tx = __builtin_amdgcn_readfirstlane(t.x), ty = __builtin_amdgcn_readfirstlane(t.y),
            tz = __builtin_amdgcn_readfirstlane(t.z), tw = __builtin_amdgcn_readfirstlane(t.w);
  const GridView<T> g = uniform_view(views + tx);
  const ColdView<T> cold{(typename ColdView<T>::P)(uintptr_t)(views + tx)};
  const int k0 = tw & 0xffff;
  tb2_any<T, CI, true, 8, NC, true>(g, cold, sm, ty & 0xffff, tz & 0xffff, ty >> 16, tz >> 16, k0, k0 + (tw >> 16), step);
}

// The batch's probes apart from its pass (as k_probes_tb2).
template <typename T, typename CI>
__global__ __launch_bounds__(PR_NT) void k_probes_tb2_batch(const GridView<T>* __restrict__ views,
                                                           const int2* __restrict__ plist, int n,
                                                           const int* __restrict__ d_step, int offset, int prev) {
  const int step = *d_step + offset;
  __shared__ double red[8];
  if ((int)blockIdx.x >= n) return;  // uniform per block
  const int2 e = plist[blockIdx.x];
  probe_tb2<T, CI, true>(views[e.x], e.y, step, (int)threadIdx.x, red);
  if (prev) probe_one(views[e.x], e.y, step - 1, (int)threadIdx.x, red + 4);
}

// ---------------------------------------------------------------------------
// probes of a one-step pass: one block per probe, the fixed FP64 order of
// probe_sum
// ---------------------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(PR_NT) void k_probes(GridView<T> g, int step) {
  step = gstep(g, step);
  __shared__ double red[4];
  if ((int)blockIdx.x >= g.n_probe) return;  // uniform per block
  probe_one(g, blockIdx.x, step, (int)threadIdx.x, red);
}

// Batched probes: entry q of the list is (grid, probe); one block each.
template <typename T>
__global__ __launch_bounds__(PR_NT) void k_probes_batch(const GridView<T>* __restrict__ views,
                                                       const int2* __restrict__ plist, int n,
                                                       const int* __restrict__ d_step, int offset) {
  __shared__ double red[4];
  if ((int)blockIdx.x >= n) return;  // uniform per block
  const int2 e = plist[blockIdx.x];
  probe_one(views[e.x], e.y, *d_step + offset, (int)threadIdx.x, red);
}

__global__ void k_add(int* p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p += v;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// Split-pass blocks: NB consecutive nodes of a plane (full waves for any
// nx).  512 on large planes, 256 (dealt in bands per XCD) on small ones: on a
// 512 x 512 plane 512 ran 2.5% faster, on a 100 x 100 plane 4% slower (and
// 128 slower on both).
inline int split_nb(const long long sxy) { return sxy >= 65536 ? 512 : 256; }

template <typename T, typename CI, int NB>
hipError_t step_split_nb(const GridView<T>& g, int step, hipStream_t st) {
  const dim3 blk(NB), grd((unsigned)((g.sxy + NB - 1) / NB), (unsigned)g.nz);
  if (g.npml > 0) {
    hipLaunchKernelGGL((k_h_split<T, CI, true, NB>), grd, blk, 0, st, g);
    hipLaunchKernelGGL((k_e_split<T, CI, true, NB>), grd, blk, 0, st, g, step);
  } else {
    hipLaunchKernelGGL((k_h_split<T, CI, false, NB>), grd, blk, 0, st, g);
    hipLaunchKernelGGL((k_e_split<T, CI, false, NB>), grd, blk, 0, st, g, step);
  }
  return hipGetLastError();
}

template <typename T, typename CI>
hipError_t step_split(const GridView<T>& g, int step, hipStream_t st) {
  return split_nb(g.sxy) == 512 ? step_split_nb<T, CI, 512>(g, step, st) : step_split_nb<T, CI, 256>(g, step, st);
}

// Oblique thin wires.  k_owire_cur: the new segment currents from E^n (the
// input field set, or with E1 the values of k_owire_e1) and the charges q^n
// (the driven segment takes its sample); k_owire_q: then the charges from
// the new currents, and the record.  Both before the step's field pass,
// which they do not depend on.  One one-wave block per segment (block
// (s, wire)): lane l sums the gather terms l, l + 64, ... in table order,
// then the 64 partial sums meet in a fixed shuffle tree, so the result does
// not depend on scheduling.  The blocks are single waves so that they find
// room on CUs that the field pass's blocks keep busy.
template <typename T, bool E1>
__global__ void __launch_bounds__(64) k_owire_cur(GridView<T> g, OWireView w, int step) {
  step = gstep(g, step);
  const OWireParam p = w.par[blockIdx.y];
  const int s = (int)blockIdx.x;
  if (s >= p.nseg) return;  // uniform per block
  double* cur = w.cur + p.seg0;
  const double* q = w.q + p.seg0 + blockIdx.y;
  const int lane = (int)threadIdx.x;
  double et = 0.0;
  for (int e = w.seg_off[p.seg0 + s] + lane, e1 = w.seg_off[p.seg0 + s + 1]; e < e1; e += 64) {
    if (E1) {
      et += w.g_w[e] * w.e1[w.g_edge[e]];
    } else {
      const long long key = w.g_key[e];
      et += w.g_w[e] * (double)g.fi[(int)(key >> 40)][key & ((1ll << 40) - 1)];
    }
  }
  for (int off = 32; off > 0; off >>= 1) et += __shfl_down(et, off, 64);
  if (lane == 0)
    cur[s] = s == p.src ? w.amp[(size_t)blockIdx.y * w.max_steps + step]
                        : cur[s] + p.dtL * (et - (q[s + 1] - q[s]) * p.invCdl);
}

template <typename T>
__global__ void __launch_bounds__(64) k_owire_q(GridView<T> g, OWireView w, int step) {
  step = gstep(g, step);
  const OWireParam p = w.par[blockIdx.y];
  const double* cur = w.cur + p.seg0;
  double* q = w.q + p.seg0 + blockIdx.y;
  const int j = (int)(blockIdx.x * 64 + threadIdx.x);
  if (j <= p.nseg) {
    const double il = j > 0 ? cur[j - 1] : 0.0, ir = j < p.nseg ? cur[j] : 0.0;
    q[j] -= ((j == 0 || j == p.nseg) ? 2.0 * p.dtdl : p.dtdl) * (ir - il);
  }
  if (j == 0 && p.rec >= 0) w.rec[(size_t)blockIdx.y * w.max_steps + step] = cur[p.rec];
}

// Junctions, after k_owire_q: that kernel moved each member end node's
// charge by its own segment's current as for an open end, so the members'
// charges sum (times their half segments) to the junction's new charge;
// they then take the shared potential, q_m = C'_m Q / sum_m C'_m len_m.  One
// thread per junction, members in table order (FP64).
__global__ void __launch_bounds__(64) k_owire_junc(OWireView w) {
  const int J = (int)(blockIdx.x * 64 + threadIdx.x);
  if (J >= w.n_junc) return;
  double Q = 0.0, cap = 0.0;
  for (int m = w.jn_off[J]; m < w.jn_off[J + 1]; ++m) {
    Q += w.q[w.jn_q[m]] * w.jn_a[m];
    cap += w.jn_c[m] * w.jn_a[m];
  }
  const double V = Q / cap;
  for (int m = w.jn_off[J]; m < w.jn_off[J + 1]; ++m) w.q[w.jn_q[m]] = w.jn_c[m] * V;
}

// The touched edges' source amplitudes of step `step`: one thread per edge
// sums its terms in increasing segment order (FP64), times the edge's Cb / dx.
template <typename T, typename CI>
__global__ void __launch_bounds__(64) k_owire_amp(GridView<T> g, OWireView w, int step) {
  step = gstep(g, step);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= w.n_edge) return;
  const long long key = w.e_key[e];
  const int a = (int)(key >> 40);
  const long long n = key & ((1ll << 40) - 1);
  double sum = 0.0;
  for (int t = w.e_off[e], t1 = w.e_off[e + 1]; t < t1; ++t) sum += w.j_w[t] * w.cur[w.j_seg[t]];
  const int cls = ((const CI*)g.cls)[n];
  const double cbdx = (double)g.ctab[cls * K_STRIDE + K_CBX + 2 * a];
  T* amp = const_cast<T*>(g.src_amp);
  amp[(size_t)w.wsrc[e] * (size_t)g.max_steps + (size_t)step] = (T)(cbdx * sum);
}

// E^{step+1} at the touched edges for a two-step pass: the step's update
// at the edge's node, recomputed from the input set as the pass will do it
// (its sources, the wires' included, and CPML).
template <typename T, typename CI, bool PML>
__global__ void __launch_bounds__(64) k_owire_e1(GridView<T> g, OWireView w, int step) {
  step = gstep(g, step);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= w.n_edge) return;
  const long long key = w.e_key[e];
  const int a = (int)(key >> 40);
  const long long n = key & ((1ll << 40) - 1);
  const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny), k = (int)(n / g.sxy);
  T v[3];
  e1_at<T, CI, PML>(g, x, y, k, step, v);
  w.e1[e] = (double)v[a];
}

template <typename T, typename CI, int NB>
hipError_t step_split_debye_nb(const GridView<T>& g, const DebyeView<T>& d, int step, hipStream_t st) {
  const dim3 blk(NB), grd((unsigned)((g.sxy + NB - 1) / NB), (unsigned)g.nz);
  if (g.npml > 0) {
    hipLaunchKernelGGL((k_h_split<T, CI, true, NB>), grd, blk, 0, st, g);
    hipLaunchKernelGGL((k_e_split_debye<T, CI, true, NB>), grd, blk, 0, st, g, d, step);
  } else {
    hipLaunchKernelGGL((k_h_split<T, CI, false, NB>), grd, blk, 0, st, g);
    hipLaunchKernelGGL((k_e_split_debye<T, CI, false, NB>), grd, blk, 0, st, g, d, step);
  }
  return hipGetLastError();
}

template <typename T, typename CI>
hipError_t step_split_debye(const GridView<T>& g, const DebyeView<T>& d, int step, hipStream_t st) {
  return split_nb(g.sxy) == 512 ? step_split_debye_nb<T, CI, 512>(g, d, step, st)
                                : step_split_debye_nb<T, CI, 256>(g, d, step, st);
}

int launch_owire_iq(int prec, const void* view, const OWireView* ow, int step, int from_e1, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const dim3 gc((unsigned)ow->max_seg, (unsigned)ow->n_wire), gq((unsigned)(ow->max_seg / 64 + 1), (unsigned)ow->n_wire);
  if (prec == 64) {
    const GridView<double>& g = *(const GridView<double>*)view;
    if (from_e1) hipLaunchKernelGGL((k_owire_cur<double, true>), gc, dim3(64), 0, st, g, *ow, step);
    else hipLaunchKernelGGL((k_owire_cur<double, false>), gc, dim3(64), 0, st, g, *ow, step);
    hipLaunchKernelGGL((k_owire_q<double>), gq, dim3(64), 0, st, g, *ow, step);
  } else {
    const GridView<float>& g = *(const GridView<float>*)view;
    if (from_e1) hipLaunchKernelGGL((k_owire_cur<float, true>), gc, dim3(64), 0, st, g, *ow, step);
    else hipLaunchKernelGGL((k_owire_cur<float, false>), gc, dim3(64), 0, st, g, *ow, step);
    hipLaunchKernelGGL((k_owire_q<float>), gq, dim3(64), 0, st, g, *ow, step);
  }
  if (ow->n_junc > 0) hipLaunchKernelGGL(k_owire_junc, dim3((unsigned)((ow->n_junc + 63) / 64)), dim3(64), 0, st, *ow);
  return (int)hipGetLastError();
}

template <typename T>
hipError_t owire_amp_t(const GridView<T>& g, int cls16, const OWireView& w, int step, hipStream_t st) {
  const dim3 grd((unsigned)((w.n_edge + 63) / 64)), blk(64);
  if (cls16) hipLaunchKernelGGL((k_owire_amp<T, uint16_t>), grd, blk, 0, st, g, w, step);
  else hipLaunchKernelGGL((k_owire_amp<T, uint8_t>), grd, blk, 0, st, g, w, step);
  return hipGetLastError();
}

template <typename T>
hipError_t owire_e1_t(const GridView<T>& g, int cls16, const OWireView& w, int step, hipStream_t st) {
  const dim3 grd((unsigned)((w.n_edge + 63) / 64)), blk(64);
  const bool pml = g.npml > 0;
  if (cls16) {
    if (pml) hipLaunchKernelGGL((k_owire_e1<T, uint16_t, true>), grd, blk, 0, st, g, w, step);
    else hipLaunchKernelGGL((k_owire_e1<T, uint16_t, false>), grd, blk, 0, st, g, w, step);
  } else {
    if (pml) hipLaunchKernelGGL((k_owire_e1<T, uint8_t, true>), grd, blk, 0, st, g, w, step);
    else hipLaunchKernelGGL((k_owire_e1<T, uint8_t, false>), grd, blk, 0, st, g, w, step);
  }
  return hipGetLastError();
}

int launch_owire_amp(int prec, const void* view, int cls16, const OWireView* ow, int step, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (prec == 64) return (int)owire_amp_t(*(const GridView<double>*)view, cls16, *ow, step, st);
  return (int)owire_amp_t(*(const GridView<float>*)view, cls16, *ow, step, st);
}

int launch_owire_e1(int prec, const void* view, int cls16, const OWireView* ow, int step, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (prec == 64) return (int)owire_e1_t(*(const GridView<double>*)view, cls16, *ow, step, st);
  return (int)owire_e1_t(*(const GridView<float>*)view, cls16, *ow, step, st);
}

int launch_step_debye(int prec, const void* view, const void* dview, int cls16, int step, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  if (prec == 64) {
    const GridView<double>& g = *(const GridView<double>*)view;
    const DebyeView<double>& d = *(const DebyeView<double>*)dview;
    e = cls16 ? step_split_debye<double, uint16_t>(g, d, step, st) : step_split_debye<double, uint8_t>(g, d, step, st);
  } else {
    const GridView<float>& g = *(const GridView<float>*)view;
    const DebyeView<float>& d = *(const DebyeView<float>*)dview;
    e = cls16 ? step_split_debye<float, uint16_t>(g, d, step, st) : step_split_debye<float, uint8_t>(g, d, step, st);
  }
  return (int)e;
}

template <typename T, typename CI, bool PML, int TX, int TY>
hipError_t launch_fused(const GridView<T>& g, int step, int kz, hipStream_t st) {
  const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + kz - 1) / kz;
  const long long nb = (long long)ntx * nty * ntz;
  if (nb > 0x7fffffff || (sizeof(CI) == 1 && g.ncls > 256)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_fused<T, CI, PML, TX, TY>), dim3((unsigned)nb), dim3(TX * TY), 0, st, g, step, kz, ntx,
                     nty);
  return hipGetLastError();
}

template <typename T, typename CI>
hipError_t step_fused(const GridView<T>& g, int step, int tile_y, int tile_z, hipStream_t st) {
  const int kz = tile_z > 0 ? tile_z : 32;
  const bool pml = g.npml > 0;
  if (tile_y == 4)
    return pml ? launch_fused<T, CI, true, 64, 4>(g, step, kz, st) : launch_fused<T, CI, false, 64, 4>(g, step, kz, st);
  return pml ? launch_fused<T, CI, true, 64, 8>(g, step, kz, st) : launch_fused<T, CI, false, 64, 8>(g, step, kz, st);
}

// Tile groups of a grid with a CPML, by the slabs a tile (halo included)
// reaches: 0 neither the x nor the y slabs (z CPML code only), 1 x slabs, 2
// y slabs, 3 both (x-y corners).  Tiles of the fused pass, 32 wide in groups 1
// and 3 and 64 wide otherwise.  FP64 (a diagnostic precision) keeps the all-axes instantiation for every group.
template <typename T, typename CI, int TY>
hipError_t launch_lists(const GridView<T>& g, int step, const int4* tiles, const int* counts, hipStream_t st,
                        hipStream_t st2, void* ev_src) {
  if (sizeof(CI) == 1 && g.ncls > 256) return hipErrorInvalidValue;
  constexpr bool D = sizeof(T) == 8;
  const int4* t = tiles;
  if (counts[0] > 0)
    hipLaunchKernelGGL((k_fused_list<T, CI, true, 64, TY, D ? 7 : 4>), dim3((unsigned)counts[0]), dim3(64 * TY), 0,
                       st, g, t, step);
  t += counts[0];
  if (counts[1] > 0)
    hipLaunchKernelGGL((k_fused_list<T, CI, true, 32, TY, D ? 7 : 5>), dim3((unsigned)counts[1]), dim3(32 * TY), 0,
                       st2, g, t, step);
  t += counts[1];
  if (counts[2] > 0)
    hipLaunchKernelGGL((k_fused_list<T, CI, true, 64, TY, D ? 7 : 6>), dim3((unsigned)counts[2]), dim3(64 * TY), 0,
                       st2, g, t, step);
  t += counts[2];
  if (counts[3] > 0)
    hipLaunchKernelGGL((k_fused_list<T, CI, true, 32, TY, 7>), dim3((unsigned)counts[3]), dim3(32 * TY), 0, st2, g, t,
                       step);
  t += counts[3];
  if (ev_src) {
    const hipError_t we = hipStreamWaitEvent(st2, (hipEvent_t)ev_src, 0);
    if (we != hipSuccess) return we;
  }
  if (counts[4] > 0)  // tiles that read an oblique wire's source amplitudes, once written
    hipLaunchKernelGGL((k_fused_list<T, CI, true, 32, TY, 7>), dim3((unsigned)counts[4]), dim3(32 * TY), 0, st2, g, t,
                       step);
  return hipGetLastError();
}

template <typename T>
hipError_t lists_any(const GridView<T>& g, int cls16, int step, int ty, const int4* tiles, const int* counts,
                     hipStream_t st, hipStream_t st2, void* ev) {
  if (ty == 4)
    return cls16 ? launch_lists<T, uint16_t, 4>(g, step, tiles, counts, st, st2, ev)
                 : launch_lists<T, uint8_t, 4>(g, step, tiles, counts, st, st2, ev);
  return cls16 ? launch_lists<T, uint16_t, 8>(g, step, tiles, counts, st, st2, ev)
               : launch_lists<T, uint8_t, 8>(g, step, tiles, counts, st, st2, ev);
}

template <typename T, typename CI, bool PML, int TY, int NC>
hipError_t launch_tb2(const GridView<T>& g, int step, int kz, int run, int prev, hipStream_t st) {
  constexpr int GRP = 64 * (TY + 4) / PR_NT;
  const int ntx = (g.nx + 59) / 60, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + kz - 1) / kz;
  const bool many = g.n_probe > PR_MANY;
  const int npb = many ? 0 : (g.n_probe + GRP - 1) / GRP;
  const long long nb = (long long)ntx * nty * ntz + npb;
  if (nb > 0x7fffffff || (NC && g.ncls > NC)) return hipErrorInvalidValue;
  if (many) probes_tb2<T, CI, PML, false>(g, MarchDebye<T>{}, step, prev, st);
  hipLaunchKernelGGL((k_tb2<T, CI, PML, TY, NC>), dim3((unsigned)nb), dim3(64 * (TY + 4)), 0, st, g, step, kz, ntx, nty,
                     npb, prev, run);
  return hipGetLastError();
}

template <typename T, typename CI, int NC>
hipError_t step_tb2(const GridView<T>& g, int step, int ty, int kz, int run, int prev, hipStream_t st) {
  const bool pml = g.npml > 0;
  if (ty == 4)
    return pml ? launch_tb2<T, CI, true, 4, NC>(g, step, kz, run, prev, st)
               : launch_tb2<T, CI, false, 4, NC>(g, step, kz, run, prev, st);
  if (ty == 12)
    return pml ? launch_tb2<T, CI, true, 12, NC>(g, step, kz, run, prev, st)
               : launch_tb2<T, CI, false, 12, NC>(g, step, kz, run, prev, st);
  return pml ? launch_tb2<T, CI, true, 8, NC>(g, step, kz, run, prev, st)
             : launch_tb2<T, CI, false, 8, NC>(g, step, kz, run, prev, st);
}

int launch_tb2_pass(int prec, const void* view, int cls16, int step, int ty, int kz, int run, int prev,
                    void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (prec == 64) {
    const GridView<double>& g = *(const GridView<double>*)view;
    return (int)(cls16 ? step_tb2<double, uint16_t, 0>(g, step, ty, kz, run, prev, st)
                       : step_tb2<double, uint8_t, 256>(g, step, ty, kz, run, prev, st));
  }
  const GridView<float>& g = *(const GridView<float>*)view;
  // 2-byte ids: the table in LDS as far as it fits (us a step, in memory / in
  // LDS: 1,300 classes on 203 x 157 x 131 with a CPML 106 / 51, 384 x 384 x 288
  // with 420 610 / 361; 1,208 on 96 x 96 x 80 24.7 / 15.9)
  if (cls16 && g.ncls > TB2_NC1) return (int)step_tb2<float, uint16_t, 0>(g, step, ty, kz, run, prev, st);
  if (!cls16) return (int)step_tb2<float, uint8_t, 256>(g, step, ty, kz, run, prev, st);
  if (g.ncls <= TB2_NC2 && ty == 8 && g.npml == 0)
    return (int)launch_tb2<float, uint16_t, false, 8, TB2_NC2>(g, step, kz, run, prev, st);
  return (int)step_tb2<float, uint16_t, TB2_NC1>(g, step, ty, kz, run, prev, st);
}

template <typename T>
hipError_t step_any(const GridView<T>& g, int cls16, int variant, int step, int tile_y, int tile_z,
                    hipStream_t st) {
  if (variant == 2)
    return cls16 ? step_fused<T, uint16_t>(g, step, tile_y, tile_z, st)
                 : step_fused<T, uint8_t>(g, step, tile_y, tile_z, st);
  return cls16 ? step_split<T, uint16_t>(g, step, st) : step_split<T, uint8_t>(g, step, st);
}

int launch_lists_step(int prec, const void* view, int cls16, int step, int tile_y, const void* tiles,
                      const int* counts, void* stream, void* stream2, void* ev_src) {
  hipStream_t st = (hipStream_t)stream, st2 = (hipStream_t)stream2;
  const int4* t = (const int4*)tiles;
  const int ty = tile_y == 4 ? 4 : 8;
  hipError_t e = prec == 64 ? lists_any<double>(*(const GridView<double>*)view, cls16, step, ty, t, counts, st, st2,
                                                ev_src)
                            : lists_any<float>(*(const GridView<float>*)view, cls16, step, ty, t, counts, st, st2,
                                               ev_src);
  return (int)e;
}

int launch_step(int prec, const void* view, int cls16, int variant, int step, int tile_y, int tile_z,
                void* stream) {
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  if (prec == 64)
    e = step_any<double>(*(const GridView<double>*)view, cls16, variant, step, tile_y, tile_z, st);
  else
    e = step_any<float>(*(const GridView<float>*)view, cls16, variant, step, tile_y, tile_z, st);
  return (int)e;
}

template <typename T>
hipError_t probes_any(const GridView<T>& g, int step, hipStream_t st) {
  if (g.n_probe <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_probes<T>), dim3((unsigned)g.n_probe), dim3(PR_NT), 0, st, g, step);
  return hipGetLastError();
}

int launch_probes(int prec, const void* view, int step, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (prec == 64) return (int)probes_any<double>(*(const GridView<double>*)view, step, st);
  return (int)probes_any<float>(*(const GridView<float>*)view, step, st);
}

template <typename T, typename CI, bool PML>
hipError_t batch_step_t(const void* views, const void* tiles, int n_tiles, int tx, int ty, const int* d_step,
                        int offset, hipStream_t st) {
  const GridView<T>* v = (const GridView<T>*)views;
  const int4* t = (const int4*)tiles;
  if (tx == 32 && ty == 8)
    hipLaunchKernelGGL((k_fused_batch<T, CI, PML, 32, 8>), dim3(n_tiles), dim3(256), 0, st, v, t, d_step, offset);
  else if (tx == 32 && ty == 16)
    hipLaunchKernelGGL((k_fused_batch<T, CI, PML, 32, 16>), dim3(n_tiles), dim3(512), 0, st, v, t, d_step, offset);
  else if (tx == 64 && ty == 8)
    hipLaunchKernelGGL((k_fused_batch<T, CI, PML, 64, 8>), dim3(n_tiles), dim3(512), 0, st, v, t, d_step, offset);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

int launch_batch_step(int prec, int cls16, int pml, const void* views, const void* tiles, int n_tiles, int tx,
                      int ty, const int* d_step, int offset, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (n_tiles <= 0) return 0;
  hipError_t e;
  if (prec == 64) {
    if (cls16) e = pml ? batch_step_t<double, uint16_t, true>(views, tiles, n_tiles, tx, ty, d_step, offset, st)
                       : batch_step_t<double, uint16_t, false>(views, tiles, n_tiles, tx, ty, d_step, offset, st);
    else e = pml ? batch_step_t<double, uint8_t, true>(views, tiles, n_tiles, tx, ty, d_step, offset, st)
                 : batch_step_t<double, uint8_t, false>(views, tiles, n_tiles, tx, ty, d_step, offset, st);
  } else {
    if (cls16) e = pml ? batch_step_t<float, uint16_t, true>(views, tiles, n_tiles, tx, ty, d_step, offset, st)
                       : batch_step_t<float, uint16_t, false>(views, tiles, n_tiles, tx, ty, d_step, offset, st);
    else e = pml ? batch_step_t<float, uint8_t, true>(views, tiles, n_tiles, tx, ty, d_step, offset, st)
                 : batch_step_t<float, uint8_t, false>(views, tiles, n_tiles, tx, ty, d_step, offset, st);
  }
  return (int)e;
}

int launch_batch_probes(int prec, const void* views, const void* plist, int n, const int* d_step, int offset,
                        void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (n <= 0) return 0;
  const dim3 grd((unsigned)n), blk(PR_NT);
  if (prec == 64)
    hipLaunchKernelGGL((k_probes_batch<double>), grd, blk, 0, st, (const GridView<double>*)views,
                       (const int2*)plist, n, d_step, offset);
  else
    hipLaunchKernelGGL((k_probes_batch<float>), grd, blk, 0, st, (const GridView<float>*)views,
                       (const int2*)plist, n, d_step, offset);
  return (int)hipGetLastError();
}

template <typename T, typename CI, int NC>
hipError_t batch_pass_t(const void* views, const void* tiles, int n_tiles, const void* plist, int n_probes,
                        const int* d_step, int offset, int prev, int run, hipStream_t st) {
  const bool many = n_probes > PR_MANY;
  const int npb = many ? 0 : (n_probes + 768 / PR_NT - 1) / (768 / PR_NT);
  if (many)
    hipLaunchKernelGGL((k_probes_tb2_batch<T, CI>), dim3((unsigned)n_probes), dim3(PR_NT), 0, st,
                       (const GridView<T>*)views, (const int2*)plist, n_probes, d_step, offset, prev);
  hipLaunchKernelGGL((k_tb2_batch<T, CI, NC>), dim3((unsigned)(npb + n_tiles)), dim3(768), 0, st,
                     (const GridView<T>*)views, (const int4*)tiles, (const int2*)plist, n_probes, npb, d_step, offset,
                     prev, run);
  return hipGetLastError();
}

int launch_batch_pass(int prec, int cls16, int ncls, const void* views, const void* tiles, int n_tiles, const void* plist,
                      int n_probes, const int* d_step, int offset, int prev, int run, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  const auto pass = [&](auto f) {
    return f(views, tiles, n_tiles, plist, n_probes, d_step, offset, prev, run, st);
  };
  if (prec == 64)
    e = pass(cls16 ? batch_pass_t<double, uint16_t, 0> : batch_pass_t<double, uint8_t, 256>);
  else
    e = pass(cls16 && ncls > TB2_NC1 ? batch_pass_t<float, uint16_t, 0>
             : !cls16                ? batch_pass_t<float, uint8_t, 256>
                                     : batch_pass_t<float, uint16_t, TB2_NC1>);
  return (int)e;
}

__global__ void k_set(int* p, int v) {
  if (threadIdx.x == 0) *p = v;
}

int launch_set(int* d, int v, void* stream) {
  hipLaunchKernelGGL(k_set, dim3(1), dim3(64), 0, (hipStream_t)stream, d, v);
  return (int)hipGetLastError();
}

int launch_add(int* d, int v, void* stream) {
  hipLaunchKernelGGL(k_add, dim3(1), dim3(64), 0, (hipStream_t)stream, d, v);
  return (int)hipGetLastError();
}

}  // namespace mi355fdtd
