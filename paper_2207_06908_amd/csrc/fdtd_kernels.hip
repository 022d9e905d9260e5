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
// temporally blocked variant: two steps per pass
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

// One two-step tile in the CPML: outputs [i0, i0+iw) x [j0, j0+jh) x [k0, k1)
// with iw <= 60, jh <= TY.  FP64 grids run their slab tiles through this one,
// a plane of every stage at a time (tb2_any).
template <typename T, typename CI, int TY>
__device__ __forceinline__ void tb2_tile(const GridView<T>& g, TB2Smem<T, TY>& sm, int i0, int j0, int iw, int jh,
                                         int k0, int k1, int step) {
  constexpr int TX = 60, NT = 64 * (TY + 4);
  constexpr bool LDS_TAB = sizeof(CI) == 1;
  const int tid = threadIdx.x, u = tid & 63, v = tid >> 6;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const unsigned sxy = (unsigned)g.sxy;
  const CI* cls = (const CI*)g.cls;
  if (LDS_TAB) {
    for (int q = tid; q < g.ncls * K_STRIDE; q += NT) sm.stab[q] = ldg(g.ctab, (unsigned)q);
  }
  auto coef = [&](int c) -> const T* { return LDS_TAB ? sm.stab + c * K_STRIDE : g.ctab + c * K_STRIDE; };

  const int x = i0 - 2 + u, y = j0 - 2 + v;
  const bool dom = x >= 0 && x < nx && y >= 0 && y < ny;
  const bool inA = dom && u <= TX + 2 && v <= TY + 2;
  const bool inB = inA && u >= 1 && v >= 1;
  const bool inC = inB && u <= TX + 1 && v <= TY + 1;
  const bool inD = inC && u >= 2 && v >= 2 && u < 2 + iw && v < 2 + jh;
  const unsigned n0 = dom ? (unsigned)x + (unsigned)nx * (unsigned)y : 0u;
  const int lx = dom ? slab_pos(x, nx, g.npml) : -1;
  const int ly = dom ? slab_pos(y, ny, g.npml) : -1;
  // (E is updated on planes k0 - 1 .. k1: the first step's cone, then the outputs)
  const SrcRange srcr = src_wave(g, n0, inB, k0 - 1, k1);
  const int tn = 2 * g.npml;
  if (v == 0) {
    const int xl = x >= 0 && x < nx ? slab_pos(x, nx, g.npml) : -1;
    for (int r = 0; r < P_NROW; ++r) sm.px[r][u] = xl >= 0 ? ldg(g.prof[0], (unsigned)(r * tn + xl)) : T(0);
  }
  if (u == 0) {
    const int yl = y >= 0 && y < ny ? slab_pos(y, ny, g.npml) : -1;
    for (int r = 0; r < P_NROW; ++r) sm.py[r][v] = yl >= 0 ? ldg(g.prof[1], (unsigned)(r * tn + yl)) : T(0);
  }
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
    const int lz = slab_pos(k, nz, g.npml);
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
        e_sources(&g, srcr.first(k), srcr.last(k), n0 + sxy * (unsigned)k, step, e1c);
      };
      if (lz >= 0) {
        const int l[3] = {lx, ly, lz};
        stage_b(l);
      } else {
        const int l[3] = {lx, ly, -1};
        stage_b(l);
      }
    }
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
      int l[3] = {lx, ly, slab_pos(km, nz, g.npml)};
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
    if (inD && km >= k0) {
      const unsigned nst = n0 + sxy * (unsigned)km;
      T e2[3];
      int l[3] = {lx, ly, slab_pos(km, nz, g.npml)};
      e_core_pf<T, true>(pf, l, coef(cp), h2c[0], h2c[1], h2c[2], sm.sh2[0][v - 1][u], h2p[0], sm.sh2[1][v][u - 1],
                        h2p[1], sm.sh2[2][v][u - 1], sm.sh2[2][v - 1][u], e1p, pse[0], pse[1], pse[2], e2);
      e_sources(&g, srcr.first(km), srcr.last(km), nst, step + 1, e2);
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

// ---------------------------------------------------------------------------
// The two-step tile of k_tb2: 64 x (TY + 4) points around a 60 x TY output
// tile, two barriers per plane.  Iteration k runs two phases, a barrier after
// each:
//   X  H^{n+1/2} of plane k (stage A) and E^{n+2} of plane k-2 (stage D);
//   Y  E^{n+1} of plane k (B) and H^{n+3/2} of plane k-1 (C).
// The two stages of a phase do not depend on each other.  Neighbours along x
// are lanes of the same wave (cross-lane moves), those along z stay in the
// thread's registers, and only the components that y neighbours need go
// through LDS: E^n (x, z) for A, H^{n+1/2} (x, z) for B, E^{n+1} (x, z) for C,
// H^{n+3/2} (x, z) for D.
//
// One block runs on a CU at a time (58 KB of LDS, up to 16 waves of at most
// 128 registers), and with everything in the caches a plane costs what its
// instructions cost, so the loop is built to issue few: uniform bases with
// one 32-bit offset per plane; points and planes outside the grid are not
// branched around (their coefficients are the table's zero row); registers
// rotate by name over three unrolled iterations, not by copies; what is
// needed rarely is read again where it is needed (ColdView).  A lane outside a stage's region
// computes a value that no lane inside reads.
//
// Measured (us per step, against one launch per CPML group of 8-row tiles
// with three barriers, four LDS planes and 2.5 times the instructions):
// 512 x 512 x 384 with a 10-cell CPML 743 (891), 203 x 157 x 131 44 (116),
// 96 x 96 x 80 14.5 (82), 48^3 without one 4.3 (38, the fused pass).  In the
// caches a plane of an 8-row tile takes 0.92 us clear of the CPML and 1.7 us
// in it; on the largest grid 12 rows take 2 us, bound by the 5 TB/s that
// the tiles draw through the L2s (a copy reaches 5.1).
// ---------------------------------------------------------------------------

template <typename T, int TY>
struct MarchSmem {
  static constexpr int R = TY + 4;
  static constexpr int PZ = 512 / sizeof(T);  // longest z profile row held here (2 npml)
  T e0[2][R][64];       // E^n (x, z), plane k
  T h1[2][R][64];       // H^{n+1/2} (x, z), plane k
  T e1[2][2][R][64];    // E^{n+1} (x, z), planes k and k-1
  T h2[2][R][64];       // H^{n+3/2} (x, z), plane k-2
  T stab[257 * K_STRIDE];  // a row of zeros, then the classes' coefficients
  T px[P_NROW][64];     // CPML profile at each lane's x
  T pz[P_NROW * PZ];    // the z table
};

// CPML profile values of a tile's points: a lane's x values in registers
// (tiles of up to 8 rows, which have them to spare) or LDS, the row's y
// values in scalar registers, z from LDS.
template <typename T, int TY>
struct ProfMarch {
  static constexpr bool XREG = TY <= 8;
  const MarchSmem<T, TY>& sm;
  int tn, u;
  T x[XREG ? P_NROW : 1];
  T y[P_NROW];  // uniform across the wave
  template <int U>
  __device__ __forceinline__ Prof3<T> at(int row, int l) const {
    if (U == 0 && XREG) return row == P_BE ? Prof3<T>{x[0], x[1], x[2]} : Prof3<T>{x[3], x[4], x[5]};
    if (U == 0) return {sm.px[row][u], sm.px[row + 1][u], sm.px[row + 2][u]};
    if (U == 1) return row == P_BE ? Prof3<T>{y[0], y[1], y[2]} : Prof3<T>{y[3], y[4], y[5]};
    const int q = row * tn + l;
    return {sm.pz[q], sm.pz[q + tn], sm.pz[q + 2 * tn]};
  }
};

// A wave-uniform value in a scalar register.
__device__ __forceinline__ float uniform(float v) {
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}
__device__ __forceinline__ double uniform(double v) {
  const unsigned long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The value of lane u + 1 (CTRL 0x130, wave_shl:1) or u - 1 (0x138,
// wave_shr:1); 0 past the wave's ends.  Every lane must be active.
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename T>
__device__ __forceinline__ T next_lane(T v) { return lane_shift<0x130>(v); }
template <typename T>
__device__ __forceinline__ T prev_lane(T v) { return lane_shift<0x138>(v); }

// A view whose members are read where they are used (by scalar loads), not
// kept in scalar registers over the whole march.
template <typename T>
struct ColdView {
  typedef const __attribute__((address_space(4))) GridView<T>* P;
  P p;
  __device__ __forceinline__ P operator->() const {
    P q = p;
    asm volatile("" : "+s"(q));
    return q;
  }
};

// A copy of the view behind p, read by scalar loads: p is the same for the
// whole block, which the compiler does not see where a table of views is
// indexed by a loaded value (it would hold every pointer in vector registers).
template <typename T>
__device__ __forceinline__ GridView<T> uniform_view(const GridView<T>* p) {
  static_assert(sizeof(GridView<T>) % 8 == 0, "copied in 8-byte words");
  constexpr int N = sizeof(GridView<T>) / 8;
  const uint64_t a = (uint64_t)(uintptr_t)p;
  const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32;
  typedef const __attribute__((address_space(4))) uint64_t* W;
  const W w = (W)u;
  struct {
    uint64_t q[N];
  } v;
#pragma unroll
  for (int i = 0; i < N; ++i) v.q[i] = w[i];
  return __builtin_bit_cast(GridView<T>, v);
}

// The state of one thread's point, registers named by plane modulo 3.
template <typename T>
struct MarchRegs {
  T e0[3][3];       // E^n
  T h0[3][3];       // H^{n-1/2}
  T h1[3][3];       // H^{n+1/2}
  T e1[3][3];       // E^{n+1}
  T h2[3][3];       // H^{n+3/2}
  T e2[3];          // E^{n+2} of D
  typedef T Pair __attribute__((ext_vector_type(2)));
  Pair ph[3][3];    // CPML state, H-type [plane][axis]
  Pair pe[3][3];    // E-type
  unsigned co[3];   // LDS row (in values) of the class
};

// One tile: outputs [i0, i0 + iw) x [j0, j0 + jh) x [k0, k1) with iw <= 60,
// jh <= TY; AX masks the axes whose CPML slabs the tile's region reaches.
//
// Points outside the grid read the column (0, 0), whose E is 0 (it lies on
// two walls); planes below the grid read plane 0, planes above it the last
// one, with E set to 0.  With the zero row as their coefficients their E
// stays 0, as the upper walls need; their H only meets the lower walls'
// zero coefficients.
template <typename T, typename CI, int TY, int AX>
struct March {
  static constexpr int TX = 60, NT = 64 * (TY + 4);
  static constexpr bool LDS_TAB = sizeof(CI) == 1;
  static constexpr bool PML = AX != 0, SX = AX & 1, SY = AX & 2, SZ = AX & 4;
  static constexpr unsigned S = sizeof(T), NONE = 0xFFFFFFFFu;

  typedef typename MarchRegs<T>::Pair Pair;
  MarchSmem<T, TY>& sm;
  ColdView<T> g;
  const T* fi[6];
  T* fo[6];
  const CI* cls;
  int nz, np, u, v, step, k0, k1;
  int lx, ly;
  unsigned n0, n0s, sxy;           // column index, its byte offset; nodes per plane
  bool dom, inD;
  // CPML state: bases, the output set's distance (values), and per axis the
  // column's byte offset, the step per plane (x, y) and the H-type pairs'
  // distance
  const T* pib[3];
  ptrdiff_t pout;
  unsigned qx, qy, qz, dx, dy, dkind[3];
  int lz[3];                       // z slab position of the planes in the three slots
  SrcRange srcr;
  ProfMarch<T, TY> pf;
  MarchRegs<T> r;
  unsigned craw;

  // coefficients [F, F + N) of a class row
  template <int F, int N>
  __device__ __forceinline__ void coef(unsigned row, T* cf) const {
#pragma unroll
    for (int q = 0; q < N; ++q)
      cf[F + q] = LDS_TAB ? sm.stab[row + F + q] : row == NONE ? T(0) : ldg(g->ctab, row + F + q);
  }
  // the row of a class id; the zero row for points and planes outside the grid
  __device__ __forceinline__ unsigned row_of(unsigned c, bool in) const {
    return LDS_TAB ? (in ? (c + 1u) * K_STRIDE : 0u) : (in ? c * K_STRIDE : NONE);
  }
  // Both kinds of CPML state of plane k (z slab position lz): H-type into
  // ph, E-type into pe (values outside the slabs are not used); and back.
  template <int A, bool LOAD>
  __device__ __forceinline__ void psi_axis(bool on, unsigned off, Pair& ph, Pair& pe) const {
    const Pair* p = (const Pair*)(LOAD ? pib[A] : pib[A] + pout);
    Pair h = ph, e = pe;
    if (on && LOAD) {
      e = ldb(p, off);
      h = ldb(p, off + dkind[A]);
    } else if (on) {
      stb((Pair*)p, off, e);
      stb((Pair*)p, off + dkind[A], h);
    }
    if (LOAD) {
      pe = e;
      ph = h;
    }
  }
  template <bool LOAD>
  __device__ __forceinline__ void psi(int k, int lzk, Pair (&ph)[3], Pair (&pe)[3]) const {
    if (SX) psi_axis<0, LOAD>(lx >= 0, qx + (unsigned)k * dx, ph[0], pe[0]);
    if (SY) psi_axis<1, LOAD>(ly >= 0, qy + (unsigned)k * dy, ph[1], pe[1]);
    if (SZ) psi_axis<2, LOAD>(lzk >= 0, qz + (unsigned)lzk * (sxy * 2u * S), ph[2], pe[2]);
  }

  // H of plane k (A and C): e and en the E of planes k and k + 1, le the
  // plane's E (x, z) in LDS.
  __device__ __forceinline__ void stage_h(int lzk, unsigned row, const T e[3], const T en[3], const T (*le)[TY + 4][64],
                                          const T hold[3], Pair (&pp)[3], T hn[3]) const {
    T cf[K_STRIDE];
    coef<K_DBX, 3>(row, cf);
    T p0[2], p1[2], p2[2];
    if (SX) p0[0] = pp[0].x, p0[1] = pp[0].y;
    if (SY) p1[0] = pp[1].x, p1[1] = pp[1].y;
    if (SZ) p2[0] = pp[2].x, p2[1] = pp[2].y;
    const int l[3] = {SX ? lx : -1, SY ? ly : -1, SZ ? lzk : -1};
    h_core_pf<T, PML>(pf, l, cf, e[0], e[1], e[2], le[0][v + 1][u], en[0], next_lane(e[1]), en[1], next_lane(e[2]),
                      le[1][v + 1][u], hold, p0, p1, p2, hn);
    if (SX) pp[0] = Pair{p0[0], p0[1]};
    if (SY) pp[1] = Pair{p1[0], p1[1]};
    if (SZ) pp[2] = Pair{p2[0], p2[1]};
  }
  // E of plane k (B and D): h and hp the H of planes k and k - 1, lh the
  // plane's H (x, z) in LDS.
  __device__ __forceinline__ void stage_e(int k, int lzk, unsigned row, const T h[3], const T hp[3], const T (*lh)[TY + 4][64],
                                          const T eold[3], int st, Pair (&pp)[3], T en[3]) const {
    T cf[K_STRIDE];
    coef<K_CAX, 6>(row, cf);
    T p0[2], p1[2], p2[2];
    if (SX) p0[0] = pp[0].x, p0[1] = pp[0].y;
    if (SY) p1[0] = pp[1].x, p1[1] = pp[1].y;
    if (SZ) p2[0] = pp[2].x, p2[1] = pp[2].y;
    const int l[3] = {SX ? lx : -1, SY ? ly : -1, SZ ? lzk : -1};
    e_core_pf<T, PML>(pf, l, cf, h[0], h[1], h[2], lh[0][v - 1][u], hp[0], prev_lane(h[1]), hp[1], prev_lane(h[2]),
                      lh[1][v - 1][u], eold, p0, p1, p2, en);
    if (SX) pp[0] = Pair{p0[0], p0[1]};
    if (SY) pp[1] = Pair{p1[0], p1[1]};
    if (SZ) pp[2] = Pair{p2[0], p2[1]};
    if (k >= srcr.klo && k <= srcr.khi)  // uniform
      e_sources(g, srcr.lo, srcr.hi, dom ? n0 + sxy * (unsigned)k : NONE, st, en);
  }

  // Iteration k, the registers of plane k in slot Q; with TAIL only what is
  // left after the last plane: D and the outputs of plane k1 - 1.
  template <int Q, bool TAIL>
  __device__ __forceinline__ void iter(int k) {
    constexpr int N1 = (Q + 1) % 3, P1 = (Q + 2) % 3, P2 = N1;  // slots of planes k+1, k-1 and k-2
    if (!TAIL) {
      // loads: class and H of plane k+1, E of plane k+2 (plane k-1's slot)
      r.co[Q] = row_of(craw, dom && k >= 0 && k < nz);
      if (k + 1 >= nz) r.e0[N1][0] = r.e0[N1][1] = r.e0[N1][2] = T(0);
      const unsigned ph = (unsigned)min(max(k + 1, 0), nz - 1) * sxy, pe = (unsigned)min(max(k + 2, 0), nz - 1) * sxy;
      craw = ldg(cls, n0 + ph);
#pragma unroll
      for (int c = 0; c < 3; ++c) r.h0[N1][c] = ldb(fi[3 + c], n0s + ph * S);
#pragma unroll
      for (int c = 0; c < 3; ++c) r.e0[P1][c] = ldb(fi[c], n0s + pe * S);
      // X: A of plane k, D of plane k-2
      if (v <= TY + 2) {
        stage_h(lz[Q], r.co[Q], r.e0[Q], r.e0[N1], sm.e0, r.h0[Q], r.ph[Q], r.h1[Q]);
        sm.h1[0][v][u] = r.h1[Q][0];
        sm.h1[1][v][u] = r.h1[Q][2];
      }
    }
    if (v >= 2 && v <= TY + 1 && k - 2 >= k0)
      stage_e(k - 2, lz[P2], r.co[P2], r.h2[P2], r.h2[Q], sm.h2, r.e1[P2], step + 1, r.pe[P2], r.e2);
    if (!TAIL) __syncthreads();
    // the outputs of plane k-2
    if (inD && k - 2 >= k0) {
      const unsigned o = n0s + (unsigned)(k - 2) * sxy * S;
#pragma unroll
      for (int c = 0; c < 3; ++c) stb(fo[c], o, r.e2[c]);
#pragma unroll
      for (int c = 0; c < 3; ++c) stb(fo[3 + c], o, r.h2[P2][c]);
      if (PML) psi<false>(k - 2, lz[P2], r.ph[P2], r.pe[P2]);
    }
    if (TAIL) {
      // (keeps the compiler from merging the three slots' tails, which would
      // put the registers they store into memory)
      asm volatile("" ::"i"(Q));
      return;
    }
    if (PML && k + 1 < nz) {  // (planes outside the grid keep finite values that no output sees)
      lz[N1] = SZ ? slab_pos(k + 1, nz, np) : -1;
      if (k + 1 >= 0) psi<true>(k + 1, lz[N1], r.ph[N1], r.pe[N1]);
    } else if (PML) {
      lz[N1] = -1;
    }
    // Y: B of plane k, C of plane k-1
    const int s1 = k & 1, s1m = s1 ^ 1;
    if (v >= 1 && v <= TY + 2 && k >= k0 - 1) {
      stage_e(k, lz[Q], r.co[Q], r.h1[Q], r.h1[P1], sm.h1, r.e0[Q], step, r.pe[Q], r.e1[Q]);
      if (v <= TY + 1 && k >= k0) {
        stage_h(lz[P1], r.co[P1], r.e1[P1], r.e1[Q], sm.e1[s1m], r.h1[P1], r.ph[P1], r.h2[P1]);
        sm.h2[0][v][u] = r.h2[P1][0];
        sm.h2[1][v][u] = r.h2[P1][2];
      }
      sm.e1[s1][0][v][u] = r.e1[Q][0];
      sm.e1[s1][1][v][u] = r.e1[Q][2];
    }
    sm.e0[0][v][u] = k + 1 >= nz ? T(0) : r.e0[N1][0];
    sm.e0[1][v][u] = k + 1 >= nz ? T(0) : r.e0[N1][2];
    __syncthreads();
  }

  __device__ __forceinline__ March(const GridView<T>& gv, ColdView<T> cold, MarchSmem<T, TY>& sm_, int i0, int j0,
                                   int iw, int jh, int k0_, int k1_, int step_)
      : sm(sm_), g(cold), nz(gv.nz), np(gv.npml), step(step_), k0(k0_), k1(k1_),
        pf{sm_, 0, 0, {}, {}} {
    const int tid = threadIdx.x, nx = gv.nx, ny = gv.ny;
    u = tid & 63;
    v = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (LDS_TAB) {
      if (tid < K_STRIDE) sm.stab[tid] = T(0);
      for (int q = tid; q < gv.ncls * K_STRIDE; q += NT) sm.stab[K_STRIDE + q] = ldg(gv.ctab, (unsigned)q);
    }
    const int x = i0 - 2 + u, y = j0 - 2 + v;
    dom = x >= 0 && x < nx && y >= 0 && y < ny;
    inD = dom && u >= 2 && u < 2 + iw && v >= 2 && v < 2 + jh;
    sxy = (unsigned)gv.sxy;
    n0 = dom ? (unsigned)x + (unsigned)nx * (unsigned)y : 0u;
    n0s = n0 * S;
    lx = SX && dom ? slab_pos(x, nx, np) : -1;
    ly = SY && y >= 0 && y < ny ? slab_pos(y, ny, np) : -1;  // uniform across the wave
    srcr = src_wave(gv, n0, dom && u >= 1 && u <= TX + 2 && v >= 1 && v <= TY + 2, k0 - 1, k1);
    pf.tn = 2 * np;
    pf.u = u;
    if (PML) {
      const int tn = 2 * np;
      if (SX) {
        const int xl = x >= 0 && x < nx ? slab_pos(x, nx, np) : -1;
#pragma unroll
        for (int q = 0; q < P_NROW; ++q) {
          if (pf.XREG) pf.x[q] = xl >= 0 ? ldg(gv.prof[0], (unsigned)(q * tn + xl)) : T(0);
          else if (v == 0) sm.px[q][u] = xl >= 0 ? ldg(gv.prof[0], (unsigned)(q * tn + xl)) : T(0);
        }
      }
#pragma unroll
      for (int q = 0; q < P_NROW; ++q) pf.y[q] = SY && ly >= 0 ? uniform(ldg(gv.prof[1], (unsigned)(q * tn + ly))) : T(0);
      if (SZ)
        for (int q = tid; q < P_NROW * tn; q += NT) sm.pz[q] = ldg(gv.prof[2], (unsigned)q);
      constexpr unsigned P = 2 * S;  // bytes of a pair
      dx = 2u * np * (unsigned)ny * P;
      dy = 2u * np * (unsigned)nx * P;
      qx = SX ? ((unsigned)max(lx, 0) + 2u * np * (unsigned)(dom ? y : 0)) * P : 0u;
      qy = SY ? ((unsigned)(dom ? x : 0) + (unsigned)nx * (unsigned)max(ly, 0)) * P : 0u;
      qz = n0 * P;
      pout = gv.pob[0] - gv.pib[0];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        pib[a] = gv.pib[a];
        asm volatile("" : "+s"(pib[a]));  // (kept, not read again in every plane)
        dkind[a] = gv.pel[a] * P;
      }
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      fi[c] = gv.fi[c];
      fo[c] = gv.fo[c];
    }
    cls = (const CI*)gv.cls;
    // plane kb, and E of plane kb + 1
    const int kb = k0 - 2;
    const unsigned pa = (unsigned)max(kb, 0) * sxy, pb = (unsigned)min(max(kb + 1, 0), nz - 1) * sxy;
    craw = ldg(cls, n0 + pa);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r.h0[0][c] = ldb(fi[3 + c], n0s + pa * S);
      r.e0[0][c] = ldb(fi[c], n0s + pa * S);
      r.e0[1][c] = ldb(fi[c], n0s + pb * S);
    }
    if (PML) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int a = 0; a < 3; ++a) r.ph[q][a] = r.pe[q][a] = Pair{T(0), T(0)};
      lz[0] = SZ && kb >= 0 ? slab_pos(kb, nz, np) : -1;
      lz[1] = lz[2] = -1;
      if (kb >= 0) psi<true>(kb, lz[0], r.ph[0], r.pe[0]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) r.h1[q][c] = r.e1[q][c] = r.h2[q][c] = r.e2[c] = T(0);
    r.co[1] = r.co[2] = row_of(0, false);
    sm.e0[0][v][u] = r.e0[0][0];
    sm.e0[1][v][u] = r.e0[0][2];
    __syncthreads();
    for (int k = kb;;) {
      iter<0, false>(k);
      if (++k > k1) { iter<1, true>(k); break; }
      iter<1, false>(k);
      if (++k > k1) { iter<2, true>(k); break; }
      iter<2, false>(k);
      if (++k > k1) { iter<0, true>(k); break; }
    }
  }
};

// Probes of a two-step pass: the intermediate step's values are recomputed
// point by point from the input set (which the pass leaves untouched) with
// the same per-point arithmetic; the second step's values are read from the
// output set.
template <typename T, typename CI, bool PML>
__device__ __forceinline__ void h1_at(const GridView<T>& g, int x, int y, int k, T h[3]) {
  h[0] = h[1] = h[2] = T(0);
  if (x < 0 || y < 0 || k < 0 || x >= g.nx || y >= g.ny || k >= g.nz) return;
  const unsigned n = (unsigned)x + (unsigned)g.nx * ((unsigned)y + (unsigned)g.ny * (unsigned)k);
  const T* cf = g.ctab + (int)ldg((const CI*)g.cls, n) * K_STRIDE;
  const T ex = ldg(g.fi[0], n), ey = ldg(g.fi[1], n), ez = ldg(g.fi[2], n);
  const T ex_j = (y + 1 < g.ny) ? ldg(g.fi[0], n + (unsigned)g.nx) : T(0);
  const T ex_k = (k + 1 < g.nz) ? ldg(g.fi[0], n + (unsigned)g.sxy) : T(0);
  const T ey_i = (x + 1 < g.nx) ? ldg(g.fi[1], n + 1) : T(0);
  const T ey_k = (k + 1 < g.nz) ? ldg(g.fi[1], n + (unsigned)g.sxy) : T(0);
  const T ez_i = (x + 1 < g.nx) ? ldg(g.fi[2], n + 1) : T(0);
  const T ez_j = (y + 1 < g.ny) ? ldg(g.fi[2], n + (unsigned)g.nx) : T(0);
  const T hold[3] = {ldg(g.fi[3], n), ldg(g.fi[4], n), ldg(g.fi[5], n)};
  int l[3] = {-1, -1, -1};
  T ps[3][2];
  if (PML) {
    slabs(g, x, y, k, l);
    psi_load(g, 1, l, x, y, k, ps);
  }
  h_core<T, PML>(g, l, cf, ex, ey, ez, ex_j, ex_k, ey_i, ey_k, ez_i, ez_j, hold, ps, h);
}

template <typename T, typename CI, bool PML>
__device__ __forceinline__ void e1_at(const GridView<T>& g, int x, int y, int k, int step, T e[3]) {
  const unsigned n = (unsigned)x + (unsigned)g.nx * ((unsigned)y + (unsigned)g.ny * (unsigned)k);
  T h[3], hi[3], hj[3], hk[3];
  h1_at<T, CI, PML>(g, x, y, k, h);
  h1_at<T, CI, PML>(g, x - 1, y, k, hi);
  h1_at<T, CI, PML>(g, x, y - 1, k, hj);
  h1_at<T, CI, PML>(g, x, y, k - 1, hk);
  const T* cf = g.ctab + (int)ldg((const CI*)g.cls, n) * K_STRIDE;
  const T eold[3] = {ldg(g.fi[0], n), ldg(g.fi[1], n), ldg(g.fi[2], n)};
  int l[3] = {-1, -1, -1};
  T ps[3][2];
  if (PML) {
    slabs(g, x, y, k, l);
    psi_load(g, 0, l, x, y, k, ps);
  }
  const SrcRange sr = src_node(g, x, y, k);
  e_core<T, PML>(g, l, n, cf, h[0], h[1], h[2], hj[0], hk[0], hi[1], hk[1], hi[2], hj[2], eold, step, ps, e, sr.lo,
                 sr.hi);
}

// Probes: PR_NT threads per probe (a block, or one of several groups of a
// larger block).  Thread `t` of the group sums terms t, t + PR_NT, ... of the
// probe in order; the lanes of each wave are then summed by a shuffle tree
// and the four wave sums in order.  Every probe kernel sums in this one FP64
// order, so that all variants, and a batch and its grids run alone, agree bit
// for bit.
constexpr int PR_NT = 256;

// Sum of `a` over the group's threads in the fixed order; `red` holds the
// group's 4 doubles of LDS.  The total is returned to every thread.
__device__ __forceinline__ double probe_sum(double a, int t, double* red) {
  for (int o = 32; o > 0; o >>= 1) a += __shfl_down(a, o, 64);
  if ((t & 63) == 0) red[t >> 6] = a;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// Probe p of a two-step pass: sample `step`, recomputed from the input set
// (which the pass leaves untouched), and with S2 sample `step` + 1, read from
// the output set.  Thread t of the group; groups past the last probe (p = -1)
// only keep the block's barriers.  `red` holds the group's 8 doubles of LDS.
template <typename T, typename CI, bool PML, bool S2>
__device__ __forceinline__ void probe_tb2(const GridView<T>& g, int p, int step, int t, double* red) {
  double a1 = 0.0, a2 = 0.0;
  const int q0 = p < 0 ? 0 : g.pr_off[p], q1 = p < 0 ? 0 : g.pr_off[p + 1];
  for (int q = q0 + t; q < q1; q += PR_NT) {
    const int c = g.term_comp[q];
    const unsigned n = (unsigned)g.term_idx[q];
    const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny), k = (int)(n / g.sxy);
    T v3[3];
    if (c < 3) e1_at<T, CI, PML>(g, x, y, k, step, v3);
    else h1_at<T, CI, PML>(g, x, y, k, v3);
    const int cc = c < 3 ? c : c - 3;
    const T v1 = cc == 0 ? v3[0] : cc == 1 ? v3[1] : v3[2];
    a1 += g.term_w[q] * (double)v1;
    if (S2) {
      const T* f = c == 0 ? g.fo[0] : c == 1 ? g.fo[1] : c == 2 ? g.fo[2] : c == 3 ? g.fo[3] : c == 4 ? g.fo[4] : g.fo[5];
      a2 += g.term_w[q] * (double)ldg((const T*)f, n);
    }
  }
  a1 = probe_sum(a1, t, red);
  if (S2) a2 = probe_sum(a2, t, red + 4);
  if (t == 0 && p >= 0) {
    g.pr_out[(long long)p * g.max_steps + step] = a1;
    if (S2) g.pr_out[(long long)p * g.max_steps + step + 1] = a2;
  }
}

// Probe p at sample `step` from the view's input fields (p = -1: none).
template <typename T>
__device__ __forceinline__ void probe_one(const GridView<T>& g, int p, int step, int t, double* red) {
  double acc = 0.0;
  const int q0 = p < 0 ? 0 : g.pr_off[p], q1 = p < 0 ? 0 : g.pr_off[p + 1];
  for (int q = q0 + t; q < q1; q += PR_NT) {
    const int c = g.term_comp[q];
    const T* f = c == 0 ? g.fi[0] : c == 1 ? g.fi[1] : c == 2 ? g.fi[2] : c == 3 ? g.fi[3] : c == 4 ? g.fi[4] : g.fi[5];
    acc += g.term_w[q] * (double)ldg(f, (unsigned)g.term_idx[q]);
  }
  acc = probe_sum(acc, t, red);
  if (t == 0 && p >= 0) g.pr_out[(long long)p * g.max_steps + step] = acc;
}

// One tile of a two-step pass by the code its CPML needs: tiles whose region
// (halo and pipeline planes included) is clear of some slabs leave their code
// out.  FP64 tiles in the CPML would spill in March's registers; they take
// the one-plane-at-a-time tile.
template <typename T, int TY>
union TileSmem {
  MarchSmem<T, TY> m;
  TB2Smem<T, TY> t;
};
template <int TY>
union TileSmem<float, TY> {
  MarchSmem<float, TY> m;
};
template <typename T, typename CI, bool PML, int TY>
__device__ __forceinline__ void tb2_any(const GridView<T>& g, ColdView<T> cold, TileSmem<T, TY>& sm, int i0, int j0,
                                        int iw, int jh, int k0, int k1, int step) {
  if constexpr (!PML) {
    March<T, CI, TY, 0>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
  } else {
    const int n = g.npml;
    const bool cx = i0 - 2 >= n && i0 + 62 <= g.nx - n, cy = j0 - 2 >= n && j0 + TY + 2 <= g.ny - n,
               cz = k0 - 2 >= n && k1 < g.nz - n;
    if (cx && cy && cz) {
      March<T, CI, TY, 0>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
    } else if constexpr (sizeof(T) == 8) {
      tb2_tile<T, CI, TY>(g, sm.t, i0, j0, iw, jh, k0, k1, step);
    } else {
      if (cx && cy) March<T, CI, TY, 4>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
      else if (cy) March<T, CI, TY, 5>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
      else if (cx) March<T, CI, TY, 6>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
      else March<T, CI, TY, 7>(g, cold, sm.m, i0, j0, iw, jh, k0, k1, step);
    }
  }
}

// Registers a lane may use: FP32 tiles with CPML code take what one block per
// CU leaves them, tiles without it stay below 80 so that two 12-wave blocks
// share a CU.
constexpr int tb2_waves(int size, bool pml, int ty) { return size == 8 ? 1 : pml || ty == 12 ? (ty + 4) / 4 : 6; }

// A whole two-step pass in one launch: blocks 0 .. npb - 1 each record a few
// probes (sample `step` recomputed from the input set and, with `prev`, the
// previous pass's second sample, step - 1, which is the input set itself),
// the others march one 60 x TY tile over kz planes.  The probes of a pass's
// last step are left to the next pass or to k_probes after the last one.
// `run`: tiles that an XCD takes in a row (xcd_runs).
template <typename T, typename CI, bool PML, int TY>
__global__ __launch_bounds__(64 * (TY + 4), tb2_waves(sizeof(T), PML, TY)) void k_tb2(GridView<T> g, int step, int kz,
                                                                                   int ntx, int nty, int npb,
                                                                                   int prev, int run) {
  step = gstep(g, step);
  __shared__ TileSmem<T, TY> sm;
  constexpr int GRP = 64 * (TY + 4) / PR_NT;  // probes per block
  __shared__ double red[12 * GRP];
  if ((int)blockIdx.x < npb) {  // uniform per block
    const int grp = (int)threadIdx.x / PR_NT, t = (int)threadIdx.x % PR_NT, q = (int)blockIdx.x * GRP + grp;
    const int p = q < g.n_probe ? q : -1;
    probe_tb2<T, CI, PML, false>(g, p, step, t, red + 12 * grp);
    if (prev) probe_one(g, p, step - 1, t, red + 12 * grp + 8);
    return;
  }
  const int tile = xcd_runs((int)blockIdx.x - npb, (int)gridDim.x - npb, run);
  const int tile_x = tile % ntx, rest = tile / ntx, k0 = (rest / nty) * kz;
  // the view is the kernel's first argument: read again where it is needed
  const ColdView<T> cold{(typename ColdView<T>::P)__builtin_amdgcn_kernarg_segment_ptr()};
  tb2_any<T, CI, PML, TY>(g, cold, sm, tile_x * 60, (rest % nty) * TY, 60, TY, k0, min(k0 + kz, g.nz), step);
}

// Batched two-step pass: as k_tb2 over a tile list that spans every grid
// (grid, i0 | iw << 16, j0 | jh << 16, k0 | kz << 16) and a list of (grid,
// probe) pairs; step index *d_step + offset.  Nearly every tile of a small
// grid is in the CPML and marches at 1.7 us a plane, instruction bound.  256
// grids of 32 to 96 cells a side with an 8-cell CPML: 1179 us a step (1473
// with one work-queue launch per CPML group and a probe launch); 64 of them
// 296, 8 of them 47 (80).
template <typename T, typename CI>
__global__ __launch_bounds__(768, tb2_waves(sizeof(T), true, 8)) void k_tb2_batch(
    const GridView<T>* __restrict__ views, const int4* __restrict__ tiles, const int2* __restrict__ plist, int n_probes,
    int npb, const int* __restrict__ d_step, int offset, int prev, int run) {
  const int step = *d_step + offset;
  __shared__ TileSmem<T, 8> sm;
  constexpr int GRP = 768 / PR_NT;
  __shared__ double red[12 * GRP];
  if ((int)blockIdx.x < npb) {  // uniform per block
    const int grp = (int)threadIdx.x / PR_NT, t = (int)threadIdx.x % PR_NT, q = (int)blockIdx.x * GRP + grp;
    const int2 e = plist[min(q, n_probes - 1)];
    const int p = q < n_probes ? e.y : -1;
    probe_tb2<T, CI, true, false>(views[e.x], p, step, t, red + 12 * grp);
    if (prev) probe_one(views[e.x], p, step - 1, t, red + 12 * grp + 8);
    return;
  }
  const int4 t = tiles[xcd_runs((int)blockIdx.x - npb, (int)gridDim.x - npb, run)];
  const int tx = __builtin_amdgcn_readfirstlane(t.x), ty = __builtin_amdgcn_readfirstlane(t.y),
            tz = __builtin_amdgcn_readfirstlane(t.z), tw = __builtin_amdgcn_readfirstlane(t.w);
  const GridView<T> g = uniform_view(views + tx);
  const ColdView<T> cold{(typename ColdView<T>::P)(uintptr_t)(views + tx)};
  const int k0 = tw & 0xffff;
  tb2_any<T, CI, true, 8>(g, cold, sm, ty & 0xffff, tz & 0xffff, ty >> 16, tz >> 16, k0, k0 + (tw >> 16), step);
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
// y slabs, 3 both (x-y corners).  Fused tiles are 32 wide in groups 1 and 3
// and 64 wide otherwise; two-step tiles are 60 wide.  FP64 (a diagnostic
// precision) keeps the all-axes instantiation for every group.
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

template <typename T, typename CI, bool PML, int TY>
hipError_t launch_tb2(const GridView<T>& g, int step, int kz, int run, int prev, hipStream_t st) {
  constexpr int GRP = 64 * (TY + 4) / PR_NT;
  const int ntx = (g.nx + 59) / 60, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + kz - 1) / kz;
  const int npb = (g.n_probe + GRP - 1) / GRP;
  const long long nb = (long long)ntx * nty * ntz + npb;
  if (nb > 0x7fffffff || (sizeof(CI) == 1 && g.ncls > 256)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_tb2<T, CI, PML, TY>), dim3((unsigned)nb), dim3(64 * (TY + 4)), 0, st, g, step, kz, ntx, nty,
                     npb, prev, run);
  return hipGetLastError();
}

template <typename T, typename CI>
hipError_t step_tb2(const GridView<T>& g, int step, int ty, int kz, int run, int prev, hipStream_t st) {
  const bool pml = g.npml > 0;
  if (ty == 4)
    return pml ? launch_tb2<T, CI, true, 4>(g, step, kz, run, prev, st)
               : launch_tb2<T, CI, false, 4>(g, step, kz, run, prev, st);
  if (ty == 12)
    return pml ? launch_tb2<T, CI, true, 12>(g, step, kz, run, prev, st)
               : launch_tb2<T, CI, false, 12>(g, step, kz, run, prev, st);
  return pml ? launch_tb2<T, CI, true, 8>(g, step, kz, run, prev, st)
             : launch_tb2<T, CI, false, 8>(g, step, kz, run, prev, st);
}

int launch_tb2_pass(int prec, const void* view, int cls16, int step, int ty, int kz, int run, int prev,
                    void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (prec == 64) {
    const GridView<double>& g = *(const GridView<double>*)view;
    return (int)(cls16 ? step_tb2<double, uint16_t>(g, step, ty, kz, run, prev, st)
                       : step_tb2<double, uint8_t>(g, step, ty, kz, run, prev, st));
  }
  const GridView<float>& g = *(const GridView<float>*)view;
  return (int)(cls16 ? step_tb2<float, uint16_t>(g, step, ty, kz, run, prev, st)
                     : step_tb2<float, uint8_t>(g, step, ty, kz, run, prev, st));
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

template <typename T, typename CI>
hipError_t batch_pass_t(const void* views, const void* tiles, int n_tiles, const void* plist, int n_probes,
                        const int* d_step, int offset, int prev, int run, hipStream_t st) {
  const int npb = (n_probes + 768 / PR_NT - 1) / (768 / PR_NT);
  hipLaunchKernelGGL((k_tb2_batch<T, CI>), dim3((unsigned)(npb + n_tiles)), dim3(768), 0, st,
                     (const GridView<T>*)views, (const int4*)tiles, (const int2*)plist, n_probes, npb, d_step, offset,
                     prev, run);
  return hipGetLastError();
}

int launch_batch_pass(int prec, int cls16, const void* views, const void* tiles, int n_tiles, const void* plist,
                      int n_probes, const int* d_step, int offset, int prev, int run, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  if (prec == 64)
    e = cls16 ? batch_pass_t<double, uint16_t>(views, tiles, n_tiles, plist, n_probes, d_step, offset, prev, run, st)
              : batch_pass_t<double, uint8_t>(views, tiles, n_tiles, plist, n_probes, d_step, offset, prev, run, st);
  else
    e = cls16 ? batch_pass_t<float, uint16_t>(views, tiles, n_tiles, plist, n_probes, d_step, offset, prev, run, st)
              : batch_pass_t<float, uint8_t>(views, tiles, n_tiles, plist, n_probes, d_step, offset, prev, run, st);
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
