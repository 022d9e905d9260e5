// fdtd_march.h -- the two-step tile and its probes (device code of the
// two-step passes).
#pragma once
#include <hip/hip_runtime.h>

#include "fdtd_dev.h"
#include "fdtd_tile.h"
#include "yee_update.h"

namespace mi355fdtd {

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
// One block of a tile in the CPML or of 12 rows runs on a CU at a time (up to 16
// waves of at most 128 registers; FP32 tiles of 8 rows without CPML code stay
// below 80, and two of 12 waves share a CU; 48 KB of LDS for 8 rows, 58 for 12,
// 124 and 155 in FP64; 72 and 134 with tables of 768 and 2,048 classes), and
// with everything in the caches a plane costs what its instructions cost, so
// the loop is built to issue few: uniform bases with
// one 32-bit offset per plane; points and planes outside the grid are not
// branched around (their coefficients are the table's zero row); registers
// rotate by name over three unrolled iterations, not by copies; what is
// needed rarely is read again where it is needed (ColdView).  A lane outside a
// stage's region computes a value that no lane inside reads.
//
// Measured (us per step, against one launch per CPML group of 8-row tiles
// with three barriers, four LDS planes and 2.5 times the instructions):
// 512 x 512 x 384 with a 10-cell CPML 743 (891), 203 x 157 x 131 46 (116),
// 96 x 96 x 80 14.5 (82), 48^3 without one 4.3 (38, the fused pass).  In the
// caches a plane of an 8-row tile takes 0.92 us clear of the CPML and 1.7 us
// in it; on the largest grid 12 rows take 2 us, bound by the 5 TB/s that
// the tiles draw through the L2s (a copy reaches 5.1).
// ---------------------------------------------------------------------------

template <typename T, int TY>
struct MarchRows {
  static constexpr int R = TY + 4;
  static constexpr int PZ = 512 / sizeof(T);  // longest z profile row held here (2 npml)
  T e0[2][R][64];       // E^n (x, z), plane k
  T h1[2][R][64];       // H^{n+1/2} (x, z), plane k
  T e1[2][2][R][64];    // E^{n+1} (x, z), planes k and k-1
  T h2[2][R][64];       // H^{n+3/2} (x, z), plane k-2
  T px[P_NROW][64];     // CPML profile at each lane's x
  T pz[P_NROW * PZ];    // the z table
};
// NC: classes whose coefficients fit the LDS table (0: none, they are read from
// memory at each use).  A table of up to 256 comes first, where offsets into it
// need no base (100 x 100 x 80 with four poles 25.0 us a step, 25.8 with the
// table behind the rows); a larger one comes last, as it would push the rows out
// of an offset's 64 KB (12 rows, 1,300 classes on 203 x 157 x 131 68 us a step,
// 104 with the table first).
template <typename T, int NC>
struct MarchTab {
  T stab[(NC + 1) * K_STRIDE];  // a row of zeros, then the classes' coefficients
};
template <typename T, int TY, int NC = 256, bool FIRST = (NC <= 256)>
struct MarchSmem : MarchTab<T, NC>, MarchRows<T, TY> {};
template <typename T, int TY, int NC>
struct MarchSmem<T, TY, NC, false> : MarchRows<T, TY>, MarchTab<T, NC> {};

// CPML profile values of a tile's points: a lane's x values in registers
// (tiles of up to 8 rows, which have them to spare) or LDS, the row's y
// values in scalar registers, z from LDS.
template <typename T, int TY>
struct ProfMarch {
  static constexpr bool XREG = TY <= 8;
  const MarchRows<T, TY>& sm;
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

// Debye media in a two-step pass: the pole currents' input set (array q =
// component * npole + pole at jin + q pitch), the output set's distance, and
// the factors.
template <typename T>
struct MarchDebye {
  const T* jin;
  ptrdiff_t jout;
  size_t pitch;
  const T* dtab;
  const unsigned char* dflag;
  T kp[D_MAXPOLE];
  int npole;
};
// MarchDebye in the kernel's arguments, read again at each use (ColdView).
template <typename T>
struct DebyeArgs {
  typedef const __attribute__((address_space(4))) MarchDebye<T>* P;
  P p;
  __device__ __forceinline__ P get() const {
    P q = p;
    asm volatile("" : "+s"(q));
    return q;
  }
};
template <typename T, int TY, int NP>
struct MarchDebyeSmem {
  T j[2][3 * NP][TY + 4][64];   // J^{n+1}, two planes
  T dt[256 * D_STRIDE];
  unsigned char fl[256];
};
template <typename T, int TY>
struct MarchDebyeSmem<T, TY, 0> {};

// The state of one thread's point, registers named by plane modulo 3.
template <typename T>
struct MarchRegs {
  unsigned dc[3];   // LDS row (in values) of the class's pole factors, NONE: no pole term
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
//
// NP > 0: Debye media of up to NP poles.  The pole currents are node-local:
// B advances J^n to J^{n+1} and D to J^{n+2}, which goes to the output set of
// the currents (neighbouring tiles still read the input set).  J^n of a plane
// is loaded an iteration before its B; J^{n+1} waits the two iterations from
// B to D in LDS, in slots that only its own thread touches.  Nodes without a
// pole term skip all of it.
template <typename T, typename CI, int TY, int AX, int NP = 0, int NC = sizeof(CI) == 1 ? 256 : 0>
struct March {
  static constexpr int TX = 60, NT = 64 * (TY + 4);
  static constexpr bool LDS_TAB = NC > 0;
  static constexpr bool PML = AX != 0, SX = AX & 1, SY = AX & 2, SZ = AX & 4;
  static constexpr unsigned S = sizeof(T), NONE = 0xFFFFFFFFu;

  typedef typename MarchRegs<T>::Pair Pair;
  MarchSmem<T, TY, NC>& sm;
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
  MarchDebyeSmem<T, TY, NP>* ds;
  DebyeArgs<T> db;
  T jn[NP > 0 ? 3 * NP : 1];       // J^n of the plane that B takes next

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
    if (k >= srcr.klo && k <= srcr.khi) {  // uniform
      const unsigned n = dom ? n0 + sxy * (unsigned)k : NONE;
      if (srcr.hi - srcr.lo <= 4) {
        e_sources(g, srcr.lo, srcr.hi, n, st, en);
      } else {
        // many sources (wires feed every edge they touch): 64 keys at a time,
        // only those of this plane taken one by one, in their order.  (A
        // tower of 15 wires, 424 segments, on 512 x 512 x 384: 798 us a step,
        // 1,575 with every source of the columns looked at in every plane.)
        for (int s0 = srcr.lo; s0 < srcr.hi; s0 += 64) {
          const int s = s0 + u;
          const bool here = s < srcr.hi && (unsigned)ldg(g->src_idx, (unsigned)s) - sxy * (unsigned)k < sxy;
          for (unsigned long long m = __ballot(here); m; m &= m - 1) {
            const int q = s0 + __builtin_ctzll(m);
            e_sources(g, q, q + 1, n, st, en);
          }
        }
      }
    }
  }

  // Pole factors and J^n of plane k (class id c) for the next B.  The arrays'
  // addresses are formed one after another (the asm statement keeps the
  // compiler from holding them all); poles beyond npole count as 0.
  __device__ __forceinline__ void load_j(int k, unsigned c, unsigned& dc) {
    dc = NONE;
    if (k < 0 || k >= nz || v < 1 || v > TY + 2) return;  // uniform
    if (dom && ds->fl[c]) {
      dc = c * D_STRIDE;
      const unsigned o = n0s + (unsigned)k * sxy * S;
      const auto d = db.get();
      const T* j = d->jin;
      const int npole = d->npole;
      const size_t pitch = d->pitch;
#pragma unroll
      for (int q = 0; q < 3 * NP; ++q) {
        jn[q] = T(0);
        if (q % NP < npole) {  // uniform
          asm volatile("" : "+s"(j));
          jn[q] = ldb(j, o);
          j += pitch;
        }
      }
    }
  }
  // E of plane k less the pole currents, and those one step later: from jn to
  // LDS (B) or from LDS to the output set (D), a component at a time to need
  // few registers.
  template <bool D>
  __device__ __forceinline__ void debye(int k, unsigned dc, const T eold[3], T e[3]) const {
    const T* f = ds->dt + dc;
    T* const jl = &ds->j[k & 1][0][v][u];
    const auto d = db.get();
    const T* out = d->jin + d->jout;
    const int npole = d->npole;
    const size_t pitch = d->pitch;
    const unsigned o = n0s + (unsigned)k * sxy * S;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T jo[NP], sum = T(0);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        jo[p] = D ? jl[(a * NP + p) * NT] : jn[a * NP + p];
        sum += f[a * 2 * D_MAXPOLE + 2 * p + 1] * jo[p];
      }
      e[a] -= sum;
      const T de = e[a] - eold[a];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const T j1 = d->kp[p] * jo[p] + f[a * 2 * D_MAXPOLE + 2 * p] * de;
        if (!D) {
          jl[(a * NP + p) * NT] = j1;
        } else if (p < npole) {  // uniform
          asm volatile("" : "+s"(out));
          if (inD) stb((T*)out, o, j1);
          out += pitch;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
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
    {
      stage_e(k - 2, lz[P2], r.co[P2], r.h2[P2], r.h2[Q], sm.h2, r.e1[P2], step + 1, r.pe[P2], r.e2);
      if constexpr (NP > 0) {
        if (r.dc[P2] != NONE) debye<true>(k - 2, r.dc[P2], r.e1[P2], r.e2);
      }
    }
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
      if constexpr (NP > 0) {
        if (r.dc[Q] != NONE) debye<false>(k, r.dc[Q], r.e0[Q], r.e1[Q]);
      }
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
    if constexpr (NP > 0) load_j(k + 1, craw, r.dc[N1]);
    __syncthreads();
  }

  __device__ __forceinline__ March(const GridView<T>& gv, ColdView<T> cold, MarchSmem<T, TY, NC>& sm_, int i0, int j0,
                                   int iw, int jh, int k0_, int k1_, int step_,
                                   MarchDebyeSmem<T, TY, NP>* ds_ = nullptr, DebyeArgs<T> db_ = {})
      : sm(sm_), g(cold), nz(gv.nz), np(gv.npml), step(step_), k0(k0_), k1(k1_),
        pf{sm_, 0, 0, {}, {}}, ds(ds_), db(db_) {
    const int tid = threadIdx.x, nx = gv.nx, ny = gv.ny;
    u = tid & 63;
    v = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (LDS_TAB) {
      if (tid < K_STRIDE) sm.stab[tid] = T(0);
      for (int q = tid; q < gv.ncls * K_STRIDE; q += NT) sm.stab[K_STRIDE + q] = ldg(gv.ctab, (unsigned)q);
    }
    if constexpr (NP > 0) {
      for (int q = tid; q < gv.ncls * D_STRIDE; q += NT) ds->dt[q] = ldg(db.p->dtab, (unsigned)q);
      for (int q = tid; q < gv.ncls; q += NT) ds->fl[q] = ldg(db.p->dflag, (unsigned)q);
      r.dc[0] = r.dc[1] = r.dc[2] = NONE;
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
// the same per-point arithmetic; the second step's are read from its output
// set by the next pass.
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
__device__ __forceinline__ void e1_at(const GridView<T>& g, int x, int y, int k, int step, T e[3],
                                      const MarchDebye<T>* db = nullptr) {
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
  const unsigned c = (unsigned)ldg((const CI*)g.cls, n);
  if (!db || !ldg(db->dflag, c)) return;
  for (int a = 0; a < 3; ++a) {
    T sum = T(0);
    for (int p = 0; p < db->npole; ++p)
      sum += ldg(db->dtab, c * D_STRIDE + (unsigned)(a * 2 * D_MAXPOLE + 2 * p + 1)) *
             ldg(db->jin + (size_t)(a * db->npole + p) * db->pitch, n);
    e[a] -= sum;
  }
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

// Probe p of a two-step pass (p = -1: none): sample `step`, recomputed from
// the input set, which the pass leaves untouched.  Thread t of the group.
template <typename T, typename CI, bool PML>
__device__ __forceinline__ void probe_tb2(const GridView<T>& g, int p, int step, int t, double* red,
                                          const MarchDebye<T>* db = nullptr) {
  double acc = 0.0;
  const int q0 = p < 0 ? 0 : g.pr_off[p], q1 = p < 0 ? 0 : g.pr_off[p + 1];
  for (int q = q0 + t; q < q1; q += PR_NT) {
    const int c = g.term_comp[q];
    const unsigned n = (unsigned)g.term_idx[q];
    const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny), k = (int)(n / g.sxy);
    T v3[3];
    if (c < 3) e1_at<T, CI, PML>(g, x, y, k, step, v3, db);
    else h1_at<T, CI, PML>(g, x, y, k, v3);
    const int cc = c < 3 ? c : c - 3;
    acc += g.term_w[q] * (double)(cc == 0 ? v3[0] : cc == 1 ? v3[1] : v3[2]);
  }
  acc = probe_sum(acc, t, red);
  if (t == 0 && p >= 0) g.pr_out[(long long)p * g.max_steps + step] = acc;
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

// Both samples of a pass with more than PR_MANY probes, in a launch of its own
// before the pass.  (The pass's own blocks hold the LDS of a tile, one to a CU,
// and three probes each: a launch less, and the faster way while they are a few
// rounds.  us a step, 1,000 and 2,000 values in the pass / 2,060 apart: 48^3
// 5.8, 8.5 / 8.4, 160^3 26.2, 29.9 / 27.2, 96 x 96 x 80 with a CPML 22.0, 27.9 /
// 19.5, 100 x 100 x 80 with four poles 35.4, 41.0 / 43.5.)  Most probes of so
// many are single values: the first `nlane` blocks take those, a lane each, 1
// << lw of them a wave; the others take the rest, a wave each, summed in
// probe_sum's order (the 0.0 of threads without a term changes no bit).  Bound
// by the loads' latency, about eight dependent rounds of them a value.  96 x 96
// x 80, us a step (a block of 256 a probe): 4,000 values 20.1 (25.6), 20,000
// 23.1 (62.0), 100,000 47.9 (243); 20,000 loops of four terms 22.8 (39.4),
// 20,000 lines of 93 53.7 (74.0).
template <typename T, typename CI, bool PML, bool DB>
__global__ __launch_bounds__(PR_NT) void k_probes_tb2(GridView<T> g, MarchDebye<T> db, int step, int prev, int nlane,
                                                      int lw) {
  step = gstep(g, step);
  const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // term q, added to both samples' sums
  auto term = [&](int q, double acc[2]) {
    const int c = g.term_comp[q], cc = c < 3 ? c : c - 3;
    const unsigned n = (unsigned)g.term_idx[q];
    const double w = g.term_w[q];
    if (prev) {
      const T* f = c == 0 ? g.fi[0] : c == 1 ? g.fi[1] : c == 2 ? g.fi[2] : c == 3 ? g.fi[3] : c == 4 ? g.fi[4] : g.fi[5];
      acc[1] += w * (double)ldg(f, n);
    }
    const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny), k = (int)(n / g.sxy);
    T v3[3];
    if (c < 3) e1_at<T, CI, PML>(g, x, y, k, step, v3, DB ? &db : nullptr);
    else h1_at<T, CI, PML>(g, x, y, k, v3);
    acc[0] += w * (double)(cc == 0 ? v3[0] : cc == 1 ? v3[1] : v3[2]);
  };
  auto record = [&](int p, const double sum[2]) {
    double* out = g.pr_out + (long long)p * g.max_steps + step;
    out[0] = sum[0];
    if (prev) out[-1] = sum[1];
  };
  double sum[2] = {0.0, 0.0};
  if ((int)blockIdx.x < nlane) {
    const int p = ((int)(blockIdx.x * (PR_NT / 64) + wave) << lw) + lane;
    if (lane >> lw || p >= g.n_probe) return;
    const int q0 = g.pr_off[p];
    if (g.pr_off[p + 1] - q0 != 1) return;
    term(q0, sum);
    record(p, sum);
    return;
  }
  const int p = ((int)blockIdx.x - nlane) * (PR_NT / 64) + wave;
  if (p >= g.n_probe) return;
  const int q0 = g.pr_off[p], q1 = g.pr_off[p + 1];
  if (q1 - q0 == 1) return;
  for (int q = q0; q < q1 && q < q0 + PR_NT; q += 64) {
    double acc[2] = {0.0, 0.0};
    for (int r = q + lane; r < q1; r += PR_NT) term(r, acc);
    for (int u = 0; u < 2; ++u) {
      for (int o = 32; o > 0; o >>= 1) acc[u] += __shfl_down(acc[u], o, 64);
      sum[u] += acc[u];
    }
  }
  if (lane == 0) record(p, sum);
}

// Its launch: up to 4,096 waves of single values.
template <typename T, typename CI, bool PML, bool DB>
void probes_tb2(const GridView<T>& g, const MarchDebye<T>& db, int step, int prev, hipStream_t st) {
  constexpr int W = PR_NT / 64;
  int lw = 0;
  while (lw < 6 && g.n_probe >> lw > 4096) ++lw;
  const int nlane = (g.n_probe + (W << lw) - 1) / (W << lw), nwave = (g.n_probe + W - 1) / W;
  hipLaunchKernelGGL((k_probes_tb2<T, CI, PML, DB>), dim3((unsigned)(nlane + nwave)), dim3(PR_NT), 0, st, g, db, step,
                     prev, nlane, lw);
}

}  // namespace mi355fdtd
