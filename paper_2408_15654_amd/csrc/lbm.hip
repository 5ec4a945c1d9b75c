// HIP kernels and C ABI of the coupled three-field lattice Boltzmann library
// (phase field f, surfactant g, flow h; arXiv:2408.15654), for gfx950.
//
// State on the device (one caller-owned workspace per simulation).  Two
// copies (ping-pong) of:
//   populations  row-interleaved: lattice row y holds the FG block (for
//                i = 0..8, nx pairs (f_i, g_i), so the two populations that
//                stream from the same source site arrive in one access) and
//                then the H block (h_1..h_8, nx each; h_0 is never read:
//                column 0 of M is e_0 and rows 1-8 of M^-1 start with 0).
//                f_i and g_i are stored as deviations f_i - w_i phi and
//                g_i - w_i psi from the rest values of the writing site;
//   rest         one record per site, (phi, psi) of the same time level:
//                the bases of those deviations;
// plus, updated in place (each site reads and writes only its own entry):
//   aux          one record per site, (ux, uy) of the previous time level
//                (the first-order time differences need it; the previous
//                level's mass flux S is recomputed from the previous phi
//                of the rest records); with a prescribed velocity, u itself;
//   scratch      float64 planes (plane-major) for host transfers and
//                read-back.
// Storage: float64, float32, or float16 deviations with per-field
// power-of-two scales; with float16 storage h is also stored as deviations,
// from 3 w_k (P + c_k . rho u) of the writing site, the rest record carries
// (phi, psi, P, rho ux, rho uy) in float32, and the previous velocity is
// rho u / rho(phi) of that record (aux holds only a prescribed velocity).
//
// A time step is one launch of lbm_step_kernel, except where
// lbm_block_kernel (grids too small to fill the device) or lbm_pair_kernel
// (large float64 and float32 grids) take several steps in one launch with
// the same results.  In lbm_step_kernel each wavefront owns a
// strip of columns, 60 with one column per lane or 124 with two (float32
// and float16 storage, even nx), plus two halo columns on each side, and
// walks down a tile of rows.  For each row it pulls the f and g deviations
// of the NEXT row, rebuilds that row's phi, psi (and sigma(psi)) from them
// and the rest values of their source sites, keeps a three-row window of
// phi, psi, sigma in registers and takes x-neighbours from adjacent lanes
// with cross-lane moves, so the 9-point stencils need no LDS and no
// barrier.  The h populations and the previous level are read for the
// current row only, and every population is written once.  Workgroups walk
// the tiles in one contiguous band per XCD.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "lbm.h"
#include "lbm_device.h"
#include "arena.h"
#include "tiling.h"

using namespace lbm;

namespace {

constexpr int kWave = 64;
constexpr int kPlanes = 26;
constexpr int kScratch = 8;
constexpr int kReduceBlocks = 1024;
constexpr int kReduceVals = 8;
constexpr int kMomentVals = 7;               // lbm_reduce_kernel's values,
constexpr unsigned kMomentMaxes = 1u << 5 | 1u << 6;  // of which 5 and 6 are maxima

// Minimum waves per SIMD the compiler schedules the step kernel for.  The
// value steers the instruction scheduler as much as the register budget:
// measured on the 2048x2048 many-drop field, 1 (no constraint) is best for
// float64 and float32 storage, 2 for float16 storage (3 spills), and 4
// spills for all.
#ifndef LBM_WAVES_F64
#define LBM_WAVES_F64 1
#endif
#ifndef LBM_WAVES_F32
#define LBM_WAVES_F32 1
#endif
#ifndef LBM_WAVES_F16
#define LBM_WAVES_F16 2
#endif

// Cache policies of the step kernel's stores (the precision structs pick
// one): non-temporal (what a step writes is read again only by the next
// step, long after it has left the caches) or the default.  Measured on the
// 2048x2048 field: non-temporal is 3% faster for float32 storage and 6% for
// float64, the default 4% faster for float16 storage.  A single simulation
// whose step traffic fits the 256 MB Infinity Cache takes default stores in
// every precision (F64C, F32C; cache_resident).
constexpr int kStoreNT = 2;
constexpr int kStoreDefault = 0;

// Storage precisions: S population type, A type of phi/psi/u/S planes,
// R arithmetic type, SCALED: populations carry power-of-two scales.
struct F64 {
  using S = double;
  using A = double;
  using R = double;
  static constexpr bool SCALED = false;
  static constexpr int kMinWaves = LBM_WAVES_F64;  // step kernel waves per SIMD
  static constexpr int kBlockWaves = 4;  // step kernel wavefronts per workgroup
  static constexpr int kStorePol = kStoreNT;  // step kernel store cache policy
  static constexpr bool HDEV = false;  // h stored raw
  static constexpr int kRest = 2;      // rest record: phi, psi
  static constexpr int kAux = 2;       // aux record: ux, uy
};
struct F32 {
  using S = float;
  using A = float;
  using R = float;
  static constexpr bool SCALED = false;
  static constexpr int kMinWaves = LBM_WAVES_F32;  // step kernel waves per SIMD
  static constexpr int kBlockWaves = 4;  // step kernel wavefronts per workgroup
  static constexpr int kStorePol = kStoreNT;  // step kernel store cache policy
  static constexpr bool HDEV = false;
  static constexpr int kRest = 2;
  static constexpr int kAux = 2;
};
struct F16 {
  using S = _Float16;
  using A = float;
  using R = float;
  static constexpr bool SCALED = true;
  static constexpr int kMinWaves = LBM_WAVES_F16;  // step kernel waves per SIMD
  // one wavefront per workgroup: 3% faster than four on the 2048x2048 field
  // (float32 and float64 storage: equal, or slower with one)
  static constexpr int kBlockWaves = 1;
  static constexpr int kStorePol = kStoreDefault;  // step kernel store cache policy
  // h_k stored as deviations from 3 w_k (P + c_k . rho u) of the storing
  // site; P and rho u join phi, psi in the rest record, and the previous
  // velocity is rho u / rho(phi) of that record, so the Navier-Stokes step
  // reads no aux record (it holds only a prescribed velocity).
  static constexpr bool HDEV = true;
  static constexpr int kRest = 5;  // rest record: phi, psi, P, rho ux, rho uy
  static constexpr int kAux = 2;   // aux record: ux, uy (prescribed flow only)
};
// The same storage with default stores: what one step writes is then read
// by the next one from the Infinity Cache while the simulation fits it.
struct F64C : F64 {
  static constexpr int kStorePol = kStoreDefault;
};
struct F32C : F32 {
  static constexpr int kStorePol = kStoreDefault;
};

template <class P>
struct Scales {
  typename P::R f, g, h;     // multiply before storing
  typename P::R fi, gi, hi;  // multiply after loading
};

// Buffer-resource memory access for the step kernel: the address is a
// wave-uniform resource (SGPRs) plus a uniform byte offset (SGPR) plus one
// per-lane 32-bit byte offset (VGPR), so no per-lane 64-bit address math.
// The third dword 0x00020000 is the raw 32-bit-element format of gfx9-family
// buffer descriptors.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
using rsrc_t = __amdgpu_buffer_rsrc_t;

// Guards around a buffer store of more than 64 bits.  Such a store reads
// its data registers over several cycles after it issues; measured on
// gfx950, registers rewritten by the very next instructions (the compiler
// leaves no gap when the store's offset is an SGPR) reached memory with
// the new values in the last lanes of each 16-lane group.  The store is
// pinned between two scheduling barriers and followed by two wait states.
__device__ __forceinline__ void wide_store_begin() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ void wide_store_guard() {
  __asm__ volatile("s_nop 1" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Byte offset of a lane whose buffer stores must not land.  The hardware
// discards a buffer store whose offset is past the resource's range: it
// checks soffset + voffset (+ 4 per further dword) against the resource's
// byte count, without 32-bit wraparound (measured on MI355X for offsets up
// to 0xFFFFFFF0 with soffset 0 to 2^31), and no memory request is made.
// Every resource of the step covers at most kDropped bytes (lbm_create
// checks it), so kDropped, and kDropped plus the few bytes added within a
// record (at most 32, below 2^32 still), is past all of them.
constexpr unsigned kDropped = 0xFFFFFF00u;

__device__ __forceinline__ rsrc_t make_rsrc(const void *base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, int(bytes),
                                           0x00020000);
}

template <class T>
struct BufIO;
template <>
struct BufIO<float> {
  static __device__ __forceinline__ float load(rsrc_t r, unsigned v, unsigned s) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
  }
  template <int POL>
  static __device__ __forceinline__ void store(float x, rsrc_t r, unsigned v, unsigned s) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, v, s, POL);
  }
};
template <>
struct BufIO<double> {
  static __device__ __forceinline__ double load(rsrc_t r, unsigned v, unsigned s) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0);
    const unsigned w0 = w[0], w1 = w[1];
    return __hiloint2double(int(w1), int(w0));
  }
  template <int POL>
  static __device__ __forceinline__ void store(double x, rsrc_t r, unsigned v, unsigned s) {
    u32x2 w;
    w[0] = unsigned(__double2loint(x));
    w[1] = unsigned(__double2hiint(x));
    __builtin_amdgcn_raw_buffer_store_b64(w, r, v, s, POL);
  }
};
template <>
struct BufIO<_Float16> {
  static __device__ __forceinline__ _Float16 load(rsrc_t r, unsigned v, unsigned s) {
    return __builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(r, v, s, 0));
  }
};

// Population load through a buffer resource, with the float16 scale where
// the storage is scaled; store of an unscaled (float32/float64) one.
template <class P>
__device__ __forceinline__ typename P::R bld(rsrc_t r, unsigned v, unsigned s,
                                             typename P::R inv) {
#pragma clang fp contract(off)
  using R = typename P::R;
  if constexpr (P::SCALED)
    return R(BufIO<typename P::S>::load(r, v, s)) * inv;
  else
    return R(BufIO<typename P::S>::load(r, v, s));
}
template <class P>
__device__ __forceinline__ void bst(typename P::R x, rsrc_t r, unsigned v, unsigned s) {
  static_assert(!P::SCALED, "float16 populations are stored packed (halves_sr)");
  BufIO<typename P::S>::template store<P::kStorePol>(typename P::S(x), r, v, s);
}

template <class P>
__device__ __forceinline__ typename P::R ld(const typename P::S *p, long long i,
                                            typename P::R inv) {
  using R = typename P::R;
  if constexpr (P::SCALED)
    return R(p[i]) * inv;
  else
    return R(p[i]);
}
template <class P>
__device__ __forceinline__ void st(typename P::S *p, long long i, typename P::R v,
                                   typename P::R scale) {
  using S = typename P::S;
  if constexpr (P::SCALED)
    p[i] = S(v * scale);
  else
    p[i] = S(v);
}

template <class P>
struct StepArgs {
  Phys<typename P::R> p;
  Scales<P> sc;
  const typename P::S *src;
  const typename P::A *src_rest;
  typename P::S *dst;
  typename P::A *dst_rest;
  typename P::A *aux;
  int *flag;
  int nx, ny, walls;
  int nstrips, rows;
  int tail_rows, tail_h;  // single-grid launches: short chunks at each band's end
};

// Row offsets and wall flags for pulling row y.
struct RowIdx {
  long long rc, rm, rp;  // offsets of rows y, y-1, y+1 (valid even at walls)
  bool bot, top;         // row y touches the bottom / top wall
};

__device__ __forceinline__ RowIdx row_index(int y, int nx, int ny, int walls) {
  RowIdx r;
  int ym = y - 1, yp = y + 1;
  r.bot = walls && y == 0;
  r.top = walls && y == ny - 1;
  if (ym < 0) ym = walls ? y : ym + ny;
  if (yp >= ny) yp = walls ? y : yp - ny;
  r.rc = (long long)y * nx;
  r.rm = (long long)ym * nx;
  r.rp = (long long)yp * nx;
  return r;
}

// Row y of the lattice for a row index that may lie one or two rows
// outside: periodic wrap, or clamped between walls (clamped rows are only
// read where the bounce-back makes their value irrelevant).
__device__ __forceinline__ int wrap_row(int y, int ny, int walls) {
  if (walls) return y < 0 ? 0 : (y >= ny ? ny - 1 : y);
  return y < 0 ? y + ny : (y >= ny ? y - ny : y);
}

// ------------------------------------------------------------------
// Memory layout (row-interleaved; x fastest inside each block).  Row y of
// the population group holds, in units of the storage type S:
//   block FG: for i = 0..8, nx pairs (f_i, g_i)      -> 18 nx values
//   block H:  for i = 1..8, nx values h_i             ->  8 nx values
// so f_i and g_i, which stream from the same source site, arrive in one
// load.  The rest group holds (phi, psi) pairs and the aux group (ux, uy)
// pairs, one per site.
__device__ __forceinline__ long long fg_idx(int i, int c, int y, int x, int nx) {
  return (long long)y * (kPlanes * nx) + (long long)(i * nx + x) * 2 + c;
}
__device__ __forceinline__ long long h_idx(int i, int y, int x, int nx) {
  return (long long)y * (kPlanes * nx) + 18LL * nx + (long long)(i - 1) * nx + x;
}
template <class P>
__device__ __forceinline__ long long rest_idx(int c, int y, int x, int nx) {
  return ((long long)y * nx + x) * P::kRest + c;
}
template <class P>
__device__ __forceinline__ long long aux_idx(int c, int y, int x, int nx) {
  return ((long long)y * nx + x) * P::kAux + c;
}

// Rows y-1, y, y+1 to pull from (valid even at walls) and the wall flags of
// row y.
struct RowN {
  int m, c, p;
  bool bot, top;
};

__device__ __forceinline__ RowN row_numbers(int y, int ny, int walls) {
  const RowIdx r = row_index(y, 1, ny, walls);
  RowN n;
  n.m = int(r.rm);
  n.c = int(r.rc);
  n.p = int(r.rp);
  n.bot = r.bot;
  n.top = r.top;
  return n;
}

// Source (row, column, direction) of population i pulled to site (x, row
// r.c): x - c_i, or across a wall the opposite population of the site
// itself (half-way bounce-back).
struct Src {
  int y, x, dir;
};
__device__ __forceinline__ Src pull_source(int i, const RowN &r, int x, int xm, int xp) {
  switch (i) {
    case 0: return {r.c, x, 0};
    case 1: return {r.c, xm, 1};
    case 3: return {r.c, xp, 3};
    case 2: return r.bot ? Src{r.c, x, 4} : Src{r.m, x, 2};
    case 5: return r.bot ? Src{r.c, x, 7} : Src{r.m, xm, 5};
    case 6: return r.bot ? Src{r.c, x, 8} : Src{r.m, xp, 6};
    case 4: return r.top ? Src{r.c, x, 2} : Src{r.p, x, 4};
    case 7: return r.top ? Src{r.c, x, 5} : Src{r.p, xp, 7};
    default: return r.top ? Src{r.c, x, 6} : Src{r.p, xm, 8};
  }
}

// Pull streaming of f and g to site (x, row) (pointer form, for the
// per-site kernels).
template <class P>
__device__ __forceinline__ void pull_fg(const typename P::S *__restrict__ s, const RowN &r,
                                        int x, int xm, int xp, int nx, typename P::R fi,
                                        typename P::R gi, typename P::R *f,
                                        typename P::R *g) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const Src q = pull_source(i, r, x, xm, xp);
    f[i] = ld<P>(s, fg_idx(q.dir, 0, q.y, q.x, nx), fi);
    g[i] = ld<P>(s, fg_idx(q.dir, 1, q.y, q.x, nx), gi);
  }
}

// Pull of h_1..h_8 (h[k] = h_{k+1}); across a wall, bounce-back with Ladd's
// moving-wall term 2 w_i rho_w (c_i.u_w)/c_s^2 = rho_w c_ix u_w / 6 for the
// diagonal populations (rho_w = rho at the site at collision time).
template <class P>
__device__ __forceinline__ void pull_h(const typename P::S *__restrict__ s, const RowN &r,
                                       int x, int xm, int xp, int nx, typename P::R inv,
                                       typename P::R rho_w, typename P::R uwb,
                                       typename P::R uwt, typename P::R *h) {
  using R = typename P::R;
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const Src q = pull_source(i, r, x, xm, xp);
    h[i - 1] = ld<P>(s, h_idx(q.dir, q.y, q.x, nx), inv);
  }
  const R kb = rho_w * uwb * R(1.0 / 6.0), kt = rho_w * uwt * R(1.0 / 6.0);
  if (r.bot) {
    h[4] += kb;
    h[5] -= kb;
  }
  if (r.top) {
    h[6] -= kt;
    h[7] += kt;
  }
}

// Rest values of the nine source sites of a row r relative to the site's
// own value: e_i = X(x - c_i) - X(x); bounced populations come from the
// site itself (e_i = 0).  v holds X at rows r-1 (m), r (c), r+1 (n) of
// columns x-1 (L), x, x+1 (R).
// Rest part of h_k under float16 storage: 3 w_k (P + c_k . j), j = rho u,
// with (sx, sy) = c_k.  The storing site subtracts it for each outgoing k
// and the receiving site adds the same expression of the same stored
// values back, so the two cancel exactly.
template <class R>
__device__ __forceinline__ R hb(R w3, R P, int sx, R jx, int sy, R jy) {
#pragma clang fp contract(off)
  R t = P;
  if (sx > 0) t += jx;
  if (sx < 0) t -= jx;
  if (sy > 0) t += jy;
  if (sy < 0) t -= jy;
  return w3 * t;
}
template <class R>
struct HRest {
  R P, jx, jy;
};
// Rest parts of the post-collision h_1..h_8 stored at one site (b[k] for
// h_{k+1}).
template <class R>
__device__ __forceinline__ void h_store_basis(const HRest<R> &v, R *b) {
#pragma clang fp contract(off)
  const R a = R(1) / R(3), d = R(1) / R(12);  // 3 w_k
  b[0] = hb(a, v.P, 1, v.jx, 0, v.jy);
  b[1] = hb(a, v.P, 0, v.jx, 1, v.jy);
  b[2] = hb(a, v.P, -1, v.jx, 0, v.jy);
  b[3] = hb(a, v.P, 0, v.jx, -1, v.jy);
  b[4] = hb(d, v.P, 1, v.jx, 1, v.jy);
  b[5] = hb(d, v.P, -1, v.jx, 1, v.jy);
  b[6] = hb(d, v.P, -1, v.jx, -1, v.jy);
  b[7] = hb(d, v.P, 1, v.jx, -1, v.jy);
}
// Rest parts of the h_1..h_8 arriving at a site from the 9-point windows
// of the stored (P, jx, jy): each from its source site x - c_k, or at a
// wall row from the site itself, where the arriving h_k left as h_-k.
template <class R>
__device__ __forceinline__ void h_arrival_basis(const Nine<R> &P, const Nine<R> &jx,
                                                const Nine<R> &jy, bool bot, bool top, R *b) {
#pragma clang fp contract(off)
  const R a = R(1) / R(3), d = R(1) / R(12);
  b[0] = hb(a, P.cL, 1, jx.cL, 0, jy.cL);
  b[2] = hb(a, P.cR, -1, jx.cR, 0, jy.cR);
  b[1] = bot ? hb(a, P.c, 0, jx.c, -1, jy.c) : hb(a, P.m, 0, jx.m, 1, jy.m);
  b[4] = bot ? hb(d, P.c, -1, jx.c, -1, jy.c) : hb(d, P.mL, 1, jx.mL, 1, jy.mL);
  b[5] = bot ? hb(d, P.c, 1, jx.c, -1, jy.c) : hb(d, P.mR, -1, jx.mR, 1, jy.mR);
  b[3] = top ? hb(a, P.c, 0, jx.c, 1, jy.c) : hb(a, P.n, 0, jx.n, -1, jy.n);
  b[6] = top ? hb(d, P.c, 1, jx.c, 1, jy.c) : hb(d, P.nR, -1, jx.nR, -1, jy.nR);
  b[7] = top ? hb(d, P.c, -1, jx.c, 1, jy.c) : hb(d, P.nL, 1, jx.nL, -1, jy.nL);
}

// The same where (bot, top) is the same on every lane: wall rows are rare, so
// they are branched to.
template <class R>
__device__ __forceinline__ void source_offsets_row(const Nine<R> &v, bool bot, bool top, R *e) {
  const R c = v.c;
  e[0] = R(0);
  e[1] = v.cL - c;
  e[3] = v.cR - c;
  e[2] = v.m - c;
  e[5] = v.mL - c;
  e[6] = v.mR - c;
  e[4] = v.n - c;
  e[7] = v.nR - c;
  e[8] = v.nL - c;
  if (bot) e[2] = e[5] = e[6] = R(0);
  if (top) e[4] = e[7] = e[8] = R(0);
}
template <class R>
__device__ __forceinline__ void source_offsets(const Nine<R> &v, bool bot, bool top, R *e) {
  const R c = v.c;
  e[0] = R(0);
  e[1] = v.cL - c;
  e[3] = v.cR - c;
  e[2] = bot ? R(0) : v.m - c;
  e[5] = bot ? R(0) : v.mL - c;
  e[6] = bot ? R(0) : v.mR - c;
  e[4] = top ? R(0) : v.n - c;
  e[7] = top ? R(0) : v.nR - c;
  e[8] = top ? R(0) : v.nL - c;
}

// Value of lane-1 / lane+1 of the wavefront: DPP wave shifts (one VALU op
// per 32 bits; lane 0 / lane 63 receive 0, which is never used).
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double from_left(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, int(b), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), 0x138, 0xf, 0xf, true);
  return __longlong_as_double((long long)((unsigned long long)(unsigned)lo |
                                          ((unsigned long long)(unsigned)hi << 32)));
}
__device__ __forceinline__ double from_right(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, int(b), 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), 0x130, 0xf, 0xf, true);
  return __longlong_as_double((long long)((unsigned long long)(unsigned)lo |
                                          ((unsigned long long)(unsigned)hi << 32)));
}

// 3x3 neighbourhood of site k of a lane that holds K adjacent columns,
// from the lane's values in rows y-1 (m), y (c), y+1 (n): neighbours
// across the lane's edge come from the adjacent lanes.
template <int K, int k, class R>
__device__ __forceinline__ Nine<R> window_k(const R *m, const R *c, const R *n) {
  Nine<R> v;
  v.m = m[k];
  v.c = c[k];
  v.n = n[k];
  if constexpr (k > 0) {
    v.mL = m[k - 1];
    v.cL = c[k - 1];
    v.nL = n[k - 1];
  } else {
    v.mL = from_left(m[K - 1]);
    v.cL = from_left(c[K - 1]);
    v.nL = from_left(n[K - 1]);
  }
  if constexpr (k < K - 1) {
    v.mR = m[k + 1];
    v.cR = c[k + 1];
    v.nR = n[k + 1];
  } else {
    v.mR = from_right(m[0]);
    v.cR = from_right(c[0]);
    v.nR = from_right(n[0]);
  }
  return v;
}

// Values of K adjacent columns pulled by one column to the right (sh = 1:
// site k takes column k-1, site 0 the last column of the lane to the
// left), to the left (sh = -1), or not at all (sh = 0).  sh is
// wavefront-uniform; at wall rows the bounced populations are not shifted.
template <int K, class R>
__device__ __forceinline__ void shift_k(const R *v, int sh, R *out) {
  R l[K], r[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    l[k] = k > 0 ? v[k > 0 ? k - 1 : 0] : from_left(v[K - 1]);
    r[k] = k < K - 1 ? v[k < K - 1 ? k + 1 : 0] : from_right(v[0]);
  }
#pragma unroll
  for (int k = 0; k < K; ++k) out[k] = sh > 0 ? l[k] : (sh < 0 ? r[k] : v[k]);
}


// Pairs through one buffer access.  Vector elements are copied to scalars
// before any reinterpretation: a bit cast applied directly to an element
// of an ext_vector reads the vector's first element.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <class T>
struct PairIO;
template <>
struct PairIO<float> {
  static __device__ __forceinline__ void load(rsrc_t r, unsigned v, unsigned s, float &a,
                                              float &b) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0);
    const unsigned w0 = w[0], w1 = w[1];
    a = __uint_as_float(w0);
    b = __uint_as_float(w1);
  }
  template <int POL>
  static __device__ __forceinline__ void store(float a, float b, rsrc_t r, unsigned v,
                                               unsigned s) {
    u32x2 w;
    w[0] = __float_as_uint(a);
    w[1] = __float_as_uint(b);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, v, s, POL);
  }
};
template <>
struct PairIO<double> {
  static __device__ __forceinline__ void load(rsrc_t r, unsigned v, unsigned s, double &a,
                                              double &b) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0);
    const unsigned w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
    a = __hiloint2double(int(w1), int(w0));
    b = __hiloint2double(int(w3), int(w2));
  }
  template <int POL>
  static __device__ __forceinline__ void store(double a, double b, rsrc_t r, unsigned v,
                                               unsigned s) {
    u32x4 w;
    w[0] = unsigned(__double2loint(a));
    w[1] = unsigned(__double2hiint(a));
    w[2] = unsigned(__double2loint(b));
    w[3] = unsigned(__double2hiint(b));
    wide_store_begin();
    __builtin_amdgcn_raw_buffer_store_b128(w, r, v, s, POL);
    wide_store_guard();
  }
};
template <>
struct PairIO<_Float16> {
  static __device__ __forceinline__ void load(rsrc_t r, unsigned v, unsigned s, _Float16 &a,
                                              _Float16 &b) {
    const unsigned w = __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0);
    const unsigned short lo = (unsigned short)(w & 0xffffu), hi = (unsigned short)(w >> 16);
    a = __builtin_bit_cast(_Float16, lo);
    b = __builtin_bit_cast(_Float16, hi);
  }
};

// Three floats through one 96-bit load.
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
struct TripleIO {
  static __device__ __forceinline__ void load(rsrc_t r, unsigned v, unsigned s, float &a,
                                              float &b, float &c) {
    const u32x3 w = __builtin_amdgcn_raw_buffer_load_b96(r, v, s, 0);
    const unsigned w0 = w[0], w1 = w[1], w2 = w[2];
    a = __uint_as_float(w0);
    b = __uint_as_float(w1);
    c = __uint_as_float(w2);
  }
};

// Four floats through one 128-bit access.
struct QuadIO {
  static __device__ __forceinline__ void load(rsrc_t r, unsigned v, unsigned s, float &a,
                                              float &b, float &c, float &d) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0);
    const unsigned w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
    a = __uint_as_float(w0);
    b = __uint_as_float(w1);
    c = __uint_as_float(w2);
    d = __uint_as_float(w3);
  }
  template <int POL>
  static __device__ __forceinline__ void store(float a, float b, float c, float d, rsrc_t r,
                                               unsigned v, unsigned s) {
    u32x4 w;
    w[0] = __float_as_uint(a);
    w[1] = __float_as_uint(b);
    w[2] = __float_as_uint(c);
    w[3] = __float_as_uint(d);
    wide_store_begin();
    __builtin_amdgcn_raw_buffer_store_b128(w, r, v, s, POL);
    wide_store_guard();
  }
};

// The row number as the loop's optimiser cannot follow it (readfirstlane
// of a wave-uniform value: the same number).  The row loop passes each
// row through it, so the byte offsets derived from the row (one per
// population plane and record) are computed where they are used, by scalar
// adds, instead of each becoming an induction variable of its own: those
// outnumbered the scalar registers, and the excess was kept in vector lanes
// at one v_readlane per use (float32 step: 28 such registers, none now;
// 1.5% faster on the 2048x2048 field).
__device__ __forceinline__ int opaque_row(int y) {
  return __builtin_amdgcn_readfirstlane(y);
}

// Byte offsets of one row in the step kernel's three groups.
struct RowOff {
  unsigned m, c, p;  // population rows y-1, y, y+1
  bool bot, top;
};

__device__ __forceinline__ RowOff row_offsets(int y, int ny, int walls, unsigned row_bytes) {
  const RowIdx r = row_index(y, 1, ny, walls);
  RowOff o;
  o.m = unsigned(r.rm) * row_bytes;
  o.c = unsigned(r.rc) * row_bytes;
  o.p = unsigned(r.rp) * row_bytes;
  o.bot = r.bot;
  o.top = r.top;
  return o;
}

// Per-lane byte offsets of columns x, x-1, x+1 inside a FG block (pairs)
// and an H block (singles).
struct ColOff {
  unsigned p0, pm, pp;  // pairs
  unsigned h0, hm, hp;  // singles
};

template <class P>
struct Pull {
  using R = typename P::R;
  using S = typename P::S;
  // f_i, g_i of the nine populations arriving at row r (one pair load each)
  static __device__ __forceinline__ void fg(rsrc_t rs, unsigned nxb, const RowOff &r,
                                            const ColOff &c, const Scales<P> &sc, R *f, R *g) {
    // nxb: bytes of one pair row (nx pairs)
    auto pair = [&](int dir, unsigned row, unsigned col, int i) {
#pragma clang fp contract(off)
      S a, b;
      PairIO<S>::load(rs, col, row + unsigned(dir) * nxb, a, b);
      if constexpr (P::SCALED) {
        f[i] = R(a) * sc.fi;
        g[i] = R(b) * sc.gi;
      } else {
        f[i] = R(a);
        g[i] = R(b);
      }
    };
    // One load per population on every path: at a wall row the source of
    // the three populations leaving through the wall is selected (uniform
    // over the wavefront), not branched to, so every row issues the same
    // sequence of memory operations.
    const bool bot = r.bot, top = r.top;
    pair(0, r.c, c.p0, 0);
    pair(1, r.c, c.pm, 1);
    pair(3, r.c, c.pp, 3);
    pair(0, bot ? r.c + 4 * nxb : r.m + 2 * nxb, c.p0, 2);
    pair(0, bot ? r.c + 7 * nxb : r.m + 5 * nxb, bot ? c.p0 : c.pm, 5);
    pair(0, bot ? r.c + 8 * nxb : r.m + 6 * nxb, bot ? c.p0 : c.pp, 6);
    pair(0, top ? r.c + 2 * nxb : r.p + 4 * nxb, c.p0, 4);
    pair(0, top ? r.c + 5 * nxb : r.p + 7 * nxb, top ? c.p0 : c.pp, 7);
    pair(0, top ? r.c + 6 * nxb : r.p + 8 * nxb, top ? c.p0 : c.pm, 8);
  }
  // h_1..h_8 arriving at row r (h[k] = h_{k+1}); hb: byte offset of the H
  // block in a row, nxh: bytes of one h row
  static __device__ __forceinline__ void h(rsrc_t rs, unsigned hb, unsigned nxh,
                                           const RowOff &r, const ColOff &c, R inv, R *out) {
    // off: byte offset of the source row and direction plane within the
    // H block; wall rows select their bounced source as in fg()
    auto one = [&](unsigned off, unsigned col, int k) {
      out[k] = bld<P>(rs, col, off + hb, inv);
    };
    const bool bot = r.bot, top = r.top;
    one(r.c, c.hm, 0);             // h_1 from x-1
    one(r.c + 2 * nxh, c.hp, 2);   // h_3 from x+1
    one(bot ? r.c + 3 * nxh : r.m + nxh, c.h0, 1);                    // h_2
    one(bot ? r.c + 6 * nxh : r.m + 4 * nxh, bot ? c.h0 : c.hm, 4);   // h_5
    one(bot ? r.c + 7 * nxh : r.m + 5 * nxh, bot ? c.h0 : c.hp, 5);   // h_6
    one(top ? r.c + nxh : r.p + 3 * nxh, c.h0, 3);                    // h_4
    one(top ? r.c + 4 * nxh : r.p + 6 * nxh, top ? c.h0 : c.hp, 6);   // h_7
    one(top ? r.c + 5 * nxh : r.p + 7 * nxh, top ? c.h0 : c.hm, 7);   // h_8
  }
};

// Moving-wall term of the bounced diagonal h populations (see pull_h).
template <class R>
__device__ __forceinline__ void wall_terms(bool bot, bool top, R rho_w, R uwb, R uwt,
                                           R *h) {
  if (bot) {
    const R kb = rho_w * uwb * R(1.0 / 6.0);
    h[4] += kb;
    h[5] -= kb;
  }
  if (top) {
    const R kt = rho_w * uwt * R(1.0 / 6.0);
    h[6] -= kt;
    h[7] += kt;
  }
}

// Strip geometry of the step kernel with K adjacent columns per lane: two
// halo columns on each side (2 / K lanes), the rest interior.
template <int K>
struct Strip {
  static constexpr int kHaloLanes = 2 / K;
  static constexpr int kCols = K * (kWave - 2 * kHaloLanes);  // interior columns
};

// s_waitcnt operand (gfx9 encoding) that waits for all vector memory
// operations only: vmcnt 0, expcnt and lgkmcnt at their maxima.
constexpr int kWaitVmcnt0 = (0xF << 8) | (0x7 << 4);

template <bool B>
struct BoolC {
  static constexpr bool value = B;
};

// f(std::integral_constant<int, k>) for k = 0 .. N-1, unrolled.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Float16 halves of a 32-bit word.
__device__ __forceinline__ float half_lo(unsigned w) {
  return float(__builtin_bit_cast(_Float16, (unsigned short)(w & 0xffffu)));
}
__device__ __forceinline__ float half_hi(unsigned w) {
  return float(__builtin_bit_cast(_Float16, (unsigned short)(w >> 16)));
}
// A widened float16 value times a scale, rounded once: written as a fused
// multiply-add with +0 so that the widening and the product are one
// mixed-precision instruction (v_fma_mix_f32).  The result is the rounded
// product, except that a product of -0 becomes +0.
__device__ __forceinline__ float scale_half(float h, float s) { return __builtin_fmaf(h, s, 0.0f); }
__device__ __forceinline__ unsigned halves(float lo, float hi) {
  const unsigned short a = __builtin_bit_cast(unsigned short, _Float16(lo)),
                       b = __builtin_bit_cast(unsigned short, _Float16(hi));
  return unsigned(a) | (unsigned(b) << 16);
}

// Float16 storage rounds stochastically.  Round-to-nearest of a slowly
// varying value makes nearly the same error every step, and those errors
// add up linearly in time; stochastic rounding makes them unbiased and
// uncorrelated.  Measured on the 100x100 convection test (u = 0.05, 2000
// steps) the phi error against float64 falls from 4.2e-3 to 1.3e-4.
//
// Integer hash (multiply-xorshift; the constants of C. Wellons' lowbias32).
__device__ __forceinline__ unsigned hash32(unsigned x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}
// Two values to packed float16, rounded stochastically: 13 bits of a hash
// of both values' float32 bits and of key are added below the 10 kept
// mantissa bits, and the sum is truncated (round toward zero), so a value
// rounds away from zero with probability equal to its fractional distance.
// The bits come from the values themselves, so the rounding is reproducible
// and changes from step to step as the values do.  (Below the smallest
// normal float16, 2^-14, more than 13 bits are dropped and the rounding
// leans toward zero: at the default scales that is below 1.5e-8 of f and g
// and 1e-9 of h.)
__device__ __forceinline__ unsigned halves_sr(float lo, float hi, unsigned key) {
  const unsigned bl = __float_as_uint(lo), bh = __float_as_uint(hi);
  const unsigned r = hash32(bl ^ ((bh << 16) | (bh >> 16)) ^ key);
  const float a = __uint_as_float(bl + (r & 0x1fffu));
  const float b = __uint_as_float(bh + ((r >> 16) & 0x1fffu));
  return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(a, b));
}
// Packed float16 words (f_i, g_i) of one site's nine scaled deviations:
// i = 1..8 rounded stochastically; their rounding errors (exact in float32)
// are added to the rest population, which stays at the site and is rounded
// to nearest.  The deviations of a site sum to zero, so the stored ones
// change the mass by that one rounding only, not by nine random ones.
// amax takes the largest magnitude packed: the conversion saturates at the
// float16 maximum 65504 without a sign of it, so the caller flags larger
// values (or NaN) as a lost state.
__device__ __forceinline__ void pack_fg(const float *f, const float *g, float sf, float sg,
                                        unsigned site, unsigned *w, float &amax) {
#pragma clang fp contract(off)
  float ef = -0.f, eg = -0.f;  // -0 + x is x: the first sum needs no add
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const float vf = f[i] * sf, vg = g[i] * sg;
    amax = fmaxf(amax, fmaxf(fabsf(vf), fabsf(vg)));
    w[i] = halves_sr(vf, vg, site * 32u + unsigned(i));
    ef += vf - half_lo(w[i]);
    eg += vg - half_hi(w[i]);
  }
  const float v0 = f[0] * sf + ef, u0 = g[0] * sg + eg;
  amax = fmaxf(amax, fmaxf(fabsf(v0), fabsf(u0)));
  w[0] = halves(v0, u0);
}
constexpr float kHalfMax = 65504.f;  // largest finite float16

// Pull streaming with two adjacent columns per lane (float32 storage, or
// scaled float16 deviations): each population is loaded at the lane's own
// two columns, one (f, g) access (16 bytes float32, 8 bytes float16) and
// one h access (8 or 4 bytes) per plane; sources, bounce-back selection
// and load order as in Pull.  The shift by c_ix is applied in registers by
// shift_fg / shift_h when the row is used, not at the load, so the loads
// of the next row stay in flight meanwhile.  Float16 words are kept packed
// until then (decode_fg / decode_h): the prefetched row then holds half the
// registers, and no conversion consumes a load early.
template <class P>
struct Pull2 {
  using R = typename P::R;
  using S = typename P::S;
  static_assert((!P::SCALED && sizeof(S) == 4) || (P::SCALED && sizeof(S) == 2),
                "float32 or scaled float16 storage");
  static __device__ __forceinline__ void fg(rsrc_t rs, unsigned nxb, const RowOff &r,
                                            unsigned col, R (*f)[9], R (*g)[9]) {
    auto quad = [&](unsigned row, int i) {
      if constexpr (sizeof(S) == 4) {
        QuadIO::load(rs, col, row, f[0][i], g[0][i], f[1][i], g[1][i]);
      } else {  // packed (f, g) words of the two columns, decoded in decode_fg
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, col, row, 0);
        const unsigned w0 = w[0], w1 = w[1];
        f[0][i] = __uint_as_float(w0);
        f[1][i] = __uint_as_float(w1);
        g[0][i] = g[1][i] = R(0);
      }
    };
    const bool bot = r.bot, top = r.top;
    quad(r.c, 0);
    quad(r.c + nxb, 1);
    quad(r.c + 3 * nxb, 3);
    quad(bot ? r.c + 4 * nxb : r.m + 2 * nxb, 2);
    quad(bot ? r.c + 7 * nxb : r.m + 5 * nxb, 5);
    quad(bot ? r.c + 8 * nxb : r.m + 6 * nxb, 6);
    quad(top ? r.c + 2 * nxb : r.p + 4 * nxb, 4);
    quad(top ? r.c + 5 * nxb : r.p + 7 * nxb, 7);
    quad(top ? r.c + 6 * nxb : r.p + 8 * nxb, 8);
  }
  // float16 storage: unpack and scale what fg() loaded.  The scaled values
  // are rounded here (no contraction into the sums that use them), so the
  // result does not depend on which copy of the row code a site runs in.
  static __device__ __forceinline__ void decode_fg(const Scales<P> &sc, R (*f)[9], R (*g)[9]) {
    if constexpr (sizeof(S) == 2) {
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        const unsigned w0 = __float_as_uint(f[0][i]), w1 = __float_as_uint(f[1][i]);
        f[0][i] = scale_half(half_lo(w0), sc.fi);
        g[0][i] = scale_half(half_hi(w0), sc.gi);
        f[1][i] = scale_half(half_lo(w1), sc.fi);
        g[1][i] = scale_half(half_hi(w1), sc.gi);
      }
    }
  }
  // float16 storage: unpack and scale what h() loaded
  static __device__ __forceinline__ void decode_h(R inv, R (*h)[8]) {
    if constexpr (sizeof(S) == 2) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const unsigned w = __float_as_uint(h[0][k]);
        h[0][k] = scale_half(half_lo(w), inv);
        h[1][k] = scale_half(half_hi(w), inv);
      }
    }
  }
  // shift of population i (1: from the left column, -1: from the right);
  // populations bounced at a wall row come from the site itself
  static __device__ __forceinline__ int shift_of(int i, bool bot, bool top) {
    switch (i) {
      case 1: return 1;
      case 3: return -1;
      case 5: return bot ? 0 : 1;
      case 6: return bot ? 0 : -1;
      case 7: return top ? 0 : -1;
      case 8: return top ? 0 : 1;
      default: return 0;
    }
  }
  static __device__ __forceinline__ void shift_fg(bool bot, bool top, R (*f)[9], R (*g)[9]) {
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const int sh = shift_of(i, bot, top);
      if (i == 2 || i == 4) continue;
      R a[2] = {f[0][i], f[1][i]}, b[2] = {g[0][i], g[1][i]}, oa[2], ob[2];
      shift_k<2>(a, sh, oa);
      shift_k<2>(b, sh, ob);
      f[0][i] = oa[0];
      f[1][i] = oa[1];
      g[0][i] = ob[0];
      g[1][i] = ob[1];
    }
  }
  static __device__ __forceinline__ void h(rsrc_t rs, unsigned hb, unsigned nxh,
                                           const RowOff &r, unsigned col, R (*out)[8]) {
    auto two = [&](unsigned off, int k) {
      if constexpr (sizeof(S) == 4) {
        PairIO<float>::load(rs, col, off + hb, out[0][k], out[1][k]);
      } else {  // packed h word of the two columns, decoded in decode_h
        const unsigned w = __builtin_amdgcn_raw_buffer_load_b32(rs, col, off + hb, 0);
        out[0][k] = __uint_as_float(w);
        out[1][k] = R(0);
      }
    };
    const bool bot = r.bot, top = r.top;
    two(r.c, 0);                                   // h_1
    two(r.c + 2 * nxh, 2);                         // h_3
    two(bot ? r.c + 3 * nxh : r.m + nxh, 1);       // h_2
    two(bot ? r.c + 6 * nxh : r.m + 4 * nxh, 4);   // h_5
    two(bot ? r.c + 7 * nxh : r.m + 5 * nxh, 5);   // h_6
    two(top ? r.c + nxh : r.p + 3 * nxh, 3);       // h_4
    two(top ? r.c + 4 * nxh : r.p + 6 * nxh, 6);   // h_7
    two(top ? r.c + 5 * nxh : r.p + 7 * nxh, 7);   // h_8
  }
  // h[k] = h_{k+1}
  static __device__ __forceinline__ void shift_h(bool bot, bool top, R (*h)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k == 1 || k == 3) continue;
      const int sh = shift_of(k + 1, bot, top);
      R a[2] = {h[0][k], h[1][k]}, o[2];
      shift_k<2>(a, sh, o);
      h[0][k] = o[0];
      h[1][k] = o[1];
    }
  }
};

// Which product of the phase-field and surfactant sources is fused
// (collide_fg): the float16 kernels take the first one written, the time
// difference; the others what the compiler used to choose for them.
template <class P, bool NS>
constexpr bool kFluxF = NS && !P::SCALED;
template <class P, bool NS, bool GENR>
constexpr bool kFluxG = NS && !P::SCALED && !(GENR && sizeof(typename P::R) == 8);

// The fused step: pull-stream + boundaries, phi/psi/sigma, stencils, forces,
// closures, three MRT collisions, store.  Each lane holds K adjacent
// columns.  The two columns on each side of the interior are halo: they
// rebuild phi, psi, sigma for the stencils of the interior columns but
// store nothing (the outermost one only serves the rebuild of the next,
// which needs the old rest values one column further out).
// The row loop is software-pipelined: the loads for row y+1 are issued
// before the arithmetic and stores of row y.
// One tile (strip x rows) of one simulation, executed by one wavefront.
// NS: velocity from the Navier-Stokes LB (h); otherwise prescribed (u held
// in aux slots 0, 1; only f and g evolve).
// K = 2 (float32 storage, even nx): every access of a lane covers two
// sites, 16 bytes per (f, g) plane and 8 per h plane.
template <class P, int K, bool GENR, bool HAS_S, bool NS>
__device__ __forceinline__ void step_tile(const StepArgs<P> &a, const int strip, const int y0,
                                          const int y1) {
  using R = typename P::R;
  using S = typename P::S;
  using A = typename P::A;
  static_assert(K == 1 || (K == 2 && sizeof(A) == 4 &&
                           ((!P::SCALED && sizeof(S) == 4) || (P::SCALED && sizeof(S) == 2))),
                "two columns per lane: float32 or float16 storage");
  constexpr int HL = Strip<K>::kHaloLanes;
  constexpr int COLS = Strip<K>::kCols;
  const int lane = threadIdx.x & (kWave - 1);
  const int nx = a.nx, ny = a.ny, walls = a.walls;
  const int x0 = strip * COLS;
  const int wl = min(COLS, nx - x0) / K;  // interior lanes (nx is a multiple of K)
  const bool interior = lane >= HL && lane < HL + wl;
  int xl = x0 - K * HL + K * min(lane, wl + 2 * HL - 1);  // first column of the lane
  xl %= nx;
  if (xl < 0) xl += nx;
  const unsigned xc = unsigned(xl);
  const unsigned xcm = xl == 0 ? unsigned(nx - 1) : xc - 1;
  const unsigned xcp = xl == nx - 1 ? 0u : xc + 1;
  constexpr unsigned ES = sizeof(S), EA = sizeof(A);
  ColOff co;
  co.p0 = xc * 2 * ES;
  co.pm = xcm * 2 * ES;
  co.pp = xcp * 2 * ES;
  co.h0 = xc * ES;
  co.hm = xcm * ES;
  co.hp = xcp * ES;
  const unsigned brest = xc * P::kRest * EA;  // this lane's first rest record in a row
  const unsigned baux = xc * P::kAux * EA;    // this lane's first aux record
  const unsigned nsites = unsigned(nx) * unsigned(ny);
  const unsigned nxb = unsigned(nx) * 2 * ES;      // one FG pair row
  const unsigned nxh = unsigned(nx) * ES;          // one h row
  const unsigned hb = 9u * nxb;                    // H block offset in a row
  const unsigned rows_s = unsigned(kPlanes) * nxh; // bytes per population row
  const unsigned rrow = unsigned(nx) * P::kRest * EA; // bytes per rest row
  const unsigned arow = unsigned(nx) * P::kAux * EA;  // bytes per aux row
  const rsrc_t rsrc = make_rsrc(a.src, unsigned(kPlanes) * nsites * ES);
  const rsrc_t rdst = make_rsrc(a.dst, unsigned(kPlanes) * nsites * ES);
  const rsrc_t rrest = make_rsrc(a.src_rest, unsigned(P::kRest) * nsites * EA);
  const rsrc_t rdrest = make_rsrc(a.dst_rest, unsigned(P::kRest) * nsites * EA);
  const rsrc_t raux = make_rsrc(a.aux, unsigned(P::kAux) * nsites * EA);
  const Phys<R> &p = a.p;
  const Scales<P> &sc = a.sc;
  // the aux records (ux, uy) of a lane's two float32 sites: one 16-byte access
  constexpr bool kAuxQuad = sizeof(A) == 4 && K == 2;
  // the step reads an aux record: the previous velocity, or the prescribed one
  constexpr bool kAuxRead = !P::HDEV || !NS;

  // old (phi, psi) of this lane's columns at row y, wrapped or clamped
  auto rest_at = [&](int y, R *X, R *Y) {
    const unsigned ro = unsigned(wrap_row(y, ny, walls)) * rrow;
    if constexpr (K == 2 && P::kRest == 2) {  // both records in one access
      QuadIO::load(rrest, brest, ro, X[0], Y[0], X[1], Y[1]);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        A u, v;
        PairIO<A>::load(rrest, brest + unsigned(k) * P::kRest * EA, ro, u, v);
        X[k] = R(u);
        Y[k] = R(v);
      }
    }
  };
  // raw stored deviations of f and g pulled to row r
  auto load_fg = [&](int r, R (*d)[9], R (*q)[9]) {
    const RowOff o = row_offsets(r, ny, walls, rows_s);
    if constexpr (K == 1)
      Pull<P>::fg(rsrc, nxb, o, co, sc, d[0], q[0]);
    else
      Pull2<P>::fg(rsrc, nxb, o, co.p0, d, q);
  };
  // loads of row y that the rebuild of row y+1 does not need
  auto load_row = [&](int y, R (*h)[8], R *uxp, R *uyp) {
    if constexpr (NS) {
      const RowOff o = row_offsets(y, ny, walls, rows_s);
      if constexpr (K == 1)
        Pull<P>::h(rsrc, hb, nxh, o, co, sc.hi, h[0]);
      else
        Pull2<P>::h(rsrc, hb, nxh, o, co.h0, h);
    }
    // u: the previous level, or the prescribed field; with float16 storage
    // the previous velocity comes from the rest record (P, rho u) instead
    if constexpr (!kAuxRead) {
#pragma unroll
      for (int k = 0; k < K; ++k) uxp[k] = uyp[k] = R(0);
    } else if constexpr (kAuxQuad) {  // (ux, uy) of both sites in one access
      QuadIO::load(raux, baux, unsigned(y) * arow, uxp[0], uyp[0], uxp[1], uyp[1]);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        A u, v;
        PairIO<A>::load(raux, baux + unsigned(k) * P::kAux * EA, unsigned(y) * arow, u, v);
        uxp[k] = R(u);
        uyp[k] = R(v);
      }
    }
  };
  // old (P, rho ux, rho uy) of this lane's columns at row y (float16
  // storage only)
  struct HR {
    R pr[K], jx[K], jy[K];
  };
  auto hrest_at = [&](int y, HR &v) {
    if constexpr (P::HDEV && NS) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        TripleIO::load(rrest, brest + unsigned(k) * P::kRest * EA + 2 * EA,
                       unsigned(wrap_row(y, ny, walls)) * rrow, v.pr[k], v.jx[k], v.jy[k]);
    }
  };
  // rebuild row r from its raw deviations: new phi, psi, sigma, and the
  // deviations relative to them (in place), given the old rest fields at
  // rows r-1, r, r+1 of the lane's columns
  auto rebuild = [&](int r, const R *Xm, const R *Xc, const R *Xn, const R *Ym, const R *Yc,
                     const R *Yn, R (*d)[9], R (*q)[9], R *ph, R *ps, R *sg) {
    const bool bot = walls && r == 0, top = walls && r == ny - 1;
    if constexpr (K == 2) {
      Pull2<P>::decode_fg(sc, d, q);
      Pull2<P>::shift_fg(bot, top, d, q);
    }
    static_for<K>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      R e[9];
      source_offsets(window_k<K, k>(Xm, Xc, Xn), bot, top, e);
      ph[k] = restream(d[k], e, Xc[k]);
      source_offsets(window_k<K, k>(Ym, Yc, Yn), bot, top, e);
      ps[k] = restream(q[k], e, Yc[k]);
      sg[k] = sigma_of(p, ps[k]);
    });
  };
  auto copy = [](R *dst, const R *src) {
#pragma unroll
    for (int k = 0; k < K; ++k) dst[k] = src[k];
  };

  // Prologue: phi, psi, sigma of rows y0 and y0-1, and the loop's first
  // prefetch.  With float32 and float64 storage every load is issued before
  // the first rebuild, so a tile starts after one round trip to memory
  // rather than three (1% faster on the 2048x2048 field for float64, 4-10%
  // shorter steps on grids too small to fill the device).  Float16 storage
  // keeps the rebuilds between the loads (3% faster there).
  constexpr bool kEarlyLoads = !P::SCALED;
  // old rest values of this lane's columns, rows y-1 .. y+2
  R X0[K], X1[K], X2[K], X3[K], Y0[K], Y1[K], Y2[K], Y3[K];
  rest_at(y0 - 1, X0, Y0);
  rest_at(y0, X1, Y1);
  rest_at(y0 + 1, X2, Y2);
  rest_at(y0 + 2, X3, Y3);
  R dc[K][9], qc[K][9];
  R phc[K], psc[K], sgc[K], phm[K], psm[K], sgm[K];
  load_fg(y0, dc, qc);
  // row y0-1, unless it is the mirror ghost below the bottom wall
  const bool ghost_below = walls && y0 == 0;
  const int ym = y0 == 0 ? ny - 1 : y0 - 1;
  R dt[K][9], qt[K][9], Xa[K], Ya[K];
  auto load_below = [&]() {
    if (!ghost_below) {
      rest_at(y0 - 2, Xa, Ya);
      load_fg(ym, dt, qt);
    }
  };
  auto rebuild_y0 = [&]() { rebuild(y0, X0, X1, X2, Y0, Y1, Y2, dc, qc, phc, psc, sgc); };
  auto rebuild_below = [&]() {
    if (ghost_below) {
      copy(phm, phc);
      copy(psm, psc);
      copy(sgm, sgc);
    } else {
      rebuild(ym, Xa, X0, X1, Ya, Y0, Y1, dt, qt, phm, psm, sgm);
    }
  };
  if (kEarlyLoads) {
    load_below();
  } else {
    rebuild_y0();
    load_below();
    rebuild_below();
  }

  // Software pipeline: the loads for row y+1 are issued before the
  // arithmetic and stores of row y.  Every iteration issues the same
  // memory operations on every path (no divergent or row-dependent branch
  // around a load or store), so the wait at the top of an iteration only
  // covers the loads it needs, not the stores just issued.
  R dn[K][9], qn[K][9];  // raw deviations of row y+1
  R hr[K][8];            // h of row y
  R uxr[K], uyr[K];
  // above the top wall the next row is the mirror ghost: the load of row
  // ny-1 keeps the sequence uniform and its values are not used
  auto next_fg_row = [&](int y) { return wrap_row(y, ny, walls); };
  load_fg(next_fg_row(y0 + 1), dn, qn);
  load_row(y0, hr, uxr, uyr);
  // rest (P, rho u) of rows y-1, y, y+1 and the prefetched y+2
  HR Hm{}, Hc{}, Hn{}, Hq{};
  if constexpr (P::HDEV && NS) {
    hrest_at(y0 - 1, Hm);
    hrest_at(y0, Hc);
    hrest_at(y0 + 1, Hn);
  }

  if (kEarlyLoads) {
    rebuild_y0();
    rebuild_below();
  }

  // Stores are issued by every lane (the same memory operations on every
  // path); a halo lane's offsets are kDropped, so the hardware discards its
  // part and only interior lanes write.
  const ColOff cs = {interior ? co.p0 : kDropped, 0u, 0u, interior ? co.h0 : kDropped, 0u, 0u};
  const unsigned brest_s = interior ? brest : kDropped, baux_s = interior ? baux : kDropped;
  bool bad = false;

  auto row_step = [&](int y, auto prefetch) {
    // rebuild the next row from the raw deviations loaded last iteration
    R phn[K], psn[K], sgn[K];
    const bool ghost = walls && y == ny - 1;
    if (!ghost) {
      rebuild(y + 1 == ny ? 0 : y + 1, X1, X2, X3, Y1, Y2, Y3, dn, qn, phn, psn, sgn);
    } else {  // mirror ghost row above the top wall
      copy(phn, phc);
      copy(psn, psc);
      copy(sgn, sgc);
    }
    R h[K][8];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < 8; ++i) h[k][i] = hr[k][i];
    if constexpr (K == 2 && NS) {
      Pull2<P>::decode_h(sc.hi, h);
      Pull2<P>::shift_h(walls && y == 0, walls && y == ny - 1, h);
    }
    R uxp[K], uyp[K], Sxp[K], Syp[K];
    copy(uxp, uxr);
    copy(uyp, uyr);
    // the previous level's mass flux, Eq. (16), from the previous phi of
    // rows y-1, y, y+1 (the rest values the rebuilds read)
    static_for<K>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if constexpr (HAS_S && NS) {
        R gx, gy;
        grad9(window_k<K, k>(X0, X1, X2), gx, gy);
        mass_flux(p, X1[k], gx, gy, Sxp[k], Syp[k]);
      } else {
        Sxp[k] = Syp[k] = R(0);
      }
    });
    if constexpr (P::HDEV && NS) {  // add back the rest parts of the arriving h
      // (no contraction: float16 storage rounds stochastically from all
      // 32 bits, so every copy of the row code must give the same bits)
      static_for<K>([&](auto kc) {
#pragma clang fp contract(off)
        constexpr int k = decltype(kc)::value;
        R b[8];
        h_arrival_basis(window_k<K, k>(Hm.pr, Hc.pr, Hn.pr), window_k<K, k>(Hm.jx, Hc.jx, Hn.jx),
                        window_k<K, k>(Hm.jy, Hc.jy, Hn.jy), walls && y == 0,
                        walls && y == ny - 1, b);
#pragma unroll
        for (int i = 0; i < 8; ++i) h[k][i] += b[i];
        const R irho = recip(p.rhoB + p.drho * (X1[k] - p.phiB));
        uxp[k] = Hc.jx[k] * irho;
        uyp[k] = Hc.jy[k] * irho;
      });
    }
    R dnn[K][9], qnn[K][9];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        dnn[k][i] = dn[k][i];
        qnn[k][i] = qn[k][i];
      }

    R X4[K], Y4[K];
    copy(X4, X3);
    copy(Y4, Y3);
    if constexpr (decltype(prefetch)::value) {
      rest_at(y + 3, X4, Y4);
      load_fg(next_fg_row(y + 2), dn, qn);
      load_row(y + 1, hr, uxr, uyr);
      hrest_at(y + 2, Hq);
    }

    const bool bot = walls && y == 0, top = walls && y == ny - 1;
    R oux[K], ouy[K];
    HR hn{};
    static_for<K>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const R php = X1[k], psp = Y1[k];
      if constexpr (NS) wall_terms(bot, top, rho_of(p, php), p.uwb, p.uwt, h[k]);

      // stencils from the register window
      const Nine<R> vphi = window_k<K, k>(phm, phc, phn);
      const Nine<R> vsig = window_k<K, k>(sgm, sgc, sgn);
      R gfx, gfy, gsx, gsy;
      grad9(vphi, gfx, gfy);
      grad9(vsig, gsx, gsy);
      const R lphi = lap9(vphi);

      Front<R> s;
      if constexpr (NS)
        site_front<R, HAS_S, !P::SCALED>(p, s, phc[k], psc[k], sgc[k], gfx, gfy, lphi, gsx, gsy, h[k], php,
                             psp, uxp[k], uyp[k], Sxp[k], Syp[k]);
      else
        site_front_prescribed<R>(p, s, phc[k], psc[k], gfx, gfy, uxp[k], uyp[k], php, psp);
      if (GENR) {
        const Nine<R> vpsi = window_k<K, k>(psm, psc, psn);
        grad9(vpsi, s.gpx, s.gpy);
      } else {
        s.gpx = s.gpy = R(0);
      }
      if constexpr (NS)
        collide_site<R, GENR, kFluxF<P, NS>, kFluxG<P, NS, GENR>>(p, s, dc[k], qc[k], h[k]);
      else
        collide_fg<R, GENR, kFluxF<P, NS>, kFluxG<P, NS, GENR>>(p, s, dc[k], qc[k]);
      if constexpr (P::HDEV && NS) {  // h as deviations from this site's new rest parts
#pragma clang fp contract(off)
        hn.pr[k] = s.P;
        hn.jx[k] = s.jx;
        hn.jy[k] = s.jy;
        R b[8];
        h_store_basis(HRest<R>{s.P, s.jx, s.jy}, b);
#pragma unroll
        for (int i = 0; i < 8; ++i) h[k][i] -= b[i];
      }
      oux[k] = s.ux;
      ouy[k] = s.uy;
      bad |= interior && !isfinite(phc[k] + psc[k] + s.ux + s.uy);
    });

    const unsigned rcs = unsigned(y) * rows_s;
    float amax = 0.f;  // largest scaled deviation stored as float16
    if constexpr (K == 1) {
      if constexpr (P::SCALED) {  // float16: packed words, stochastic rounding
        unsigned w[9];
        pack_fg(dc[0], qc[0], sc.f, sc.g, unsigned(y) * unsigned(nx) + xc, w, amax);
#pragma unroll
        for (int i = 0; i < 9; ++i)
          __builtin_amdgcn_raw_buffer_store_b32(w[i], rdst, cs.p0,
                                                rcs + unsigned(i) * nxb, P::kStorePol);
      } else {
#pragma unroll
        for (int i = 0; i < 9; ++i)
          PairIO<S>::template store<P::kStorePol>(S(dc[0][i]), S(qc[0][i]), rdst, cs.p0,
                           rcs + unsigned(i) * nxb);
      }
      if constexpr (NS && P::SCALED) {
        const unsigned key = (unsigned(y) * unsigned(nx) + xc) * 32u + 16u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float v = h[0][i] * sc.h;
          amax = fmaxf(amax, fabsf(v));
          __builtin_amdgcn_raw_buffer_store_b16(
              (unsigned short)(halves_sr(v, 0.f, key + unsigned(i)) & 0xffffu),
              rdst, cs.h0, rcs + hb + unsigned(i) * nxh, P::kStorePol);
        }
      } else if constexpr (NS) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          bst<P>(h[0][i], rdst, cs.h0, rcs + hb + unsigned(i) * nxh);
      }
      if constexpr (P::HDEV && NS) {  // (phi, psi, P, rho ux) and rho uy
        QuadIO::store<P::kStorePol>(phc[0], psc[0], hn.pr[0], hn.jx[0], rdrest,
                                    brest_s, unsigned(y) * rrow);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(hn.jy[0]), rdrest,
                                              brest_s + 4 * EA, unsigned(y) * rrow,
                                              P::kStorePol);
      } else {
        PairIO<A>::template store<P::kStorePol>(A(phc[0]), A(psc[0]), rdrest, brest_s,
                                                unsigned(y) * rrow);
      }
      if constexpr (!P::HDEV && NS)
        PairIO<A>::template store<P::kStorePol>(A(oux[0]), A(ouy[0]), raux, baux_s,
                                                unsigned(y) * arow);
    } else if constexpr (sizeof(S) == 4) {
#pragma unroll
      for (int i = 0; i < 9; ++i)
        QuadIO::store<P::kStorePol>(dc[0][i], qc[0][i], dc[1][i], qc[1][i], rdst,
                                    cs.p0, rcs + unsigned(i) * nxb);
      if constexpr (NS) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          PairIO<S>::template store<P::kStorePol>(
              h[0][i], h[1][i], rdst, cs.h0, rcs + hb + unsigned(i) * nxh);
      }
      QuadIO::store<P::kStorePol>(phc[0], psc[0], phc[1], psc[1], rdrest,
                                  brest_s, unsigned(y) * rrow);
      if constexpr (NS)
        QuadIO::store<P::kStorePol>(oux[0], ouy[0], oux[1], ouy[1], raux,
                                    baux_s, unsigned(y) * arow);
    } else {  // float16 deviations, scaled: four halves per (f, g) plane, two per h plane
      const unsigned site = unsigned(y) * unsigned(nx) + xc;
      unsigned w0[9], w1[9];
      pack_fg(dc[0], qc[0], sc.f, sc.g, site, w0, amax);
      pack_fg(dc[1], qc[1], sc.f, sc.g, site + 1u, w1, amax);
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        u32x2 w;
        w[0] = w0[i];
        w[1] = w1[i];
        __builtin_amdgcn_raw_buffer_store_b64(w, rdst, cs.p0, rcs + unsigned(i) * nxb,
                                              P::kStorePol);
      }
      if constexpr (NS) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float v0 = h[0][i] * sc.h, v1 = h[1][i] * sc.h;
          amax = fmaxf(amax, fmaxf(fabsf(v0), fabsf(v1)));
          __builtin_amdgcn_raw_buffer_store_b32(
              halves_sr(v0, v1, site * 32u + 16u + unsigned(i)),
              rdst, cs.h0, rcs + hb + unsigned(i) * nxh, P::kStorePol);
        }
      }
      if constexpr (P::HDEV && NS) {
        // the two 5-float rest records (40 bytes) as 16 + 16 + 8 bytes
        QuadIO::store<P::kStorePol>(phc[0], psc[0], hn.pr[0], hn.jx[0], rdrest,
                                    brest_s, unsigned(y) * rrow);
        QuadIO::store<P::kStorePol>(hn.jy[0], phc[1], psc[1], hn.pr[1], rdrest,
                                    brest_s + 4 * EA, unsigned(y) * rrow);
        PairIO<A>::template store<P::kStorePol>(hn.jx[1], hn.jy[1], rdrest,
                                                brest_s + 8 * EA, unsigned(y) * rrow);
      } else {
#pragma unroll
        for (int k = 0; k < K; ++k)
          PairIO<A>::template store<P::kStorePol>(phc[k], psc[k], rdrest,
                                                  brest_s + unsigned(k) * P::kRest * EA,
                                                  unsigned(y) * rrow);
      }
    }

    // a deviation beyond the float16 range was stored saturated: the state
    // is lost, as with a non-finite value
    if constexpr (P::SCALED) bad |= interior && !(amax <= kHalfMax);

    // slide the windows
    copy(phm, phc);
    copy(psm, psc);
    copy(sgm, sgc);
    copy(phc, phn);
    copy(psc, psn);
    copy(sgc, sgn);
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        dc[k][i] = dnn[k][i];
        qc[k][i] = qnn[k][i];
      }
    copy(X0, X1);
    copy(X1, X2);
    copy(X2, X3);
    copy(X3, X4);
    copy(Y0, Y1);
    copy(Y1, Y2);
    copy(Y2, Y3);
    copy(Y3, Y4);
    if constexpr (P::HDEV && NS) {
      Hm = Hc;
      Hc = Hn;
      Hn = Hq;
    }
  };

  // The first row needs the loads just issued in any case.  Waiting for
  // them here leaves nothing of the prologue in flight at the loop head,
  // so the waits placed there serve only the previous iteration's loads
  // (long complete) instead of also holding back on its stores.
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  // (This loop form, with its own trip counter and the row after the loop
  // taken from it, and the wall and wrap tests written on y itself, gives
  // a loop body with 1% fewer instructions: 1.5% faster for float32 and 1%
  // for float64 storage on the 2048x2048 field, same bits.)
  int y = y0;
  for (int i = y0; i < y1 - 1; ++i, ++y) row_step(opaque_row(y), BoolC<true>{});
  row_step(y, BoolC<false>{});  // the last row prefetches nothing
  if (bad) *a.flag = 1;
}

// Grid size of the single-grid step kernel: rounds of kXcds workgroups,
// enough for the band with the most tiles.
template <class P>
int step_grid(const StepArgs<P> &a) {
  int most = 0;
  for (int x = 0; x < kXcds; ++x)
    most = std::max(most, band_of(x, a.ny, a.rows, a.tail_rows, a.tail_h).nchunks);
  return kXcds * ((most * a.nstrips + P::kBlockWaves - 1) / P::kBlockWaves);
}

// One time step of one simulation: one wavefront per tile.  The hardware
// deals workgroups to the XCDs round-robin, so workgroup b runs on XCD
// b % 8 and takes the (b / 8)-th group of tiles of that XCD's band of rows:
// the halo rows a tile shares with the tiles above and below are read
// through the same L2 (measured on 2048x2048, float32 storage: reads past
// L2 fell from 226 to 160 bytes per site at equal speed).  Tiles are
// strip-major (consecutive wavefronts take adjacent strips of the same
// rows, so each row streams contiguously from memory).  Each band is
// dispatched in order, so its last chunks are the ones still running when
// the launch drains; they are short, which shortens the drain.
template <class P, int K, bool GENR, bool HAS_S, bool NS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P::kMinWaves)))
lbm_step_kernel(const StepArgs<P> a) {
  // the wavefront index is the same on every lane: make it a scalar so all
  // row arithmetic and row offsets stay in SGPRs
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const Band b = band_of(int(blockIdx.x % kXcds), a.ny, a.rows, a.tail_rows, a.tail_h);
  const int tile = int(blockIdx.x / kXcds) * P::kBlockWaves + wave;
  const int chunk = tile / a.nstrips;
  if (chunk >= b.nchunks) return;  // whole wavefronts only
  const bool full = chunk < b.nlong;
  const int y0 = full ? b.y0 + chunk * a.rows : b.ys + (chunk - b.nlong) * a.tail_h;
  const int y1 = full ? min(y0 + a.rows, b.ys) : min(y0 + a.tail_h, b.y1);
  step_tile<P, K, GENR, HAS_S, NS>(a, tile - chunk * a.nstrips, y0, y1);
}


// ------------------------------------------------- several steps per launch

// Block step: one workgroup advances a 16 x 16 block of sites `steps` time
// steps in LDS, one thread per site, and stores the sites whose every
// dependence lay inside the block.  A step reaches two sites in every
// direction (a site pulls from its neighbours, and its stencils need the
// phi, psi, sigma that its neighbours rebuild from theirs), so `steps` steps
// leave 16 - 2 (2 steps - 1) sites a side, the blocks of neighbouring
// workgroups overlap, and no workgroup waits for another.
//
// What bounds it: latency.  On a grid too small to fill the device a step of
// lbm_step_kernel is one wavefront's walk (6.5 us for float32 storage: three
// row rebuilds and a collision of two columns in one wavefront, 1700 vector
// instructions, after a round trip to memory and between two launches).
// Here a launch costs 3.0 us once (launch, loads, stores) and each step
// 1.5 us (one rebuild and one collision per wavefront, 700 instructions at
// one wavefront per SIMD, and two barriers); float64 2.3 us, float16 2.9 us.
// Measured per step on MI355X, lbm_step_kernel -> this (steps per launch):
// 64^2 float32 6.5 -> 2.7 us (3), float64 7.2 -> 3.1 us (3), float16
// 7.9 -> 4.0 us (3); 128^2 float32 6.6 -> 3.4 us (2); 256x128 float32
// 6.8 -> 4.0 us (2).  Larger blocks (32 x 16, 32 x 32 threads) waste fewer
// sites but put 2 and 4 wavefronts on a SIMD: 64^2 float32 3.3 us, 256x128
// 4.3 and 8.3 us.  Asking for 3 or 4 wavefronts per SIMD spills (256x128:
// 4.9 and 7.2 us).
//
// Each XCD takes a contiguous run of blocks: with blocks dealt round-robin
// the lines that neighbouring blocks share came through two L2s (256x128
// float32 6.3 us per step).
//
// The arithmetic of a site is that of step_tile, bit for bit, in every
// precision: the float16 kernels by their compilation pass, the others by
// the expressions spelled out with fused() (lbm_device.h).
constexpr int kBlockSide = 16;
constexpr int kBlockMaxSteps = 3;

template <class P>
struct BlockArgs {
  StepArgs<P> s;
  typename P::A *aux_out;  // new previous velocity (s.aux is read by several blocks)
  int steps;               // time steps of this launch
  int ntx, ntiles;         // blocks per row of blocks, in all
};

// Columns and rows of the block on each side that the last of `steps` steps
// cannot form.  Float16 storage with even nx rounds h in pairs of columns,
// both of which must be formed, and starts its blocks on even columns.
template <class P>
__host__ __device__ constexpr int block_halo_x(int steps) {
  return P::SCALED ? 2 * steps : 2 * steps - 1;
}
__host__ __device__ constexpr int block_halo_y(int steps) { return 2 * steps - 1; }

// Value of the other lane of an even/odd pair of lanes (quad permutation
// 1, 0, 3, 2).
__device__ __forceinline__ float pair_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));
}

template <class T>
struct Two {
  T a, b;
};

template <class P, bool GENR, bool HAS_S, bool NS>
__global__ void __launch_bounds__(kBlockSide * kBlockSide)
lbm_block_kernel(const BlockArgs<P> ba) {
  using R = typename P::R;
  using S = typename P::S;
  using A = typename P::A;
  constexpr int B = kBlockSide, N = B * B;
  static_assert(B > 2 * block_halo_x<P>(kBlockMaxSteps), "no site left after the last step");
  constexpr unsigned ES = sizeof(S), EA = sizeof(A);
  constexpr int NH = NS ? 8 : 1, NR = P::HDEV && NS ? 3 : 1;
  // one step's post-collision state of the block, in storage form, and the
  // scalars of the level being formed
  __shared__ Two<S> l_fg[8][N];       // f_i, g_i, i = 1..8
  __shared__ S l_h[NH][N];            // h_1..h_8
  __shared__ Two<A> l_rest[2][N];     // phi, psi of two levels
  __shared__ A l_sig[N];
  __shared__ A l_hr[NR][N];           // float16 storage: P, rho ux, rho uy

  const StepArgs<P> &a = ba.s;
  const Phys<R> &p = a.p;
  const Scales<P> &sc = a.sc;
  const int nx = a.nx, ny = a.ny, walls = a.walls, steps = ba.steps;
  const int hx = block_halo_x<P>(steps), hy = block_halo_y(steps);
  // workgroup b runs on XCD b % 8: each XCD takes a contiguous run of blocks,
  // which read the columns and rows they share through one L2
  const int per = int(gridDim.x) / kXcds;
  const int tile = int(blockIdx.x % kXcds) * per + int(blockIdx.x / kXcds);
  if (tile >= ba.ntiles) return;
  const int ty = tile / ba.ntx, tx = tile - ty * ba.ntx;
  const int lx = int(threadIdx.x) % B, ly = int(threadIdx.x) / B;
  const int gx = tx * (B - 2 * hx) - hx + lx, gy = ty * (B - 2 * hy) - hy + ly;
  const bool owned = lx >= hx && lx < B - hx && ly >= hy && ly < B - hy && gx < nx && gy < ny;
  int x = gx % nx, y = gy % ny;
  if (x < 0) x += nx;
  if (y < 0) y += ny;
  if (walls) y = gy < 0 ? 0 : (gy >= ny ? ny - 1 : gy);  // rows past a wall are never used
  const bool bot = walls && y == 0, top = walls && y == ny - 1;
  const bool even = P::SCALED && nx % 2 == 0;  // h rounded in pairs of columns

  // neighbours in the block; at a wall the stencils' row beyond it is the
  // wall row itself
  const int k0 = ly * B + lx;
  const int dl = lx > 0 ? -1 : 0, dr = lx < B - 1 ? 1 : 0;
  const int dm = ly > 0 && !bot ? -B : 0, dp = ly < B - 1 && !top ? B : 0;
  auto nine = [&](auto get) {
    Nine<R> v;
    v.mL = R(get(k0 + dm + dl));
    v.m = R(get(k0 + dm));
    v.mR = R(get(k0 + dm + dr));
    v.cL = R(get(k0 + dl));
    v.c = R(get(k0));
    v.cR = R(get(k0 + dr));
    v.nL = R(get(k0 + dp + dl));
    v.n = R(get(k0 + dp));
    v.nR = R(get(k0 + dp + dr));
    return v;
  };
  R d[9], q[9], h[8];
  Nine<R> X, Y, HP, HX, HY;  // previous level: phi, psi; P, rho ux, rho uy
  R uxp = R(0), uyp = R(0);
  bool bad = false;
  const unsigned ux_ = unsigned(x), uy_ = unsigned(y), unx = unsigned(nx);
  const unsigned nxb = unx * 2 * ES, nxh = unx * ES, hb = 9u * nxb;
  const unsigned rows_s = unsigned(kPlanes) * nxh;

  auto decode = [&](const Two<S> &w, int i) {
#pragma clang fp contract(off)
    if constexpr (P::SCALED) {
      d[i] = even ? scale_half(float(w.a), sc.fi) : R(w.a) * sc.fi;
      q[i] = even ? scale_half(float(w.b), sc.gi) : R(w.b) * sc.gi;
    } else {
      d[i] = R(w.a);
      q[i] = R(w.b);
    }
  };
  auto decode_h = [&](S w, int k) {
#pragma clang fp contract(off)
    if constexpr (P::SCALED)
      h[k] = even ? scale_half(float(w), sc.hi) : R(w) * sc.hi;
    else
      h[k] = R(w);
  };

  {  // first step: the state comes from memory
    const unsigned nsites = unx * unsigned(ny);
    const rsrc_t rsrc = make_rsrc(a.src, unsigned(kPlanes) * nsites * ES);
    const rsrc_t rrest = make_rsrc(a.src_rest, unsigned(P::kRest) * nsites * EA);
    const rsrc_t raux = make_rsrc(a.aux, unsigned(P::kAux) * nsites * EA);
    const unsigned xm = x == 0 ? unx - 1 : ux_ - 1, xp = x == nx - 1 ? 0u : ux_ + 1;
    const unsigned ym = y == 0 ? (walls ? 0u : unsigned(ny - 1)) : uy_ - 1;
    const unsigned yp = y == ny - 1 ? (walls ? uy_ : 0u) : uy_ + 1;
    const unsigned rc = uy_ * rows_s, rm = ym * rows_s, rp = yp * rows_s;
    Two<S> w[9];
    auto pair = [&](unsigned row, unsigned col, int i) {
      PairIO<S>::load(rsrc, row + col * 2 * ES, 0, w[i].a, w[i].b);
    };
    pair(rc, ux_, 0);
    pair(rc + nxb, xm, 1);
    pair(rc + 3 * nxb, xp, 3);
    pair(bot ? rc + 4 * nxb : rm + 2 * nxb, ux_, 2);
    pair(bot ? rc + 7 * nxb : rm + 5 * nxb, bot ? ux_ : xm, 5);
    pair(bot ? rc + 8 * nxb : rm + 6 * nxb, bot ? ux_ : xp, 6);
    pair(top ? rc + 2 * nxb : rp + 4 * nxb, ux_, 4);
    pair(top ? rc + 5 * nxb : rp + 7 * nxb, top ? ux_ : xp, 7);
    pair(top ? rc + 6 * nxb : rp + 8 * nxb, top ? ux_ : xm, 8);
    auto rest = [&](unsigned yy, unsigned xx, R &u, R &v) {
      A s, t;
      PairIO<A>::load(rrest, (yy * unx + xx) * (P::kRest * EA), 0, s, t);
      u = R(s);
      v = R(t);
    };
    rest(ym, xm, X.mL, Y.mL);
    rest(ym, ux_, X.m, Y.m);
    rest(ym, xp, X.mR, Y.mR);
    rest(uy_, xm, X.cL, Y.cL);
    rest(uy_, ux_, X.c, Y.c);
    rest(uy_, xp, X.cR, Y.cR);
    rest(yp, xm, X.nL, Y.nL);
    rest(yp, ux_, X.n, Y.n);
    rest(yp, xp, X.nR, Y.nR);
    if constexpr (P::HDEV && NS) {
      auto hrest = [&](unsigned yy, unsigned xx, R &u, R &v, R &t) {
        TripleIO::load(rrest, (yy * unx + xx) * (P::kRest * EA) + 2 * EA, 0, u, v, t);
      };
      hrest(ym, xm, HP.mL, HX.mL, HY.mL);
      hrest(ym, ux_, HP.m, HX.m, HY.m);
      hrest(ym, xp, HP.mR, HX.mR, HY.mR);
      hrest(uy_, xm, HP.cL, HX.cL, HY.cL);
      hrest(uy_, ux_, HP.c, HX.c, HY.c);
      hrest(uy_, xp, HP.cR, HX.cR, HY.cR);
      hrest(yp, xm, HP.nL, HX.nL, HY.nL);
      hrest(yp, ux_, HP.n, HX.n, HY.n);
      hrest(yp, xp, HP.nR, HX.nR, HY.nR);
    }
    S wh[8];
    if constexpr (NS) {
      auto one = [&](unsigned row, unsigned col, int k) {
        wh[k] = BufIO<S>::load(rsrc, row + hb + col * ES, 0);
      };
      one(rc, xm, 0);
      one(rc + 2 * nxh, xp, 2);
      one(bot ? rc + 3 * nxh : rm + nxh, ux_, 1);
      one(bot ? rc + 6 * nxh : rm + 4 * nxh, bot ? ux_ : xm, 4);
      one(bot ? rc + 7 * nxh : rm + 5 * nxh, bot ? ux_ : xp, 5);
      one(top ? rc + nxh : rp + 3 * nxh, ux_, 3);
      one(top ? rc + 4 * nxh : rp + 6 * nxh, top ? ux_ : xp, 6);
      one(top ? rc + 5 * nxh : rp + 7 * nxh, top ? ux_ : xm, 7);
    }
    if constexpr (!P::HDEV || !NS) {
      A s, t;
      PairIO<A>::load(raux, (uy_ * unx + ux_) * (P::kAux * EA), 0, s, t);
      uxp = R(s);
      uyp = R(t);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) decode(w[i], i);
    if constexpr (NS) {
#pragma unroll
      for (int k = 0; k < 8; ++k) decode_h(wh[k], k);
    }
  }

  for (int t = 0;; ++t) {
    // rebuild phi, psi, sigma of the new level from the pulled deviations
    R e[9];
    source_offsets(X, bot, top, e);
    const R ph = restream(d, e, X.c);
    source_offsets(Y, bot, top, e);
    const R ps = restream(q, e, Y.c);
    const R sg = sigma_of(p, ps);
    Two<A> rec;
    rec.a = A(ph);
    rec.b = A(ps);
    l_rest[t & 1][k0] = rec;
    l_sig[k0] = A(sg);
    // the previous level's mass flux, Eq. (16)
    R Sxp = R(0), Syp = R(0);
    if constexpr (HAS_S && NS) {
      R fx, fy;
      grad9(X, fx, fy);
      mass_flux(p, X.c, fx, fy, Sxp, Syp);
    }
    if constexpr (P::HDEV && NS) {  // rest parts of the arriving h
#pragma clang fp contract(off)
      R b[8];
      h_arrival_basis(HP, HX, HY, bot, top, b);
#pragma unroll
      for (int i = 0; i < 8; ++i) h[i] += b[i];
      const R irho = recip(p.rhoB + p.drho * (X.c - p.phiB));
      uxp = HX.c * irho;
      uyp = HY.c * irho;
    }
    if constexpr (NS) wall_terms(bot, top, rho_of(p, X.c), p.uwb, p.uwt, h);
    const R php = X.c, psp = Y.c;
    __syncthreads();
    const Nine<R> vphi = nine([&](int k) { return l_rest[t & 1][k].a; });
    const Nine<R> vsig = nine([&](int k) { return l_sig[k]; });
    R gfx, gfy, gsx, gsy;
    grad9(vphi, gfx, gfy);
    grad9(vsig, gsx, gsy);
    const R lphi = lap9(vphi);
    Front<R> s;
    if constexpr (NS)
      site_front<R, HAS_S, !P::SCALED>(p, s, ph, ps, sg, gfx, gfy, lphi, gsx, gsy, h, php, psp, uxp, uyp,
                           Sxp, Syp);
    else
      site_front_prescribed<R>(p, s, ph, ps, gfx, gfy, uxp, uyp, php, psp);
    if constexpr (GENR) {
      const Nine<R> vpsi = nine([&](int k) { return l_rest[t & 1][k].b; });
      grad9(vpsi, s.gpx, s.gpy);
    } else {
      s.gpx = s.gpy = R(0);
    }
    if constexpr (NS)
      collide_site<R, GENR, kFluxF<P, NS>, kFluxG<P, NS, GENR>>(p, s, d, q, h);
    else
      collide_fg<R, GENR, kFluxF<P, NS>, kFluxG<P, NS, GENR>>(p, s, d, q);
    if constexpr (P::HDEV && NS) {
#pragma clang fp contract(off)
      R b[8];
      h_store_basis(HRest<R>{s.P, s.jx, s.jy}, b);
#pragma unroll
      for (int i = 0; i < 8; ++i) h[i] -= b[i];
    }
    bad |= owned && !isfinite(ph + ps + s.ux + s.uy);

    // storage form
    Two<S> w[9];
    S wh[8];
    if constexpr (P::SCALED) {
      const unsigned site = uy_ * unx + ux_;
      unsigned pw[9];
      float amax = 0.f;
      pack_fg(d, q, sc.f, sc.g, site, pw, amax);
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        const unsigned short lo = (unsigned short)(pw[i] & 0xffffu), hi = (unsigned short)(pw[i] >> 16);
        w[i].a = __builtin_bit_cast(_Float16, lo);
        w[i].b = __builtin_bit_cast(_Float16, hi);
      }
      if constexpr (NS) {
        const bool odd = ux_ & 1u;
        const unsigned key = (even ? site - (ux_ & 1u) : site) * 32u + 16u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float v = h[i] * sc.h;
          amax = fmaxf(amax, fabsf(v));
          const float o = even ? pair_lane(v) : 0.f;
          const unsigned hw = halves_sr(even && odd ? o : v, even && odd ? v : o, key + unsigned(i));
          const unsigned short s16 = (unsigned short)(even && odd ? hw >> 16 : hw & 0xffffu);
          wh[i] = __builtin_bit_cast(_Float16, s16);
        }
      }
      bad |= owned && !(amax <= kHalfMax);
    } else {
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        w[i].a = S(d[i]);
        w[i].b = S(q[i]);
      }
      if constexpr (NS) {
#pragma unroll
        for (int k = 0; k < 8; ++k) wh[k] = S(h[k]);
      }
    }

    if (t == steps - 1) {  // last step: the sites of this block's interior to memory
      if (owned) {
        S *const dst = a.dst;
        const long long rowb = (long long)y * (kPlanes * nx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
          *reinterpret_cast<Two<S> *>(dst + rowb + 2LL * (i * nx + x)) = w[i];
        if constexpr (NS) {
#pragma unroll
          for (int k = 0; k < 8; ++k) dst[rowb + 18LL * nx + (long long)k * nx + x] = wh[k];
        }
        A *const r = a.dst_rest + ((long long)y * nx + x) * P::kRest;
        r[0] = A(ph);
        r[1] = A(ps);
        if constexpr (P::HDEV && NS) {
          r[2] = s.P;
          r[3] = s.jx;
          r[4] = s.jy;
        }
        if constexpr (!P::HDEV && NS) {
          A *const u = ba.aux_out + ((long long)y * nx + x) * P::kAux;
          u[0] = A(s.ux);
          u[1] = A(s.uy);
        }
      }
      break;
    }

#pragma unroll
    for (int i = 1; i < 9; ++i) l_fg[i - 1][k0] = w[i];
    if constexpr (NS) {
#pragma unroll
      for (int k = 0; k < 8; ++k) l_h[k][k0] = wh[k];
    }
    if constexpr (P::HDEV && NS) {
      l_hr[0][k0] = s.P;
      l_hr[1][k0] = s.jx;
      l_hr[2][k0] = s.jy;
    } else if constexpr (NS) {
      uxp = s.ux;
      uyp = s.uy;
    }
    decode(w[0], 0);
    __syncthreads();

    // next step: the state comes from LDS
    const int cm = ly > 0 ? -B : 0, cp = ly < B - 1 ? B : 0;
    decode(l_fg[0][k0 + dl], 1);
    decode(l_fg[2][k0 + dr], 3);
    decode(bot ? l_fg[3][k0] : l_fg[1][k0 + cm], 2);
    decode(bot ? l_fg[6][k0] : l_fg[4][k0 + cm + dl], 5);
    decode(bot ? l_fg[7][k0] : l_fg[5][k0 + cm + dr], 6);
    decode(top ? l_fg[1][k0] : l_fg[3][k0 + cp], 4);
    decode(top ? l_fg[4][k0] : l_fg[6][k0 + cp + dr], 7);
    decode(top ? l_fg[5][k0] : l_fg[7][k0 + cp + dl], 8);
    if constexpr (NS) {
      decode_h(l_h[0][k0 + dl], 0);
      decode_h(l_h[2][k0 + dr], 2);
      decode_h(bot ? l_h[3][k0] : l_h[1][k0 + cm], 1);
      decode_h(bot ? l_h[6][k0] : l_h[4][k0 + cm + dl], 4);
      decode_h(bot ? l_h[7][k0] : l_h[5][k0 + cm + dr], 5);
      decode_h(top ? l_h[1][k0] : l_h[3][k0 + cp], 3);
      decode_h(top ? l_h[4][k0] : l_h[6][k0 + cp + dr], 6);
      decode_h(top ? l_h[5][k0] : l_h[7][k0 + cp + dl], 7);
    }
    X = nine([&](int k) { return l_rest[t & 1][k].a; });
    Y = nine([&](int k) { return l_rest[t & 1][k].b; });
    if constexpr (P::HDEV && NS) {
      HP = nine([&](int k) { return l_hr[0][k]; });
      HX = nine([&](int k) { return l_hr[1][k]; });
      HY = nine([&](int k) { return l_hr[2][k]; });
    }
  }
  if (bad) *a.flag = 1;
}

// ------------------------------------------------- two steps per launch, rows

// Two-step kernel (large grids, float32 and float64 storage, Navier-Stokes
// flow): a wavefront walks down a strip of columns as lbm_step_kernel's does,
// one column per lane, and takes each row through two time steps.  The first
// step's row j goes to LDS; the second step pulls rows j-2, j-1, j of it to
// rebuild row j-1, and stores row j-2.  The populations so cross memory once
// per two steps.  A step reaches two sites in every direction: 56 of the 64
// columns are stored, and the first step walks two more rows at each end.
//
// What bounds it: vector issue for float32 (about 1450 instructions per row of
// two steps; the vector units of 2048^2 are 71% busy by the counters), where a
// step per launch is bound by memory (1.0 GB per step); for float64 latency
// too (55% busy).  Two float32 wavefronts share a SIMD (185-200 registers,
// 18 KB of LDS each), one float64 wavefront has it alone (420-450 registers,
// 4 of them spilled, 36 KB).  Two columns per lane need 430 registers for
// float32: 135 us per step on 2048^2 against 132.
// Measured per step on MI355X, lbm_step_kernel -> this: float32 1024^2
// 47.0 -> 37.0 us, 2048x1024 97.9 -> 69.1, 2048^2 196 -> 132, 4096^2
// 799 -> 485; float64 1023x769 77.4 -> 55.6, 2048^2 362 -> 229.

// LDS of one wavefront: the rows of the first step's state that the second
// still has to pull from, in rings over the rows.  Populations that stream
// up are pulled last and kept longest; one that a wall sends back is pulled
// from its own row instead.  Columns are offset by 1, so that the shifted
// reads of the edge lanes stay inside a row (their values are not used).
//
// Lanes read columns that other lanes wrote, so a row's writes must stay
// before the reads that follow them, and those before the next row's writes.
// The hardware runs a wavefront's LDS operations in order; lds_in_order()
// between them holds the compiler to it (for one lane the addresses differ,
// so nothing else does).
template <class P>
struct PairLds {
  using S = typename P::S;
  static constexpr int W = kWave + 2;
  Two<S> up[3][3][W];   // (f, g)_2, 5, 6 of rows j-2 .. j
  Two<S> mid[2][3][W];  // (f, g)_0, 1, 3 of rows j-1, j
  Two<S> dn[2][3][W];   // (f, g)_4, 7, 8 of rows j-1, j
  S hup[4][3][W];       // h_2, 5, 6 of rows j-3 .. j
  S hmid[3][2][W];      // h_1, 3 of rows j-2 .. j
  S hdn[3][3][W];       // h_4, 7, 8 of rows j-2 .. j
};

static_assert(kPairCols == kWave - 2 * kPairHalo, "a wavefront's columns");

// Orders the wavefront's LDS operations before this point before those after
// it, for the compiler alone: no instruction.
__device__ __forceinline__ void lds_in_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <class P>
struct PairArgs {
  StepArgs<P> s;
  typename P::A *aux_out;  // new previous velocity (s.aux is read by several wavefronts)
  int tiles;               // per XCD
};

// phi, psi, sigma of one site.
template <class R>
struct Scalars {
  R ph, ps, sg;
};

// Rows [y0, y1) of one strip, two steps, by one wavefront.
template <class P, bool GENR, bool HAS_S>
__device__ __forceinline__ void pair_tile(const StepArgs<P> &a, typename P::A *aux_out,
                                          const int strip, const int y0, const int y1,
                                          PairLds<P> &ls) {
  using R = typename P::R;
  using S = typename P::S;
  using A = typename P::A;
  static_assert(!P::SCALED, "float64 or float32 storage");
  const int lane = threadIdx.x & (kWave - 1);
  const int nx = a.nx, ny = a.ny, walls = a.walls;
  const int x0 = strip * kPairCols;
  const int wl = min(kPairCols, nx - x0);
  const bool interior = lane >= kPairHalo && lane < kPairHalo + wl;
  int xl = x0 - kPairHalo + min(lane, wl + 2 * kPairHalo - 1);
  xl %= nx;
  if (xl < 0) xl += nx;
  const unsigned xc = unsigned(xl);
  const unsigned xcm = xl == 0 ? unsigned(nx - 1) : xc - 1;
  const unsigned xcp = xl == nx - 1 ? 0u : xc + 1;
  constexpr unsigned ES = sizeof(S), EA = sizeof(A);
  const ColOff co = {xc * 2 * ES, xcm * 2 * ES, xcp * 2 * ES, xc * ES, xcm * ES, xcp * ES};
  const unsigned brest = xc * P::kRest * EA, baux = xc * P::kAux * EA;
  const unsigned nsites = unsigned(nx) * unsigned(ny);
  const unsigned nxb = unsigned(nx) * 2 * ES, nxh = unsigned(nx) * ES, hb = 9u * nxb;
  const unsigned rows_s = unsigned(kPlanes) * nxh;
  const unsigned rrow = unsigned(nx) * P::kRest * EA, arow = unsigned(nx) * P::kAux * EA;
  const rsrc_t rsrc = make_rsrc(a.src, unsigned(kPlanes) * nsites * ES);
  const rsrc_t rdst = make_rsrc(a.dst, unsigned(kPlanes) * nsites * ES);
  const rsrc_t rrest = make_rsrc(a.src_rest, unsigned(P::kRest) * nsites * EA);
  const rsrc_t rdrest = make_rsrc(a.dst_rest, unsigned(P::kRest) * nsites * EA);
  const rsrc_t raux = make_rsrc(a.aux, unsigned(P::kAux) * nsites * EA);
  const rsrc_t rauxo = make_rsrc(aux_out, unsigned(P::kAux) * nsites * EA);
  const Phys<R> &p = a.p;
  const Scales<P> &sc = a.sc;
  const int c = lane + 1;  // this lane's column in an LDS row

  // Row numbers run two past each end of the tile and may lie outside the
  // grid: wrapped, or clamped between walls (such rows are never used).
  auto rest_at = [&](int r, R &X, R &Y) {
    A u, v;
    PairIO<A>::load(rrest, brest, unsigned(wrap_row(r, ny, walls)) * rrow, u, v);
    X = R(u);
    Y = R(v);
  };
  auto load_fg = [&](int r, R *d, R *q) {
    Pull<P>::fg(rsrc, nxb, row_offsets(wrap_row(r, ny, walls), ny, walls, rows_s), co, sc, d, q);
  };
  auto load_row = [&](int r, R *h, R &ux, R &uy) {
    const int y = wrap_row(r, ny, walls);
    Pull<P>::h(rsrc, hb, nxh, row_offsets(y, ny, walls, rows_s), co, sc.hi, h);
    A u, v;
    PairIO<A>::load(raux, baux, unsigned(y) * arow, u, v);
    ux = R(u);
    uy = R(v);
  };
  auto at_bottom = [&](int r) { return walls && r == 0; };
  auto at_top = [&](int r) { return walls && r == ny - 1; };
  auto window = [](R m, R v, R n) { return window_k<1, 0>(&m, &v, &n); };
  // phi, psi, sigma of row r from its pulled deviations and the previous
  // level's phi (X) and psi (Y) of rows r-1, r, r+1
  auto rebuild = [&](int r, R Xm, R Xc, R Xn, R Ym, R Yc, R Yn, R *d, R *q) {
    const bool bot = at_bottom(r), top = at_top(r);
    Scalars<R> v;
    R e[9];
    source_offsets_row(window(Xm, Xc, Xn), bot, top, e);
    v.ph = restream(d, e, Xc);
    source_offsets_row(window(Ym, Yc, Yn), bot, top, e);
    v.ps = restream(q, e, Yc);
    v.sg = sigma_of(p, v.ps);
    return v;
  };
  // collision of row r, in place on d, q, h: from the level's scalars of rows
  // r-1, r, r+1 and the previous level's phi of the same rows, psi and u
  auto collide_row = [&](int r, const Scalars<R> &m, const Scalars<R> &v, const Scalars<R> &n,
                         R Xm, R Xc, R Xn, R Yc, R uxp, R uyp, R *d, R *q, R *h, R &ux, R &uy) {
    R Sxp = R(0), Syp = R(0);
    if constexpr (HAS_S) {
      R fx, fy;
      grad9(window(Xm, Xc, Xn), fx, fy);
      mass_flux(p, Xc, fx, fy, Sxp, Syp);
    }
    wall_terms(at_bottom(r), at_top(r), rho_of(p, Xc), p.uwb, p.uwt, h);
    const Nine<R> vphi = window(m.ph, v.ph, n.ph), vsig = window(m.sg, v.sg, n.sg);
    R gfx, gfy, gsx, gsy;
    grad9(vphi, gfx, gfy);
    grad9(vsig, gsx, gsy);
    const R lphi = lap9(vphi);
    Front<R> s;
    site_front<R, HAS_S, true>(p, s, v.ph, v.ps, v.sg, gfx, gfy, lphi, gsx, gsy, h, Xc, Yc, uxp,
                               uyp, Sxp, Syp);
    if constexpr (GENR) {
      grad9(window(m.ps, v.ps, n.ps), s.gpx, s.gpy);
    } else {
      s.gpx = s.gpy = R(0);
    }
    collide_site<R, GENR, kFluxF<P, true>, kFluxG<P, true, GENR>>(p, s, d, q, h);
    ux = s.ux;
    uy = s.uy;
  };

  // Memory: X, Y are phi, psi of rows j-1 .. j+2; dn, qn the raw deviations
  // of row j+1; hr, uxr, uyr h and u of row j.
  R X0, X1, X2, X3, Y0, Y1, Y2, Y3;
  R dc[9], qc[9], dn[9], qn[9], hr[8], uxr, uyr;
  // First step's level: scalars of rows j-1 (m), j (v) and deviations of row
  // j; after its collision phi, psi, u of rows j-1, j-2 and phi of row j-3,
  // the previous level of the second step.
  Scalars<R> m1, v1;
  R f1 = R(0), f2 = R(0), f3 = R(0), s1 = R(0), s2 = R(0);
  R ux1 = R(0), uy1 = R(0), ux2 = R(0), uy2 = R(0);
  // Second step's level: scalars of rows j-3 (m), j-2 (v), deviations of j-2.
  Scalars<R> m2 = {R(0), R(0), R(0)}, v2 = {R(0), R(0), R(0)};
  R dd[9] = {}, qd[9] = {};
  const int j0 = y0 - 2;
  {
    R dt[9], qt[9], Xa, Ya;
    rest_at(j0 - 1, X0, Y0);
    rest_at(j0, X1, Y1);
    rest_at(j0 + 1, X2, Y2);
    rest_at(j0 + 2, X3, Y3);
    load_fg(j0, dc, qc);
    rest_at(j0 - 2, Xa, Ya);
    load_fg(j0 - 1, dt, qt);
    load_fg(j0 + 1, dn, qn);
    load_row(j0, hr, uxr, uyr);
    v1 = rebuild(j0, X0, X1, X2, Y0, Y1, Y2, dc, qc);
    m1 = rebuild(j0 - 1, Xa, X0, X1, Ya, Y0, Y1, dt, qt);
  }
  // halo lanes' stores are dropped by the hardware, as in step_tile
  const unsigned cs_p = interior ? co.p0 : kDropped, cs_h = interior ? co.h0 : kDropped;
  const unsigned brest_s = interior ? brest : kDropped, baux_s = interior ? baux : kDropped;
  bool bad = false;
  int r3 = 0, r2 = 0, r4 = 0;  // ring slots of row j

  // Row j of the first step; then of the second, row j-1 rebuilt (if second)
  // and row j-2 collided and stored (if STORE).
  auto row = [&](int j, auto store, bool second) {
    constexpr bool STORE = decltype(store)::value;
    const int r3b = r3 == 0 ? 2 : r3 - 1, r3c = r3b == 0 ? 2 : r3b - 1;  // rows j-1, j-2
    const int r2b = r2 ^ 1, r4b = (r4 + 2) & 3, r4c = (r4 + 1) & 3;      // j-1; j-2, j-3
    Scalars<R> n1 = rebuild(j + 1, X1, X2, X3, Y1, Y2, Y3, dn, qn);
    R h[8], dk[9], qk[9], X4, Y4;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = hr[i];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      dk[i] = dn[i];
      qk[i] = qn[i];
    }
    const R uxp = uxr, uyp = uyr;
    rest_at(j + 3, X4, Y4);
    load_fg(j + 2, dn, qn);
    load_row(j + 1, hr, uxr, uyr);
    // at a wall the stencils' row beyond it is the wall row itself
    if (at_bottom(j)) m1 = v1;
    if (at_top(j)) n1 = v1;
    R ux, uy;
    collide_row(j, m1, v1, n1, X0, X1, X2, Y1, uxp, uyp, dc, qc, h, ux, uy);
    bad |= interior && j >= y0 && j < y1 && !isfinite(v1.ph + v1.ps + ux + uy);
    auto w = [&](int i) { return Two<S>{S(dc[i]), S(qc[i])}; };
    lds_in_order();  // after the last row's reads
    ls.up[r3][0][c] = w(2);
    ls.up[r3][1][c] = w(5);
    ls.up[r3][2][c] = w(6);
    ls.mid[r2][0][c] = w(0);
    ls.mid[r2][1][c] = w(1);
    ls.mid[r2][2][c] = w(3);
    ls.dn[r2][0][c] = w(4);
    ls.dn[r2][1][c] = w(7);
    ls.dn[r2][2][c] = w(8);
    ls.hup[r4][0][c] = S(h[1]);
    ls.hup[r4][1][c] = S(h[4]);
    ls.hup[r4][2][c] = S(h[5]);
    ls.hmid[r3][0][c] = S(h[0]);
    ls.hmid[r3][1][c] = S(h[2]);
    ls.hdn[r3][0][c] = S(h[3]);
    ls.hdn[r3][1][c] = S(h[6]);
    ls.hdn[r3][2][c] = S(h[7]);
    lds_in_order();  // before this row's reads

    Scalars<R> n2 = {R(0), R(0), R(0)};
    R de[9], qe[9];
    if (second) {
      const bool bot = at_bottom(j - 1), top = at_top(j - 1);
      auto get = [&](const Two<S> *row, int i) {
        const Two<S> t = row[c];
        de[i] = R(t.a);
        qe[i] = R(t.b);
      };
      get(ls.mid[r2b][0], 0);
      get(ls.mid[r2b][1] - 1, 1);
      get(ls.mid[r2b][2] + 1, 3);
      get(bot ? ls.dn[r2b][0] : ls.up[r3c][0], 2);
      get(bot ? ls.dn[r2b][1] : ls.up[r3c][1] - 1, 5);
      get(bot ? ls.dn[r2b][2] : ls.up[r3c][2] + 1, 6);
      get(top ? ls.up[r3b][0] : ls.dn[r2][0], 4);
      get(top ? ls.up[r3b][1] : ls.dn[r2][1] + 1, 7);
      get(top ? ls.up[r3b][2] : ls.dn[r2][2] - 1, 8);
      n2 = rebuild(j - 1, f2, f1, v1.ph, s2, s1, v1.ps, de, qe);
    }
    if constexpr (STORE) {
      const int y = j - 2;
      const bool bot = at_bottom(y), top = at_top(y);
      R g[8];
      auto get = [&](const S *row, int k) { g[k] = R(row[c]); };
      get(ls.hmid[r3c][0] - 1, 0);
      get(ls.hmid[r3c][1] + 1, 2);
      get(bot ? ls.hdn[r3c][0] : ls.hup[r4c][0], 1);
      get(bot ? ls.hdn[r3c][1] : ls.hup[r4c][1] - 1, 4);
      get(bot ? ls.hdn[r3c][2] : ls.hup[r4c][2] + 1, 5);
      get(top ? ls.hup[r4b][0] : ls.hdn[r3b][0], 3);
      get(top ? ls.hup[r4b][1] : ls.hdn[r3b][1] + 1, 6);
      get(top ? ls.hup[r4b][2] : ls.hdn[r3b][2] - 1, 7);
      if (bot) {
        m2 = v2;
        f3 = f2;
      }
      Scalars<R> nn = n2;
      R fn = f1;
      if (top) {
        nn = v2;
        fn = f2;
      }
      R ox, oy;
      collide_row(y, m2, v2, nn, f3, f2, fn, s2, ux2, uy2, dd, qd, g, ox, oy);
      bad |= interior && !isfinite(v2.ph + v2.ps + ox + oy);
      const unsigned rcs = unsigned(y) * rows_s;
#pragma unroll
      for (int i = 0; i < 9; ++i)
        PairIO<S>::template store<P::kStorePol>(S(dd[i]), S(qd[i]), rdst, cs_p,
                                                rcs + unsigned(i) * nxb);
#pragma unroll
      for (int i = 0; i < 8; ++i) bst<P>(g[i], rdst, cs_h, rcs + hb + unsigned(i) * nxh);
      PairIO<A>::template store<P::kStorePol>(A(v2.ph), A(v2.ps), rdrest, brest_s,
                                              unsigned(y) * rrow);
      PairIO<A>::template store<P::kStorePol>(A(ox), A(oy), rauxo, baux_s, unsigned(y) * arow);
    }

    // slide the windows
    if (second) {
      m2 = v2;
      v2 = n2;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        dd[i] = de[i];
        qd[i] = qe[i];
      }
    }
    f3 = f2;
    f2 = f1;
    f1 = v1.ph;
    s2 = s1;
    s1 = v1.ps;
    ux2 = ux1;
    uy2 = uy1;
    ux1 = ux;
    uy1 = uy;
    m1 = v1;
    v1 = n1;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      dc[i] = dk[i];
      qc[i] = qk[i];
    }
    X0 = X1;
    X1 = X2;
    X2 = X3;
    X3 = X4;
    Y0 = Y1;
    Y1 = Y2;
    Y2 = Y3;
    Y3 = Y4;
    r3 = r3 == 2 ? 0 : r3 + 1;
    r2 ^= 1;
    r4 = (r4 + 1) & 3;
  };

  // The waits leave nothing of one loop in flight at the head of the next
  // (see step_tile); the first four rows feed the second step only.
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  int j = j0;
  for (int i = 0; i < 4; ++i, ++j) row(opaque_row(j), BoolC<false>{}, i >= 2);
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  for (int i = y0; i < y1; ++i, ++j) row(opaque_row(j), BoolC<true>{}, true);
  if (bad) *a.flag = 1;
}

// One wavefront per tile (pair_tile_of).
template <class P, bool GENR, bool HAS_S>
__global__ void __launch_bounds__(kWave)
lbm_pair_kernel(const PairArgs<P> pa) {
  __shared__ PairLds<P> ls;
  const StepArgs<P> &a = pa.s;
  const PairTile t = pair_tile_of(int(blockIdx.x % kXcds), int(blockIdx.x / kXcds), a.ny, pa.tiles,
                                  a.nstrips);
  if (t.y0 < t.y1) pair_tile<P, GENR, HAS_S>(a, pa.aux_out, t.strip, t.y0, t.y1, ls);
}

// ------------------------------------------------------------ batched step

// A tile of the batched step: which simulation, which strip and row chunk.
struct TileRef {
  int inst, strip, chunk, pad;
};

// Per simulation of a batch: the step arguments for both ping-pong
// parities, the parity at the start of the captured chunk, and how many of
// the chunk's launches it takes part in.
template <class P>
struct BatchInst {
  StepArgs<P> a[2];
  int parity, steps, pad[2];
};

// Constant address space: loads through it with a wavefront-uniform address
// become scalar loads.  The qualifier exists only in the device pass.
#if defined(__HIP_DEVICE_COMPILE__)
#define LBM_CONST __attribute__((address_space(4)))
#else
#define LBM_CONST
#endif

// Launch k of a captured chunk for every simulation of one kernel variant.
// Persistent: gridDim.x * P::kBlockWaves wavefronts walk the tile list with a fixed
// stride; the tile count and the per-simulation descriptors are read from
// device memory (scalar loads), so a captured graph stays valid when the
// batch's membership changes between chunks.  Every wavefront leaves the
// loop after at most ceil(ntiles / stride) tiles.
template <class P, int K, bool GENR, bool HAS_S, bool NS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P::kMinWaves)))
lbm_batch_step_kernel(const BatchInst<P> *insts, const TileRef *tiles, const int *ntiles,
                      int k) {
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int nt = *(const LBM_CONST int *)(ntiles);
  const int stride = int(gridDim.x) * P::kBlockWaves;
  for (int t = int(blockIdx.x) * P::kBlockWaves + wave; t < nt; t += stride) {
    const TileRef tr = ((const LBM_CONST TileRef *)(tiles))[t];
    const LBM_CONST BatchInst<P> *bi =
        (const LBM_CONST BatchInst<P> *)(insts) + tr.inst;
    if (k >= bi->steps) continue;
    const StepArgs<P> a = bi->a[(bi->parity + k) & 1];
    const int y0 = tr.chunk * a.rows;
    step_tile<P, K, GENR, HAS_S, NS>(a, tr.strip, y0, min(y0 + a.rows, a.ny));
  }
}

// ------------------------------------------------------------ site kernels

// Neighbour of site (x, y) at offset (dx, dy) in {-1,0,1}^2: periodic in x;
// periodic in y or, between walls, the wall row itself (mirror ghost).
__device__ __forceinline__ void nbr_xy(int x, int y, int dx, int dy, int nx, int ny,
                                       int walls, int &xx, int &yy) {
  xx = x + dx;
  yy = y + dy;
  xx = xx < 0 ? xx + nx : (xx >= nx ? xx - nx : xx);
  if (walls) {
    yy = yy < 0 ? 0 : (yy >= ny ? ny - 1 : yy);
  } else {
    yy = yy < 0 ? yy + ny : (yy >= ny ? yy - ny : yy);
  }
}

// The 9-point neighbourhood of site (x, y) of a field given by an index
// function idx(y, x).
template <class R, class F>
__device__ __forceinline__ Nine<R> gather9(F get, int x, int y, int nx, int ny, int walls) {
  auto v9 = [&](int dx, int dy) {
    int xx, yy;
    nbr_xy(x, y, dx, dy, nx, ny, walls, xx, yy);
    return R(get(yy, xx));
  };
  Nine<R> v;
  v.mL = v9(-1, -1);
  v.m = v9(0, -1);
  v.mR = v9(1, -1);
  v.cL = v9(-1, 0);
  v.c = v9(0, 0);
  v.cR = v9(1, 0);
  v.nL = v9(-1, 1);
  v.n = v9(0, 1);
  v.nR = v9(1, 1);
  return v;
}

template <class P>
struct SiteArgs {
  const typename P::S *src;
  const typename P::A *src_rest;
  typename P::S *dst;
  typename P::A *dst_rest;
  typename P::A *aux;
  double *scratch;  // kScratch float64 planes
  Scales<P> sc;
  long long plane;
  int nx, ny, walls;
  int ns;  // 1: velocity from the Navier-Stokes LB; 0: prescribed (aux slots 0, 1)
};

// Initial state in float64: post-collision populations := equilibria of
// Eqs. (22), (26), (30) with P = 0 and S of Eq. (16) from the gradient of
// the initial phi; previous level := the initial fields.  Inputs are
// scratch planes 0-3 (phi, psi, ux, uy).  f and g are stored as deviations
// from w_i times the STORED rest value, so storing phi, psi in a narrower
// type leaves the populations themselves exact up to their own rounding.
template <class P>
__global__ void __launch_bounds__(256)
lbm_init_kernel(const SiteArgs<P> a, const Phys<double> p) {
  using A = typename P::A;
  using R = typename P::R;
  const long long n = (long long)a.nx * a.ny;
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int nx = a.nx;
  const int x = int(k % nx), y = int(k / nx);
  const long long pl = a.plane;
  const double *phi0 = a.scratch, *psi0 = a.scratch + pl;
  const double *ux0 = a.scratch + 2 * pl, *uy0 = a.scratch + 3 * pl;
  const Nine<double> v = gather9<double>(
      [&](int yy, int xx) { return phi0[(long long)yy * nx + xx]; }, x, y, nx, a.ny, a.walls);
  double gx, gy;
  grad9(v, gx, gy);
  const double phi = phi0[k], psi = psi0[k], ux = ux0[k], uy = uy0[k];
  const double gn = sqrt(gx * gx + gy * gy);
  const double inv = 1.0 / (gn + p.eps_n);
  const double delta = p.c4W * ((p.phiA - phi) * (phi - p.phiB));
  const double Sx = p.Mdrho * (gx - delta * gx * inv);
  const double Sy = p.Mdrho * (gy - delta * gy * inv);
  const double rho = rho_of(p, phi);
  const double jx = rho * ux, jy = rho * uy;
  const double Ax = jx - Sx, Ay = jy - Sy, Au = Ax * ux + Ay * uy;
  const int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  const int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  const double w[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                       1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
  const double phis = double(A(phi)), psis = double(A(psi));
  // float16 storage: h relative to the rest parts of the STORED (P = 0, rho u)
  R hbase[8] = {};
  if constexpr (P::HDEV) {
    const HRest<R> v = {R(0), R(A(jx)), R(A(jy))};
    h_store_basis(v, hbase);
  }
  for (int i = 0; i < 9; ++i) {
    const double cu = cx[i] * ux + cy[i] * uy;
    st<P>(a.dst, fg_idx(i, 0, y, x, nx), R(w[i] * (phi - phis) + w[i] * phi * 3.0 * cu),
          a.sc.f);
    st<P>(a.dst, fg_idx(i, 1, y, x, nx), R(w[i] * (psi - psis) + w[i] * psi * 3.0 * cu),
          a.sc.g);
    if (i > 0) {
      const double cj = cx[i] * jx + cy[i] * jy;
      const double cA = cx[i] * Ax + cy[i] * Ay;
      st<P>(a.dst, h_idx(i, y, x, nx),
            R(w[i] * (3.0 * cj + 4.5 * cA * cu - 1.5 * Au) - double(hbase[i - 1])), a.sc.h);
    }
  }
  a.dst_rest[rest_idx<P>(0, y, x, nx)] = A(phi);
  a.dst_rest[rest_idx<P>(1, y, x, nx)] = A(psi);
  if (!a.ns) {  // prescribed velocity, held in aux slots 0, 1 for good
    a.aux[aux_idx<P>(0, y, x, nx)] = A(ux);
    a.aux[aux_idx<P>(1, y, x, nx)] = A(uy);
    return;
  }
  if constexpr (P::HDEV) {
    a.dst_rest[rest_idx<P>(2, y, x, nx)] = A(0);
    a.dst_rest[rest_idx<P>(3, y, x, nx)] = A(jx);
    a.dst_rest[rest_idx<P>(4, y, x, nx)] = A(jy);
  } else {
    a.aux[aux_idx<P>(0, y, x, nx)] = A(ux);
    a.aux[aux_idx<P>(1, y, x, nx)] = A(uy);
  }
}

// Read-back, pass 1: phi, psi, sigma of the current level into scratch
// planes 5-7 (arithmetic type R), by the same streaming as the step.
template <class P>
__global__ void __launch_bounds__(256)
lbm_macro_scalars_kernel(const SiteArgs<P> a, const Phys<typename P::R> p) {
  using R = typename P::R;
  const long long n = (long long)a.nx * a.ny;
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int nx = a.nx;
  const int x = int(k % nx), y = int(k / nx);
  const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const long long pl = a.plane;
  const RowN r = row_numbers(y, a.ny, a.walls);
  R d[9], q[9], e[9];
  pull_fg<P>(a.src, r, x, xm, xp, nx, a.sc.fi, a.sc.gi, d, q);
  const auto *rs = a.src_rest;
  const Nine<R> vx = gather9<R>([&](int yy, int xx) { return rs[rest_idx<P>(0, yy, xx, nx)]; },
                                x, y, nx, a.ny, a.walls);
  source_offsets(vx, r.bot, r.top, e);
  const R phi = restream(d, e, vx.c);
  const Nine<R> vy = gather9<R>([&](int yy, int xx) { return rs[rest_idx<P>(1, yy, xx, nx)]; },
                                x, y, nx, a.ny, a.walls);
  source_offsets(vy, r.bot, r.top, e);
  const R psi = restream(q, e, vy.c);
  R *out = reinterpret_cast<R *>(a.scratch + 5 * pl);
  out[k] = phi;
  out[pl + k] = psi;
  out[2 * pl + k] = sigma_of(p, psi);
}

// Read-back, pass 2: u and P by the same closures as the step, float64
// phi, psi, ux, uy, P into scratch planes 0-4.
template <class P, bool HAS_S>
__global__ void __launch_bounds__(256)
lbm_macro_fields_kernel(const SiteArgs<P> a, const Phys<typename P::R> p) {
  using R = typename P::R;
  const long long n = (long long)a.nx * a.ny;
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int nx = a.nx;
  const int x = int(k % nx), y = int(k / nx);
  const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const long long pl = a.plane;
  const R *sc = reinterpret_cast<const R *>(a.scratch + 5 * pl);
  const Nine<R> vphi = gather9<R>([&](int yy, int xx) { return sc[(long long)yy * nx + xx]; },
                                  x, y, nx, a.ny, a.walls);
  const R *ss = sc + 2 * pl;
  const Nine<R> vsig = gather9<R>([&](int yy, int xx) { return ss[(long long)yy * nx + xx]; },
                                  x, y, nx, a.ny, a.walls);
  R gfx, gfy, gsx, gsy;
  grad9(vphi, gfx, gfy);
  grad9(vsig, gsx, gsy);
  const R lphi = lap9(vphi);
  const R php = R(a.src_rest[rest_idx<P>(0, y, x, nx)]);
  const R psp = R(a.src_rest[rest_idx<P>(1, y, x, nx)]);
  if (!a.ns) {  // prescribed velocity: u as given, P = 0
    a.scratch[k] = double(vphi.c);
    a.scratch[pl + k] = double(sc[pl + k]);
    a.scratch[2 * pl + k] = double(a.aux[aux_idx<P>(0, y, x, nx)]);
    a.scratch[3 * pl + k] = double(a.aux[aux_idx<P>(1, y, x, nx)]);
    a.scratch[4 * pl + k] = 0.0;
    return;
  }
  // the previous level's mass flux from the previous phi, as in the step
  R Sxp = R(0), Syp = R(0);
  if constexpr (HAS_S) {
    const auto *rs = a.src_rest;
    const Nine<R> vq = gather9<R>(
        [&](int yy, int xx) { return R(rs[rest_idx<P>(0, yy, xx, nx)]); }, x, y, nx, a.ny,
        a.walls);
    R gqx, gqy;
    grad9(vq, gqx, gqy);
    mass_flux(p, php, gqx, gqy, Sxp, Syp);
  }
  const RowN r = row_numbers(y, a.ny, a.walls);
  R h[8];
  pull_h<P>(a.src, r, x, xm, xp, nx, a.sc.hi, rho_of(p, php), p.uwb, p.uwt, h);
  R uxp, uyp;
  if constexpr (P::HDEV) {
    const auto *rs = a.src_rest;
    auto g = [&](int c) {
      return gather9<R>([&](int yy, int xx) { return rs[rest_idx<P>(c, yy, xx, nx)]; }, x, y,
                        nx, a.ny, a.walls);
    };
    const Nine<R> vP = g(2), vjx = g(3), vjy = g(4);
    R b[8];
    h_arrival_basis(vP, vjx, vjy, r.bot, r.top, b);
    for (int i = 0; i < 8; ++i) h[i] += b[i];
    const R irho = R(1) / rho_of(p, php);
    uxp = vjx.c * irho;
    uyp = vjy.c * irho;
  } else {
    uxp = R(a.aux[aux_idx<P>(0, y, x, nx)]);
    uyp = R(a.aux[aux_idx<P>(1, y, x, nx)]);
  }
  Front<R> s;
  site_front<R, HAS_S, !P::SCALED>(p, s, vphi.c, sc[pl + k], vsig.c, gfx, gfy, lphi, gsx, gsy, h, php,
                       psp, uxp, uyp, Sxp, Syp);
  a.scratch[k] = double(s.phi);
  a.scratch[pl + k] = double(s.psi);
  a.scratch[2 * pl + k] = double(s.ux);
  a.scratch[3 * pl + k] = double(s.uy);
  a.scratch[4 * pl + k] = double(s.P);
}

// Float64 reductions over scratch planes 0-3 (phi, psi, ux, uy): per-block
// partial sums in a fixed order (wavefront shuffles, then LDS), then one
// block adds the partials in a fixed order.  Deterministic.
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_down(v, o, kWave);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_down(v, o, kWave));
  return v;
}

__global__ void __launch_bounds__(256)
lbm_reduce_kernel(const double *scratch, long long plane, long long n,
                  const Phys<double> p, double *partials) {
  double acc[kReduceVals] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (long long)gridDim.x * blockDim.x) {
    const double phi = scratch[k], psi = scratch[plane + k];
    const double ux = scratch[2 * plane + k], uy = scratch[3 * plane + k];
    const double rho = rho_of(p, phi);
    const double u2 = ux * ux + uy * uy;
    acc[0] += phi;
    acc[1] += psi;
    acc[2] += rho * ux;
    acc[3] += rho * uy;
    acc[4] += 0.5 * rho * u2;
    acc[5] = fmax(acc[5], sqrt(u2));
    if (!isfinite(phi + psi + ux + uy)) acc[6] = 1.0;
  }
  __shared__ double lds[kReduceVals][256 / kWave];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  for (int j = 0; j < 7; ++j) {
    const double v = (j == 5 || j == 6) ? wave_max(acc[j]) : wave_sum(acc[j]);
    if (lane == 0) lds[j][wv] = v;
  }
  __syncthreads();
  if (threadIdx.x < 7) {
    const int j = threadIdx.x;
    double v = lds[j][0];
    for (int q = 1; q < 256 / kWave; ++q)
      v = (j == 5 || j == 6) ? fmax(v, lds[j][q]) : v + lds[j][q];
    partials[blockIdx.x * kReduceVals + j] = v;
  }
}

// Adds the blocks' partials in block order (maxima for the values of MAXES),
// deterministically, and appends *flag (if given) as a double.  One dependent
// chain of at most kReduceBlocks additions per value: what bounds it is how
// soon the next operand is there, so all partials are first brought into LDS
// by the whole workgroup (walking them from memory, one round trip per few
// additions, took 168 us for 1024 blocks; this takes 16 us, 4 us for 128).  The sums and
// the maxima are walked by different wavefronts.
constexpr int kFinalThreads = 256;
template <int NV, int STRIDE, unsigned MAXES>
__global__ void __launch_bounds__(kFinalThreads)
lbm_final_kernel(const double *partials, int nblocks, const int *flag, double *out) {
  __shared__ double col[NV][kReduceBlocks + 2];  // padded: columns start in different banks
#pragma unroll 8
  for (int i = int(threadIdx.x); i < nblocks * STRIDE; i += kFinalThreads) {
    const double v = partials[i];
    if (i % STRIDE < NV) col[i % STRIDE][i / STRIDE] = v;
  }
  __syncthreads();
  const int j = int(threadIdx.x) & (kWave - 1), wv = int(threadIdx.x) / kWave;
  if (j >= NV || wv > 1 || (wv == 1) != bool(MAXES >> j & 1u)) return;
  auto walk = [&](auto add) {
    constexpr int U = 32;  // operands on their way while the last ones are added
    double v = col[j][0], q[U];
    int b = 1;
    if (b + U <= nblocks) {
#pragma unroll
      for (int k = 0; k < U; ++k) q[k] = col[j][b + k];
      for (b += U; b + U <= nblocks; b += U) {
        double r[U];
#pragma unroll
        for (int k = 0; k < U; ++k) r[k] = col[j][b + k];
#pragma unroll
        for (int k = 0; k < U; ++k) {
          v = add(v, q[k]);
          q[k] = r[k];
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) v = add(v, q[k]);
    }
    for (; b < nblocks; ++b) v = add(v, col[j][b]);
    return v;
  };
  out[j] = wv == 0 ? walk([](double x, double y) { return x + y; })
                   : walk([](double x, double y) { return fmax(x, y); });
  if (flag && j == 0) out[NV] = double(*flag);
}

// Blocks of a reduction over n sites: those beyond the sites would add zeros.
int reduce_blocks(long long n) {
  return int(std::min<long long>(kReduceBlocks, (n + 255) / 256));
}

// Shape diagnostics of fluid A from the float64 phi of scratch plane 0:
// c = (phi - phiB)/(phiA - phiB).  Pass 1 sums c, c cos/sin of the periodic
// angles of x and y, c y, and |grad phi|; pass 2 sums c dx^2, c dx dy,
// c dy^2 about the centroid (minimum image along periodic directions).
// Per-block partials in a fixed order, as in lbm_reduce_kernel.
constexpr int kShapeVals = 7;
template <int PASS>
__global__ void __launch_bounds__(256)
lbm_shape_kernel(const double *phi, int nx, int ny, int walls, double phiA, double phiB,
                 double cx, double cy, double *partials) {
  double acc[kShapeVals] = {0, 0, 0, 0, 0, 0, 0};
  const long long n = (long long)nx * ny;
  const double inv = 1.0 / (phiA - phiB);
  const double tx = 2.0 * M_PI / nx, ty = 2.0 * M_PI / ny;
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (long long)gridDim.x * blockDim.x) {
    const int x = int(k % nx), y = int(k / nx);
    const double c = (phi[k] - phiB) * inv;
    if (PASS == 1) {
      const Nine<double> v = gather9<double>(
          [&](int yy, int xx) { return phi[(long long)yy * nx + xx]; }, x, y, nx, ny, walls);
      double gx, gy;
      grad9(v, gx, gy);
      acc[0] += c;
      acc[1] += c * cos(tx * x);
      acc[2] += c * sin(tx * x);
      acc[3] += c * cos(ty * y);
      acc[4] += c * sin(ty * y);
      acc[5] += c * y;
      acc[6] += sqrt(gx * gx + gy * gy);
    } else {
      double dx = x - cx;
      dx -= nx * rint(dx / nx);
      double dy = y - cy;
      if (!walls) dy -= ny * rint(dy / ny);
      acc[0] += c * dx * dx;
      acc[1] += c * dx * dy;
      acc[2] += c * dy * dy;
    }
  }
  __shared__ double lds[kShapeVals][256 / kWave];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  for (int j = 0; j < kShapeVals; ++j) {
    const double v = wave_sum(acc[j]);
    if (lane == 0) lds[j][wv] = v;
  }
  __syncthreads();
  if (threadIdx.x < kShapeVals) {
    const int j = threadIdx.x;
    double v = lds[j][0];
    for (int q = 1; q < 256 / kWave; ++q) v += lds[j][q];
    partials[blockIdx.x * kShapeVals + j] = v;
  }
}

// ------------------------------------------------------------------ host

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

size_t storage_size(int prec) {
  return prec == LBM_FP64 ? 8 : (prec == LBM_FP32 ? 4 : 2);
}
size_t field_size(int prec) { return prec == LBM_FP64 ? 8 : 4; }
// fields per site of the rest record (ping-pong) and the aux record
int rest_fields(int prec) { return prec == LBM_FP16DEV ? F16::kRest : F32::kRest; }
int aux_fields(int prec) { return prec == LBM_FP16DEV ? F16::kAux : F32::kAux; }

struct Layout {
  long long plane;  // elements per plane
  size_t pop_bytes, rest_bytes, aux_bytes, scratch_bytes, partial_bytes;
  size_t off_pop[2], off_rest[2], off_aux, off_scratch, off_partial, off_flag, total;
};

Layout make_layout(const lbm_params &p) {
  Layout L;
  const long long n = (long long)p.nx * p.ny;
  L.plane = (long long)align_up((size_t)n, 64);
  L.pop_bytes = align_up((size_t)kPlanes * n * storage_size(p.precision), 256);
  L.rest_bytes = align_up((size_t)rest_fields(p.precision) * n * field_size(p.precision), 256);
  L.aux_bytes = align_up((size_t)aux_fields(p.precision) * n * field_size(p.precision), 256);
  L.scratch_bytes = align_up((size_t)kScratch * L.plane * 8, 256);
  L.partial_bytes = align_up((size_t)(kReduceBlocks + 1) * kReduceVals * 8, 256);
  size_t o = 0;
  for (int c = 0; c < 2; ++c) {
    L.off_pop[c] = o;
    o += L.pop_bytes;
    L.off_rest[c] = o;
    o += L.rest_bytes;
  }
  L.off_aux = o;
  o += L.aux_bytes;
  L.off_scratch = o;
  o += L.scratch_bytes;
  L.off_partial = o;
  o += L.partial_bytes;
  L.off_flag = o;
  o += 256;
  L.total = o;
  return L;
}

std::string g_create_error;

const char *validate(const lbm_params *p) {
  if (!p) return "params is NULL";
  if (p->nx < 3 || p->ny < 3) return "nx and ny must be >= 3";
  if ((long long)p->nx * p->ny > (1LL << 31)) return "grid too large";
  if (p->walls_y != 0 && p->walls_y != 1) return "walls_y must be 0 or 1";
  if (p->eos != LBM_EOS_LINEAR && p->eos != LBM_EOS_LANGMUIR) return "unknown eos";
  if (p->precision != LBM_FP64 && p->precision != LBM_FP32 && p->precision != LBM_FP16DEV)
    return "unknown precision";
  if (p->flow != LBM_FLOW_NS && p->flow != LBM_FLOW_PRESCRIBED) return "unknown flow";
  {
    // the step kernel addresses each population copy through one buffer
    // resource with 32-bit byte offsets, and its halo lanes store at
    // kDropped, which must lie past every resource
    const unsigned long long sites = (unsigned long long)p->nx * p->ny;
    if (kPlanes * sites * storage_size(p->precision) > kDropped)
      return "grid too large: 26 population planes must fit in 4 GiB";
    if (rest_fields(p->precision) * sites * field_size(p->precision) > kDropped)
      return "grid too large: the rest records must fit in 4 GiB";
  }
  if (!(p->phiA > p->phiB)) return "phiA must exceed phiB";
  if (!(p->W > 0)) return "W must be > 0";
  if (!(p->M > 0) || !(p->D > 0)) return "M and D must be > 0 (tau > 1/2)";
  if (!(p->rhoA > 0) || !(p->rhoB > 0)) return "densities must be > 0";
  if (!(p->muA > 0) || !(p->muB > 0)) return "viscosities must be > 0";
  if (!(p->r >= 0)) return "r must be >= 0";
  if (!(p->sigma0 >= 0)) return "sigma0 must be >= 0";
  const double fin[] = {p->u_wall_bot, p->u_wall_top, p->beta, p->gx, p->gy};
  for (double v : fin)
    if (!std::isfinite(v)) return "non-finite parameter";
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      if (!(p->s_free[a][b] > 0 && p->s_free[a][b] < 2)) return "free rates must lie in (0, 2)";
  for (int a = 0; a < 3; ++a) {
    const double s = p->fp16_scale[a];
    if (s == 0) continue;
    int e;
    if (!(s > 0) || std::frexp(s, &e) != 0.5 || e < -29 || e > 31)  // s = 2^(e-1)
      return "fp16_scale entries must be 0 or powers of two in [2^-30, 2^30]";
  }
  return nullptr;
}

template <class R>
Phys<R> make_phys(const lbm_params &q) {
  Phys<R> p;
  const double dphi = q.phiA - q.phiB;
  const double drho = (q.rhoA - q.rhoB) / dphi;
  p.phiA = R(q.phiA);
  p.phiB = R(q.phiB);
  p.phiAB = R(q.phiA + q.phiB);
  p.c4W = R(4.0 / (q.W * dphi));
  p.cbulk = R(24.0 / (q.W * dphi * dphi * dphi * dphi));
  p.cW = R(1.5 * q.W / (dphi * dphi));
  p.rhoB = R(q.rhoB);
  p.drho = R(drho);
  p.muB = R(q.muB);
  p.dmu = R((q.muA - q.muB) / dphi);
  p.Mdrho = R(q.M * drho);
  p.gx = R(q.gx);
  p.gy = R(q.gy);
  p.sigma0 = R(q.sigma0);
  p.beta = R(q.beta);
  p.r = R(q.r);
  p.rm1 = R(q.r - 1.0);
  p.s1f = R(1.0 / (3.0 * q.M + 0.5));
  p.s2f = R(q.s_free[0][0]);
  p.s3f = R(q.s_free[0][1]);
  p.s4f = R(q.s_free[0][2]);
  p.s1g = R(1.0 / (3.0 * q.D + 0.5));
  p.s2g = R(q.s_free[1][0]);
  p.s3g = R(q.s_free[1][1]);
  p.s4g = R(q.s_free[1][2]);
  p.s3h = R(q.s_free[2][1]);
  p.s4h = R(q.s_free[2][2]);
  p.uwb = R(q.u_wall_bot);
  p.uwt = R(q.u_wall_top);
  p.psi_max = R(1.0 - 1e-9);
  // 1e-4 of the largest gradient of the equilibrium profile: inside drops,
  // where |grad phi| can fall below delta(phi), the sharpening flux must not
  // become anti-diffusive (it would amplify rounding differences)
  p.eps_n = R(1e-4 * dphi / q.W);
  p.eos = q.eos;
  return p;
}

// Default float16 scales: deviations of f and g are at most a few 1e-2 of
// their field, h_i are O(w_i (3P + 3 c.rho u)); the scales put the expected
// magnitudes near 2^4..2^8, well inside float16's normal range.
void fp16_scales(const lbm_params &q, double out[3]) {
  const double dflt[3] = {4096.0, 4096.0, 65536.0};
  for (int a = 0; a < 3; ++a) out[a] = q.fp16_scale[a] > 0 ? q.fp16_scale[a] : dflt[a];
}

template <class P>
Scales<P> make_scales(const lbm_params &q) {
  using R = typename P::R;
  Scales<P> s;
  double v[3] = {1.0, 1.0, 1.0};
  if (P::SCALED) fp16_scales(q, v);
  s.f = R(v[0]);
  s.g = R(v[1]);
  s.h = R(v[2]);
  s.fi = R(1.0 / v[0]);
  s.gi = R(1.0 / v[1]);
  s.hi = R(1.0 / v[2]);
  return s;
}

}  // namespace

struct lbm_handle {
  lbm_params p;
  Layout L;
  hipStream_t stream;
  char *ws;
  int cur;
  int64_t step;
  bool valid;
  int rows;
  int tail_rows, tail_h;  // short chunks at the end of each band (taper_of)
  bool genr, has_s, ns;
  bool resident;  // step stores with the default cache policy (cache_resident)
  int waves_resident;  // step wavefronts the device holds at once (0: unknown)
  int pair_plan;       // tiles per XCD of the two-step kernel (pair_tiles_of)
  int pair_tiles;      // the plan in use: 0 under a tile height set by the caller
  int block_plan;      // steps per launch of the block kernel (plan_block_steps)
  int block_steps;     // the plan in use: 0 under a tile height set by the caller
  bool of_batch;       // transfers of a batch's simulations always use staging
  bool block_short;    // its launches of one step pay (one_step_pays)
  std::string kernel;  // the step kernel variant, as a profiler names it
  std::string kernel_of_several;  // the kernel of several steps per launch, if planned
  std::string err;
  double *fixed_scratch;  // this device's copy of the static read-back scratch
};

// One launch of the block kernel: its steps, and where it reads the previous
// velocity and writes the new one.
struct BlockLaunch {
  int steps;
  const void *aux_in;
  void *aux_out;
};

// Step launches: compiled in both passes of this file (see lbm_f16_part).
namespace {

void *pops(lbm_handle *h, int which) { return h->ws + h->L.off_pop[which]; }
void *rest(lbm_handle *h, int which) { return h->ws + h->L.off_rest[which]; }
void *auxp(lbm_handle *h) { return h->ws + h->L.off_aux; }
double *scratch(lbm_handle *h) { return reinterpret_cast<double *>(h->ws + h->L.off_scratch); }
double *partials(lbm_handle *h) { return reinterpret_cast<double *>(h->ws + h->L.off_partial); }
int *flagp(lbm_handle *h) { return reinterpret_cast<int *>(h->ws + h->L.off_flag); }

// Columns per lane of the step kernel: two for float32 and float16 storage
// when nx is even (each lane's pair of columns then never straddles the
// periodic seam), else one.
int sites_per_lane(const lbm_params &p) {
  return p.precision != LBM_FP64 && p.nx % 2 == 0 ? 2 : 1;
}
// Whether a grid lies where default stores beat non-temporal ones: measured
// for float32 and float64 storage on single grids from 256x128 to 2048^2,
// the default is 6-25% faster (the written populations are read back from
// the Infinity Cache) from 250 k to 1.25 M sites with float32 storage and
// from 125 k to 625 k sites with float64 storage (64-320 MB of step traffic
// at the 256 and 512 bytes per site the step moved when those measurements
// were taken), and equal or slower outside.
bool cache_resident(const lbm_params &p) {
  const double sites = double(p.nx) * double(p.ny);
  if (p.precision == LBM_FP32) return sites >= 250e3 && sites <= 1.25e6;
  if (p.precision == LBM_FP64) return sites >= 125e3 && sites <= 625e3;
  return false;
}

int strips_of(const lbm_params &p) {
  const int cols = sites_per_lane(p) == 2 ? Strip<2>::kCols : Strip<1>::kCols;
  return (p.nx + cols - 1) / cols;
}

template <class P>
StepArgs<P> step_args(const lbm_handle *h, int cur) {
  lbm_handle *hh = const_cast<lbm_handle *>(h);
  StepArgs<P> a;
  a.p = make_phys<typename P::R>(h->p);
  a.sc = make_scales<P>(h->p);
  a.src = static_cast<const typename P::S *>(pops(hh, cur));
  a.src_rest = static_cast<const typename P::A *>(rest(hh, cur));
  a.dst = static_cast<typename P::S *>(pops(hh, cur ^ 1));
  a.dst_rest = static_cast<typename P::A *>(rest(hh, cur ^ 1));
  a.aux = static_cast<typename P::A *>(auxp(hh));
  a.flag = flagp(hh);
  a.nx = h->p.nx;
  a.ny = h->p.ny;
  a.walls = h->p.walls_y;
  a.nstrips = strips_of(h->p);
  a.rows = h->rows;
  a.tail_rows = 0;  // batched tiles come from the tile list
  a.tail_h = 1;
  return a;
}

// One step launch; with waves_per_cu set, instead the number of this
// variant's wavefronts one compute unit holds at once.
template <class P, int K, bool GENR, bool HAS_S, bool NS>
hipError_t launch_step(lbm_handle *h, int *waves_per_cu) {
  if (waves_per_cu) {
    int blocks = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &blocks, lbm_step_kernel<P, K, GENR, HAS_S, NS>, kWave * P::kBlockWaves, 0);
    *waves_per_cu = blocks * P::kBlockWaves;
    return e;
  }
  StepArgs<P> a = step_args<P>(h, h->cur);
  a.tail_rows = h->tail_rows;
  a.tail_h = h->tail_h;
  hipLaunchKernelGGL((lbm_step_kernel<P, K, GENR, HAS_S, NS>), dim3(step_grid<P>(a)),
                     dim3(kWave * P::kBlockWaves), 0, h->stream, a);
  return hipGetLastError();
}

template <class P, int K>
hipError_t launch_step_prec(lbm_handle *h, int *waves_per_cu) {
  if (!h->ns)
    return h->genr ? launch_step<P, K, true, false, false>(h, waves_per_cu)
                   : launch_step<P, K, false, false, false>(h, waves_per_cu);
  if (h->genr)
    return h->has_s ? launch_step<P, K, true, true, true>(h, waves_per_cu)
                    : launch_step<P, K, true, false, true>(h, waves_per_cu);
  return h->has_s ? launch_step<P, K, false, true, true>(h, waves_per_cu)
                  : launch_step<P, K, false, false, true>(h, waves_per_cu);
}

// Blocks a launch of `steps` steps takes.
int block_count(const lbm_params &p, int steps) {
  const int hx = p.precision == LBM_FP16DEV ? block_halo_x<F16>(steps) : block_halo_x<F32>(steps);
  const int w = kBlockSide - 2 * hx, t = kBlockSide - 2 * block_halo_y(steps);
  const long long n = (long long)((p.nx + w - 1) / w) * ((p.ny + t - 1) / t);
  return int(std::min<long long>(n, 1 << 30));
}

// A launch of the block kernel; with blocks_per_cu set, instead the number of
// its workgroups one compute unit holds at once.
template <class P, bool GENR, bool HAS_S, bool NS>
hipError_t launch_block_as(lbm_handle *h, const BlockLaunch &l, int *blocks_per_cu) {
  if (blocks_per_cu)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        blocks_per_cu, lbm_block_kernel<P, GENR, HAS_S, NS>, kBlockSide * kBlockSide, 0);
  BlockArgs<P> b;
  b.s = step_args<P>(h, h->cur);
  b.s.aux = static_cast<typename P::A *>(const_cast<void *>(l.aux_in));
  b.aux_out = static_cast<typename P::A *>(l.aux_out);
  b.steps = l.steps;
  const int w = kBlockSide - 2 * block_halo_x<P>(l.steps);
  b.ntx = (h->p.nx + w - 1) / w;
  b.ntiles = block_count(h->p, l.steps);
  hipLaunchKernelGGL((lbm_block_kernel<P, GENR, HAS_S, NS>),
                     dim3((b.ntiles + kXcds - 1) / kXcds * kXcds),
                     dim3(kBlockSide * kBlockSide), 0, h->stream, b);
  return hipGetLastError();
}

// A launch of the two-step kernel; with waves_per_cu set, instead the number
// of its wavefronts one compute unit holds at once.
template <class P, bool GENR, bool HAS_S>
hipError_t launch_pair_as(lbm_handle *h, const BlockLaunch &l, int *waves_per_cu) {
  if (waves_per_cu)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(waves_per_cu,
                                                        lbm_pair_kernel<P, GENR, HAS_S>, kWave, 0);
  PairArgs<P> b;
  b.s = step_args<P>(h, h->cur);
  b.s.aux = static_cast<typename P::A *>(const_cast<void *>(l.aux_in));
  b.s.nstrips = pair_strips(h->p.nx);
  b.aux_out = static_cast<typename P::A *>(l.aux_out);
  b.tiles = h->pair_tiles;
  hipLaunchKernelGGL((lbm_pair_kernel<P, GENR, HAS_S>), dim3(kXcds * b.tiles), dim3(kWave), 0,
                     h->stream, b);
  return hipGetLastError();
}

template <class P>
hipError_t launch_pair(lbm_handle *h, const BlockLaunch &l, int *w) {
  if (h->genr)
    return h->has_s ? launch_pair_as<P, true, true>(h, l, w)
                    : launch_pair_as<P, true, false>(h, l, w);
  return h->has_s ? launch_pair_as<P, false, true>(h, l, w)
                  : launch_pair_as<P, false, false>(h, l, w);
}

template <class P>
hipError_t launch_block(lbm_handle *h, const BlockLaunch &l, int *blocks_per_cu) {
  int *w = blocks_per_cu;
  if (!h->ns)
    return h->genr ? launch_block_as<P, true, false, false>(h, l, w)
                   : launch_block_as<P, false, false, false>(h, l, w);
  if (h->genr)
    return h->has_s ? launch_block_as<P, true, true, true>(h, l, w)
                    : launch_block_as<P, true, false, true>(h, l, w);
  return h->has_s ? launch_block_as<P, false, true, true>(h, l, w)
                  : launch_block_as<P, false, false, true>(h, l, w);
}

template <class P, int K, bool GENR, bool HAS_S, bool NS>
void launch_batch(int blocks, hipStream_t st, const void *desc, const TileRef *tiles,
                  const int *count, int k) {
  hipLaunchKernelGGL((lbm_batch_step_kernel<P, K, GENR, HAS_S, NS>), dim3(blocks),
                     dim3(kWave * P::kBlockWaves), 0, st,
                     static_cast<const BatchInst<P> *>(desc), tiles, count, k);
}

template <class P, int K>
void launch_batch_prec(int c, int blocks, hipStream_t st, const void *desc,
                       const TileRef *tiles, const int *count, int k) {
  switch (c & 7) {
    case 0: launch_batch<P, K, false, false, true>(blocks, st, desc, tiles, count, k); break;
    case 1: launch_batch<P, K, false, true, true>(blocks, st, desc, tiles, count, k); break;
    case 2: launch_batch<P, K, true, false, true>(blocks, st, desc, tiles, count, k); break;
    case 3: launch_batch<P, K, true, true, true>(blocks, st, desc, tiles, count, k); break;
    case 4: launch_batch<P, K, false, false, false>(blocks, st, desc, tiles, count, k); break;
    default: launch_batch<P, K, true, false, false>(blocks, st, desc, tiles, count, k); break;
  }
}

}  // namespace

// The float16 step kernels are compiled in a second pass of this file
// (LBM_F16_PART) that fuses a multiply and an add only within one source
// expression (-ffp-contract=on, done by the front end and so the same in
// every inlined copy).  Float16 storage rounds stochastically from all 32
// bits of each value, so every copy of the row code must give the same
// bits for the results not to depend on the tile height; the float32 and
// float64 kernels keep the compiler's default fusion (1-2% faster) and are
// tile-height independent with it.
namespace lbm_f16_part {
hipError_t step(lbm_handle *h, int *waves_per_cu);
hipError_t block(lbm_handle *h, const BlockLaunch &l, int *blocks_per_cu);
void batch(int c, int blocks, hipStream_t st, const void *desc, const void *tiles,
           const int *count, int k);
}  // namespace lbm_f16_part

#ifdef LBM_F16_PART
namespace lbm_f16_part {
hipError_t step(lbm_handle *h, int *waves_per_cu) {
  return sites_per_lane(h->p) == 2 ? launch_step_prec<F16, 2>(h, waves_per_cu)
                                   : launch_step_prec<F16, 1>(h, waves_per_cu);
}
hipError_t block(lbm_handle *h, const BlockLaunch &l, int *blocks_per_cu) {
  return launch_block<F16>(h, l, blocks_per_cu);
}
void batch(int c, int blocks, hipStream_t st, const void *desc, const void *tiles,
           const int *count, int k) {
  const TileRef *t = static_cast<const TileRef *>(tiles);
  if (c / 8 == int(LBM_FP16DEV))
    launch_batch_prec<F16, 1>(c, blocks, st, desc, t, count, k);
  else
    launch_batch_prec<F16, 2>(c, blocks, st, desc, t, count, k);
}
}  // namespace lbm_f16_part
#else

namespace {

lbm_status fail(lbm_handle *h, lbm_status s, const std::string &msg) {
  if (h)
    h->err = msg;
  else
    g_create_error = msg;
  return s;
}

lbm_status hip_check(lbm_handle *h, hipError_t e, const char *what) {
  if (e == hipSuccess) return LBM_OK;
  return fail(h, LBM_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}


// ---- host transfers.  Copies between the caller's pageable memory and the
// device go through pinned staging in chunks: the device copies at the rate
// of the link (57 GB/s pinned, against 18 GB/s read and 29 GB/s written for
// pageable memory), and for large ones worker threads copy between staging
// and the caller's memory meanwhile and take the page faults of memory the
// caller has not touched yet, which cost one thread more than the link does
// (128 MB: 2.4 ms on the link, 7-8 ms of first touches).  Only the calling
// thread makes HIP calls: a new thread's first one takes about 3 ms.
// Measured, direct -> this: the five fields of 64^2 0.16 -> 0.05 ms, 512^2
// 0.64 -> 0.43, 1024^2 2.35 -> 1.6, 1448^2 4.7 -> 3.0, 2048^2 (168 MB) 17 ->
// 4.8; initial fields of 1448^2 4.0 -> 3.2, of 2048^2 8 -> 3.7 ms.

constexpr size_t kChunkBytes = 2u << 20;  // a huge page of host memory
constexpr int kSlots = 12;                // chunks in staging
constexpr int kWorkers = 6;
// Size of the largest piece from which threads help.  malloc maps blocks of 32
// MiB and more afresh, in huge pages where the caller asks for them; smaller
// ones may come from its heap, whose pages come singly, and six threads that
// fault those in at once take longer than one and hold up the caller (the
// fields of 1023x769, 6 MB each, in new memory: 5-9 ms with threads, 2.8-4
// without, 3.9-5.1 for direct copies; of 2048^2, 34 MB each, 5 ms with
// threads, 17 direct).
constexpr size_t kThreadedBytes = 32u << 20;

// To the device, staging without threads pays for initial fields of up to
// kOneWrite (one copy instead of four) and of more than kManyWrites (their
// check goes on while the chunk before is copied).  Between these, and for a
// checkpoint, it is one more pass over host memory.  Directly and through
// staging: initial fields of 128^2 (0.5 MB) 0.075 and 0.060 ms, 192^2 0.092
// and 0.091, 288^2 0.13 and 0.19, 576^2 (10.6 MB) 0.46 and 0.47, 768^2 0.77
// and 0.73; float32 checkpoints of 160^2 0.13 and 0.17, 384^2 0.50 and 0.53,
// 512^2 (27 MB the largest part) 0.86 and 0.86, 576^2 with threads 1.31 and
// 1.12.
constexpr size_t kOneWrite = 1u << 20;
constexpr size_t kManyWrites = 12u << 20;
// Not in a batch, whose simulations step meanwhile: with the joiners' initial
// fields copied directly, the served burst of twelve float32 solves took 16 to
// 20 ms (every other run 19 or more), through staging 15 to 16.

// Making staging costs as much as it saves in several small transfers, so a
// program's first two of up to kAtOnce, say the initial fields and the result
// of one solve, go without (StagingPool::take); but not fields that fit in the
// smallest staging.  Create, init, read, destroy, directly and with staging:
// float32 32^2 0.160 and 0.134 ms, 64^2 0.160 and 0.153, 256^2 (2.6 MB read)
// 0.32 and 0.50, 320^2 0.42 and 0.55, 384^2 0.64 and 0.73, 512^2 (10.5 MB)
// 1.07 and 0.94; a checkpoint of 160^2 set and got 0.36 and 0.47.
constexpr size_t kAtOnce = 8u << 20;
constexpr size_t kLeastStaging = 1u << 18;

// Asks for the whole pages of [mem, mem + n), which is about to be written, in
// one call: new pages taken one fault at a time cost 0.45 us each.  Does
// nothing where the kernel does not know the request.
inline void want_pages(char *mem, size_t n) {
  constexpr uintptr_t kPage = 4096;
  constexpr int kPopulateWrite = 23;  // MADV_POPULATE_WRITE
  const uintptr_t from = (reinterpret_cast<uintptr_t>(mem) + kPage - 1) / kPage * kPage;
  const uintptr_t to = (reinterpret_cast<uintptr_t>(mem) + n) / kPage * kPage;
  if (to >= from + 16 * kPage) (void)madvise(reinterpret_cast<void *>(from), to - from, kPopulateWrite);
}

// Makes `dev` the calling thread's current device while it lives.
class OnDevice {
 public:
  explicit OnDevice(int dev) {
    ok_ = hipGetDevice(&before_) == hipSuccess &&
          (before_ == dev || hipSetDevice(dev) == hipSuccess);
    back_ = ok_ && before_ != dev;
  }
  ~OnDevice() {
    if (back_) (void)hipSetDevice(before_);
  }
  OnDevice(const OnDevice &) = delete;
  OnDevice &operator=(const OnDevice &) = delete;
  bool ok() const { return ok_; }

 private:
  int before_ = 0;
  bool ok_, back_;
};

struct Staging {
  char *mem = nullptr;  // the sticky flag's copy, then the chunks
  size_t bytes = 0;
  int device = -1;      // of the events: streams of others refuse them
  hipEvent_t done[kSlots] = {};
};
constexpr size_t kStagingHead = 256;

// Idle staging buffers: at most kIdle of them (24 MiB each at most), freed
// when the last handle is destroyed.
class StagingPool {
 public:
  void enter() {
    std::lock_guard<std::mutex> lock(mu_);
    ++handles_;
  }
  void leave() {
    Staging all[kIdle];
    int n = 0;
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (--handles_ == 0) {
        while (count_ > 0) all[n++] = idle_[--count_];
        small_ = 0;
      }
    }
    while (n > 0) release(all[--n]);
  }
  // A buffer of at least `bytes` for a stream of `device` (false: none to be
  // had, or for this `small` transfer none worth making).
  bool take(size_t bytes, int device, bool small, Staging *out) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      for (int i = 0; i < count_; ++i)
        if (idle_[i].bytes >= bytes && idle_[i].device == device) {
          *out = idle_[i];
          idle_[i] = idle_[--count_];
          return true;
        }
      if (small && small_ < kSmallOnes) {
        ++small_;
        return false;
      }
    }
    const OnDevice on(device);
    Staging s;
    s.device = device;
    s.bytes = kLeastStaging;
    while (s.bytes < bytes) s.bytes *= 2;
    s.bytes = std::min(s.bytes, kStagingHead + kSlots * kChunkBytes);
    bool ok = on.ok() &&
              hipHostMalloc(reinterpret_cast<void **>(&s.mem), s.bytes, hipHostMallocPortable) ==
                  hipSuccess;
    if (!ok) s.mem = nullptr;
    for (int w = 0; w < kSlots && ok; ++w)
      ok = hipEventCreateWithFlags(&s.done[w], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
      release(s);
      (void)hipGetLastError();
      return false;
    }
    *out = s;
    return true;
  }
  void give(Staging s) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (count_ < kIdle) {
        idle_[count_++] = s;
        return;
      }
      for (Staging &o : idle_)  // keep the larger ones
        if (o.bytes < s.bytes) std::swap(o, s);
    }
    release(s);
  }

 private:
  static constexpr int kIdle = 2;
  static constexpr int kSmallOnes = 2;
  int small_ = 0;  // those gone without since the first of the live handles
  static void release(Staging &s) {
    for (hipEvent_t e : s.done)
      if (e) (void)hipEventDestroy(e);
    if (s.mem) (void)hipHostFree(s.mem);
  }
  std::mutex mu_;
  Staging idle_[kIdle];
  int count_ = 0;
  long long handles_ = 0;
};
StagingPool g_staging;

// Device memory and the caller's, to be copied either way.
struct Piece {
  char *dev;
  char *host;
  size_t bytes;
};

struct NoCheck {
  bool operator()(int, const char *, size_t) const { return true; }
};

// Whether the runtime knows this memory: pinned, managed or of a device.
bool known_memory(const void *p) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
  (void)hipGetLastError();
  return false;
}

hipError_t clear_flag(lbm_handle *h) {
  return hipMemsetAsync(flagp(h), 0, sizeof(int), h->stream);
}

// transfer() without staging.
template <class Check>
hipError_t copy_directly(lbm_handle *h, const Piece *pieces, int npieces, bool planes,
                         bool to_device, int *flag, bool *refused, Check check) {
  hipError_t e = hipSuccess;
  if (flag) {
    e = hipMemcpyAsync(flag, flagp(h), sizeof(int), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess || *flag) return e;
  }
  for (int i = 0; i < npieces && e == hipSuccess; ++i) {
    if (to_device && !check(i, pieces[i].host, pieces[i].bytes)) {
      *refused = true;
      break;
    }
    e = to_device ? hipMemcpyAsync(pieces[i].dev, pieces[i].host, pieces[i].bytes,
                                   hipMemcpyHostToDevice, h->stream)
                  : hipMemcpyAsync(pieces[i].host, pieces[i].dev, pieces[i].bytes,
                                   hipMemcpyDeviceToHost, h->stream);
  }
  if (e == hipSuccess && to_device && !planes) e = clear_flag(h);
  const hipError_t last = hipStreamSynchronize(h->stream);
  return e != hipSuccess ? e : last;
}

// Copies the pieces on h's stream, to the device or from it, and waits for
// them.  From the device: the sticky flag is read first (*flag), and nothing
// reaches the caller's memory if it is set.  To the device: `check` sees all
// of the host memory; if it refuses some, the copy ends (*refused).  planes:
// the pieces are scratch planes one after another, whose gaps may be copied;
// without, they are a checkpoint, and the sticky flag is cleared behind it.
template <class Check>
hipError_t transfer(lbm_handle *h, const Piece *pieces, int npieces, bool planes, bool to_device,
                    int *flag, bool *refused, Check check) {
  // Pinned memory of the caller's takes part in the copies as it is.  Directly
  // and through staging: the five fields of 1448^2 1.63 and 3.06 ms, of 2048^2
  // 3.19 and 4.39; initial fields of 1448^2 1.87 and 2.94.
  for (int i = 0; i < npieces; ++i)
    if (known_memory(pieces[i].host))
      return copy_directly(h, pieces, npieces, planes, to_device, flag, refused, check);
  if (npieces == 0) planes = false;
  size_t total = 0;
  for (int i = 0; i < npieces; ++i) total += pieces[i].bytes;
  const size_t span = planes ? size_t(pieces[npieces - 1].dev + pieces[npieces - 1].bytes -
                                      pieces[0].dev) : total;
  size_t largest = 0;
  for (int i = 0; i < npieces; ++i) largest = std::max(largest, pieces[i].bytes);
  int threads = largest >= kThreadedBytes ? kWorkers : 0;
  if (to_device && threads == 0 && !h->of_batch &&
      !(planes && (span <= kOneWrite || span > kManyWrites)))
    return copy_directly(h, pieces, npieces, planes, to_device, flag, refused, check);
  // Small transfers are one chunk, scratch planes one device copy.  Larger
  // ones are cut where the caller's memory passes from one huge page to the
  // next: two workers that touch one page first would both clear it.
  const bool single = span <= kChunkBytes;
  // The cuts are whole doubles from the start of the piece, which may stand
  // on any address: `check` sees every value whole.
  auto first_part = [&](const Piece &p) {
    const size_t to_page =
        (kChunkBytes - reinterpret_cast<uintptr_t>(p.host) % kChunkBytes) / 8 * 8;
    return std::min(p.bytes, to_page ? to_page : kChunkBytes);
  };
  auto parts_of = [&](const Piece &p) {
    return 1 + (long long)((p.bytes - first_part(p) + kChunkBytes - 1) / kChunkBytes);
  };
  long long chunks = single ? 1 : 0;
  for (int i = 0; i < npieces && !single; ++i) chunks += parts_of(pieces[i]);
  const int slots = int(std::min<long long>(chunks, kSlots));
  Staging st;
  int device = -1;
  const size_t bytes = kStagingHead + (single ? span : slots * kChunkBytes);
  const bool small =
      span < kAtOnce && !h->of_batch && !(planes && bytes <= kLeastStaging);
  if (hipStreamGetDevice(h->stream, &device) != hipSuccess ||
      !g_staging.take(bytes, device, small, &st)) {
    (void)hipGetLastError();  // no staging to be had
    return copy_directly(h, pieces, npieces, planes, to_device, flag, refused, check);
  }
  auto slot = [&](long long k) { return st.mem + kStagingHead + size_t(k % slots) * kChunkBytes; };
  // f(piece, offset in it, bytes, offset in the slot) for the parts of chunk
  // k, until one is false
  auto each_part = [&](long long k, auto f) {
    size_t at = 0;
    for (int i = 0; i < npieces; ++i) {
      const Piece &p = pieces[i];
      if (single) {
        if (planes) at = size_t(p.dev - pieces[0].dev);
        if (!f(i, size_t(0), p.bytes, at)) return false;
        at += p.bytes;
        continue;
      }
      const long long n = parts_of(p);
      if (k < n) {
        const size_t off = k == 0 ? 0 : first_part(p) + size_t(k - 1) * kChunkBytes;
        return f(i, off, k == 0 ? first_part(p) : std::min(kChunkBytes, p.bytes - off), size_t(0));
      }
      k -= n;
    }
    return true;
  };
  auto host_part = [&](long long k) {  // between the slot and the caller's memory
    return each_part(k, [&](int i, size_t off, size_t n, size_t in_slot) {
      char *const mem = pieces[i].host + off;
      if (!to_device) {
        if (threads == 0) want_pages(mem, n);
        std::memcpy(mem, slot(k) + in_slot, n);
        return true;
      }
      if (!check(i, mem, n)) return false;
      std::memcpy(slot(k) + in_slot, mem, n);
      return true;
    });
  };
  auto device_part = [&](long long k) {  // between the slot and the device
    hipError_t e = hipSuccess;
    if (single && planes)
      return to_device ? hipMemcpyAsync(pieces[0].dev, slot(0), span, hipMemcpyHostToDevice,
                                        h->stream)
                       : hipMemcpyAsync(slot(0), pieces[0].dev, span, hipMemcpyDeviceToHost,
                                        h->stream);
    each_part(k, [&](int i, size_t off, size_t n, size_t in_slot) {
      e = to_device ? hipMemcpyAsync(pieces[i].dev + off, slot(k) + in_slot, n,
                                     hipMemcpyHostToDevice, h->stream)
                    : hipMemcpyAsync(slot(k) + in_slot, pieces[i].dev + off, n,
                                     hipMemcpyDeviceToHost, h->stream);
      return e == hipSuccess;
    });
    return e != hipSuccess || single ? e : hipEventRecord(st.done[k % slots], h->stream);
  };
  auto device_done = [&](long long k) {
    return single ? hipStreamSynchronize(h->stream) : hipEventSynchronize(st.done[k % slots]);
  };
  // The last chunk of each slot that the workers may take up, and that they
  // have finished; worker w has chunks w, w + threads, ...
  std::atomic<long long> open[kSlots], closed[kSlots];
  for (int i = 0; i < kSlots; ++i) {
    open[i] = to_device ? i : -1;  // every slot is empty at first
    closed[i] = -1;
  }
  std::atomic<bool> stop{false}, bad{false};
  auto work = [&](int w) {
    for (long long k = w; k < chunks; k += threads) {
      while (open[k % slots] < k) {
        if (stop) return;
        std::this_thread::yield();
      }
      if (!host_part(k)) {
        bad = stop = true;
        return;
      }
      closed[k % slots] = k;
    }
  };
  std::thread pool[kWorkers];
  int started = 0;
  for (; started < threads; ++started) {
    try {
      pool[started] = std::thread(work, started);
    } catch (...) {  // no thread to be had
      break;
    }
  }
  if (started < threads) {  // some chunks would have no worker: none takes any
    stop = true;
    for (int w = 0; w < started; ++w) pool[w].join();
    stop = false;
    started = threads = 0;
    for (int i = 0; i < kSlots; ++i) closed[i] = -1;
  }
  // chunk k has passed between its slot and the caller's memory
  auto host_done = [&](long long k) {
    if (threads == 0) return true;
    while (closed[k % slots] < k && !stop) std::this_thread::yield();
    return closed[k % slots] >= k;
  };
  hipError_t e = hipSuccess;
  if (to_device) {
    long long waited = 0;  // chunks the device has read
    for (long long k = 0; k < chunks && e == hipSuccess && !stop; ++k) {
      // half the slots stay with the workers
      for (; waited <= k - std::max(1, slots / 2) && e == hipSuccess; ++waited) {
        e = device_done(waited);
        open[waited % slots] = waited + slots;
      }
      if (e != hipSuccess) break;
      if (threads == 0 && !host_part(k)) {
        bad = true;
        break;
      }
      if (!host_done(k)) break;
      e = device_part(k);
    }
  } else {
    int *const flag_copy = reinterpret_cast<int *>(st.mem);
    if (flag)
      e = hipMemcpyAsync(flag_copy, flagp(h), sizeof(int), hipMemcpyDeviceToHost, h->stream);
    long long next = 0;  // first chunk the device has not been asked for
    for (long long k = 0; k < chunks && e == hipSuccess; ++k) {
      for (; next < chunks && next < k + slots && e == hipSuccess; ++next) {
        if (next >= slots && next > k && threads > 0 && closed[next % slots] < next - slots) break;
        if (next >= slots && !host_done(next - slots)) break;
        e = device_part(next);
      }
      if (e == hipSuccess) e = device_done(k);
      if (e != hipSuccess) break;
      if (flag && k == 0 && *static_cast<volatile int *>(flag_copy)) break;
      if (threads == 0)
        host_part(k);
      else
        open[k % slots] = k;
    }
    if (e == hipSuccess && chunks == 0) e = hipStreamSynchronize(h->stream);
    if (flag) *flag = *static_cast<volatile int *>(flag_copy);
    for (long long k = std::max(0LL, chunks - slots);
         k < chunks && e == hipSuccess && !(flag && *flag); ++k)
      host_done(k);
  }
  stop = true;
  for (int w = 0; w < started; ++w) pool[w].join();
  if (refused) *refused = bad;
  // nothing of the staging may be in flight when it goes back
  if (e == hipSuccess && to_device && !planes) e = clear_flag(h);
  if (to_device || e != hipSuccess || (flag && *flag)) {
    const hipError_t last = hipStreamSynchronize(h->stream);
    if (e == hipSuccess) e = last;
  }
  g_staging.give(st);
  return e;
}

template <class P>
SiteArgs<P> site_args(lbm_handle *h) {
  SiteArgs<P> a;
  a.src = static_cast<const typename P::S *>(pops(h, h->cur));
  a.src_rest = static_cast<const typename P::A *>(rest(h, h->cur));
  a.dst = static_cast<typename P::S *>(pops(h, h->cur));
  a.dst_rest = static_cast<typename P::A *>(rest(h, h->cur));
  a.aux = static_cast<typename P::A *>(auxp(h));
  a.scratch = scratch(h);
  a.sc = make_scales<P>(h->p);
  a.plane = h->L.plane;
  a.nx = h->p.nx;
  a.ny = h->p.ny;
  a.walls = h->p.walls_y;
  a.ns = h->ns ? 1 : 0;
  return a;
}


int default_rows(const lbm_params &p, bool in_batch = false) {
  const long long strips = strips_of(p);
  // Many short tiles keep the wavefronts' start-up and drain phases
  // staggered; the two extra halo rows per tile are served mostly from
  // cache.  Measured on 2048x2048: 2 rows for float32 with two columns per
  // lane, 3 with one, 5 for float16 storage with two (1% over 4), 4 for
  // float16 with one and for float64 storage.  In a batch of the serving
  // mix (128^2 to 1024^2) float16 storage with two columns is 2% faster
  // with 4 rows than with 5.
  const long long target = p.precision == LBM_FP32 ? 24576 : 16384;
  const bool two = sites_per_lane(p) == 2;
  const long long lo = p.precision == LBM_FP32 ? (two ? 2 : 3)
                     : p.precision == LBM_FP16DEV && two && !in_batch ? 5 : 4;
  long long rows = strips * p.ny / target;
  if (rows < lo) rows = lo;
  if (rows > 64) rows = 64;
  return int(rows);
}


// One step of h (or, with waves_per_cu set, the occupancy of its kernel).
hipError_t run_step(lbm_handle *h, int *waves_per_cu = nullptr) {
  int *w = waves_per_cu;
  switch (h->p.precision) {
    case LBM_FP64:
      return h->resident ? launch_step_prec<F64C, 1>(h, w) : launch_step_prec<F64, 1>(h, w);
    case LBM_FP32:
      if (sites_per_lane(h->p) == 2)
        return h->resident ? launch_step_prec<F32C, 2>(h, w) : launch_step_prec<F32, 2>(h, w);
      return h->resident ? launch_step_prec<F32C, 1>(h, w) : launch_step_prec<F32, 1>(h, w);
    default: return lbm_f16_part::step(h, w);
  }
}

// Several steps of h in one launch (or, with blocks_per_cu set, the occupancy
// of its block kernel).
hipError_t run_block(lbm_handle *h, const BlockLaunch &l, int *blocks_per_cu = nullptr) {
  switch (h->p.precision) {
    case LBM_FP64: return launch_block<F64C>(h, l, blocks_per_cu);
    case LBM_FP32: return launch_block<F32C>(h, l, blocks_per_cu);
    default: return lbm_f16_part::block(h, l, blocks_per_cu);
  }
}

// Two steps of h in one launch (or, with waves_per_cu set, the occupancy of
// its two-step kernel).
hipError_t run_pair(lbm_handle *h, const BlockLaunch &l, int *waves_per_cu = nullptr) {
  if (h->p.precision == LBM_FP64)
    return h->resident ? launch_pair<F64C>(h, l, waves_per_cu)
                       : launch_pair<F64>(h, l, waves_per_cu);
  return h->resident ? launch_pair<F32C>(h, l, waves_per_cu) : launch_pair<F32>(h, l, waves_per_cu);
}

// lbm_step_kernel's shortest walks, with one column per lane in float32
// arithmetic: tiles of one row (5.5 us; with two columns 6.8, in float64 7.3),
// and float16 storage's of two (6.4 to 7.1).
bool short_walk(const lbm_handle *h) {
  if (h->p.precision == LBM_FP64 || sites_per_lane(h->p) == 2) return false;
  return h->rows == 1 || h->p.precision == LBM_FP16DEV;
}

// Whether a launch of the block kernel with one step is faster than
// lbm_step_kernel's: where its blocks all run at once, and the walk that it
// replaces is not among the shortest, which a block's fixed part outweighs:
//  * float64: 32^2 to 222^2 7.3 -> 6.3 us to 8.1 -> 7.3, but with a prescribed
//    velocity 4.8 -> 5.0 and 5.5 -> 6.0;
//  * float32 and float16 with two columns per lane, or one where the tiles are
//    of two rows: float32 60^2 6.8 -> 5.8, 260^2 (361 blocks) 7.7 -> 7.4, 300^2
//    (484) 7.65 -> 7.7; float16 160^2 8.4 -> 7.1; prescribed float16 280^2
//    (400) 7.2 -> 6.4, 290^2 (441) 7.1 -> 7.7; float32 280^2 6.0 -> 5.9, 310^2
//    (529) 6.0 -> 6.7;
//  * not over the shortest walks: float32 61x60 5.5 -> 5.7, 201x200 6.0 -> 6.4;
//    float16 161x160 6.7 -> 7.0, 257x159 7.1 -> 7.2; prescribed float32 161x160
//    4.8 -> 5.1, float16 221x220 5.5 -> 6.0, 283x220 6.4 -> 6.55.
bool one_step_pays(const lbm_handle *h, int cus, int resident) {
  const int blocks = block_count(h->p, 1);
  if (blocks > resident) return false;
  if (h->p.precision == LBM_FP64) return h->ns;
  return !short_walk(h) && 3 * blocks <= 5 * cus;
}

// Time steps per launch of the block kernel, 0 where lbm_step_kernel is
// faster.  A launch whose blocks all run at once costs its fixed part plus
// its steps, and a second round of blocks doubles it, so the most steps are
// taken whose blocks fit:
//  * 3 (kBlockMaxSteps), if each block has a compute unit to itself (more steps leave 2 x 2
//    sites of a block).  float32 96^2, 256 blocks: 2.65 us per step against
//    3.36 with 2; 108^2, 324 blocks: 3.03 against 3.39 for float32, but
//    5.46 against 3.84 for float64, of which a compute unit holds one block.
//  * 2, if they are all resident: float64 160^2, 256 blocks, 3.98 us against
//    6.33 with 1 and 7.9 for lbm_step_kernel; 176^2, 324 blocks, 6.67 against
//    6.53 with 1.  float32 with the Navier-Stokes flow also gains where two
//    rounds take them, but not over tiles of one row with one column per lane.
//    With equal densities 256^2, 676 blocks, 7.2 us -> 6.2, 316^2, 1024 blocks,
//    7.4 -> 7.05, 231x230, 552 blocks, 5.85 -> 6.1; with different ones, whose
//    blocks take longer, 256^2 7.5 -> 6.7, 280^2, 784 blocks, 7.7 -> 7.5, 281x280,
//    812, 7.6 -> 7.7, 320x300, 960, 7.5 -> 7.85.
//  * 1, if that pays (one_step_pays).
// Calls of a few steps, and what is left of longer ones, take launches of one
// step where they pay, else lbm_step_kernel (block_share).
int plan_block_steps(lbm_handle *h, int cus, int resident) {
  if (cus <= 0 || resident <= 0) return 0;
  h->block_short = one_step_pays(h, cus, resident);
  if (block_count(h->p, kBlockMaxSteps) <= cus) return kBlockMaxSteps;
  const int sixteenths = h->p.precision != LBM_FP32 || !h->ns || short_walk(h) ? 16
                         : h->has_s                                            ? 25
                                                                               : 32;
  if (block_count(h->p, 2) <= resident * sixteenths / 16) return 2;
  return h->block_short ? 1 : 0;
}

// Steps of a call of n that launches of the block kernel take, and the number
// of these: as few as can be with at most `most` steps each, at least two
// where `one` step in a launch does not pay.  The call's launches are as many
// as its steps but for an even number, since each goes from one copy of the
// state to the other, and steps that a caller captures and replays have to end
// on the copy that as many single steps end on.  `even`: the launches have to
// be even in number.
struct BlockShare {
  int64_t steps, launches;
};
BlockShare block_share(int64_t n, int most, bool one, bool even) {
  if (n < 2) return {0, 0};
  for (int64_t steps = even ? n - n % 2 : n; steps > 0; steps -= even ? 2 : 1) {
    int64_t launches = (steps + most - 1) / most;
    launches += (steps - launches) % 2;
    if (launches <= (one ? steps : steps / 2)) return {steps, launches};
  }
  return {0, 0};
}

// Default tile height of a single simulation.  A step costs about one
// wavefront's walk down its tile (3-5 us per row) when every wavefront of
// the launch fits on the device at once, so a grid too small to fill the
// device takes the shortest tiles that still fit in one round (measured:
// 1-row tiles make a 64x64 step 1.5-3x faster than the heights tuned for
// large grids).  Larger grids keep those heights (default_rows).
int single_rows(const lbm_handle *h) {
  const int lo = default_rows(h->p);
  const long long strips = strips_of(h->p);
  if (h->waves_resident <= 0) return lo;
  for (int r = 1; r < lo; ++r)
    if (strips * ((h->p.ny + r - 1) / r) <= h->waves_resident) return r;
  return lo;
}

// Short chunks at the end of each XCD's band of a single-grid step (see
// lbm_step_kernel).  When the last tiles are dispatched, the device holds
// tiles at every stage of their walk and idles for about the length of one
// tile's walk as they finish; 1-row chunks make that walk short.  About
// one round of the XCD's wavefront slots takes short chunks, and at most a
// quarter of the band: more would add the prologue of a tile (rebuilding
// the rows before its first) to more of the grid.  Measured on 2048x2048
// (bitwise the same results): float32 storage 198.6 -> 196.2 us per step
// with 15 rows of 1-row chunks per band, float64 365.8 -> 363.1 us with 3,
// float16 storage unchanged; 512x512 float32, 16 rows of 64 in short
// chunks: 15.8 us, 18.8 without, 17.2 with 48.
// Where the band's tiles all run at once, the short chunks must not make a
// second round: a chunk that waits for a slot costs a whole walk.  Only as
// many rows are cut short as still fit.  us per step, a quarter of the band in
// short chunks -> those that fit: float64 330^2 17.9 -> 13.9 (none fits), 370^2
// 20.9 -> 18.4, 410^2 22.5 -> 19.8, 450^2 23.5 -> 22.8; float16 640^2 28.6 ->
// 23.7, 704^2 34.3 -> 31.1, 768^2 35.5 -> 31.5, 1024x512 35.0 -> 31.1, 896^2
// 42.6 -> 40.3, 960^2 44.1 -> 43.2; float32 630^2 23.9 -> 22.0, 571^2 18.1 ->
// 16.9.  Not for float32 tiles of 3 rows, three wavefronts to a SIMD: 619^2
// 20.5 -> 19.4, but 635^2 21.0 -> 21.9, 605x660 20.8 -> 22.1.
void taper_of(lbm_handle *h) {
  h->tail_h = 1;
  h->tail_rows = 0;
  if (h->rows <= h->tail_h || h->waves_resident <= 0) return;
  const long long round = h->waves_resident / (kXcds * strips_of(h->p));  // chunks
  h->tail_rows = int(std::min<long long>(round * h->tail_h, h->p.ny / kXcds / 4));
  const int band = (h->p.ny + kXcds - 1) / kXcds;
  auto chunks = [&] {
    return (band - h->tail_rows + h->rows - 1) / h->rows + h->tail_rows / h->tail_h;
  };
  if ((band + h->rows - 1) / h->rows <= round && !(h->p.precision == LBM_FP32 && h->rows > 2))
    while (h->tail_rows > 0 && chunks() > round) --h->tail_rows;
}

// Tile plan of a single-grid step: the tile height (single_rows) and the
// short chunks at each band's end (taper_of).  Float16 storage with two
// columns per lane instead gives every wavefront slot of an XCD one tile
// of the band, when such tiles are at most 24 rows high, and walks the few
// rows left over in 1-row chunks after them: that step is short of vector
// issue, and tall tiles rebuild fewer rows before their first.  Measured on
// 2048x2048: 15 tiles of 17 rows per band and 17 one-row tiles, 159.0 us
// per step against 173.6 with 5-row tiles (float32 and float64 storage are
// 15-20% slower with tiles that tall: their halo rows are no longer shared
// through L2); neutral on 1024x1024 (4 rows) and not applied to taller
// bands (2048x4096, 4096x4096: no gain or slower).
void plan_tiles(lbm_handle *h) {
  h->rows = single_rows(h);
  taper_of(h);
  if (h->p.precision != LBM_FP16DEV || sites_per_lane(h->p) != 2 || h->waves_resident <= 0)
    return;
  const long long per_round = h->waves_resident / (kXcds * strips_of(h->p));  // chunks
  const int band = h->p.ny / kXcds;
  if (per_round < 1 || band / per_round < h->rows || band / per_round > 24) return;
  h->rows = int(band / per_round);
  h->tail_rows = int(band - per_round * h->rows);
  h->tail_h = 1;
}

// The template arguments of the step kernel run_step launches for h, in the
// order a profiler prints them: storage, columns per lane, r != 1,
// rho_A != rho_B, Navier-Stokes velocity.
const char *storage_name_of(const lbm_handle *h, bool resident) {
  return h->p.precision == LBM_FP64   ? (resident ? "F64C" : "F64")
         : h->p.precision == LBM_FP32 ? (resident ? "F32C" : "F32")
                                      : "F16";
}
const char *name_of(bool v) { return v ? "true" : "false"; }
std::string kernel_name_of(const lbm_handle *h) {
  return std::string("lbm_step_kernel<") + storage_name_of(h, h->resident) + ", " +
         std::to_string(sites_per_lane(h->p)) + ", " + name_of(h->genr) + ", " +
         name_of(h->has_s) + ", " + name_of(h->ns) + ">";
}
std::string kernel_of_several_of(const lbm_handle *h) {
  if (h->block_plan > 0)
    return std::string("lbm_block_kernel<") + storage_name_of(h, true) + ", " +
           name_of(h->genr) + ", " + name_of(h->has_s && h->ns) + ", " + name_of(h->ns) + ">";
  if (h->pair_plan > 0)
    return std::string("lbm_pair_kernel<") + storage_name_of(h, h->resident) + ", " +
           name_of(h->genr) + ", " + name_of(h->has_s) + ">";
  return h->kernel;
}

// Wavefronts of h's step kernel the current device holds at once (0 if the
// runtime cannot tell).
int query_waves_resident(lbm_handle *h) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      run_step(h, &per_cu) != hipSuccess) {
    (void)hipGetLastError();  // leave no error behind for the next call
    return 0;
  }
  return cus * per_cu;
}

// Steps per launch of h's block kernel on the current device.
int query_block_steps(lbm_handle *h) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      run_block(h, BlockLaunch{}, &per_cu) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return plan_block_steps(h, cus, cus * per_cu);
}

// Tiles per XCD of h's two-step kernel on the current device, 0 where
// lbm_step_kernel is used: where pair_tiles_of says so, for float16 storage
// (its step is bound by vector issue, which two steps per launch do not
// lower) and for a prescribed velocity.
int query_pair_tiles(lbm_handle *h) {
  int dev = 0, cus = 0, per_cu = 0;
  if (h->p.precision == LBM_FP16DEV || !h->ns) return 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      run_pair(h, BlockLaunch{}, &per_cu) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  const double least =
      pair_least_rows(h->p.precision == LBM_FP32, h->p.nx % 2 != 0, h->genr, h->has_s);
  return pair_tiles_of(h->p.nx, h->p.ny, cus * per_cu / kXcds, least);
}

template <class P>
hipError_t launch_macros(lbm_handle *h, double *sc, long long plane) {
  SiteArgs<P> a = site_args<P>(h);
  a.scratch = sc;
  a.plane = plane;
  const long long n = (long long)h->p.nx * h->p.ny;
  const int blocks = int((n + 255) / 256);
  const Phys<typename P::R> p = make_phys<typename P::R>(h->p);
  hipLaunchKernelGGL((lbm_macro_scalars_kernel<P>), dim3(blocks), dim3(256), 0, h->stream,
                     a, p);
  if (h->has_s)
    hipLaunchKernelGGL((lbm_macro_fields_kernel<P, true>), dim3(blocks), dim3(256), 0,
                       h->stream, a, p);
  else
    hipLaunchKernelGGL((lbm_macro_fields_kernel<P, false>), dim3(blocks), dim3(256), 0,
                       h->stream, a, p);
  return hipGetLastError();
}

// The macroscopic fields of the current level into kScratch float64 planes
// of `plane` elements at sc (default: the handle's own scratch).
hipError_t run_macros(lbm_handle *h, double *sc, long long plane) {
  switch (h->p.precision) {
    case LBM_FP64: return launch_macros<F64>(h, sc, plane);
    case LBM_FP32: return launch_macros<F32>(h, sc, plane);
    default: return launch_macros<F16>(h, sc, plane);
  }
}
hipError_t run_macros(lbm_handle *h) { return run_macros(h, scratch(h), h->L.plane); }

// Read-back scratch of lbm_moments_async in static device memory, for
// callers that cannot allocate: kScratch float64 planes of at most
// kFixedSites sites, then the reduction partials.  Each device holds its own
// copy for the life of the process (32.1 MiB); host code reaches it only
// through the address hipGetSymbolAddress gives for that device.
constexpr long long kFixedSites = 1LL << 19;
constexpr long long kFixedDoubles = kScratch * kFixedSites + kReduceBlocks * kReduceVals;
static __device__ __align__(256) double fixed_scratch[kFixedDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_fixed_mu;
double *g_fixed_ptr[kMaxDevices];  // per device, resolved once

// This device's address of fixed_scratch (nullptr if it cannot be had),
// resolved once per device with that device current.
double *fixed_scratch_of(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_fixed_mu);
  if (!g_fixed_ptr[dev]) {
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess) return nullptr;
    if (cur != dev && hipSetDevice(dev) != hipSuccess) return nullptr;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(fixed_scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_fixed_ptr[dev] = static_cast<double *>(ptr);
  }
  return g_fixed_ptr[dev];
}

template <class P>
hipError_t launch_init(lbm_handle *h) {
  SiteArgs<P> a = site_args<P>(h);
  const long long n = (long long)h->p.nx * h->p.ny;
  const Phys<double> p = make_phys<double>(h->p);
  hipLaunchKernelGGL((lbm_init_kernel<P>), dim3(int((n + 255) / 256)), dim3(256), 0,
                     h->stream, a, p);
  return hipGetLastError();
}

hipError_t run_init(lbm_handle *h) {
  switch (h->p.precision) {
    case LBM_FP64: return launch_init<F64>(h);
    case LBM_FP32: return launch_init<F32>(h);
    default: return launch_init<F16>(h);
  }
}

// The moments of the read-back planes at sc into res (kMomentVals values,
// and the sticky flag after them if given).
hipError_t launch_moments(lbm_handle *h, const double *sc, long long plane, double *part,
                          const int *flag, double *res) {
  const long long n = (long long)h->p.nx * h->p.ny;
  const int blocks = reduce_blocks(n);
  hipLaunchKernelGGL(lbm_reduce_kernel, dim3(blocks), dim3(256), 0, h->stream, sc, plane, n,
                     make_phys<double>(h->p), part);
  hipLaunchKernelGGL((lbm_final_kernel<kMomentVals, kReduceVals, kMomentMaxes>), dim3(1),
                     dim3(kFinalThreads), 0, h->stream, (const double *)part, blocks, flag, res);
  return hipGetLastError();
}

// The three parts of the state after the step counter of a checkpoint.
struct StatePieces {
  Piece p[3];
  StatePieces(lbm_handle *h, int cur, char *host) {
    char *const pop = host + sizeof(int64_t), *const rst = pop + h->L.pop_bytes;
    p[0] = Piece{static_cast<char *>(pops(h, cur)), pop, h->L.pop_bytes};
    p[1] = Piece{static_cast<char *>(rest(h, cur)), rst, h->L.rest_bytes};
    p[2] = Piece{static_cast<char *>(auxp(h)), rst + h->L.rest_bytes, h->L.aux_bytes};
  }
};

lbm_status nonfinite(lbm_handle *h) {
  h->valid = false;
  return fail(h, LBM_ENONFINITE, "the device produced a non-finite value");
}

}  // namespace

extern "C" {

size_t lbm_workspace_bytes(const lbm_params *params) {
  if (validate(params)) return 0;
  return make_layout(*params).total;
}

lbm_status lbm_create(const lbm_params *params, void *dev_ws, size_t ws_bytes,
                      void *hip_stream, lbm_handle **out) {
  if (!out) return fail(nullptr, LBM_EINVAL, "out is NULL");
  *out = nullptr;
  if (const char *m = validate(params)) return fail(nullptr, LBM_EINVAL, m);
  const Layout L = make_layout(*params);
  if (!dev_ws) return fail(nullptr, LBM_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(dev_ws) % 256)
    return fail(nullptr, LBM_EINVAL, "workspace must be 256-byte aligned");
  if (ws_bytes < L.total) return fail(nullptr, LBM_ENOMEM, "workspace too small");
  lbm_handle *h = new (std::nothrow) lbm_handle();
  if (!h) return fail(nullptr, LBM_ENOMEM, "out of host memory");
  h->p = *params;
  h->L = L;
  h->stream = static_cast<hipStream_t>(hip_stream);
  h->ws = static_cast<char *>(dev_ws);
  h->cur = 0;
  h->step = 0;
  h->valid = false;
  h->rows = default_rows(*params);
  h->genr = params->r != 1.0;
  h->ns = params->flow == LBM_FLOW_NS;
  h->has_s = h->ns && params->rhoA != params->rhoB;
  h->resident = cache_resident(*params);
  h->waves_resident = query_waves_resident(h);
  plan_tiles(h);
  h->block_plan = h->block_steps = query_block_steps(h);
  h->pair_plan = h->pair_tiles = query_pair_tiles(h);
  h->of_batch = false;
  h->kernel = kernel_name_of(h);
  h->kernel_of_several = kernel_of_several_of(h);
  int dev = -1;
  h->fixed_scratch = hipStreamGetDevice(h->stream, &dev) == hipSuccess ? fixed_scratch_of(dev)
                                                                      : nullptr;
  (void)hipGetLastError();
  g_staging.enter();
  *out = h;
  return LBM_OK;
}

lbm_status lbm_init_fields(lbm_handle *h, const double *phi, const double *psi,
                           const double *ux, const double *uy) {
  if (!h) return LBM_EINVAL;
  if (!phi || !psi || !ux || !uy) return fail(h, LBM_EINVAL, "NULL field");
  const size_t n = size_t(h->p.nx) * size_t(h->p.ny);
  double *sc = scratch(h);
  const double *src[4] = {phi, psi, ux, uy};
  Piece pieces[4];
  for (int j = 0; j < 4; ++j)
    pieces[j] = Piece{reinterpret_cast<char *>(sc + j * h->L.plane),
                      reinterpret_cast<char *>(const_cast<double *>(src[j])), n * sizeof(double)};
  const bool langmuir = h->p.eos == LBM_EOS_LANGMUIR;
  std::atomic<int> why{0};
  bool refused = false;
  hipError_t e = transfer(h, pieces, 4, true, true, nullptr, &refused,
                          [&](int piece, const char *at, size_t bytes) {
    typedef double anywhere __attribute__((aligned(1)));
    const anywhere *const v = reinterpret_cast<const anywhere *>(at);
    const size_t m = bytes / sizeof(double);
    // |x| <= max rejects infinities and NaN alike; no branch per value
    int bad = 0, big = 0;
    for (size_t k = 0; k < m; ++k) bad |= !(std::fabs(v[k]) <= std::numeric_limits<double>::max());
    if (langmuir && piece == 1)
      for (size_t k = 0; k < m; ++k) big |= v[k] >= 1.0;
    if (bad | big) why |= bad ? 1 : 2;
    return !(bad | big);
  });
  if (e == hipSuccess && refused)
    return fail(h, LBM_EINVAL, why & 1 ? "non-finite initial value" : "Langmuir EOS needs psi < 1");
  if (e != hipSuccess) return hip_check(h, e, "copying initial fields");
  // from here on the stored state is being replaced: a failure leaves no
  // valid state (LBM_ESTATE until a later init or set_state succeeds)
  h->valid = false;
  h->cur = 0;
  e = run_init(h);
  if (e == hipSuccess) e = clear_flag(h);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_check(h, e, "initialising");
  h->step = 0;
  h->valid = true;
  return LBM_OK;
}

lbm_status lbm_step(lbm_handle *h, int64_t nsteps) {
  if (!h) return LBM_EINVAL;
  if (nsteps < 0) return fail(h, LBM_EINVAL, "nsteps < 0");
  if (!h->valid) return fail(h, LBM_ESTATE, "no valid state");
  bool launched = false;
  auto after = [&](hipError_t e, int steps) {
    if (e != hipSuccess) {
      // the launches already enqueued still run: the state is no longer the
      // one before the call, nor a known number of steps past it
      if (launched) h->valid = false;
      return hip_check(h, e, "launching the step kernel");
    }
    launched = true;
    h->cur ^= 1;
    h->step += steps;
    return LBM_OK;
  };
  int64_t left = nsteps;
  // Launches of several steps read the previous velocity where others write
  // it, so they cannot update it in place: they write it alternately to the
  // scratch planes and back, an even number of them.
  const bool flips = h->ns && h->p.precision != LBM_FP16DEV;
  void *const aux[2] = {auxp(h), flips ? scratch(h) : auxp(h)};
  auto alternate = [&](int64_t launches, int64_t steps, auto run) {
    for (int64_t i = 0; i < launches; ++i) {
      const int64_t rest = launches - i;
      const BlockLaunch l = {int((steps + rest - 1) / rest), aux[i % 2], aux[(i + 1) % 2]};
      const lbm_status st = after(run(l), l.steps);
      if (st != LBM_OK) return st;
      steps -= l.steps;
      left -= l.steps;
    }
    return LBM_OK;
  };
  if (h->block_steps > 0) {
    const BlockShare share = block_share(left, h->block_steps, h->block_short, flips);
    const lbm_status st = alternate(share.launches, share.steps,
                                    [&](const BlockLaunch &l) { return run_block(h, l); });
    if (st != LBM_OK) return st;
  } else if (h->pair_tiles > 0) {
    const int64_t launches = left / 4 * 2;
    const lbm_status st = alternate(launches, 2 * launches,
                                    [&](const BlockLaunch &l) { return run_pair(h, l); });
    if (st != LBM_OK) return st;
  }
  for (; left > 0; --left) {
    const lbm_status st = after(run_step(h), 1);
    if (st != LBM_OK) return st;
  }
  return LBM_OK;
}

lbm_status lbm_read_fields(lbm_handle *h, double *phi, double *psi, double *ux,
                           double *uy, double *P) {
  if (!h) return LBM_EINVAL;
  if (!h->valid) return fail(h, LBM_ESTATE, "no valid state");
  hipError_t e = run_macros(h);
  if (e != hipSuccess) return hip_check(h, e, "launching read-back kernels");
  double *dst[5] = {phi, psi, ux, uy, P};
  Piece pieces[5];
  int n = 0;
  for (int j = 0; j < 5; ++j)
    if (dst[j])
      pieces[n++] = Piece{reinterpret_cast<char *>(scratch(h) + j * h->L.plane),
                          reinterpret_cast<char *>(dst[j]),
                          size_t(h->p.nx) * size_t(h->p.ny) * sizeof(double)};
  int flag = 0;
  e = transfer(h, pieces, n, true, false, &flag, nullptr, NoCheck{});
  if (e != hipSuccess) return hip_check(h, e, "reading fields");
  return flag ? nonfinite(h) : LBM_OK;
}

lbm_status lbm_moments(lbm_handle *h, lbm_moments_t *out) {
  if (!h) return LBM_EINVAL;
  if (!out) return fail(h, LBM_EINVAL, "out is NULL");
  if (!h->valid) return fail(h, LBM_ESTATE, "no valid state");
  hipError_t e = run_macros(h);
  if (e != hipSuccess) return hip_check(h, e, "launching read-back kernels");
  double *part = partials(h);
  double *res = part + kReduceBlocks * kReduceVals;
  e = launch_moments(h, scratch(h), h->L.plane, part, flagp(h), res);
  double v[kReduceVals];
  static_assert(kMomentVals + 1 <= kReduceVals, "the flag follows the moments");
  if (e == hipSuccess)
    e = hipMemcpyAsync(v, res, sizeof v, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_check(h, e, "reducing");
  if (v[kMomentVals] != 0.0) return nonfinite(h);
  out->step = h->step;
  out->sum_phi = v[0];
  out->sum_psi = v[1];
  out->mom_x = v[2];
  out->mom_y = v[3];
  out->kinetic = v[4];
  out->max_u = v[5];
  out->nonfinite = v[6] != 0.0;
  out->pad = 0;
  if (out->nonfinite) {
    h->valid = false;
    return fail(h, LBM_ENONFINITE, "non-finite macroscopic field");
  }
  return LBM_OK;
}

lbm_status lbm_moments_async(lbm_handle *h, double *dev_out) {
  if (!h) return LBM_EINVAL;
  if (!dev_out) return fail(h, LBM_EINVAL, "dev_out is NULL");
  if (!h->valid) return fail(h, LBM_ESTATE, "no valid state");
  const long long n = (long long)h->p.nx * h->p.ny;
  if (n > kFixedSites)
    return fail(h, LBM_EINVAL, "grid has more than 524288 sites, the capacity of the static "
                               "read-back scratch of lbm_moments_async (use lbm_moments)");
  double *base = h->fixed_scratch;
  if (!base) return fail(h, LBM_EDEVICE, "no address of the static read-back scratch");
  const long long plane = (long long)align_up((size_t)n, 64);
  hipError_t e = run_macros(h, base, plane);
  if (e != hipSuccess) return hip_check(h, e, "launching read-back kernels");
  double *part = base + kScratch * kFixedSites;
  return hip_check(h, launch_moments(h, base, plane, part, nullptr, dev_out),
                   "launching the reductions");
}

lbm_status lbm_shape(lbm_handle *h, lbm_shape_t *out) {
  if (!h) return LBM_EINVAL;
  if (!out) return fail(h, LBM_EINVAL, "out is NULL");
  if (!h->valid) return fail(h, LBM_ESTATE, "no valid state");
  hipError_t e = run_macros(h);
  if (e != hipSuccess) return hip_check(h, e, "launching read-back kernels");
  const lbm_params &p = h->p;
  const double *phi = scratch(h);
  double *part = partials(h);
  double *res = part + kReduceBlocks * kShapeVals;
  const int blocks = reduce_blocks((long long)p.nx * p.ny);
  auto pass = [&](int which, double cx, double cy, double *v) -> hipError_t {
    if (which == 1)
      hipLaunchKernelGGL(lbm_shape_kernel<1>, dim3(blocks), dim3(256), 0, h->stream,
                         phi, p.nx, p.ny, p.walls_y, p.phiA, p.phiB, cx, cy, part);
    else
      hipLaunchKernelGGL(lbm_shape_kernel<2>, dim3(blocks), dim3(256), 0, h->stream,
                         phi, p.nx, p.ny, p.walls_y, p.phiA, p.phiB, cx, cy, part);
    hipLaunchKernelGGL((lbm_final_kernel<kShapeVals, kShapeVals, 0u>), dim3(1),
                       dim3(kFinalThreads), 0, h->stream, (const double *)part, blocks,
                       (const int *)flagp(h), res);
    hipError_t e2 = hipGetLastError();
    if (e2 == hipSuccess)
      e2 = hipMemcpyAsync(v, res, sizeof(double) * (kShapeVals + 1), hipMemcpyDeviceToHost,
                          h->stream);
    if (e2 == hipSuccess) e2 = hipStreamSynchronize(h->stream);
    return e2;
  };
  double s1[kShapeVals + 1], s2[kShapeVals + 1];  // the flag follows the values
  e = pass(1, 0.0, 0.0, s1);
  if (e != hipSuccess) return hip_check(h, e, "shape pass 1");
  if (s1[kShapeVals] != 0.0) return nonfinite(h);
  const double area = s1[0];
  if (!(area > 0.0)) return fail(h, LBM_EINVAL, "no fluid A in the domain");
  auto circ = [](double c, double s, int n) {
    double a = std::atan2(s, c) * n / (2.0 * M_PI);
    a = std::fmod(a, double(n));
    return a < 0 ? a + n : a;
  };
  const double cx = circ(s1[1], s1[2], p.nx);
  const double cy = p.walls_y ? s1[5] / area : circ(s1[3], s1[4], p.ny);
  e = pass(2, cx, cy, s2);
  if (e != hipSuccess) return hip_check(h, e, "shape pass 2");
  const double ixx = s2[0] / area, ixy = s2[1] / area, iyy = s2[2] / area;
  const double tr = ixx + iyy, det = ixx * iyy - ixy * ixy;
  const double disc = std::sqrt(std::max(tr * tr / 4 - det, 0.0));
  const double L = 2 * std::sqrt(tr / 2 + disc), B = 2 * std::sqrt(std::max(tr / 2 - disc, 0.0));
  out->area = area;
  out->cx = cx;
  out->cy = cy;
  out->Ixx = ixx;
  out->Ixy = ixy;
  out->Iyy = iyy;
  out->length = s1[6] / (p.phiA - p.phiB);
  out->taylor_D = (L + B) > 0 ? (L - B) / (L + B) : 0.0;
  out->angle = 0.5 * std::atan2(2 * ixy, ixx - iyy);
  return LBM_OK;
}

size_t lbm_state_bytes(const lbm_handle *h) {
  if (!h) return 0;
  return sizeof(int64_t) + h->L.pop_bytes + h->L.rest_bytes + h->L.aux_bytes;
}

lbm_status lbm_get_state(lbm_handle *h, void *host_buf, size_t bytes) {
  if (!h) return LBM_EINVAL;
  if (!host_buf || bytes != lbm_state_bytes(h)) return fail(h, LBM_EINVAL, "bad buffer");
  if (!h->valid) return fail(h, LBM_ESTATE, "no valid state");
  int flag = 0;
  const StatePieces parts(h, h->cur, static_cast<char *>(host_buf));
  const hipError_t e = transfer(h, parts.p, 3, false, false, &flag, nullptr, NoCheck{});
  if (e != hipSuccess) return hip_check(h, e, "saving state");
  if (flag) return nonfinite(h);
  std::memcpy(host_buf, &h->step, sizeof(int64_t));
  return LBM_OK;
}

lbm_status lbm_set_state(lbm_handle *h, const void *host_buf, size_t bytes) {
  if (!h) return LBM_EINVAL;
  if (!host_buf || bytes != lbm_state_bytes(h)) return fail(h, LBM_EINVAL, "bad buffer");
  int64_t step;
  std::memcpy(&step, host_buf, sizeof(int64_t));
  // the stored state is overwritten from here on: a failure leaves no valid
  // state (LBM_ESTATE until a later init or set_state succeeds)
  h->valid = false;
  h->cur = 0;
  const StatePieces parts(h, 0, static_cast<char *>(const_cast<void *>(host_buf)));
  bool refused = false;
  const hipError_t e = transfer(h, parts.p, 3, false, true, nullptr, &refused, NoCheck{});
  if (e != hipSuccess) return hip_check(h, e, "restoring state");
  h->step = step;
  h->valid = true;
  return LBM_OK;
}

void lbm_destroy(lbm_handle *h) {
  if (!h) return;
  // work enqueued by lbm_step may still be writing the caller's workspace;
  // finish it before the caller can release or reuse that memory
  (void)hipStreamSynchronize(h->stream);
  delete h;
  g_staging.leave();
}

const char *lbm_last_error(const lbm_handle *h) {
  return h ? h->err.c_str() : g_create_error.c_str();
}

lbm_status lbm_set_tile_rows(lbm_handle *h, int32_t rows) {
  if (!h) return LBM_EINVAL;
  if (rows < 0 || rows > 4096) return fail(h, LBM_EINVAL, "rows out of range");
  if (rows == 0) {
    plan_tiles(h);
    h->block_steps = h->block_plan;
    h->pair_tiles = h->pair_plan;
  } else {
    h->rows = rows;
    taper_of(h);
    h->block_steps = h->pair_tiles = 0;
  }
  return LBM_OK;
}

lbm_status lbm_get_tile_plan(const lbm_handle *h, int32_t *plan) {
  if (!h || !plan) return LBM_EINVAL;
  plan[0] = h->rows;
  plan[1] = h->tail_rows;
  plan[2] = h->tail_h;
  return LBM_OK;
}

const char *lbm_step_plan(const lbm_handle *h, int32_t *steps) {
  if (!h) return "lbm_step_kernel";
  const bool several = h->block_steps > 0 || h->pair_tiles > 0;
  if (steps) *steps = !several ? 1 : h->block_steps > 0 ? h->block_steps : 2;
  return several ? h->kernel_of_several.c_str() : h->kernel.c_str();
}

const char *lbm_step_kernel_name(const lbm_handle *h) {
  return h ? h->kernel.c_str() : "lbm_step_kernel";
}

}  // extern "C"

// ------------------------------------------------------------ batch runtime

namespace {

// Kernel variants: storage precision x prescribed velocity x (r != 1) x
// (rho_A != rho_B); float32 and float16 storage with two columns per lane
// are a fourth and a fifth group after the three precisions.
constexpr int kClasses = 40;
int class_of(const lbm_handle *h) {
  int group = int(h->p.precision);
  if (sites_per_lane(h->p) == 2) group = h->p.precision == LBM_FP32 ? 3 : 4;
  return group * 8 + (h->ns ? 0 : 4) + (h->genr ? 2 : 0) + (h->has_s ? 1 : 0);
}

size_t desc_size(int prec) {
  switch (prec) {
    case LBM_FP64: return sizeof(BatchInst<F64>);
    case LBM_FP32: return sizeof(BatchInst<F32>);
    default: return sizeof(BatchInst<F16>);
  }
}

template <class P>
void fill_desc(void *dst, const lbm_handle *h, int steps) {
  BatchInst<P> d;
  std::memset(&d, 0, sizeof d);
  d.a[0] = step_args<P>(h, 0);
  d.a[1] = step_args<P>(h, 1);
  d.parity = h->cur;
  d.steps = steps;
  std::memcpy(dst, &d, sizeof d);
}


// Storage precision of a kernel variant class (its descriptor array).
int class_precision(int c) {
  const int g = c / 8;
  return g == 3 ? int(LBM_FP32) : (g == 4 ? int(LBM_FP16DEV) : g);
}

void launch_batch_class(int c, int blocks, hipStream_t st, const void *desc,
                        const TileRef *tiles, const int *count, int k) {
  switch (c / 8) {
    case LBM_FP64: launch_batch_prec<F64, 1>(c, blocks, st, desc, tiles, count, k); break;
    case LBM_FP32: launch_batch_prec<F32, 1>(c, blocks, st, desc, tiles, count, k); break;
    case 3: launch_batch_prec<F32, 2>(c, blocks, st, desc, tiles, count, k); break;
    default: lbm_f16_part::batch(c, blocks, st, desc, tiles, count, k); break;
  }
}

}  // namespace

struct lbm_batch {
  hipStream_t stream = nullptr;   // the caller's stream: all work goes here
  hipStream_t capture = nullptr;  // library stream used only to record graphs
  hipStream_t admit = nullptr;    // library stream for joiners' copies and init
  // The streams that a chunk's kernel variants run on, besides the caller's,
  // and the events that tie them to it: made with the first batch of several
  // variants.  Three lanes and the admission stream are the four hardware
  // queues of a process.
  static constexpr int kLanes = 3;
  hipStream_t lane[kLanes] = {};   // [0] stays nullptr: the caller's stream
  hipEvent_t tie[kLanes] = {};     // [0] the start of a chunk, then each lane's end
  char *ws = nullptr;
  size_t ws_bytes = 0;
  int max_inst = 0;
  lbm_host::Arena arena;
  struct Inst {
    lbm_handle *h = nullptr;  // nullptr: free id
    size_t off = 0, bytes = 0;
    int64_t remaining = 0;
    int up_steps = -1, up_parity = -1;  // what the device descriptor holds
  };
  std::vector<Inst> inst;
  // device metadata (from the workspace) and pinned host staging
  size_t meta_off = 0, meta_bytes = 0;
  char *d_desc[3] = {nullptr, nullptr, nullptr};
  int *d_count = nullptr;
  TileRef *d_tiles = nullptr;
  size_t tiles_off = 0, tiles_cap = 0;
  char *h_desc[3] = {nullptr, nullptr, nullptr};
  int *h_count = nullptr;
  TileRef *h_tiles = nullptr;
  size_t h_tiles_cap = 0;
  int class_off[kClasses] = {}, class_n[kClasses] = {};
  bool tiles_dirty = true;
  lbm_schedule sched = {0, 0, 32, 0};
  int cus = 256;
  std::map<std::string, hipGraphExec_t> graphs;
  std::string err;
};

namespace {

lbm_status bfail(const lbm_batch *b, lbm_status s, const std::string &msg) {
  if (b)
    const_cast<lbm_batch *>(b)->err = msg;
  else
    g_create_error = msg;
  return s;
}

lbm_status bhip(lbm_batch *b, hipError_t e, const char *what) {
  if (e == hipSuccess) return LBM_OK;
  return bfail(b, LBM_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

void clear_graphs(lbm_batch *b) {
  for (auto &kv : b->graphs) (void)hipGraphExecDestroy(kv.second);
  b->graphs.clear();
}

size_t meta_bytes_for(int max_inst) {
  size_t m = 0;
  for (int p = 0; p < 3; ++p) m += align_up(desc_size(p) * size_t(max_inst), 256);
  return m + align_up(sizeof(int) * kClasses, 256);
}

// Rebuild the tile lists (after a change of membership or schedule):
// simulations grouped by kernel variant, each strip-major.
lbm_status rebuild_tiles(lbm_batch *b) {
  size_t total = 0;
  for (auto &in : b->inst) {
    if (!in.h) continue;
    lbm_handle *h = in.h;
    h->rows = b->sched.rows > 0 ? b->sched.rows : default_rows(h->p, true);
    const size_t strips = strips_of(h->p);
    total += strips * size_t((h->p.ny + h->rows - 1) / h->rows);
  }
  hipError_t e = hipStreamSynchronize(b->stream);  // staging and tiles idle
  if (e != hipSuccess) return bhip(b, e, "synchronising");
  if (total > b->tiles_cap) {  // grow the device tile list
    const size_t cap = std::max(total, 2 * b->tiles_cap);
    if (b->d_tiles) b->arena.release(b->tiles_off, b->tiles_cap * sizeof(TileRef));
    b->d_tiles = nullptr;
    b->tiles_cap = 0;
    size_t off;
    if (!b->arena.alloc_top(cap * sizeof(TileRef), &off))
      return bfail(b, LBM_ENOMEM, "workspace too small for the tile list");
    b->tiles_off = off;
    b->tiles_cap = cap;
    b->d_tiles = reinterpret_cast<TileRef *>(b->ws + off);
    clear_graphs(b);
  }
  if (total > b->h_tiles_cap) {
    const size_t cap = std::max(total, 2 * b->h_tiles_cap);
    if (b->h_tiles) (void)hipHostFree(b->h_tiles);
    b->h_tiles = nullptr;
    b->h_tiles_cap = 0;
    e = hipHostMalloc(reinterpret_cast<void **>(&b->h_tiles), cap * sizeof(TileRef));
    if (e != hipSuccess) return bhip(b, e, "allocating pinned staging");
    b->h_tiles_cap = cap;
  }
  size_t n = 0;
  for (int c = 0; c < kClasses; ++c) {
    b->class_off[c] = int(n);
    for (int id = 0; id < b->max_inst; ++id) {
      const lbm_handle *h = b->inst[id].h;
      if (!h || class_of(h) != c) continue;
      const int strips = strips_of(h->p);
      const int chunks = (h->p.ny + h->rows - 1) / h->rows;
      for (int ch = 0; ch < chunks; ++ch)
        for (int st = 0; st < strips; ++st) b->h_tiles[n++] = TileRef{id, st, ch, 0};
    }
    b->class_n[c] = int(n) - b->class_off[c];
    b->h_count[c] = b->class_n[c];
  }
  if (n) {
    e = hipMemcpyAsync(b->d_tiles, b->h_tiles, n * sizeof(TileRef), hipMemcpyHostToDevice,
                       b->stream);
    if (e != hipSuccess) return bhip(b, e, "uploading tiles");
  }
  e = hipMemcpyAsync(b->d_count, b->h_count, sizeof(int) * kClasses, hipMemcpyHostToDevice,
                     b->stream);
  if (e != hipSuccess) return bhip(b, e, "uploading tile counts");
  for (auto &in : b->inst) in.up_steps = -1;  // rows may have changed
  b->tiles_dirty = false;
  return LBM_OK;
}

// Upload the descriptors of simulations whose (parity, steps this chunk)
// changed.  Synchronises only when something must be written.
lbm_status update_descs(lbm_batch *b, int K) {
  bool need = false;
  for (auto &in : b->inst)
    if (in.h && (in.up_steps != int(std::min<int64_t>(K, in.remaining)) ||
                 in.up_parity != in.h->cur))
      need = true;
  if (!need) return LBM_OK;
  hipError_t e = hipStreamSynchronize(b->stream);  // staging idle
  if (e != hipSuccess) return bhip(b, e, "synchronising");
  for (int id = 0; id < b->max_inst; ++id) {
    auto &in = b->inst[id];
    if (!in.h) continue;
    const int steps = int(std::min<int64_t>(K, in.remaining));
    if (in.up_steps == steps && in.up_parity == in.h->cur) continue;
    const int p = in.h->p.precision;
    char *hd = b->h_desc[p] + size_t(id) * desc_size(p);
    switch (p) {
      case LBM_FP64: fill_desc<F64>(hd, in.h, steps); break;
      case LBM_FP32: fill_desc<F32>(hd, in.h, steps); break;
      default: fill_desc<F16>(hd, in.h, steps); break;
    }
    e = hipMemcpyAsync(b->d_desc[p] + size_t(id) * desc_size(p), hd, desc_size(p),
                       hipMemcpyHostToDevice, b->stream);
    if (e != hipSuccess) return bhip(b, e, "uploading descriptors");
    in.up_steps = steps;
    in.up_parity = in.h->cur;
  }
  return LBM_OK;
}

int class_blocks(const lbm_batch *b, int c) {
  const int waves = b->sched.grid_waves > 0 ? b->sched.grid_waves : b->class_n[c];
  const int prec = class_precision(c);
  const int wpb = prec == LBM_FP16DEV ? F16::kBlockWaves
                : prec == LBM_FP64    ? F64::kBlockWaves
                                      : F32::kBlockWaves;
  return std::max(1, (waves + wpb - 1) / wpb);
}

// The graph of K launches of each of n variants, one after the other in every
// step, captured once per (K, variants, their places in the tile list, grid
// shapes, tile storage).
lbm_status get_graph(lbm_batch *b, int K, const int *variants, int n, hipGraphExec_t *out) {
  std::string key = std::to_string(K) + ":" +
                    std::to_string(reinterpret_cast<uintptr_t>(b->d_tiles));
  for (int i = 0; i < n; ++i) {
    const int c = variants[i];
    key += ":" + std::to_string(c) + "@" + std::to_string(b->class_off[c]) + "/" +
           std::to_string(class_blocks(b, c));
  }
  auto it = b->graphs.find(key);
  if (it != b->graphs.end()) {
    *out = it->second;
    return LBM_OK;
  }
  hipError_t e = hipStreamBeginCapture(b->capture, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return bhip(b, e, "beginning graph capture");
  for (int k = 0; k < K; ++k)
    for (int i = 0; i < n; ++i) {
      const int c = variants[i];
      launch_batch_class(c, class_blocks(b, c), b->capture, b->d_desc[class_precision(c)],
                         b->d_tiles + b->class_off[c], b->d_count + c, k);
    }
  hipGraph_t g = nullptr;
  hipError_t e2 = hipGetLastError();
  e = hipStreamEndCapture(b->capture, &g);
  if (e2 != hipSuccess) e = e2;
  hipGraphExec_t x = nullptr;
  if (e == hipSuccess) e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
  if (g) (void)hipGraphDestroy(g);
  if (e != hipSuccess) return bhip(b, e, "capturing the batch graph");
  b->graphs[key] = x;
  *out = x;
  return LBM_OK;
}

// The streams and events of the first `lanes` lanes, on the device of the
// caller's stream, whatever device is current: its events are recorded there.
hipError_t make_lanes(lbm_batch *b, int lanes) {
  if (b->tie[lanes - 1]) return hipSuccess;  // made last
  int dev = 0;
  hipError_t e = hipStreamGetDevice(b->stream, &dev);
  if (e != hipSuccess) return e;
  const OnDevice on(dev);
  if (!on.ok()) return hipErrorInvalidDevice;
  for (int i = 1; i < lanes && e == hipSuccess; ++i)
    if (!b->lane[i]) e = hipStreamCreateWithFlags(&b->lane[i], hipStreamNonBlocking);
  for (int i = 0; i < lanes && e == hipSuccess; ++i)
    if (!b->tie[i]) e = hipEventCreateWithFlags(&b->tie[i], hipEventDisableTiming);
  return e;
}

// K steps of every variant present.  The simulations of different variants
// do not touch each other, and one variant alone may not fill the device, so
// they run side by side, each with a graph of its own: the largest first, each
// on the lane with the least work so far.  The caller's stream waits for all
// of them.  Measured, one after the other -> side by side: twelve served
// float32 solves (three variants of 21, 15 and 11 us per step) 18.7 -> 13.2
// ms, 22 -> 18.5 ms when the batch is new; nine float16 ones 19.0 -> 12.1 ms;
// 180 steps of 32 channels (two variants, 80 and 27 us) 19.1 -> 17.5 ms.
// Lanes and more graphs cost 20-40 us per chunk, and gain the steps of all but
// the longest variant.  us per chunk, one graph -> lanes: of 2 steps, three
// variants of one 32x32 field 101 -> 121, of two 200x200 223 -> 140; of 4, 197 ->
// 198 and 441 -> 232, but two variants of one 32x16 field 92 -> 111 and of one
// 512x256 119 -> 128; of 5, these 118 -> 118 and 151 -> 151; of 8, 166 -> 146 and
// 220 -> 204.  So two variants use them from 6 steps, three and more from 4, and
// shorter chunks stay one graph on the caller's stream.
int lane_steps(int variants) { return variants == 2 ? 6 : 4; }

lbm_status launch_chunk(lbm_batch *b, int K) {
  int order[kClasses], present = 0;
  for (int c = 0; c < kClasses; ++c)
    if (b->class_n[c]) order[present++] = c;
  std::sort(order, order + present, [&](int x, int y) {
    return b->class_n[x] != b->class_n[y] ? b->class_n[x] > b->class_n[y] : x < y;
  });
  hipError_t e = hipSuccess;
  if (b->graphs.size() + size_t(present) > 96) {
    e = hipStreamSynchronize(b->stream);  // no launch still uses them
    if (e != hipSuccess) return bhip(b, e, "synchronising");
    clear_graphs(b);
  }
  int lanes = K >= lane_steps(present) ? std::min(present, lbm_batch::kLanes) : 1;
  if (lanes > 1) {  // a caller's capture sees its own stream only
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(b->stream, &cap) != hipSuccess) {
      (void)hipGetLastError();
      lanes = 1;
    }
    if (cap != hipStreamCaptureStatusNone) lanes = 1;
  }
  if (lanes > 1 && make_lanes(b, lanes) != hipSuccess) {  // none to be had: one after the other
    (void)hipGetLastError();
    lanes = 1;
  }
  hipGraphExec_t graph[kClasses];
  const int graphs = lanes > 1 ? present : 1;
  for (int i = 0; i < graphs; ++i) {
    const lbm_status st = get_graph(b, K, order + i, lanes > 1 ? 1 : present, &graph[i]);
    if (st != LBM_OK) return st;
  }
  if (lanes > 1) e = hipEventRecord(b->tie[0], b->stream);
  for (int i = 1; i < lanes && e == hipSuccess; ++i)
    e = hipStreamWaitEvent(b->lane[i], b->tie[0], 0);
  long long load[lbm_batch::kLanes] = {};
  bool started[kClasses] = {};  // on lanes: the variants whose steps are enqueued
  for (int i = 0; i < graphs && e == hipSuccess; ++i) {
    const int to = int(std::min_element(load, load + lanes) - load);
    load[to] += b->class_n[order[i]];
    e = hipGraphLaunch(graph[i], to ? b->lane[to] : b->stream);
    started[order[i]] = lanes > 1 && e == hipSuccess;
  }
  // Also after an error: what was started has to end before the caller's
  // stream goes on.
  for (int i = 1; i < lanes; ++i) {
    hipError_t e2 = hipEventRecord(b->tie[i], b->lane[i]);
    if (e2 == hipSuccess) e2 = hipStreamWaitEvent(b->stream, b->tie[i], 0);
    if (e2 != hipSuccess) (void)hipStreamSynchronize(b->lane[i]);
    if (e == hipSuccess) e = e2;
  }
  // Of a chunk that failed, the started variants step on the device all the
  // same: their simulations are no longer where they were, nor known to be a
  // chunk further.
  for (auto &in : b->inst)
    if (e != hipSuccess && in.h && in.remaining > 0 && started[class_of(in.h)]) {
      in.h->valid = false;
      in.remaining = 0;
    }
  return bhip(b, e, "launching the batch graphs");
}

bool schedule_ok(const lbm_schedule *s) {
  return s && s->rows >= 0 && s->rows <= 4096 && s->grid_waves >= 0 &&
         s->grid_waves <= (1 << 22) && s->chunk >= 1 && s->chunk <= 1024 && s->reserved == 0;
}

}  // namespace

extern "C" {

size_t lbm_batch_instance_bytes(const lbm_params *params) {
  return lbm_workspace_bytes(params);
}

size_t lbm_batch_overhead_bytes(int32_t max_instances) {
  if (max_instances < 1 || max_instances > 65536) return 0;
  return meta_bytes_for(max_instances);
}

lbm_status lbm_batch_create(int32_t max_instances, void *dev_ws, size_t ws_bytes,
                            void *hip_stream, lbm_batch **out) {
  if (!out) return bfail(nullptr, LBM_EINVAL, "out is NULL");
  *out = nullptr;
  if (max_instances < 1 || max_instances > 65536)
    return bfail(nullptr, LBM_EINVAL, "max_instances must be in 1..65536");
  if (!dev_ws) return bfail(nullptr, LBM_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(dev_ws) % 256)
    return bfail(nullptr, LBM_EINVAL, "workspace must be 256-byte aligned");
  const size_t meta = meta_bytes_for(max_instances);
  if (ws_bytes < meta) return bfail(nullptr, LBM_ENOMEM, "workspace smaller than metadata");
  lbm_batch *b = new (std::nothrow) lbm_batch();
  if (!b) return bfail(nullptr, LBM_ENOMEM, "out of host memory");
  b->stream = static_cast<hipStream_t>(hip_stream);
  b->ws = static_cast<char *>(dev_ws);
  b->ws_bytes = ws_bytes;
  b->max_inst = max_instances;
  b->inst.resize(max_instances);
  b->arena.reset(ws_bytes);
  size_t off = 0;
  b->arena.alloc(meta, &off);  // first block: offset 0
  b->meta_off = off;
  b->meta_bytes = meta;
  size_t o = off;
  for (int p = 0; p < 3; ++p) {
    b->d_desc[p] = b->ws + o;
    o += align_up(desc_size(p) * size_t(max_instances), 256);
  }
  b->d_count = reinterpret_cast<int *>(b->ws + o);
  hipError_t e = hipSuccess;
  for (int p = 0; p < 3 && e == hipSuccess; ++p)
    e = hipHostMalloc(reinterpret_cast<void **>(&b->h_desc[p]),
                      desc_size(p) * size_t(max_instances));
  if (e == hipSuccess)
    e = hipHostMalloc(reinterpret_cast<void **>(&b->h_count), sizeof(int) * kClasses);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->capture, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->admit, hipStreamNonBlocking);
  int dev = 0;
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess)
    e = hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) {
    const std::string m = std::string("creating the batch: ") + hipGetErrorString(e);
    lbm_batch_destroy(b);
    return bfail(nullptr, LBM_EDEVICE, m);
  }
  *out = b;
  return LBM_OK;
}

lbm_status lbm_batch_submit(lbm_batch *b, const lbm_params *params, const double *phi,
                            const double *psi, const double *ux, const double *uy,
                            int64_t nsteps, int32_t *id) {
  if (!b) return LBM_EINVAL;
  if (!id) return bfail(b, LBM_EINVAL, "id is NULL");
  if (nsteps < 0) return bfail(b, LBM_EINVAL, "nsteps < 0");
  if (const char *m = validate(params)) return bfail(b, LBM_EINVAL, m);
  int slot = -1;
  for (int i = 0; i < b->max_inst; ++i)
    if (!b->inst[i].h) {
      slot = i;
      break;
    }
  if (slot < 0) return bfail(b, LBM_ENOMEM, "no free simulation id");
  const size_t bytes = lbm_workspace_bytes(params);
  size_t off;
  if (!b->arena.alloc(bytes, &off))
    return bfail(b, LBM_ENOMEM, "not enough contiguous free workspace");
  // The new simulation's fields are copied in and initialised on the
  // batch's admission stream, so the simulations already stepping on the
  // caller's stream keep running meanwhile.  Its block of the workspace is
  // free of device work: a retire releases a block only after the stream
  // has finished every launch that used it.  It joins the launches of the
  // next lbm_batch_step, which are enqueued after this call has waited for
  // the initialisation to complete.
  lbm_handle *h = nullptr;
  lbm_status st = lbm_create(params, b->ws + off, bytes, b->admit, &h);
  if (st == LBM_OK) {
    h->of_batch = true;
    st = lbm_init_fields(h, phi, psi, ux, uy);
    if (st != LBM_OK) {
      bfail(b, st, h->err);
      lbm_destroy(h);
      h = nullptr;
    }
  } else {
    bfail(b, st, g_create_error);
  }
  if (st != LBM_OK) {
    b->arena.release(off, bytes);
    return st;
  }
  h->stream = b->stream;  // reads and steps from now on go to the caller's stream
  auto &in = b->inst[slot];
  in.h = h;
  in.off = off;
  in.bytes = bytes;
  in.remaining = nsteps;
  in.up_steps = in.up_parity = -1;
  b->tiles_dirty = true;
  *id = slot;
  return LBM_OK;
}

lbm_status lbm_batch_step(lbm_batch *b, int64_t nsteps) {
  if (!b) return LBM_EINVAL;
  if (nsteps < 0) return bfail(b, LBM_EINVAL, "nsteps < 0");
  while (nsteps > 0) {
    int64_t most = 0;
    for (auto &in : b->inst)
      if (in.h) most = std::max(most, in.remaining);
    if (most == 0) break;  // nothing left to run
    if (b->tiles_dirty) {
      lbm_status st = rebuild_tiles(b);
      if (st != LBM_OK) return st;
    }
    const int K = int(std::min<int64_t>({nsteps, int64_t(b->sched.chunk), most}));
    lbm_status st = update_descs(b, K);
    if (st != LBM_OK) return st;
    st = launch_chunk(b, K);
    if (st != LBM_OK) return st;
    for (auto &in : b->inst) {
      if (!in.h) continue;
      const int s = int(std::min<int64_t>(K, in.remaining));
      in.h->cur ^= s & 1;
      in.h->step += s;
      in.remaining -= s;
    }
    nsteps -= K;
  }
  return LBM_OK;
}

lbm_status lbm_batch_remaining(const lbm_batch *b, int32_t id, int64_t *remaining) {
  if (!b) return LBM_EINVAL;
  if (!remaining || id < 0 || id >= b->max_inst || !b->inst[id].h)
    return bfail(b, LBM_EINVAL, "unknown simulation id");
  *remaining = b->inst[id].remaining;
  return LBM_OK;
}

lbm_status lbm_batch_read_fields(lbm_batch *b, int32_t id, double *phi, double *psi,
                                 double *ux, double *uy, double *P) {
  if (!b) return LBM_EINVAL;
  if (id < 0 || id >= b->max_inst || !b->inst[id].h)
    return bfail(b, LBM_EINVAL, "unknown simulation id");
  lbm_handle *h = b->inst[id].h;
  lbm_status st = lbm_read_fields(h, phi, psi, ux, uy, P);
  if (st != LBM_OK) bfail(b, st, h->err);
  return st;
}

lbm_status lbm_batch_moments(lbm_batch *b, int32_t id, lbm_moments_t *out) {
  if (!b) return LBM_EINVAL;
  if (id < 0 || id >= b->max_inst || !b->inst[id].h)
    return bfail(b, LBM_EINVAL, "unknown simulation id");
  lbm_handle *h = b->inst[id].h;
  lbm_status st = lbm_moments(h, out);
  if (st != LBM_OK) bfail(b, st, h->err);
  return st;
}

lbm_status lbm_batch_shape(lbm_batch *b, int32_t id, lbm_shape_t *out) {
  if (!b) return LBM_EINVAL;
  if (id < 0 || id >= b->max_inst || !b->inst[id].h)
    return bfail(b, LBM_EINVAL, "unknown simulation id");
  lbm_handle *h = b->inst[id].h;
  lbm_status st = lbm_shape(h, out);
  if (st != LBM_OK) bfail(b, st, h->err);
  return st;
}

lbm_status lbm_batch_retire(lbm_batch *b, int32_t id) {
  if (!b) return LBM_EINVAL;
  if (id < 0 || id >= b->max_inst || !b->inst[id].h)
    return bfail(b, LBM_EINVAL, "unknown simulation id");
  hipError_t e = hipStreamSynchronize(b->stream);  // no launch still uses it
  if (e != hipSuccess) return bhip(b, e, "synchronising");
  auto &in = b->inst[id];
  lbm_destroy(in.h);
  b->arena.release(in.off, in.bytes);
  in = lbm_batch::Inst();
  b->tiles_dirty = true;
  return LBM_OK;
}

size_t lbm_batch_free_bytes(const lbm_batch *b) { return b ? b->arena.largest() : 0; }

lbm_status lbm_batch_set_schedule(lbm_batch *b, const lbm_schedule *s) {
  if (!b) return LBM_EINVAL;
  if (!schedule_ok(s)) return bfail(b, LBM_EINVAL, "schedule out of range");
  b->sched = *s;
  b->tiles_dirty = true;
  return LBM_OK;
}

lbm_status lbm_batch_get_schedule(const lbm_batch *b, lbm_schedule *s) {
  if (!b) return LBM_EINVAL;
  if (!s) return bfail(b, LBM_EINVAL, "s is NULL");
  *s = b->sched;
  return LBM_OK;
}

lbm_status lbm_batch_autotune(lbm_batch *b, int64_t probe_steps, lbm_schedule *chosen) {
  if (!b) return LBM_EINVAL;
  if (probe_steps < 1) return bfail(b, LBM_EINVAL, "probe_steps < 1");
  const lbm_schedule keep = b->sched;
  std::vector<lbm_schedule> cands;
  for (int rows : {0, 4, 8, 16})
    for (int per_cu : {0, 4, 8, 16})
      cands.push_back(lbm_schedule{rows, per_cu * b->cus, keep.chunk, 0});
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) return bhip(b, e, "creating events");
  lbm_schedule best = keep;
  double best_t = -1.0;
  lbm_status st = LBM_OK;
  for (const auto &c : cands) {
    b->sched = c;
    b->tiles_dirty = true;
    double work = 0.0;  // site updates in the timed probe
    for (auto &in : b->inst)
      if (in.h)
        work += double(in.h->p.nx) * in.h->p.ny * double(std::min(probe_steps, in.remaining));
    if (work == 0.0) break;
    st = lbm_batch_step(b, std::min<int64_t>(probe_steps, c.chunk));  // builds graphs
    if (st != LBM_OK) break;
    work = 0.0;
    for (auto &in : b->inst)
      if (in.h)
        work += double(in.h->p.nx) * in.h->p.ny * double(std::min(probe_steps, in.remaining));
    if (work == 0.0) break;
    e = hipEventRecord(e0, b->stream);
    if (e == hipSuccess) st = lbm_batch_step(b, probe_steps);
    if (e == hipSuccess && st == LBM_OK) e = hipEventRecord(e1, b->stream);
    if (e == hipSuccess && st == LBM_OK) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess && st == LBM_OK) e = hipEventElapsedTime(&ms, e0, e1);
    if (e != hipSuccess || st != LBM_OK) break;
    const double t = double(ms) / work;
    if (best_t < 0.0 || t < best_t) {
      best_t = t;
      best = c;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (e != hipSuccess) {
    b->sched = keep;
    b->tiles_dirty = true;
    return bhip(b, e, "timing the autotuner probes");
  }
  if (st != LBM_OK) {
    b->sched = keep;
    b->tiles_dirty = true;
    return st;
  }
  b->sched = best;
  b->tiles_dirty = true;
  if (chosen) *chosen = best;
  return LBM_OK;
}

void lbm_batch_destroy(lbm_batch *b) {
  if (!b) return;
  (void)hipStreamSynchronize(b->stream);
  clear_graphs(b);
  for (auto &in : b->inst)
    if (in.h) lbm_destroy(in.h);
  for (int p = 0; p < 3; ++p)
    if (b->h_desc[p]) (void)hipHostFree(b->h_desc[p]);
  if (b->h_count) (void)hipHostFree(b->h_count);
  if (b->h_tiles) (void)hipHostFree(b->h_tiles);
  for (hipStream_t st : b->lane)
    if (st) (void)hipStreamDestroy(st);
  for (hipEvent_t ev : b->tie)
    if (ev) (void)hipEventDestroy(ev);
  if (b->capture) (void)hipStreamDestroy(b->capture);
  if (b->admit) (void)hipStreamDestroy(b->admit);
  delete b;
}

const char *lbm_batch_last_error(const lbm_batch *b) {
  return b ? b->err.c_str() : g_create_error.c_str();
}

}  // extern "C"

#endif  // LBM_F16_PART
