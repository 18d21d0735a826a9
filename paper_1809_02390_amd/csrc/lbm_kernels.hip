// HIP kernels and C-ABI entry points of the self-tuning-EOS D2Q9 library
// (gfx950).  See include/lbm.h for the contract of every entry point.
//
// Data layout, x fastest.  State buffers (state_layout) interleave rows,
// population i of node (x, y) at element (9 y + i) nx + x (FP32 states
// larger than 4 GiB are read with band-relative or 64-bit offsets,
// wide_state).  The adjoint state interleaves its eleven fields the same
// way when its offsets fit 32 bits, else it holds eleven planes P =
// plane_elems apart (nx*ny rounded up to 64 plus a pad, so that the planes
// do not start at one offset modulo a large power of two); the 2-byte
// reference densities and the caller's plain arrays hold planes of nx*ny.  Two caller-owned
// buffers A and B alternate; the buffer that is
// read by the next step holds the post-collision populations of the previous
// step at their source node ("pull" streaming: f_i(x, t) = src_i(x - e_i)).
//
// Storages (one template parameter of every kernel):
//   F32   f-bar stored as float;
//   F16 / BF16  f-bar stored in two bytes as S (f-bar - f_ref), with f_ref the
//         rest equilibrium at the reference density rho~ of the node the
//         population streams to.  rho~ is that node's density of the previous
//         step in binary16, kept in two planes that alternate like A and B.
//         The encoder takes the neighbour densities from the LDS tile it
//         already holds for the force stencil; the decoder reads its own rho~.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "lbm.h"
#include "lbm_cell.h"
#include "lbm_internal.h"

namespace lbm {
namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return code;
}

#define HIP_OK(expr)                                                                    \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return fail(LBM_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// ---------------------------------------------------------------------------
// Velocity set (supplement Eq. 3) as compile-time tables
// ---------------------------------------------------------------------------
constexpr int kCx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int kCy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// ---------------------------------------------------------------------------
// Storage policies
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint16_t f32_to_f16(float v) { return __half_as_ushort(__float2half_rn(v)); }
__device__ __forceinline__ float f16_to_f32(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// binary32 -> bfloat16, round to nearest even (one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t f32_to_bf16(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// The reference density rho~ of a node: its density rounded to binary16.
__device__ __forceinline__ float ref_density(float rho) { return f16_to_f32(f32_to_f16(rho)); }

struct StoreF32 {
  using E = float;
  static constexpr int ES = 4;
  static constexpr bool kRef = false;
};

template <int KIND>
struct Store16 {
  using E = uint16_t;
  static constexpr int ES = 2;
  static constexpr bool kRef = true;
  __device__ static float to_f32(uint16_t h) { return KIND == LBM_FP16 ? f16_to_f32(h) : bf16_to_f32(h); }
  __device__ static uint16_t from_f32(float v) { return KIND == LBM_FP16 ? f32_to_f16(v) : f32_to_bf16(v); }
};

// ---------------------------------------------------------------------------
// Addressing: per-plane base pointers (uniform) and 32-bit byte offsets
// ---------------------------------------------------------------------------
// i mod n.  Tile coordinates lie within one period of [0, n) except on
// lattices narrower than a tile, which alone take the integer division.
__device__ __forceinline__ int wrap(int i, int n) {
  if (i >= n)
    i -= n;
  else if (i < 0)
    i += n;
  if ((unsigned)i >= (unsigned)n) {
    i %= n;
    if (i < 0) i += n;
  }
  return i;
}

// Row offsets (row * rp * ES, rp the row pitch) of rows y, y-1, y+1 and column offsets
// (x * ES) of columns x, x-1, x+1 of a node, periodic.
template <int ES>
struct NodeAddr {
  unsigned r0, rm, rp, c0, cm, cp;
};

// One multiplication per node; the neighbours' offsets are the node's plus
// or minus one row (column), or the opposite edge.
template <int ES>
__device__ __forceinline__ NodeAddr<ES> node_addr(int x, int y, int nx, int ny, unsigned rp, int yb = 0) {
  // rows relative to row yb; with yb > 0 (band addressing) y never wraps
  const unsigned rb = ES * rp, r0 = rb * (unsigned)(y - yb), rlast = rb * (unsigned)(ny - 1 - yb);
  const unsigned c0 = ES * (unsigned)x, clast = ES * (unsigned)(nx - 1);
  return {r0, y == 0 ? rlast : r0 - rb, y == ny - 1 ? rb * (unsigned)(-yb) : r0 + rb,
          c0, x == 0 ? clast : c0 - ES, x == nx - 1 ? 0u : c0 + ES};
}

template <typename E>
__device__ __forceinline__ E ldb(const char* __restrict__ base, unsigned off) {
  return *reinterpret_cast<const E*>(base + off);
}

// Store that is left in the caches (kStream false) or streamed past them.
template <bool kStream, typename E>
__device__ __forceinline__ void put(E v, char* base, unsigned off) {
  E* p = reinterpret_cast<E*>(base + off);
  if constexpr (kStream)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <typename E>
struct Planes {
  const char* p[9];
};

template <typename E>
__device__ __forceinline__ Planes<E> planes(const void* src, size_t N) {
  Planes<E> P;
#pragma unroll
  for (int i = 0; i < 9; ++i) P.p[i] = reinterpret_cast<const char*>(reinterpret_cast<const E*>(src) + (size_t)i * N);
  return P;
}

template <typename E>
struct OutPlanes {
  char* p[9];
};

template <typename E>
__device__ __forceinline__ OutPlanes<E> out_planes(void* dst, size_t N) {
  OutPlanes<E> P;
#pragma unroll
  for (int i = 0; i < 9; ++i) P.p[i] = reinterpret_cast<char*>(reinterpret_cast<E*>(dst) + (size_t)i * N);
  return P;
}

// Elements from one plane of an internal buffer (A/B state, checkpoint,
// adjoint state) to the next: nx*ny rounded up to 64, plus LBM_PLANE_PAD
// bytes, so that the planes do not all start at one offset modulo a large
// power of two (the streams of the nine planes then spread over the HBM
// channels).  The 2-byte reference planes and the caller's plain arrays use
// nx*ny.
#ifndef LBM_PLANE_PAD
#define LBM_PLANE_PAD 16640
#endif
__host__ __device__ __forceinline__ size_t plane_elems(int nx, int ny, int es) {
  return ((size_t)nx * ny + 63) / 64 * 64 + (size_t)(LBM_PLANE_PAD / es);
}

// Layout of a state buffer (A/B, checkpoint): elements from one population
// to the next (ps) and from one lattice row to the next (rp).  States
// interleave rows -- the nine populations of a lattice row are nine
// consecutive buffer rows, population i of node (x, y) at (9 y + i) nx + x.
// A wave's nine loads (stores) of a row segment then fall within 9 nx
// elements instead of nine planes apart, which keeps more of them in open
// DRAM pages (a data-movement kernel with the step's access pattern moves
// 3-6 % more bytes per second; the FP32 step gains 7 % at 4096^2, the
// 2-byte steps 1 %).
struct Layout {
  size_t ps;    // elements between populations
  unsigned rp;  // elements between lattice rows
};
__host__ __device__ __forceinline__ Layout state_layout(int nx, int, int) { return {(size_t)nx, 9u * (unsigned)nx}; }

// Byte offsets of a state from uniform bases fit the 32-bit lane offsets
// when 9 es nx ny < 2^32 (always for the 2-byte storages; FP32 lattices up
// to 119M nodes): kAbs.  Larger FP32 states are read per tile relative to
// the band of rows the tile reads (kBand: tile rows whose halo stays inside
// the lattice) or with 64-bit addresses (kWide: the tile rows that wrap),
// in two launches, so that the wide path adds no registers to the kernel
// that runs nearly every tile.
enum { kAbs = 0, kBand = 1, kWide = 2 };
__host__ __device__ __forceinline__ bool wide_state(int nx, int ny, int es) {
  return 9ull * (unsigned long long)es * (unsigned long long)nx * (unsigned long long)ny > 0xFFFFFFFFull;
}

// Tile rows of one launch: local tile row r is row r0 + r for r < na, else
// r1 + (r - na) (the wide launch takes the rows at both ends).
struct TileRows {
  int r0, na, r1;
};
__device__ __forceinline__ int tile_row(const TileRows& t, int r) { return r < t.na ? t.r0 + r : t.r1 + (r - t.na); }

// Layout of an adjoint state buffer: eleven fields (L_0..L_8, A_x, A_y)
// with rows interleaved like the FP32 state when every byte offset fits 32
// bits (44 nx ny < 2^32), else eleven planes plane_elems apart.
__host__ __device__ __forceinline__ Layout adj_layout(int nx, int ny) {
  if (44ull * (unsigned long long)nx * (unsigned long long)ny <= 0xFFFFFFFFull)
    return {(size_t)nx, 11u * (unsigned)nx};
  return {plane_elems(nx, ny, 4), (unsigned)nx};
}

// Raw stored values arriving at a node: raw_i = src_i(x - e_i).
template <typename E>
__device__ __forceinline__ void pull_raw(const Planes<E>& P, const NodeAddr<sizeof(E)>& a, E* r) {
  r[0] = ldb<E>(P.p[0], a.r0 + a.c0);
  r[1] = ldb<E>(P.p[1], a.r0 + a.cm);
  r[2] = ldb<E>(P.p[2], a.rm + a.c0);
  r[3] = ldb<E>(P.p[3], a.r0 + a.cp);
  r[4] = ldb<E>(P.p[4], a.rp + a.c0);
  r[5] = ldb<E>(P.p[5], a.rm + a.cm);
  r[6] = ldb<E>(P.p[6], a.rm + a.cp);
  r[7] = ldb<E>(P.p[7], a.rp + a.cp);
  r[8] = ldb<E>(P.p[8], a.rp + a.cm);
}

// Populations arriving at node (x, y) from a row-interleaved FP32 state,
// any node (periodic wrap), with 64-bit addresses (kWide).
__device__ __forceinline__ void pull_rows(const char* __restrict__ base, int x, int y, int nx, int ny, float* r) {
  const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
  const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const int row[9] = {y, y, ym, y, yp, ym, ym, yp, yp};  // source of population i: (x, y) - e_i
  const int col[9] = {x, xm, x, xp, x, xm, xp, xp, xm};
#pragma unroll
  for (int i = 0; i < 9; ++i)
    r[i] = *reinterpret_cast<const float*>(base + 4 * (((size_t)row[i] * 9 + i) * nx + col[i]));
}

// Decode the raw values of a node into f_i (FP32).  rref is the node's
// stored reference density (binary16 bits; ignored for F32).
template <class St>
__device__ __forceinline__ void decode(const typename St::E* r, uint16_t rref, const RefPoly<float>& q, float* f) {
  if constexpr (St::kRef) {
    const float rt = f16_to_f32(rref);
    const float ref[3] = {ref_value(q, 0, rt), ref_value(q, 1, rt), ref_value(q, 2, rt)};
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = ref[velocity_class(i)] + St::to_f32(r[i]) * q.inv_scale;
  } else {
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = r[i];
  }
}

// Encode f-bar_i of one node given the reference densities of the nine
// nodes its populations stream to (index i: x + e_i).
template <class St>
__device__ __forceinline__ void encode(const float* f, const float* rdest, const RefPoly<float>& q,
                                       typename St::E* out) {
  if constexpr (St::kRef) {
#pragma unroll
    for (int i = 0; i < 9; ++i) out[i] = St::from_f32((f[i] - ref_value(q, velocity_class(i), rdest[i])) * q.scale);
  } else {
#pragma unroll
    for (int i = 0; i < 9; ++i) out[i] = f[i];
  }
}

// ---------------------------------------------------------------------------
// Tiles: TX x TY nodes per workgroup of TX x WY threads; each thread owns
// NPT = TY/WY nodes of one column.  The tile plus a one-node ring of
// densities is staged in LDS for the force stencil; ring nodes pull their
// own populations (L2 hits: neighbouring tiles run on the same XCD).
// ---------------------------------------------------------------------------
template <int TX_, int TY_, int WY_>
struct TileShape {
  static constexpr int TX = TX_, TY = TY_, WY = WY_, NPT = TY / WY, LW = TX + 2;
  static constexpr int NRING = 2 * LW + 2 * TY, NTHREADS = TX * WY, LDS = (TY + 2) * LW;
  static_assert(TY % WY == 0, "rows per thread");
  static_assert(NRING <= NTHREADS, "one ring node per thread");
};

// Tiles of the step kernel (TX, TY, WY), per storage; compile-time tuning
// knobs.  StepTile on lattices beyond the caches (launch_step): FP32 (bound
// by HBM) 256 x 8 in 1024-thread workgroups, 2-byte storages (bound by the
// vector ALU) 128 x 8 in 512, two nodes per thread.  NearTile below: one node
// per thread, so that more, shorter waves cover each other's loads.
#ifndef LBM_STEP_TILE_F32
#define LBM_STEP_TILE_F32 256, 8, 4
#endif
#ifndef LBM_STEP_TILE_16
#define LBM_STEP_TILE_16 128, 8, 4
#endif
#ifndef LBM_NEAR_TILE_F32
#define LBM_NEAR_TILE_F32 64, 4, 4
#endif
#ifndef LBM_NEAR_TILE_16
#define LBM_NEAR_TILE_16 64, 8, 8
#endif
template <class St>
using StepTile =
    std::conditional_t<St::kRef, TileShape<LBM_STEP_TILE_16>, TileShape<LBM_STEP_TILE_F32>>;
template <class St>
using NearTile =
    std::conditional_t<St::kRef, TileShape<LBM_NEAR_TILE_16>, TileShape<LBM_NEAR_TILE_F32>>;
using MomTile = TileShape<64, 16, 4>;

// Several steps per launch where that is faster; compiled with
// -DLBM_FUSE_STEPS=0 every call takes single steps.
#ifndef LBM_FUSE_STEPS
#define LBM_FUSE_STEPS 1
#endif
constexpr bool kFuseSteps = LBM_FUSE_STEPS;

// Division by a launch constant d (d >= 1): quotients of n < 2^31 from one
// high multiplication by m = floor(2^32 / d) (2^32 - 1 for d = 1), at most
// one too small, and a correction.
struct Divisor {
  unsigned d, m;
};
inline Divisor make_divisor(unsigned d) { return {d, d == 1 ? 0xFFFFFFFFu : (unsigned)((1ull << 32) / d)}; }
__device__ __forceinline__ unsigned div_mod(unsigned n, const Divisor& v, unsigned& rem) {
  unsigned q = (unsigned)(((unsigned long long)n * v.m) >> 32), r = n - q * v.d;
  if (r >= v.d) r -= v.d, ++q;
  rem = r;
  return q;
}

// Order in which a launch visits the tiles of an ntx x nty grid.
//
// Across the eight XCDs of the chip: workgroups are dealt to the XCDs
// round-robin by dispatch index, so dispatch b runs on XCD b % 8.  Each XCD
// gets one contiguous run of the order, so that the tiles whose halo lines
// overlap share that XCD's L2.
//
// Within the order: vertical strips of `strip` tile columns (1 <= strip <=
// ntx), band by band within a strip; the tile that shares a halo line with
// the tile above it comes `strip` tiles later, whatever the lattice width,
// so the line is still in L2 when it is read again.  Full strips first, then
// a narrower one.  The host passes the divisors (Divisor), so that a wave
// reaches its first load after about 30 scalar instructions and one round of
// scalar loads; dividing in the kernel took about 150, a latency in front of
// the loads of every workgroup.  Measured, us per step before and after:
// two-step kernel 44.0 / 40.8 at 2048^2, 152 / 151 at 4096^2; one-step FP32
// 206 / 199 and FP16 176 / 170 at 4096^2, FP16 53.0 / 48.6 at 2048^2;
// adjoint 9.34 / 9.01 at 512^2, 108 / 105.5 at 2048^2, 402 / 396 at 4096^2.
//
// Launches whose stores stay in the caches (stream_stores) alternate between
// the order and its reverse within each XCD: the next launch then starts on
// what the last one wrote last, which the caches still hold.  Measured, us
// per step, one order / alternating: two-step kernel 42.4 / 40.7 at 2048^2,
// 89.9 / 87.3 at 3000^2; FP16 163.5 / 158.0 at 4000^2; adjoint 116 / 109 at
// 2050 x 2047.
struct TileOrder {
  unsigned xq, xr;            // tiles / 8, tiles % 8
  unsigned reverse;           // 1: each XCD's run backwards
  unsigned full;              // full strips
  Divisor per, strip, last;   // tiles per full strip; its columns; columns of the narrower strip
};
inline TileOrder make_order(int ntx, int nty, int strip, bool reverse) {
  const unsigned n = (unsigned)ntx * nty, w = (unsigned)(ntx % strip);
  return {n >> 3, n & 7, reverse ? 1u : 0u, (unsigned)(ntx / strip), make_divisor((unsigned)strip * nty),
          make_divisor((unsigned)strip), make_divisor(w ? w : 1)};
}

// Tile (tx, ty) of dispatch b: a bijection onto the grid for any ntx, nty.
// Without branches, so that the launch constants arrive in one round of
// scalar loads.  Returns the dispatch that visits the tile in the forward
// order: one number per tile, whichever way the launch runs.
__device__ __forceinline__ unsigned order_tile(unsigned b, const TileOrder& o, int& tx, int& ty) {
  const unsigned xcd = b & 7, last = o.xq - (xcd < o.xr ? 0u : 1u);
  const unsigned l = (b >> 3) + o.reverse * (last - 2u * (b >> 3));
  const unsigned t = xcd * o.xq + (xcd < o.xr ? xcd : o.xr) + l;
  unsigned rem, c;
  const unsigned s = div_mod(t, o.per, rem);
  const bool narrow = s >= o.full;
  const Divisor v = {narrow ? o.last.d : o.strip.d, narrow ? o.last.m : o.strip.m};
  ty = (int)div_mod(rem, v, c);
  tx = (int)(s * o.strip.d + c);
  return l << 3 | xcd;
}

// Coordinates (hx, hy) in the (TY+2) x LW density tile of ring slot t:
// slots [0, LW) the top row, [LW, 2 LW) the bottom row, then the left and
// the right column (TY nodes each).  Selects rather than branches: every
// ring thread of a wave takes the same instructions.
template <class S>
__device__ __forceinline__ void ring_slot(int t, int& hx, int& hy) {
  const bool row = t < 2 * S::LW, bottom = t >= S::LW, right = t >= 2 * S::LW + S::TY;
  const int c = t - 2 * S::LW - (right ? S::TY : 0);  // column slots: row index - 1
  hx = row ? (bottom ? t - S::LW : t) : (right ? S::LW - 1 : 0);
  hy = row ? (bottom ? S::TY + 1 : 0) : c + 1;
}

// Stored values of one tile held in registers: NPT own nodes per thread and,
// for the first NRING threads, one ring node; plus their reference densities.
template <class S, class St>
struct TileRegs {
  typename St::E raw[S::NPT][9];
  typename St::E rraw[9];
  uint16_t rref[S::NPT];
  uint16_t rrref;
};

// Whether the tile at (x0, y0), its ring and the ring's pull sources lie
// inside the lattice without wrapping (the common case on large lattices).
template <class S>
__device__ __forceinline__ bool interior_tile(int x0, int y0, int nx, int ny) {
  return x0 >= 2 && y0 >= 2 && x0 + S::TX + 2 <= nx && y0 + S::TY + 2 <= ny;
}

// Issue the loads of the tile at (x0, y0); ring loads first.  P holds the
// population bases of lattice row yb (0, or the tile's band origin y0 - 2
// for kBand); offsets count rows from there.  kInterior (interior_tile
// true): every population's pull shift goes into its uniform base, so the
// nine loads of a node share one offset register.  kWideAddr: 64-bit
// addresses from the state's base P.p[0] (FP32, rows that wrap).  kRing
// false: the own nodes only.
template <class S, class St, bool kInterior = false, bool kWideAddr = false, bool kRing = true>
__device__ __forceinline__ void issue_tile(const Planes<typename St::E>& P, const uint16_t* __restrict__ rho_ref,
                                           int nx, int ny, int x0, int y0, int yb, TileRegs<S, St>& R) {
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * S::TX + tx;
  if constexpr (kWideAddr) {
    static_assert(sizeof(typename St::E) == 4 && !St::kRef, "64-bit addressing is for FP32 states");
    if (kRing && tid < S::NRING) {
      int hx, hy;
      ring_slot<S>(tid, hx, hy);
      pull_rows(P.p[0], wrap(x0 + hx - 1, nx), wrap(y0 + hy - 1, ny), nx, ny, R.rraw);
    }
    const int xw = wrap(x0 + tx, nx);
#pragma unroll
    for (int k = 0; k < S::NPT; ++k) pull_rows(P.p[0], xw, wrap(y0 + ty + k * S::WY, ny), nx, ny, R.raw[k]);
    return;
  } else if constexpr (kInterior) {
    using E = typename St::E;
    const unsigned rb = St::ES * state_layout(nx, ny, St::ES).rp;
    Planes<E> Q;  // Q_i + offset(x) = P_i + offset(x - e_i)
#pragma unroll
    for (int i = 0; i < 9; ++i) Q.p[i] = P.p[i] - (ptrdiff_t)kCy[i] * rb - kCx[i] * St::ES;
    const char* rref = reinterpret_cast<const char*>(rho_ref);  // reference plane, row pitch 2 nx bytes
    if (kRing && tid < S::NRING) {
      int hx, hy;
      ring_slot<S>(tid, hx, hy);
      const unsigned off = (unsigned)(y0 + hy - 1 - yb) * rb + (unsigned)(x0 + hx - 1) * St::ES;
#pragma unroll
      for (int i = 0; i < 9; ++i) R.rraw[i] = ldb<E>(Q.p[i], off);
      if constexpr (St::kRef) R.rrref = ldb<uint16_t>(rref, 2u * ((unsigned)(y0 + hy - 1) * nx + (unsigned)(x0 + hx - 1)));
    }
    const unsigned off0 = (unsigned)(y0 + ty - yb) * rb + (unsigned)(x0 + tx) * St::ES;
#pragma unroll
    for (int k = 0; k < S::NPT; ++k) {
      const unsigned off = off0 + (unsigned)(k * S::WY) * rb;
#pragma unroll
      for (int i = 0; i < 9; ++i) R.raw[k][i] = ldb<E>(Q.p[i], off);
      if constexpr (St::kRef) R.rref[k] = ldb<uint16_t>(rref, 2u * ((unsigned)(y0 + ty + k * S::WY) * nx + (unsigned)(x0 + tx)));
    }
    // Distinct markers end the two load paths, so the compiler cannot sink
    // their last loads into the join (which would force 64-bit per-lane
    // addresses on this path).
    asm volatile("; tile loads issued: interior" ::: "memory");
    return;
  }
  if (kRing && tid < S::NRING) {
    int hx, hy;
    ring_slot<S>(tid, hx, hy);
    const int gx = wrap(x0 + hx - 1, nx), gy = wrap(y0 + hy - 1, ny);
    pull_raw<typename St::E>(P, node_addr<St::ES>(gx, gy, nx, ny, state_layout(nx, ny, St::ES).rp, yb), R.rraw);
    if constexpr (St::kRef) R.rrref = ldb<uint16_t>(reinterpret_cast<const char*>(rho_ref), 2u * ((unsigned)gy * nx + (unsigned)gx));
  }
  const int xw = wrap(x0 + tx, nx);
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    const int yw = wrap(y0 + ty + k * S::WY, ny);
    pull_raw<typename St::E>(P, node_addr<St::ES>(xw, yw, nx, ny, state_layout(nx, ny, St::ES).rp, yb), R.raw[k]);
    if constexpr (St::kRef) R.rref[k] = ldb<uint16_t>(reinterpret_cast<const char*>(rho_ref), 2u * ((unsigned)yw * nx + (unsigned)xw));
  }
  asm volatile("; tile loads issued: edge" ::: "memory");
}

// The three class values of the reference equilibrium at the reference
// density of a tile node (2-byte storages), times -S, staged for the
// encoders of the node's neighbours: sref[class * LDS + pos] (the encoder
// is then one fused multiply-add, S f + (-S f_ref)).
template <class S>
__device__ __forceinline__ void stage_ref(const RefPoly<float>& q, float rho, int pos, float* sref) {
  const float rt = ref_density(rho);
#pragma unroll
  for (int c = 0; c < 3; ++c) sref[c * S::LDS + pos] = -q.scale * ref_value(q, c, rt);
}

// Decode the tile, stage densities of the tile and its ring into
// srho[(TY+2)][LW], keep the own nodes' populations and densities in
// registers.
template <class S, class St>
__device__ __forceinline__ void stage_tile(const TileRegs<S, St>& R, const RefPoly<float>& q,
                                           float (&f)[S::NPT][9], float (&rho)[S::NPT], float* srho,
                                           float* sref) {
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * S::TX + tx;
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    decode<St>(R.raw[k], St::kRef ? R.rref[k] : 0, q, f[k]);
    rho[k] = density(f[k]);
    const int pos = (ty + k * S::WY + 1) * S::LW + tx + 1;
    srho[pos] = rho[k];
    if (St::kRef && sref) stage_ref<S>(q, rho[k], pos, sref);
  }
  if (tid < S::NRING) {
    int hx, hy;
    ring_slot<S>(tid, hx, hy);
    float fr[9];
    decode<St>(R.rraw, St::kRef ? R.rrref : 0, q, fr);
    const float r = density(fr);
    srho[hy * S::LW + hx] = r;
    if (St::kRef && sref) stage_ref<S>(q, r, hy * S::LW + hx, sref);
  }
}

// The stencil neighbours of tile position (hx, hy), indexed like the
// populations: nb[i] = rho(x + e_i) (nb[0] = rho(x)).
template <class S>
__device__ __forceinline__ void neighbours(const float* srho, int hx, int hy, float* nb) {
  const float* r = srho + hy * S::LW + hx;
#pragma unroll
  for (int i = 0; i < 9; ++i) nb[i] = r[kCy[i] * S::LW + kCx[i]];
}

// Step kernel: one tile per workgroup, tiles ordered across the XCDs by
// order_tile so that neighbouring tiles (whose halo lines overlap) run on the
// same XCD and share its L2.
template <class S, class St, int kMode, bool kStream>
__global__ __launch_bounds__(S::NTHREADS) void step_kernel(const void* __restrict__ src, void* __restrict__ dst,
                                                           const uint16_t* __restrict__ ref_in,
                                                           uint16_t* __restrict__ ref_out, int nx, int ny,
                                                           TileOrder order, Coef<float> c, RefPoly<float> q,
                                                           TileRows rows) {
  using E = typename St::E;
  __shared__ float srho[S::LDS];
  __shared__ float sref[St::kRef ? 3 * S::LDS : 1];
  const Layout L = state_layout(nx, ny, St::ES);
  const size_t N = L.ps, rowb = (size_t)St::ES * L.rp;
  int tx, ty;
  order_tile(blockIdx.x, order, tx, ty);
  const int x0 = tx * S::TX, y0 = tile_row(rows, ty) * S::TY;
  float f[S::NPT][9];
  float rho[S::NPT];
  {
    TileRegs<S, St> R;
    const int yb = kMode == kBand ? y0 - 2 : 0;  // loads: rows counted from yb
    const char* sb = static_cast<const char*>(src) + (size_t)yb * rowb;
    if constexpr (kMode == kWide)
      issue_tile<S, St, false, true>(planes<E>(src, N), ref_in, nx, ny, x0, y0, 0, R);
    else if (interior_tile<S>(x0, y0, nx, ny))
      issue_tile<S, St, true>(planes<E>(sb, N), ref_in, nx, ny, x0, y0, yb, R);
    else
      issue_tile<S, St, false>(planes<E>(sb, N), ref_in, nx, ny, x0, y0, yb, R);
    stage_tile<S, St>(R, q, f, rho, srho, St::kRef ? sref : nullptr);
  }
  __syncthreads();
  const int x = x0 + threadIdx.x;
  if (x >= nx) return;
  // stores: rows counted from row 0 (kAbs) or from the tile's first row
  const int ys = kMode == kAbs ? 0 : y0;
  const OutPlanes<E> Q = out_planes<E>(static_cast<char*>(dst) + (size_t)ys * rowb, N);
  const unsigned rb = St::ES * L.rp;
  const unsigned o0 = rb * (unsigned)(y0 - ys + threadIdx.y) + St::ES * (unsigned)x;
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    const int ly = threadIdx.y + k * S::WY, y = y0 + ly;
    if (y >= ny) break;
    float nb[9];
    neighbours<S>(srho, threadIdx.x + 1, ly + 1, nb);
    float gx, gy;
    stencil(nb[1], nb[2], nb[3], nb[4], nb[5], nb[6], nb[7], nb[8], gx, gy);
    collide_node<float, St::kRef>(f[k], rho[k], gx, gy, c);
    E out[9];
    if constexpr (St::kRef) {
      // f-bar_i streams to x + e_i: encode it against that node's reference
      const int pos = (ly + 1) * S::LW + threadIdx.x + 1;
#pragma unroll
      for (int i = 0; i < 9; ++i)
        out[i] = St::from_f32(fmaf(f[k][i], q.scale, sref[velocity_class(i) * S::LDS + pos + kCy[i] * S::LW + kCx[i]]));
    } else {
#pragma unroll
      for (int i = 0; i < 9; ++i) out[i] = f[k][i];
    }
    const unsigned o = o0 + (unsigned)(k * S::WY) * rb;
    if constexpr (St::kRef)  // 2 nx ny < 2^32 for every 2-byte state: a 32-bit offset from the plane
      *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ref_out) + 2u * ((unsigned)y * nx + (unsigned)x)) =
          f32_to_f16(nb[0]);
#pragma unroll
    for (int i = 0; i < 9; ++i) put<kStream>(out[i], Q.p[i], o);
  }
}

// ---------------------------------------------------------------------------
// Two time steps per launch (FP32 storage).  A workgroup advances a TX x TY
// tile from the state of time t to that of t + 2 without storing t + 1:
//   (A) pull f(t) onto the tile plus a three-node ring and stage the
//       densities of that region in LDS;
//   (B) collide the tile plus a two-node ring (step t), streaming each
//       post-collision population in LDS to the node it arrives at, if that
//       node lies on the tile or its one-node ring;
//   (C) form the densities of the tile and its ring at t + 1;
//   (D) collide the tile (step t + 1) and store f-bar.
// Every node is updated by the operations of step_kernel in the same order
// (density, stencil, collide_node), so two fused steps give the bits of two
// single steps.  Per two lattice updates the tile moves 36 B of each node in
// and 36 B out, half the bytes of two single steps, for (TX+4)(TY+4)
// collisions instead of TX TY in step t (64 x 24 tiles: 12 % more per
// update over the two steps), so the kernel is bound by the vector ALU
// rather than by HBM.  The tile is 64 x 24 in 512 threads (70 KB of LDS, two
// workgroups per CU; measured at 4096^2 against 64 x 16 in 256 or 512
// threads, 32 x 32, 64 x 20, 64 x 32, 128 x 16 and other thread counts).
// kMid also stores the state of t + 1 (the checkpoint driver keeps every
// state), past the caches: no launch reads it soon (1100^2, us per step,
// streamed / cached: 17.5 / 18.6; 2050 x 2048 61.2 / 64.5).
// ---------------------------------------------------------------------------
template <int TX_, int TY_, int WY_>
struct Tile2Shape {
  static constexpr int TX = TX_, TY = TY_, WY = WY_, NTHREADS = TX * WY;
  static constexpr int W1 = TX + 6, H1 = TY + 6;  // loaded region: the tile and a three-node ring
  static constexpr int KA = (H1 + WY - 1) / WY;   // loaded nodes of the tile's columns per thread
  static constexpr int NSIDE = 6 * H1;            // loaded nodes left and right of the tile's columns
  static constexpr int KD = TY / WY;              // tile nodes per thread
  // the tile and its one-node ring (positions as in TileShape: LW, ring_slot)
  static constexpr int LW = TX + 2, NRING = 2 * LW + 2 * TY, G = (TY + 2) * LW;
  static_assert(TY % WY == 0, "rows per thread");
  static_assert(NSIDE <= NTHREADS && NRING <= NTHREADS, "one side node and one ring node per thread");
};
#ifndef LBM_STEP2_TILE
#define LBM_STEP2_TILE 64, 24, 8
#endif
using Step2Tile = Tile2Shape<LBM_STEP2_TILE>;

// Whether the loaded region of the tile at (x0, y0) and its pull sources lie
// inside the lattice without wrapping.
template <class S>
__device__ __forceinline__ bool interior_tile2(int x0, int y0, int nx, int ny) {
  return x0 >= 4 && y0 >= 4 && x0 + S::TX + 4 <= nx && y0 + S::TY + 4 <= ny;
}

// Stencil gradient at position pos of an LDS density tile lw nodes wide.
template <int LWD>
__device__ __forceinline__ void stencil_at(const float* s, int pos, float& gx, float& gy) {
  float nb[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) nb[i] = s[pos + kCy[i] * LWD + kCx[i]];
  stencil(nb[1], nb[2], nb[3], nb[4], nb[5], nb[6], nb[7], nb[8], gx, gy);
}

// Stream the post-collision populations of the node at position (X, Y) of
// the loaded region to the tile-plus-ring positions they arrive at: sg[i G +
// (Y - 2 + e_iy) LW + X - 2 + e_ix], skipped where that lies outside.
template <class S, bool kCheckX>
__device__ __forceinline__ void push_node(const float* f, int X, int Y, float* sg) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int X2 = X - 2 + kCx[i], Y2 = Y - 2 + kCy[i];
    const bool in = (unsigned)Y2 < (unsigned)(S::TY + 2) && (!kCheckX || (unsigned)X2 < (unsigned)S::LW);
    if (in) sg[i * S::G + Y2 * S::LW + X2] = f[i];
  }
}

template <class S, bool kMid, bool kStream>
__global__ __launch_bounds__(S::NTHREADS) void step2_kernel(const float* __restrict__ src, float* __restrict__ mid,
                                                            float* __restrict__ dst, int nx, int ny,
                                                            TileOrder order, Coef<float> c) {
  __shared__ float s1[S::W1 * S::H1];  // densities at t of the loaded region; then at t + 1 of tile + ring
  __shared__ float sg[9 * S::G];       // populations arriving at the tile and its ring at t + 1
  const size_t rowb = (size_t)36 * nx;  // bytes from one lattice row of a state to the next
  // rb: the same in 32 bits (offsets within a tile's rows); pb: bytes from
  // one population of a row to the next
  const unsigned rb = 36u * (unsigned)nx, pb = 4u * (unsigned)nx;
  int tx, ty;
  order_tile(blockIdx.x, order, tx, ty);
  const int x0 = tx * S::TX, y0 = ty * S::TY;
  const int lx = threadIdx.x, ly = threadIdx.y, tid = ly * S::TX + lx;
  // side node of this thread: column sc of the six outside the tile's columns
  const int sY = tid / 6, sc = tid - 6 * sY, sX = sc < 3 ? sc : S::TX + sc;
  const bool side = tid < S::NSIDE;
  float fa[S::KA][9], fs[9];
  // (A) f(t) arriving at the loaded region, position (X, Y) = node (x0 - 3 + X, y0 - 3 + Y)
  if (interior_tile2<S>(x0, y0, nx, ny)) {
    // rows counted from y0 - 4; each population's pull shift in its uniform base
    const char* sb = reinterpret_cast<const char*>(src) + (size_t)(y0 - 4) * rowb;
    const char* Q[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) Q[i] = sb + (ptrdiff_t)i * pb - (ptrdiff_t)kCy[i] * rb - kCx[i] * 4;
    const unsigned o0 = (unsigned)(ly + 1) * rb + 4u * (unsigned)(x0 + lx);
#pragma unroll
    for (int k = 0; k < S::KA; ++k)
      if (k * S::WY < S::H1 - (S::WY - 1) || ly + k * S::WY < S::H1) {
        const unsigned o = o0 + (unsigned)(k * S::WY) * rb;
#pragma unroll
        for (int i = 0; i < 9; ++i) fa[k][i] = ldb<float>(Q[i], o);
      }
    if (side) {
      const unsigned o = (unsigned)(sY + 1) * rb + 4u * (unsigned)(x0 - 3 + sX);
#pragma unroll
      for (int i = 0; i < 9; ++i) fs[i] = ldb<float>(Q[i], o);
    }
    asm volatile("; two-step loads issued: interior" ::: "memory");
  } else {
    const char* base = reinterpret_cast<const char*>(src);
    const int xw = wrap(x0 + lx, nx);
#pragma unroll
    for (int k = 0; k < S::KA; ++k)
      if (k * S::WY < S::H1 - (S::WY - 1) || ly + k * S::WY < S::H1)
        pull_rows(base, xw, wrap(y0 - 3 + ly + k * S::WY, ny), nx, ny, fa[k]);
    if (side) pull_rows(base, wrap(x0 - 3 + sX, nx), wrap(y0 - 3 + sY, ny), nx, ny, fs);
    asm volatile("; two-step loads issued: edge" ::: "memory");
  }
  float ra[S::KA], rs = 0.f;
#pragma unroll
  for (int k = 0; k < S::KA; ++k) {
    const int Y = ly + k * S::WY;
    if (Y < S::H1) {
      ra[k] = density(fa[k]);
      s1[Y * S::W1 + lx + 3] = ra[k];
    }
  }
  if (side) {
    rs = density(fs);
    s1[sY * S::W1 + sX] = rs;
  }
  __syncthreads();
  // (B) step t on the tile and a two-node ring (Y in [1, H1 - 1), X in [1, W1 - 1))
#pragma unroll
  for (int k = 0; k < S::KA; ++k) {
    const int Y = ly + k * S::WY;
    if (Y >= 1 && Y < S::H1 - 1) {
      float gx, gy;
      stencil_at<S::W1>(s1, Y * S::W1 + lx + 3, gx, gy);
      collide_node<float>(fa[k], ra[k], gx, gy, c);
      push_node<S, false>(fa[k], lx + 3, Y, sg);
    }
  }
  if (side && sc >= 1 && sc <= 4 && sY >= 1 && sY < S::H1 - 1) {
    float gx, gy;
    stencil_at<S::W1>(s1, sY * S::W1 + sX, gx, gy);
    collide_node<float>(fs, rs, gx, gy, c);
    push_node<S, true>(fs, sX, sY, sg);
  }
  __syncthreads();
  // (C) densities at t + 1 of the tile (own nodes, kept in registers) and its ring
  float fd[S::KD][9], rd[S::KD];
  float* const s2 = s1;
#pragma unroll
  for (int k = 0; k < S::KD; ++k) {
    const int pos = (ly + k * S::WY + 1) * S::LW + lx + 1;
#pragma unroll
    for (int i = 0; i < 9; ++i) fd[k][i] = sg[i * S::G + pos];
    rd[k] = density(fd[k]);
    s2[pos] = rd[k];  // the densities of step t are no longer read (barrier above)
  }
  if (tid < S::NRING) {
    int hx, hy;
    ring_slot<S>(tid, hx, hy);
    const int pos = hy * S::LW + hx;
    float fr[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) fr[i] = sg[i * S::G + pos];
    s2[pos] = density(fr);
  }
  __syncthreads();
  // (D) step t + 1 on the tile; with kMid first the state of t + 1, f-bar_i
  // of each tile node, which LDS holds where it streamed to
  const int x = x0 + lx;
  if (x >= nx) return;
  char* const ob = reinterpret_cast<char*>(dst) + (size_t)y0 * rowb;
  char* const mb = kMid ? reinterpret_cast<char*>(mid) + (size_t)y0 * rowb : nullptr;
#pragma unroll
  for (int k = 0; k < S::KD; ++k) {
    const int r = ly + k * S::WY;
    if (y0 + r >= ny) break;
    if constexpr (kMid) {
      const int pos = (r + 1) * S::LW + lx + 1;
      const unsigned o = (unsigned)r * rb + 4u * (unsigned)x;
#pragma unroll
      for (int i = 0; i < 9; ++i)
        put<true>(sg[i * S::G + pos + kCy[i] * S::LW + kCx[i]], mb + i * pb, o);
    }
    float gx, gy;
    stencil_at<S::LW>(s2, (r + 1) * S::LW + lx + 1, gx, gy);
    collide_node<float>(fd[k], rd[k], gx, gy, c);
    const unsigned o = (unsigned)r * rb + 4u * (unsigned)x;
#pragma unroll
    for (int i = 0; i < 9; ++i) put<kStream>(fd[k][i], ob + i * pb, o);
  }
}

// ---------------------------------------------------------------------------
// Two time steps per launch on large lattices (FP32 storage), marching: a
// workgroup walks down a strip of kMarchCols columns, one thread per column
// of the strip and its halo and one row per iteration, with both steps as a
// pipeline of rows behind the row being loaded.  Iteration m (rows counted
// from the first of the workgroup's segment)
//   (B) collides row m - 5 of step t, whose stencil reads the densities of
//       rows m - 6 .. m - 4, and pushes its populations to the rows they
//       stream to;
//   (A) stages the densities of row m - 3, which the iteration before
//       loaded, and issues the loads of row m - 2;
//   (D) collides row m - 9 of step t + 1 and stores it;
//   (C) takes back the nine populations that have arrived at row m - 7 and
//       stages its densities.
// A phase reads only what earlier iterations left in LDS, so an iteration
// has one barrier.  The rows in flight are held in rings of four slots (two
// for populations that move up, which are read one iteration after their
// write), indexed by constants: the loop is unrolled four times.  Every node
// is updated by the operations of step_kernel in the same order.
//
// What bounds it: the vector ALU, as in step2_kernel, but without that
// kernel's halo of a 64 x 24 tile (12 % more collisions), its side nodes,
// row tests and addresses: 254 instructions per update at 4096^2 against 283
// (and 230 of arithmetic).  One workgroup of 1024 threads per CU: its barrier
// keeps the waves of a SIMD together, where four workgroups of 256 drift
// apart and leave the SIMD to the slowest at the end (4096^2: 147 us per
// step), and a wide strip has few partial lines.  The 32 columns left of the
// strip put the first thread's loads and the stores on 128-byte lines
// (16384 x 8192: 972 us; with 16 columns, storing 992 of the 1024, 1006).  A
// segment costs about eight rows more than it has, while the pipeline fills
// (16 us for its first eight iterations of 3.3) and drains.
// Measured, us per step, step2_kernel / this: 2880^2 79.0 / 76.1, 3072^2 86.7
// / 83.2, 5000 x 3000 142.9 / 126.4, 4096^2 142.9 / 131.9, 4097 x 4093 155.3 /
// 138.4, 6000 x 5000 266.6 / 229.7, 8192^2 542 / 487, 16384 x 8192 1103 / 975.
// ---------------------------------------------------------------------------
constexpr int kMarchThreads = 1024, kMarchLeft = 32, kMarchCols = 960;
static_assert(kMarchLeft + kMarchCols + 3 <= kMarchThreads, "a thread per column of the strip and its halo");

// Segments of `rows` rows: first full_blocks workgroups on the full strips,
// one segment each; then those of the narrower last strip, whose segments
// take `lanes` threads (whole waves) and share a workgroup.
struct MarchGrid {
  unsigned full_blocks, segs;  // segs: per strip
  Divisor full, lanes;         // full: full strips
  int rows;
};

template <bool kStream>
__global__ __launch_bounds__(kMarchThreads) void march_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                                              int nx, int ny, MarchGrid grid, Coef<float> c) {
  constexpr int W = kMarchThreads + 2;  // thread X at X + 1
  __shared__ float s1[4][W], s2[4][W];  // densities at t, t + 1
  // populations at t + 1 where they arrive, by velocity: along the row, down, up
  __shared__ float gh[4][3][W], gu[4][3][W], gd[2][3][W];
  const int X = threadIdx.x;
  unsigned strip, lane = X;
  unsigned seg = div_mod(blockIdx.x, grid.full, strip);
  if (blockIdx.x >= grid.full_blocks) {
    strip = grid.full.d;
    const unsigned part = __builtin_amdgcn_readfirstlane(div_mod((unsigned)X, grid.lanes, lane));
    const unsigned parts = (unsigned)kMarchThreads / grid.lanes.d;
    seg = part < parts ? (blockIdx.x - grid.full_blocks) * parts + part : ~0u;
  }
  const int x0 = (int)strip * kMarchCols, w = min(kMarchCols, nx - x0);
  // waves past the strip or the lattice leave; barriers wait for the others only
  if (seg >= grid.segs || __builtin_amdgcn_readfirstlane(lane) >= (unsigned)(kMarchLeft + w + 3)) return;
  const int y0 = (int)seg * grid.rows, h = min(grid.rows, ny - y0);
  const int x = x0 - kMarchLeft + (int)lane;
  const size_t rowb = (size_t)36 * nx;
  const unsigned pb = 4u * (unsigned)nx;
  // byte offsets of the column and its neighbours
  unsigned oc = 4u * (unsigned)wrap(x, nx), om = 4u * (unsigned)wrap(x - 1, nx), op = 4u * (unsigned)wrap(x + 1, nx);
  const bool own = lane >= (unsigned)kMarchLeft && lane < (unsigned)(kMarchLeft + w);
  const char* const base = reinterpret_cast<const char*>(src);
  int yn = wrap(y0 - 2, ny);  // rows y - 1, y, y + 1 of the next row to load
  const char* pm = base + (size_t)wrap(y0 - 4, ny) * rowb;
  const char* p0 = base + (size_t)wrap(y0 - 3, ny) * rowb;
  const char* pp = base + (size_t)yn * rowb;
  char* out = reinterpret_cast<char*>(dst) + (size_t)y0 * rowb;
  unsigned xb = 4u * (unsigned)X;  // byte offset of the thread's column within an LDS row
  auto at = [&](float* row, int d) __attribute__((always_inline)) -> float& {
    return *reinterpret_cast<float*>(reinterpret_cast<char*>(row) + 4 * (d + 1) + xb);
  };
  float F[4][9], G[4][9];
  auto pull = [&](float* f) __attribute__((always_inline)) {
    // keeps the offsets 32 bits wide beside a scalar base
    asm volatile("" : "+v"(oc), "+v"(om), "+v"(op));
#pragma unroll
    for (int i = 0; i < 9; ++i)
      f[i] = ldb<float>((kCy[i] == 0 ? p0 : (kCy[i] > 0 ? pm : pp)) + (size_t)i * pb,
                        kCx[i] == 0 ? oc : (kCx[i] > 0 ? om : op));
    pm = p0;
    p0 = pp;
    yn = yn + 1 == ny ? 0 : yn + 1;
    pp = yn == 0 ? base : pp + rowb;
  };
  auto collide = [&](float* f, float (&s)[4][W], int row) __attribute__((always_inline)) {
    float nb[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) nb[i] = at(s[(row + kCy[i]) & 3], kCx[i]);
    float gx, gy;
    stencil(nb[1], nb[2], nb[3], nb[4], nb[5], nb[6], nb[7], nb[8], gx, gy);
    collide_node<float>(f, nb[0], gx, gy, c);
  };
  auto iteration = [&](auto slot, int m) __attribute__((always_inline)) {
    constexpr int I = decltype(slot)::value;
    // LDS addresses are formed in every iteration: kept across iterations they
    // take 12 registers, three more than there are (16 waves: 128), and the
    // spills' traffic costs 3 % (4096^2: 134.6 / 131.1 us per step)
    asm volatile("" : "+v"(xb));
    if (m >= 3 && m <= h + 6) {
      float* const f = F[(I + 2) & 3];
      collide(f, s1, I + 2);
      at(gh[(I + 2) & 3][0], 0) = f[0];
      at(gh[(I + 2) & 3][1], 1) = f[1];
      at(gh[(I + 2) & 3][2], -1) = f[3];
      at(gu[(I + 3) & 3][0], 0) = f[2];
      at(gu[(I + 3) & 3][1], 1) = f[5];
      at(gu[(I + 3) & 3][2], -1) = f[6];
      at(gd[(I + 1) & 1][0], 0) = f[4];
      at(gd[(I + 1) & 1][1], -1) = f[7];
      at(gd[(I + 1) & 1][2], 1) = f[8];
    }
    if (m <= h + 5) at(s1[I], 0) = density(F[I]);
    if (m <= h + 4) pull(F[(I + 1) & 3]);
    if (m >= 9 && m <= h + 8) {
      float* const f = G[(I + 2) & 3];
      collide(f, s2, I + 2);
      // the nine rows of populations as one buffer; halo columns store beyond its end, that is nowhere
      const auto rs = __builtin_amdgcn_make_buffer_rsrc(out, 0, 9u * pb, 0x00020000);
      asm volatile("" : "+v"(oc));
      const unsigned so = own ? oc : 1u << 31;
#pragma unroll
      for (int i = 0; i < 9; ++i)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f[i]), rs, so, i * pb, kStream ? 2 : 0);
      out += rowb;
    }
    if (m >= 6 && m <= h + 7) {
      float* const g = G[I];
      g[0] = at(gh[I][0], 0);
      g[1] = at(gh[I][1], 0);
      g[3] = at(gh[I][2], 0);
      g[2] = at(gu[I][0], 0);
      g[5] = at(gu[I][1], 0);
      g[6] = at(gu[I][2], 0);
      g[4] = at(gd[I & 1][0], 0);
      g[7] = at(gd[I & 1][1], 0);
      g[8] = at(gd[I & 1][2], 0);
      at(s2[I], 0) = density(g);
    }
    __syncthreads();
  };
  pull(F[0]);
  for (int m = 0; m < h + 9; m += 4) {
    iteration(std::integral_constant<int, 0>{}, m);
    iteration(std::integral_constant<int, 1>{}, m + 1);
    iteration(std::integral_constant<int, 2>{}, m + 2);
    iteration(std::integral_constant<int, 3>{}, m + 3);
  }
}

// ---------------------------------------------------------------------------
// Several time steps per launch on small lattices (every storage).  A
// workgroup advances a TX x TY tile by k <= K steps.  Each thread owns one
// node of the tile plus a ring of 2 k - 1 nodes, numbered from the inside
// out: the tile first, then ring after ring.  Per step
//   (1) the density of every node still valid goes to LDS;
//   (2) its nodes but the outermost ring collide and push f-bar, encoded as
//       the storage holds it, to the LDS slots of the nodes it streams to;
//       tile nodes store f-bar where the caller wants the state;
//   (3) every node takes its nine populations back.
// A step shrinks the valid part by two rings (one the stencil reads, one the
// populations cross), so each phase works on a prefix of the threads and
// whole waves drop out as it shrinks.  Every node is updated by the
// operations of step_kernel in the same order, the 2-byte storages rounding
// every state as it does, so k fused steps give the bits of k single steps.
//
// What bounds it: not bandwidth (a whole 256^2 state is 2.4 MB) and not the
// vector ALU, but one wave's chain of instructions.  A launch costs about
// 2.8 us before its first collision (the gap between dependent launches, the
// kernel arguments, the first loads, cold instruction fetch), and a step a
// further 0.8 us when each SIMD holds one wave (1870 cycles: 1340 for the
// collision, at one instruction per five cycles, the rest LDS and barriers).
// So: as many steps per launch as the recomputed rings allow; one node per
// thread, which spreads the collisions over all SIMDs; and the steps as a
// loop over one copy of the code, since instructions executed once cost
// their fetch (a straight line of 2048 takes 3.8 us longer than a loop).
// ---------------------------------------------------------------------------
template <int TX_, int TY_, int K_>
struct TileKShape {
  static constexpr int TX = TX_, TY = TY_, K = K_, R = 2 * K - 1;
  static constexpr int W = TX + 2 * R, H = TY + 2 * R, N = W * H;
  static constexpr int NT = (N + 63) / 64 * 64;
  static_assert(NT <= 1024, "one node per thread");
  // nodes of the tile and its first j rings
  static constexpr __host__ __device__ int prefix(int j) { return (TX + 2 * j) * (TY + 2 * j); }
};

// Position (X, Y) in the W x H region of thread t < N: ring j around the box
// of the tile and its first j - 1 rings is the row above the box, the row
// below, then the column to its left and the one to its right.
template <class S>
__device__ __forceinline__ void ring_node(int t, int& X, int& Y) {
  int j = 0;
#pragma unroll
  for (int m = 0; m < S::R; ++m) j += t >= S::prefix(m);
  const int w = S::TX + 2 * j, h = S::TY + 2 * j - 2, u = t - (w - 2) * h;  // ring: rows of w nodes, columns of h
  const bool row = u < 2 * w;
  const int n = row ? w : h, v = row ? u : u - 2 * w;
  const bool second = v >= n;
  const int along = second ? v - n : v;  // position along the row or column
  X = S::R - j + (row ? along : (second ? w - 1 : 0));
  Y = S::R - j + (row ? (second ? h + 1 : 0) : along + 1);
  if (j == 0) X = S::R + t % S::TX, Y = S::R + t / S::TX;
}

// States a launch of k steps writes: p[s] receives the state after step
// s + 1 (null: not stored).
template <int K>
struct StepOuts {
  void* p[K];
};

template <class S, class St>
__global__ __launch_bounds__(S::NT) void stepk_kernel(const void* __restrict__ src, StepOuts<S::K> outs,
                                                      const uint16_t* __restrict__ ref_in,
                                                      uint16_t* __restrict__ ref_out, int nx, int ny,
                                                      TileOrder order, int k, Coef<float> c, RefPoly<float> q) {
  using E = typename St::E;
  __shared__ E sf[9 * S::N];                         // populations arriving at each node
  __shared__ float srho[S::N];                       // densities
  __shared__ float sref[St::kRef ? 3 * S::N : 1];    // -S f_ref of each velocity class (2-byte storages)
  const Layout L = state_layout(nx, ny, St::ES);
  int tx, ty;
  order_tile(blockIdx.x, order, tx, ty);
  const int tid = threadIdx.x;
  int X, Y;
  ring_node<S>(tid, X, Y);
  const int x = tx * S::TX - S::R + X, y = ty * S::TY - S::R + Y, pos = Y * S::W + X;
  const bool own = tid < S::TX * S::TY && x < nx && y < ny;
  const unsigned off = St::ES * ((unsigned)y * L.rp + (unsigned)x);
  float f[9], ref[3];
  // f(t) arriving at the tile and its first 2 k - 1 rings
  if (tid < (S::TX + 4 * k - 2) * (S::TY + 4 * k - 2)) {
    const int xw = wrap(x, nx), yw = wrap(y, ny);
    E r[9];
    pull_raw<E>(planes<E>(src, L.ps), node_addr<St::ES>(xw, yw, nx, ny, L.rp), r);
    decode<St>(r, St::kRef ? ref_in[(unsigned)yw * nx + (unsigned)xw] : 0, q, f);
  }
#pragma unroll 1
  for (int s = k - 1, j = 0;; --s, ++j) {  // s steps follow this one
    // nodes that collide (the tile and 2 s rings), nodes whose density they read (one ring more)
    const int nc = (S::TX + 4 * s) * (S::TY + 4 * s), nd = (S::TX + 4 * s + 2) * (S::TY + 4 * s + 2);
    float rho = 0.0f;
    if (tid < nd) {
      rho = density(f);
      srho[pos] = rho;
      if constexpr (St::kRef) {
        const float rt = ref_density(rho);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          ref[m] = ref_value(q, m, rt);
          sref[m * S::N + pos] = -q.scale * ref[m];
        }
      }
    }
    __syncthreads();
    if (tid < nc) {
      float gx, gy;
      stencil_at<S::W>(srho, pos, gx, gy);
      collide_node<float, St::kRef>(f, rho, gx, gy, c);
      E o[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        if constexpr (St::kRef)
          o[i] = St::from_f32(fmaf(f[i], q.scale, sref[velocity_class(i) * S::N + pos + kCy[i] * S::W + kCx[i]]));
        else
          o[i] = f[i];
      }
      char* const out = static_cast<char*>(outs.p[j]);
      if (out && own) {
        // rows of whole 128-byte lines are streamed (every state of 256^2
        // stored: 2.37 us per step against 2.52), shorter ones left to merge
        // in the caches (16 x 16 tiles, 620^2: 7.6 against 11.6)
#pragma unroll
        for (int i = 0; i < 9; ++i) put<S::TX * sizeof(E) >= 128>(o[i], out + (size_t)i * L.ps * St::ES, off);
        if constexpr (St::kRef)
          if (s == 0) ref_out[(unsigned)y * nx + (unsigned)x] = f32_to_f16(rho);
      }
      if (s > 0) {
#pragma unroll
        for (int i = 0; i < 9; ++i) sf[i * S::N + pos + kCy[i] * S::W + kCx[i]] = o[i];
      }
    }
    if (s == 0) break;
    __syncthreads();
    // the part still valid: the tile and 2 s - 1 rings.  The next barrier
    // separates these reads from the next step's pushes.
    if (tid < (S::TX + 4 * s - 2) * (S::TY + 4 * s - 2)) {
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        if constexpr (St::kRef)
          f[i] = fmaf(St::to_f32(sf[i * S::N + pos]), q.inv_scale, ref[velocity_class(i)]);
        else
          f[i] = sf[i * S::N + pos];
      }
    }
  }
}

// The value of the lane kOff higher (kOff a power of two) in every lane that
// kOff does not carry across its 64, 32 or 16 lanes; elsewhere some lane's.
// Register permutes (DPP within a row of 16 lanes, row and half swaps above)
// instead of a trip through LDS.
template <int kOff>
__device__ __forceinline__ unsigned lane_up(unsigned v) {
  if constexpr (kOff == 32) {
    return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
  } else if constexpr (kOff == 16) {
    return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
  } else {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + kOff, 0xF, 0xF, true);  // row_shl:kOff
  }
}
template <int kOff>
__device__ __forceinline__ double lane_up(double v) {
  const unsigned long long b = __double_as_longlong(v);
  const unsigned lo = lane_up<kOff>((unsigned)b), hi = lane_up<kOff>((unsigned)(b >> 32));
  return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// Sum over the wave in lane 0: lane i adds lane i + 32, then + 16, ..., + 1.
__device__ __forceinline__ double wave_sum(double v) {
  v += lane_up<32>(v);
  v += lane_up<16>(v);
  v += lane_up<8>(v);
  v += lane_up<4>(v);
  v += lane_up<2>(v);
  v += lane_up<1>(v);
  return v;
}

// Deterministic FP64 sum of three per-thread values over a block, into the
// slot partials[3 slot .. 3 slot + 2] (on top of `before`, the slot's sum so
// far, in threads 0 .. 2): a fixed tree inside each wave, then the waves'
// sums in wave order.  red holds 3 doubles per wave of LDS; it may alias LDS
// the block read before the call.  The end of a workgroup waits for it, so
// the tree stays in registers and the caller loads `before` early (adjoint
// step of 64^2, 64 x 8 tiles: 7.33 us with the tree through LDS and the slot
// read here, 6.79 with the slot read early, 6.61 with both).
template <class S>
__device__ __forceinline__ void block_sum3(const double* in, double* red, double* __restrict__ partials,
                                           unsigned slot, double before) {
  constexpr int NW = S::NTHREADS / 64;
  const int tid = threadIdx.y * S::TX + threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double v[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) v[k] = wave_sum(in[k]);
  __syncthreads();  // red may alias LDS read above
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) red[k * NW + wave] = v[k];
  __syncthreads();
  if (tid < 3) {
    double s = red[tid * NW];
    for (int w = 1; w < NW; ++w) s += red[tid * NW + w];
    partials[(size_t)slot * 3 + tid] = before + s;
  }
}

// Moments: rho and u of main Eq. 5 plus per-workgroup FP64 partial sums of
// mass and lattice momentum (reduced in a fixed order; a tile's sums go to
// the slot of its raster index).  kVel false: rho and the sums only, which
// need neither the ring nor the force.  Bound by HBM: 48 B per node with the
// three fields, 146 us at 4096^2 for a kernel that only moves them; loads
// from uniform bases on interior tiles and the tile order of the step took
// it from 194 us there and from 1636 at 16384 x 8192 (64-bit addresses on
// every tile).
template <class St, int kMode, bool kVel>
__global__ __launch_bounds__(MomTile::NTHREADS) void moments_kernel(
    const void* __restrict__ src, const uint16_t* __restrict__ ref_in, float* __restrict__ rho_out,
    float* __restrict__ ux_out, float* __restrict__ uy_out, double* __restrict__ partials, int nx, int ny, int ntx,
    TileOrder order, Coef<float> c, RefPoly<float> q, TileRows rows) {
  using S = MomTile;
  using E = typename St::E;
  __shared__ float srho[kVel ? S::LDS : 1];
  __shared__ double sred[3 * (S::NTHREADS / 64)];
  const Layout L = state_layout(nx, ny, St::ES);
  int tx, tr;
  order_tile(blockIdx.x, order, tx, tr);
  const int ty = tile_row(rows, tr), x0 = tx * S::TX, y0 = ty * S::TY;
  float f[S::NPT][9];
  float rho[S::NPT];
  {
    TileRegs<S, St> R;
    const int yb = kMode == kBand ? y0 - 2 : 0;
    const char* sb = static_cast<const char*>(src) + (size_t)yb * St::ES * L.rp;
    if constexpr (kMode == kWide)
      issue_tile<S, St, false, true, kVel>(planes<E>(src, L.ps), ref_in, nx, ny, x0, y0, 0, R);
    else if (interior_tile<S>(x0, y0, nx, ny))
      issue_tile<S, St, true, false, kVel>(planes<E>(sb, L.ps), ref_in, nx, ny, x0, y0, yb, R);
    else
      issue_tile<S, St, false, false, kVel>(planes<E>(sb, L.ps), ref_in, nx, ny, x0, y0, yb, R);
    if constexpr (kVel) {
      stage_tile<S, St>(R, q, f, rho, srho, nullptr);
      __syncthreads();
    } else {
#pragma unroll
      for (int k = 0; k < S::NPT; ++k) decode<St>(R.raw[k], St::kRef ? R.rref[k] : 0, q, f[k]);
    }
  }
  const int x = x0 + threadIdx.x;
  double sm = 0.0, sx = 0.0, sy = 0.0;
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    const int ly = threadIdx.y + k * S::WY, y = y0 + ly;
    if (x >= nx || y >= ny) continue;
    float m[9];
    forward_moments(f[k], m);
    const size_t o = (size_t)y * nx + x;
    if (rho_out) rho_out[o] = m[0];
    if constexpr (kVel) {
      float nb[9], gx, gy;
      neighbours<S>(srho, threadIdx.x + 1, ly + 1, nb);
      stencil(nb[1], nb[2], nb[3], nb[4], nb[5], nb[6], nb[7], nb[8], gx, gy);
      const NodeState<float> s = node_state(m[0], m[3], m[5], gx, gy, c);
      if (ux_out) ux_out[o] = s.ux;
      if (uy_out) uy_out[o] = s.uy;
    }
    sm += (double)m[0];
    sx += (double)m[3];
    sy += (double)m[5];
  }
  const double v[3] = {sm, sx, sy};
  block_sum3<S>(v, sred, partials, (unsigned)(ty * ntx + tx), 0.0);
}

// Sum of the per-workgroup partials in a fixed order: each thread adds a
// strided subset in order, then block_sum3 over the 256 threads.  kClear:
// the partials are zeroed once read.  One workgroup is bound by the latency
// of its loads, so each thread keeps kAhead of them in flight (131072
// partials took 231 us one at a time, 16384 29 us).
constexpr int RED = 256;
struct FlatBlock {
  static constexpr int TX = RED, NTHREADS = RED;
};
template <bool kClear>
__global__ __launch_bounds__(RED) void finish_sums(double* __restrict__ partials, int nblocks,
                                                   double* __restrict__ out) {
  __shared__ double red[3 * (RED / 64)];
  constexpr int kAhead = 8;
  double a[3] = {0.0, 0.0, 0.0};
  int b = threadIdx.x;
  for (; b + (kAhead - 1) * RED < nblocks; b += kAhead * RED) {
    double v[kAhead][3];
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) v[j][k] = partials[(size_t)(b + j * RED) * 3 + k];
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        a[k] += v[j][k];
        if constexpr (kClear) partials[(size_t)(b + j * RED) * 3 + k] = 0.0;
      }
  }
  for (; b < nblocks; b += RED)
    for (int k = 0; k < 3; ++k) {
      a[k] += partials[(size_t)b * 3 + k];
      if constexpr (kClear) partials[(size_t)b * 3 + k] = 0.0;
    }
  block_sum3<FlatBlock>(a, red, out, 0, 0.0);  // one block: its slot is out[0..2]
}

// Halo coordinates (hx, hy) of the entries p = tid, tid + NTHREADS, ... of
// a W-wide row-major table, stepped without divisions: one division for the
// first entry, then NTHREADS = DY W + DX per step.
template <int W, int NTHREADS>
struct HaloWalk {
  static constexpr int DY = NTHREADS / W, DX = NTHREADS % W;
  int hx, hy;
  __device__ __forceinline__ explicit HaloWalk(int p) : hx(p % W), hy(p / W) {}
  __device__ __forceinline__ void next() {
    hx += DX;
    hy += DY;
    if (hx >= W) hx -= W, ++hy;
  }
};

// Store the post-streaming populations f of node (x, y) into the pull
// layout: f_i goes to slot (i, x - e_i), where pull_raw reads it, encoded
// against the reference density of (x, y), which is also written (2-byte
// storages).  kWideAddr: 64-bit addresses (states above 4 GiB).
template <class St, bool kWideAddr, bool kStream>
__device__ __forceinline__ void put_node(int x, int y, int nx, int ny, const float* f, const RefPoly<float>& q,
                                         void* dst, uint16_t* ref_out) {
  using E = typename St::E;
  const Layout L = state_layout(nx, ny, St::ES);
  float rd[9];
  if constexpr (St::kRef) {
    const float r = ref_density(density(f));
    *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ref_out) + 2u * ((unsigned)y * nx + (unsigned)x)) = f32_to_f16(r);
#pragma unroll
    for (int i = 0; i < 9; ++i) rd[i] = r;
  }
  E o[9];
  encode<St>(f, rd, q, o);
  if constexpr (kWideAddr) {
    char* const base = static_cast<char*>(dst);
    const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
    const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int row = kCy[i] == 0 ? y : (kCy[i] > 0 ? ym : yp), col = kCx[i] == 0 ? x : (kCx[i] > 0 ? xm : xp);
      put<kStream>(o[i], base + ((size_t)row * L.rp + (size_t)i * L.ps) * St::ES, St::ES * (unsigned)col);
    }
  } else {
    const OutPlanes<E> Q = out_planes<E>(dst, L.ps);
    const NodeAddr<St::ES> a = node_addr<St::ES>(x, y, nx, ny, L.rp);
#pragma unroll
    for (int i = 0; i < 9; ++i)
      put<kStream>(o[i], Q.p[i],
                   (kCy[i] == 0 ? a.r0 : (kCy[i] > 0 ? a.rm : a.rp)) + (kCx[i] == 0 ? a.c0 : (kCx[i] > 0 ? a.cm : a.cp)));
  }
}

// One thread per node o of the lattice, in row order; width: make_divisor(nx).
// These kernels move 40 (init), 72 (set, get) or 80 (adjoint seed) bytes per
// node and are bound by HBM.
constexpr int BLK = 256;
__device__ __forceinline__ bool flat_node(int nx, int ny, const Divisor& width, unsigned& o, int& x, int& y) {
  o = blockIdx.x * BLK + threadIdx.x;
  if (o >= (unsigned)nx * (unsigned)ny) return false;
  unsigned rem;
  y = (int)div_mod(o, width, rem);
  x = (int)rem;
  return true;
}

// Initial state: f^eq(rho0, u0, eta(rho0)) at every node.  Sets *flag on a
// density outside (0, 4/b) or a non-finite input.  kRest: no velocities
// given.
template <class St, bool kWideAddr, bool kStream, bool kRest>
__global__ __launch_bounds__(BLK) void init_kernel(const float* __restrict__ rho0, const float* __restrict__ ux0,
                                                   const float* __restrict__ uy0, void* __restrict__ dst,
                                                   uint16_t* __restrict__ ref_out, int nx, int ny, Divisor width,
                                                   Coef<float> c, RefPoly<float> q, int* flag) {
  unsigned o;
  int x, y;
  if (!flat_node(nx, ny, width, o, x, y)) return;
  const float r = rho0[o];
  bool bad = !(r > 0.0f && c.b4 * r < 1.0f);
  float f[9];
  if constexpr (kRest) {
    equilibrium_rest(r, c, f);
  } else {
    const float ux = ux0 ? ux0[o] : 0.0f, uy = uy0 ? uy0[o] : 0.0f;
    bad = bad || !isfinite(ux) || !isfinite(uy);
    equilibrium_node(r, ux, uy, c, f);
  }
  if (bad) *flag = 1;  // any thread, the same value
  put_node<St, kWideAddr, kStream>(x, y, nx, ny, f, q, dst, ref_out);
}

// The initial state at rest of lattices that stream past the caches
// (launch_init), by tiles: the three class values of every node of the tile
// and its ring go to LDS, and each slot of the pull layout takes its own from
// there, so that whole aligned rows are stored.  One node per thread
// (init_kernel) stores rows shifted by the streaming, whose ends share lines
// with the next workgroup's (us of lbm_init with its wait, one node per thread /
// by tiles: FP32 4096^2 160 / 107, 8192^2 629 / 378, 16384 x 8192 1324 / 889, in
// tiles of 256 x 8 in 512 threads; FP16 4096^2 111 / 68, 8192^2 384 / 322, 16384
// x 8192 768 / 677, in tiles of 64 x 16).  On lattices the caches hold it gains
// nothing.
template <int TX_, int TY_, int WY_>
struct InitShape {
  static constexpr int TX = TX_, TY = TY_, WY = WY_, NPT = TY / WY, LW = TX + 2;
  static constexpr int NTHREADS = TX * WY, LDS = (TY + 2) * LW;
};
template <class St>
using InitTile = std::conditional_t<St::kRef, InitShape<64, 16, 4>, InitShape<256, 8, 2>>;

template <class St>
__global__ __launch_bounds__(InitTile<St>::NTHREADS) void init_rest_kernel(const float* __restrict__ rho0,
                                                                      void* __restrict__ dst,
                                                                      uint16_t* __restrict__ ref_out, int nx, int ny,
                                                                      TileOrder order, Coef<float> c,
                                                                      RefPoly<float> q, int* flag) {
  using S = InitTile<St>;
  using E = typename St::E;
  __shared__ E sv[3 * S::LDS];
  int tx, ty;
  order_tile(blockIdx.x, order, tx, ty);
  const int x0 = tx * S::TX, y0 = ty * S::TY, tid = threadIdx.y * S::TX + threadIdx.x;
  constexpr int kRounds = (S::LDS + S::NTHREADS - 1) / S::NTHREADS;
  float r[kRounds];
  {
    HaloWalk<S::LW, S::NTHREADS> w(tid);
#pragma unroll
    for (int k = 0; k < kRounds; ++k, w.next())
      if (tid + k * S::NTHREADS < S::LDS)
        r[k] = ldb<float>(reinterpret_cast<const char*>(rho0),
                          4u * ((unsigned)wrap(y0 + w.hy - 1, ny) * (unsigned)nx + (unsigned)wrap(x0 + w.hx - 1, nx)));
  }
  HaloWalk<S::LW, S::NTHREADS> w(tid);
  bool bad = false;
#pragma unroll
  for (int k = 0; k < kRounds; ++k, w.next()) {
    const int p = tid + k * S::NTHREADS;
    if (p >= S::LDS) break;
    bad = bad || !(r[k] > 0.0f && c.b4 * r[k] < 1.0f);
    float f[9];
    equilibrium_rest(r[k], c, f);
    E o[9];
    float rd[9];
    if constexpr (St::kRef) {
      const float rt = ref_density(density(f));
#pragma unroll
      for (int i = 0; i < 9; ++i) rd[i] = rt;
      const int x = x0 + w.hx - 1, y = y0 + w.hy - 1;
      if (w.hx >= 1 && w.hx <= S::TX && w.hy >= 1 && w.hy <= S::TY && x < nx && y < ny)
        *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(ref_out) + 2u * ((unsigned)y * nx + (unsigned)x)) =
            f32_to_f16(rt);
    }
    encode<St>(f, rd, q, o);
    sv[p] = o[0], sv[S::LDS + p] = o[1], sv[2 * S::LDS + p] = o[5];
  }
  if (bad) *flag = 1;  // any thread, the same value
  __syncthreads();
  const int x = x0 + threadIdx.x;
  if (x >= nx) return;
  const Layout L = state_layout(nx, ny, St::ES);
  char* const base = static_cast<char*>(dst) + (size_t)y0 * L.rp * St::ES;
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    const int ly = threadIdx.y + k * S::WY;
    if (y0 + ly >= ny) break;
    const unsigned off = St::ES * ((unsigned)ly * L.rp + (unsigned)x);  // rows of the tile: below 2^32 (launch_init)
    const int pos = (ly + 1) * S::LW + threadIdx.x + 1;
#pragma unroll
    for (int i = 0; i < 9; ++i)
      put<true>(sv[velocity_class(i) * S::LDS + pos + kCy[i] * S::LW + kCx[i]], base + (size_t)i * L.ps * St::ES, off);
  }
}

// Load a post-streaming state.  kShiftLoads (FP32, launch_set): the shift of
// the streaming goes into the loads, so that whole rows are stored; else into
// the stores (put_node).
template <class St, bool kWideAddr, bool kShiftLoads, bool kStream>
__global__ __launch_bounds__(BLK) void set_state_kernel(const float* __restrict__ fin, void* __restrict__ dst,
                                                        uint16_t* __restrict__ ref_out, int nx, int ny, Divisor width,
                                                        RefPoly<float> q) {
  unsigned o;
  int x, y;
  if (!flat_node(nx, ny, width, o, x, y)) return;
  const Planes<float> F = planes<float>(fin, (size_t)nx * ny);
  if constexpr (kShiftLoads) {
    // a permutation: slot (i, x) is f_i of node x + e_i
    const Layout L = state_layout(nx, ny, 4);
    const NodeAddr<4> a = node_addr<4>(x, y, nx, ny, (unsigned)nx);
    char* const base = static_cast<char*>(dst) + (kWideAddr ? (size_t)y * L.rp * 4 : 0);
    const unsigned off = 4u * ((kWideAddr ? 0u : (unsigned)y * L.rp) + (unsigned)x);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const unsigned from = (kCy[i] == 0 ? a.r0 : (kCy[i] > 0 ? a.rp : a.rm)) + (kCx[i] == 0 ? a.c0 : (kCx[i] > 0 ? a.cp : a.cm));
      put<kStream>(ldb<float>(F.p[i], from), base + (size_t)i * L.ps * 4, off);
    }
  } else {
    float f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = ldb<float>(F.p[i], 4u * o);
    put_node<St, kWideAddr, kStream>(x, y, nx, ny, f, q, dst, ref_out);
  }
}

// Export the post-streaming state f(t).  kLaneStores: stores at per-lane 64-bit
// addresses instead of uniform bases and one 32-bit offset (lbm_get_state).
template <class St, bool kWideAddr, bool kLaneStores>
__global__ __launch_bounds__(BLK) void get_state_kernel(const void* __restrict__ src,
                                                        const uint16_t* __restrict__ ref_in, float* __restrict__ fout,
                                                        int nx, int ny, Divisor width, RefPoly<float> q) {
  using E = typename St::E;
  unsigned o;
  int x, y;
  if (!flat_node(nx, ny, width, o, x, y)) return;
  E raw[9];
  const Layout L = state_layout(nx, ny, St::ES);
  if constexpr (kWideAddr)
    pull_rows(static_cast<const char*>(src), x, y, nx, ny, raw);
  else
    pull_raw<E>(planes<E>(src, L.ps), node_addr<St::ES>(x, y, nx, ny, L.rp), raw);
  float f[9];
  decode<St>(raw, St::kRef ? ref_in[o] : 0, q, f);
  const size_t N = (size_t)nx * ny;
  if constexpr (kLaneStores) {
#pragma unroll
    for (int i = 0; i < 9; ++i) fout[(size_t)i * N + o] = f[i];
  } else {
    const OutPlanes<float> F = out_planes<float>(fout, N);
#pragma unroll
    for (int i = 0; i < 9; ++i) put<false>(f[i], F.p[i], 4u * o);
  }
}

// ---------------------------------------------------------------------------
// Adjoint (reverse mode) of the FP32 step
//
// The adjoint of time t is Lambda_i(x) = dL/d f_i(x, t) for the post-
// streaming populations.  It is kept as eleven planes {L_0..L_8, A_x, A_y}:
//   Lambda_i(x) = L_i(x) + nu(x),   nu(z) = sum_j w_j e_j . A(z - e_j),
// where A(y) = dL/d g(y) for the stencil gradient g of main Eq. 12 at y and
// nu(z) is dL/d rho(z) through the eight stencils that read rho(z).  Keeping
// A instead of adding nu to all nine planes saves a second sweep: the next
// adjoint step forms nu on its tile from a two-node halo of A.
//
// One adjoint step, for every node y (forward state of time t, adjoint of
// time t+1):
//   lam-bar_i(y) = Lambda_i(y + e_i, t+1)   (streaming moved f-bar_i(y) to y + e_i)
//   (L_i(y), A(y), dtheta) = transposed Jacobian of the collision at y
//                            (rho and g recomputed as the forward step has them)
// ---------------------------------------------------------------------------
#ifndef LBM_ADJ_TILE
#define LBM_ADJ_TILE 64, 8, 4
#endif
using AdjTile = TileShape<LBM_ADJ_TILE>;
// Small lattices: half as wide and one node per thread.  The parameter terms
// of the two nodes one thread of AdjTile sweeps (four rows apart) are added
// in FP32 first here too (adjoint_tile), so the sums differ only in their
// FP64 order.
using AdjTileSmall = TileShape<32, 8, 8>;

template <class S>
struct AdjLds {
  static constexpr int AW = S::TX + 4, AH = S::TY + 4, NA = AW * AH;
  static constexpr int NRED = 3 * (S::NTHREADS / 64);  // doubles of the block reduction (one per wave)
  // floats of the LDS buffer that holds the A halo, then the reduction
  static constexpr int NSA = 2 * NA > 2 * NRED ? 2 * NA : 2 * NRED;
};

// A on the tile plus a two-node ring ((TY+4) x (TX+4) nodes), held in
// registers by the thread that stages it: halo node p = tid + r * NTHREADS.
template <class S>
struct AHalo {
  static constexpr int R = (AdjLds<S>::NA + S::NTHREADS - 1) / S::NTHREADS;
  float v[R][2];
};

// 32-bit byte offsets from the A planes' bases: (y rp + x) 4 < 44 nx ny for
// interleaved rows (44 nx ny < 2^32) and < 4 nx ny for planes.
template <class S, bool kInterior = false>
__device__ __forceinline__ void load_a(const float* __restrict__ ax, const float* __restrict__ ay, int nx, int ny,
                                       unsigned rp, int x0, int y0, AHalo<S>& h) {
  using L = AdjLds<S>;
  const int tid = threadIdx.y * S::TX + threadIdx.x;
  HaloWalk<L::AW, S::NTHREADS> w(tid);
#pragma unroll
  for (int r = 0; r < AHalo<S>::R; ++r) {
    const int p = tid + r * S::NTHREADS;
    if (p >= L::NA) break;
    const unsigned yy = kInterior ? (unsigned)(y0 + w.hy - 2) : (unsigned)wrap(y0 + w.hy - 2, ny);
    const unsigned xx = kInterior ? (unsigned)(x0 + w.hx - 2) : (unsigned)wrap(x0 + w.hx - 2, nx);
    const unsigned off = 4u * (yy * rp + xx);
    h.v[r][0] = ldb<float>(reinterpret_cast<const char*>(ax), off);
    h.v[r][1] = ldb<float>(reinterpret_cast<const char*>(ay), off);
    w.next();
  }
}

// The A halo (load_a's registers) into sa[2][AH][AW], a barrier, then nu on
// the tile plus a one-node ring into snu[(TY+2)][LW], and a barrier.
template <class S>
__device__ __forceinline__ void put_nu(const AHalo<S>& h, float* sa, float* snu) {
  using L = AdjLds<S>;
  const int tid = threadIdx.y * S::TX + threadIdx.x;
#pragma unroll
  for (int r = 0; r < AHalo<S>::R; ++r) {
    const int p = tid + r * S::NTHREADS;
    if (p >= L::NA) break;
    sa[p] = h.v[r][0];
    sa[L::NA + p] = h.v[r][1];
  }
  __syncthreads();
  const float third = 1.0f / 3.0f, twelfth = 1.0f / 12.0f;
  const float* sx = sa;
  const float* sy = sa + L::NA;
  HaloWalk<S::LW, S::NTHREADS> w(tid);
  for (int p = tid; p < S::LDS; p += S::NTHREADS, w.next()) {
    const int hx = w.hx, hy = w.hy;
    const int c = (hy + 1) * L::AW + hx + 1;  // the same node in the A halo
    // axis neighbours z - e_j: E -> c-1, W -> c+1, N -> c-AW, S -> c+AW
    const float axis = (sx[c - 1] - sx[c + 1]) + (sy[c - L::AW] - sy[c + L::AW]);
    // diagonals: NE -> c-AW-1 (Ax+Ay), NW -> c-AW+1 (Ay-Ax), SW -> c+AW+1 -(Ax+Ay), SE -> c+AW-1 (Ax-Ay)
    const float diag = (sx[c - L::AW - 1] + sy[c - L::AW - 1]) + (sy[c - L::AW + 1] - sx[c - L::AW + 1]) -
                       (sx[c + L::AW + 1] + sy[c + L::AW + 1]) + (sx[c + L::AW - 1] - sy[c + L::AW - 1]);
    snu[p] = third * axis + twelfth * diag;
  }
  __syncthreads();
}

// nu of the tile plus a one-node ring from the A planes (load_a, put_nu).
template <class S, bool kInterior = false>
__device__ __forceinline__ void stage_nu(const float* __restrict__ ax, const float* __restrict__ ay, int nx, int ny,
                                         unsigned rp, int x0, int y0, float* sa, float* snu) {
  AHalo<S> h;
  load_a<S, kInterior>(ax, ay, nx, ny, rp, x0, y0, h);
  put_nu<S>(h, sa, snu);
}

// Deterministic FP64 block sum of three per-thread FP32 values, added to a
// slot of partials (a tile always adds to the same slot, so sums over many
// launches are reproducible bit for bit).
template <class S>
__device__ __forceinline__ void block_accumulate(const float* th, double* red, double* __restrict__ partials,
                                                 unsigned slot, double before) {
  const double v[3] = {(double)th[0], (double)th[1], (double)th[2]};
  block_sum3<S>(v, red, partials, slot, before);
}

// One tile of the adjoint step (kInterior: interior_tile holds, no wrap).
// Every global load (the forward populations with their ring, the A halo and
// the adjoint populations of the own nodes) is issued before the first
// barrier.
template <class S, bool kInterior, int kMode, bool kStream>
__device__ __forceinline__ void adjoint_tile(const float* __restrict__ fsrc, const float* __restrict__ adj_in,
                                             float* __restrict__ adj_out, int nx, int ny, int x0, int y0,
                                             const Coef<float>& c, float* srho, float* snu, float* sa, float* th) {
  const Layout A = adj_layout(nx, ny);
  const size_t N = A.ps;
  const Planes<float> P = planes<float>(adj_in, N);
  const unsigned rb = 4u * A.rp;
  const int x = x0 + threadIdx.x;
  const unsigned o0 = rb * (unsigned)(y0 + threadIdx.y) + 4u * (unsigned)x;
  float f[S::NPT][9];
  float rho[S::NPT];
  float lb[S::NPT][9];
  AHalo<S> h;
  {
    TileRegs<S, StoreF32> R;
    const Layout Ls = state_layout(nx, ny, 4);
    const int yb = kMode == kBand ? y0 - 2 : 0;  // forward state: rows counted from yb
    if constexpr (kMode == kWide)
      issue_tile<S, StoreF32, false, true>(planes<float>(fsrc, Ls.ps), nullptr, nx, ny, x0, y0, 0, R);
    else
      issue_tile<S, StoreF32, kInterior>(planes<float>(reinterpret_cast<const char*>(fsrc) + (size_t)yb * 4 * Ls.rp, Ls.ps),
                                         nullptr, nx, ny, x0, y0, yb, R);
    load_a<S, kInterior>(adj_in + 9 * N, adj_in + 10 * N, nx, ny, A.rp, x0, y0, h);
    // lam-bar_i(y) = L_i(y + e_i) (+ nu(y + e_i) below)
#pragma unroll
    for (int k = 0; k < S::NPT; ++k) {
      const int y = y0 + threadIdx.y + k * S::WY;
      if (x >= nx || y >= ny) break;
      const unsigned o = o0 + (unsigned)(k * S::WY) * rb;
      if constexpr (kInterior) {
#pragma unroll
        for (int i = 0; i < 9; ++i) lb[k][i] = ldb<float>(P.p[i] + (ptrdiff_t)kCy[i] * rb + kCx[i] * 4, o);
      } else {
        const NodeAddr<4> a = node_addr<4>(x, y, nx, ny, A.rp);
        lb[k][0] = ldb<float>(P.p[0], a.r0 + a.c0);
        lb[k][1] = ldb<float>(P.p[1], a.r0 + a.cp);
        lb[k][2] = ldb<float>(P.p[2], a.rp + a.c0);
        lb[k][3] = ldb<float>(P.p[3], a.r0 + a.cm);
        lb[k][4] = ldb<float>(P.p[4], a.rm + a.c0);
        lb[k][5] = ldb<float>(P.p[5], a.rp + a.cp);
        lb[k][6] = ldb<float>(P.p[6], a.rp + a.cm);
        lb[k][7] = ldb<float>(P.p[7], a.rm + a.cm);
        lb[k][8] = ldb<float>(P.p[8], a.rm + a.cp);
      }
    }
    stage_tile<S, StoreF32>(R, RefPoly<float>{}, f, rho, srho, nullptr);
  }
  put_nu<S>(h, sa, snu);  // its barriers cover srho too
  ThetaTerms<float> own{};
  struct {
    char* p[11];
  } Q;
#pragma unroll
  for (int i = 0; i < 11; ++i) Q.p[i] = reinterpret_cast<char*>(adj_out) + (size_t)i * N * 4;
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    const int ly = threadIdx.y + k * S::WY, y = y0 + ly;
    if (x >= nx || y >= ny) break;
    const int hx = threadIdx.x + 1, hy = ly + 1, pos = hy * S::LW + hx;
    float nb[9];
    neighbours<S>(srho, hx, hy, nb);
    float gx, gy;
    stencil(nb[1], nb[2], nb[3], nb[4], nb[5], nb[6], nb[7], nb[8], gx, gy);
#pragma unroll
    for (int i = 0; i < 9; ++i) lb[k][i] += snu[pos + kCy[i] * S::LW + kCx[i]];
    float lf[9], agx = 0.0f, agy = 0.0f;
    ThetaTerms<float> t;
    collide_node_vjp<float>(f[k], gx, gy, c, lb[k], lf, agx, agy, t);
    if constexpr (S::NPT > 1)
      add_theta(t, c, th);
    else
      own = t;
    const unsigned o = o0 + (unsigned)(k * S::WY) * rb;
    // uniform field bases and one 32-bit lane offset for the eleven stores
#pragma unroll
    for (int i = 0; i < 9; ++i) put<kStream>(lf[i], Q.p[i], o);
    put<kStream>(agx, Q.p[9], o);
    put<kStream>(agy, Q.p[10], o);
  }
  if constexpr (S::NPT == 1) {
    // rows 0 .. 3 add the terms of the node four rows below to their own
    static_assert(S::WY == 8 && AdjTile::TY == 8 && AdjTile::WY == 4, "the pairs of AdjTile");
    static_assert(4 * sizeof(ThetaTerms<float>) / 4 * (S::NTHREADS / 2) <= 4 * AdjLds<S>::NSA, "LDS of the A halo");
    const int tid = threadIdx.y * S::TX + threadIdx.x;
    ThetaTerms<float>* const pair = reinterpret_cast<ThetaTerms<float>*>(sa);
    if (tid >= S::NTHREADS / 2) pair[tid - S::NTHREADS / 2] = own;  // sa was last read ahead of put_nu's last barrier
    __syncthreads();
    if (tid < S::NTHREADS / 2) {
      add_theta(own, c, th);
      add_theta(pair[tid], c, th);
    }
  }
}

template <class S, int kMode, bool kStream>
__global__ __launch_bounds__(S::NTHREADS) void adjoint_step_kernel(const float* __restrict__ fsrc,
                                                                   const float* __restrict__ adj_in,
                                                                   float* __restrict__ adj_out,
                                                                   double* __restrict__ partials, int nx, int ny,
                                                                   TileOrder order, Coef<float> c,
                                                                   TileRows rows) {
  using L = AdjLds<S>;
  __shared__ float srho[S::LDS];
  __shared__ float snu[S::LDS];
  __shared__ __align__(8) float sa[L::NSA];
  int tx, ty;
  const unsigned slot = order_tile(blockIdx.x, order, tx, ty);
  // the slot's sum so far, loaded ahead of the sweep
  const int tid = threadIdx.y * S::TX + threadIdx.x;
  const double before = tid < 3 ? partials[(size_t)slot * 3 + tid] : 0.0;
  const int x0 = tx * S::TX, y0 = tile_row(rows, ty) * S::TY;
  float th[3] = {0.0f, 0.0f, 0.0f};
  if constexpr (kMode == kWide)  // the tile rows that wrap: never interior
    adjoint_tile<S, false, kWide, kStream>(fsrc, adj_in, adj_out, nx, ny, x0, y0, c, srho, snu, sa, th);
  else if (interior_tile<S>(x0, y0, nx, ny))
    adjoint_tile<S, true, kMode, kStream>(fsrc, adj_in, adj_out, nx, ny, x0, y0, c, srho, snu, sa, th);
  else
    adjoint_tile<S, false, kMode, kStream>(fsrc, adj_in, adj_out, nx, ny, x0, y0, c, srho, snu, sa, th);
  block_accumulate<S>(th, reinterpret_cast<double*>(sa), partials, slot, before);
}

// Lambda = L + nu on the tile, then either exported (kInit false) or taken
// through the adjoint of the initial equilibrium (kInit true): dL/d rho0 and
// the parameter terms that enter through eta(rho0).
template <class S, bool kInit>
__global__ __launch_bounds__(S::NTHREADS) void adjoint_finish_kernel(
    const float* __restrict__ adj, float* __restrict__ out, const float* __restrict__ rho0,
    const float* __restrict__ ux0, const float* __restrict__ uy0, double* __restrict__ partials, int nx, int ny,
    int ntx, Coef<float> c) {
  using L = AdjLds<S>;
  __shared__ float snu[S::LDS];
  __shared__ __align__(8) float sa[L::NSA];
  const size_t N = (size_t)nx * ny;
  const Layout A = adj_layout(nx, ny);
  const int x0 = (blockIdx.x % ntx) * S::TX, y0 = (blockIdx.x / ntx) * S::TY;
  const int tid = threadIdx.y * S::TX + threadIdx.x;
  const double before = kInit && tid < 3 ? partials[(size_t)blockIdx.x * 3 + tid] : 0.0;
  stage_nu<S>(adj + 9 * A.ps, adj + 10 * A.ps, nx, ny, A.rp, x0, y0, sa, snu);
  float th[3] = {0.0f, 0.0f, 0.0f};
  const int x = x0 + threadIdx.x;
#pragma unroll
  for (int k = 0; k < S::NPT; ++k) {
    const int ly = threadIdx.y + k * S::WY, y = y0 + ly;
    if (x >= nx || y >= ny) break;
    const float nu = snu[(ly + 1) * S::LW + threadIdx.x + 1];
    const size_t o = (size_t)y * nx + x, oa = (size_t)y * A.rp + x;
    float lam[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) lam[i] = adj[(size_t)i * A.ps + oa] + nu;
    if constexpr (kInit) {
      out[o] = equilibrium_vjp<float>(rho0[o], ux0 ? ux0[o] : 0.0f, uy0 ? uy0[o] : 0.0f, c, lam, th);
    } else {
#pragma unroll
      for (int i = 0; i < 9; ++i) out[(size_t)i * N + o] = lam[i];
    }
  }
  if constexpr (kInit) block_accumulate<S>(th, reinterpret_cast<double*>(sa), partials, blockIdx.x, before);
}

// Adjoint state (adj_layout) from a plain Lambda (planes nx*ny apart):
// L = lam, A = 0.
template <bool kStream>
__global__ __launch_bounds__(BLK) void adjoint_seed_kernel(const float* __restrict__ lam, float* __restrict__ adj,
                                                          int nx, int ny, Divisor width) {
  unsigned o;
  int x, y;
  if (!flat_node(nx, ny, width, o, x, y)) return;
  const Layout A = adj_layout(nx, ny);
  const Planes<float> F = planes<float>(lam, (size_t)nx * ny);
  char* const base = reinterpret_cast<char*>(adj);
  const unsigned oa = 4u * ((unsigned)y * A.rp + (unsigned)x);  // < 2^32 in both layouts
#pragma unroll
  for (int i = 0; i < 9; ++i) put<kStream>(ldb<float>(F.p[i], 4u * o), base + (size_t)i * A.ps * 4, oa);
  put<kStream>(0.0f, base + 9 * A.ps * 4, oa);
  put<kStream>(0.0f, base + 10 * A.ps * 4, oa);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
Coef<float> make_coef(const lbm_derived& d, double varpi, double a, double b) {
  Coef<double> c{};
  const double se = d.s_e, sp = d.s_p, sq = d.s_q, seps = d.s_eps, k = d.k, h = d.h, bs = d.bs;
  c.g2 = d.g2;
  c.kp = d.kp;
  c.rt = d.rt;
  c.a = a;
  c.b4 = 0.25 * b;
  c.kprt = d.kp * d.rt;
  c.e_rho = 0.5 * d.g2 - d.kp * a;
  c.de_rho = d.g2 - 2.0 * d.kp * a;
  c.alpha2 = d.alpha2;
  c.beta2 = d.beta2;
  c.k_seps_h = 0.5 * k * seps;
  c.h_sq_h = 0.5 * h * sq;
  c.b_sq = bs * sq;
  c.b_sq_h = 0.5 * bs * sq;
  c.om_e = 1.0 - 0.5 * se;
  c.om_eps = 1.0 - 0.5 * seps;
  c.om_q = 1.0 - 0.5 * sq;
  c.om_p = 1.0 - 0.5 * sp;
  c.two_om_e = 2.0 - se;
  c.two_om_p = 2.0 - sp;
  c.one_m_seps = 1.0 - seps;
  c.one_m_sq = 1.0 - sq;
  c.cR11 = -(se / (4.0 * varpi)) * (9.0 * (1.0 - k) - 2.0 * (3.0 * k + h));
  c.cR17 = -(3.0 * sp * (2.0 - se)) / (4.0 * (2.0 - sp)) * (9.0 * (1.0 - k) + 2.0 * (3.0 * k + h));
  c.cR18 = 12.0 * sp * (2.0 - se) / (2.0 - sp) * (3.0 * k + h);
  c.cT1 = 1.5 * (2.0 - se);
  c.one_mk = 1.0 - k;
  c.twok_h = 2.0 * k + h;
  c.cX1 = 4.5 * (2.0 - se) * (2.0 * k + h);
  c.cT1a = c.cT1 * (1.0 - k);
  c.cT1b = c.cT1 * (2.0 * k + h);
  c.cR71 = -(se * (2.0 - sp)) / (4.0 * varpi * (2.0 - se)) * (3.0 - 4.0 * bs);
  c.cR77 = -(3.0 * sp / 4.0) * (3.0 + 4.0 * bs);
  c.cT7 = 0.5 * (2.0 - sp);
  c.two_b = 2.0 * bs;
  c.cX7 = -3.0 * (2.0 - sp) * bs;
  c.cR81 = se * (2.0 - sp) / (varpi * (2.0 - se)) * bs;
  c.cR88 = 6.0 * sp * bs;
  c.cT8 = -0.5 * (2.0 - sp) * bs;
  c.cX8 = 1.5 * (2.0 - sp) * bs;
  c.s_e = se;
  c.kq2 = k * (0.5 * se - 1.0) * seps;
  c.s_eps = seps;
  c.s_p = sp;
  c.q1 = (se - c.kq2) * 0.5 * d.g2;
  c.q7 = sp * d.g2 / 12.0;
  c.q2 = seps * 0.5 * d.g2;
  c.s_q = sq;
  c.w_r11 = -c.cR11 / 36.0, c.w_r17 = -c.cR17 / 36.0, c.w_r18 = -c.cR18 / 36.0;
  c.w_t1a = -c.cT1a / 36.0, c.w_x1 = -c.cX1 / 36.0, c.w_t1b = c.cT1b / 36.0, c.w_q1 = c.q1 / 36.0;
  c.w_seps = seps / 36.0, c.w_q2 = c.q2 / 36.0, c.w_sq = sq / 12.0;
  c.w_r71 = -c.cR71 / 4.0, c.w_r77 = -c.cR77 / 4.0, c.w_t7 = -c.cT7 / 4.0, c.w_x7 = -c.cX7 / 4.0;
  c.w_t7b = -c.cT7 * c.two_b / 4.0, c.w_q7 = c.q7 / 4.0;
  c.w_r81 = -c.cR81 / 4.0, c.w_r88 = -c.cR88 / 4.0, c.w_x8 = -c.cX8 / 4.0, c.w_t8 = -c.cT8 / 4.0;
  Coef<float> f;
  const double* src = reinterpret_cast<const double*>(&c);
  float* dstp = reinterpret_cast<float*>(&f);
  static_assert(sizeof(Coef<double>) == 2 * sizeof(Coef<float>), "Coef layout");
  for (size_t i = 0; i < sizeof(Coef<float>) / sizeof(float); ++i) dstp[i] = (float)src[i];
  return f;
}

// Reference populations of the 2-byte storages.  eta(rho) of the model
// (p_LBE = (rho + eta)/3 with the CS pressure) is replaced by its cubic
// least-squares fit on [0, 1.25 rho_l]; any smooth fit keeps encoder and
// decoder consistent, a closer one keeps the stored deviations small.  The
// class values are those of the rest equilibrium:
//   rest  (16 rho + (4 beta2 - 8) eta)/36,  axis rho/9 - (1 + beta2) eta/18,
//   diag  rho/36 + (4 + beta2) eta/36.
RefPoly<float> make_refpoly(const lbm_derived& d, double a, double b, int storage) {
  const int n = 257;
  const double rmax = 1.25 * d.rho_l;
  double A[4][4] = {}, B[4] = {};
  for (int j = 0; j < n; ++j) {
    const double r = rmax * 0.5 * (1.0 - std::cos(M_PI * j / (n - 1)));
    const double v = 0.25 * b * r, w = 1.0 - v;
    const double z = (1.0 + v + v * v - v * v * v) / (w * w * w);
    const double p = d.kp * (r * d.rt * z - a * r * r) + 0.5 * d.g2 * r * r;
    const double eta = 3.0 * p - r;
    const double bas[4] = {1.0, r, r * r, r * r * r};
    for (int u = 0; u < 4; ++u) {
      B[u] += bas[u] * eta;
      for (int v2 = 0; v2 < 4; ++v2) A[u][v2] += bas[u] * bas[v2];
    }
  }
  // Gaussian elimination with partial pivoting (4x4)
  double e[4];
  for (int col = 0; col < 4; ++col) {
    int piv = col;
    for (int r = col + 1; r < 4; ++r)
      if (std::fabs(A[r][col]) > std::fabs(A[piv][col])) piv = r;
    for (int u = 0; u < 4; ++u) std::swap(A[col][u], A[piv][u]);
    std::swap(B[col], B[piv]);
    for (int r = col + 1; r < 4; ++r) {
      const double fac = A[r][col] / A[col][col];
      for (int u = col; u < 4; ++u) A[r][u] -= fac * A[col][u];
      B[r] -= fac * B[col];
    }
  }
  for (int r = 3; r >= 0; --r) {
    double s = B[r];
    for (int u = r + 1; u < 4; ++u) s -= A[r][u] * e[u];
    e[r] = s / A[r][r];
  }
  const double be = d.beta2;
  const double lin[3] = {16.0 / 36.0, 1.0 / 9.0, 1.0 / 36.0};  // coefficient of rho
  const double eta_c[3] = {(4.0 * be - 8.0) / 36.0, -(1.0 + be) / 18.0, (4.0 + be) / 36.0};
  RefPoly<float> q{};
  for (int cls = 0; cls < 3; ++cls)
    for (int u = 0; u < 4; ++u) q.c[cls][u] = (float)(eta_c[cls] * e[u] + (u == 1 ? lin[cls] : 0.0));
  const double S = storage == LBM_FP16 ? 4096.0 : 1.0;
  q.scale = (float)S;
  q.inv_scale = (float)(1.0 / S);
  return q;
}

}  // namespace
}  // namespace lbm

// Scratch of lbm_moments_noalloc: the per-workgroup FP64 partial sums of the
// moments kernel, in a fixed device array instead of memory the library
// allocates (callers that cannot allocate).  Every device holds its own copy
// until the process ends; host code uses the device address taken by
// hipGetSymbolAddress, never this name.  Calls on one device share it.
constexpr size_t kNoallocScratchDoubles = 262144;  // 2 MiB: 87381 workgroups of 64 x 16 nodes
static __device__ __align__(256) double scratch[kNoallocScratchDoubles];

namespace lbm {
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[kMaxDevices];  // address of `scratch` on each device, once taken

// Address of the static scratch on `device`, which must be the current
// device; taken once per device.  nullptr if the runtime cannot give it.
double* noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) == hipSuccess) g_scratch_dev[device] = static_cast<double*>(p);
  }
  return g_scratch_dev[device];
}
}  // namespace
}  // namespace lbm

using namespace lbm;

namespace {
// Results of a call that returns them to the host: written by the kernel
// itself into pinned memory and read after the stream has finished.  A copy
// to the caller's memory took another launch and a staging copy: kernel,
// copy and wait 24 us, kernel and wait 11 us.
struct alignas(64) HostWord {
  double sums[3];
  int flag;
};

// One pinned page of them for the process (allocating one per context took
// 25-80 us of lbm_create), handed out under a lock; contexts beyond 64 get
// an allocation of their own.
constexpr int kHostWords = 64;
std::mutex g_host_mu;
HostWord* g_host_page;
uint64_t g_host_used;

hipError_t take_host_word(HostWord** out) {
  std::lock_guard<std::mutex> lock(g_host_mu);
  if (!g_host_page) {
    hipError_t e = hipHostMalloc(reinterpret_cast<void**>(&g_host_page), kHostWords * sizeof(HostWord),
                                 hipHostMallocPortable);
    if (e != hipSuccess) {
      g_host_page = nullptr;
      return e;
    }
  }
  if (g_host_used == ~0ull) return hipHostMalloc(reinterpret_cast<void**>(out), sizeof(HostWord), hipHostMallocPortable);
  const int i = __builtin_ctzll(~g_host_used);
  g_host_used |= 1ull << i;
  *out = g_host_page + i;
  return hipSuccess;
}

// The word's last kernel has finished.
void give_host_word(HostWord* w) {
  std::lock_guard<std::mutex> lock(g_host_mu);
  if (w >= g_host_page && w < g_host_page + kHostWords)
    g_host_used &= ~(1ull << (w - g_host_page));
  else
    (void)hipHostFree(w);
}
}  // namespace

struct lbm_ctx {
  lbm_params p;
  lbm_derived d;
  Coef<float> c;
  RefPoly<float> q;
  void* buf[2];
  uint16_t* ref[2];  // reference-density planes (2-byte storages)
  int cur;           // buffer holding the pull source of the next step
  bool ready;        // state initialised
  int64_t t;
  hipStream_t stream;
  int device;
  bool reverse;      // direction of the last launch with cached stores (with_stores)
  int cus;           // compute units of the device (tile-shape choice)
  int nblocks;       // workgroups of the moments tile grid
  double* scratch;   // nblocks*3 partials of the moments
  int adj_blocks;    // workgroups of the adjoint tile grid
  double* theta;     // adj_blocks*3 accumulated partials of dL/dtheta
  HostWord* host;    // results the kernels write for the host (pinned), and its device address
  HostWord* host_dev;
  double* noalloc;   // the static scratch on this device (lbm_moments_noalloc), or nullptr
};

namespace {

template <class S>
int tiles_x(int nx) { return (nx + S::TX - 1) / S::TX; }

// Tile columns per strip of the tile order (TileOrder) for tiles tx nodes
// wide on a lattice nx nodes wide.  Measured on MI355X for the FP32 step and
// the adjoint, which stream their bytes from HBM: raster order up to 2048
// nodes, beyond that strips a quarter of the lattice wide and at least 1024
// nodes (4096^2: 1024-node strips, +5 %; 16384 x 8192: 4096-node strips,
// +13 % over raster).  The 2-byte steps, bound by the vector ALU, keep
// raster order (one strip).
int strip_width(int nx, int tx, bool raster) {
  const int ntx = (nx + tx - 1) / tx;
  if (raster || nx <= 2048) return ntx;
  const int nodes = nx / 4 < 1024 ? 1024 : nx / 4;
  const int w = nodes / tx;
  return w < 1 ? 1 : (w > ntx ? ntx : w);
}

// Tile columns per strip for the tiles of one node per thread, on an ntx x nty
// grid where strip_width gives `strip`: at most 32, else the tile that shares
// halo lines with the one above it comes after that XCD's L2 has let them go,
// or on another XCD (FP32, us per step, strip_width / at most 32: 50000 x 6 8.7
// / 6.0, 100000 x 30 42.4 / 35.2, 16384 x 200 36.2 / 36.2).  2-byte lattices
// in raster order only if an XCD's run is less than a row of tiles, that is
// below eight of them (20000 x 10 7.7 / 6.0, 16000 x 12 6.0 / 4.95, 6000 x 48
// 6.23 / 6.15, but 10000 x 200 18.8 / 19.1).
int near_strip_width(int strip, int nty, bool raster) { return strip > 32 && (!raster || nty < 8) ? 32 : strip; }
template <class S>
int tiles_total(int nx, int ny) { return tiles_x<S>(nx) * ((ny + S::TY - 1) / S::TY); }

// Tile rows [lo, hi) whose reads stay inside the lattice (t TY >= 2 and
// t TY + TY + 2 <= ny): the kBand launch of a wide state.
template <class S>
void band_rows(int ny, int& lo, int& hi) {
  lo = (2 + S::TY - 1) / S::TY;
  hi = ny >= S::TY + 2 ? (ny - S::TY - 2) / S::TY + 1 : 0;
  if (hi < lo) hi = lo;
}

// Launch fn(mode, rows, nrows) over every tile row of a lattice: one kAbs
// launch, or for a wide FP32 state a kBand launch over the band rows and a
// kWide launch over the rows at both ends.
template <class S, bool kFP32, class Fn>
void for_tile_rows(int nx, int ny, Fn&& fn) {
  const int nty = (ny + S::TY - 1) / S::TY;
  if constexpr (kFP32) {
    if (wide_state(nx, ny, 4)) {
      // a band of TY + 4 rows must fit 32-bit offsets (lattices up to about
      // 9M nodes wide); wider ones take 64-bit addresses on every tile row
      if (36ull * (unsigned long long)nx * (S::TY + 4) >= (1ull << 32)) {
        fn(std::integral_constant<int, kWide>{}, TileRows{0, nty, 0}, nty);
        return;
      }
      int lo, hi;
      band_rows<S>(ny, lo, hi);
      if (hi > lo) fn(std::integral_constant<int, kBand>{}, TileRows{lo, hi - lo, 0}, hi - lo);
      fn(std::integral_constant<int, kWide>{}, TileRows{0, lo, hi}, lo + nty - hi);
      return;
    }
  }
  fn(std::integral_constant<int, kAbs>{}, TileRows{0, nty, 0}, nty);
}

// Whether a kernel streams the state it writes (non-temporal stores) or
// leaves it in the caches.  bytes: the state written; row: bytes of one of
// its rows; most: the bytes of source and destination together up to which
// the next launch still finds part of them there.
//
// Three ranges, measured with every size between (us per step, streamed /
// cached; step2 is the two-step kernel, L2 4 MiB on each of 8 XCDs, memory
// cache 256 MiB):
//  - up to half the L2s the end of the launch, which writes them back, costs
//    more than the next launch gains (a little earlier where rows do not
//    start on 64 bytes): one step 640^2 5.50 / 6.46, 672^2 6.07 / 6.90, 688^2
//    8.12 / 7.04, 661 x 660 6.44 / 6.85, 666^2 7.25 / 6.95; FP16 870^2 9.0 /
//    9.4, 910^2 11.3 / 10.2, 992^2 12.8 / 12.0; adjoint 608^2 13.8 / 15.0,
//    624^2 17.3 / 16.5;
//  - rows that do not start on 64 bytes share lines between workgroups, and
//    cached stores merge them: step2 1100^2 15.9 / 14.1, 4097 x 4093 166 /
//    159, FP16 4097 x 4093 197 / 180, adjoint 493 / 440;
//  - else cached while the caches hold enough of it.  The one-step FP32 and
//    adjoint kernels and the two-step kernel that stores both states, which
//    HBM bounds, gain while the memory cache holds source and destination
//    (one step 1792^2 46.0 / 38.6, 2048^2 57.8 / 57.8, 4096^2 199 / 211;
//    adjoint 1600^2 67.8 / 65.8, 2048^2 109.8 / 110.5; both states 1536^2
//    32.7 / 31.1, 2048^2 53.3 / 54.3), the kernels the vector ALU bounds up
//    to about 640 MB (step2 2048^2 42.4 / 40.7, 3000^2 91.3 / 87.3, 4096^2
//    143.6 / 146; FP16 2048^2 48.9 / 44.9, 4000^2 164 / 158, 8192^2 627 /
//    634).
constexpr unsigned long long kCachedHbm = 288ull << 20, kCachedAlu = 640ull << 20;
bool stream_stores(unsigned long long bytes, unsigned long long row, unsigned long long most) {
  const bool aligned = row % 64 == 0;
  if (bytes < (aligned ? 16ull : 15ull) << 20) return true;
  return aligned && 2 * bytes > most;
}

// The same for the kernels of one node per thread that write a whole state
// (initial, loaded and seeded states).  Rows that do not start on 64 bytes share
// their lines with other rows, which streamed stores write in parts (us,
// streamed / cached: FP32 set_state 3 x 100000 17.5 / 7.6, 10 x 34000 8.3 / 5.4,
// 600^2 4.6 / 4.3; adjoint seed 3 x 100000 23.8 / 8.9, 380^2 3.8 / 3.3).  Whole
// rows are streamed past the caches (seed 2048^2 48 / 65, 2400^2 65 / 80) and,
// as by the step, up to half the L2s, there from about 7 MiB on (set_state
// 352 x 380 (4.6 MiB) 3.36 / 3.24, 480^2 (7.9) 3.05 / 3.46, 640^2 (14.1) 3.7 /
// 4.45, 720^2 (17.8) 5.97 / 5.63; seed 480^2 3.3 / 3.6, 1200 x 300 3.8 / 4.5).
bool past_caches(unsigned long long bytes, unsigned long long row) { return row % 64 == 0 && 2 * bytes > kCachedHbm; }
bool stream_rows(unsigned long long bytes, unsigned long long row) {
  return past_caches(bytes, row) || (row % 64 == 0 && bytes >= 7ull << 20 && bytes < 16ull << 20);
}

// Call fn with v as std::bool_constant.
template <class Fn>
void with_bool(bool v, Fn&& fn) {
  if (v)
    fn(std::true_type{});
  else
    fn(std::false_type{});
}

// Call fn(stream, reverse) for one launch (or the launches of one step):
// stream as std::bool_constant, and whether the tiles run backwards, which
// cached launches do every other time.
template <class Fn>
void with_stores(lbm_ctx* ctx, bool stream, Fn&& fn) {
  if (stream) return fn(std::true_type{}, false);
  ctx->reverse = !ctx->reverse;
  fn(std::false_type{}, ctx->reverse);
}

// One step of storage St with tile shape S from the buffer src (and its
// reference plane) to dst, on the context's stream.
template <class St, class S>
void launch_step_tiles(lbm_ctx* ctx, bool stream, const void* src, void* dst, const uint16_t* ref_in,
                       uint16_t* ref_out) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, ntx = tiles_x<S>(nx), strip = strip_width(nx, S::TX, St::kRef);
  auto columns = [&](int nrows) { return S::NPT == 1 ? near_strip_width(strip, nrows, St::kRef) : strip; };
  with_stores(ctx, stream, [&](auto str, bool reverse) {
    for_tile_rows<S, !St::kRef>(nx, ny, [&](auto mode, TileRows rows, int nrows) {
      step_kernel<S, St, decltype(mode)::value, decltype(str)::value>
          <<<ntx * nrows, dim3(S::TX, S::WY), 0, ctx->stream>>>(
              src, dst, ref_in, ref_out, nx, ny, make_order(ntx, nrows, columns(nrows), reverse), ctx->c, ctx->q, rows);
    });
  });
}

// Whether one 2-byte step takes the 64 x 4 tiles of FP32: at most one 64 x 8
// tile per two CUs, where the launch is as long as one workgroup (us, 64 x 4 /
// 64 x 8: 64^2 3.5 / 3.7, 160^2 3.6 / 3.8, 256^2 3.65 / 3.8, 10 x 1000 3.8 / 4.1),
// unless the last tile column has only up to eight nodes (waves with so few
// active lanes run slower, and 64 x 4 tiles have twice as many: 200^2 4.9 / 3.95,
// 72^2 4.85 / 4.5, 8 x 1000 5.0 / 3.95).
template <class St>
bool small_2byte(int nx, int ny, int cus) {
  return St::kRef && (nx - 1) % 64 >= 8 && 2 * tiles_total<NearTile<St>>(nx, ny) <= cus;
}

// One step: NearTile while the 256 MiB memory cache holds source and
// destination, StepTile beyond.  Measured, us per step, NearTile / StepTile
// (FP32 on small lattices: 128 x 8): FP32 512^2 4.72 / 5.05, 560^2 5.00 /
// 6.33, 1000 x 700 9.4 / 12.4, 2085 x 1035 25.5 / 30.2, 1900^2 39.1 / 44.7,
// 1984^2 59.7 / 57.6, 2048^2 68.1 / 57.8, 4096^2 257 / 197; FP16 1000 x 700
// 8.36 / 9.79, 1024^2 12.4 / 14.0, 2048^2 38.7 / 45.0, 2560^2 64.8 / 66.0,
// 3072^2 103.9 / 99.2, 4096^2 167.1 / 162.7, 8192^2 634 / 618.  The per-node
// arithmetic does not depend on the tile, so both give the same bits.
template <class St>
void launch_step(lbm_ctx* ctx, const void* src, void* dst, const uint16_t* ref_in, uint16_t* ref_out) {
  const int nx = ctx->p.nx, ny = ctx->p.ny;
  const unsigned long long bytes = (9ull * St::ES + (St::kRef ? 2 : 0)) * nx * ny;
  const bool stream = stream_stores(bytes, (unsigned long long)St::ES * nx, St::kRef ? kCachedAlu : kCachedHbm);
  if (small_2byte<St>(nx, ny, ctx->cus))
    launch_step_tiles<St, NearTile<StoreF32>>(ctx, stream, src, dst, ref_in, ref_out);
  else if (2 * bytes <= 256ull << 20)
    launch_step_tiles<St, NearTile<St>>(ctx, stream, src, dst, ref_in, ref_out);
  else
    launch_step_tiles<St, StepTile<St>>(ctx, stream, src, dst, ref_in, ref_out);
}

// Two FP32 steps per launch (step2_kernel), on lattices too large for
// stepk_kernel: tiles of 64 x 24 or of 64 x 16 (mid_tile_first).  The tiles
// address TY + 8 rows of 36 nx bytes from one base with 32-bit offsets,
// which bounds the width (about 3.7M nodes); wider lattices take single
// steps.
using Step2Mid = Tile2Shape<64, 16, 8>;
static_assert(Step2Mid::TY <= Step2Tile::TY, "the width bound of the large tile covers the other");

bool use_step2(const lbm_ctx* ctx) {
  const unsigned long long band = 36ull * (unsigned long long)ctx->p.nx * (Step2Tile::TY + 8);
  return ctx->p.storage == LBM_FP32 && band < (1ull << 32);
}

// src (time t) -> dst (time t + 2), and mid (time t + 1) if kMid.
template <class S, bool kMid>
void launch_step2_on(lbm_ctx* ctx, const void* src, void* mid, void* dst) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, ntx = tiles_x<S>(nx), nt = tiles_total<S>(nx, ny);
  with_stores(ctx, stream_stores(36ull * nx * ny, 4ull * nx, kMid ? kCachedHbm : kCachedAlu), [&](auto str, bool reverse) {
    step2_kernel<S, kMid, decltype(str)::value><<<nt, dim3(S::TX, S::WY), 0, ctx->stream>>>(
        static_cast<const float*>(src), static_cast<float*>(mid), static_cast<float*>(dst), nx, ny,
        make_order(ntx, nt / ntx, strip_width(nx, S::TX, false), reverse), ctx->c);
  });
}
// k steps of storage St per launch on small lattices (stepk_kernel).
using StepKTiny = TileKShape<4, 4, 4>;
using StepKSmall = TileKShape<8, 8, 4>;
using StepKWide = TileKShape<32, 8, 3>;
using StepKLast = TileKShape<16, 16, 2>;

// 16 x 16 tiles per CU, in tenths, up to which stepk_kernel advances an FP32
// lattice two steps faster than the two-step kernel, whose time goes by the
// turns the CUs take through its tiles.  Measured, us per 20 steps, 16 x 16 /
// 64 x 16 / 64 x 24 tiles, 16 x 16 tiles per CU in brackets:
//  - at most one 64 x 16 tile per CU: 400^2 (2.4) 77 / 82 / 99, 432^2 (2.8) 78
//    / 82 / 98, 6000 x 24 (2.9) 97 / 89 / 95, 448^2 (3.1) 86 / 83 / 99, 2000 x
//    112 (3.4) 98 / 84 / 97, 512^2 (4.0) 93 / 81 / 98;
//  - else one 64 x 24 tile: 520^2 (4.3) 104 / 120 / 105, 544^2 (4.5) 107 / 112
//    / 97, 100 x 3000 (5.1) 112 / 111 / 98, 600^2 (5.6) 120 / 111 / 98, 16000 x
//    24 (7.8) 164 / 131 / 106;
//  - else two 64 x 16 tiles: 72 x 3400 (4.2) 100 / 121 / 155, 20000 x 5 (4.9)
//    87 / 91 / 110, 608^2 (5.6) 120 / 111 / 142, 200 x 1800 (5.7) 118 / 121 /
//    154, 700^2 (7.6) 151 / 130 / 160;
//  - else: 712^2 (7.9) 161 / 171 / 160, 740^2 (8.6) 164 / 167 / 163.
// Storing every state as well (us for 8 steps): 380^2 (2.3) 31.3 / 32.2 / 38.6,
// 400^2 (2.4) 35.0 / 33.3 / 41.0.  The two-step kernel streams the state
// between, and beyond one 64 x 16 tile per CU wins only with rows on 64 bytes:
// 544^2 (4.5) 47.6 / 50.9 / 44.8, 576^2 (5.1) 51.6 / 51.1 / 45.7, 4064 x 89
// (6.0) 59.5 / - / 51.4, 640^2 (6.3) 58.7 / 51.7 / 65.6, but 568^2 (5.1) 52.4 /
// 52.1 / 53.7, 300 x 1200 (5.6) 53.6 / 56.7 / 61.2, 620^2 (5.9) 54.5 / 58.2 /
// 68.0, 660^2 (6.9) 64.5 / 64.5 / 71.0; and on one row of tiles 10000 x 16 (2.4)
// 31.9 / 34.0.
// The odd step behind two-step launches finds its instructions cold, which
// costs it about 2.5 us more than behind stepk_kernel's short loop: n steps in
// a call (us, 16 x 16 tiles / the two-step kernel), n = 3: 440^2 (3.1) 12.9 /
// 13.4, 520^2 15.4 / 16.6, 600^2 17.5 / 18.0, 620^2 (5.9) 17.9 / 19.8, 640^2 (6.3)
// 18.5 / 16.6; n = 5: 440^2 21.1 / 22.1, 540^2 26.2 / 25.5, 600^2 29.6 / 27.2, 620^2
// 30.0 / 31.1; n = 7: 620^2 42.1 / 42.5.  Not on wide lattices, where the rows of
// 16 x 16 tiles lie far apart in the launch (n = 3: 1200 x 300 17.9 / 18.7, 2000
// x 180 20.6 / 19.7, 4064 x 89 26.9 / 18.1).
template <bool kChain>
int last_tile_limit(const lbm_ctx* ctx, int n) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, cus = ctx->cus;
  const int mid = tiles_total<Step2Mid>(nx, ny);
  const bool odd = n % 2 && n < 8 && nx <= 1800;
  if (mid <= cus) return kChain ? (ny <= 16 ? 31 : 23) : (odd ? 31 : 29);
  if (kChain && nx % 16) return 65;
  if (tiles_total<Step2Tile>(nx, ny) <= cus) return !kChain && odd && n == 3 ? 60 : 42;
  if (mid <= 2 * cus) return !kChain && odd ? 60 : 55;
  return kChain ? 65 : 85;
}

// The tile of stepk_kernel (1 .. 4, in the order above) for n steps, or 0 where
// the other kernels are faster.  The more steps per launch, the smaller the tile
// has to be for one thread per node of it and its rings; a tile is taken
// while the lattice gives the CUs one (4 x 4) or two of them.  Measured, us
// per step, 4 x 4 / 8 x 8 / 32 x 8 / 16 x 16 tiles / without stepk_kernel:
//   FP32  64^2 1.43 / 1.55 / 1.97 / 2.43 / 2.69    128^2 2.09 / 1.60 / 2.11 / 2.39 / 2.73
//         200 x 160 3.33 / 2.04 / 2.21 / 2.64 / 2.90    256^2 5.55 / 2.76 / 2.18 / 2.54 / 2.83
//         350^2 9.26 / 4.06 / 2.77 / 3.23 / 3.54    400^2 11.6 / 4.94 / 3.97 / 3.70 / 4.18
//   FP16  64^2 1.66 / 1.80 / 2.23 / 2.61 / 4.06    256^2 9.3 / 3.39 / 2.40 / 2.76 / 3.59
//         350^2 16.4 / 5.43 / 3.17 / 3.56 / 4.86    400^2 20.8 / 6.59 / 4.31 / 4.16 / 5.08
// The last tile ends where the kernels with larger tiles fill the chip: FP32
// by last_tile_limit; 2-byte (16 x 16 / single steps) 500^2 5.2 / 5.4, 560^2
// 6.2 / 6.4, 600^2 6.57 / 6.27, 640^2 7.56 / 6.92, 700^2 8.26 / 6.95.  Single
// 2-byte steps also win where 16 x 16 tiles hold more rows past the lattice
// than the 64 x 8 tiles of the single step: from three tiles per CU on, more
// than 2.2 of them per 64 x 8 tile (16 x 16 / single, tiles per CU and per 64 x
// 8 tile in brackets): 20000 x 4 5.45 / 4.35 (4.9, 4.0), 10000 x 24 7.1 / 5.35
// (4.9, 2.7), 4800 x 40 5.65 / 5.1 (3.5, 2.4), 3000 x 72 5.55 / 5.25 (3.7,
// 2.2), but 4000 x 40 4.65 / 5.0 (2.9, 2.4), 5500 x 24 4.7 / 4.8 (2.7, 2.7),
// 16000 x 9 4.95 / 6.3 (3.9, 2.0).
template <class St, bool kChain>
int stepk_shape(const lbm_ctx* ctx, int n) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, cus = ctx->cus;
  if (tiles_total<StepKTiny>(nx, ny) <= cus) return 1;
  if (tiles_total<StepKSmall>(nx, ny) <= 2 * cus) return 2;
  if (tiles_total<StepKWide>(nx, ny) <= 2 * cus) return 3;
  const int t = tiles_total<StepKLast>(nx, ny);
  if constexpr (St::kRef) {
    const bool sparse = t > 3 * cus && 10 * t > 22 * tiles_total<NearTile<St>>(nx, ny);
    return !sparse && 2 * t <= 11 * cus ? 4 : 0;
  } else {
    return 10 * t <= last_tile_limit<kChain>(ctx, n) * cus ? 4 : 0;
  }
}

// Whether the 64 x 16 tile finishes the lattice first: the CUs work through
// ceil(tiles / CUs) workgroups each, and one of its takes 0.73 of the time of
// one of 64 x 24.  Where the larger tile leaves its last turn nearly empty
// the smaller one wins (us per step, 64 x 24 / 64 x 16, workgroups per CU in
// brackets): 830^2 8.5 / 8.7 (1.8 / 2.6), 900^2 11.0 / 10.4 (2.2 / 3.3), 1024^2
// 11.9 / 11.5 (2.7 / 4), 1100^2 14.1 / 13.5 (3.2 / 4.9), 1200^2 14.9 / 15.4
// (3.7 / 5.6), 1500^2 21.5 / 23.3 (5.9 / 8.8).
bool mid_tile_first(const lbm_ctx* ctx) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, cus = ctx->cus;
  const long long large = (tiles_total<Step2Tile>(nx, ny) + cus - 1) / cus;
  const long long mid = (tiles_total<Step2Mid>(nx, ny) + cus - 1) / cus;
  return 73 * mid < 100 * large;
}

// Launch of march_kernel: as many segments as give every CU `rounds`
// workgroups in turn, the number of rounds that costs the fewest iterations.
struct MarchPlan {
  int rounds, rows, segs, blocks, lanes;
};
constexpr int kMarchFill = 8;  // rows that filling and draining a segment's pipeline costs

MarchPlan march_plan(int nx, int ny, int cus) {
  const int full = nx / kMarchCols, rest = nx % kMarchCols;
  const int lanes = rest ? (rest + kMarchLeft + 3 + 63) / 64 * 64 : kMarchThreads, parts = kMarchThreads / lanes;
  MarchPlan best{0, 0, 0, 0, lanes};
  long long least = 0;
  for (int r = 1; r <= 4; ++r)
    for (int rows = (int)((long long)ny * full / ((long long)r * cus)) + 1; rows <= ny; ++rows) {
      const int segs = (ny + rows - 1) / rows;
      const long long blocks = (long long)full * segs + (rest ? (segs + parts - 1) / parts : 0);
      if (blocks > (long long)r * cus) continue;
      const long long cost = (long long)r * (rows + kMarchFill);
      if (best.rounds == 0 || cost < least) best = {r, rows, segs, (int)blocks, lanes}, least = cost;
      break;
    }
  return best;
}

// Whether march_kernel takes the two steps: a full strip, and iterations that
// would advance at most 1.3 times the lattice's nodes if every CU spent each
// on a full row of a strip.  Measured, that ratio and us per step, step2_kernel
// / march_kernel: 16384 x 8192 1.07 1103 / 975, 8192^2 1.10 542 / 487, 4096^2
// 1.14 142.9 / 131.9, 1000 x 20000 1.19 177.0 / 168.3, 2880^2 1.24 79.0 / 76.1,
// 3000^2 1.26 86.2 / 82.2, 960 x 8192 1.28 72.8 / 73.0, 2700^2 1.35 70.7 / 69.8,
// 2304^2 1.44 53.4 / 52.2, 2560^2 1.46 63.9 / 64.5, 2048^2 1.52 40.1 / 40.1.
bool use_march(const lbm_ctx* ctx, MarchPlan& plan) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, cus = ctx->cus;
  const long long nodes = (long long)nx * ny, row = (long long)cus * kMarchCols;  // row: nodes an iteration advances
  if (nx < kMarchCols || 3 * nodes < 10 * kMarchFill * row) return false;
  plan = march_plan(nx, ny, cus);
  return plan.rounds && 10 * plan.rounds * (plan.rows + kMarchFill) * row <= 13 * nodes;
}

void launch_march(lbm_ctx* ctx, const MarchPlan& plan, const void* src, void* dst) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, full = nx / kMarchCols;
  const MarchGrid grid{(unsigned)(full * plan.segs), (unsigned)plan.segs, make_divisor((unsigned)full),
                       make_divisor((unsigned)plan.lanes), plan.rows};
  with_bool(stream_stores(36ull * nx * ny, 4ull * nx, kCachedAlu), [&](auto stream) {
    march_kernel<decltype(stream)::value><<<plan.blocks, kMarchThreads, 0, ctx->stream>>>(
        static_cast<const float*>(src), static_cast<float*>(dst), nx, ny, grid, ctx->c);
  });
}

template <bool kMid>
void launch_step2(lbm_ctx* ctx, const void* src, void* mid, void* dst) {
  if constexpr (!kMid)
    if (MarchPlan plan; use_march(ctx, plan)) return launch_march(ctx, plan, src, dst);
  if (mid_tile_first(ctx))
    launch_step2_on<Step2Mid, kMid>(ctx, src, mid, dst);
  else
    launch_step2_on<Step2Tile, kMid>(ctx, src, mid, dst);
}

// Call fn with the tile of stepk_shape (1 .. 4).
template <class Fn>
void with_stepk(int shape, Fn&& fn) {
  switch (shape) {
    case 1: fn(StepKTiny{}); break;
    case 2: fn(StepKSmall{}); break;
    case 3: fn(StepKWide{}); break;
    default: fn(StepKLast{}); break;
  }
}

// k steps from the buffer src; a single step is the step kernel's.
template <class St, class S>
void launch_stepk(lbm_ctx* ctx, const void* src, const StepOuts<S::K>& outs, int k, const uint16_t* ref_in,
                  uint16_t* ref_out) {
  if (k == 1) return launch_step<St>(ctx, src, outs.p[0], ref_in, ref_out);
  const int nx = ctx->p.nx, ny = ctx->p.ny, ntx = tiles_x<S>(nx), nt = tiles_total<S>(nx, ny);
  stepk_kernel<S, St><<<nt, S::NT, 0, ctx->stream>>>(src, outs, ref_in, ref_out, nx, ny,
                                                     make_order(ntx, nt / ntx, ntx, false), k, ctx->c, ctx->q);
}

// Whether the adjoint step takes AdjTileSmall: at most three of its tiles per
// CU.  A step is then as long as one wave's instructions, which one node per
// thread halves: us per step, two nodes / one, 64^2 6.62 / 5.32, 256^2 7.05 /
// 5.74, 400^2 9.96 / 8.61, but 450^2 10.3 / 10.7, 512^2 10.9 / 11.0.  A last
// tile column of up to eight nodes costs the wider tile most: waves with so
// few active lanes ran the sweep three times slower (70 x 64 12.8 / 5.4).  Also
// on lattices one of its tiles wide, which the wider tile sweeps with as many
// workgroups and half their lanes or more idle (1 x 16000 24.5 / 13.1, 8 x 50000
// 66 / 34, 32 x 20000 27.6 / 17.7, but 33 x 20000 26.0 / 26.0).
bool small_adjoint(const lbm_ctx* ctx) {
  using S = AdjTileSmall;
  return ctx->p.nx <= S::TX || tiles_total<S>(ctx->p.nx, ctx->p.ny) <= 3 * ctx->cus;
}

int check_ctx(const lbm_ctx* ctx, bool need_state) {
  if (!ctx) return fail(LBM_EINVAL, "context is NULL");
  if (need_state && !ctx->ready) return fail(LBM_ESTATE, "state not initialised (call lbm_init or lbm_set_state)");
  return LBM_OK;
}

int set_device(const lbm_ctx* ctx) {
  int cur = -1;
  HIP_OK(hipGetDevice(&cur));
  if (cur != ctx->device) HIP_OK(hipSetDevice(ctx->device));
  return LBM_OK;
}

// Workgroups of one node per thread; lbm_create admits 9 nx ny < 2^31, so
// the count fits a grid dimension.
unsigned grid1(size_t n) { return static_cast<unsigned>((n + BLK - 1) / BLK); }

// Call fn(wide, stream): 64-bit addresses for FP32 states above 4 GiB, and the
// store policy.
template <class St, class Fn>
void with_state_access(const lbm_ctx* ctx, bool stream, Fn&& fn) {
  with_bool(stream, [&](auto str) {
    if constexpr (St::kRef)
      fn(std::false_type{}, str);
    else
      with_bool(wide_state(ctx->p.nx, ctx->p.ny, 4), [&](auto wide) { fn(wide, str); });
  });
}

// Queue the initial state (init_rest_kernel where it streams, at rest, and
// its tiles' rows fit 32-bit offsets; else init_kernel).  init_kernel stores
// rows shifted by the streaming, which the caches merge better in FP32 (with
// velocities, us, streamed / cached: 2880^2 108 / 93, 3600^2 183 / 144, 8192^2
// 667 / 651; 2-byte 3200^2 74 / 87, 4096^2 111 / 124).
template <class St>
void launch_init(const lbm_ctx* ctx, const float* rho0, const float* ux0, const float* uy0) {
  const int nx = ctx->p.nx, ny = ctx->p.ny;
  const bool rest = !ux0 && !uy0;
  int* const flag = &ctx->host_dev->flag;
  const unsigned long long row = 9ull * St::ES * nx;
  with_state_access<St>(ctx, past_caches(row * ny, row / 9), [&](auto wide, auto stream) {
    using S = InitTile<St>;
    if constexpr (decltype(stream)::value)
      if (rest && row * S::TY < 1ull << 32) {
        const int ntx = tiles_x<S>(nx), nt = tiles_total<S>(nx, ny);
        init_rest_kernel<St><<<nt, dim3(S::TX, S::WY), 0, ctx->stream>>>(
            rho0, ctx->buf[0], ctx->ref[0], nx, ny, make_order(ntx, nt / ntx, strip_width(nx, S::TX, false), false),
            ctx->c, ctx->q, flag);
        return;
      }
    with_bool(rest, [&](auto r) {
      init_kernel<St, decltype(wide)::value, St::kRef && decltype(stream)::value, decltype(r)::value>
          <<<grid1((size_t)nx * ny), BLK, 0, ctx->stream>>>(rho0, ux0, uy0, ctx->buf[0], ctx->ref[0], nx, ny,
                                                           make_divisor(nx), ctx->c, ctx->q, flag);
    });
  });
}

// Queue the loaded state f.  FP32 states that are streamed (stream_rows), and
// those whose populations the memory cache does not hold beside the caller's,
// take the shift in the loads (us, loads / stores: 1584 x 2392 45.4 / 46.5, 3000
// x 8000 325 / 341, streamed 2400^2 62 / 77, 8192^2 816 / 920), the others in
// the stores, which the caches merge (300 x 2800 11.3 / 10.6, 1000^2 12.5 /
// 12.0, 1500^2 26.7 / 26.3).  2-byte states store shifted rows, streamed only
// in two ranges of sizes and not short ones (us, streamed / cached: 760^2 (9.9
// MiB) 5.4 / 5.0, 820^2 (11.5) 6.0 / 6.5, 1000 x 800 (13.7) 6.9 / 7.9, 4 x 100000
// (6.9) 9.9 / 7.2; 4000^2 188 / 167, 8192^2 766 / 732; with the step and the
// export behind, 440^2 (3.3) 13.4 / 13.4, 500^2 (4.3) 14.5 / 15.1, 600^2 (6.2)
// 18.5 / 19.6, 660^2 (7.5) 21.0 / 20.6, 760^2 25.4 / 23.1).
template <class St>
void launch_set(const lbm_ctx* ctx, const float* f) {
  const int nx = ctx->p.nx, ny = ctx->p.ny;
  const unsigned long long row = (unsigned long long)St::ES * nx, bytes = 9 * row * ny;
  const unsigned long long half = bytes >> 19;  // half MiB
  const bool stream =
      St::kRef ? row >= 512 && ((half >= 8 && half < 14) || (half >= 21 && half < 32)) : stream_rows(bytes, row);
  with_state_access<St>(ctx, stream, [&](auto wide, auto str) {
    with_bool(!St::kRef && (stream || 2 * bytes > 256ull << 20), [&](auto loads) {
      constexpr bool kLoads = !St::kRef && decltype(loads)::value;
      set_state_kernel<St, decltype(wide)::value, kLoads, decltype(str)::value && (kLoads || St::kRef)>
          <<<grid1((size_t)nx * ny), BLK, 0, ctx->stream>>>(f, ctx->buf[0], ctx->ref[0], nx, ny, make_divisor(nx),
                                                           ctx->q);
    });
  });
}

// Call fn with the storage policy of the context.
template <class Fn>
int with_storage(const lbm_ctx* ctx, Fn&& fn) {
  switch (ctx->p.storage) {
    case LBM_FP32: return fn(StoreF32{});
    case LBM_FP16: return fn(Store16<LBM_FP16>{});
    default: return fn(Store16<LBM_BF16>{});
  }
}

}  // namespace

extern "C" {

const char* lbm_last_error(void) { return g_err; }

int lbm_derive(const lbm_params* p, lbm_derived* out) {
  if (!out) return fail(LBM_EINVAL, "out is NULL");
  return lbm::derive(p, out, g_err, sizeof g_err);
}

int lbm_sigma_paper(double width, double tr, double a, double b, double r_gas, double* sigma_out) {
  if (!sigma_out) return fail(LBM_EINVAL, "sigma_out is NULL");
  if (!(width > 0) || !(tr > 0 && tr < 1) || !(a > 0) || !(b > 0) || !(r_gas > 0))
    return fail(LBM_EINVAL, "invalid parameter: width, a, b, r_gas > 0 and 0 < tr < 1 required");
  int st = lbm::sigma_paper(width, tr, a, b, r_gas, sigma_out);
  return st ? fail(st, "no two-phase coexistence found at tr = %g", tr) : LBM_OK;
}

size_t lbm_state_bytes(const lbm_params* p) {
  char msg[256];
  if (lbm::validate(p, msg, sizeof msg)) return 0;
  const int es = p->storage == LBM_FP32 ? 4 : 2;
  return (size_t)9 * plane_elems(p->nx, p->ny, es) * es;
}

size_t lbm_ref_bytes(const lbm_params* p) {
  char msg[256];
  if (lbm::validate(p, msg, sizeof msg) || p->storage == LBM_FP32) return 0;
  return (size_t)2 * p->nx * p->ny * 2;
}

int lbm_create(lbm_ctx** out, const lbm_params* p, void* f_a, void* f_b, void* rho_ref, void* stream) {
  if (!out) return fail(LBM_EINVAL, "out is NULL");
  *out = nullptr;
  lbm_derived d;
  int st = lbm::derive(p, &d, g_err, sizeof g_err);
  if (st) return st;
  if (!f_a || !f_b || f_a == f_b) return fail(LBM_EINVAL, "f_a and f_b must be two distinct device buffers");
  if (p->storage != LBM_FP32 && !rho_ref)
    return fail(LBM_EINVAL, "the 2-byte storages need the reference-density buffer rho_ref");
  lbm_ctx* c = new (std::nothrow) lbm_ctx{};
  if (!c) return fail(LBM_EHIP, "out of host memory");
  c->p = *p;
  c->d = d;
  c->c = make_coef(d, p->varpi, p->a, p->b);
  c->q = make_refpoly(d, p->a, p->b, p->storage);
  c->buf[0] = f_a;
  c->buf[1] = f_b;
  const size_t N = (size_t)p->nx * p->ny;
  c->ref[0] = p->storage == LBM_FP32 ? nullptr : reinterpret_cast<uint16_t*>(rho_ref);
  c->ref[1] = p->storage == LBM_FP32 ? nullptr : reinterpret_cast<uint16_t*>(rho_ref) + N;
  c->cur = 0;
  c->ready = false;
  c->t = 0;
  c->stream = (hipStream_t)stream;
  c->nblocks = tiles_total<MomTile>(p->nx, p->ny);
  hipError_t e = hipGetDevice(&c->device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device);
  if (p->storage == LBM_FP32)
    c->adj_blocks = small_adjoint(c) ? tiles_total<AdjTileSmall>(p->nx, p->ny) : tiles_total<AdjTile>(p->nx, p->ny);
  const size_t mom_doubles = 3 * (size_t)c->nblocks, th_doubles = 3 * (size_t)c->adj_blocks;
  if (e == hipSuccess) e = hipMalloc(&c->scratch, sizeof(double) * (mom_doubles + th_doubles));
  if (e == hipSuccess) e = hipMemsetAsync(c->scratch, 0, sizeof(double) * (mom_doubles + th_doubles), c->stream);
  if (e == hipSuccess) e = take_host_word(&c->host);
  if (e == hipSuccess) e = hipHostGetDevicePointer(reinterpret_cast<void**>(&c->host_dev), c->host, 0);
  if (e != hipSuccess) {
    if (c->scratch) (void)hipFree(c->scratch);
    if (c->host) give_host_word(c->host);
    delete c;
    return fail(LBM_EHIP, "lbm_create: %s", hipGetErrorString(e));
  }
  c->theta = c->scratch + mom_doubles;
  c->noalloc = noalloc_scratch(c->device);  // c->device is current here
  *out = c;
  return LBM_OK;
}

int lbm_set_stream(lbm_ctx* ctx, void* stream) {
  if (int st = check_ctx(ctx, false)) return st;
  const hipStream_t next = (hipStream_t)stream;
  if (next != ctx->stream) {
    // work queued on the old stream precedes everything issued on the new one
    if (int st = set_device(ctx)) return st;
    hipEvent_t ev;
    HIP_OK(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    hipError_t e = hipEventRecord(ev, ctx->stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(next, ev, 0);
    (void)hipEventDestroy(ev);  // released once the wait has been satisfied
    if (e != hipSuccess) return fail(LBM_EHIP, "lbm_set_stream: %s", hipGetErrorString(e));
  }
  ctx->stream = next;
  return LBM_OK;
}

int lbm_init(lbm_ctx* ctx, const float* rho0, const float* ux0, const float* uy0) {
  if (int st = check_ctx(ctx, false)) return st;
  if (!rho0) return fail(LBM_EINVAL, "rho0 is NULL");
  if (int st = set_device(ctx)) return st;
  ctx->host->flag = 0;  // no kernel that sets it is in flight: this call waits for its own
  int st = with_storage(ctx, [&](auto store) -> int {
    launch_init<decltype(store)>(ctx, rho0, ux0, uy0);
    HIP_OK(hipGetLastError());
    return LBM_OK;
  });
  if (st) return st;
  HIP_OK(hipStreamSynchronize(ctx->stream));
  if (ctx->host->flag) {
    ctx->ready = false;
    return fail(LBM_EINVAL, "rho0 must be finite and in (0, 4/b), u0 finite");
  }
  ctx->cur = 0;
  ctx->t = 0;
  ctx->ready = true;
  return LBM_OK;
}

int lbm_set_state(lbm_ctx* ctx, const float* f) {
  if (int st = check_ctx(ctx, false)) return st;
  if (!f) return fail(LBM_EINVAL, "f is NULL");
  if (int st = set_device(ctx)) return st;
  int st = with_storage(ctx, [&](auto store) -> int {
    launch_set<decltype(store)>(ctx, f);
    HIP_OK(hipGetLastError());
    return LBM_OK;
  });
  if (st) return st;
  ctx->cur = 0;
  ctx->t = 0;
  ctx->ready = true;
  return LBM_OK;
}

int lbm_get_state(lbm_ctx* ctx, float* f) {
  if (int st = check_ctx(ctx, true)) return st;
  if (!f) return fail(LBM_EINVAL, "f is NULL");
  if (int st = set_device(ctx)) return st;
  const int nx = ctx->p.nx, ny = ctx->p.ny;
  return with_storage(ctx, [&](auto store) -> int {
    using St = decltype(store);
    auto go = [&](auto wide, auto lane) {
      get_state_kernel<St, decltype(wide)::value, decltype(lane)::value>
          <<<grid1((size_t)nx * ny), BLK, 0, ctx->stream>>>(ctx->buf[ctx->cur], ctx->ref[ctx->cur], f, nx, ny,
                                                           make_divisor(nx), ctx->q);
    };
    // 2-byte states whose populations the memory cache does not hold take
    // per-lane store addresses (FP16, us, from uniform bases / per lane: 2880^2
    // 85.4 / 79.9, 4097^2 200 / 191, 6000^2 364 / 342, but 5000 x 1000 47.1 /
    // 48.8, 640^2 4.9 / 4.8; FP32 the same either way)
    if constexpr (St::kRef)
      with_bool(36ull * nx * ny > 256ull << 20, [&](auto lane) { go(std::false_type{}, lane); });
    else
      with_bool(wide_state(nx, ny, 4), [&](auto wide) { go(wide, std::false_type{}); });
    HIP_OK(hipGetLastError());
    return LBM_OK;
  });
}

int lbm_step(lbm_ctx* ctx, int32_t n) {
  if (int st = check_ctx(ctx, true)) return st;
  if (n < 0) return fail(LBM_EINVAL, "n must be >= 0");
  if (n == 0) return LBM_OK;
  if (int st = set_device(ctx)) return st;
  int st = with_storage(ctx, [&](auto store) -> int {
    using St = decltype(store);
    if (const int shape = kFuseSteps ? stepk_shape<St, false>(ctx, n) : 0) {
      with_stepk(shape, [&](auto tile) {
        using S = decltype(tile);
        // as few launches as K steps each allow, of about equal length; for n
        // a multiple of 4 an even number, so that a captured call ends on the
        // buffer it started from
        int32_t launches = n / S::K + (n % S::K != 0);
        if (n % 4 == 0) launches += launches & 1;
        for (int32_t left = n; launches > 0; --launches) {
          const int a = ctx->cur, b = ctx->cur ^ 1, k = left / launches + (left % launches != 0);
          StepOuts<S::K> outs{};
          outs.p[k - 1] = ctx->buf[b];
          launch_stepk<St, S>(ctx, ctx->buf[a], outs, k, ctx->ref[a], ctx->ref[b]);
          left -= k;
          ctx->cur = b;
        }
      });
      HIP_OK(hipGetLastError());
      return LBM_OK;
    }
    for (int32_t s = 0; s < n;) {
      const int a = ctx->cur, b = ctx->cur ^ 1;
      if (kFuseSteps && std::is_same_v<St, StoreF32> && n - s >= 2 && use_step2(ctx)) {
        launch_step2<false>(ctx, ctx->buf[a], nullptr, ctx->buf[b]);
        s += 2;
      } else {
        launch_step<St>(ctx, ctx->buf[a], ctx->buf[b], ctx->ref[a], ctx->ref[b]);
        ++s;
      }
      ctx->cur = b;
    }
    HIP_OK(hipGetLastError());
    return LBM_OK;
  });
  if (st) return st;
  ctx->t += n;
  return LBM_OK;
}

namespace {
// The moments kernel over the current state, its per-workgroup partials
// into `partials` (3 per workgroup of tiles_total<MomTile>).
int launch_moments(const lbm_ctx* ctx, float* rho, float* ux, float* uy, double* partials) {
  using S = MomTile;
  return with_storage(ctx, [&](auto store) -> int {
    using St = decltype(store);
    const int nx = ctx->p.nx, ny = ctx->p.ny, ntx = tiles_x<S>(nx);
    with_bool(ux || uy, [&](auto vel) {
      for_tile_rows<S, !St::kRef>(nx, ny, [&](auto mode, TileRows rows, int nrows) {
        moments_kernel<St, decltype(mode)::value, decltype(vel)::value>
            <<<ntx * nrows, dim3(S::TX, S::WY), 0, ctx->stream>>>(
                ctx->buf[ctx->cur], ctx->ref[ctx->cur], rho, ux, uy, partials, nx, ny, ntx,
                make_order(ntx, nrows, strip_width(nx, S::TX, false), false), ctx->c, ctx->q, rows);
      });
    });
    HIP_OK(hipGetLastError());
    return LBM_OK;
  });
}
}  // namespace

int lbm_moments(lbm_ctx* ctx, float* rho, float* ux, float* uy, double totals[3]) {
  if (int st = check_ctx(ctx, true)) return st;
  if (int st = set_device(ctx)) return st;
  if (int st = launch_moments(ctx, rho, ux, uy, ctx->scratch)) return st;
  if (!totals) return LBM_OK;
  finish_sums<false><<<1, RED, 0, ctx->stream>>>(ctx->scratch, ctx->nblocks, ctx->host_dev->sums);
  HIP_OK(hipGetLastError());
  HIP_OK(hipStreamSynchronize(ctx->stream));
  for (int k = 0; k < 3; ++k) totals[k] = ctx->host->sums[k];
  for (int k = 0; k < 3; ++k)
    if (!std::isfinite(totals[k])) return fail(LBM_ENONFINITE, "non-finite total (%d): the state has diverged", k);
  return LBM_OK;
}

int lbm_moments_noalloc(lbm_ctx* ctx, float* rho, float* ux, float* uy, double* totals_dev) {
  if (!ctx) return fail(LBM_EINVAL, "context is NULL");
  if (3 * (size_t)ctx->nblocks > kNoallocScratchDoubles)
    return fail(LBM_EINVAL,
                "lbm_moments_noalloc: a %d x %d lattice needs %zu doubles of scratch, the static maximum is %zu "
                "(%zu workgroups of 64 x 16 nodes); use lbm_moments",
                ctx->p.nx, ctx->p.ny, 3 * (size_t)ctx->nblocks, kNoallocScratchDoubles, kNoallocScratchDoubles / 3);
  if (int st = check_ctx(ctx, true)) return st;
  if (!ctx->noalloc) return fail(LBM_EHIP, "lbm_moments_noalloc: the static scratch has no device address");
  if (int st = set_device(ctx)) return st;
  if (int st = launch_moments(ctx, rho, ux, uy, ctx->noalloc)) return st;
  if (totals_dev) {
    finish_sums<false><<<1, RED, 0, ctx->stream>>>(ctx->noalloc, ctx->nblocks, totals_dev);
    HIP_OK(hipGetLastError());
  }
  return LBM_OK;
}

size_t lbm_checkpoint_bytes(const lbm_params* p) {
  const size_t s = lbm_state_bytes(p);
  return s == 0 || p->storage == LBM_FP32 ? s : s + (size_t)2 * p->nx * p->ny;
}

int lbm_save_state(lbm_ctx* ctx, void* dst) {
  if (int st = check_ctx(ctx, true)) return st;
  if (!dst) return fail(LBM_EINVAL, "dst is NULL");
  if (int st = set_device(ctx)) return st;
  const size_t sb = lbm_state_bytes(&ctx->p);
  HIP_OK(hipMemcpyAsync(dst, ctx->buf[ctx->cur], sb, hipMemcpyDeviceToDevice, ctx->stream));
  if (ctx->p.storage != LBM_FP32)
    HIP_OK(hipMemcpyAsync(static_cast<char*>(dst) + sb, ctx->ref[ctx->cur], (size_t)2 * ctx->p.nx * ctx->p.ny,
                          hipMemcpyDeviceToDevice, ctx->stream));
  return LBM_OK;
}

int lbm_load_state(lbm_ctx* ctx, const void* src, int64_t t) {
  if (int st = check_ctx(ctx, false)) return st;
  if (!src) return fail(LBM_EINVAL, "src is NULL");
  if (t < 0) return fail(LBM_EINVAL, "t must be >= 0");
  if (int st = set_device(ctx)) return st;
  const size_t sb = lbm_state_bytes(&ctx->p);
  HIP_OK(hipMemcpyAsync(ctx->buf[0], src, sb, hipMemcpyDeviceToDevice, ctx->stream));
  if (ctx->p.storage != LBM_FP32)
    HIP_OK(hipMemcpyAsync(ctx->ref[0], static_cast<const char*>(src) + sb, (size_t)2 * ctx->p.nx * ctx->p.ny,
                          hipMemcpyDeviceToDevice, ctx->stream));
  ctx->cur = 0;
  ctx->t = t;
  ctx->ready = true;
  return LBM_OK;
}

namespace {
int need_fp32(const lbm_ctx* ctx, const char* what) {
  if (ctx->p.storage != LBM_FP32) return fail(LBM_EINVAL, "%s is available for LBM_FP32 storage only", what);
  return LBM_OK;
}
}  // namespace

int lbm_step_saved(lbm_ctx* ctx, const void* src, void* dst) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "lbm_step_saved")) return st;
  if (!src || !dst || src == dst) return fail(LBM_EINVAL, "src and dst must be two distinct device buffers");
  if (int st = set_device(ctx)) return st;
  launch_step<StoreF32>(ctx, src, dst, nullptr, nullptr);
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

int lbm_step_saved_chain(lbm_ctx* ctx, void* const* bufs, int32_t n) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "lbm_step_saved_chain")) return st;
  if (n < 0) return fail(LBM_EINVAL, "n must be >= 0");
  if (n == 0) return LBM_OK;
  if (!bufs) return fail(LBM_EINVAL, "bufs is NULL");
  for (int32_t j = 0; j < n; ++j)
    if (!bufs[j] || !bufs[j + 1] || bufs[j] == bufs[j + 1])
      return fail(LBM_EINVAL, "bufs[%d] and bufs[%d] must be two distinct device buffers", j, j + 1);
  if (int st = set_device(ctx)) return st;
  if (const int shape = kFuseSteps ? stepk_shape<StoreF32, true>(ctx, n) : 0) {
    with_stepk(shape, [&](auto tile) {
      using S = decltype(tile);
      for (int32_t j = 0; j < n;) {
        // up to K steps, each state a buffer the launch neither reads nor writes otherwise
        StepOuts<S::K> outs{};
        int k = 0;
        for (bool fresh = true; fresh && k < S::K && j + k < n; k += fresh) {
          for (int i = 0; i <= k; ++i) fresh = fresh && bufs[j + i] != bufs[j + k + 1];
          if (fresh) outs.p[k] = bufs[j + k + 1];
        }
        launch_stepk<StoreF32, S>(ctx, bufs[j], outs, k, nullptr, nullptr);
        j += k;
      }
    });
    HIP_OK(hipGetLastError());
    return LBM_OK;
  }
  for (int32_t j = 0; j < n;) {
    // two steps per launch where the state two steps on goes to a third buffer
    if (kFuseSteps && n - j >= 2 && use_step2(ctx) && bufs[j + 2] != bufs[j]) {
      launch_step2<true>(ctx, bufs[j], bufs[j + 1], bufs[j + 2]);
      j += 2;
    } else {
      launch_step<StoreF32>(ctx, bufs[j], bufs[j + 1], nullptr, nullptr);
      ++j;
    }
  }
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

size_t lbm_adjoint_bytes(const lbm_params* p) {
  char msg[256];
  if (lbm::validate(p, msg, sizeof msg) || p->storage != LBM_FP32) return 0;
  return (size_t)11 * plane_elems(p->nx, p->ny, 4) * sizeof(float);
}

int lbm_adjoint_seed(lbm_ctx* ctx, const float* lam, void* adj) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (!lam || !adj) return fail(LBM_EINVAL, "lam and adj must be device buffers");
  if (int st = set_device(ctx)) return st;
  const int nx = ctx->p.nx, ny = ctx->p.ny;
  with_bool(stream_rows(44ull * nx * ny, 4ull * nx), [&](auto stream) {
    adjoint_seed_kernel<decltype(stream)::value><<<grid1((size_t)nx * ny), BLK, 0, ctx->stream>>>(
        lam, static_cast<float*>(adj), nx, ny, make_divisor(nx));
  });
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

// One adjoint step on the context's stream (split like the forward step for
// wide FP32 states).  Blocks of both launches add into the partial-sum
// slots 0 .. grid-1 in launch order, so the sums stay reproducible.
extern "C++" {
template <class S>
static void launch_adjoint_tiles(lbm_ctx* ctx, const void* f_t, const void* adj_next, void* adj_out) {
  const int nx = ctx->p.nx, ny = ctx->p.ny, ntx = tiles_x<S>(nx);
  with_stores(ctx, stream_stores(44ull * nx * ny, 4ull * nx, kCachedHbm), [&](auto str, bool reverse) {
    for_tile_rows<S, true>(nx, ny, [&](auto mode, TileRows rows, int nrows) {
      adjoint_step_kernel<S, decltype(mode)::value, decltype(str)::value>
          <<<ntx * nrows, dim3(S::TX, S::WY), 0, ctx->stream>>>(
              static_cast<const float*>(f_t), static_cast<const float*>(adj_next), static_cast<float*>(adj_out),
              ctx->theta, nx, ny, make_order(ntx, nrows, strip_width(nx, S::TX, false), reverse), ctx->c, rows);
    });
  });
}
static void launch_adjoint(lbm_ctx* ctx, const void* f_t, const void* adj_next, void* adj_out) {
  if (small_adjoint(ctx))
    launch_adjoint_tiles<AdjTileSmall>(ctx, f_t, adj_next, adj_out);
  else
    launch_adjoint_tiles<AdjTile>(ctx, f_t, adj_next, adj_out);
}
}  // extern "C++"

int lbm_adjoint_step(lbm_ctx* ctx, const void* f_t, const void* adj_next, void* adj_out) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (!f_t || !adj_next || !adj_out || adj_next == adj_out)
    return fail(LBM_EINVAL, "f_t, adj_next and adj_out must be device buffers, adj_next != adj_out");
  if (int st = set_device(ctx)) return st;
  launch_adjoint(ctx, f_t, adj_next, adj_out);
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

int lbm_adjoint_run(lbm_ctx* ctx, const void* const* f_states, int32_t n, void* adj_a, void* adj_b,
                    int32_t* which) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (n < 0) return fail(LBM_EINVAL, "n must be >= 0");
  if (!which) return fail(LBM_EINVAL, "which is NULL");
  if (!adj_a || !adj_b || adj_a == adj_b) return fail(LBM_EINVAL, "adj_a and adj_b must be two distinct device buffers");
  if (n > 0 && !f_states) return fail(LBM_EINVAL, "f_states is NULL");
  for (int32_t j = 0; j < n; ++j)
    if (!f_states[j]) return fail(LBM_EINVAL, "f_states[%d] is NULL", j);
  if (int st = set_device(ctx)) return st;
  void* buf[2] = {adj_a, adj_b};
  int cur = 0;
  for (int32_t j = n - 1; j >= 0; --j) {
    launch_adjoint(ctx, f_states[j], buf[cur], buf[cur ^ 1]);
    cur ^= 1;
  }
  HIP_OK(hipGetLastError());
  *which = cur;
  return LBM_OK;
}

int lbm_adjoint_get(lbm_ctx* ctx, const void* adj, float* lam) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (!adj || !lam) return fail(LBM_EINVAL, "adj and lam must be device buffers");
  if (int st = set_device(ctx)) return st;
  using S = AdjTile;
  adjoint_finish_kernel<S, false><<<tiles_total<S>(ctx->p.nx, ctx->p.ny), dim3(S::TX, S::WY), 0, ctx->stream>>>(
      static_cast<const float*>(adj), lam, nullptr, nullptr, nullptr, nullptr, ctx->p.nx, ctx->p.ny,
      tiles_x<S>(ctx->p.nx), ctx->c);
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

int lbm_adjoint_init(lbm_ctx* ctx, const float* rho0, const float* ux0, const float* uy0, const void* adj0,
                     float* drho0) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (!rho0 || !adj0 || !drho0) return fail(LBM_EINVAL, "rho0, adj0 and drho0 must be device buffers");
  if (int st = set_device(ctx)) return st;
  using S = AdjTile;
  adjoint_finish_kernel<S, true><<<tiles_total<S>(ctx->p.nx, ctx->p.ny), dim3(S::TX, S::WY), 0, ctx->stream>>>(
      static_cast<const float*>(adj0), drho0, rho0, ux0, uy0, ctx->theta, ctx->p.nx, ctx->p.ny,
      tiles_x<S>(ctx->p.nx), ctx->c);
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

namespace {
// Queue the sum of the accumulated dL/dtheta into the context's pinned words.
int launch_theta(const lbm_ctx* ctx, bool clear) {
  with_bool(clear, [&](auto c) {
    finish_sums<decltype(c)::value><<<1, RED, 0, ctx->stream>>>(ctx->theta, ctx->adj_blocks, ctx->host_dev->sums);
  });
  HIP_OK(hipGetLastError());
  return LBM_OK;
}

// Wait for it.
int wait_theta(const lbm_ctx* ctx, double dtheta[3]) {
  HIP_OK(hipStreamSynchronize(ctx->stream));
  for (int k = 0; k < 3; ++k) dtheta[k] = ctx->host->sums[k];
  for (int k = 0; k < 3; ++k)
    if (!std::isfinite(dtheta[k])) return fail(LBM_ENONFINITE, "non-finite parameter gradient (%d)", k);
  return LBM_OK;
}
}  // namespace

int lbm_adjoint_theta(lbm_ctx* ctx, double dtheta[3], int32_t reset) {
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (int st = set_device(ctx)) return st;
  if (!dtheta) {
    if (reset) HIP_OK(hipMemsetAsync(ctx->theta, 0, 3 * sizeof(double) * (size_t)ctx->adj_blocks, ctx->stream));
    return LBM_OK;
  }
  if (int st = launch_theta(ctx, reset != 0)) return st;
  return wait_theta(ctx, dtheta);
}

int lbm_adjoint_params(lbm_ctx* ctx, double dparams[3], double dtheta[3], int32_t reset) {
  if (!dparams) return fail(LBM_EINVAL, "dparams is NULL");
  if (int st = check_ctx(ctx, false)) return st;
  if (int st = need_fp32(ctx, "the adjoint")) return st;
  if (int st = set_device(ctx)) return st;
  if (int st = launch_theta(ctx, reset != 0)) return st;
  // the parameter map's Jacobian (a few hundred us of host work) while the
  // device finishes the sweep
  double th[3], jac[9];
  char msg[sizeof g_err];
  const int bad = lbm::param_jacobian(&ctx->p, ctx->d, jac, msg, sizeof msg);
  if (int st = wait_theta(ctx, th)) return st;
  if (bad) return fail(bad, "%s", msg);
  for (int j = 0; j < 3; ++j) dparams[j] = jac[j] * th[0] + jac[3 + j] * th[1] + jac[6 + j] * th[2];
  if (dtheta)
    for (int k = 0; k < 3; ++k) dtheta[k] = th[k];
  return LBM_OK;
}

int lbm_param_jacobian(const lbm_params* p, double jac[9]) {
  if (!jac) return fail(LBM_EINVAL, "jac is NULL");
  lbm_derived d;
  if (int st = lbm::derive(p, &d, g_err, sizeof g_err)) return st;
  return lbm::param_jacobian(p, d, jac, g_err, sizeof g_err);
}

int64_t lbm_time(const lbm_ctx* ctx) { return ctx ? ctx->t : -1; }

int lbm_get_derived(const lbm_ctx* ctx, lbm_derived* out) {
  if (int st = check_ctx(ctx, false)) return st;
  if (!out) return fail(LBM_EINVAL, "out is NULL");
  *out = ctx->d;
  return LBM_OK;
}

void lbm_destroy(lbm_ctx* ctx) {
  if (!ctx) return;
  if (ctx->scratch) {
    int cur = -1;
    const bool other = hipGetDevice(&cur) == hipSuccess && cur != ctx->device;
    if (other) (void)hipSetDevice(ctx->device);
    (void)hipFree(ctx->scratch);  // waits for the context's work in flight
    if (ctx->host) give_host_word(ctx->host);
    if (other) (void)hipSetDevice(cur);
  }
  delete ctx;
}

}  // extern "C"
