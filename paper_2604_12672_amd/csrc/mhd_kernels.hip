// mhd_kernels.hip -- gfx950 kernels of the explicit MHD step.
//
// stage_kernel: one SSP-RK stage (Sect. 2.9) fused into one launch.  A block
// marches up a segment of z planes of a 14 x 14 column tile, with a ring of
// halo columns around it for the three-cell stencils: 16 x 16 columns, plus
// 64 ring cells two columns out that only feed the x/y stencils.  Its waves
// have one role each and work on different planes of the march at the same
// time; what one computes at a step the others read at the next, so a step
// needs one barrier.  At step i
//   the column waves turn plane i into primitive deviations (EOS included),
//     stage them in LDS, reconstruct cell i-1 of their column along z, solve
//     the z-face between cells i-2 and i-1 and update the cells of plane i-2;
//   the x-face waves compute the Contact-CT edges E_y on the z-face below
//     plane i-2, update B_x and B_z of plane i-3 and B_y of plane i-4, and
//     reconstruct and solve the x-faces of plane i-1;
//   the y-face waves compute the edges E_x on the z-face below plane i-2 and
//     E_z of plane i-2, convert the ring cells of plane i, and reconstruct
//     and solve the y-faces of plane i-1.  Their lanes run along y, so that
//     the y neighbour is the next lane, as the x neighbour is in the others.
// In FP32 the x- and y-face work is done by the same waves, one after the
// other.  Neighbour exchanges inside a 16-lane row use lane shuffles, the
// others go through LDS.  Fluxes and EMFs on tile borders are recomputed by
// both neighbouring blocks from identical inputs with the same code, so every
// face and edge value is single-valued (div B stays at round-off) without
// atomics or a global EMF array.
#include <hip/hip_runtime.h>

#include <cfloat>

#include "mhd_device.h"
#include "mhd_internal.h"

namespace mhd {

// Row neighbours inside a 16-lane DPP row (one tile row): row_shr:1 reads
// lane-1, row_shl:1 reads lane+1; the lane at the row edge gets 0 (its
// result is never used).  Must be called with all lanes active.
__device__ __forceinline__ int dpp_shr1(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x111, 0xf, 0xf, true);
}
__device__ __forceinline__ int dpp_shl1(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x101, 0xf, 0xf, true);
}
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(dpp_shr1(__float_as_int(v)));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(dpp_shl1(__float_as_int(v)));
}
__device__ __forceinline__ double from_left(double v) {
  const int lo = dpp_shr1(__double2loint(v)), hi = dpp_shr1(__double2hiint(v));
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_right(double v) {
  const int lo = dpp_shl1(__double2loint(v)), hi = dpp_shl1(__double2hiint(v));
  return __hiloint2double(hi, lo);
}

// z plane or face q of a periodic z with n planes, -2 <= q <= n + 1 (also
// for n = 1: two steps of n reach the range; a division would cost more)
__device__ __forceinline__ int zwrap(int q, int n) {
  if (q < 0) q += n;
  if (q < 0) q += n;
  if (q >= n) q -= n;
  if (q >= n) q -= n;
  return q;
}
// z plane q -> stored plane and mirror flag (reflecting walls)
__device__ __forceinline__ int zsource(const Phys &ph, int q, int &mirror) {
  mirror = 0;
  if (q >= 0 && q < ph.nz) return q;
  if (!ph.reflect) return zwrap(q, ph.nz);
  mirror = 1;
  return q < 0 ? -1 - q : 2 * ph.nz - 1 - q;
}
// z face index f (0..nz for walls) -> stored face
__device__ __forceinline__ int zface(const Phys &ph, int f) {
  return ph.reflect ? f : zwrap(f, ph.nz);
}

// Element access through a plane's address and a lane's column.  The plane
// address (array + field + plane) must be the same for every lane of the
// wave: it is held in scalar registers (the asm's "s" constraint; a base
// the compiler holds in vector registers fails the build with an illegal
// vector-to-scalar copy instead of being narrowed to one lane), and the
// column is a 32-bit byte offset (planes stay below 4 GiB, checked at
// grid creation), so the access takes the scalar-base form of the global
// load and store and costs the vector unit no 64-bit address arithmetic.
// The empty asm statements keep the compiler from folding the scalar base
// into a per-lane address; lane_off re-states a column offset in the basic
// block of its accesses, since the compiler chooses the address form block
// by block.
__device__ __forceinline__ uint32_t lane_off(uint32_t o) {
  asm("" : "+v"(o));
  return o;
}
template <typename T>
__device__ __forceinline__ T plane_ld(const T *base, uint32_t off) {
  using G = const __attribute__((address_space(1))) char;
  using GT = const __attribute__((address_space(1))) T;
  G *b = (G *)base;
  asm("" : "+s"(b));
  return *(GT *)(b + off);
}
template <typename T>
__device__ __forceinline__ void plane_st(T *base, uint32_t off, T v) {
  using G = __attribute__((address_space(1))) char;
  using GT = __attribute__((address_space(1))) T;
  G *b = (G *)base;
  asm("" : "+s"(b));
  *(GT *)(b + off) = v;
}

// byte offsets of a lane's column and of its +x and +y neighbours in a plane
struct ColOff {
  uint32_t c, xp, yp;
};
__device__ __forceinline__ ColOff col_off(const Phys &ph, int gi, int gip, int gj, int gjp) {
  return {(uint32_t)(((size_t)gj * ph.nx + gi) * 8), (uint32_t)(((size_t)gj * ph.nx + gip) * 8),
          (uint32_t)(((size_t)gjp * ph.nx + gi) * 8)};
}

template <typename R, bool GR>
struct Cfg {
  static constexpr int NF = GR ? 10 : 8;  // cell fields kept per cell
};

// Reconstruction of one cell along `axis` (0 x, 1 y, 2 z) from its two
// neighbours (Sect. 2.5): the cell's lower-face value lo (R state of face
// i-1/2) and upper-face value hi (L state of face i+1/2), in the face frame
// of the axis (n = axis, t1 = axis+1, t2 = axis+2).  Van Leer: limited
// linear slope; PPH: the unlimited parabola whose averages over the three
// cells are the cell values, lo = (2 m + 5 c - p)/6, hi = (-m + 5 c + 2 p)/6.
template <typename R, bool GR>
__device__ __forceinline__ void recon_cell(int axis, const R *m, const R *c,
                                           const R *p, Side<R> &lo, Side<R> &hi,
                                           bool pph) {
  const int vn = Q_VX + axis, v1 = Q_VX + (axis + 1) % 3, v2 = Q_VX + (axis + 2) % 3;
  const int b1 = Q_BX + (axis + 1) % 3, b2 = Q_BX + (axis + 2) % 3;
  auto rec_vl = [&](int f, R &l, R &h) {
    const R s = R(0.5) * vanleer<R>(c[f] - m[f], p[f] - c[f]);
    l = c[f] - s;
    h = c[f] + s;
  };
  auto rec_pph = [&](int f, R &l, R &h) {
    const R sixth = R(1.0 / 6.0);
    l = (R(2) * m[f] + R(5) * c[f] - p[f]) * sixth;
    h = (R(5) * c[f] - m[f] + R(2) * p[f]) * sixth;
  };
  // one uniform branch per cell and axis, not per field
  auto all = [&](auto rec) {
    rec(Q_RHO, lo.drho, hi.drho);
    rec(vn, lo.vn, hi.vn);
    rec(v1, lo.v1, hi.v1);
    rec(v2, lo.v2, hi.v2);
    rec(Q_P, lo.dp, hi.dp);
    rec(b1, lo.b1, hi.b1);
    rec(b2, lo.b2, hi.b2);
    if (GR) {
      rec(Q_GE, lo.dge, hi.dge);
      rec(Q_GC, lo.dgc, hi.dgc);
    } else {
      lo.dge = hi.dge = lo.dgc = hi.dgc = R(0);
    }
  };
  if (pph)
    all(rec_pph);
  else
    all(rec_vl);
}

template <typename R>
__device__ __forceinline__ Side<R> side_from_left(const Side<R> &s) {
  Side<R> o;
  o.drho = from_left(s.drho);
  o.vn = from_left(s.vn);
  o.v1 = from_left(s.v1);
  o.v2 = from_left(s.v2);
  o.dp = from_left(s.dp);
  o.b1 = from_left(s.b1);
  o.b2 = from_left(s.b2);
  o.dge = from_left(s.dge);
  o.dgc = from_left(s.dgc);
  return o;
}

// face flux -> conserved order (rho, m_x, m_y, m_z, E)
template <typename R>
__device__ __forceinline__ void to_cons(int axis, const R F[7], R out[5]) {
  out[0] = F[0];
  out[1 + axis] = F[1];
  out[1 + (axis + 1) % 3] = F[2];
  out[1 + (axis + 2) % 3] = F[3];
  out[4] = F[4];
}

// Copy the packed guess network into LDS (all threads; caller syncs).
__device__ __forceinline__ void stage_mlp(const void *src, void *dst, int tid, int nthreads) {
  const uint4 *s4 = (const uint4 *)src;
  uint4 *d4 = (uint4 *)dst;
  for (int i = tid; i < (int)(sizeof(MlpLds) / 16); i += nthreads) d4[i] = s4[i];
}

// The arguments of one stage launch, passed as the kernel's only argument,
// so that they start at offset 0 of the kernel-argument segment.
struct StageArgs {
  Phys ph;
  StagePtrs p;
  double ca, cb, cc, dt_host;  // U^(s+1) = cb U^(s) + ca U^n - cc dt (div F - S)(U^(s))
  int tiles, full, share;      // the split of the work over the blocks (see the kernel)
};

// The stage's arguments read again from the argument segment, as a view
// the compiler cannot hoist (the asm hides that the address is the same
// each time).  Inside the plane loop the kernel keeps more uniform values
// live (pointers, constants, field offsets, branch conditions) than the
// 102 scalar registers hold; the compiler then parks the excess in lanes
// of vector registers and pays one v_readlane per 32-bit word at every
// use.  Taken from this view once per plane, the values are scalar loads
// (through the scalar cache, no vector issue slot) near their use.
__device__ __forceinline__ const StageArgs &stage_args_view() {
  using KA = const __attribute__((address_space(4))) StageArgs;
  KA *a = (KA *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return *(const StageArgs *)a;
}

// Threads of a stage block: the columns' four waves and, in FP64, four each
// for the x-faces and the y-faces, in FP32 four for both.  The split is by
// registers: one wave that does all of a column needs 382 of them in FP64
// (one wave per SIMD, every latency exposed), a third of it fits the 168 of
// three waves per SIMD; in FP32 a half fits 128 (two blocks of two waves per
// SIMD), a third would have to fit 80 for two blocks and spills.  Only the
// ideal-gas variants without optional features fit as they are (164 registers
// in FP64, 123 in FP32; on one plane 164 and 110).  Vector registers spilled by
// the others, and on one plane: FP64 ideal gas with features 16 (27), gas +
// radiation 7 (50), with features 34 (50); FP32 3 (9), 3 (0) and 13 (26).
// 256^3 stratified box per launch, one wave per column -> split: FP64 3.07 ->
// 1.95 ms (the launch's 770 M vector instructions take 1.3 ms to issue),
// 250 x 250 x 310 in FP32 1.81 -> 1.59 ms.
template <typename R>
constexpr int stage_threads() {
  return sizeof(R) == 8 ? 3 * NTHREADS : 2 * NTHREADS;
}

// One block of stage_kernel in LDS.  Planes are held by parity: a plane
// written during one step of the march is read during the next one, on the
// other side of that step's barrier, while the next plane goes to the other
// half.
constexpr int LW = TT + 2;  // staged plane edge: columns -2 .. 15
constexpr int LP = LW * LW;
// exchanged face and edge values: 16 x 16 with an odd pitch (the y-face
// waves walk a plane column by column) and one row and column of margin
// below, so that a lower neighbour's index is in the array for every lane; an
// upper neighbour's index past the last row (a halo lane's, whose value is
// not used) falls into the next plane or the margin after the last one
constexpr int EP = TT + 1;
constexpr int EN = EP * (TT + 1);
template <typename R, bool GR, bool XF>
struct StageLds {
  static constexpr int NF = Cfg<R, GR>::NF;
  R w[2][NF][LP];           // cell primitives (deviations)
  R bx[2][EN], by[2][EN];   // fields on the lower x and y faces
  R fx[2][5][EN];           // x-face conserved flux
  R fy[2][5][EN];           // y-face conserved flux
  R xez[2][EN];             // x-face E_z
  R yez[2][EN];             // y-face E_z
  R zex[2][EN], zey[2][EN]; // z-face E_x, E_y
  R zm[2][EN];              // z-face mass flux
  R rz[2][EN];              // cell reference E_z
  R ex[2][EN], ez[2][EN];   // edge E_x, E_z
  R margin[EP];
  // rows of the launch's table (see StagePtrs) of planes i-3 .. i+1: uniform
  // per plane, so every read is a broadcast
  double tab[8][TAB_N];
  uint8_t fl[XF ? 2 : 1][XF ? EN : 1];         // flattening flags
  unsigned long long nst[GR ? 3 : 1][NTHREADS / 64];
};

// A segment of the block's work, planes z0 .. z1-1 of one column tile, and a
// thread's column in it.  What follows from the thread's number is worked
// out again at each step: held over the march it would cost registers the
// face solves need, and a value spilled to scratch is read back through the
// queue of the global loads, behind every load in flight.
struct StageTile {
  int z0, z1;
  int tid;         // thread of the role, 0 .. 255
  bool owner;      // the block updates this column
  bool xedge, yedge;  // the column's upper x / y face wraps
  uint32_t col;    // byte offset of the column in a plane
};
struct StageIdx {
  int w, e;        // index of the column in a staged plane, in an exchanged plane
};
__device__ __forceinline__ int restate(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
// lanes of a row along x: column (tid % 16 - 1, tid / 16 - 1)
__device__ __forceinline__ StageIdx idx_rows(int tid) {
  const int q = restate(tid), r = q / TT;
  return {q + 2 * r + LW + 1, q + r + EP + 1};
}
// lanes of a row along y: column (tid / 16 - 1, tid % 16 - 1)
__device__ __forceinline__ StageIdx idx_cols(int tid) {
  const int q = restate(tid), r = q / TT, l = q % TT;
  return {l * LW + r + LW + 1, l * EP + r + EP + 1};
}
__device__ __forceinline__ ColOff tile_off(const Phys &ph, const StageTile &t) {
  const uint32_t row = (uint32_t)ph.nx * 8;
  return {t.col, t.xedge ? t.col - (row - 8) : t.col + 8,
          t.yedge ? t.col - row * (uint32_t)(ph.ny - 1) : t.col + row};
}

// A value that is not set on every path below: the register starts a new
// life here (no instruction), so that its old value does not stay live up to
// this point.
template <typename T>
__device__ __forceinline__ void renew(T &x) {
  asm("" : "=v"(x));
}
template <typename R, bool GR>
__device__ __forceinline__ void renew_side(Side<R> &s) {
  renew(s.drho);
  renew(s.vn);
  renew(s.v1);
  renew(s.v2);
  renew(s.dp);
  renew(s.b1);
  renew(s.b2);
  if (GR) {
    renew(s.dge);
    renew(s.dgc);
  }
}

// Entry `lane` of the table rows of plane i (mirror / wrap applied): the
// cell's entries, then those of its lower face.
__device__ __forceinline__ double table_request(const Phys &ph, const StagePtrs &p, int i,
                                                int lane) {
  int mir;
  const int kk = zsource(ph, i, mir);
  const int fk = ph.reflect ? max(0, min(i, ph.nz)) : zwrap(i, ph.nz);
  // the two rows are at most two apart: one base for both
  const int k0 = min(kk, fk);
  double v;
  renew(v);
  if (lane < TAB_N)
    v = plane_ld(p.table + (size_t)k0 * TAB_N,
                 lane_off((uint32_t)(((lane < TAB_FACE ? kk : fk) - k0) * TAB_N + lane) * 8));
  return v;
}

// What a wave carries from one step of the march to the next: reconstructed
// states, fluxes and EMFs (st, listed at each role) and the global values
// requested at the end of a step for the next one.
constexpr int ST_N = 14, PRE_N = 12;  // column waves
constexpr int XST_N = 10, XPRE_N = 6, YST_N = 8;  // face waves

// raw values of one cell: U, the six faces, the temperature guess
__device__ __forceinline__ void request_cell(const Phys &ph, const StagePtrs &p, ColOff co, int kk,
                                             double *pre) {
  const size_t plane = (size_t)ph.nx * ph.ny;
  const size_t n = plane * ph.nz;
  const size_t pk = (size_t)kk * plane;
  const int kp = ph.reflect ? kk + 1 : zwrap(kk + 1, ph.nz);
  const uint32_t o = lane_off(co.c), ox = lane_off(co.xp), oy = lane_off(co.yp);
#pragma unroll
  for (int f = 0; f < 5; ++f) pre[f] = plane_ld(p.Us + f * n + pk, o);
  pre[5] = plane_ld(p.Bxs + pk, o);
  pre[6] = plane_ld(p.Bys + pk, o);
  pre[7] = plane_ld(p.Bxs + pk, ox);
  pre[8] = plane_ld(p.Bys + pk, oy);
  pre[9] = plane_ld(p.Bzs + pk, o);
  pre[10] = plane_ld(p.Bzs + (size_t)kp * plane, o);
  pre[11] = p.Tin ? plane_ld(p.Tin + pk, lane_off(co.c)) : 0.0;
}

// primitive deviations of the requested cell, as R, with the mirror image
// applied
template <typename R, bool GR>
__device__ __forceinline__ void prim_cell(const Phys &ph, const double *pre, const double bg[4],
                                          int mirror, R *w, PrimOut &o, int maxit) {
  const double b[3] = {0.5 * (pre[5] + pre[7]), 0.5 * (pre[6] + pre[8]), 0.5 * (pre[9] + pre[10])};
  cons2prim<GR>(ph, pre, b, pre[11], bg, o, maxit);
  constexpr int NF = Cfg<R, GR>::NF;
#pragma unroll
  for (int f = 0; f < NF; ++f) w[f] = (R)o.w[f];
  if (mirror) {
    w[Q_VZ] = -w[Q_VZ];
    w[Q_BZ] = -w[Q_BZ];
  }
}

// Ring cells two columns outside the tile (they only feed the x/y
// stencils): the first 16 lanes of each of four waves take one of the four
// sides, so that every SIMD carries the same extra work.
struct RingCell {
  bool on;
  int w;       // index in a staged plane
  ColOff co;
};
__device__ __forceinline__ RingCell ring_cell(const Phys &ph, int X0, int Y0, int tid) {
  const int wv = tid >> 6, lane = tid & 63;
  int ci = lane - 1, cj = lane - 1;
  if (wv == 0) ci = -2;
  if (wv == 1) ci = TT - 1;
  if (wv == 2) cj = -2;
  if (wv == 3) cj = TT - 1;
  return {lane < 16, (cj + 2) * LW + (ci + 2),
          col_off(ph, wrapi(X0 + ci, ph.nx), wrapi(X0 + ci + 1, ph.nx), wrapi(Y0 + cj, ph.ny),
                  wrapi(Y0 + cj + 1, ph.ny))};
}

// FLAT: a grid of one plane.  Every plane of the march is the same one, so
// its cells are converted once (step z0-1, into both slots), its faces solved
// once (step z0+1), and steps z0-2 and z0 are left out.  Where a step needs
// values of the plane below or above, its own are those.
template <bool FLAT>
__device__ __forceinline__ bool skip_step(int i, int z0) {
  return FLAT && (i == z0 - 2 || i == z0);
}

// the requested ring cell of plane i to the staged plane
template <typename R, bool GR, bool XF, bool FLAT>
__device__ __forceinline__ void ring_step(const StageArgs &A, StageLds<R, GR, XF> &S,
                                          const RingCell &rc, int i, const double *pre, int &bad) {
  constexpr int NF = Cfg<R, GR>::NF;
  int mir;
  (void)zsource(A.ph, i, mir);
  if (rc.on) {
    const double *bg = S.tab[i & 7];
    PrimOut o;
    R Wr[NF];
    prim_cell<R, GR>(A.ph, pre, bg, mir, Wr, o, A.p.newton_cap);
    bad |= o.bad;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      S.w[i & 1][f][rc.w] = Wr[f];
      if (FLAT) S.w[~i & 1][f][rc.w] = Wr[f];
    }
  }
}
// ... and the request of plane i
__device__ __forceinline__ void ring_request(const Phys &ph, const StagePtrs &p, const RingCell &rc,
                                             int i, double (&pre)[PRE_N]) {
  int mir;
  const int kk = zsource(ph, i, mir);
#pragma unroll
  for (int f = 0; f < PRE_N; ++f) renew(pre[f]);
  if (rc.on) request_cell(ph, p, rc.co, kk, pre);
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ double uniform(double x) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                          __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// Error bits and Newton statistics of a thread.
struct StageCount {
  unsigned it = 0, mx = 0, fb = 0;
  int bad = 0;
};

// Column waves, step i: primitives of plane i, the z-face between cells i-2
// and i-1, the update of the cells of plane i-2.
// st: 0..8 upper z-face state of cell i-2, 9..13 z-face flux of the face i-2.
template <typename R, bool GR, bool XF, bool FLAT>
__device__ __forceinline__ void column_steps(const StageArgs &args, StageLds<R, GR, XF> &S,
                                             const StageTile &t, double cdt, StageCount &n) {
  constexpr int NF = Cfg<R, GR>::NF;
  // FP32 with the optional features: the update is finished at the top of the
  // next step, so its values arrive over the barrier and are not live beside
  // the forcing (spilled registers 21 -> 3 with the ideal gas, 34 -> 13 with gas
  // + radiation; turbulence box at 384^3 38.4 -> 31.2 ms for two steps, others
  // 1 % faster); the other variants lose 0 to 4 % that way
  constexpr bool LATE = sizeof(R) == 4 && XF;
  const int z0 = t.z0, z1 = t.z1;
  R st[ST_N];
#pragma unroll
  for (int f = 0; f < ST_N; ++f) st[f] = R(0);
  double pre[PRE_N];
  double us[5], u0[5], r[5];  // the update in progress: U^(s), U^n, divergence
#pragma unroll
  for (int f = 0; f < 5; ++f) us[f] = u0[f] = r[f] = 0.0;
  int fk = 0, fc = 0;  // flags of the column's cells i-2 and i-1
  {
    const Phys &ph = args.ph;
    int mir0;
    const int k0 = zsource(ph, z0 - 2, mir0);
    request_cell(ph, args.p, tile_off(ph, t), k0, pre);
  }
  // coefficients of the forcing of the column
  R fco[XF ? 3 * FZB : 1];
  if (XF && args.p.fcoef) {
    const size_t plane = (size_t)args.ph.nx * args.ph.ny;
#pragma unroll
    for (int d = 0; d < 3 * FZB; ++d)
      fco[XF ? d : 0] = plane_ld((const R *)args.p.fcoef + d * plane, lane_off(t.col / (8 / sizeof(R))));
  }
  for (int i = z0 - 2; i <= z1 + 3; ++i) {
    if (skip_step<FLAT>(i, z0)) continue;
    const StageArgs &A = stage_args_view();
    const Phys &ph = A.ph;
    const StagePtrs &p = A.p;
    const double ca = A.ca, cb = A.cb;
    const size_t plane = (size_t)ph.nx * ph.ny;
    const size_t ncell = plane * ph.nz;
    const int b = i & 1, pb = b ^ 1;
    // finishes the update of the cells of plane k
    auto finish = [&](int k) {
      const double *tab = S.tab[k & 7];
      // sources S - S_hat: gravity on the density deviation, rho g.v,
      // heating, forcing (Sect. 2.1, eq. wb2)
      double s1 = 0.0, s2 = 0.0, s3 = (us[0] - tab[0]) * ph.gz;
      double s4 = us[3] * ph.gz + tab[4];
      if (XF && p.fcoef) {
        // the forcing of this cell from its column's coefficients
        double fo[3];
#pragma unroll
        for (int c3 = 0; c3 < 3; ++c3) {
          double f = 0.0;
#pragma unroll
          for (int d = 0; d < FZB; ++d)
            f += (double)fco[XF ? c3 * FZB + d : 0] * tab[5 + d];
          fo[c3] = f;
        }
        s1 += us[0] * fo[0];
        s2 += us[0] * fo[1];
        s3 += us[0] * fo[2];
        s4 += us[1] * fo[0] + us[2] * fo[1] + us[3] * fo[2];
      }
      r[1] -= s1;
      r[2] -= s2;
      r[3] -= s3;
      r[4] -= s4;
      const size_t pq = (size_t)k * plane;
      const uint32_t o = lane_off(t.col);
#pragma unroll
      for (int f = 0; f < 5; ++f)
        plane_st(p.Uo + f * ncell + pq, o, cb * us[f] - cdt * r[f] + ca * u0[f]);
    };
    if (LATE && i >= z0 + 3 && i <= z1 + 2 && t.owner) finish(i - 3);
    if (i <= z1 + 1) {
      const StageIdx ix = idx_rows(t.tid);
      const int w = ix.w, e = ix.e;
      int mir;
      const int kk = zsource(ph, i, mir);
      int fn = 0;  // flag of cell i (a mirror image carries its source's)
      if (XF && p.flat) fn = plane_ld(p.flat + (size_t)kk * plane, lane_off(t.col >> 3));
      double bzf = 0.0;
      if (i >= z0 + 1)
        bzf = plane_ld(p.Bzs + (size_t)zface(ph, i - 1) * plane, lane_off(t.col));
      // primitives of plane i, staged for the face waves
      R Wn[NF];
      if (!FLAT || i < z0) {
        const double *bg = S.tab[i & 7];
        PrimOut o;
        prim_cell<R, GR>(ph, pre, bg, mir, Wn, o, p.newton_cap);
        S.bx[b][e] = (R)pre[5];
        S.by[b][e] = (R)pre[6];
        if (GR) {
          if (t.owner && (FLAT ? i < z0 : i >= z0 && i < z1)) {
            if (p.Tout) plane_st(p.Tout + (size_t)kk * plane, lane_off(t.col), o.T);
            n.it += o.iters;
            n.mx = (unsigned)o.iters > n.mx ? o.iters : n.mx;
            n.fb += o.fallback;
          }
        }
        n.bad |= o.bad;
      }
      if (XF && (!FLAT || i < z0)) S.fl[b][e] = (uint8_t)fn;
      // own cells i-2 (its slot is the one plane i goes to; only this thread
      // reads or writes that slot) and i-1
      R Wm[NF], Wc[NF];
      if (!FLAT) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          Wm[f] = S.w[b][f][w];
          Wc[f] = S.w[pb][f][w];
          S.w[b][f][w] = Wn[f];
        }
      } else if (i < z0) {
#pragma unroll
        for (int f = 0; f < NF; ++f) S.w[b][f][w] = S.w[pb][f][w] = Wn[f];
        S.bx[pb][e] = S.bx[b][e];
        S.by[pb][e] = S.by[b][e];
        if (XF) S.fl[XF ? pb : 0][XF ? e : 0] = (uint8_t)fn;
      } else {
#pragma unroll
        for (int f = 0; f < NF; ++f) Wm[f] = Wc[f] = Wn[f] = S.w[b][f][w];
      }
      Side<R> topn;  // upper z-face state of cell i-1
      R fzc[5];
      renew_side<R, GR>(topn);
#pragma unroll
      for (int f = 0; f < 5; ++f) renew(fzc[f]);
      if (FLAT && i > z0 + 1) {
        // both z-faces carry the flux of step z0+1
#pragma unroll
        for (int f = 0; f < 5; ++f) fzc[f] = st[9 + f];
      } else if (i >= z0) {
        Side<R> botn;
        recon_cell<R, GR>(2, Wm, Wc, Wn, botn, topn,
                          ph.recon == MHD_RECON_PPH && !(XF && fc));
        if (i >= z0 + 1) {
          const int f = i - 1;
          const double *bg = S.tab[f & 7] + TAB_FACE;
          const FaceBg<R> bgf = {(R)bg[0], (R)bg[1], (R)bg[2], (R)bg[3]};
          Side<R> topk = {st[0], st[1], st[2], st[3], st[4], st[5], st[6], st[7], st[8]};
          if (FLAT) topk = topn;
          R fz[7];
          face_flux<R, GR>(XF && (fk | fc) != 0, topk, botn, (R)bzf, bgf, (R)ph.gamma,
                           (R)ph.igm1, ph.xi_mode, (R)ph.mach_cut, (R)ph.imach_cut, fz);
          // mass flux for the species: the lower face of cell i-1 (and the
          // top wall), written once, by the block that owns the cell
          if (XF && p.mfz && t.owner && (f < z1 || (ph.reflect && f == ph.nz)))
            plane_st(p.mfz + (size_t)f * plane, lane_off(t.col), (double)fz[0]);
          to_cons<R>(2, fz, fzc);
          S.zey[b][e] = -fz[5];  // z-face E_y = -F_z[B_x]
          S.zex[b][e] = fz[6];   // z-face E_x = +F_z[B_y]
          S.zm[b][e] = fz[0];
          if (FLAT) {
            S.zey[pb][e] = -fz[5];
            S.zex[pb][e] = fz[6];
            S.zm[pb][e] = fz[0];
          }
        }
      }
      // cells of plane i-2: their flux divergence, and the values of the update
      // that the next step finishes; then the next plane's cells.  All are in
      // flight over the barrier.
      const int kc = max(i - 2, 0);
      const size_t pqc = (size_t)kc * plane;
      const bool upd = i >= z0 + 2 && t.owner;
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        renew(us[f]);
        u0[f] = 0.0;
      }
      if (upd) {
        const uint32_t o = lane_off(t.col);
#pragma unroll
        for (int f = 0; f < 5; ++f) us[f] = plane_ld(p.Us + f * ncell + pqc, o);
      }
      if (upd && ca != 0.0) {
        const uint32_t o = lane_off(t.col);
#pragma unroll
        for (int f = 0; f < 5; ++f) u0[f] = plane_ld(p.U0 + f * ncell + pqc, o);
      }
#pragma unroll
      for (int f = 0; f < PRE_N; ++f) renew(pre[f]);
      if (!FLAT && i <= z1) {
        int mirn;
        const int kn = zsource(ph, i + 1, mirn);
        request_cell(ph, p, tile_off(ph, t), kn, pre);
      }
      {
        const StageIdx ix = idx_rows(t.tid);
        const int e = ix.e;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          const R fxl = S.fx[pb][f][e], fyl = S.fy[pb][f][e];
          const double acc = ((double)S.fx[pb][f][e + 1] - (double)fxl) * ph.idx +
                             ((double)S.fy[pb][f][e + EP] - (double)fyl) * ph.idy;
          r[f] = acc + ((double)fzc[f] - (double)st[9 + f]) * ph.idz;
          // mass fluxes for the species: the lower x and y faces
          if (XF && f == 0 && p.mfx && upd) {
            plane_st(p.mfx + pqc, lane_off(t.col), (double)fxl);
            plane_st(p.mfy + pqc, lane_off(t.col), (double)fyl);
          }
        }
      }
      if (!LATE && upd) finish(i - 2);
      st[0] = topn.drho;
      st[1] = topn.vn;
      st[2] = topn.v1;
      st[3] = topn.v2;
      st[4] = topn.dp;
      st[5] = topn.b1;
      st[6] = topn.b2;
      st[7] = GR ? topn.dge : R(0);
      st[8] = GR ? topn.dgc : R(0);
#pragma unroll
      for (int f = 0; f < 5; ++f) st[9 + f] = fzc[f];
      fk = fc;
      fc = fn;
    }
    __syncthreads();
  }
}

// Face states of one face direction (AX 0: x, 1: y) at the lane's lower
// face: reconstructs the own cell from the staged plane; the L state is the
// upper value of the cell one down the axis, the previous lane of the row.
template <typename R, bool GR, int AX>
__device__ __forceinline__ void face_states(const R (*W)[LP], int w, bool pph, R *Wc,
                                            Side<R> &L, Side<R> &Rt) {
  constexpr int NF = Cfg<R, GR>::NF;
  constexpr int ST = AX == 0 ? 1 : LW;
  R m[NF], u[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    m[f] = W[f][w - ST];
    Wc[f] = W[f][w];
    u[f] = W[f][w + ST];
  }
  Side<R> hi;
  recon_cell<R, GR>(AX, m, Wc, u, Rt, hi, pph);
  L = side_from_left<R>(hi);
}

// background at the x- and y-faces of plane k
template <typename R, bool GR, bool XF>
__device__ __forceinline__ FaceBg<R> cell_bg(const StageLds<R, GR, XF> &S, int k) {
  const double *bg = S.tab[k & 7];
  return {(R)bg[0], (R)bg[1], (R)bg[2], (R)bg[3]};
}

// x-face waves, step i: the edges E_y on the z-face i-2 and the updates of
// B_x and B_z (plane i-3) and B_y (plane i-4), then the x-faces of plane i-1.
// st: 0 x-face E_y, 1 its mass flux, 2 the cell's reference E_y (plane
// i-2), 3..5 the same of plane i-3, 6 edge E_y, 7 edge E_x (z-face i-3),
// 8, 9 edge E_z of plane i-4, own and right.
template <typename R, bool GR, bool XF>
__device__ __forceinline__ void xedge_step(const StageArgs &A, StageLds<R, GR, XF> &S,
                                           const StageTile &t, double cdt, int i, R (&st)[XST_N],
                                           const double (&pre)[XPRE_N]) {
  const int z0 = t.z0, z1 = t.z1;
  const Phys &ph = A.ph;
  const StagePtrs &p = A.p;
  const double ca = A.ca, cb = A.cb;
  const size_t plane = (size_t)ph.nx * ph.ny;
  const int b = i & 1, pb = b ^ 1;
  const StageIdx ix = idx_rows(t.tid);
  const int e = ix.e;
  R ey_n = 0;
  if (i >= z0 + 2 && i <= z1 + 2) {
    // E_y at (ci-1/2, cj, i-2): a = z (z-faces at ci, ci-1), b = x
    // (x-faces at planes i-2, i-3)
    const R zey = S.zey[pb][e], zm = S.zm[pb][e];
    const R zey_l = from_left(zey), zm_l = from_left(zm);
    const R r_l = from_left(st[2]), rp_l = from_left(st[5]);
    ey_n = ct_edge<R>(zey, zey_l, st[0], st[3], st[2], st[5], r_l, rp_l, zm, zm_l,
                      st[1], st[4]);
    // a reflecting wall carries no tangential EMF
    if (ph.reflect && (i == 2 || i - 2 == ph.nz)) ey_n = R(0);
  }
  if (i >= z0 + 3) {
    const R ex_n = S.ex[pb][e], ex_u = S.ex[pb][e + EP];
    const R ez_c = S.ez[pb][e], ez_u = S.ez[pb][e + EP], ez_r = S.ez[pb][e + 1];
    const R ey_p = st[6], ey_r = from_right(ey_p);
    if (t.owner && i <= z1 + 2) {
      const size_t px = (size_t)(i - 3) * plane;
      const double rbx = ((double)ez_u - (double)ez_c) * ph.idy -
                         ((double)ey_n - (double)ey_p) * ph.idz;
      plane_st(p.Bxo + px, lane_off(t.col), cb * pre[0] - cdt * rbx + ca * pre[3]);
    }
    if (t.owner && i <= z1 + 2 && !(ph.reflect && i == 3)) {
      const size_t px = (size_t)(i - 3) * plane;
      const double rbz = ((double)ey_r - (double)ey_p) * ph.idx -
                         ((double)ex_u - (double)ex_n) * ph.idy;
      plane_st(p.Bzo + px, lane_off(t.col), cb * pre[2] - cdt * rbz + ca * pre[5]);
    }
    if (t.owner && i >= z0 + 4) {
      const double rby = ((double)ex_n - (double)st[7]) * ph.idz -
                         ((double)st[9] - (double)st[8]) * ph.idx;
      plane_st(p.Byo + (size_t)(i - 4) * plane, lane_off(t.col),
               cb * pre[1] - cdt * rby + ca * pre[4]);
    }
    st[7] = ex_n;
    st[8] = ez_c;
    st[9] = ez_r;
  }
  st[6] = ey_n;
}
template <typename R, bool GR, bool XF, bool FLAT>
__device__ __forceinline__ void xface_step(const StageArgs &A, StageLds<R, GR, XF> &S,
                                           const StageTile &t, int i, R (&st)[XST_N],
                                           double (&pre)[XPRE_N]) {
  constexpr int NF = Cfg<R, GR>::NF;
  const Phys &ph = A.ph;
  const StagePtrs &p = A.p;
  const double ca = A.ca;
  const int z0 = t.z0, z1 = t.z1;
  const size_t plane = (size_t)ph.nx * ph.ny;
  const int b = i & 1, pb = b ^ 1;
  const StageIdx ix = idx_rows(t.tid);
  const int e = ix.e;
  if (i >= z0 && i <= (FLAT ? z1 : z1 + 1)) {
    st[3] = st[0];
    st[4] = st[1];
    st[5] = st[2];
    int fc = 0;
    if (XF) fc = S.fl[XF ? pb : 0][XF ? e : 0];
    R Wc[NF];
    Side<R> L, Rt;
    face_states<R, GR, 0>(S.w[pb], ix.w, ph.recon == MHD_RECON_PPH && !(XF && fc), Wc, L, Rt);
    st[2] = -(Wc[Q_VZ] * Wc[Q_BX] - Wc[Q_VX] * Wc[Q_BZ]);
    const bool hll = XF && (fc | dpp_shr1(fc)) != 0;  // cells ci-1 and ci
    R fx[7], fxc[5];
    face_flux<R, GR>(hll, L, Rt, S.bx[pb][e], cell_bg(S, i - 1), (R)ph.gamma,
                     (R)ph.igm1, ph.xi_mode, (R)ph.mach_cut, (R)ph.imach_cut, fx);
    to_cons<R>(0, fx, fxc);
#pragma unroll
    for (int f = 0; f < 5; ++f) S.fx[b][f][e] = fxc[f];
    S.xez[b][e] = -fx[5];  // x-face E_z = -F_x[B_y]
    st[0] = fx[6];       // x-face E_y = +F_x[B_z]
    st[1] = fx[0];
    if (FLAT) {
      st[3] = st[0];
      st[4] = st[1];
      st[5] = st[2];
    }
  }
  // the face fields the next step updates
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    renew(pre[f]);
    pre[3 + f] = 0.0;
  }
  const bool next = i >= z0 + 2 && t.owner;
  const size_t nx = (size_t)max(0, min(i - 2, z1 - 1)) * plane;
  const size_t ny = (size_t)max(0, min(max(i - 3, z0), z1 - 1)) * plane;
  if (next) {
    const uint32_t o = lane_off(t.col);
    pre[0] = plane_ld(p.Bxs + nx, o);
    pre[1] = plane_ld(p.Bys + ny, o);
    pre[2] = plane_ld(p.Bzs + nx, o);
  }
  if (next && ca != 0.0) {
    const uint32_t o = lane_off(t.col);
    pre[3] = plane_ld(p.Bx0 + nx, o);
    pre[4] = plane_ld(p.By0 + ny, o);
    pre[5] = plane_ld(p.Bz0 + nx, o);
  }
}

// y-face waves (lanes of a row run along y), step i: the edges E_x on the
// z-face i-2 and E_z of plane i-2, then the y-faces of plane i-1.
// st: 0 y-face E_x, 1 its E_z, 2 its mass flux, 3, 4 the cell's reference
// E_x, E_z (plane i-2), 5..7 E_x, mass flux, reference E_x of plane i-3.
template <typename R, bool GR, bool XF>
__device__ __forceinline__ void yedge_step(const StageArgs &A, StageLds<R, GR, XF> &S,
                                           const StageTile &t, int i, R (&st)[YST_N]) {
  const int z0 = t.z0, z1 = t.z1;
  const Phys &ph = A.ph;
  const int b = i & 1, pb = b ^ 1;
  const StageIdx ix = idx_cols(t.tid);
  const int e = ix.e;
  if (i >= z0 + 2 && i <= z1 + 2) {
    // E_x at (ci, cj-1/2, i-2): a = y (y-faces at planes i-2, i-3), b = z
    // (z-faces at cj, cj-1)
    const R zex = S.zex[pb][e], zm = S.zm[pb][e];
    const R zex_d = from_left(zex), zm_d = from_left(zm);
    const R rx_d = from_left(st[3]), rxp_d = from_left(st[7]);
    R ex_n = ct_edge<R>(st[0], st[5], zex, zex_d, st[3], rx_d, st[7], rxp_d, st[2],
                        st[6], zm, zm_d);
    if (ph.reflect && (i == 2 || i - 2 == ph.nz)) ex_n = R(0);
    S.ex[b][e] = ex_n;
    // E_z at (ci-1/2, cj-1/2, i-2): a = x, b = y
    const R xez = S.xez[pb][e], xm = S.fx[pb][0][e];
    const R xez_d = from_left(xez), xm_d = from_left(xm);
    const R yez_l = S.yez[pb][e - 1], ym_l = S.fy[pb][0][e - 1], rz_l = S.rz[pb][e - 1];
    const R rz_d = from_left(st[4]), rz_ld = from_left(rz_l);
    S.ez[b][e] = ct_edge<R>(xez, xez_d, st[1], yez_l, st[4], rz_l, rz_d, rz_ld, xm, xm_d,
                            st[2], ym_l);
  }
}
template <typename R, bool GR, bool XF, bool FLAT>
__device__ __forceinline__ void yface_step(const StageArgs &A, StageLds<R, GR, XF> &S,
                                           const StageTile &t, int i, R (&st)[YST_N]) {
  constexpr int NF = Cfg<R, GR>::NF;
  const Phys &ph = A.ph;
  const int z0 = t.z0, z1 = t.z1;
  const int b = i & 1, pb = b ^ 1;
  const StageIdx ix = idx_cols(t.tid);
  const int e = ix.e;
  if (i >= z0 && i <= (FLAT ? z1 : z1 + 1)) {
    st[5] = st[0];
    st[6] = st[2];
    st[7] = st[3];
    int fc = 0;
    if (XF) fc = S.fl[XF ? pb : 0][XF ? e : 0];
    R Wc[NF];
    Side<R> L, Rt;
    face_states<R, GR, 1>(S.w[pb], ix.w, ph.recon == MHD_RECON_PPH && !(XF && fc), Wc, L, Rt);
    st[3] = -(Wc[Q_VY] * Wc[Q_BZ] - Wc[Q_VZ] * Wc[Q_BY]);
    st[4] = -(Wc[Q_VX] * Wc[Q_BY] - Wc[Q_VY] * Wc[Q_BX]);
    S.rz[b][e] = st[4];
    const bool hll = XF && (fc | dpp_shr1(fc)) != 0;  // cells cj-1 and cj
    R fy[7], fyc[5];
    face_flux<R, GR>(hll, L, Rt, S.by[pb][e], cell_bg(S, i - 1), (R)ph.gamma,
                     (R)ph.igm1, ph.xi_mode, (R)ph.mach_cut, (R)ph.imach_cut, fy);
    to_cons<R>(1, fy, fyc);
#pragma unroll
    for (int f = 0; f < 5; ++f) S.fy[b][f][e] = fyc[f];
    S.yez[b][e] = fy[6];  // y-face E_z = +F_y[B_x]
    st[0] = -fy[5];     // y-face E_x = -F_y[B_z]
    st[1] = fy[6];
    st[2] = fy[0];
    if (FLAT) {
      st[5] = st[0];
      st[6] = st[2];
      st[7] = st[3];
    }
  }
}

// March of the face waves.  FP64: x-faces and y-faces in waves of their own
// (DO_X or DO_Y); FP32: both in one wave.
template <typename R, bool GR, bool XF, bool FLAT, bool DO_X, bool DO_Y>
__device__ __forceinline__ void face_steps(const StageArgs &args, StageLds<R, GR, XF> &S,
                                           const StageTile &t, const RingCell &rc, double cdt, int wv, int lane,
                                           int &bad) {
  // The ring cells go first with the gas + radiation EOS, whose inversion has
  // the longest way to go (the registers of its 12 values are then free for
  // the edges: 5.17 -> 4.92 ms for three steps of a 170 x 190 x 150 box in
  // FP64), else after the edges, which hide the values' latency
  constexpr bool RING = DO_Y, FIRST = GR;
  const int z0 = t.z0, z1 = t.z1;
  R xst[XST_N], yst[YST_N];
#pragma unroll
  for (int f = 0; f < XST_N; ++f) xst[f] = R(0);
#pragma unroll
  for (int f = 0; f < YST_N; ++f) yst[f] = R(0);
  double pre[XPRE_N] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, rpre[PRE_N];
  if (RING) ring_request(args.ph, args.p, rc, z0 - 2, rpre);
  // the table row of the next plane is stored during a step, requested at
  // the end of the step before
  double tab = 0.0;
  if (DO_X && wv == 0) tab = table_request(args.ph, args.p, z0 - 1, lane);
  for (int i = z0 - 2; i <= z1 + 3; ++i) {
    if (skip_step<FLAT>(i, z0)) continue;
    const StageArgs &A = stage_args_view();
    const bool ring = RING && i <= (FLAT ? z0 - 1 : z1 + 1);
    if (FIRST && ring) ring_step<R, GR, XF, FLAT>(A, S, rc, i, rpre, bad);
    if (DO_X) xedge_step<R, GR, XF>(A, S, t, cdt, i, xst, pre);
    if (DO_Y) yedge_step<R, GR, XF>(A, S, t, i, yst);
    if (DO_X && wv == 0 && lane < TAB_N) S.tab[(i + 1) & 7][lane] = tab;
    if (!FIRST && ring) ring_step<R, GR, XF, FLAT>(A, S, rc, i, rpre, bad);
    if (DO_X) xface_step<R, GR, XF, FLAT>(A, S, t, i, xst, pre);
    if (DO_Y) yface_step<R, GR, XF, FLAT>(A, S, t, i, yst);
    if (RING && !FLAT && i <= z1) ring_request(A.ph, A.p, rc, i + 1, rpre);
    renew(tab);
    if (DO_X && wv == 0) tab = table_request(A.ph, A.p, min(i + 2, z1 + 1), lane);
    __syncthreads();
  }
}

// XF: the optional features of a stage (forcing modes, shock-flattening
// flags, species mass fluxes); the variant without them carries none of
// their code, pointers or registers.
template <typename R, bool GR, bool XF, bool FLAT>
__device__ __forceinline__ void stage_block(const StageArgs &args, StageLds<R, GR, XF> &S) {
  const StagePtrs &p = args.p;

  // the first four waves are the columns', the others the faces'; the role
  // is the same for every lane of a wave
  const int role = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NTHREADS);
  const int tid = threadIdx.x % NTHREADS;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave of the role
  const int lx = tid % TT, ly = tid / TT;
  const double cdt = uniform(args.cc * (p.dt_dev ? *p.dt_dev : args.dt_host));
  StageCount n;
  // The launch's items of work: the planes of one tile, first whole columns
  // of planes (args.full for every block), then the columns of the remaining
  // tiles cut in segments of args.share planes.  Tiles run fastest, so the
  // blocks march up neighbouring tiles at the same heights, and the logical
  // order gives each XCD a contiguous run of them: they share its L2.
  const int nblk = gridDim.x, lb = xcd_logical_block(blockIdx.x, nblk);
  // Issue priority of the waves with the longest way to the step's barrier:
  // FP32 the face waves (250 x 250 x 310 11.04 -> 10.69 ms for three steps, gas
  // + radiation 256^3 12.23 -> 11.85, with forcing 384^3 32.7 -> 31.0 for two;
  // the column waves first: 5 % slower), FP64 with the gas + radiation EOS the
  // x-face waves (170 x 190 x 150 4.92 -> 4.80); the ideal-gas FP64 roles are
  // even, and any order of them loses 1 to 7 %.
  if (role == 1 && (sizeof(R) == 4 || GR)) __builtin_amdgcn_s_setprio(2);
  for (int it = 0;; ++it) {
    const StageArgs &A = stage_args_view();
    const Phys &ph = A.ph;
    int tile, z0, z1;
    if (it < A.full) {
      tile = it * nblk + lb;
      z0 = 0;
      z1 = ph.nz;
    } else {
      const int rest = A.tiles - A.full * nblk;
      const int j = (it - A.full) * nblk + lb;
      const int seg = rest > 0 ? j / rest : 0;
      z0 = seg * A.share;
      if (rest <= 0 || z0 >= ph.nz) break;
      z1 = min(ph.nz, z0 + A.share);
      tile = A.full * nblk + (j - seg * rest);
    }
    const int ntx = (ph.nx + TB - 1) / TB;
    tile = __builtin_amdgcn_readfirstlane(tile);
    z0 = __builtin_amdgcn_readfirstlane(z0);
    z1 = __builtin_amdgcn_readfirstlane(z1);
    const int X0 = (tile % ntx) * TB, Y0 = (tile / ntx) * TB;
    const int gx = X0 + lx - 1, gy = Y0 + ly - 1;
    const int gi = wrapi(gx, ph.nx), gj = wrapi(gy, ph.ny);
    const RingCell rc = ring_cell(ph, X0, Y0, tid);
    StageTile t;
    t.z0 = z0;
    t.z1 = z1;
    t.tid = tid;
    t.owner = lx >= 1 && lx <= TB && ly >= 1 && ly <= TB && gx < ph.nx && gy < ph.ny;
    t.xedge = gi + 1 == ph.nx;
    t.yedge = gj + 1 == ph.ny;
    t.col = (uint32_t)(((size_t)gj * ph.nx + gi) * 8);
    // the first plane's table row; the face waves bring one a step
    if (role == 1 && wv == 0) {
      const double v = table_request(ph, A.p, z0 - 2, tid & 63);
      if ((tid & 63) < TAB_N) {
        S.tab[(z0 - 2) & 7][tid & 63] = v;
        if (FLAT)
          for (int r = 0; r < 8; ++r) S.tab[r][tid & 63] = v;
      }
    }
    __syncthreads();
    if (role == 0)
      column_steps<R, GR, XF, FLAT>(A, S, t, cdt, n);
    else if constexpr (sizeof(R) == 4)
      face_steps<R, GR, XF, FLAT, true, true>(A, S, t, rc, cdt, wv, tid & 63, n.bad);
    else if (role == 1)
      face_steps<R, GR, XF, FLAT, true, false>(A, S, t, rc, cdt, wv, tid & 63, n.bad);
    else
      face_steps<R, GR, XF, FLAT, false, true>(A, S, t, rc, cdt, wv, tid & 63, n.bad);
  }
  if (n.bad) atomicOr(p.flags, n.bad);
  if (GR) {
    // Newton statistics: wave totals of the column waves, then the block's
    unsigned long long a = n.it, m = n.mx, f = n.fb;
    for (int o = 32; o > 0; o >>= 1) {
      a += __shfl_xor(a, o);
      f += __shfl_xor(f, o);
      const unsigned long long mo = __shfl_xor(m, o);
      m = mo > m ? mo : m;
    }
    if (role == 0 && (tid & 63) == 0) {
      S.nst[0][tid >> 6] = a;
      S.nst[GR ? 1 : 0][tid >> 6] = m;
      S.nst[GR ? 2 : 0][tid >> 6] = f;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long a = 0, m = 0, f = 0;
      for (int v = 0; v < NTHREADS / 64; ++v) {
        a += S.nst[0][v];
        m = S.nst[GR ? 1 : 0][v] > m ? S.nst[GR ? 1 : 0][v] : m;
        f += S.nst[GR ? 2 : 0][v];
      }
      atomicAdd(&p.newton_stats[0], a);
      atomicMax(&p.newton_stats[1], m);
      atomicAdd(&p.newton_stats[2], f);
    }
  }
}

template <typename R, bool GR, bool XF>
__global__ __launch_bounds__(stage_threads<R>(), sizeof(R) == 4 ? 4 : 3) void stage_kernel(
    StageArgs args) {
  __shared__ StageLds<R, GR, XF> S;
  stage_block<R, GR, XF, false>(args, S);
}

// The stage of a grid of one plane (2D runs): five steps of the march instead
// of seven, one of them with face solves instead of three, and cells converted
// once instead of four times.  Bound as stage_kernel is: by the chain of one
// march where the tiles are few, by FP64 issue where they are many.  A variant
// of its own because the same tests in stage_kernel cost the other grids 1 to
// 2 %.  64 x 64 vortex, 20 steps 1062 -> 721 us; 4000 x 3000, 3 steps 28.7 ->
// 15.8 ms; 1000 x 1010 gas + radiation in split precision, 5 steps 3.59 -> 2.63.
template <typename R, bool GR, bool XF>
__global__ __launch_bounds__(stage_threads<R>(), sizeof(R) == 4 ? 4 : 3) void plane_stage_kernel(
    StageArgs args) {
  __shared__ StageLds<R, GR, XF> S;
  stage_block<R, GR, XF, true>(args, S);
}

static_assert(sizeof(MlpLds) % 16 == 0, "MlpLds is copied in 16-byte words");
size_t mlp_bytes() { return sizeof(MlpLds); }

// One plane: a reflecting z needs two, so its neighbours along z are itself.
static bool one_plane(const Phys &ph) { return ph.nz == 1; }

template <typename R, bool GR>
static auto stage_variant(bool xf, bool flat) -> void (*)(StageArgs) {
  if (flat) return xf ? plane_stage_kernel<R, GR, true> : plane_stage_kernel<R, GR, false>;
  return xf ? stage_kernel<R, GR, true> : stage_kernel<R, GR, false>;
}

template <typename R, bool GR>
static void launch_stage_g(const Ctx &c, const StagePtrs &p, double a, double b, double cc,
                           double dt_host, dim3 grid) {
  hipLaunchKernelGGL((stage_variant<R, GR>(p.fcoef || p.flat || p.mfx || p.mfy || p.mfz,
                                           one_plane(c.ph))),
                     grid, dim3(stage_threads<R>()), 0, c.stream,
                     StageArgs{c.ph, p, a, b, cc, dt_host, c.stage_tiles, c.stage_full,
                               c.stage_share});
}

template <typename R>
static void launch_stage_t(const Ctx &c, const StagePtrs &p, double a, double b, double cc,
                           double dt_host, dim3 grid) {
  if (!c.ph.gasrad)
    launch_stage_g<R, false>(c, p, a, b, cc, dt_host, grid);
  else
    launch_stage_g<R, true>(c, p, a, b, cc, dt_host, grid);
}

// the variant the context's stages run (occupancy for the segment length;
// forcing modes set later only change the variant, not the result)
template <typename R>
static const void *stage_fn(const Ctx &c) {
  const bool xf = c.d.flatten || c.d.nspecies > 0;
  return c.ph.gasrad ? (const void *)stage_variant<R, true>(xf, one_plane(c.ph))
                     : (const void *)stage_variant<R, false>(xf, one_plane(c.ph));
}

int stage_blocks_per_cu(const Ctx &c) {
  const bool split = c.d.precision == MHD_PREC_SPLIT;
  const void *f = split ? stage_fn<float>(c) : stage_fn<double>(c);
  const int nt = split ? stage_threads<float>() : stage_threads<double>();
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, nt, 0) != hipSuccess || nb < 1)
    nb = 1;
  return nb;
}

hipError_t launch_stage(const Ctx &c, const StagePtrs &p, double a, double b,
                        double cc, double dt_host) {
  dim3 grid(c.stage_blocks);
  if (c.d.precision == MHD_PREC_SPLIT)
    launch_stage_t<float>(c, p, a, b, cc, dt_host, grid);
  else
    launch_stage_t<double>(c, p, a, b, cc, dt_host, grid);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// CFL time step (eq. cfl): per-cell signal speed, block max, final max
// ---------------------------------------------------------------------------

constexpr int RED_THREADS = 256;
constexpr int RED_BLOCKS = CFL_MAX_BLOCKS;

template <bool GR, bool ML>
// Three waves per SIMD at least: the variant with the learned guess would
// otherwise take 176 registers (two waves) and wait on memory; at 168 it
// spills one register and runs 11 % faster (184 -> 163 us a launch over 128^3
// and 256^3 in turn); the other variants use 50 and 70.
__global__ __launch_bounds__(RED_THREADS) __attribute__((amdgpu_waves_per_eu(3))) void
signal_speed_kernel(
    Phys ph, const double *__restrict__ U, const double *__restrict__ Bx,
    const double *__restrict__ By, const double *__restrict__ Bz,
    const double *__restrict__ T, const void *mlp, double *__restrict__ partial,
    int *flags, double *__restrict__ Tout, double *__restrict__ Pout) {
  __shared__ __attribute__((aligned(16))) char sMlpRaw[ML ? sizeof(MlpLds) : 16];
  const MlpLds &sMlp = *reinterpret_cast<const MlpLds *>(sMlpRaw);
  if (ML) {
    stage_mlp(mlp, sMlpRaw, threadIdx.x, RED_THREADS);
    __syncthreads();
  }
  const size_t plane = (size_t)ph.nx * ph.ny;
  const size_t n = plane * ph.nz;
  const int lane = threadIdx.x & 63;
  double smax = 0.0;
  int bad = 0;
  // uniform trip count: lanes past the end redo the last cell and drop it
  for (size_t base = (size_t)blockIdx.x * blockDim.x; base < n;
       base += (size_t)gridDim.x * blockDim.x) {
    const bool valid = base + threadIdx.x < n;
    const size_t q = valid ? base + threadIdx.x : n - 1;
    int i, j, k;
    cell_ijk(ph, q, i, j, k);
    const int ip = i + 1 == ph.nx ? 0 : i + 1;
    const int jp = j + 1 == ph.ny ? 0 : j + 1;
    const int kp = ph.reflect ? k + 1 : (k + 1 == ph.nz ? 0 : k + 1);
    double u[5], b[3];
#pragma unroll
    for (int f = 0; f < 5; ++f) u[f] = U[f * n + q];
    b[0] = 0.5 * (Bx[q] + Bx[q - i + ip]);
    b[1] = 0.5 * (By[q] + By[q + (size_t)(jp - j) * ph.nx]);
    b[2] = 0.5 * (Bz[q] + Bz[(size_t)kp * plane + (q - (size_t)k * plane)]);
    const double zero[4] = {0, 0, 0, 0};
    double tg = (GR && !ML && T) ? T[q] : 0.0;
    if (ML) {
      float x0, x1;
      mlp_inputs(ph, u[0], specific_eint(u, b), x0, x1);
      tg = mlp_guess_wave(ph, sMlp, x0, x1, lane);
    }
    PrimOut o;
    cons2prim<GR>(ph, u, b, tg, zero, o, ML ? ph.newton_maxit_mlp : ph.newton_maxit);
    if (!valid) continue;
    bad |= o.bad;
    // the converged temperature is the best guess the next stage can get
    if (GR && Tout) Tout[q] = o.T;
    if (Pout) Pout[q] = o.w[Q_P];  // thermal pressure for the flattening detector
    const double rho = u[0];
    const double P = o.w[Q_P];
    const double a2 = o.w[Q_GC] * P / rho;
    const double b2 = (b[0] * b[0] + b[1] * b[1] + b[2] * b[2]) / rho;
    const double v[3] = {o.w[Q_VX], o.w[Q_VY], o.w[Q_VZ]};
    const double ids[3] = {ph.idx, ph.idy, ph.idz};
    double sum = 0.0;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      if (!ph.dims_active[s]) continue;
      const double bs2 = b[s] * b[s] / rho;
      double disc = (a2 + b2) * (a2 + b2) - 4.0 * a2 * bs2;
      disc = disc > 0.0 ? disc : 0.0;
      const double cf = sqrt(0.5 * ((a2 + b2) + sqrt(disc)));
      sum += (fabs(v[s]) + cf) * ids[s];
    }
    smax = sum > smax ? sum : smax;
    if (!(sum < INFINITY)) bad |= 1;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double t = __shfl_xor(smax, o);
    smax = t > smax ? t : smax;
  }
  __shared__ double sm[RED_THREADS / 64];
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = smax;
  if (bad) atomicOr(flags, bad);
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = 0.0;
    for (int w = 0; w < RED_THREADS / 64; ++w) m = sm[w] > m ? sm[w] : m;
    partial[blockIdx.x] = m;
  }
}

__global__ void finish_dt_kernel(const double *__restrict__ partial, int nb,
                                 double cfl, double *dt_out, double *smax_out) {
  __shared__ double sm[RED_THREADS];
  double m = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) m = partial[i] > m ? partial[i] : m;
  sm[threadIdx.x] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) sm[threadIdx.x] = sm[threadIdx.x + s] > sm[threadIdx.x] ? sm[threadIdx.x + s] : sm[threadIdx.x];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *smax_out = sm[0];
    *dt_out = cfl / sm[0];
  }
}

int cfl_partial_blocks(size_t ncell) {
  const size_t nb = (ncell + RED_THREADS - 1) / RED_THREADS;
  return (int)(nb < (size_t)RED_BLOCKS ? nb : (size_t)RED_BLOCKS);
}

hipError_t launch_signal_speed_raw(const Phys &ph, hipStream_t stream, bool learned,
                                   const double *U, const double *Bx, const double *By,
                                   const double *Bz, const double *T, const void *mlp,
                                   double *partial, int *flags, double cfl, double *dt_dev,
                                   double *smax_out, double *Tout, double *Pout) {
  const int nb = cfl_partial_blocks((size_t)ph.nx * ph.ny * ph.nz);
  if (!ph.gasrad)
    hipLaunchKernelGGL((signal_speed_kernel<false, false>), dim3(nb), dim3(RED_THREADS), 0,
                       stream, ph, U, Bx, By, Bz, T, mlp, partial, flags, nullptr, Pout);
  else if (learned)
    hipLaunchKernelGGL((signal_speed_kernel<true, true>), dim3(nb), dim3(RED_THREADS), 0,
                       stream, ph, U, Bx, By, Bz, T, mlp, partial, flags, Tout, Pout);
  else
    hipLaunchKernelGGL((signal_speed_kernel<true, false>), dim3(nb), dim3(RED_THREADS), 0,
                       stream, ph, U, Bx, By, Bz, T, mlp, partial, flags, Tout, Pout);
  hipLaunchKernelGGL(finish_dt_kernel, dim3(1), dim3(RED_THREADS), 0, stream, partial, nb, cfl,
                     dt_dev, smax_out);
  return hipGetLastError();
}

hipError_t launch_signal_speed(const Ctx &c, const double *U, const double *Bx,
                               const double *By, const double *Bz,
                               const double *T, double cfl, double *dt_dev, double *Tout,
                               double *Pout) {
  return launch_signal_speed_raw(c.ph, c.stream, c.d.eos_guess == MHD_GUESS_MLP, U, Bx, By, Bz,
                                 T, c.mlp, c.red, c.flags, cfl, dt_dev, c.red + RED_BLOCKS, Tout,
                                 Pout);
}

// ---------------------------------------------------------------------------
// initial temperature (bracketed solve) for the previous-T guess
// ---------------------------------------------------------------------------

// T of every cell: Newton from Tg when given, else the bracketed solve
__global__ void init_temperature_kernel(Phys ph, const double *__restrict__ U,
                                        const double *__restrict__ Bx,
                                        const double *__restrict__ By,
                                        const double *__restrict__ Bz,
                                        const double *__restrict__ Tg,
                                        double *__restrict__ T, int *flags) {
  const size_t plane = (size_t)ph.nx * ph.ny;
  const size_t n = plane * ph.nz;
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (size_t)gridDim.x * blockDim.x) {
    int i, j, k;
    cell_ijk(ph, q, i, j, k);
    const int ip = i + 1 == ph.nx ? 0 : i + 1;
    const int jp = j + 1 == ph.ny ? 0 : j + 1;
    const int kp = ph.reflect ? k + 1 : (k + 1 == ph.nz ? 0 : k + 1);
    double u[5], b[3];
    for (int f = 0; f < 5; ++f) u[f] = U[f * n + q];
    b[0] = 0.5 * (Bx[q] + Bx[q - i + ip]);
    b[1] = 0.5 * (By[q] + By[q + (size_t)(jp - j) * ph.nx]);
    b[2] = 0.5 * (Bz[q] + Bz[(size_t)kp * plane + (q - (size_t)k * plane)]);
    const double zero[4] = {0, 0, 0, 0};
    PrimOut o;
    cons2prim<true>(ph, u, b, Tg ? Tg[q] : NAN, zero, o);
    if (o.bad) atomicOr(flags, o.bad);
    T[q] = o.T;
  }
}

hipError_t launch_init_temperature(const Ctx &c, const double *U,
                                   const double *Bx, const double *By,
                                   const double *Bz, const double *Tg, double *T) {
  int nb = (int)((c.ncell + 255) / 256);
  nb = nb < 4096 ? nb : 4096;
  hipLaunchKernelGGL(init_temperature_kernel, dim3(nb), dim3(256), 0, c.stream, c.ph, U, Bx, By,
                     Bz, Tg, T, c.flags);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// learned initial guess of every cell of a state (before each stage in the
// learned mode): the stage kernel reads it as its temperature guess
// ---------------------------------------------------------------------------

// With polish the guess is polished by FP64 Newton right here (at most
// newton_maxit_mlp steps, then the bracketed solve) and the converged
// temperature is stored in its place, so the stage's own Newton starts
// converged: the iterations run in this small kernel at full occupancy
// instead of in the register-bound stage.  Their statistics go to stats
// (nullable).  With P != nullptr (shock flattening) the thermal pressure
// the detector needs is stored as well.
__global__ __launch_bounds__(256) void mlp_guess_kernel(Phys ph, const double *__restrict__ U,
                                                        const double *__restrict__ Bx,
                                                        const double *__restrict__ By,
                                                        const double *__restrict__ Bz,
                                                        const void *mlp,
                                                        double *__restrict__ Tg,
                                                        double *__restrict__ P, int *flags,
                                                        int polish,
                                                        unsigned long long *stats) {
  __shared__ __attribute__((aligned(16))) char sMlpRaw[sizeof(MlpLds)];
  const MlpLds &sMlp = *reinterpret_cast<const MlpLds *>(sMlpRaw);
  stage_mlp(mlp, sMlpRaw, threadIdx.x, 256);
  __syncthreads();
  const size_t plane = (size_t)ph.nx * ph.ny;
  const size_t n = plane * ph.nz;
  const int lane = threadIdx.x & 63;
  // every lane of a wave runs the matrix passes; lanes past the end repeat
  // the last cell and store nothing
  // cell data of one cell: U and the six faces (read at the top of each
  // pass: without a prefetch of the next cell the kernel fits 160 registers
  // and three waves per SIMD, which hide the latency better)
  auto fetch = [&](size_t q, double u[5], double f[6]) {
    int i, j, k;
    cell_ijk(ph, q, i, j, k);
    const int ip = i + 1 == ph.nx ? 0 : i + 1;
    const int jp = j + 1 == ph.ny ? 0 : j + 1;
    const int kp = ph.reflect ? k + 1 : (k + 1 == ph.nz ? 0 : k + 1);
#pragma unroll
    for (int c = 0; c < 5; ++c) u[c] = U[c * n + q];
    f[0] = Bx[q];
    f[1] = Bx[q - i + ip];
    f[2] = By[q];
    f[3] = By[q + (size_t)(jp - j) * ph.nx];
    f[4] = Bz[q];
    f[5] = Bz[(size_t)kp * plane + (q - (size_t)k * plane)];
  };
  const size_t stride = (size_t)gridDim.x * 256;
  size_t base = (size_t)blockIdx.x * 256;
  unsigned long long nit = 0, nmax = 0, nfb = 0;
  for (; base < n; base += stride) {
    const bool valid = base + threadIdx.x < n;
    const size_t q = valid ? base + threadIdx.x : n - 1;
    double u[5], b[3], fn[6];
    fetch(q, u, fn);
    b[0] = 0.5 * (fn[0] + fn[1]);
    b[1] = 0.5 * (fn[2] + fn[3]);
    b[2] = 0.5 * (fn[4] + fn[5]);
    float x0, x1;
    const double e = specific_eint(u, b);
    mlp_inputs(ph, u[0], e, x0, x1);
    const double t = mlp_guess_wave(ph, sMlp, x0, x1, lane);
    if (!valid) continue;
    if (!polish) {
      Tg[q] = t;
      continue;
    }
    const double zero_bg[4] = {0.0, 0.0, 0.0, 0.0};
    PrimOut o;
    cons2prim<true>(ph, u, b, t, zero_bg, o, ph.newton_maxit_mlp);
    if (o.bad) atomicOr(flags, o.bad);
    nit += o.iters;
    nmax = o.iters > nmax ? o.iters : nmax;
    nfb += o.fallback;
    Tg[q] = o.T;
    if (P) P[q] = o.w[Q_P];  // full pressure: the background passed is zero
  }
  if (stats) {
    // block totals of the Newton statistics
    __shared__ unsigned long long s_it[4], s_fb[4], s_mx[4];
    for (int o = 32; o > 0; o >>= 1) {
      nit += __shfl_xor(nit, o);
      nfb += __shfl_xor(nfb, o);
      const unsigned long long m = __shfl_xor(nmax, o);
      nmax = m > nmax ? m : nmax;
    }
    if (lane == 0) {
      s_it[threadIdx.x >> 6] = nit;
      s_fb[threadIdx.x >> 6] = nfb;
      s_mx[threadIdx.x >> 6] = nmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long a = 0, f = 0, m = 0;
      for (int w = 0; w < 4; ++w) {
        a += s_it[w];
        f += s_fb[w];
        m = s_mx[w] > m ? s_mx[w] : m;
      }
      atomicAdd(&stats[0], a);
      atomicMax(&stats[1], m);
      atomicAdd(&stats[2], f);
    }
  }
}

hipError_t launch_mlp_guess(const Ctx &c, const double *U, const double *Bx, const double *By,
                            const double *Bz, double *Tg, double *P, bool polish,
                            unsigned long long *stats) {
  long long nb = (long long)((c.ncell + 255) / 256);
  nb = nb < 8192 ? nb : 8192;
  hipLaunchKernelGGL(mlp_guess_kernel, dim3((unsigned)nb), dim3(256), 0, c.stream, c.ph, U, Bx,
                     By, Bz, c.mlp, Tg, P, c.flags, polish ? 1 : 0, stats);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// batch temperature inversion T(rho, e_int) (EOS microbenchmark and guess
// quality): guess from an array, the learned network or the bracket
// ---------------------------------------------------------------------------

template <bool ML>
__global__ __launch_bounds__(256) void eos_solve_kernel(
    Phys ph, const double *__restrict__ rho, const double *__restrict__ e,
    const double *__restrict__ tguess, long long n, const void *mlp,
    double *__restrict__ T, double *__restrict__ T0, unsigned long long *stats, int *flags) {
  __shared__ __attribute__((aligned(16))) char sMlpRaw[ML ? sizeof(MlpLds) : 16];
  const MlpLds &sMlp = *reinterpret_cast<const MlpLds *>(sMlpRaw);
  if (ML) {
    stage_mlp(mlp, sMlpRaw, threadIdx.x, 256);
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  unsigned long long it = 0, mx = 0, fb = 0;
  int bad = 0;
  // the next sample's inputs are requested before this one is solved
  const long long stride = (long long)gridDim.x * blockDim.x;
  long long base = (long long)blockIdx.x * blockDim.x;
  double rn = 0.0, en = 0.0, gn = NAN;
  if (base < n) {
    const long long q0 = base + threadIdx.x < n ? base + threadIdx.x : n - 1;
    rn = rho[q0];
    en = e[q0];
    if (tguess) gn = tguess[q0];
  }
  for (; base < n; base += stride) {
    const bool valid = base + threadIdx.x < n;
    const long long q = valid ? base + threadIdx.x : n - 1;
    const double r = rn, ee = en;
    double g = gn;
    if (base + stride < n) {
      const long long qn =
          base + stride + threadIdx.x < n ? base + stride + threadIdx.x : n - 1;
      rn = rho[qn];
      en = e[qn];
      if (tguess) gn = tguess[qn];
    }
    if (ML) {
      float x0, x1;
      mlp_inputs(ph, r, ee, x0, x1);
      g = mlp_guess_wave(ph, sMlp, x0, x1, lane);
    }
    double t = NAN;
    int iters = 0, fallback = 0;
    int rc = 1;
    if (r > 0.0 && ee > 0.0)
      rc = eos_temperature(ph, r, ee, g, ML ? ph.newton_maxit_mlp : ph.newton_maxit, t, iters,
                           fallback);
    if (!valid) continue;
    T[q] = t;
    if (T0) T0[q] = g;
    it += iters;
    mx = iters > mx ? iters : mx;
    fb += fallback;
    bad |= rc ? 2 : 0;
  }
  if (bad) atomicOr(flags, bad);
  if (!stats) return;  // block-uniform: no statistics requested
  // statistics: wave, then block totals, one set of atomics per block
  for (int o = 32; o > 0; o >>= 1) {
    it += __shfl_xor(it, o);
    fb += __shfl_xor(fb, o);
    const unsigned long long m2 = __shfl_xor(mx, o);
    mx = m2 > mx ? m2 : mx;
  }
  __shared__ unsigned long long s_st[3][4];
  const int wv = threadIdx.x >> 6;
  if (lane == 0) {
    s_st[0][wv] = it;
    s_st[1][wv] = mx;
    s_st[2][wv] = fb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long a = 0, m = 0, f = 0;
    for (int w = 0; w < 4; ++w) {
      a += s_st[0][w];
      m = s_st[1][w] > m ? s_st[1][w] : m;
      f += s_st[2][w];
    }
    atomicAdd(&stats[0], a);
    atomicMax(&stats[1], m);
    atomicAdd(&stats[2], f);
  }
}

hipError_t launch_eos_solve(const Ctx &c, const double *rho, const double *e,
                            const double *tguess, long long n, double *T, double *T0,
                            bool stats) {
  // With the network three rounds of the three resident blocks per CU: each
  // block stages the 17.5 KB of weights, 8192 blocks for a few hundred samples
  // each (4.0 M samples 67.7 -> 63.3 us a call, 16.8 M 256 -> 254, 0.3 M the
  // same; two rounds 65.0, four 64.8, one 66.8)
  const long long cap = c.d.eos_guess == MHD_GUESS_MLP ? 9ll * c.cus : 8192;
  long long nb = (n + 255) / 256;
  nb = nb < cap ? nb : cap;
  unsigned long long *st = stats ? c.nstats : nullptr;
  if (c.d.eos_guess == MHD_GUESS_MLP)
    hipLaunchKernelGGL(eos_solve_kernel<true>, dim3((unsigned)nb), dim3(256), 0, c.stream, c.ph,
                       rho, e, tguess, n, c.mlp, T, T0, st, c.flags);
  else
    hipLaunchKernelGGL(eos_solve_kernel<false>, dim3((unsigned)nb), dim3(256), 0, c.stream, c.ph,
                       rho, e, tguess, n, c.mlp, T, T0, st, c.flags);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// diagnostics: div B (eq. divb), |B_face| max, conservation totals
// ---------------------------------------------------------------------------

constexpr int DIAG_BLOCKS = 1024;
constexpr int NDIAG = 9;  // divb max, divb^2 sum, |B| max, 5 totals, bflux_x0

__global__ __launch_bounds__(256) void diag_kernel(Phys ph, const double *__restrict__ U,
                                                   const double *__restrict__ Bx,
                                                   const double *__restrict__ By,
                                                   const double *__restrict__ Bz,
                                                   double *__restrict__ part) {
  const size_t plane = (size_t)ph.nx * ph.ny;
  const size_t n = plane * ph.nz;
  const double dmin = fmin(ph.dx, fmin(ph.dy, ph.dz));
  double v[NDIAG];
  for (int f = 0; f < NDIAG; ++f) v[f] = 0.0;
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (size_t)gridDim.x * blockDim.x) {
    int i, j, k;
    cell_ijk(ph, q, i, j, k);
    const int ip = i + 1 == ph.nx ? 0 : i + 1;
    const int jp = j + 1 == ph.ny ? 0 : j + 1;
    const int kp = ph.reflect ? k + 1 : (k + 1 == ph.nz ? 0 : k + 1);
    const double bxl = Bx[q], bxr = Bx[q - i + ip];
    const double byl = By[q], byr = By[q + (size_t)(jp - j) * ph.nx];
    const double bzl = Bz[q], bzr = Bz[(size_t)kp * plane + (q - (size_t)k * plane)];
    const double d = ((bxr - bxl) * ph.idx + (byr - byl) * ph.idy + (bzr - bzl) * ph.idz) * dmin;
    v[0] = fmax(v[0], fabs(d));
    v[1] += d * d;
    v[2] = fmax(v[2], fmax(fabs(bxl), fmax(fabs(byl), fabs(bzl))));
    if (ph.reflect && k == ph.nz - 1) v[2] = fmax(v[2], fabs(bzr));
    for (int f = 0; f < 5; ++f) v[3 + f] += U[f * n + q];
    if (i == 0) v[8] += bxl;
  }
  __shared__ double sm[NDIAG][256];
  for (int f = 0; f < NDIAG; ++f) sm[f][threadIdx.x] = v[f];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      sm[0][threadIdx.x] = fmax(sm[0][threadIdx.x], sm[0][threadIdx.x + s]);
      sm[2][threadIdx.x] = fmax(sm[2][threadIdx.x], sm[2][threadIdx.x + s]);
      sm[1][threadIdx.x] += sm[1][threadIdx.x + s];
      for (int f = 3; f < NDIAG; ++f) sm[f][threadIdx.x] += sm[f][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x < NDIAG) part[(size_t)threadIdx.x * DIAG_BLOCKS + blockIdx.x] = sm[threadIdx.x][0];
}

hipError_t launch_diagnostics(const Ctx &c, const double *U, const double *Bx,
                              const double *By, const double *Bz, double *out) {
  hipLaunchKernelGGL(diag_kernel, dim3(DIAG_BLOCKS), dim3(256), 0, c.stream, c.ph, U, Bx, By, Bz,
                     c.red);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  static thread_local double host[NDIAG * DIAG_BLOCKS];
  e = hipMemcpyAsync(host, c.red, sizeof(double) * NDIAG * DIAG_BLOCKS, hipMemcpyDeviceToHost,
                     c.stream);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(c.stream);
  if (e != hipSuccess) return e;
  // fixed-order host reduction of the block partials
  for (int f = 0; f < NDIAG; ++f) {
    long double s = 0.0L;
    double m = 0.0;
    for (int b = 0; b < DIAG_BLOCKS; ++b) {
      const double x = host[(size_t)f * DIAG_BLOCKS + b];
      if (f == 0 || f == 2)
        m = x > m ? x : m;
      else
        s += x;
    }
    out[f] = (f == 0 || f == 2) ? m : (double)s;
  }
  return hipSuccess;
}

__global__ void zero_walls_kernel(double *Bz, size_t plane, size_t top) {
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < plane;
       q += (size_t)gridDim.x * blockDim.x) {
    Bz[q] = 0.0;
    Bz[top + q] = 0.0;
  }
}

hipError_t launch_zero_walls(const Ctx &c, double *Bz) {
  const size_t plane = (size_t)c.ph.nx * c.ph.ny;
  int nb = (int)((plane + 255) / 256);
  nb = nb < 1024 ? nb : 1024;
  hipLaunchKernelGGL(zero_walls_kernel, dim3(nb), dim3(256), 0, c.stream, Bz, plane,
                     plane * (size_t)c.ph.nz);
  return hipGetLastError();
}

}  // namespace mhd
