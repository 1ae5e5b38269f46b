// Matrix-free application of the finite-difference 6x6 hole Hamiltonian and
// the fused Chebyshev recurrence step
//
//     Y = alpha (H - shift) X + beta Y_old
//
// (the filter of the Rayleigh-Chebyshev subspace iteration, paper Sec. II.B).
//
// H in the |L S> basis (paper Eq. LK) is, per spin block, a 19-point stencil:
//   faces    -(E0/h^2) [ (L-M) S_ii + M (S_x + S_y + S_z) ]     on every component
//   edges    E0 N Ksym_ab coupling orbital components a <-> b (4 diagonal
//            neighbours in the (a,b) plane, two L-shaped Peierls paths averaged)
//   on-site  the orbital 3x3 block V + H_eps(r), the kinetic centre, spin-orbit
//            and Zeeman (a constant 6x6, evaluated in closed form)
// with L = g1+4g2, M = g1-2g2, N = 6 g3.
//
// Kernel design (gfx950): a workgroup owns a tile of (x, y) columns of one vector
// and marches along z.  Each plane (with a one-point halo ring) is staged through
// LDS once; every thread reads its 19-point neighbourhood from LDS and "pushes" the
// plane's contributions into three register accumulators for the output planes z-1,
// z and z+1.  The x-z and y-z edge couplings of a plane therefore need only that
// plane's x/y neighbours, so one plane of LDS per vector suffices.  Planes are
// double-buffered in LDS (one barrier per plane).  Output plane z-1 is complete after
// plane z has been pushed and is written straight to memory (alpha, beta and the old
// block fused in).  Workgroups are mapped to XCDs in contiguous runs so that the
// vectors of one tile share an L2.  Two ways of staging a plane: copies of whole rows
// (stencil_kernel) and through registers (stencil_pipe_kernel); launch_t chooses.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "hkp_internal.h"
#include "stencil_ops.h"

namespace hkp {

namespace {

using namespace sten;

template <typename T>
struct KArgs {
  const T* in;
  long long in_bstride;
  const void* old;
  long long old_bstride;
  void* out;
  long long out_bstride;
  const T* D;
  long long D_bstride;
  const T* ptab;   // [nz][kFoldRow] complex: folded phases per plane (field on)
  const double* ptab64;   // the same in double, and [nx] complex the y-links' phase along x
  const double* utab64;   // (Bz != 0)
  const double* coef;
  int coef_stride;
  double alpha, shift, beta;
  const int* active;
  const int* lock;
  const int* work;
  int batch;
  int vfirst;
  int zsplit;   // z-ranges that the grid leaves room for
  int zfixed;   // z-ranges of the launch, or 0: from the live count
  ZCut cut;     // the planes in zfixed ranges
  float c0;
  float cus, icus;   // compute units of the device, and their reciprocal
  int stream;   // blocks beyond the cache: the old block and the output pass it by
  int nx, ny, nz, nvec;
  int tiles_x, tiles_y;
  int vgroup;   // vectors of one tile run side by side (1: vector-major)
  double h;     // weighted inputs: the grid spacing
  StencilConsts<T> k;
};

// Which (member, vector, tile, z range) this workgroup works on; false: none.
// Workgroup order: groups of vgroup vectors; inside a group the vectors of
// one tile are adjacent (they share the tile's on-site fields in L2) and the
// tiles follow each other (neighbouring tiles march z side by side on one XCD,
// so the halo rows they share hit in L2).  vgroup = 1 is vector-major order,
// vgroup = nvec tile-major order.  With a work table the order runs over the
// live (virtual) vectors of all members and the rest of the grid exits.
// Launches with few live workgroups (locked vectors, converged members, small grids
// and groups) split every (vector, tile) into zs z-ranges so that more workgroups
// share the chip evenly; a range recomputes one plane on each side.  The grid holds
// zsplit x the unsplit count; the split is decided from the live count, uniformly
// for the whole launch (z_ranges).
struct Place {
  int b, vec, tile, zc;
  ZCut cut;
};

template <typename T>
__device__ __forceinline__ bool find_place(const KArgs<T>& a, Place* p) {
  const int ntiles = a.tiles_x * a.tiles_y;
  const int nv = a.work ? a.work[a.batch] : 0;   // live vectors
  const int nlw = a.work ? nv * ntiles : (int)gridDim.x / a.zsplit;
  int zs = 1;
  p->cut = a.cut;
  if (a.zsplit > 1) {
    zs = a.zfixed;
    if (zs == 0) {
      const ZRanges z = z_ranges(nlw, a.nz, a.zsplit, a.c0, a.cus, a.icus);
      zs = __builtin_amdgcn_readfirstlane(z.zs);
      const ZCut c = z_cut(a.nz, z);
      p->cut.q = __builtin_amdgcn_readfirstlane(c.q);
      p->cut.r = __builtin_amdgcn_readfirstlane(c.r);
      p->cut.m = (unsigned)__builtin_amdgcn_readfirstlane((int)c.m);
    }
  }
  const int nlive = nlw * zs;
  if (nlive <= 0 || (int)blockIdx.x >= nlive) return false;
  int logical = xcd_remap(blockIdx.x, nlive);
  p->zc = logical / nlw;   // z range outermost: one range of all tiles per XCD run
  logical -= p->zc * nlw;
  if (a.work) {
    const int g = logical / (a.vgroup * ntiles);
    const int within = logical - g * a.vgroup * ntiles;
    const int gsize = min(a.vgroup, nv - g * a.vgroup);
    p->tile = within / gsize;
    const int u = g * a.vgroup + (within - p->tile * gsize);
    int b = 0;
    while (a.work[b + 1] <= u) ++b;
    p->b = b;
    p->vec = (a.lock ? a.lock[b] : 0) + (u - a.work[b]);
    return true;
  }
  const int per_b = ntiles * a.nvec;
  p->b = logical / per_b;
  const int r = logical - p->b * per_b;
  const int g = r / (a.vgroup * ntiles);
  const int within = r - g * a.vgroup * ntiles;
  const int gsize = min(a.vgroup, a.nvec - g * a.vgroup);
  p->tile = within / gsize;
  p->vec = a.vfirst + g * a.vgroup + (within - p->tile * gsize);
  if (a.active && !a.active[p->b]) return false;
  return !(a.lock && p->vec < a.lock[p->b]);   // converged vectors are not filtered
}

// (in scalar registers, so that everything derived from it is uniform to the compiler)
template <typename T>
__device__ __forceinline__ bool place_workgroup(const KArgs<T>& a, Place* p) {
  if (!find_place(a, p)) return false;
  p->b = __builtin_amdgcn_readfirstlane(p->b);
  p->vec = __builtin_amdgcn_readfirstlane(p->vec);
  p->tile = __builtin_amdgcn_readfirstlane(p->tile);
  p->zc = __builtin_amdgcn_readfirstlane(p->zc);
  return true;
}

// the coefficients alpha, shift, beta of this launch's step for member b
template <typename T>
__device__ __forceinline__ void step_coef(const KArgs<T>& a, int b, T* alpha, T* shift, T* beta) {
  if (a.coef) {
    const double* c = a.coef + (long long)b * a.coef_stride;
    *alpha = (T)c[0];
    *shift = (T)c[1];
    *beta = (T)c[2];
  } else {
    *alpha = (T)a.alpha;
    *shift = (T)a.shift;
    *beta = (T)a.beta;
  }
}

// barrier for LDS traffic alone: global loads and stores stay in flight across it
// (__syncthreads would wait for every store to reach memory)
__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

// waves per SIMD that the register budget is held to: FP32 four (128 registers; the
// general phases' recurrence step would spill: three), FP64 two
template <typename T>
constexpr int pipe_waves(int ph, bool old, int ty) {
  return sizeof(T) == 4 && ty > 1 ? (ph == 2 && old ? 3 : 4) : 2;
}

// Register-staged march.  A tile is TX x (64 / TX x TY) columns: a wave covers 64 / TX
// rows of TX columns of one spin, so grids that 64-wide tiles would pad (nx = 96, 75)
// keep their lanes busy.  Plane z + 2 is loaded into registers while plane z is
// computed, and written to LDS one step later.  One wait per step, at its top, covers
// every load issued a whole step before (that plane, the on-site fields, the old
// block) and the stores of the step before it; then come this step's stores and
// loads, then the arithmetic.  Nothing that was just issued is waited for, and the
// barrier at the end waits for LDS alone.
// A lane's offsets are 32-bit bytes from a uniform base; TY = 1 (nx beyond 2^22) takes
// 64-bit ones.
// WGT: the input is formed on its way to LDS, vector 4 c + i from vector i times 1 or a
// coordinate about the box centre (the g-matrices' twelve weighted vectors are never
// stored: of 256 x 48 x 48 429 us for the sixteen, 441 from stored ones and 161 to store
// them; the four that share their inputs run side by side).
template <typename T, typename TO, typename TW, int PH, bool STR, int TX, int TY, int NC = 6,
          bool WGT = false>
__global__ void __launch_bounds__(64 * TY * (NC / 3), pipe_waves<T>(PH, !std::is_same<TO, void>::value, TY))
stencil_pipe_kernel(KArgs<T> a) {
  static_assert(NC == 6 || (NC == 3 && PH == 0), "spin-free vectors carry no field terms");
  constexpr bool kWide = TY == 1;
  constexpr int RH = (64 / TX) * TY;        // rows of the tile
  constexpr int W = TX + 2, ROWS = RH + 2;
  constexpr int PLANE = W * ROWS;
  constexpr int NT = 64 * TY * (NC / 3);
  constexpr int NS = (PLANE + NT - 1) / NT;
  constexpr int BUF = NC * PLANE;
  constexpr bool kOld = !std::is_same<TO, void>::value;
  using TOv = std::conditional_t<kOld, TO, T>;
  __shared__ cx<T> lds[2 * BUF];

  Place pl;
  if (!place_workgroup(a, &pl)) return;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int tx0 = (pl.tile % a.tiles_x) * TX, ty0 = (pl.tile / a.tiles_x) * RH;
  // output planes [o0, o1) of this range; input planes p0..p1 feed them
  const int o0 = range_begin(pl.zc, pl.cut), o1 = range_begin(pl.zc + 1, pl.cut);
  const int p0 = o0 > 0 ? o0 - 1 : 0, p1 = o1 < nz ? o1 : nz - 1;
  const unsigned nxy = (unsigned)nx * (unsigned)ny;
  const unsigned N = nxy * (unsigned)nz;   // 6 N < 2^31 (checked on the host)
  const int lane = threadIdx.x;
  const int lx = lane & (TX - 1), ly = threadIdx.y * (64 / TX) + lane / TX;
  // the spin is uniform across a wave (64 consecutive threads share threadIdx.z)
  const int sp = __builtin_amdgcn_readfirstlane(threadIdx.z);
  const int tid = lane + 64 * ((int)threadIdx.y + TY * sp);
  const int gx = tx0 + lx, gy = ty0 + ly;
  const bool mine = gx < nx && gy < ny;
  const int X = 3 * sp, F = 3 - X;      // own and flipped-spin component offsets

  T alpha, shift, beta;
  step_coef(a, pl.b, &alpha, &shift, &beta);
  const bool has_old = kOld && a.old != nullptr && beta != (T)0;

  // bases at this tile's first row (uniform); lane offsets in bytes from there
  const size_t row0 = (size_t)ty0 * nx;
  const long long vb = (long long)pl.vec * NC * N;
  const T* in = a.in + 2 * ((long long)pl.b * a.in_bstride +
                            (WGT ? (long long)(pl.vec & 3) * NC * N : vb));
  // (without an old block its loads read the block's first entry and are not used)
  const TOv* oldp = has_old ? reinterpret_cast<const TOv*>(a.old) +
                                  2 * ((long long)pl.b * a.old_bstride + vb + (long long)X * N + row0)
                            : reinterpret_cast<const TOv*>(a.in);
  const unsigned oldN = has_old ? N : 0u, oldxy = has_old ? nxy : 0u;
  TW* outp = reinterpret_cast<TW*>(a.out) +
             2 * ((long long)pl.b * a.out_bstride + vb + (long long)X * N + row0);
  const T* D = a.D + (long long)pl.b * a.D_bstride + row0;
  using Off = std::conditional_t<kWide, size_t, unsigned>;
  // base + a lane's offset; the empty statement keeps the offset's extension to 64 bits
  // beside the access, where it folds into the instruction's address
  auto ptr = [](auto* base, Off bytes) {
    using P = std::conditional_t<std::is_const<std::remove_pointer_t<decltype(base)>>::value,
                                 const char*, char*>;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(bytes));
#endif
    return reinterpret_cast<decltype(base)>(reinterpret_cast<P>(base) + bytes);
  };
  const StencilConsts<T> k = a.k;
  const T dgs = sp == 0 ? k.dgU : k.dgD;
  const T ax = sp == 0 ? k.aUx : k.aDx, ay = sp == 0 ? k.aUy : k.aDy,
          az = sp == 0 ? k.aUz : k.aDz;
  const T sd3 = sp == 0 ? -k.d3 : k.d3;   // sign of the d3 f_Z and f_X spin-flip terms
  const T sby = sp == 0 ? -k.by : k.by;   // (bx -+ i by)

  // halo-tile slots this thread stages (a slot outside the grid loads the tile's first
  // column and stores zero); offsets are from the tile's first row or the row above it
  const int up = ty0 > 0 ? 1 : 0;
  const T* inr = in + 2 * (row0 - (size_t)(up * nx));
  Off soff[NS];
  int sidx[NS];
  bool sval[NS];
  T wgt[WGT ? NS : 1];   // a slot's weight (x, y), and the plane's (z)
  const int waxis = WGT ? pl.vec >> 2 : 0;
  auto centred = [&](int i, int n) { return (T)((i - 0.5 * (n - 1)) * a.h); };
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int slot = tid + s * NT;
    const int row = slot / W, colx = slot - row * W;
    const int x = tx0 + colx - 1, y = ty0 + row - 1;
    if constexpr (WGT)
      wgt[s] = waxis == 1 ? centred(x, nx) : waxis == 2 ? centred(y, ny) : (T)1;
    sval[s] = slot < PLANE && x >= 0 && x < nx && y >= 0 && y < ny;
    soff[s] = sval[s] ? (Off)((Off)(row - 1 + up) * (Off)nx + (Off)x) * (Off)sizeof(cx<T>)
                      : (Off)tx0 * (Off)sizeof(cx<T>);
    sidx[s] = slot < PLANE ? slot : -1;
  }
  const Off col = mine ? (Off)ly * (Off)nx + (Off)gx : (Off)tx0;
  const Off colT = col * (Off)sizeof(T), colO = has_old ? col * (Off)sizeof(cx<TOv>) : (Off)0,
            colW = col * (Off)sizeof(cx<TW>);
  const int lb = (ly + 1) * W + (lx + 1);   // this thread's centre in an LDS plane
  cx<double> ux = mk<double>(1, 0);
  if constexpr (PH == 2) ux = ld(a.utab64 + 2 * (gx < nx ? gx : nx - 1));
  // the folded phases' rows, from plane p0 on (advanced: a product per plane costs more)
  const T* frow = a.ptab + (PH != 0 ? fold_offset(p0) : 0);
  const double* frow64 = a.ptab64 + (PH == 2 ? fold_offset(p0) : 0);

  const bool stream = a.stream != 0;

  constexpr int ND = STR ? 6 : 1;
  struct Set {          // what a step needs besides the plane: loaded one step ahead
    T d[ND];            // on-site fields of the plane (d00 d11 d22 d12 d02 d01, or V)
    cx<TOv> old[3];     // old block of the plane before it
  };
  // a plane's offset, kept out of the compiler's induction variables so that every
  // access stays a uniform base plus a 32-bit lane offset
  auto plane = [&](int z, unsigned stride) -> size_t {
    return (size_t)(unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)z * stride));
  };
  cx<T> R[NS][NC];
  auto fetch = [&](int z) {
    const T* q = inr + 2 * plane(z, nxy);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int c = 0; c < NC; ++c) R[s][c] = ld(ptr(q + 2 * (size_t)((unsigned)c * N), soff[s]));
  };
  auto commit = [&](int z) {
    cx<T>* dst = lds + (z & 1) * BUF;
    const T wz = WGT && waxis == 3 ? centred(z < nz ? z : nz - 1, nz) : (T)1;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (PLANE % NT != 0 && sidx[s] < 0) continue;
      if constexpr (WGT)
#pragma unroll
        for (int c = 0; c < NC; ++c) R[s][c] = scl(wgt[s] * wz, R[s][c]);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        dst[c * PLANE + sidx[s]] = sval[s] ? R[s][c] : mk<T>(0, 0);
    }
  };
  auto load_fields = [&](int z, Set& t) {
    const T* q = D + plane(z, nxy);
#pragma unroll
    for (int i = 0; i < ND; ++i) t.d[i] = *ptr(q + (size_t)i * N, colT);
  };
  auto load_old = [&](int z, Set& t) {
    if constexpr (kOld) {
      const TOv* q = oldp + 2 * plane(z, oldxy);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const TOv* p = ptr(q + 2 * (size_t)(i * oldN), colO);
        t.old[i] = stream ? ld_stream(p) : ld(p);
      }
    }
  };
  cx<T> acc0[3], acc1[3], res[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) acc0[i] = acc1[i] = res[i] = mk<T>(0, 0);
  auto store = [&](int z) {
    if (!mine) return;
    TW* q = outp + 2 * plane(z, nxy);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      TW* p = ptr(q + 2 * (size_t)i * N, colW);
      if (stream) stg_stream<TW>(p, 0, res[i]); else stg<TW>(p, 0, res[i]);
    }
  };
  auto finish = [&](const Set& t) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      res[i] = scl(alpha, acc0[i]);
      if constexpr (kOld)
        if (has_old) res[i] = fma_s(res[i], beta, mk<T>((T)t.old[i].r, (T)t.old[i].i));
    }
  };

  // step z: plane z + 1 to LDS, the finished plane z - 2 to memory, then the loads for
  // step z + 1 and beyond, then plane z (which completes plane z - 1)
  auto step = [&](int z, const Set& cur, Set& nxt) {
    commit(z + 1);
    if (z - 2 >= o0) store(z - 2);
    fetch(z + 2 < p1 ? z + 2 : p1);
    load_fields(z + 1 < nz ? z + 1 : z, nxt);
    load_old(z < o1 ? (z > o0 ? z : o0) : o1 - 1, nxt);
    const Fold<T> f = load_fold<T, PH>(frow, frow64, ux);
    if constexpr (PH != 0) frow += fold_offset(1);
    if constexpr (PH == 2) frow64 += fold_offset(1);
    const T d00 = cur.d[0], d11 = cur.d[STR ? 1 : 0], d22 = cur.d[STR ? 2 : 0];
    const T d12 = STR ? cur.d[STR ? 3 : 0] : (T)0;
    const T d02 = STR ? cur.d[STR ? 4 : 0] : (T)0;
    const T d01 = STR ? cur.d[STR ? 5 : 0] : (T)0;
    cx<T> acc2[3];
    push_plane<T, PH, STR, NC, PLANE, W>(lds + (z & 1) * BUF + lb, X, F, k, dgs, ax, ay, az, sd3,
                                         sby, shift, f, d00, d11, d22, d12, d02, d01, acc0, acc1,
                                         acc2);
    finish(cur);
    settle(acc1);
    settle(acc2);
    settle(res);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      acc0[i] = acc1[i];
      acc1[i] = acc2[i];
    }
    lds_barrier();
  };

  Set A, B;
  fetch(p0);
  load_fields(p0, A);
  load_old(o0, A);
  commit(p0);
  fetch(p0 < p1 ? p0 + 1 : p1);
  lds_barrier();
  int z = p0;
  for (; z + 1 <= p1; z += 2) {
    step(z, A, B);
    step(z + 1, B, A);
  }
  if (z <= p1) {
    step(z, A, B);
    A = B;
    ++z;
  }
  // z = p1 + 1: plane z - 2 is in res; with p1 the grid's last plane (o1 = nz), plane
  // z - 1 has no successor to complete it
  if (z - 2 >= o0) store(z - 2);
  if (o1 == nz) {
    finish(A);
    store(nz - 1);
  }
}

// Row-copy march, for grids of whole 64-wide tiles: the 64 interior elements of every
// halo-tile row go global -> LDS directly (global_load_lds, no registers), issued one
// plane ahead and waited for at the end of the step; the two x-halo columns use
// ordinary loads.
// NC = 6: the full spinor (a wave per spin and row).  NC = 3: a spin-free orbital
// vector (X, Y, Z of one spin; no spin-orbit or field terms, so nothing couples
// it to the other spin): one wave per row and half the bytes.
template <typename T, typename TO, typename TW, int PH, bool STR, int TY, int NC = 6>
__global__ void __launch_bounds__(64 * TY * (NC / 3))
stencil_kernel(KArgs<T> a) {
  static_assert(NC == 6 || (NC == 3 && PH == 0), "spin-free vectors carry no field terms");
  static_assert(sizeof(T) == 8, "a lane copies one complex entry of 16 bytes");
  constexpr int C0 = 1;   // column of x = tx0 in an LDS row: left halo, 64 interior, right halo
  constexpr int W = 66;
  constexpr int ROWS = TY + 2;
  constexpr int SLOTS = W * ROWS;
  constexpr int PLANE = SLOTS;        // elements per (buffer, component) plane
  constexpr int NT = 64 * TY * (NC / 3);   // (x, y, spin) threads
  // double-buffered plane: [component][row][col] each (two distinct arrays, so the
  // compiler can tell the buffer being read from the one being filled)
  __shared__ cx<T> lds0[NC * PLANE];
  __shared__ cx<T> lds1[NC * PLANE];
  auto bufp = [&](auto BUF) -> cx<T>* {
    if constexpr (decltype(BUF)::value == 0) return lds0; else return lds1;
  };

  Place pl;
  if (!place_workgroup(a, &pl)) return;
  const int b = pl.b, vec = pl.vec, tile = pl.tile, zc = pl.zc;
  const int tx0 = (tile % a.tiles_x) * 64;
  const int ty0 = (tile / a.tiles_x) * TY;

  const int nx = a.nx, ny = a.ny, nz = a.nz;
  // output planes [o0, o1) of this range; input planes p0..p1 feed them
  const int o0 = range_begin(zc, pl.cut), o1 = range_begin(zc + 1, pl.cut);
  const int p0 = o0 > 0 ? o0 - 1 : 0, p1 = o1 < nz ? o1 : nz - 1;
  const unsigned nxy = (unsigned)nx * (unsigned)ny;
  const unsigned N = nxy * (unsigned)nz;   // 6 N < 2^31 (checked on the host)
  const int lx = threadIdx.x, ly = threadIdx.y;
  // the spin is uniform across a wave (64 consecutive threads share threadIdx.z)
  const int sp = __builtin_amdgcn_readfirstlane(threadIdx.z);
  const int tid = lx + 64 * (ly + TY * sp);
  const int gx = tx0 + lx, gy = ty0 + ly;
  const bool mine = gx < nx && gy < ny;
  const int X = 3 * sp, F = 3 - X;      // own and flipped-spin component offsets

  T alpha, shift, beta;
  step_coef(a, b, &alpha, &shift, &beta);
  // TO = void: a launch without an old block (a step of the product-form filter,
  // or H X), compiled without its loads
  constexpr bool kOld = !std::is_same<TO, void>::value;
  using TOv = std::conditional_t<kOld, TO, T>;
  const bool has_old = kOld && a.old != nullptr && beta != (T)0;

  // uniform (scalar) bases; lane offsets are 32-bit element indices
  const T* __restrict__ in = a.in + 2 * ((long long)b * a.in_bstride + (long long)vec * NC * N);
  const TOv* __restrict__ oldp = has_old
      ? reinterpret_cast<const TOv*>(a.old) +
            2 * ((long long)b * a.old_bstride + (long long)vec * NC * N + (long long)X * N)
      : nullptr;
  TW* __restrict__ outp = reinterpret_cast<TW*>(a.out) +
                          2 * ((long long)b * a.out_bstride + (long long)vec * NC * N +
                               (long long)X * N);
  const T* __restrict__ D = a.D + (long long)b * a.D_bstride;
  const StencilConsts<T> k = a.k;
  // spin-dependent constants (sp is wave-uniform: scalar selects)
  const T dgs = sp == 0 ? k.dgU : k.dgD;
  const T ax = sp == 0 ? k.aUx : k.aDx, ay = sp == 0 ? k.aUy : k.aDy,
          az = sp == 0 ? k.aUz : k.aDz;
  const T sd3 = sp == 0 ? -k.d3 : k.d3;   // sign of the d3 f_Z and f_X spin-flip terms
  const T sby = sp == 0 ? -k.by : k.by;   // (bx -+ i by)

  const unsigned col = mine ? (unsigned)(gy * nx + gx) : 0u;
  const int gxc = gx < nx ? gx : nx - 1;
  const int lb = (ly + 1) * W + (lx + C0);   // this thread's centre in an LDS plane

  cx<T> acc0[3], acc1[3], oldv[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) acc0[i] = acc1[i] = oldv[i] = mk<T>(0, 0);

  // row copies spread over the workgroup's waves
  constexpr int NW = TY * (NC / 3);
  const int wave = __builtin_amdgcn_readfirstlane(ly + TY * sp);
  auto dma_plane = [&](int z, auto BUF) {
    cx<T>* dst = bufp(BUF);
    const unsigned zo = (unsigned)z * nxy;
    for (int j = wave; j < NC * ROWS; j += NW) {
      const int c = j / ROWS, r = j % ROWS;
      const int y = ty0 + r - 1;
      if (y < 0 || y >= ny) continue;
      const T* src = in + 2 * (size_t)((unsigned)c * N + zo + (unsigned)(y * nx + tx0)) +
                     2 * lx;
      dma16(src, dst + c * PLANE + r * W + C0);
    }
  };
  // x-halo columns: element e of 12 ROWS per plane (side, component, row)
  const int he = tid;
  const bool hown = he < 2 * NC * ROWS;
  const int hside = he & 1, hc = (he >> 1) % NC, hr = (he >> 1) / NC;
  const int hx = hside ? tx0 + 64 : tx0 - 1, hy = ty0 + hr - 1;
  const bool hval = hown && hx >= 0 && hx < nx && hy >= 0 && hy < ny;
  const unsigned hoff = hval ? (unsigned)(hc * N + hy * nx + hx) : 0u;
  const int hidx = hc * PLANE + hr * W + (hside ? C0 + 64 : C0 - 1);
  auto halo_load = [&](int z) -> cx<T> {
    cx<T> v = mk<T>(0, 0);
    if (hval) v = ld(in + 2 * (size_t)(hoff + (unsigned)z * nxy));
    return v;
  };
  auto halo_commit = [&](cx<T> v, auto BUF) {
    if (hown) bufp(BUF)[hidx] = v;
  };

  auto load_old = [&](int z) {
    if (!kOld || !has_old || !mine) return;
    const unsigned o = (unsigned)z * nxy + col;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const TOv* p = oldp + 2 * (size_t)((unsigned)i * N + o);
      cx<TOv> q = a.stream ? ld_stream(p) : ld(p);
      oldv[i] = mk<T>((T)q.r, (T)q.i);
    }
  };
  auto finalize = [&](int z) {
    if (!mine) return;
    const unsigned o = (unsigned)z * nxy + col;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      cx<T> r = scl(alpha, acc0[i]);
      if (kOld && has_old) r = fma_s(r, beta, oldv[i]);
      const long long w = (long long)((unsigned)i * N + o);
      if (a.stream) stg_stream<TW>(outp, w, r); else stg<TW>(outp, w, r);
    }
  };

  cx<double> ux = mk<double>(1, 0);
  if constexpr (PH == 2) ux = ld(a.utab64 + 2 * gxc);
  const T* frow = a.ptab + (PH != 0 ? fold_offset(p0) : 0);   // as in the staged march
  const double* frow64 = a.ptab64 + (PH == 2 ? fold_offset(p0) : 0);

  // on-site fields of this column, loaded one plane ahead (d00 d11 d22 d12 d02 d01;
  // without strain only the first)
  constexpr int ND = STR ? 6 : 1;
  auto load_d = [&](int z, T (&d)[ND]) {
    const unsigned pz = (unsigned)z * nxy + col;
#pragma unroll
    for (int i = 0; i < ND; ++i) d[i] = D[(unsigned)i * N + pz];
  };
  T cd[ND];
  load_d(p0, cd);

  auto step = [&](int z, auto BUF) {
    constexpr int cur = decltype(BUF)::value;
    // loads in the order they are needed (the memory counter retires them in
    // order): the next plane's on-site fields, the old block for the output plane,
    // the next plane's halo, the next plane's rows (into the buffer that is not being
    // read; the barrier at the end of the step publishes it and retires this one)
    T nd[ND];
    load_d(z + 1 < nz ? z + 1 : z, nd);
    if (z - 1 >= o0) load_old(z - 1);
    cx<T> hv = mk<T>(0, 0);
    const bool more = z + 1 <= p1;
    if (more) {
      hv = halo_load(z + 1);
      dma_plane(z + 1, IC<1 - cur>{});
    }
    // (indices stay inside cd for ND = 1; the strain terms are then zero)
    const T d00 = cd[0], d11 = cd[STR ? 1 : 0], d22 = cd[STR ? 2 : 0];
    const T d12 = STR ? cd[STR ? 3 : 0] : (T)0;
    const T d02 = STR ? cd[STR ? 4 : 0] : (T)0;
    const T d01 = STR ? cd[STR ? 5 : 0] : (T)0;
    const cx<T>* L = bufp(IC<cur>{}) + lb;
    cx<T> acc2[3];
    const Fold<T> f = load_fold<T, PH>(frow, frow64, ux);
    if constexpr (PH != 0) frow += fold_offset(1);
    if constexpr (PH == 2) frow64 += fold_offset(1);
    push_plane<T, PH, STR, NC, PLANE, W>(L, X, F, k, dgs, ax, ay, az, sd3, sby, shift, f, d00,
                                         d11, d22, d12, d02, d01, acc0, acc1, acc2);

    // the output plane's stores (and the wait for the old block, which the
    // compiler extends to every load in flight, the next plane's copy included)
    // after all of this plane's arithmetic
    settle(acc1);
    settle(acc2);
    if (z - 1 >= o0) finalize(z - 1);
    if (more) halo_commit(hv, IC<1 - cur>{});
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      acc0[i] = acc1[i];
      acc1[i] = acc2[i];
    }
#pragma unroll
    for (int i = 0; i < ND; ++i) cd[i] = nd[i];
    __syncthreads();
  };

  // rows outside the grid are never loaded: zero both buffers once
  for (int i = tid; i < NC * PLANE; i += NT) {
    lds0[i] = mk<T>(0, 0);
    lds1[i] = mk<T>(0, 0);
  }
  __syncthreads();
  halo_commit(halo_load(p0), IC<0>{});
  dma_plane(p0, IC<0>{});
  __syncthreads();
  for (int z = p0; z <= p1; z += 2) {
    step(z, IC<0>{});
    if (z + 1 <= p1) step(z + 1, IC<1>{});
  }
  if (o1 == nz) {   // the last plane has no successor to complete it
    load_old(nz - 1);
    finalize(nz - 1);
  }
}

template <typename T, typename TO, typename TW, int PH, bool STR, int NC = 6>
hipError_t launch_t(const StencilLaunch& L, const StencilConsts<double>& c, hipStream_t s) {
  KArgs<T> a;
  a.in = reinterpret_cast<const T*>(L.in);
  a.in_bstride = L.in_bstride;
  a.old = L.old;
  a.old_bstride = L.old_bstride;
  a.out = L.out;
  a.out_bstride = L.out_bstride;
  a.D = reinterpret_cast<const T*>(L.D);
  a.D_bstride = L.D_bstride;
  a.ptab = reinterpret_cast<const T*>(L.ptab);
  a.ptab64 = L.ptab64;
  a.utab64 = L.utab64;
  a.coef = L.coef.coef;
  a.coef_stride = L.coef.stride;
  a.alpha = L.coef.alpha;
  a.shift = L.coef.shift;
  a.beta = L.coef.beta;
  a.active = L.active;
  a.lock = L.lock;
  a.work = L.work;
  a.batch = L.batch;
  a.nx = L.nx;
  a.ny = L.ny;
  a.nz = L.nz;
  const bool part = L.vcount > 0;
  if (part && (L.work || L.batch != 1)) return hipErrorInvalidValue;
  a.nvec = part ? L.vcount : L.nvec;
  a.vgroup = L.vgroup < 1 ? 1 : (L.vgroup > a.nvec ? a.nvec : L.vgroup);
  a.vfirst = part ? L.vfirst : 0;
  long long vectors = (long long)a.nvec * L.batch;
  if (L.work) vectors = table_vectors(vectors, L.vlive, L.vmost);
  // The old block (read for the last time) and the output pass the caches by where the
  // launch's blocks exceed the memory-side cache: they would only push out what is
  // read again (on-site fields, halo rows; a 40-vector FP32 step of 256 x 48 x 48: 711
  // us, 763 cached).  Blocks that fit are kept, for the next step to read (4 vectors:
  // 59 us, 72 streamed).
  const size_t entries = (size_t)vectors * NC * L.nx * L.ny * L.nz;
  a.stream = entries * (2 * sizeof(T) + 2 * sizeof(TW) +
                        (L.old && L.old != L.out ? 2 * (L.old_fp64 ? 8 : 4) : 0)) > kCacheBytes;
  a.k = cast_consts<T>(c);
  a.h = L.h;
  const int ty = L.tile_y;
  constexpr unsigned NSP = NC / 3;   // spin waves per row
  auto go = [&](auto kernel, int tx, int rows, int waves) {
    a.tiles_x = (L.nx + tx - 1) / tx;
    a.tiles_y = (L.ny + rows - 1) / rows;
    const long long nwg = (long long)a.tiles_x * a.tiles_y * vectors;
    if (nwg <= 0) return hipSuccess;
    // z split: 0 never, 1 as balances the launch (z_split), 2 always in two (tests)
    a.c0 = sizeof(T) == 8 ? 2.2f : (std::is_same<TO, void>::value ? 2.6f : 2.0f);
    const int cus = device_cus();
    a.cus = (float)cus;
    a.icus = 1.0f / (float)cus;
    a.zsplit = 1;
    ZRanges fixed{1, 1.0f};
    if (L.zsplit >= 2) {
      a.zsplit = 2;
      if (L.nz >= 8) fixed = ZRanges{2, 0.5f};
    } else if (L.zsplit == 1) {
      const ZSplit z = z_split(nwg, L.nz, L.work && L.vlive < 0, a.c0, cus);
      a.zsplit = z.room;
      fixed = z.fixed;
    }
    a.zfixed = fixed.zs;
    a.cut = z_cut(L.nz, fixed.zs > 0 ? fixed : ZRanges{1, 1.0f});
    if (nwg * a.zsplit > 0x7fffffffLL) return hipErrorInvalidValue;
    kernel<<<dim3((unsigned)(nwg * a.zsplit)), dim3(64, waves, NSP), 0, s>>>(a);
    return hipGetLastError();
  };
  constexpr bool can_weight = sizeof(T) == 8 && std::is_same<TO, void>::value && PH == 0 && NC == 6;
  if constexpr (can_weight) {
    if (L.weighted) {
      if (L.nvec != 16 || part || L.batch != 1 || L.work) return hipErrorInvalidValue;
      if (L.nx > (1 << 22)) return go(stencil_pipe_kernel<T, TO, TW, PH, STR, 64, 1, NC, true>, 64, 1, 1);
      return L.nx <= 16 ? go(stencil_pipe_kernel<T, TO, TW, PH, STR, 16, 2, NC, true>, 16, 8, 2)
                        : go(stencil_pipe_kernel<T, TO, TW, PH, STR, 32, 2, NC, true>, 32, 4, 2);
    }
  } else if (L.weighted) {
    return hipErrorInvalidValue;
  }
  // Row copies or register staging.  FP64 on whole 64-wide tiles copies rows (its step
  // in cache-sized groups: 58 us copied, 61 staged, 2 vectors of 256 x 48 x 48; 14
  // orbitals of 128 x 37 x 37 63 and 68; H X of 40 vectors 1057 and 1081).  FP32 is
  // staged (12 vectors of 128 x 40 x 40: 63 us, 67 copied; 40 vectors of 256 x 48 x 48
  // 718 and 722; without an old block 4 vectors 45 and 53), and so is any other nx:
  // 32-wide tiles keep the lanes that 64-wide ones pad away (FP32 product step, 40
  // vectors of 96 x 32 x 32: 66 us, 64-wide staged 100; 75 x 31 x 29: 77 and 98),
  // 16-wide ones only where a 32-wide tile would be half empty.
  constexpr bool copy = sizeof(T) == 8;
  if constexpr (copy) {
    if (L.dma && L.nx % 64 == 0) {
      switch (ty) {
        case 1: return go(stencil_kernel<T, TO, TW, PH, STR, 1, NC>, 64, 1, 1);
        case 2: return go(stencil_kernel<T, TO, TW, PH, STR, 2, NC>, 64, 2, 2);
        case 4: return go(stencil_kernel<T, TO, TW, PH, STR, 4, NC>, 64, 4, 4);
        default: return hipErrorInvalidValue;
      }
    }
  }
  // one row and 64-bit lane offsets where a lane's 32-bit byte offset could overflow
  // (tile rows x nx x 16 bytes)
  const int waves = L.nx > (1 << 22) ? 1 : ty;
  switch (waves) {
    case 1: return go(stencil_pipe_kernel<T, TO, TW, PH, STR, 64, 1, NC>, 64, 1, 1);
    case 2:
      return L.nx <= 16 ? go(stencil_pipe_kernel<T, TO, TW, PH, STR, 16, 2, NC>, 16, 8, 2)
                        : go(stencil_pipe_kernel<T, TO, TW, PH, STR, 32, 2, NC>, 32, 4, 2);
    case 4: return go(stencil_pipe_kernel<T, TO, TW, PH, STR, 32, 4, NC>, 32, 8, 4);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, typename TO, typename TW>
hipError_t launch_ph(const StencilLaunch& L, const StencilConsts<double>& c, hipStream_t s) {
  // 0: no field; 1: Bz = 0 (all link phases uniform over a z-plane); 2: general
  const int ph = L.ptab == nullptr ? 0 : (L.phase_general ? 2 : 1);
  if (L.ncomp == 3) {   // spin-free orbital vectors: zero field only
    if (ph != 0) return hipErrorInvalidValue;
    return L.strain ? launch_t<T, TO, TW, 0, true, 3>(L, c, s)
                    : launch_t<T, TO, TW, 0, false, 3>(L, c, s);
  }
  if (ph == 2)
    return L.strain ? launch_t<T, TO, TW, 2, true>(L, c, s) : launch_t<T, TO, TW, 2, false>(L, c, s);
  if (ph == 1)
    return L.strain ? launch_t<T, TO, TW, 1, true>(L, c, s) : launch_t<T, TO, TW, 1, false>(L, c, s);
  return L.strain ? launch_t<T, TO, TW, 0, true>(L, c, s) : launch_t<T, TO, TW, 0, false>(L, c, s);
}

}  // namespace

int device_cus() {
  static std::atomic<int> known[64];   // per device, 0: not asked yet
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return kCUs;
  }
  int n = known[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    return kCUs;
  }
  known[dev].store(n, std::memory_order_relaxed);
  return n;
}

StencilConsts<double> make_consts(const hkp_material& m, double h, const double B[3]) {
  const double L = m.gamma1 + 4.0 * m.gamma2, M = m.gamma1 - 2.0 * m.gamma2;
  const double Nn = 6.0 * m.gamma3;
  const double eh = kE0 / (h * h);
  StencilConsts<double> c;
  c.cLM = -eh * (L - M);
  c.cM = -eh * M;
  c.czZ = -eh * L;
  c.cN8 = -kE0 * Nn / (8.0 * h * h);
  const double k0 = 2.0 * eh * (L + 2.0 * M);
  const double d3 = m.delta_so_eV / 3.0;
  const double zb = kMuB * B[2];
  c.dgU = k0 + d3 + zb;
  c.dgD = k0 + d3 - zb;
  const double g = kMuB * (3.0 * m.kappa - 1.0);
  c.aUx = g * B[0];
  c.aUy = g * B[1];
  c.aUz = g * B[2] - d3;
  c.aDx = g * B[0];
  c.aDy = g * B[1];
  c.aDz = g * B[2] + d3;
  c.d3 = d3;
  c.bx = kMuB * B[0];
  c.by = kMuB * B[1];
  return c;
}

template <typename T>
StencilConsts<T> cast_consts(const StencilConsts<double>& c) {
  StencilConsts<T> o;
  o.cLM = (T)c.cLM; o.cM = (T)c.cM; o.czZ = (T)c.czZ; o.cN8 = (T)c.cN8;
  o.dgU = (T)c.dgU; o.dgD = (T)c.dgD;
  o.aUx = (T)c.aUx; o.aUy = (T)c.aUy; o.aUz = (T)c.aUz;
  o.aDx = (T)c.aDx; o.aDy = (T)c.aDy; o.aDz = (T)c.aDz;
  o.d3 = (T)c.d3; o.bx = (T)c.bx; o.by = (T)c.by;
  return o;
}
template StencilConsts<double> cast_consts<double>(const StencilConsts<double>&);
template StencilConsts<float> cast_consts<float>(const StencilConsts<double>&);

hipError_t launch_stencil(const StencilLaunch& L, const StencilConsts<double>& c,
                          hipStream_t s) {
  if (L.fp64) {
    if (!L.out_fp64) return hipErrorInvalidValue;
    return L.old ? launch_ph<double, double, double>(L, c, s)
                 : launch_ph<double, void, double>(L, c, s);
  }
  if (!L.old)   // no old block: H X, or a step of the product-form filter
    return L.out_fp64 ? launch_ph<float, void, double>(L, c, s)
                      : launch_ph<float, void, float>(L, c, s);
  // FP32 stencil: old may be FP64 (the first recurrence step reads X) and the
  // output FP64 (the last step feeds the FP64 orthonormalisation)
  if (L.old_fp64) {
    return L.out_fp64 ? launch_ph<float, double, double>(L, c, s)
                      : launch_ph<float, double, float>(L, c, s);
  }
  return L.out_fp64 ? launch_ph<float, float, double>(L, c, s)
                    : launch_ph<float, float, float>(L, c, s);
}

}  // namespace hkp
