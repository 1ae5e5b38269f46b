// Complex helpers and the per-plane arithmetic of the finite-difference hole
// Hamiltonian in the |L S> basis (paper Eq. LK, with the Bir-Pikus, Zeeman and
// Peierls terms of Eq. HNI), shared by the one-step and the two-step stencil
// kernels.  Device code only; included by the stencil sources.
#pragma once

#include "hkp_internal.h"

namespace hkp {
namespace sten {

template <typename T> struct V2;
template <> struct V2<double> { using type = double2; };
template <> struct V2<float> { using type = float2; };

template <typename T>
struct cx {
  T r, i;
};

template <typename T>
__device__ __forceinline__ cx<T> mk(T r, T i) { return cx<T>{r, i}; }
template <typename T>
__device__ __forceinline__ cx<T> add(cx<T> a, cx<T> b) { return {a.r + b.r, a.i + b.i}; }
template <typename T>
__device__ __forceinline__ cx<T> sub(cx<T> a, cx<T> b) { return {a.r - b.r, a.i - b.i}; }
template <typename T>
__device__ __forceinline__ cx<T> scl(T s, cx<T> a) { return {s * a.r, s * a.i}; }
// a + s * b
template <typename T>
__device__ __forceinline__ cx<T> fma_s(cx<T> a, T s, cx<T> b) {
  return {fma(s, b.r, a.r), fma(s, b.i, a.i)};
}
template <typename T>
__device__ __forceinline__ cx<T> mul(cx<T> a, cx<T> b) {
  return {fma(a.r, b.r, -a.i * b.i), fma(a.r, b.i, a.i * b.r)};
}
template <typename T>
__device__ __forceinline__ cx<T> conj(cx<T> a) { return {a.r, -a.i}; }
// i * a
template <typename T>
__device__ __forceinline__ cx<T> mul_i(cx<T> a) { return {-a.i, a.r}; }
// acc + c a + conj(c) b  (c carries a real stencil coefficient times a link phase)
template <typename T>
__device__ __forceinline__ cx<T> wsum_acc(cx<T> acc, cx<T> c, cx<T> a, cx<T> b) {
  cx<T> d = sub(a, b), s = add(a, b);
  return {fma(-c.i, d.i, fma(c.r, s.r, acc.r)), fma(c.i, d.r, fma(c.r, s.i, acc.i))};
}
// acc + c a - conj(c) b
template <typename T>
__device__ __forceinline__ cx<T> wdiff_acc(cx<T> acc, cx<T> c, cx<T> a, cx<T> b) {
  cx<T> d = sub(a, b), s = add(a, b);
  return {fma(-c.i, s.i, fma(c.r, d.r, acc.r)), fma(c.i, s.r, fma(c.r, d.i, acc.i))};
}

template <typename T>
__device__ __forceinline__ cx<T> ld(const T* p) {
  typename V2<T>::type v = *reinterpret_cast<const typename V2<T>::type*>(p);
  return {v.x, v.y};
}
template <typename TW, typename T>
__device__ __forceinline__ void stg(void* base, long long idx, cx<T> v) {
  typename V2<TW>::type o;
  o.x = static_cast<TW>(v.r);
  o.y = static_cast<TW>(v.i);
  reinterpret_cast<typename V2<TW>::type*>(base)[idx] = o;
}

// Streams touched once per launch (the previous iterate, the output) go through
// the cache with the non-temporal policy, so that they do not push the on-site
// fields and the input rows, which later workgroups of the same XCD reuse, out
// of the L2.
typedef float nt_f2 __attribute__((ext_vector_type(2)));
typedef double nt_d2 __attribute__((ext_vector_type(2)));
template <typename T> struct NT2;
template <> struct NT2<float> { using type = nt_f2; };
template <> struct NT2<double> { using type = nt_d2; };
template <typename T>
__device__ __forceinline__ cx<T> ld_stream(const T* p) {
  const typename NT2<T>::type v =
      __builtin_nontemporal_load(reinterpret_cast<const typename NT2<T>::type*>(p));
  return {v.x, v.y};
}
template <typename TW, typename T>
__device__ __forceinline__ void stg_stream(void* base, long long idx, cx<T> v) {
  typename NT2<TW>::type o;
  o.x = static_cast<TW>(v.r);
  o.y = static_cast<TW>(v.i);
  __builtin_nontemporal_store(o, reinterpret_cast<typename NT2<TW>::type*>(base) + idx);
}



// 16 bytes per lane, global -> LDS without registers: lane t's bytes land at
// lds + 16 t (lds is wave-uniform).  The builtin exists only for the device
// pass; the host pass sees an empty body so the kernel's host stub is emitted.
__device__ __forceinline__ void dma16(const void* g, void* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
#endif
}

// Ends the computation of these accumulators here: an empty asm statement that
// takes them as register inputs (it emits nothing), placed before a plane's
// output stores, stops the compiler from sinking this plane's arithmetic past
// the stores.  The stores need the old block, and the wait for it also waits for
// the next plane's copy issued after it; with the arithmetic done first, that
// copy is in flight during all of it.
template <typename T>
__device__ __forceinline__ void settle(const cx<T> (&a)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) asm volatile("" ::"v"(a[i].r), "v"(a[i].i));
}

template <int V>
struct IC {
  static constexpr int value = V;
};

// acc + c a, acc + conj(c) a
template <typename T>
__device__ __forceinline__ cx<T> mac(cx<T> acc, cx<T> c, cx<T> a) {
  return {fma(-c.i, a.i, fma(c.r, a.r, acc.r)), fma(c.i, a.r, fma(c.r, a.i, acc.i))};
}
template <typename T>
__device__ __forceinline__ cx<T> mac_conj(cx<T> acc, cx<T> c, cx<T> a) {
  return {fma(c.i, a.i, fma(c.r, a.r, acc.r)), fma(-c.i, a.r, fma(c.r, a.i, acc.i))};
}

// The link phases of one plane folded with the stencil coefficients (w, v: x- and
// y-link phases; m, 0, p: planes z-1, z, z+1):
//   xo, xa   x faces of the other two orbitals and of |X>:  cM w0, (cLM + cM) w0
//   yo, ya   y faces of the others and of |Y>:              cM v0, (cLM + cM) v0
//   e0..e3   x-y corners: the sum is e0 f++ + conj(e1) f-- + e2 f+- + conj(e3) f-+
//            (f by the signs of dx, dy); uniform phases have e1 = e0, e3 = e2.  With
//            Bz != 0 they are the bare phases and the sum is scaled by cN8: as numbers
//            near 2 their FP32 roundings agree, and cancel between the corners
//   cu, cd   x-z edges pushed to z-1 and z+1:  cN8 (wm + w0), -cN8 (wp + w0)
//   du, dd   y-z edges:                        cN8 (vm + v0), -cN8 (vp + v0)
template <typename T>
struct Fold {
  cx<T> xo, xa, yo, ya, e0, e1, e2, e3, cu, cd, du, dd;
};

template <typename T>
using Const = const __attribute__((address_space(4))) T;   // uniform tables: scalar loads

// The folded phases of plane z from the table (kFoldRow complex entries a plane, in
// the order of Fold; see launch_phase_tables); where Bz != 0 this column's, with u its
// phase along x: those products are formed in double from the double table, so an
// FP32 constant is rounded once.  One scalar load per plane in place of about 40 vector operations
// per wave and plane to fold them (a sixth of the plane's arithmetic).
// (row, row64: the plane's rows of the two tables)
template <typename T, int PH>
__device__ __forceinline__ Fold<T> load_fold(const T* row, const double* row64, cx<double> u) {
  Fold<T> f;
  if constexpr (PH != 0) {
    Const<T>* t = (Const<T>*)row;
    auto at = [&](int i) { return mk<T>(t[2 * i], t[2 * i + 1]); };
    f.xo = at(0);
    f.xa = at(1);
    f.yo = at(2);
    f.ya = at(3);
    f.e0 = at(4);
    f.e1 = at(5);
    f.e2 = at(6);
    f.e3 = at(7);
    f.cu = at(8);
    f.cd = at(9);
    f.du = at(10);
    f.dd = at(11);
    if constexpr (PH == 2) {
      Const<double>* t64 = (Const<double>*)row64;
      auto by = [&](cx<double> ph, int i) {
        const cx<double> r = mul(ph, mk<double>(t64[2 * i], t64[2 * i + 1]));
        return mk<T>((T)r.r, (T)r.i);
      };
      const cx<double> uc = conj(u);
      f.yo = by(u, 2);
      f.ya = by(u, 3);
      f.e0 = by(u, 4);
      f.e1 = by(u, 5);
      f.e2 = by(uc, 6);
      f.e3 = by(uc, 7);
      f.du = by(u, 10);
      f.dd = by(u, 11);
    }
  }
  return f;
}

// Contributions of one input plane z of one spin's three orbital components
// (this thread's column; the plane sits in LDS as [component][row][column] with
// plane stride PLANE and row width W, L pointing at this column's centre) to
// the output planes z-1 (added to acc0), z (added to acc1) and z+1 (written to
// acc2).  X / F: component offsets of this thread's spin and of the other one.
// f: the plane's folded phases (PH != 0; this column's where Bz != 0, PH == 2).
// d..: the on-site orbital block of this column at plane z.  In-plane terms (faces,
// x-y edges, on-site, spin-orbit and Zeeman) go to plane z; the z faces and the
// x-z / y-z edges of the plane are pushed to z-1 and z+1.
template <typename T, int PH, bool STR, int NC, int PLANE, int W>
__device__ __forceinline__ void push_plane(
    const cx<T>* L, int X, int F, const StencilConsts<T>& k, T dgs, T ax, T ay, T az, T sd3,
    T sby, T shift, const Fold<T>& f,
    T d00, T d11, T d22, T d12, T d02, T d01, cx<T> (&acc0)[3], cx<T> (&acc1)[3],
    cx<T> (&acc2)[3]) {
  auto at = [&](int c, int dy, int dx) { return L[c * PLANE + dy * W + dx]; };

  {
    // faces in the plane (this spin's three orbitals); the coefficient of the
    // x faces is (L-M) + M on |X> and M on |Y>, |Z> (y faces: on |Y> and the
    // others), folded with the link phase into one complex constant per plane
    if constexpr (PH != 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        acc1[i] = wsum_acc(acc1[i], i == 0 ? f.xa : f.xo, at(X + i, 0, 1), at(X + i, 0, -1));
        acc1[i] = wsum_acc(acc1[i], i == 1 ? f.ya : f.yo, at(X + i, 1, 0), at(X + i, -1, 0));
      }
    } else {
      const T cLMM = k.cLM + k.cM;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const cx<T> sx = add(at(X + i, 0, 1), at(X + i, 0, -1));
        const cx<T> sy = add(at(X + i, 1, 0), at(X + i, -1, 0));
        acc1[i] = fma_s(acc1[i], i == 0 ? cLMM : k.cM, sx);
        acc1[i] = fma_s(acc1[i], i == 1 ? cLMM : k.cM, sy);
      }
    }
  }
  {
    // x-y edges (in plane): couple X <-> Y
    const cx<T> fY_pp = at(X + 1, 1, 1), fY_pm = at(X + 1, -1, 1);
    const cx<T> fY_mp = at(X + 1, 1, -1), fY_mm = at(X + 1, -1, -1);
    const cx<T> fX_pp = at(X, 1, 1), fX_pm = at(X, -1, 1);
    const cx<T> fX_mp = at(X, 1, -1), fX_mm = at(X, -1, -1);
    if constexpr (PH == 2) {
      const cx<T> eY = mac_conj(mac(mac_conj(mul(f.e0, fY_pp), f.e1, fY_mm), f.e2, fY_pm), f.e3,
                                fY_mp);
      const cx<T> eX = mac_conj(mac(mac_conj(mul(f.e0, fX_pp), f.e1, fX_mm), f.e2, fX_pm), f.e3,
                                fX_mp);
      acc1[0] = fma_s(acc1[0], k.cN8, eY);
      acc1[1] = fma_s(acc1[1], k.cN8, eX);
    } else if constexpr (PH == 1) {
      acc1[0] = wsum_acc(wsum_acc(acc1[0], f.e0, fY_pp, fY_mm), f.e2, fY_pm, fY_mp);
      acc1[1] = wsum_acc(wsum_acc(acc1[1], f.e0, fX_pp, fX_mm), f.e2, fX_pm, fX_mp);
    } else {
      cx<T> eY = sub(add(fY_pp, fY_mm), add(fY_pm, fY_mp));
      cx<T> eX = sub(add(fX_pp, fX_mm), add(fX_pm, fX_mp));
      const T c2 = k.cN8 + k.cN8;
      acc1[0] = fma_s(acc1[0], c2, eY);
      acc1[1] = fma_s(acc1[1], c2, eX);
    }
  }
  {
    const cx<T> oX = at(X, 0, 0), oY = at(X + 1, 0, 0), oZ = at(X + 2, 0, 0);
    // z faces: pushed to z-1 and z+1
    acc0[0] = fma_s(acc0[0], k.cM, oX);
    acc0[1] = fma_s(acc0[1], k.cM, oY);
    acc0[2] = fma_s(acc0[2], k.czZ, oZ);
    acc2[0] = scl(k.cM, oX);
    acc2[1] = scl(k.cM, oY);
    acc2[2] = scl(k.czZ, oZ);
    // x-z and y-z edges of this plane, pushed to z-1 (sz = +1) and z+1 (sz = -1)
    const cx<T> xpZ = at(X + 2, 0, 1), xmZ = at(X + 2, 0, -1);
    const cx<T> xpX = at(X, 0, 1), xmX = at(X, 0, -1);
    const cx<T> ypZ = at(X + 2, 1, 0), ymZ = at(X + 2, -1, 0);
    const cx<T> ypY = at(X + 1, 1, 0), ymY = at(X + 1, -1, 0);
    if constexpr (PH != 0) {
      acc0[0] = wdiff_acc(acc0[0], f.cu, xpZ, xmZ);
      acc0[2] = wdiff_acc(wdiff_acc(acc0[2], f.cu, xpX, xmX), f.du, ypY, ymY);
      acc0[1] = wdiff_acc(acc0[1], f.du, ypZ, ymZ);
      acc2[0] = wdiff_acc(acc2[0], f.cd, xpZ, xmZ);
      acc2[2] = wdiff_acc(wdiff_acc(acc2[2], f.cd, xpX, xmX), f.dd, ypY, ymY);
      acc2[1] = wdiff_acc(acc2[1], f.dd, ypZ, ymZ);
    } else {
      const T c2 = k.cN8 + k.cN8;
      const cx<T> dxZ = sub(xpZ, xmZ), dxX = sub(xpX, xmX);
      const cx<T> dyZ = sub(ypZ, ymZ), dyY = sub(ypY, ymY);
      acc0[0] = fma_s(acc0[0], c2, dxZ);
      acc0[2] = fma_s(acc0[2], c2, add(dxX, dyY));
      acc0[1] = fma_s(acc0[1], c2, dyZ);
      acc2[0] = fma_s(acc2[0], -c2, dxZ);
      acc2[2] = fma_s(acc2[2], -c2, add(dxX, dyY));
      acc2[1] = fma_s(acc2[1], -c2, dyZ);
    }

    // ---- on-site: orbital block (V + strain), constants, SO/Zeeman
    const T dg = dgs - shift;
    cx<T> r0v = scl(d00 + dg, oX), r1v = scl(d11 + dg, oY), r2v = scl(d22 + dg, oZ);
    if constexpr (STR) {
      r0v = fma_s(fma_s(r0v, d01, oY), d02, oZ);
      r1v = fma_s(fma_s(r1v, d01, oX), d12, oZ);
      r2v = fma_s(fma_s(r2v, d02, oX), d12, oY);
    }
    // i (a x u)
    if constexpr (PH != 0) {
      r0v = add(r0v, mul_i(sub(scl(ay, oZ), scl(az, oY))));
      r1v = add(r1v, mul_i(sub(scl(az, oX), scl(ax, oZ))));
      r2v = add(r2v, mul_i(sub(scl(ax, oY), scl(ay, oX))));
    } else {
      r0v = fma_s(r0v, -az, mul_i(oY));
      r1v = fma_s(r1v, az, mul_i(oX));
    }
    // spin flip: up <- -d3 (v_Z, -i v_Z, -v_X + i v_Y) + (bx - i by) v   (v = down)
    //            dn <- -d3 (-v_Z, -i v_Z, v_X + i v_Y) + (bx + i by) v   (v = up)
    // i.e. r_X += s d3 v_Z, r_Y += d3 i v_Z, r_Z += -d3 i v_Y - s d3 v_X with
    // s = -1 (up), +1 (down)
    if constexpr (NC == 6) {   // spin-free vectors have no other spin to couple to
      const cx<T> f0 = at(F, 0, 0), f1 = at(F + 1, 0, 0), f2 = at(F + 2, 0, 0);
      r0v = fma_s(r0v, sd3, f2);
      r1v = fma_s(r1v, k.d3, mul_i(f2));
      r2v = fma_s(fma_s(r2v, -k.d3, mul_i(f1)), -sd3, f0);
      if constexpr (PH != 0) {
        const cx<T> bz = mk<T>(k.bx, sby);
        r0v = add(r0v, mul(bz, f0));
        r1v = add(r1v, mul(bz, f1));
        r2v = add(r2v, mul(bz, f2));
      }
    }
    acc1[0] = add(acc1[0], r0v);
    acc1[1] = add(acc1[1], r1v);
    acc1[2] = add(acc1[2], r2v);
  }
}

}  // namespace sten
}  // namespace hkp
