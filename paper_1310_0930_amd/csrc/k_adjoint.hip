// Hand-written adjoint (vector-Jacobian product) of one gather + Boris push +
// move + split + Esirkepov deposit pass: out of LDS per tile of sorted
// particles, or one thread per particle in global memory.
//
// Given the adjoints of the step's outputs -- lamX^{n+1} (positions, in cell
// units), lamU^{n+1/2} (momenta) and lamJ^{n+1/2} (the current, produced by
// the transpose of the field advance) -- each thread recomputes its particle's
// forward pass from the state at step n and propagates the adjoints back:
// through the charge-conserving deposit (segment end points as functions of
// the path's ends and of the crossing fractions f = (P - X0)/(X1 - X0)),
// the move X1 = X0 + dt u/(gamma dx), the Boris rotation and the gather,
// whose transpose scatters lamE^n, lamB^n (atomics).  The result
// overwrites lamX, lamU with their values at step n and adds to lamE, lamB.
// The map is differentiated along the branch the forward takes (cell and
// piece choices, crossing structure), where it is smooth.
#include "k_particle.h"

namespace pic {

// d w_i / d xi of the order-n weights of one piece.
template <int ORDER, typename R>
__device__ __forceinline__ void shape_deriv(R xi, R* d) {
  if (ORDER == 1) {
    d[0] = R(-1);
    d[1] = R(1);
  } else if (ORDER == 2) {
    d[0] = xi - R(0.5);
    d[1] = R(-2) * xi;
    d[2] = R(0.5) + xi;
  } else if (ORDER == 3) {
    const R s = R(1) - xi;
    d[0] = R(-0.5) * s * s;
    d[1] = xi * (R(1.5) * xi - R(2));
    d[2] = R(0.5) + xi - R(1.5) * xi * xi;
    d[3] = R(0.5) * xi * xi;
  } else {
    const R a = R(1) - R(2) * xi, b = R(1) + R(2) * xi;
    d[0] = R(-1.0 / 48.0) * a * a * a;
    d[1] = R(1.0 / 96.0) * (R(-44) + xi * (R(48) + xi * (R(48) - R(64) * xi)));
    d[2] = xi * (R(-1.25) + xi * xi);
    d[3] = R(1.0 / 96.0) * (R(44) + xi * (R(48) + xi * (R(-48) - R(64) * xi)));
    d[4] = R(1.0 / 48.0) * b * b * b;
  }
}

// Global sample index of component comp (0..2 E/J-like, 3..5 B-like) at
// lattice (x, y, z); -1 outside the domain of an open axis.
template <typename R>
__device__ __forceinline__ int sample_index(const KParams<R>& P, int dims, bool isb, int c, int x,
                                            int y, int z) {
  const int sx = isb ? (c != 0) : (c == 0);
  const int sy = isb ? (c != 1) : (c == 1);
  const int sz = isb ? (c != 2) : (c == 2);
  const int ix = axis_slot(x, P.n[0], P.bc[0] == PIC_BC_OPEN, sx);
  const int iy = axis_slot(y, P.n[1], P.bc[1] == PIC_BC_OPEN, sy);
  const int iz = dims == 3 ? axis_slot(z, P.n[2], P.bc[2] == PIC_BC_OPEN, sz) : 0;
  if (ix < 0 || iy < 0 || iz < 0) return -1;
  return ix + P.n[0] * (iy + P.n[1] * iz);
}

// Sample access of the adjoint helpers.  ref(comp, first) fixes the first
// stencil node of a field component (0..2 E, 3..5 B), at(r, i, j, k) reads the
// field and add(r, i, j, k, v) adds to its adjoint at compile-time offsets from
// it; jref and jat do the same for lamJ.  AdjGlobal goes to the global arrays
// with the domain's wrap and open faces; AdjLds to a tile's LDS regions
// (coordinates relative to the tile origin), the lamE/lamB region accumulating
// in double.
template <int DIMS, typename R>
struct AdjGlobal {
  const KParams<R>& P;
  const DFields<R>& F;
  R* const* lamE;
  R* const* lamB;
  R* const* lamJ;
  struct Ref {
    int comp, x, y, z;
  };
  __device__ __forceinline__ Ref ref(int comp, const int* b) const { return {comp, b[0], b[1], b[2]}; }
  __device__ __forceinline__ int index(const Ref& r, int i, int j, int k) const {
    return sample_index<R>(P, DIMS, r.comp >= 3, r.comp % 3, r.x + i, r.y + j, r.z + k);
  }
  __device__ __forceinline__ R at(const Ref& r, int i, int j, int k) const {
    const int g = index(r, i, j, k);
    return g < 0 ? R(0) : (r.comp >= 3 ? F.B[r.comp - 3] : F.E[r.comp])[g];
  }
  __device__ __forceinline__ void add(const Ref& r, int i, int j, int k, R v) const {
    const int g = index(r, i, j, k);
    if (g >= 0) atomicAdd(&(r.comp >= 3 ? lamB[r.comp - 3] : lamE[r.comp])[g], v);
  }
  __device__ __forceinline__ Ref jref(int comp, const int* b) const { return ref(comp, b); }
  __device__ __forceinline__ R jat(const Ref& r, int i, int j, int k) const {
    const int g = index(r, i, j, k);
    return g < 0 ? R(0) : lamJ[r.comp][g];
  }
};

// Phases of the LDS adjoint.  In 2D one kernel does a particle's whole step
// (PDA_ALL).  In 3D a tile's E/B, lamJ and lamE/lamB (in double) together
// exceed a CU's LDS, and one particle's whole step needs more than 200
// registers, so that a CU held 8 wavefronts and neither its LDS nor its
// arithmetic was half used (96x80x64 quadratic FP32: 1237 us); there PDA_BACK
// goes from the step's outputs back to the adjoints of the interpolated fields
// (E/B and lamJ in LDS; 262 us, the VALU 73 % busy) and leaves those six values
// in scratch, and PDA_GATHER transposes the gather (E/B and lamE/lamB in LDS;
// 535 us, the LDS 69 % busy: 162 double adds of at least 8 LDS cycles per
// 64 particles; as 64-bit integers on one scale per tile the adds took 395 us,
// but a tile's small adjoints lost their digits beside its large ones, at 1e-14
// of them half of their value).
enum { PDA_ALL = 0, PDA_BACK = 1, PDA_GATHER = 2 };

// Region of one workgroup of the LDS adjoint: the push tile, cut along z
// into S slabs when the phase's regions (E/B and lamJ in the working
// precision, lamE/lamB in double) of a whole 3D tile exceed a CU's LDS.
// Each slab keeps the tile's drift allowance and stencil reach; x and y are
// the tile's.
template <int DIMS, int ORDER, typename R, int PHASE, int NT2>
struct AdjGeo : Geo<DIMS, ORDER, R> {
  using B = Geo<DIMS, ORDER, R>;
  using Rc = typename B::Rc;
  static constexpr bool has_lj = PHASE != PDA_GATHER, has_leb = PHASE != PDA_BACK;
  // padded: the field region's rows and planes are the push's, which the sort
  // spreads the lanes by; else they are dense
  static constexpr size_t bytes(int tz, bool padded) {
    const int nz = DIMS == 3 ? tz + 2 * B::AZ + Rc::g_hi - Rc::g_lo : 1;
    const int mz = DIMS == 3 ? tz + 2 * B::AZ + Rc::d_hi - Rc::d_lo : 1;
    return (sizeof(R) * 6 + (has_leb ? sizeof(double) * 6 : 0)) *
               (size_t)((padded ? B::ep : B::ex * B::ex) * nz) +
           (has_lj ? sizeof(R) * 3 * (size_t)(B::jx * B::jx * mz) : 0);
  }
  static constexpr size_t LDS_MAX = 160 * 1024;
  // the gather's transpose needs few registers: 16 wavefronts in FP32
  static constexpr int NT = DIMS == 2 ? NT2 : PHASE == PDA_GATHER && sizeof(R) == 4 ? 1024 : 512;
  // wavefronts per SIMD to keep registers for: up to quadratic order in FP32
  // two workgroups of PDA_BACK share a CU (in 2D, where there are 512 tiles for
  // 256 CUs, the spills cost more: 512x256 quadratic FP32 138 against 129 us)
  static constexpr int WPE = PHASE == PDA_BACK && sizeof(R) == 4 && ORDER <= 2 ? 4 : 1;
  // with several slabs each wavefront queues the particles of its slab:
  // 128 indices per wavefront
  static constexpr int QCAP = 128;
  static constexpr size_t queue_bytes = sizeof(int) * QCAP * (NT / 64);
  static constexpr int pick(bool padded) {
    if (DIMS == 2) return 1;
    for (int s = 1; s <= B::TZ; s *= 2)
      if (B::TZ % s == 0 && bytes(B::TZ / s, padded) + (s > 1 ? queue_bytes : 0) <= LDS_MAX) return s;
    return 0;
  }
  static constexpr bool fits = pick(false) > 0;
  static constexpr int S = fits ? pick(false) : 1;
  // workgroups whose regions share a CU's LDS
  static constexpr size_t per_cu(bool padded) {
    return LDS_MAX / (bytes(B::TZ / S, padded) + (S > 1 ? queue_bytes : 0) + 64);
  }
  // padded where that costs no slab and no workgroup on a CU (2D linear FP32,
  // 512x256 at 16 per cell: 87 -> 81 us)
  static constexpr bool pad = pick(true) == S && per_cu(true) == per_cu(false);
  static constexpr int TZ = B::TZ / S;
  static constexpr int ez = DIMS == 3 ? TZ + 2 * B::AZ + Rc::g_hi - Rc::g_lo : 1;
  static constexpr int es = pad ? B::es : B::ex, ep = pad ? B::ep : B::ex * B::ex;
  static constexpr int e_vol = ep * ez, e_cnt = B::ex * B::ex * ez;
  static constexpr int jz = DIMS == 3 ? TZ + 2 * B::AZ + Rc::d_hi - Rc::d_lo : 1;
  static constexpr int j_vol = B::jx * B::jx * jz;
};

template <int DIMS, int ORDER, typename R, class G>
struct AdjLds {
  lds_ptr<const R> eb;   // E^n (0..2), B^n (3..5) over the field region
  lds_ptr<const R> lj;   // lamJ over the current region
  lds_ptr<double> leb;   // lamE (0..2), lamB (3..5) over the field region
  struct Ref {
    lds_ptr<const R> f;
    lds_ptr<double> l;
  };
  template <typename T>
  static __device__ __forceinline__ lds_ptr<T> pin(lds_ptr<T> p) {
    uint32_t a = (uint32_t)(uintptr_t)p;
    asm volatile("" : "+v"(a));
    return (lds_ptr<T>)(uintptr_t)a;
  }
  // one register per array, so that every access is an immediate offset
  __device__ __forceinline__ Ref ref(int comp, const int* b) const {
    const int i = (DIMS == 3 ? (b[2] - G::e_lo_z) * G::ep : 0) + (b[1] - G::e_lo) * G::es +
                  (b[0] - G::e_lo) + comp * G::e_vol;
    return {pin<const R>(eb + i), pin<double>(leb + i)};
  }
  // single reads, as in the push's gather
  __device__ __forceinline__ R at(const Ref& r, int i, int j, int k) const {
    using vptr = __attribute__((address_space(3))) const volatile R*;
    return ((vptr)r.f)[k * G::ep + j * G::es + i];
  }
  __device__ __forceinline__ void add(const Ref& r, int i, int j, int k, R v) const {
    __hip_atomic_fetch_add(&r.l[k * G::ep + j * G::es + i], (double)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ lds_ptr<const R> jref(int comp, const int* b) const {
    return pin<const R>(lj + (DIMS == 3 ? (b[2] - G::j_lo_z) * G::jx * G::jx : 0) +
                        (b[1] - G::j_lo) * G::jx + (b[0] - G::j_lo) + comp * G::j_vol);
  }
  __device__ __forceinline__ R jat(lds_ptr<const R> r, int i, int j, int k) const {
    using vptr = __attribute__((address_space(3))) const volatile R*;
    return ((vptr)r)[(k * G::jx + j) * G::jx + i];
  }
};

// Transpose of the gather of component COMP, whose weights and their
// derivatives per axis are w and dw, from its first stencil node: every node's
// adjoint receives w lam, and lX the derivative of the interpolated value times
// lam.  The sums over the stencil are nested (x, then y, then z), two products
// per sample.  A plane's samples are read before anything is added: the LDS
// answers in order, and a read behind an add waits for it (3D cubic FP32 in one
// kernel, 24x16x20: 293 -> 228 us).
template <int DIMS, int ORDER, typename R, class Acc>
__device__ __forceinline__ void gather_vjp_comp(const Acc& ac, int comp, const int* first,
                                                const R (*w)[ORDER + 1], const R (*dw)[ORDER + 1],
                                                R lam, R* lX) {
  constexpr int M = ORDER + 1;
  constexpr int MZ = DIMS == 3 ? M : 1;
  const auto r = ac.ref(comp, first);
  R g[3] = {R(0), R(0), R(0)};
#pragma unroll
  for (int k = 0; k < MZ; ++k) {
    R s = R(0), dy = R(0), dx = R(0);
    const R lz = DIMS == 3 ? w[2][k] * lam : lam;
    R fp[M][M];
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
      for (int i = 0; i < M; ++i) fp[j][i] = ac.at(r, i, j, k);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      R sx = R(0), dxx = R(0);
      const R lyz = w[1][j] * lz;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const R f = fp[j][i];
        sx += w[0][i] * f;
        dxx += dw[0][i] * f;
        ac.add(r, i, j, k, w[0][i] * lyz);
      }
      s += w[1][j] * sx;
      dy += dw[1][j] * sx;
      dx += w[1][j] * dxx;
    }
    g[0] += (DIMS == 3 ? w[2][k] : R(1)) * dx;
    g[1] += (DIMS == 3 ? w[2][k] : R(1)) * dy;
    if (DIMS == 3) g[2] += dw[2][k] * s;
  }
#pragma unroll
  for (int d = 0; d < DIMS; ++d) lX[d] += lam * g[d];
}

// Transpose of the gather over the six components.
template <int DIMS, int ORDER, typename R, class Acc>
__device__ __forceinline__ void gather_vjp(const Acc& ac, const int* c3, const R* o, const R* lEp,
                                           const R* lBp, R* lX) {
  constexpr int M = ORDER + 1;
  R wn[3][M], ws[3][M], dn[3][M], dsg[3][M];
  int bn[3] = {c3[0], c3[1], c3[2]}, bs[3] = {c3[0], c3[1], c3[2]};
#pragma unroll
  for (int d = 0; d < DIMS; ++d) {
    R xi;
    bn[d] += piece_node<ORDER>(o[d], xi) - ORDER / 2;
    shape<ORDER>(xi, wn[d]);
    shape_deriv<ORDER>(xi, dn[d]);
    bs[d] += piece_stag<ORDER>(o[d], xi) - ORDER / 2;
    shape<ORDER>(xi, ws[d]);
    shape_deriv<ORDER>(xi, dsg[d]);
  }
  auto one = [&](auto comp_c) {
    constexpr int comp = decltype(comp_c)::value;
    constexpr bool isb = comp >= 3;
    constexpr int c = isb ? comp - 3 : comp;
    R w[3][M], dw[3][M];
    int first[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {  // staggered along c (E_c), along the two others (B_c)
      const bool st = isb ? (d != c) : (d == c);
#pragma unroll
      for (int i = 0; i < M; ++i) {
        if (d >= DIMS) continue;
        w[d][i] = st ? ws[d][i] : wn[d][i];
        dw[d][i] = st ? dsg[d][i] : dn[d][i];
      }
      first[d] = st ? bs[d] : bn[d];
    }
    gather_vjp_comp<DIMS, ORDER, R>(ac, comp, first, w, dw, isb ? lBp[c] : lEp[c], lX);
  };
  one(std::integral_constant<int, 0>{});
  one(std::integral_constant<int, 1>{});
  one(std::integral_constant<int, 2>{});
  one(std::integral_constant<int, 3>{});
  one(std::integral_constant<int, 4>{});
  one(std::integral_constant<int, 5>{});
}

// Transpose of the Boris step u -> u' under (Ep, Bp), recomputing its
// intermediates: in lamU' ; out lamU, lamEp, lamBp.
template <typename R>
__device__ __forceinline__ void boris_vjp(R hqm, const R* u, const R* E, const R* B, const R* lu1,
                                          R* lu, R* lE, R* lB) {
  R um[3], t[3], s[3], up[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) um[c] = u[c] + hqm * E[c];
  const R gm = sqrt(R(1) + um[0] * um[0] + um[1] * um[1] + um[2] * um[2]);
  const R hg = hqm / gm;
#pragma unroll
  for (int c = 0; c < 3; ++c) t[c] = hg * B[c];
  const R tt = t[0] * t[0] + t[1] * t[1] + t[2] * t[2];
  const R f = R(2) / (R(1) + tt);
#pragma unroll
  for (int c = 0; c < 3; ++c) s[c] = f * t[c];
  up[0] = um[0] + (um[1] * t[2] - um[2] * t[1]);
  up[1] = um[1] + (um[2] * t[0] - um[0] * t[2]);
  up[2] = um[2] + (um[0] * t[1] - um[1] * t[0]);
  // u' = uq + hqm E, uq = um + up x s
  R luq[3], lum[3], lup[3], ls[3], lt[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    luq[c] = lu1[c];
    lE[c] = hqm * lu1[c];
    lum[c] = luq[c];
  }
  // c = a x b: lam_a = b x lam_c, lam_b = lam_c x a
  lup[0] = s[1] * luq[2] - s[2] * luq[1];
  lup[1] = s[2] * luq[0] - s[0] * luq[2];
  lup[2] = s[0] * luq[1] - s[1] * luq[0];
  ls[0] = luq[1] * up[2] - luq[2] * up[1];
  ls[1] = luq[2] * up[0] - luq[0] * up[2];
  ls[2] = luq[0] * up[1] - luq[1] * up[0];
  // up = um + um x t
#pragma unroll
  for (int c = 0; c < 3; ++c) lum[c] += lup[c];
  lum[0] += t[1] * lup[2] - t[2] * lup[1];
  lum[1] += t[2] * lup[0] - t[0] * lup[2];
  lum[2] += t[0] * lup[1] - t[1] * lup[0];
  lt[0] = lup[1] * um[2] - lup[2] * um[1];
  lt[1] = lup[2] * um[0] - lup[0] * um[2];
  lt[2] = lup[0] * um[1] - lup[1] * um[0];
  // s = f t, f = 2/(1 + t.t)
  const R lf = ls[0] * t[0] + ls[1] * t[1] + ls[2] * t[2];
  const R ltt = R(-0.5) * f * f * lf;
#pragma unroll
  for (int c = 0; c < 3; ++c) lt[c] += f * ls[c] + R(2) * t[c] * ltt;
  // t = (hqm/gm) B
  R bl = R(0);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lB[c] = hg * lt[c];
    bl += B[c] * lt[c];
  }
  const R lgm = -hg / gm * bl;
  // gm = sqrt(1 + um.um); um = u + hqm E
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lum[c] += um[c] / gm * lgm;
    lu[c] = lum[c];
    lE[c] += hqm * lum[c];
  }
}

// Transpose of the Esirkepov deposit of one segment: gathers lamJ over the
// segment's stencil and returns lam(xa), lam(xb) per axis and lam(fz).
template <int DIMS, int ORDER, typename R, class Acc>
__device__ __forceinline__ void deposit_segment_vjp(const KParams<R>& P, const Acc& ac,
                                                    const int* c3, const int* base, const R* xa,
                                                    const R* xb, R q, R fz, R* lxa, R* lxb,
                                                    R& lfz) {
  constexpr int M = ORDER + 1;
  constexpr R twelfth = R(1.0 / 12.0);
  // mean weights Sm = S0 + dS/2 and differences dS; the transverse factor is
  // A = Sm_a Sm_b + dS_a dS_b / 12
  R Sm[DIMS][M], dS[DIMS][M], lSm[DIMS][M], ldS[DIMS][M];
#pragma unroll
  for (int d = 0; d < DIMS; ++d) {
    shape<ORDER>(xa[d], Sm[d]);
    dshape<ORDER>(xa[d], xb[d], dS[d]);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      Sm[d][i] += R(0.5) * dS[d][i];
      lSm[d][i] = ldS[d][i] = R(0);
    }
  }
  const int first[3] = {c3[0] + base[0], c3[1] + base[1], c3[2] + base[2]};
  lfz = R(0);
#pragma unroll
  for (int c = 0; c < DIMS; ++c) {
    const int a = (c + 1) % DIMS, b = DIMS == 3 ? (c + 2) % 3 : a;
    const R qj = q * P.jfac[c];
    R Pc[ORDER], lP[ORDER];
    R run = R(0);
#pragma unroll
    for (int i = 0; i < ORDER; ++i) {
      run += dS[c][i];
      Pc[i] = qj * run;
      lP[i] = R(0);
    }
    const auto r = ac.jref(c, first);
#pragma unroll
    for (int ib = 0; ib < (DIMS == 3 ? M : 1); ++ib) {
      const R sb = DIMS == 3 ? Sm[b][ib] : R(1);
      const R db = DIMS == 3 ? twelfth * dS[b][ib] : R(0);
      R ls = R(0), ld = R(0);  // sums over ia for axis b
#pragma unroll
      for (int ia = 0; ia < M; ++ia) {
        const R A = DIMS == 3 ? Sm[a][ia] * sb + dS[a][ia] * db : Sm[a][ia];
        R lA = R(0);
#pragma unroll
        for (int ic = 0; ic < ORDER; ++ic) {
          int L[3] = {0, 0, 0};
          L[c] = ic;
          L[a] = ia;
          if (DIMS == 3) L[b] = ib;
          const R g = ac.jat(r, L[0], L[1], L[2]);
          lA += g * Pc[ic];
          lP[ic] += g * A;
        }
        lSm[a][ia] += lA * sb;
        if (DIMS == 3) {
          ldS[a][ia] += lA * db;
          ls += lA * Sm[a][ia];
          ld += lA * dS[a][ia];
        }
      }
      if (DIMS == 3) {
        lSm[b][ib] += ls;
        ldS[b][ib] += twelfth * ld;
      }
    }
    // P_c[ic] = qj * sum_{i <= ic} dS_c[i]
    R acc = R(0);
#pragma unroll
    for (int i = ORDER - 1; i >= 0; --i) {
      acc += lP[i];
      ldS[c][i] += qj * acc;
    }
  }
  if (DIMS == 2) {  // the out-of-plane current
    const auto r = ac.jref(2, first);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      const R dj = twelfth * dS[1][j];
      R ls = R(0), ld = R(0);
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const R g = ac.jat(r, i, j, 0);
        lfz += g * (Sm[0][i] * Sm[1][j] + dS[0][i] * dj);
        const R gf = g * fz;
        lSm[0][i] += gf * Sm[1][j];
        ldS[0][i] += gf * dj;
        ls += gf * Sm[0][i];
        ld += gf * dS[0][i];
      }
      lSm[1][j] += ls;
      ldS[1][j] += twelfth * ld;
    }
  }
  // Sm = S(xa) + dS/2, dS = S(xb) - S(xa)
#pragma unroll
  for (int d = 0; d < DIMS; ++d) {
    R da[M], db[M];
    shape_deriv<ORDER>(xa[d], da);
    shape_deriv<ORDER>(xb[d], db);
    R la = R(0), lb = R(0);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const R l = ldS[d][i] + R(0.5) * lSm[d][i];
      la += (lSm[d][i] - l) * da[i];
      lb += l * db[i];
    }
    lxa[d] = la;
    lxb[d] = lb;
  }
}

// Transpose of the whole split deposit: lamX0, lamX1 (cell units, relative
// to the old cell) and lam(vz) for the 2D out-of-plane current.
template <int DIMS, int ORDER, typename R, class Acc>
__device__ __forceinline__ void deposit_vjp(const KParams<R>& P, const Acc& ac, const int* c3,
                                            const R* o0, const int* sh, const R* o1, R q, R vz,
                                            R* lX0, R* lX1, R& lvz) {
  Split<DIMS, R> S;
  split_path<DIMS, ORDER, R>(S, o0, sh, o1);
  R lt[DIMS + 2];
#pragma unroll
  for (int j = 0; j < DIMS + 2; ++j) lt[j] = R(0);
  lvz = R(0);
  for (int s = 0; s <= S.m; ++s) {
    R xa[3], xb[3], ft, lxa[3], lxb[3], lfz;
    int base[3];
    segment_ends<DIMS, ORDER, R>(S, s, xa, xb, base, ft);
    deposit_segment_vjp<DIMS, ORDER, R>(P, ac, c3, base, xa, xb, q, q * vz * ft, lxa, lxb, lfz);
    R ta = R(0), tbb = R(1);
#pragma unroll
    for (int j = 0; j < DIMS + 2; ++j) {
      if (j == s) ta = S.tb[j];
      if (j == s + 1) tbb = S.tb[j];
    }
    // xa = X0 + ta (X1 - X0), xb = X0 + tb (X1 - X0) (up to the piece shift)
    R la = R(0), lb = R(0);
#pragma unroll
    for (int d = 0; d < DIMS; ++d) {
      lX0[d] += lxa[d] * (R(1) - ta) + lxb[d] * (R(1) - tbb);
      lX1[d] += lxa[d] * ta + lxb[d] * tbb;
      la += lxa[d] * S.dl[d];
      lb += lxb[d] * S.dl[d];
    }
    // fz = q vz (tb - ta)
    lvz += lfz * q * (tbb - ta);
    la -= lfz * q * vz;
    lb += lfz * q * vz;
#pragma unroll
    for (int j = 0; j < DIMS + 2; ++j) {
      if (j == s) lt[j] += la;
      if (j == s + 1) lt[j] += lb;
    }
  }
  // crossing fractions f_d = (P_d - X0_d)/(X1_d - X0_d)
#pragma unroll
  for (int d = 0; d < DIMS; ++d) {
    if (!S.cr[d]) continue;
    R l = R(0), f = R(0);
#pragma unroll
    for (int j = 1; j <= DIMS; ++j)
      if (j == S.jd[d]) {
        l = lt[j];
        f = S.tb[j];
      }
    lX0[d] += l * (f - R(1)) / S.dl[d];
    lX1[d] += l * (-f) / S.dl[d];
  }
}

// Forward pass of one particle kept for its adjoint: the gather, the Boris
// push and the move (state s becomes step n+1's, u0 keeps u^{n-1/2}).
template <typename R>
struct FwdPart {
  R Ep[3], Bp[3], u0[3], o1[3], vz;
  int sh[3];
  bool small;
};

template <int DIMS, int ORDER, typename R, class FAcc>
__device__ __forceinline__ bool forward_part(const KParams<R>& P, const FAcc& acc, PState<R>& s,
                                             FwdPart<R>& f, DevFlags* flg) {
  gather<DIMS, ORDER, R>(acc, s.o, f.Ep, f.Bp);
#pragma unroll
  for (int c = 0; c < 3; ++c) f.u0[c] = s.u[c];
  return push_move<DIMS, R>(P, s, f.Ep, f.Bp, f.sh, f.o1, f.vz, f.small, flg);
}

// Adjoint of one particle's step from its forward pass, as far back as the
// interpolated fields; c3 are the cell's coordinates in the accessor's frame.
// Reads lam at slot p (adjoints of x^{n+1}, u^{n+1/2}); gives lX0 (the adjoint
// of x^n without the gather's part), lu0 (of u^{n-1/2}), lEp and lBp.
template <int DIMS, int ORDER, typename R, class Acc>
__device__ __forceinline__ void adjoint_back(const KParams<R>& P, const Acc& ac, const int* c3,
                                             const PState<R>& s0, const PState<R>& s1,
                                             const FwdPart<R>& f, const DParts<R>& lam, int p,
                                             R* lX0, R* lu0, R* lEp, R* lBp) {
  const R u1[3] = {s1.u[0], s1.u[1], s1.u[2]};
  const R gam = sqrt(R(1) + u1[0] * u1[0] + u1[1] * u1[1] + u1[2] * u1[2]);
  // adjoints arriving from step n+1
  R lX1[3] = {R(0), R(0), R(0)}, lu1[3];
  lX0[0] = lX0[1] = lX0[2] = R(0);
#pragma unroll
  for (int d = 0; d < DIMS; ++d) lX1[d] = lam.off[d][p];
#pragma unroll
  for (int c = 0; c < 3; ++c) lu1[c] = lam.u[c][p];
  // deposit
  R lvz;
  deposit_vjp<DIMS, ORDER, R>(P, ac, c3, s0.o, f.sh, f.o1, s0.q, f.vz, lX0, lX1, lvz);
  // move: X1 = X0 + dt/dx u/gamma, vz = u_z/gamma
  R ld[3] = {R(0), R(0), R(0)};
  R dot = R(0);
#pragma unroll
  for (int d = 0; d < DIMS; ++d) {
    lX0[d] += lX1[d];
    ld[d] = lX1[d] * P.dtdx[d];
    dot += ld[d] * u1[d];
  }
  dot += lvz * u1[2];
  const R ig = R(1) / gam, ig3 = ig * ig * ig;
#pragma unroll
  for (int c = 0; c < 3; ++c) lu1[c] += (ld[c] + (c == 2 ? lvz : R(0))) * ig - u1[c] * ig3 * dot;
  // Boris
  boris_vjp<R>(P.hqm, f.u0, f.Ep, f.Bp, lu1, lu0, lEp, lBp);
}

// The whole step: overwrites lam at slot p with the adjoints of x^n, u^{n-1/2}.
template <int DIMS, int ORDER, typename R, class Acc>
__device__ __forceinline__ void adjoint_part(const KParams<R>& P, const Acc& ac, const int* c3,
                                             const PState<R>& s0, const PState<R>& s1,
                                             const FwdPart<R>& f, const DParts<R>& lam, int p) {
  R lX0[3], lu0[3], lEp[3], lBp[3];
  adjoint_back<DIMS, ORDER, R>(P, ac, c3, s0, s1, f, lam, p, lX0, lu0, lEp, lBp);
  gather_vjp<DIMS, ORDER, R>(ac, c3, s0.o, lEp, lBp, lX0);
#pragma unroll
  for (int d = 0; d < DIMS; ++d) lam.off[d][p] = lX0[d];
#pragma unroll
  for (int c = 0; c < 3; ++c) lam.u[c][p] = lu0[c];
}

// One thread per particle, everything in global memory: all particles, or
// (list != NULL) the flg->ndefer particles of the list followed by those
// from *tail on (the particles no tile covers).
template <int DIMS, int ORDER, typename R>
__global__ void __launch_bounds__(256) k_push_deposit_adjoint(KParams<R> P, DParts<R> pa,
                                                              DFields<R> F, DFields<R> L,
                                                              DParts<R> lam, DevFlags* flg,
                                                              int np, const int* list,
                                                              const int* tail) {
  const int open0 = P.bc[0] == PIC_BC_OPEN, open1 = P.bc[1] == PIC_BC_OPEN;
  const int open2 = DIMS == 3 && P.bc[2] == PIC_BC_OPEN;
  const int nl = list ? (int)flg->ndefer : 0;
  const int t0 = list ? *tail : 0;
  const int n = nl + (np - t0);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
    const int p = t < nl ? list[t] : t0 + (t - nl);
    PState<R> s = load_particle<DIMS, R>(pa, p, P.q_const);
    if (s.cl < 0) continue;
    int c3[3];
    if (!decode<DIMS, R>(P, s, c3, flg)) continue;
    GlobalFields<R> acc{F.E, F.B, c3[0], c3[1], c3[2], P.n[0], P.n[1], P.n[2],
                        open0, open1, open2, DIMS};
    const PState<R> s0 = s;
    FwdPart<R> f;
    if (!forward_part<DIMS, ORDER, R>(P, acc, s, f, flg)) continue;
    AdjGlobal<DIMS, R> ac{P, F, L.E, L.B, L.J};
    adjoint_part<DIMS, ORDER, R>(P, ac, c3, s0, s, f, lam, p);
  }
}

// The same out of LDS, one workgroup per tile of sorted particles, or per z
// slab of one (AdjGeo): the phase's regions are staged, lamE/lamB accumulate in
// double in LDS and are added to the global arrays once.  Every slab reads all
// of its tile's particles and takes those whose cell is in the slab, the first
// and last slabs also the allowance below and above the tile.  Particles
// outside the tile's drift allowance, or moving half a cell or more, go to the
// list for the global-memory kernel (entered by PDA_ALL or PDA_BACK, which has
// one slab); PDA_BACK leaves zeros in `lam_eb` (6 arrays of np) for the ones
// that moved too far or became non-finite, and PDA_GATHER skips zeros.
template <int DIMS, int ORDER, typename R, int PHASE, int NT2>
__global__ void __launch_bounds__((AdjGeo<DIMS, ORDER, R, PHASE, NT2>::NT),
                                  (AdjGeo<DIMS, ORDER, R, PHASE, NT2>::WPE)) k_pda_tile(
    KParams<R> P, DParts<R> pa, DFields<R> F, DFields<R> L, DParts<R> lam, R* __restrict__ lam_eb,
    long np, const int* __restrict__ starts, int* __restrict__ deferred, DevFlags* flg) {
  using G = AdjGeo<DIMS, ORDER, R, PHASE, NT2>;
  static_assert(G::fits, "one-cell slabs fit");
  constexpr int S = G::S;
  __shared__ R s_eb[6 * G::e_vol];
  __shared__ R s_lj[G::has_lj ? 3 * G::j_vol : 1];
  __shared__ double s_leb[G::has_leb ? 6 * G::e_vol : 1];
  const int grp = blockIdx.x >> 3;
  const int tile = (blockIdx.x & 7) * P.per_xcd + grp / S;
  const int slab = grp % S;
  if (tile >= P.ntiles) return;
  const int pbeg = starts[tile], pend = starts[tile + 1];
  if (pbeg == pend) return;
  int org[3];
  tile_origin<DIMS, ORDER, R>(P, tile, org);
  const int tor[3] = {org[0], org[1], org[2]};
  org[2] += slab * G::TZ;
  const int open0 = P.bc[0] == PIC_BC_OPEN, open1 = P.bc[1] == PIC_BC_OPEN;
  const int open2 = DIMS == 3 && P.bc[2] == PIC_BC_OPEN;
  const int str1 = P.n[0], str2 = P.n[0] * P.n[1];
  {
    constexpr int NR = (G::e_cnt + G::NT - 1) / G::NT;
    R stage[NR][6];
    stage_load<DIMS, ORDER, R, NR, G>(P, F, org, stage, (int)threadIdx.x, G::NT);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int r = threadIdx.x + k * G::NT;
      if (r < G::e_cnt) {
        const int e = r / (G::ex * G::ex) * G::ep + (r / G::ex) % G::ex * G::es + r % G::ex;
#pragma unroll
        for (int c = 0; c < 6; ++c) s_eb[c * G::e_vol + e] = stage[k][c];
      }
    }
  }
  if constexpr (G::has_lj) {
    for (int r = threadIdx.x; r < G::j_vol; r += G::NT) {  // lamJ_c, staggered along c
      const int lx = r % G::jx, ly = (r / G::jx) % G::jx, lz = r / (G::jx * G::jx);
      int sx[2], sy[2], sz[2] = {0, 0};
      axis_slots(org[0] + G::j_lo + lx, P.n[0], open0, 1, sx);
      axis_slots(org[1] + G::j_lo + ly, P.n[1], open1, str1, sy);
      if (DIMS == 3) axis_slots(org[2] + G::j_lo_z + lz, P.n[2], open2, str2, sz);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int ix = sx[c == 0], iy = sy[c == 1], iz = sz[c == 2];
        s_lj[c * G::j_vol + r] = (ix >= 0 && iy >= 0 && iz >= 0) ? L.J[c][ix + iy + iz] : R(0);
      }
    }
  }
  if constexpr (G::has_leb)
    for (int i = threadIdx.x; i < 6 * G::e_vol; i += G::NT) s_leb[i] = 0.0;
  __syncthreads();
  const AdjLds<DIMS, ORDER, R, G> ac{(lds_ptr<const R>)s_eb, (lds_ptr<const R>)s_lj,
                                     (lds_ptr<double>)s_leb};
  // the cell relative to the tile (periodic fold); false outside the tile's
  // drift allowance
  auto locate = [&](const int* c3, int* l) {
    bool fast = true;
#pragma unroll
    for (int d = 0; d < DIMS; ++d) {
      const int Td = d == 2 ? G::B::TZ : G::T;
      const int Ad = d == 2 ? G::AZ : G::A;
      int v = c3[d] - tor[d];
      if (P.bc[d] == PIC_BC_PERIODIC) {
        v = v < 0 ? v + P.n[d] : v;
        if (v >= Td + Ad) v -= P.n[d];
      }
      l[d] = v;
      fast = fast && v >= -Ad && v < Td + Ad;
    }
    return fast;
  };
  auto defer = [&](int p) { deferred[atomicAdd(&flg->ndefer, 1u)] = p; };
  // one particle whose cell l (relative to the slab) is in the region
  auto work = [&](int p, const PState<R>& s0, const int* l) {
    if constexpr (PHASE == PDA_GATHER) {
      R v[6];
      bool any = false;
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        v[c] = lam_eb[c * np + p];
        any = any || v[c] != R(0);  // (also for NaN)
      }
      if (!any) return;
      R lX[3] = {R(0), R(0), R(0)};
      gather_vjp<DIMS, ORDER, R>(ac, l, s0.o, v, v + 3, lX);
#pragma unroll
      for (int d = 0; d < DIMS; ++d) lam.off[d][p] += lX[d];
    } else {
      const LdsFields<DIMS, ORDER, R, G> acc{
          (lds_ptr<const R>)s_eb,
          (l[2] - G::e_lo_z) * G::ep + (l[1] - G::e_lo) * G::es + (l[0] - G::e_lo)};
      PState<R> s = s0;
      FwdPart<R> f;
      bool ok = forward_part<DIMS, ORDER, R>(P, acc, s, f, flg);
      if (ok && !f.small) {
        defer(p);
        ok = false;
      }
      if constexpr (PHASE == PDA_ALL) {
        if (ok) adjoint_part<DIMS, ORDER, R>(P, ac, l, s0, s, f, lam, p);
      } else {
        R lX0[3], lu0[3], v[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
        if (ok) {
          adjoint_back<DIMS, ORDER, R>(P, ac, l, s0, s, f, lam, p, lX0, lu0, v, v + 3);
#pragma unroll
          for (int d = 0; d < DIMS; ++d) lam.off[d][p] = lX0[d];
#pragma unroll
          for (int c = 0; c < 3; ++c) lam.u[c][p] = lu0[c];
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) lam_eb[c * np + p] = v[c];
      }
    }
  };
  if constexpr (S == 1) {
    for (int p = pbeg + threadIdx.x; p < pend; p += G::NT) {
      const PState<R> s = load_particle<DIMS, R>(pa, p, P.q_const);
      if (s.cl < 0) continue;
      int c3[3] = {0, 0, 0}, l[3] = {0, 0, 0};
      if (!decode<DIMS, R>(P, s, c3, flg)) continue;
      if (locate(c3, l))
        work(p, s, l);
      else if (PHASE != PDA_GATHER)
        defer(p);
    }
  } else {
    static_assert(PHASE != PDA_BACK, "particles are deferred once");
    // Every slab scans all of the tile's particles, a slab's share is about
    // 1/S of them: each wavefront queues the indices of its slab's particles
    // (allowance cells below and above the tile go to the end slabs) and
    // runs whole 64-lane batches from the queue's end (at most 63 wait when
    // 64 more arrive, so 128 entries suffice).
    __shared__ int s_own[G::NT / 64][G::QCAP];
    const int lane = threadIdx.x & 63;
    int* q = s_own[threadIdx.x >> 6];
    int qn = 0;  // uniform over the wavefront
    for (int b = pbeg + (threadIdx.x & ~63);; b += G::NT) {
      const bool more = b < pend;
      if (more) {
        const int p = b + lane;
        bool own = false;
        if (p < pend) {
          const PState<R> s = load_particle<DIMS, R>(pa, p, P.q_const);
          int c3[3] = {0, 0, 0}, l[3] = {0, 0, 0};
          if (s.cl >= 0 && decode<DIMS, R>(P, s, c3, flg)) {
            if (locate(c3, l))
              own = (l[2] < 0 ? 0 : (l[2] / G::TZ < S ? l[2] / G::TZ : S - 1)) == slab;
            else if (PHASE == PDA_ALL && slab == 0)
              defer(p);
          }
        }
        const unsigned long long m = __ballot(own);
        if (own) q[qn + (int)__popcll(m & ((1ull << lane) - 1ull))] = p;
        qn += (int)__popcll(m);
      }
      if (qn >= 64 || (!more && qn > 0)) {
        __builtin_amdgcn_wave_barrier();
        const int cnt = qn < 64 ? qn : 64;
        const int p = lane < cnt ? q[qn - cnt + lane] : -1;
        __builtin_amdgcn_wave_barrier();
        qn -= cnt;
        if (p >= 0) {
          const PState<R> s = load_particle<DIMS, R>(pa, p, P.q_const);
          int c3[3] = {0, 0, 0}, l[3] = {0, 0, 0};
          decode<DIMS, R>(P, s, c3, flg);
          locate(c3, l);
          l[2] -= slab * G::TZ;
          work(p, s, l);
        }
      }
      if (!more) break;
    }
  }
  if constexpr (!G::has_leb) return;
  __syncthreads();
  // lamE, lamB of the region (its halo overlaps the neighbouring regions')
  for (int r = threadIdx.x; r < G::e_cnt; r += G::NT) {
    const int lx = r % G::ex, ly = (r / G::ex) % G::ex, lz = r / (G::ex * G::ex);
    const int t = lz * G::ep + ly * G::es + lx;
    int sx[2], sy[2], sz[2] = {0, 0};
    axis_slots(org[0] + G::e_lo + lx, P.n[0], open0, 1, sx);
    axis_slots(org[1] + G::e_lo + ly, P.n[1], open1, str1, sy);
    if (DIMS == 3) axis_slots(org[2] + G::e_lo_z + lz, P.n[2], open2, str2, sz);
#pragma unroll
    for (int c = 0; c < 6; ++c) {  // E_c staggered along c, B_c along the two others
      const int e = c < 3 ? c : c - 3;
      const bool isb = c >= 3;
      const int ix = sx[isb ? (e != 0) : (e == 0)];
      const int iy = sy[isb ? (e != 1) : (e == 1)];
      const int iz = sz[isb ? (e != 2) : (e == 2)];
      const double v = G::has_leb ? s_leb[c * G::e_vol + t] : 0.0;
      if (v != 0.0 && ix >= 0 && iy >= 0 && iz >= 0) atomicAdd(&(isb ? L.B : L.E)[e][ix + iy + iz], (R)v);
    }
  }
}

static __global__ void k_adj_reset(DevFlags* flg) { flg->ndefer = 0u; }

template <int DIMS, int ORDER, typename R>
int launch_pda(const pic_ctx* ctx, const pic_particles* p, const pic_fields* f,
                      const pic_fields* lf, pic_particles* lp, void* ws, hipStream_t s) {
  KParams<R> P = make_params<R>(ctx);
  WsLayout Lw = ws_layout(ctx, p->np);
  DParts<R> pa, la;
  pa.cell = p->cell;
  la.cell = nullptr;
  for (int d = 0; d < 3; ++d) {
    pa.off[d] = (R*)p->off[d];
    pa.u[d] = (R*)p->u[d];
    la.off[d] = (R*)lp->off[d];
    la.u[d] = (R*)lp->u[d];
  }
  pa.q = (R*)p->q;
  pa.id = nullptr;
  la.q = nullptr;
  la.id = nullptr;
  DFields<R> F, L;
  for (int c = 0; c < 3; ++c) {
    F.E[c] = (R*)f->E[c];
    F.B[c] = (R*)f->B[c];
    F.J[c] = nullptr;
    L.E[c] = (R*)lf->E[c];
    L.B[c] = (R*)lf->B[c];
    L.J[c] = (R*)lf->J[c];
  }
  if (p->np == 0) return 0;
  DevFlags* flg = (DevFlags*)((char*)ws + Lw.flags);
  const long blocks = (p->np + 255) / 256;
  const unsigned gblocks = (unsigned)(blocks < 8192 ? blocks : 8192);
  // the LDS tile path needs tile bins for these np particles in this
  // workspace (any particle order is then handled correctly: a particle
  // outside the allowance of the tile whose range holds it takes the
  // global-memory kernel)
  if (ctx->sorted_np == p->np && ctx->sorted_ws == ws) {
    const int* starts = (const int*)((char*)ws + Lw.starts);
    int* deferred = (int*)((char*)ws + Lw.tmp_cell);
    R* lam_eb = (R*)((char*)ws + Lw.tmp_real);  // (the sort's scratch, free here)
    k_adj_reset<<<dim3(1), dim3(1), 0, s>>>(flg);
    auto phase = [&](auto ph, auto nt) {
      constexpr int PH = decltype(ph)::value, NT2 = decltype(nt)::value;
      using G = AdjGeo<DIMS, ORDER, R, PH, NT2>;
      k_pda_tile<DIMS, ORDER, R, PH, NT2><<<dim3(8 * P.per_xcd * G::S), dim3(G::NT), 0, s>>>(
          P, pa, F, L, la, lam_eb, (long)p->np, starts, deferred, flg);
    };
    const std::integral_constant<int, PDA_ALL> all{};
    const std::integral_constant<int, 512> nt512{};
    if constexpr (DIMS == 2) {
      // 8 wavefronts where a CU has at most two tiles, 4 where it has more.  Of
      // the forms with more than 128 registers (all but linear FP32) one
      // workgroup of 8 or two of 4 are on a CU; a wavefront more per SIMD hides
      // more of a tile's own latencies, and two tiles side by side hide each
      // other's staging and flush, which counts once tiles queue for CUs.  Us with
      // 8 and with 4: 300x200, 247 tiles, FP32 quadratic 45 and 61, cubic 72 and
      // 92; 512x256, 512 tiles, FP32 quadratic right after a sort 133 and 129, a
      // laser rollout of 10 steps, whose particles have drifted, 3516 and 3650;
      // 1024x1024, 4096 tiles, FP32 quadratic 568 and 436, cubic 1000 and 857,
      // FP64 linear 501 and 444.  Linear FP32 and cubic FP64 (which takes so many
      // registers with 4 that no two fit) are the faster with 8 at every size
      // (1024x1024: 277 and 293, 1201 and 1341).
      constexpr bool wide = (sizeof(R) == 4 && ORDER == 1) || (sizeof(R) == 8 && ORDER == 3);
      if (wide || P.ntiles <= 2 * ctx->cu_count)
        phase(all, nt512);
      else if constexpr (!wide)
        phase(all, std::integral_constant<int, 256>{});
    } else {
      // One kernel over the tile's slabs for linear shapes, whose regions leave
      // one or two slabs (96x80x64: FP32 310 us and 344 in two phases, FP64 609
      // and 669), and where every slab has a CU to itself, so that the two
      // phases' chains of latencies would only come one after the other (24x16x20,
      // 18 tiles: FP32 quadratic 139 and 208 us, cubic 228 and 359, quartic 242
      // and 404, FP64 quadratic 147 and 189; with 288 slabs, 48x48x32 FP32
      // quadratic, 269 and 228).  FP64 cubic does not fit and quartic gains
      // nothing.
      constexpr bool one = sizeof(R) == 4 || ORDER <= 2;
      bool done = false;
      if constexpr (one) {
        using G = AdjGeo<DIMS, ORDER, R, PDA_ALL, 512>;
        if (ORDER == 1 || P.ntiles * G::S <= ctx->cu_count) {
          phase(all, nt512);
          done = true;
        }
      }
      if constexpr (ORDER > 1)
        if (!done) {
          phase(std::integral_constant<int, PDA_BACK>{}, nt512);
          phase(std::integral_constant<int, PDA_GATHER>{}, nt512);
        }
    }
    k_push_deposit_adjoint<DIMS, ORDER, R><<<dim3(gblocks), dim3(256), 0, s>>>(
        P, pa, F, L, la, flg, (int)p->np, deferred, starts + P.ntiles);
    return (int)hipGetLastError();
  }
  k_push_deposit_adjoint<DIMS, ORDER, R><<<dim3(gblocks), dim3(256), 0, s>>>(
      P, pa, F, L, la, flg, (int)p->np, nullptr, nullptr);
  return (int)hipGetLastError();
}

// The instantiations are compiled one by one (the build defines PIC_DIMS,
// PIC_ORDER and PIC_REAL), the dispatch in a part of its own: one compiler takes
// many times as long for all of them.
#define PIC_INST(HOW, DD, OO, RR) \
  HOW template int launch_pda<DD, OO, RR>( \
      const pic_ctx* ctx, const pic_particles* p, const pic_fields* f, \
      const pic_fields* lf, pic_particles* lp, void* ws, hipStream_t s);
#ifdef PIC_DIMS
PIC_INST(, PIC_DIMS, PIC_ORDER, PIC_REAL)
#else
#define PIC_EXTERN(DD, OO) PIC_INST(extern, DD, OO, float) PIC_INST(extern, DD, OO, double)
PIC_EXTERN(2, 1) PIC_EXTERN(2, 2) PIC_EXTERN(2, 3) PIC_EXTERN(2, 4)
PIC_EXTERN(3, 1) PIC_EXTERN(3, 2) PIC_EXTERN(3, 3) PIC_EXTERN(3, 4)

int launch_push_deposit_adjoint(const pic_ctx* ctx, const pic_particles* p, const pic_fields* f,
                                const pic_fields* lam_f, pic_particles* lam_p, void* ws,
                                hipStream_t s) {
  const int D = ctx->cfg.dims, O = ctx->cfg.order;
  const bool dbl = ctx->cfg.real_bytes == 8;
#define PIC_PDA(DD, OO)                                                          \
  if (D == DD && O == OO)                                                        \
    return dbl ? launch_pda<DD, OO, double>(ctx, p, f, lam_f, lam_p, ws, s)     \
               : launch_pda<DD, OO, float>(ctx, p, f, lam_f, lam_p, ws, s);
  PIC_PDA(2, 1) PIC_PDA(2, 2) PIC_PDA(2, 3) PIC_PDA(2, 4)
  PIC_PDA(3, 1) PIC_PDA(3, 2) PIC_PDA(3, 3) PIC_PDA(3, 4)
#undef PIC_PDA
  return (int)hipErrorInvalidValue;
}
#endif

}  // namespace pic
