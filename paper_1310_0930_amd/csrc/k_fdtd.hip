// FDTD (Yee) field advance: B -= dt/2 C E; E += dt (C^T B - J); B -= dt/2 C E.
//
// The paper advances the fields with the finite-difference time-domain method
// (Sec. 2), a local, nearest-neighbour solver chosen for its small
// communication volume (Sec. 3).  C is the forward-difference curl of E at
// the B positions and C^T (its transpose) the backward-difference curl of B
// at the E positions.  One thread updates the three components of a short
// z column of cells (one cell in 2D and on small grids).
//
// Open faces: the tangential E samples on the first and last node planes of
// an open axis are advanced with the first-order Mur condition
// F0^{n+1} = F1^n + (dt - dx)/(dt + dx) (F1^{n+1} - F0^n), F1 the next sample
// inward.  Samples on two open faces (edges) follow along the lower such
// axis.  Samples beyond the last node (half-integer positions) are outside
// the domain, are never written and are read as zero.
#include <type_traits>

#include "k_common.h"

namespace pic {

struct FdParams {
  int n[3];
  int open[3];
  int dims;
  FastDiv dn0, dn1;
};

__device__ __forceinline__ void decompose(const FdParams& P, int idx, int& i, int& j, int& k) {
  const uint32_t rest = P.dn0.div((uint32_t)idx);
  i = idx - (int)rest * P.n[0];
  if (P.dims == 3) {
    const uint32_t r2 = P.dn1.div(rest);
    j = (int)(rest - r2 * P.n[1]);
    k = (int)r2;
  } else {
    j = (int)rest;
    k = 0;
  }
}

// Is the slot (i,j,k) of a component with staggering (sx,sy,sz) inside?
__device__ __forceinline__ bool inside(const FdParams& P, int i, int j, int k, int sx, int sy, int sz) {
  if (P.open[0] && i > P.n[0] - 1 - sx) return false;
  if (P.open[1] && j > P.n[1] - 1 - sy) return false;
  if (P.dims == 3 && P.open[2] && k > P.n[2] - 1 - sz) return false;
  return true;
}

// Block index with the 8 XCDs each taking a contiguous range of blocks
// (consecutive block ids are dealt round-robin to the XCDs): the neighbour
// rows and planes a stencil reads then sit in the same XCD's L2.  The grid
// must be a multiple of 8 blocks; the mapping is a permutation of it.
__device__ __forceinline__ int xcd_block() {
  const int per = gridDim.x >> 3;
  return (blockIdx.x & 7) * per + (blockIdx.x >> 3);
}

__host__ inline unsigned xcd_grid(long ncell) {
  const long g = (ncell + 255) / 256;
  return (unsigned)((g + 7) / 8 * 8);
}

// A thread's column: KC consecutive z planes (one cell in 2D) at (i, j).
// RAGGED: KC does not divide the number of planes and the last column is
// shorter; the test for its end keeps the planes' loads from going out
// together (128^3 periodic, whole advance: 42.6 us with it and 41.2 without in
// FP32, 79.3 and 75.0 in FP64).
// Consecutive threads take consecutive x, so every load and store is
// coalesced; the column's index arithmetic and wraps are formed once, the z
// neighbour of one plane is the next plane's own sample, kept in registers,
// and the x neighbour is the adjacent lane's sample, passed across the
// wavefront (only a lane at the wavefront's or the row's end loads it).
__device__ __forceinline__ int column_start(const FdParams& P, int t, int kc, int& i, int& j,
                                            int& k0) {
  const uint32_t q0 = P.dn0.div((uint32_t)t);  // t / n0
  i = t - (int)q0 * P.n[0];
  const uint32_t q1 = P.dn1.div(q0);  // column block along z
  j = (int)(q0 - q1 * P.n[1]);
  k0 = (int)q1 * kc;
  return i + P.n[0] * (j + P.n[1] * k0);
}

// One component of a curl, ha da - hb db (da: the difference along the first
// of the two other axes, db along the second; an axis a 2D grid does not have
// drops out).  STEP: summed term by term, the first product rounded before the
// second is fused to it (open and 2D grids, whose laser runs amplify any change
// of rounding); else as the compiler contracts the expression.
template <bool STEP, bool HAS_A, bool HAS_B, typename R>
__device__ __forceinline__ R curl_of(R ha, R da, R hb, R db) {
  if constexpr (STEP) {
    R acc = R(0);
    if constexpr (HAS_A) acc += ha * da;
    if constexpr (HAS_B) acc -= hb * db;
    return acc;
  } else {
    return ha * da - hb * db;
  }
}

// B -= h C E (forward differences).  OPEN: some axis is open; B_c is
// staggered along the two other axes, where the last plane of an open axis is
// outside (its wrapped neighbours are read but not used).
template <typename R, int DIMS, int KC, bool OPEN, bool RAGGED>
__global__ void __launch_bounds__(256) k_half_b(FdParams P, const R* __restrict__ E0,
                                                const R* __restrict__ E1,
                                                const R* __restrict__ E2, R* __restrict__ B0,
                                                R* __restrict__ B1, R* __restrict__ B2, R hx, R hy,
                                                R hz, int ncol) {
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= ncol) return;
  int i, j, k0;
  int idx = column_start(P, t, KC, i, j, k0);
  const int plane = P.n[0] * P.n[1];
  const int ip = i + 1 < P.n[0] ? 1 : 1 - P.n[0];
  const int jp = j + 1 < P.n[1] ? P.n[0] : P.n[0] - plane;
  const int lane = threadIdx.x & 63;
  const bool own = lane < 63 && i + 1 < P.n[0];  // the x neighbour is the next lane's sample
  const bool inx = !OPEN || !P.open[0] || i + 1 < P.n[0];
  const bool iny = !OPEN || !P.open[1] || j + 1 < P.n[1];
  R exk = E0[idx], eyk = E1[idx];  // E_x, E_y at plane k
#pragma unroll
  for (int kk = 0; kk < KC; ++kk, idx += plane) {
    const int k = k0 + kk;
    if (RAGGED && k >= P.n[2]) break;
    R ex1 = exk, ey1 = eyk;
    if (DIMS == 3) {
      const int kp = k + 1 < P.n[2] ? plane : plane - P.n[2] * plane;
      ex1 = E0[idx + kp];
      ey1 = E1[idx + kp];
    }
    const bool inz = !OPEN || DIMS == 2 || !P.open[2] || k + 1 < P.n[2];
    const R ez = E2[idx];
    R ezx = __shfl_down(ez, 1, 64), eyx = __shfl_down(eyk, 1, 64);
    if (!own) {
      ezx = E2[idx + ip];
      eyx = E1[idx + ip];
    }
    constexpr bool Z = DIMS == 3, S = OPEN || !Z;
    if (iny && inz) B0[idx] -= curl_of<S, true, Z, R>(hy, E2[idx + jp] - ez, hz, ey1 - eyk);
    if (inx && inz) B1[idx] -= curl_of<S, Z, true, R>(hz, ex1 - exk, hx, ezx - ez);
    if (inx && iny) B2[idx] -= curl_of<S, true, true, R>(hx, eyx - eyk, hy, E0[idx + jp] - exk);
    exk = ex1;
    eyk = ey1;
  }
}

// Mur updates of the face samples of one component next to the interior
// sample at idx, which the calling thread has just advanced from `old` to
// `nw`: along axis a (sa = -1 or +1: the open face lies one sample below or
// above; 0: no face), along axis b, and of the edge both meet in (along a,
// the lower axis).  No other thread reads or writes these samples.
template <typename R>
__device__ __forceinline__ void mur_faces(R* __restrict__ E, int idx, int sa, int stra, R ka,
                                          int sb, int strb, R kb, R old, R nw) {
  if (sa != 0) {
    const int fa = idx + sa * stra;
    E[fa] = old + ka * (nw - E[fa]);
  }
  if (sb != 0) {
    const int fb = idx + sb * strb;
    const R fo = E[fb], fn = old + kb * (nw - fo);
    E[fb] = fn;
    if (sa != 0) {
      const int ed = fb + sa * stra;
      E[ed] = fo + ka * (fn - E[ed]);
    }
  }
}

// E += g C^T B - dt J (backward differences) on the interior samples.  OPEN:
// the Mur update of a face sample needs its inner neighbour before and after
// this step, so the thread that advances the inner neighbour does it too (the
// face samples used to be saved to memory and updated by 2 to 12 small
// launches, and only grids periodic along every axis took columns:
// 250x131x121, open y and z, FP32: the whole advance 167 -> 95 us, 5.0 TB/s
// of the 30 reals per cell that the three in-place passes move, where a large
// copy reaches 4.7: some of what one pass leaves the next still finds in cache).
template <typename R, int DIMS, int KC, bool OPEN, bool RAGGED>
__global__ void __launch_bounds__(256) k_advance_e(
    FdParams P, R* __restrict__ E0, R* __restrict__ E1, R* __restrict__ E2,
    const R* __restrict__ B0, const R* __restrict__ B1, const R* __restrict__ B2,
    const R* __restrict__ J0, const R* __restrict__ J1, const R* __restrict__ J2, R gx, R gy, R gz,
    R kx, R ky, R kz, R dt, int ncol) {
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= ncol) return;
  int i, j, k0;
  int idx = column_start(P, t, KC, i, j, k0);
  const int plane = P.n[0] * P.n[1];
  const int im = i > 0 ? -1 : P.n[0] - 1;
  const int jm = j > 0 ? -P.n[0] : plane - P.n[0];
  const int lane = threadIdx.x & 63;
  const bool own = lane > 0 && i > 0;  // the -x neighbour is the previous lane's sample
  // in: inside along a staggered axis; at: on an open face; sx..: next to one
  const bool inx = !OPEN || !P.open[0] || i + 1 < P.n[0], iny = !OPEN || !P.open[1] || j + 1 < P.n[1];
  const bool atx = OPEN && P.open[0] && (i == 0 || i == P.n[0] - 1);
  const bool aty = OPEN && P.open[1] && (j == 0 || j == P.n[1] - 1);
  const int sx = OPEN && P.open[0] ? (i == 1 ? -1 : i == P.n[0] - 2 ? 1 : 0) : 0;
  const int sy = OPEN && P.open[1] ? (j == 1 ? -1 : j == P.n[1] - 2 ? 1 : 0) : 0;
  R bxm = R(0), bym = R(0);  // B_x, B_y at plane k - 1
  if (DIMS == 3) {
    const int km = k0 > 0 ? -plane : (P.n[2] - 1) * plane;
    bxm = B0[idx + km];
    bym = B1[idx + km];
  }
#pragma unroll
  for (int kk = 0; kk < KC; ++kk, idx += plane) {
    const int k = k0 + kk;
    if (RAGGED && k >= P.n[2]) break;
    constexpr bool Z = DIMS == 3, S = OPEN || !Z;
    const R bx = B0[idx], by = B1[idx], bz = B2[idx];
    R bzx = __shfl_up(bz, 1, 64), byx = __shfl_up(by, 1, 64);
    if (!own) {
      bzx = B2[idx + im];
      byx = B1[idx + im];
    }
    const bool inz = !OPEN || DIMS == 2 || !P.open[2] || k + 1 < P.n[2];
    const bool atz = OPEN && DIMS == 3 && P.open[2] && (k == 0 || k == P.n[2] - 1);
    const int sz = OPEN && DIMS == 3 && P.open[2] ? (k == 1 ? -1 : k == P.n[2] - 2 ? 1 : 0) : 0;
    if (inx && !aty && !atz) {
      const R old = E0[idx];
      const R nw = old + (curl_of<S, true, Z, R>(gy, bz - B2[idx + jm], gz, by - bym) - dt * J0[idx]);
      E0[idx] = nw;
      if (OPEN && (sy | sz)) mur_faces<R>(E0, idx, sy, P.n[0], ky, sz, plane, kz, old, nw);
    }
    if (iny && !atx && !atz) {
      const R old = E1[idx];
      const R nw = old + (curl_of<S, Z, true, R>(gz, bx - bxm, gx, bz - bzx) - dt * J1[idx]);
      E1[idx] = nw;
      if (OPEN && (sx | sz)) mur_faces<R>(E1, idx, sx, 1, kx, sz, plane, kz, old, nw);
    }
    if (inz && !atx && !aty) {
      const R old = E2[idx];
      const R nw = old + (curl_of<S, true, true, R>(gx, by - byx, gy, bx - B0[idx + jm]) - dt * J2[idx]);
      E2[idx] = nw;
      if (OPEN && (sx | sy)) mur_faces<R>(E2, idx, sx, 1, kx, sy, P.n[0], ky, old, nw);
    }
    bxm = bx;
    bym = by;
  }
}

static FdParams fd_params(const pic_config& cf, bool& any_open) {
  FdParams P;
  P.dims = cf.dims;
  any_open = false;
  for (int d = 0; d < 3; ++d) {
    P.n[d] = d < cf.dims ? cf.n[d] : 1;
    P.open[d] = d < cf.dims && cf.bc[d] == PIC_BC_OPEN;
    any_open = any_open || P.open[d];
  }
  P.dn0.init((uint32_t)P.n[0]);
  P.dn1.init((uint32_t)P.n[1]);
  return P;
}

// Planes per thread of the 3D kernels; below FD_COL_CELLS cells one plane, so
// that every CU still gets some eight wavefronts to hide the loads' latency.
constexpr int FD_KC = 4;
constexpr long FD_COL_CELLS = 1L << 19;

template <typename R, int DIMS, int KC, bool OPEN, bool RAGGED>
static int launch_fa_t(const pic_ctx* ctx, const FdParams& P, const pic_fields* f, hipStream_t s) {
  const pic_config& cf = ctx->cfg;
  const R dt = (R)cf.dt;
  R h[3], g[3], kp[3];
  for (int d = 0; d < 3; ++d) {
    h[d] = (R)(0.5 * cf.dt / cf.dx[d]);
    g[d] = (R)(cf.dt / cf.dx[d]);
    kp[d] = (R)((cf.dt - cf.dx[d]) / (cf.dt + cf.dx[d]));
  }
  R* E[3];
  R* B[3];
  R* J[3];
  for (int c = 0; c < 3; ++c) {
    E[c] = (R*)f->E[c];
    B[c] = (R*)f->B[c];
    J[c] = (R*)f->J[c];
  }
  const int ncol = P.n[0] * P.n[1] * ((P.n[2] + KC - 1) / KC);
  const dim3 grid(xcd_grid(ncol)), block(256);  // a multiple of 8 blocks (xcd_block)
  k_half_b<R, DIMS, KC, OPEN, RAGGED><<<grid, block, 0, s>>>(
      P, E[0], E[1], E[2], B[0], B[1], B[2], h[0], h[1], h[2], ncol);
  k_advance_e<R, DIMS, KC, OPEN, RAGGED><<<grid, block, 0, s>>>(
      P, E[0], E[1], E[2], B[0], B[1], B[2], J[0], J[1], J[2], g[0], g[1], g[2], kp[0], kp[1],
      kp[2], dt, ncol);
  k_half_b<R, DIMS, KC, OPEN, RAGGED><<<grid, block, 0, s>>>(
      P, E[0], E[1], E[2], B[0], B[1], B[2], h[0], h[1], h[2], ncol);
  return (int)hipGetLastError();
}

template <typename R>
static int launch_fa(const pic_ctx* ctx, const pic_fields* f, hipStream_t s) {
  bool open;
  const FdParams P = fd_params(ctx->cfg, open);
  auto go = [&](auto dims, auto kc, auto ragged) {
    constexpr int D = decltype(dims)::value, KC = decltype(kc)::value;
    constexpr bool RAGGED = decltype(ragged)::value;
    return open ? launch_fa_t<R, D, KC, true, RAGGED>(ctx, P, f, s)
                : launch_fa_t<R, D, KC, false, RAGGED>(ctx, P, f, s);
  };
  const std::integral_constant<int, 1> one{};
  const std::integral_constant<int, 2> two{};
  const std::integral_constant<int, 3> three{};
  const std::integral_constant<int, FD_KC> col{};
  if (P.dims == 2) return go(two, one, std::false_type{});
  if ((long)P.n[0] * P.n[1] * P.n[2] < FD_COL_CELLS) return go(three, one, std::false_type{});
  return P.n[2] % FD_KC ? go(three, col, std::true_type{}) : go(three, col, std::false_type{});
}

int launch_field_advance(const pic_ctx* ctx, const pic_fields* f, hipStream_t s) {
  return ctx->cfg.real_bytes == 8 ? launch_fa<double>(ctx, f, s) : launch_fa<float>(ctx, f, s);
}

// ------------------------------------------------------------------ adjoint
// Transpose of the field advance (for the hand-written adjoint of the step).
// The advance is linear in (E, B, J); with mu the adjoint of E^{n+1} after
// the last half step, its transpose is, in reverse order:
//   mu = lamE - h C^T mask(lamB)                  (the last half step)
//   Mur updates transposed, edges then faces
//   lamJ = -dt mu on the samples the Yee update advances, 0 elsewhere
//   lamB += dt C mu_interior = -C lamJ
//   lamE = mu (+ the direct F1^n terms of Mur);   lamE -= h C^T mask(lamB)
// where mask() keeps the B samples inside the domain (the only ones the
// forward updates or reads).  Three passes: k_adj_e_mur (the first three
// lines, and the F1^n terms), k_adj_b, k_adj_e.  The middle pass reads mu from
// lamJ, which is zero exactly where the forward does not advance, so that
// lamE can already hold the sum with the Mur terms and no array is kept
// beside them (512x256, open y, FP32: 9 launches of about 4.5 us before, now 3;
// a rollout of 10 steps forward and back 4.00 -> 3.80 ms).

// h C^T lamB at one sample: component c, (i, j, k), lamB read only inside the
// domain.
template <typename R, int DIMS, bool OPEN>
struct AdjCurlB {
  const FdParams& P;
  const R* B[3];
  R h[3];
  __device__ __forceinline__ R value(int comp, int i, int j, int k) const {
    if (OPEN && !inside(P, i, j, k, comp != 0, comp != 1, comp != 2)) return R(0);
    return B[comp][i + P.n[0] * (j + P.n[1] * k)];
  }
  // value one sample lower along axis d (0 beyond an open face)
  __device__ __forceinline__ R lower(int comp, int i, int j, int k, int d) const {
    int L[3] = {i, j, k};
    L[d] -= 1;
    if (L[d] < 0) {
      if (OPEN && P.open[d]) return R(0);
      L[d] += P.n[d];
    }
    return value(comp, L[0], L[1], L[2]);
  }
  __device__ __forceinline__ R operator()(int c, int i, int j, int k) const {
    const int a = (c + 1) % 3, b = (c + 2) % 3;
    R curl = R(0);
    if (a < DIMS) curl += h[a] * (value(b, i, j, k) - lower(b, i, j, k, a));
    if (b < DIMS) curl -= h[b] * (value(a, i, j, k) - lower(a, i, j, k, b));
    return curl;
  }
};

// mu, lamJ and the Mur terms of one cell.  The forward's Mur update of a face
// sample F0 <- F1^n + kappa (F1 - F0^n) transposes to mu1 += kappa mu0,
// x1 += mu0, mu0 <- -kappa mu0 (x: the direct terms, summed into lamE): the
// thread of the inner neighbour does it, for its face samples along the two
// axes a < b other than the component's and, first, the edge both meet in
// (which the forward takes from the face sample along b).  Face samples are
// otherwise untouched here: their own threads skip them.
template <typename R, int DIMS, bool OPEN>
__global__ void __launch_bounds__(256) k_adj_e_mur(FdParams P, R* __restrict__ L0,
                                                   R* __restrict__ L1, R* __restrict__ L2,
                                                   const R* __restrict__ B0,
                                                   const R* __restrict__ B1,
                                                   const R* __restrict__ B2, R* __restrict__ J0,
                                                   R* __restrict__ J1, R* __restrict__ J2, R hx,
                                                   R hy, R hz, R kx, R ky, R kz, R dt, int ncell) {
  const int idx = xcd_block() * blockDim.x + threadIdx.x;
  if (idx >= ncell) return;
  int i, j, k;
  decompose(P, idx, i, j, k);
  R* Lm[3] = {L0, L1, L2};
  R* J[3] = {J0, J1, J2};
  const AdjCurlB<R, DIMS, OPEN> curl{P, {B0, B1, B2}, {hx, hy, hz}};
  const int L[3] = {i, j, k};
  const int str[3] = {1, P.n[0], P.n[0] * P.n[1]};
  const R kap[3] = {kx, ky, kz};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int a = c == 0 ? 1 : 0, b = c == 2 ? 1 : 2;  // the other axes, a < b
    const bool in = !OPEN || inside(P, i, j, k, c == 0, c == 1, c == 2);
    bool face = false;
    int sa = 0, sb = 0;  // the open face one sample away along a, b
    if (OPEN) {
      if (P.open[a]) {
        face = face || L[a] == 0 || L[a] == P.n[a] - 1;
        sa = L[a] == 1 ? -1 : L[a] == P.n[a] - 2 ? 1 : 0;
      }
      if (b < DIMS && P.open[b]) {
        face = face || L[b] == 0 || L[b] == P.n[b] - 1;
        sb = L[b] == 1 ? -1 : L[b] == P.n[b] - 2 ? 1 : 0;
      }
    }
    if (!in) {  // outside: only the transposed curl, no advance
      Lm[c][idx] -= curl(c, i, j, k);
      J[c][idx] = R(0);
      continue;
    }
    if (face) {
      J[c][idx] = R(0);
      continue;
    }
    R mu = Lm[c][idx] - curl(c, i, j, k), x = R(0);
    if (OPEN && (sa | sb)) {
      auto mu_at = [&](int da, int db) {
        int M[3] = {i, j, k};
        M[a] += da;
        M[b] += db;
        return Lm[c][idx + da * str[a] + db * str[b]] - curl(c, M[0], M[1], M[2]);
      };
      R xb = R(0), mub = R(0);
      if (sb) mub = mu_at(0, sb);
      if (sa && sb) {  // the edge, taken from the face sample along b
        const R e = mu_at(sa, sb);
        mub += kap[a] * e;
        xb = e;
        Lm[c][idx + sa * str[a] + sb * str[b]] = -kap[a] * e;
      }
      if (sa) {
        const R f = mu_at(sa, 0);
        mu += kap[a] * f;
        x += f;
        Lm[c][idx + sa * str[a]] = -kap[a] * f;
      }
      if (sb) {
        mu += kap[b] * mub;
        x += mub;
        Lm[c][idx + sb * str[b]] = -kap[b] * mub + xb;
      }
    }
    J[c][idx] = -dt * mu;
    Lm[c][idx] = mu + x;
  }
}

// lamB -= C lamJ on the inside B samples (forward differences; lamJ = -dt mu
// on the samples the forward advances, 0 on the others).
template <typename R, int DIMS, bool OPEN>
__global__ void __launch_bounds__(256) k_adj_b(FdParams P, const R* __restrict__ J0,
                                               const R* __restrict__ J1, const R* __restrict__ J2,
                                               R* __restrict__ B0, R* __restrict__ B1,
                                               R* __restrict__ B2, R gx, R gy, R gz, int ncell) {
  const int idx = xcd_block() * blockDim.x + threadIdx.x;
  if (idx >= ncell) return;
  int i, j, k;
  decompose(P, idx, i, j, k);
  const R* J[3] = {J0, J1, J2};
  R* B[3] = {B0, B1, B2};
  const R g[3] = {gx, gy, gz};  // 1 / dx_d
  const int L[3] = {i, j, k};
  const int str[3] = {1, P.n[0], P.n[0] * P.n[1]};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (OPEN && !inside(P, i, j, k, c != 0, c != 1, c != 2)) continue;
    const int a = (c + 1) % 3, b = (c + 2) % 3;
    // inside along an open axis means a neighbour: only periodic axes wrap
    auto diff = [&](int v, int d) {
      const int up = L[d] + 1 < P.n[d] ? str[d] : str[d] - P.n[d] * str[d];
      return J[v][idx + up] - J[v][idx];
    };
    R acc = R(0);
    if (a < DIMS) acc += g[a] * diff(b, a);
    if (b < DIMS) acc -= g[b] * diff(a, b);
    B[c][idx] -= acc;
  }
}

// lamE -= h C^T lamB over every E sample, lamB read only inside the domain.
template <typename R, int DIMS, bool OPEN>
__global__ void __launch_bounds__(256) k_adj_e(FdParams P, R* __restrict__ L0, R* __restrict__ L1,
                                               R* __restrict__ L2, const R* __restrict__ B0,
                                               const R* __restrict__ B1, const R* __restrict__ B2,
                                               R hx, R hy, R hz, int ncell) {
  const int idx = xcd_block() * blockDim.x + threadIdx.x;
  if (idx >= ncell) return;
  int i, j, k;
  decompose(P, idx, i, j, k);
  R* Lm[3] = {L0, L1, L2};
  const AdjCurlB<R, DIMS, OPEN> curl{P, {B0, B1, B2}, {hx, hy, hz}};
#pragma unroll
  for (int c = 0; c < 3; ++c) Lm[c][idx] -= curl(c, i, j, k);
}

template <typename R, int DIMS, bool OPEN>
static int launch_fa_adj_t(const pic_ctx* ctx, const FdParams& P, const pic_fields* lam,
                           hipStream_t s) {
  const pic_config& cf = ctx->cfg;
  R h[3], g[3], kp[3];
  for (int d = 0; d < 3; ++d) {
    h[d] = (R)(0.5 * cf.dt / cf.dx[d]);
    g[d] = (R)(1.0 / cf.dx[d]);
    kp[d] = (R)((cf.dt - cf.dx[d]) / (cf.dt + cf.dx[d]));
  }
  R* E[3];
  R* B[3];
  R* J[3];
  for (int c = 0; c < 3; ++c) {
    E[c] = (R*)lam->E[c];
    B[c] = (R*)lam->B[c];
    J[c] = (R*)lam->J[c];
  }
  const int ncell = P.n[0] * P.n[1] * P.n[2];
  const dim3 grid(xcd_grid(ncell)), block(256);
  k_adj_e_mur<R, DIMS, OPEN><<<grid, block, 0, s>>>(P, E[0], E[1], E[2], B[0], B[1], B[2], J[0],
                                                    J[1], J[2], h[0], h[1], h[2], kp[0], kp[1],
                                                    kp[2], (R)cf.dt, ncell);
  k_adj_b<R, DIMS, OPEN><<<grid, block, 0, s>>>(P, J[0], J[1], J[2], B[0], B[1], B[2], g[0], g[1],
                                                g[2], ncell);
  k_adj_e<R, DIMS, OPEN><<<grid, block, 0, s>>>(P, E[0], E[1], E[2], B[0], B[1], B[2], h[0], h[1],
                                                h[2], ncell);
  return (int)hipGetLastError();
}

template <typename R>
static int launch_fa_adj(const pic_ctx* ctx, const pic_fields* lam, hipStream_t s) {
  bool open;
  const FdParams P = fd_params(ctx->cfg, open);
  if (P.dims == 2)
    return open ? launch_fa_adj_t<R, 2, true>(ctx, P, lam, s)
                : launch_fa_adj_t<R, 2, false>(ctx, P, lam, s);
  return open ? launch_fa_adj_t<R, 3, true>(ctx, P, lam, s)
              : launch_fa_adj_t<R, 3, false>(ctx, P, lam, s);
}

int launch_field_advance_adjoint(const pic_ctx* ctx, const pic_fields* lam, hipStream_t s) {
  return ctx->cfg.real_bytes == 8 ? launch_fa_adj<double>(ctx, lam, s)
                                  : launch_fa_adj<float>(ctx, lam, s);
}

}  // namespace pic
