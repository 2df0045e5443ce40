// FP64 diagnostics, kept off the timed loop: charge density from the stored
// cells and offsets, Gauss's-law and continuity residuals, field and kinetic
// energies.
//
// Charge conservation is the property the paper's deposit is chosen for
// (Sec. 5.2: a charge-conserving method for the virtual trajectories); these
// residuals measure it in double precision against the positions the push
// actually stored, whatever precision the push ran in.
#include "k_common.h"

namespace pic {

struct DiagParams {
  int n[3];
  int open[3];
  int dims, order, margin;
  double dx[3], dt, dV;
  FastDiv dn0, dn1;
  int ncell;
};

// Node-centred B-spline weights in double (same polynomials as the push).
template <int ORDER>
__device__ __forceinline__ int node_weights(double o, double* w) {
  double xi;
  int k;
  if (ORDER & 1) {
    k = 0;
    xi = o;
  } else {
    k = o >= 0.5;
    xi = k ? o - 1.0 : o;
  }
  if (ORDER == 1) {
    w[0] = 1.0 - xi;
    w[1] = xi;
  } else if (ORDER == 2) {
    const double a = 0.5 - xi, b = 0.5 + xi;
    w[0] = 0.5 * a * a;
    w[1] = 0.75 - xi * xi;
    w[2] = 0.5 * b * b;
  } else if (ORDER == 3) {
    const double s = 1.0 - xi, t2 = xi * xi, t3 = t2 * xi;
    w[0] = s * s * s / 6.0;
    w[1] = (4.0 - 6.0 * t2 + 3.0 * t3) / 6.0;
    w[2] = (1.0 + 3.0 * xi + 3.0 * t2 - 3.0 * t3) / 6.0;
    w[3] = t3 / 6.0;
  } else {
    const double a = 1.0 - 2.0 * xi, b = 1.0 + 2.0 * xi, t2 = xi * xi;
    w[0] = a * a * a * a / 384.0;
    w[1] = (19.0 + xi * (-44.0 + xi * (24.0 + xi * (16.0 - 16.0 * xi)))) / 96.0;
    w[2] = (115.0 + t2 * (-120.0 + 48.0 * t2)) / 192.0;
    w[3] = (19.0 + xi * (44.0 + xi * (24.0 + xi * (-16.0 - 16.0 * xi)))) / 96.0;
    w[4] = b * b * b * b / 384.0;
  }
  return k - ORDER / 2;
}

template <int DIMS, int ORDER, typename R>
__global__ void k_deposit_rho(DiagParams P, const int* __restrict__ cell, const R* o0, const R* o1,
                              const R* o2, const R* q, double qc, long np, double* __restrict__ rho) {
  const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (p >= np) return;
  const int cl = cell[p];
  if (cl < 0 || cl >= P.ncell) return;
  const R* off[3] = {o0, o1, o2};
  const double qp = q ? (double)q[p] : qc;
  const uint32_t rest = P.dn0.div((uint32_t)cl);
  int c3[3];
  c3[0] = cl - (int)rest * P.n[0];
  c3[1] = DIMS == 3 ? (int)(rest - P.dn1.div(rest) * P.n[1]) : (int)rest;
  c3[2] = DIMS == 3 ? (int)P.dn1.div(rest) : 0;
  constexpr int M = ORDER + 1;
  double w[3][M];
  int b[3] = {0, 0, 0};
  for (int d = 0; d < DIMS; ++d) {
    const double o = (double)off[d][p];
    if (!(o >= 0.0 && o < 1.0)) return;
    b[d] = node_weights<ORDER>(o, w[d]);
  }
  constexpr int MZ = DIMS == 3 ? M : 1;
  for (int k = 0; k < MZ; ++k) {
    const int iz = DIMS == 3 ? axis_slot(c3[2] + b[2] + k, P.n[2], P.open[2], 0) : 0;
    if (iz < 0) continue;
    const double wz = DIMS == 3 ? w[2][k] : 1.0;
    for (int j = 0; j < M; ++j) {
      const int iy = axis_slot(c3[1] + b[1] + j, P.n[1], P.open[1], 0);
      if (iy < 0) continue;
      for (int i = 0; i < M; ++i) {
        const int ix = axis_slot(c3[0] + b[0] + i, P.n[0], P.open[0], 0);
        if (ix < 0) continue;
        atomicAdd(&rho[ix + P.n[0] * (iy + P.n[1] * iz)], qp * w[0][i] * w[1][j] * wz);
      }
    }
  }
}

// Sum over a wavefront (every lane active).
__device__ __forceinline__ double wave_sum(double v) {
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int d = 32; d > 0; d >>= 1) v = fmax(v, __shfl_xor(v, d, 64));
  return v;
}

// Kinetic energy of one particle's mass density (m = |q| / |q/m|, minv =
// 1 / |q/m|): m (gamma - 1).
__device__ __forceinline__ double kinetic(double qp, double minv, double ux, double uy, double uz) {
  return fabs(qp) * minv * (sqrt(1.0 + ux * ux + uy * uy + uz * uz) - 1.0);
}

// A workgroup's [sum m (gamma - 1), live count] to part[0], part[1].
template <int NT>
__device__ __forceinline__ void store_kinetic(double wk, double alive, double* part) {
  __shared__ double red[2][NT / 64];
  wk = wave_sum(wk);
  alive = wave_sum(alive);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = wk;
    red[1][threadIdx.x >> 6] = alive;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double v = 0.0;
    for (int w = 0; w < NT / 64; ++w) v += red[threadIdx.x][w];
    part[threadIdx.x] = v;
  }
}

// The same charge density for particles binned by the last sort, one
// workgroup per tile: the tile's charges are summed in an LDS region (the
// tile, the push's drift allowance around it and the stencil reach) with
// double-precision LDS atomics and added to rho once per region node, so
// the global atomics fall from (n+1)^D per particle to one per region node.
// Particles that drifted beyond the allowance add to rho directly.
//
// Bound by the LDS atomics, (n+1)^D per particle.  The region's strides
// agree, modulo the 16 eight-byte banks, with those by which the sort spread
// the lanes of a wavefront (dense rows and planes make them collide).  With
// part the kernel also takes the particles' kinetic energy, whose loads hide
// behind the atomics (FP32, quadratic, 10M particles on one MI355X: 179 us, the
// LDS busy 71 % of them; before 200 us and 48 us for a pass of their own).  The
// sums stay in double: as 64-bit integers on one scale they took 123 us, but a
// weight then keeps no digits of its own, and nodes at the edge of a plasma,
// which hold only small weights, were off by 1e-12 (2D quadratic) to 2e-6
// (quartic) of their charge.
struct RhoTiles {
  int ntile[3];
  const int* starts;  // tile t holds particles starts[t] .. starts[t+1]-1
};

constexpr int like_mod16(int least, int want) { return least + ((want - least) % 16 + 16) % 16; }

template <int DIMS, int ORDER, typename R>
__global__ void __launch_bounds__(256) k_rho_tile(DiagParams P, RhoTiles Tl,
                                                  const int* __restrict__ cell, const R* o0,
                                                  const R* o1, const R* o2, const R* q, double qc,
                                                  const R* u0, const R* u1, const R* u2, double minv,
                                                  double* __restrict__ rho, double* __restrict__ part) {
  using G = Geo<DIMS, ORDER, R>;
  // nodes a particle reaches relative to its cell: LO .. HI
  constexpr int LO = -(ORDER / 2), HI = ORDER / 2 + 1;
  constexpr int RX = G::T + 2 * G::A + ORDER + 1;
  constexpr int RZ = DIMS == 3 ? G::TZ + 2 * G::AZ + ORDER + 1 : 1;
  static_assert(HI - LO <= ORDER + 1, "the region holds every node a particle reaches");
  constexpr int RS = like_mod16(RX, G::sgl ? G::es : G::jb);
  constexpr int RP = DIMS == 3 ? like_mod16(RS * (RX - 1) + RX, G::sgl ? G::ep : G::jc) : RS * RX;
  __shared__ double reg[RP * RZ];
  const int t = blockIdx.x;
  const int beg = Tl.starts[t], end = Tl.starts[t + 1];
  if (beg == end) {
    if (part && threadIdx.x < 2) part[2 * (long)t + threadIdx.x] = 0.0;
    return;
  }
  const int org[3] = {(t % Tl.ntile[0]) * G::T, ((t / Tl.ntile[0]) % Tl.ntile[1]) * G::T,
                      DIMS == 3 ? (t / (Tl.ntile[0] * Tl.ntile[1])) * G::TZ : 0};
  const int rlo[3] = {org[0] - G::A + LO, org[1] - G::A + LO, DIMS == 3 ? org[2] - G::AZ + LO : 0};
  for (int r = threadIdx.x; r < RP * RZ; r += blockDim.x) reg[r] = 0.0;
  __syncthreads();
  const R* off[3] = {o0, o1, o2};
  constexpr int M = ORDER + 1;
  constexpr int MZ = DIMS == 3 ? M : 1;
  double wk = 0.0, alive = 0.0;
  for (int p = beg + threadIdx.x; p < end; p += blockDim.x) {
    const int cl = cell[p];
    const double qp = q ? (double)q[p] : qc;
    double o[3] = {0.0, 0.0, 0.0};
    for (int d = 0; d < DIMS; ++d) o[d] = (double)off[d][p];
    if (part && cl >= 0) {
      wk += kinetic(qp, minv, u0[p], u1[p], u2[p]);
      alive += 1.0;
    }
    if (cl < 0 || cl >= P.ncell) continue;
    const uint32_t rest = P.dn0.div((uint32_t)cl);
    int c3[3];
    c3[0] = cl - (int)rest * P.n[0];
    c3[1] = DIMS == 3 ? (int)(rest - P.dn1.div(rest) * P.n[1]) : (int)rest;
    c3[2] = DIMS == 3 ? (int)P.dn1.div(rest) : 0;
    double w[3][M];
    int b[3] = {0, 0, 0};
    bool ok = true;
    for (int d = 0; d < DIMS; ++d) {
      ok = ok && o[d] >= 0.0 && o[d] < 1.0;
      if (ok) b[d] = node_weights<ORDER>(o[d], w[d]);
    }
    if (!ok) continue;
    if (DIMS == 2) w[2][0] = 1.0;
    // cell relative to the tile (periodic image inside the allowance)
    int l[3] = {0, 0, 0};
    bool inside = true;
    for (int d = 0; d < DIMS; ++d) {
      const int Td = d == 2 ? G::TZ : G::T, Ad = d == 2 ? G::AZ : G::A;
      int v = c3[d] - org[d];
      if (!P.open[d]) {
        v = v < 0 ? v + P.n[d] : v;
        if (v >= Td + Ad) v -= P.n[d];
      }
      l[d] = v;
      inside = inside && v >= -Ad && v < Td + Ad;
    }
    if (inside) {
      double* at = reg + (l[0] + G::A - LO + b[0]) + (l[1] + G::A - LO + b[1]) * RS +
                   (DIMS == 3 ? (l[2] + G::AZ - LO + b[2]) * RP : 0);
#pragma unroll
      for (int k = 0; k < MZ; ++k)
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const double wjk = qp * w[1][j] * w[2][k];
#pragma unroll
          for (int i = 0; i < M; ++i) atomicAdd(at + i + j * RS + k * RP, wjk * w[0][i]);
        }
      continue;
    }
    for (int k = 0; k < MZ; ++k)
      for (int j = 0; j < M; ++j)
        for (int i = 0; i < M; ++i) {
          const int iz = DIMS == 3 ? axis_slot(c3[2] + b[2] + k, P.n[2], P.open[2], 0) : 0;
          const int iy = axis_slot(c3[1] + b[1] + j, P.n[1], P.open[1], 0);
          const int ix = axis_slot(c3[0] + b[0] + i, P.n[0], P.open[0], 0);
          if (ix >= 0 && iy >= 0 && iz >= 0)
            atomicAdd(&rho[ix + P.n[0] * (iy + P.n[1] * iz)], qp * w[0][i] * w[1][j] * w[2][k]);
        }
  }
  __syncthreads();
  for (int r = threadIdx.x; r < RX * RX * RZ; r += blockDim.x) {
    const int rx = r % RX, ry = (r / RX) % RX, rz = r / (RX * RX);
    const double v = reg[rx + ry * RS + rz * RP];
    if (v == 0.0) continue;
    const int ix = axis_slot(rlo[0] + rx, P.n[0], P.open[0], 0);
    const int iy = axis_slot(rlo[1] + ry, P.n[1], P.open[1], 0);
    const int iz = DIMS == 3 ? axis_slot(rlo[2] + rz, P.n[2], P.open[2], 0) : 0;
    if (ix >= 0 && iy >= 0 && iz >= 0) atomicAdd(&rho[ix + P.n[0] * (iy + P.n[1] * iz)], v);
  }
  if (part) store_kinetic<256>(wk, alive, part + 2 * (long)t);
}

// Per-block partials: [max|G|, max|rho|, sum C^2, max|C|, sum drho^2, sum E^2+B^2]
constexpr int NPART = 6;
__device__ __forceinline__ bool part_is_max(int k) { return k == 0 || k == 1 || k == 3; }
// Blocks of the field and (for particles without a sort's bins) particle sums
// at most: 8 and 4 workgroups per CU, each taking several cells or particles.
constexpr int FIELD_BLOCKS = 2048, PART_BLOCKS = 1024;

template <typename R>
__global__ void __launch_bounds__(256) k_diag_fields(DiagParams P, const R* E0, const R* E1, const R* E2, const R* B0,
                              const R* B1, const R* B2, const R* J0, const R* J1, const R* J2,
                              const double* __restrict__ rho, const double* __restrict__ rho_prev,
                              const double* __restrict__ gref, double* __restrict__ gout,
                              double* __restrict__ part) {
  __shared__ double red[NPART][4];
  double v[NPART] = {0, 0, 0, 0, 0, 0};
  // (unsigned: the last stride may pass 2^31)
  for (uint32_t cell = blockIdx.x * blockDim.x + threadIdx.x; cell < (uint32_t)P.ncell;
       cell += gridDim.x * blockDim.x) {
    const int idx = (int)cell;
    const uint32_t rest = P.dn0.div((uint32_t)idx);
    int L[3];
    L[0] = idx - (int)rest * P.n[0];
    L[1] = P.dims == 3 ? (int)(rest - P.dn1.div(rest) * P.n[1]) : (int)rest;
    L[2] = P.dims == 3 ? (int)P.dn1.div(rest) : 0;
    const R* E[3] = {E0, E1, E2};
    const R* B[3] = {B0, B1, B2};
    const R* J[3] = {J0, J1, J2};
    bool interior = true;
    for (int d = 0; d < P.dims; ++d)
      if (P.open[d] && (L[d] < P.margin || L[d] > P.n[d] - 1 - P.margin)) interior = false;
    // Yee divergence at the node (backward differences)
    double divE = 0.0, divJ = 0.0;
    for (int d = 0; d < P.dims; ++d) {
      int M[3] = {L[0], L[1], L[2]};
      M[d] -= 1;
      if (M[d] < 0) {
        if (P.open[d]) continue;  // not interior; value unused
        M[d] += P.n[d];
      }
      const int im = M[0] + P.n[0] * (M[1] + P.n[1] * M[2]);
      divE += ((double)E[d][idx] - (double)E[d][im]) / P.dx[d];
      divJ += ((double)J[d][idx] - (double)J[d][im]) / P.dx[d];
    }
    const double r = rho[idx];
    double G = divE - r - (gref ? gref[idx] : 0.0);
    if (gout) gout[idx] = interior ? G : 0.0;
    v[1] = fmax(v[1], fabs(r));
    if (interior) {
      v[0] = fmax(v[0], fabs(G));
      if (rho_prev) {
        const double dr = (r - rho_prev[idx]) / P.dt;
        const double C = dr + divJ;
        v[2] += C * C;
        v[3] = fmax(v[3], fabs(C));
        v[4] += dr * dr;
      }
    }
    double wf = 0.0;
    for (int c = 0; c < 3; ++c) {
      bool ie = true, ib = true;
      for (int d = 0; d < P.dims; ++d) {
        if (!P.open[d]) continue;
        if (L[d] > P.n[d] - 1 - (d == c ? 1 : 0)) ie = false;
        if (L[d] > P.n[d] - 1 - (d != c ? 1 : 0)) ib = false;
      }
      if (ie) wf += (double)E[c][idx] * (double)E[c][idx];
      if (ib) wf += (double)B[c][idx] * (double)B[c][idx];
    }
    v[5] += wf;
  }
#pragma unroll
  for (int k = 0; k < NPART; ++k) {
    v[k] = part_is_max(k) ? wave_max(v[k]) : wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
  const int k = threadIdx.x;
  if (k < NPART) {
    double t = red[k][0];
    for (int w = 1; w < 4; ++w) t = part_is_max(k) ? fmax(t, red[k][w]) : t + red[k][w];
    part[(long)blockIdx.x * NPART + k] = t;
  }
}

// Per-block partials: [sum m (gamma-1), live count]
template <typename R>
__global__ void __launch_bounds__(256) k_diag_particles(const int* __restrict__ cell, const R* u0, const R* u1,
                                 const R* u2, const R* q, double qc, double minv, long np,
                                 double* __restrict__ part) {
  double wk = 0.0, alive = 0.0;
  for (long p = blockIdx.x * (long)blockDim.x + threadIdx.x; p < np; p += (long)gridDim.x * blockDim.x) {
    if (cell[p] < 0) continue;
    wk += kinetic(q ? (double)q[p] : qc, minv, u0[p], u1[p], u2[p]);
    alive += 1.0;
  }
  store_kinetic<256>(wk, alive, part + 2 * (long)blockIdx.x);
}

// The sums over a species' partials and its status words, added to those of
// the species before it; with the field partials (nf blocks) of the first.
// One workgroup; the host then reads the one record (before: all partials,
// 0.3 MB at 1.25M cells, and the status words of each species in a copy of
// their own).
struct DiagSums {
  double field[NPART];
  double kin[2];
  unsigned long long slowpath;
  unsigned long long flags;
};
static_assert(sizeof(DiagSums) % sizeof(double) == 0, "a whole number of doubles");
constexpr int FINAL_NT = 1024;
__global__ void __launch_bounds__(FINAL_NT) k_diag_final(const double* __restrict__ fpart, int nf,
                                                         const double* __restrict__ ppart, int npp,
                                                         const DevFlags* __restrict__ flg, bool first,
                                                         DiagSums* __restrict__ out) {
  __shared__ double red[NPART + 2][FINAL_NT / 64];
  double v[NPART + 2];
#pragma unroll
  for (int k = 0; k < NPART + 2; ++k) v[k] = 0.0;
  for (int b = threadIdx.x; b < nf; b += FINAL_NT)
#pragma unroll
    for (int k = 0; k < NPART; ++k) {
      const double x = fpart[(long)b * NPART + k];
      v[k] = part_is_max(k) ? fmax(v[k], x) : v[k] + x;
    }
  for (int b = threadIdx.x; b < npp; b += FINAL_NT) {
    v[NPART] += ppart[2 * (long)b];
    v[NPART + 1] += ppart[2 * (long)b + 1];
  }
#pragma unroll
  for (int k = 0; k < NPART + 2; ++k) {
    v[k] = k < NPART && part_is_max(k) ? wave_max(v[k]) : wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
  const int k = threadIdx.x;
  if (k < NPART + 2) {
    const bool mx = k < NPART && part_is_max(k);
    double t = red[k][0];
    for (int w = 1; w < FINAL_NT / 64; ++w) t = mx ? fmax(t, red[k][w]) : t + red[k][w];
    if (k >= NPART)
      out->kin[k - NPART] = first ? t : out->kin[k - NPART] + t;
    else if (first)
      out->field[k] = t;
  }
  if (threadIdx.x == 0) {
    out->slowpath = (first ? 0ull : out->slowpath) + flg->slowpath;
    out->flags = (first ? 0ull : out->flags) | flg->flags;
  }
}

__global__ void k_fill_d(double* a, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    a[i] = 0.0;
}

static DiagParams diag_params(const pic_ctx* ctx) {
  const pic_config& c = ctx->cfg;
  DiagParams P;
  P.dims = c.dims;
  P.order = c.order;
  P.margin = 1 + c.order / 2;
  P.dV = 1.0;
  for (int d = 0; d < 3; ++d) {
    P.n[d] = d < c.dims ? c.n[d] : 1;
    P.open[d] = d < c.dims && c.bc[d] == PIC_BC_OPEN;
    P.dx[d] = c.dx[d];
    if (d < c.dims) P.dV *= c.dx[d];
  }
  P.dt = c.dt;
  P.dn0.init((uint32_t)P.n[0]);
  P.dn1.init((uint32_t)P.n[1]);
  P.ncell = P.n[0] * P.n[1] * P.n[2];
  return P;
}

// Where the tile kernel is to leave a species' kinetic partials (part null:
// not wanted).
struct KinParts {
  double minv;
  double* part;
};

template <int DIMS, int ORDER, typename R>
static void rho_t(const DiagParams& P, const pic_particles* p, double qc, double* rho,
                  const RhoTiles* tiles, int ntiles, const KinParts& kin, hipStream_t s) {
  const long np = p->np;
  if (np == 0) return;
  if (tiles) {
    k_rho_tile<DIMS, ORDER, R><<<dim3((unsigned)ntiles), dim3(256), 0, s>>>(
        P, *tiles, p->cell, (const R*)p->off[0], (const R*)p->off[1], (const R*)p->off[2],
        (const R*)p->q, qc, (const R*)p->u[0], (const R*)p->u[1], (const R*)p->u[2], kin.minv, rho,
        kin.part);
    return;
  }
  k_deposit_rho<DIMS, ORDER, R><<<dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s>>>(
      P, p->cell, (const R*)p->off[0], (const R*)p->off[1], (const R*)p->off[2], (const R*)p->q, qc,
      np, rho);
}

// The tile kernel needs the bins of a sort of these very arrays in this
// workspace (the particles may have moved since).
static bool binned(const pic_ctx* ctx, const pic_particles* p, const void* ws) {
  return ws && p->np > 0 && ctx->sorted_cell == p->cell && ctx->sorted_ws == ws &&
         ctx->sorted_np == p->np;
}

static int deposit_rho(const pic_ctx* ctx, const pic_particles* p, double* rho, void* ws,
                       hipStream_t s, bool accumulate, const KinParts& kin) {
  DiagParams P = diag_params(ctx);
  RhoTiles T;
  const bool tiled = binned(ctx, p, ws);
  if (tiled) {
    for (int d = 0; d < 3; ++d) T.ntile[d] = ctx->ntile[d];
    T.starts = (const int*)((const char*)ws + ws_layout(ctx, p->np).starts);
  }
  const RhoTiles* tiles = tiled ? &T : nullptr;
  if (!accumulate)
    k_fill_d<<<dim3((unsigned)((P.ncell + 255) / 256 < 4096 ? (P.ncell + 255) / 256 : 4096)),
               dim3(256), 0, s>>>(rho, P.ncell);
  const bool dbl = ctx->cfg.real_bytes == 8;
  const int D = P.dims, O = P.order;
  const double qc = ctx->cfg.q_const;
#define PIC_RHO(DD, OO)                                                 \
  if (D == DD && O == OO) {                                             \
    if (dbl)                                                            \
      rho_t<DD, OO, double>(P, p, qc, rho, tiles, ctx->ntiles, kin, s); \
    else                                                                \
      rho_t<DD, OO, float>(P, p, qc, rho, tiles, ctx->ntiles, kin, s);  \
  }
  PIC_RHO(2, 1) PIC_RHO(2, 2) PIC_RHO(2, 3) PIC_RHO(2, 4)
  PIC_RHO(3, 1) PIC_RHO(3, 2) PIC_RHO(3, 3) PIC_RHO(3, 4)
#undef PIC_RHO
  return (int)hipGetLastError();
}

int launch_deposit_rho(const pic_ctx* ctx, const pic_particles* p, double* rho, void* ws,
                       hipStream_t s, bool accumulate) {
  return deposit_rho(ctx, p, rho, ws, s, accumulate, KinParts{0.0, nullptr});
}

// Blocks of the field sums, and offsets (doubles) of the parts of a
// workspace's diagnostics scratch: the sums, the field partials, the
// particle partials.
static long field_blocks(long ncell) {
  const long g = (ncell + 255) / 256;
  return g < FIELD_BLOCKS ? g : FIELD_BLOCKS;
}
constexpr long SUMS_LEN = sizeof(DiagSums) / sizeof(double);

// Diagnostics of one or more species sharing the fields: rho is the sum of
// the species' charge densities; the kinetic energy sums every species'
// mass density (q over q/m) times gamma - 1.  Each species' particle
// partials go to the diagnostics scratch of its own workspace.
template <typename R>
static int diag_t(int ns, const pic_ctx* const* ctx, const pic_particles* const* p,
                  void* const* ws, const pic_fields* f, const double* rho_prev,
                  const double* gauss_ref, double* rho_out, double* gauss_out, pic_diag* out,
                  hipStream_t s) {
  DiagParams P = diag_params(ctx[0]);
  const unsigned gf = (unsigned)field_blocks(P.ncell);
  double* part0 = (double*)((char*)ws[0] + ws_layout(ctx[0], p[0]->np).diag);
  DiagSums* sums = (DiagSums*)part0;
  for (int k = 0; k < ns; ++k) {
    const double minv = 1.0 / fabs(ctx[k]->cfg.q_over_m);
    double* ppart = (double*)((char*)ws[k] + ws_layout(ctx[k], p[k]->np).diag) + SUMS_LEN +
                    (size_t)gf * NPART;
    int err = deposit_rho(ctx[k], p[k], rho_out, ws[k], s, k > 0, KinParts{minv, ppart});
    if (err) return err;
    if (!binned(ctx[k], p[k], ws[k]))
      k_diag_particles<R><<<dim3(PART_BLOCKS), dim3(256), 0, s>>>(
          p[k]->cell, (const R*)p[k]->u[0], (const R*)p[k]->u[1], (const R*)p[k]->u[2],
          (const R*)p[k]->q, ctx[k]->cfg.q_const, minv, p[k]->np, ppart);
  }
  k_diag_fields<R><<<dim3(gf), dim3(256), 0, s>>>(
      P, (const R*)f->E[0], (const R*)f->E[1], (const R*)f->E[2], (const R*)f->B[0],
      (const R*)f->B[1], (const R*)f->B[2], (const R*)f->J[0], (const R*)f->J[1],
      (const R*)f->J[2], rho_out, rho_prev, gauss_ref, gauss_out, part0 + SUMS_LEN);
  for (int k = 0; k < ns; ++k) {
    const double* ppart = (const double*)((const char*)ws[k] + ws_layout(ctx[k], p[k]->np).diag) +
                          SUMS_LEN + (size_t)gf * NPART;
    const int npp = binned(ctx[k], p[k], ws[k]) ? ctx[k]->ntiles : PART_BLOCKS;
    k_diag_final<<<dim3(1), dim3(FINAL_NT), 0, s>>>(part0 + SUMS_LEN, k == 0 ? (int)gf : 0, ppart,
                                                    npp, (const DevFlags*)ws[k], k == 0, sums);
  }
  int err = (int)hipGetLastError();
  if (err) return err;
  DiagSums h;
  if ((err = (int)hipMemcpyAsync(&h, sums, sizeof(h), hipMemcpyDeviceToHost, s))) return err;
  if ((err = (int)hipStreamSynchronize(s))) return err;
  const double gmax = h.field[0], rmax = h.field[1], c2 = h.field[2], cmax = h.field[3],
               d2 = h.field[4], wf = h.field[5];
  out->gauss_max = gmax;
  out->rho_max = rmax;
  out->gauss_rel = rmax > 0 ? gmax / rmax : 0.0;
  out->cont_max = rho_prev ? cmax : 0.0;
  out->cont_rel_l2 = (rho_prev && d2 > 0) ? sqrt(c2 / d2) : 0.0;
  out->cont_rel_inf = (rho_prev && rmax > 0) ? cmax / (rmax / P.dt) : 0.0;
  out->w_field = 0.5 * wf * P.dV;
  out->w_kin = h.kin[0] * P.dV;
  out->n_alive = (int64_t)h.kin[1];
  out->flags = (uint32_t)h.flags;
  out->n_slowpath = (int64_t)h.slowpath;
  return 0;
}

int launch_diagnostics(int ns, const pic_ctx* const* ctx, const pic_particles* const* p,
                       void* const* ws, const pic_fields* f, const double* rho_prev,
                       const double* gauss_ref, double* rho_out, double* gauss_out, pic_diag* out,
                       hipStream_t s) {
  return ctx[0]->cfg.real_bytes == 8
             ? diag_t<double>(ns, ctx, p, ws, f, rho_prev, gauss_ref, rho_out, gauss_out, out, s)
             : diag_t<float>(ns, ctx, p, ws, f, rho_prev, gauss_ref, rho_out, gauss_out, out, s);
}

long diag_len(const pic_config& cf, int ntiles) {
  long ncell = 1;
  for (int d = 0; d < cf.dims; ++d) ncell *= cf.n[d];
  return SUMS_LEN + field_blocks(ncell) * NPART + 2 * (long)(ntiles > PART_BLOCKS ? ntiles : PART_BLOCKS);
}

}  // namespace pic
