// DG stage kernels for 2D Euler on a periodic face-list mesh (static Voronoi).
//
// Same method as the Cartesian kernels (Sec. 2.2 weak form, HLL face flux,
// limiter of Sec. 2.5, SSP-RK2), on general polygons: two Gauss points per
// edge, the 4-point principal-axis volume rule (points c -+ sqrt(2 lambda_k/V)
// e_k of the second-moment matrix M, weights V/4: exact for quadratics), and
// the per-cell 2x2 inverse of M for the gradients.
//
// Work decomposition.  Cells are split into blocks of up to 256 consecutive
// indices (a space-filling-curve numbering makes a block compact).  The host
// lists, per block, its "halo" (the outside cells that share a face with it)
// and every face incident to one of its cells ("slots": faces on the block
// boundary appear in both blocks), each slot with its two cells' block-local
// indices and one geometry record (unit normal, length, face-centroid offset
// from L's centroid, offset from L's centroid to R's periodic image), and per
// cell its incidences (slot, side) with the face-centroid offset from the
// cell's own centroid.  One workgroup per block, limit on read:
//   0. the raw coefficients of the block's cells and of its halo go to LDS;
//   1. each cell of the block is limited from its neighbours' means in LDS and
//      its incidences' face-centroid offsets; each halo cell from the global
//      face lists (its neighbours' means gathered); the limited gradients
//      replace the raw ones in LDS;
//   2. the slots' Riemann problems (HLL at both Gauss points, which sit at the
//      face centroid -+ A/(2 sqrt 3) along the tangent) go to an LDS table as
//      the weighted sum and half-difference of the two fluxes and A n, half
//      the slots at a time;
//   3. each cell gathers its incidences from that table (a segmented
//      reduction, no atomics);
//   4. the volume term, M^-1 and the RK combination (stage 2 takes Pi(U^n),
//      which stage 1 wrote, for the combination).
// Loads of later phases that depend on nothing the block computes (incidence
// ranges and entries, geometry, Pi(U^n), the first pass's slots) are issued
// before the first barrier, so that their latency overlaps phase 0.
// A stand-alone limiter kernel (k_fl_lim) serves dg_limit.  The discrete
// adjoint of a step sweeps the same blocks (k_adjfl_L, k_adjfl_msg) and transposes the
// limiter over the global incidence lists.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "dg_internal.h"
#include "dg_math.h"

namespace dg {

// Device arrays of a face-list mesh (allocated at create, in the mesh's
// working precision for geometry).
struct FLDev {
  int ncells, nblocks, max_slots;
  int64_t ninc;       // incidences of the global CSR (2 x faces)
  int* blk_cell0;     // [nblocks+1] first cell of each block
  int* blk_slot0;     // [nblocks+1] first slot of each block
  int* blk_halo0;     // [nblocks+1] first halo entry of each block
  int* halo_cell;     // global index of each halo cell
  int* slot_lr;       // [nslots] block-local L | R << 16 (own cell i: i; halo h: nown + h)
  void* slot_geo;     // [nslots][8] nx, ny, A, x_f - c_L (2), c_R' - c_L (2), 0
  int* cell_inc0;     // [ncells+1] block-local CSR start (global index into cell_inc)
  int* cell_inc;      // slot_local*2 + side | neighbour's block-local index << 16,
                      // each cell's incidences by slot
  void* inc_rf;       // [per cell_inc entry][2] face centroid - the cell's own centroid
  void* cell_geo;     // [ncells][8] 1/V, V Minv00, V Minv01, V Minv11, a1x, a1y, a2x, a2y
  int* lim_inc0;      // [ncells+1] global CSR for k_fl_lim, halo cells and the CFL bound
  int* lim_nbr;       // neighbour cell of each incidence
  void* lim_geo;      // [ninc][2] face-centroid offsets, then [ninc][2] A n outward
  void* cell_perim;   // [ncells] sum of face lengths
  // the discrete adjoint (its limiter gathers over the global CSR)
  int* inc_face;      // [ninc] face id << 1 | side (0: the cell is L) of each incidence
};

namespace {

constexpr int kBlock = 256;      // cells of a block at most (one thread each)
constexpr int kMaxSlots = 1024;  // distinct faces of a block
constexpr int kMaxHalo = 128;    // outside neighbours of a block
constexpr int kHalf = 512;       // slots per pass of the LDS flux table
constexpr int kLocal = kBlock + kMaxHalo;

template <typename T>
struct PF {
  const T* __restrict__ in;
  const T* __restrict__ ua;
  T* __restrict__ out;
  T* __restrict__ lim_out;  // stage 1: Pi(in) of each cell (NULL: not kept)
  const double* dt_dev;
  double dt_host;
  int* status;
  double* dtpart;
  int ncells, nc;
  T gamma;
  const int* blk_cell0;
  const int* blk_slot0;
  const int* blk_halo0;
  const int* halo_cell;
  const int* slot_lr;
  const T* slot_geo;
  const int* cell_inc0;
  const int* cell_inc;
  const T* inc_rf;
  const T* cell_geo;
  const int* lim_inc0;
  const int* lim_nbr;
  const T* lim_geo;  // face-centroid offsets (the limiter)
  const T* lim_an;   // A n outward (the CFL bound)
  const T* perim;
};

template <typename T>
__device__ __forceinline__ void load12(const T* __restrict__ U, int nc, int e, T* q) {
#pragma unroll
  for (int k = 0; k < 12; ++k) q[k] = U[k * nc + e];
}

// HLL flux along the unit normal n (Davis speeds), F = a F_L + b F_R + c dU.
template <typename T>
__device__ __forceinline__ void hll_n(const T* uL, const T* uR, T nx, T ny, T gamma, T* F,
                                      bool& bad) {
  const T gm1 = gamma - T(1);
  T irL = rcp(uL[0]), irR = rcp(uR[0]);
  T vxL = uL[1] * irL, vyL = uL[2] * irL, vxR = uR[1] * irR, vyR = uR[2] * irR;
  T pL = gm1 * (uL[3] - T(0.5) * (uL[1] * vxL + uL[2] * vyL));
  T pR = gm1 * (uR[3] - T(0.5) * (uR[1] * vxR + uR[2] * vyR));
  bad |= !(uL[0] > T(0)) || !(uR[0] > T(0)) || !(pL > T(0)) || !(pR > T(0));
  T cL = sqrt_pos(gamma * pL * irL), cR = sqrt_pos(gamma * pR * irR);
  T vnL = vxL * nx + vyL * ny, vnR = vxR * nx + vyR * ny;
  T SL = fmin(vnL - cL, vnR - cR), SR = fmax(vnL + cL, vnR + cR);
  T FL[4] = {uL[0] * vnL, uL[1] * vnL + pL * nx, uL[2] * vnL + pL * ny, (uL[3] + pL) * vnL};
  T FR[4] = {uR[0] * vnR, uR[1] * vnR + pR * nx, uR[2] * vnR + pR * ny, (uR[3] + pR) * vnR};
  T inv = rcp(SR - SL);
  T a = SR * inv, b = -SL * inv, c = SL * SR * inv;
  const bool left = SL >= T(0), right = SR <= T(0);
  a = left ? T(1) : (right ? T(0) : a);
  b = left ? T(0) : (right ? T(1) : b);
  c = (left || right) ? T(0) : c;
#pragma unroll
  for (int k = 0; k < 4; ++k) F[k] = fma(a, FL[k], fma(b, FR[k], c * (uR[k] - uL[k])));
}

// ------------------------------------------------------------- limiter --
template <typename T>
__global__ __launch_bounds__(256) void k_fl_lim(PF<T> p) {
  // blocks mapped XCD by XCD: neighbouring blocks (Morton-ordered cells) share
  // their neighbours' means in the same L2
  const int e = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (e >= p.ncells) return;
  T q[12];
  load12(p.in, p.nc, e, q);
  T hi[4], lo[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) hi[v] = lo[v] = q[3 * v];
  // Incidences are taken kBatch at a time, every load of a batch issued before
  // any is used (a per-incidence loop waits out one gather chain per face);
  // padding slots repeat the cell itself, which changes no max, min or bound.
  constexpr int kBatch = 8;
  const int i0 = p.lim_inc0[e], i1 = p.lim_inc0[e + 1];
  for (int b0 = i0; b0 < i1; b0 += kBatch) {
    int nb[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) nb[u] = b0 + u < i1 ? p.lim_nbr[b0 + u] : e;
    T m[kBatch][4];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[u][v] = p.in[(3 * v) * p.nc + nb[u]];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        hi[v] = fmax(hi[v], m[u][v]);
        lo[v] = fmin(lo[v], m[u][v]);
      }
  }
  T alpha[4] = {T(1), T(1), T(1), T(1)};
  for (int b0 = i0; b0 < i1; b0 += kBatch) {
    T rx[kBatch], ry[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = b0 + u < i1 ? b0 + u : b0;
      rx[u] = p.lim_geo[2 * i];
      ry[u] = p.lim_geo[2 * i + 1];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T d = q[3 * v + 1] * rx[u] + q[3 * v + 2] * ry[u];
        // psi = (max - phi)/d for d > 0, (min - phi)/d for d < 0, 1 for d = 0
        const T num = d > T(0) ? hi[v] - q[3 * v] : lo[v] - q[3 * v];
        const T psi = d > T(0) ? div_small(num, d) : (d < T(0) ? div_small(-num, -d) : T(1));
        alpha[v] = fmin(alpha[v], psi);
      }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    p.out[(3 * v) * p.nc + e] = q[3 * v];
    p.out[(3 * v + 1) * p.nc + e] = alpha[v] * q[3 * v + 1];
    p.out[(3 * v + 2) * p.nc + e] = alpha[v] * q[3 * v + 2];
  }
}

// ------------------------------------------------------------ stage --
// alpha = min(1, min_f psi_f) of one conserved variable (Sec. 2.5): psi from
// the face-centroid increment d = g . (x_f - c) and the bounds hi, lo of the
// means of the cell and its face neighbours.
template <typename T>
__device__ __forceinline__ T psi_of(T d, T phi, T hi, T lo) {
  const T num = d > T(0) ? hi - phi : lo - phi;
  return d > T(0) ? div_small(num, d) : (d < T(0) ? div_small(-num, -d) : T(1));
}

// Limit the gradients of q (12 coefficients, means untouched) of a block cell
// whose incidences are [i0, i1) of the block-local CSR, from the block-local
// means m[v][local] in LDS.  Incidences are taken kInc at a time with all
// their loads in flight; padding entries repeat the cell itself (no change to
// a bound, psi = 1).
constexpr int kInc = 4;
constexpr int kPre = 2 * kInc;  // incidences of a cell loaded ahead (two batches)

// Incidence i's entries of the block-local CSR for the batch starting at b0
// (padding repeats the batch's first entry, a batch past the end the cell's
// first, so every index stays inside the cell's list).  Only the entries are
// loaded ahead; the offsets of the alpha pass are loaded where they are used,
// with nothing they wait on.
__device__ __forceinline__ int batch_index(int b0, int u, int i0, int i1) {
  return b0 + u < i1 ? b0 + u : (b0 < i1 ? b0 : i0);
}

struct IncPre {  // a cell's first kPre incidences, loaded before the block's first barrier
  int inc[kPre];
};

template <typename T>
__device__ __forceinline__ void load_inc_pre(const PF<T>& p, int i0, int i1, IncPre& a) {
#pragma unroll
  for (int u = 0; u < kPre; ++u)
    a.inc[u] = p.cell_inc[batch_index(i0 + (u / kInc) * kInc, u % kInc, i0, i1)];
}

template <typename T>
__device__ __forceinline__ void limit_block_cell(const PF<T>& p, int i0, int i1, int self,
                                                 const T (*m)[kLocal], T* q,
                                                 const IncPre& pre) {
  T hi[4], lo[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) hi[v] = lo[v] = q[3 * v];
  T alpha[4] = {T(1), T(1), T(1), T(1)};
  auto bound = [&](int nbu) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const T mm = m[3 * v][nbu];
      hi[v] = fmax(hi[v], mm);
      lo[v] = fmin(lo[v], mm);
    }
  };
  auto limit_by = [&](T rx, T ry) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      alpha[v] = fmin(alpha[v], psi_of(q[3 * v + 1] * rx + q[3 * v + 2] * ry, q[3 * v],
                                       hi[v], lo[v]));
  };
  // batches of kInc in incidence order, the first two from registers
#pragma unroll
  for (int u = 0; u < kPre; ++u) {
    const int b0 = i0 + (u / kInc) * kInc;
    if (b0 < i1) bound(b0 + u % kInc < i1 ? (pre.inc[u] >> 16) : self);
  }
  for (int b0 = i0 + kPre; b0 < i1; b0 += kInc) {
    int nb[kInc];
#pragma unroll
    for (int u = 0; u < kInc; ++u) nb[u] = b0 + u < i1 ? (p.cell_inc[b0 + u] >> 16) : self;
#pragma unroll
    for (int u = 0; u < kInc; ++u) bound(nb[u]);
  }
  for (int b0 = i0; b0 < i1; b0 += kInc) {
    T rx[kInc], ry[kInc];
#pragma unroll
    for (int u = 0; u < kInc; ++u) {
      const int i = b0 + u < i1 ? b0 + u : b0;
      rx[u] = p.inc_rf[2 * (size_t)i];
      ry[u] = p.inc_rf[2 * (size_t)i + 1];
    }
#pragma unroll
    for (int u = 0; u < kInc; ++u) limit_by(rx[u], ry[u]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    q[3 * v + 1] *= alpha[v];
    q[3 * v + 2] *= alpha[v];
  }
}

// The same limiter for a cell outside the block (a halo cell) from the global
// face lists: neighbour means gathered from `U`, eight incidences at a time
// with all their loads in flight (padding repeats the cell itself).  The
// cell's incidence range and first eight neighbours come preloaded.
constexpr int kHB = 8;
struct HaloPre {
  int i0, i1;
  int nb[kHB];
};

template <typename T>
__device__ __forceinline__ void load_halo_pre(const PF<T>& p, int e, HaloPre& a) {
  a.i0 = p.lim_inc0[e];
  a.i1 = p.lim_inc0[e + 1];
#pragma unroll
  for (int u = 0; u < kHB; ++u) a.nb[u] = a.i0 + u < a.i1 ? p.lim_nbr[a.i0 + u] : e;
}

template <typename T>
__device__ __forceinline__ void limit_global_cell(const PF<T>& p, const T* __restrict__ U, int e,
                                                  T* q, const HaloPre& pre) {
  T hi[4], lo[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) hi[v] = lo[v] = q[3 * v];
  const int i0 = pre.i0, i1 = pre.i1;
  auto bounds = [&](const int* nb) {
    T m[kHB][4];
#pragma unroll
    for (int u = 0; u < kHB; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[u][v] = U[(3 * v) * p.nc + nb[u]];
#pragma unroll
    for (int u = 0; u < kHB; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        hi[v] = fmax(hi[v], m[u][v]);
        lo[v] = fmin(lo[v], m[u][v]);
      }
  };
  T alpha[4] = {T(1), T(1), T(1), T(1)};
  auto limit_by = [&](const T* rx, const T* ry) {
#pragma unroll
    for (int u = 0; u < kHB; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        alpha[v] = fmin(alpha[v], psi_of(q[3 * v + 1] * rx[u] + q[3 * v + 2] * ry[u], q[3 * v],
                                         hi[v], lo[v]));
  };
  if (i0 < i1) bounds(pre.nb);
  for (int b0 = i0 + kHB; b0 < i1; b0 += kHB) {
    int nb[kHB];
#pragma unroll
    for (int u = 0; u < kHB; ++u) nb[u] = b0 + u < i1 ? p.lim_nbr[b0 + u] : e;
    bounds(nb);
  }
  for (int b0 = i0; b0 < i1; b0 += kHB) {
    T rx[kHB], ry[kHB];
#pragma unroll
    for (int u = 0; u < kHB; ++u) {
      const int i = b0 + u < i1 ? b0 + u : b0;
      rx[u] = p.lim_geo[2 * i];
      ry[u] = p.lim_geo[2 * i + 1];
    }
    limit_by(rx, ry);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    q[3 * v + 1] *= alpha[v];
    q[3 * v + 2] *= alpha[v];
  }
}

// One stage (MODE kRhs, kStage1, kStage2) of a block of cells; LIM: limit on
// read (Pi of `in`, and in stage 2 Pi of `ua` for the combination).
template <typename T, int MODE, bool LIM>
__global__ __launch_bounds__(kBlock) void k_fl_step(PF<T> p) {
  __shared__ T cU[12][kLocal];  // coefficients of the block's and the halo's cells
  __shared__ T sF[10][kHalf];   // per slot: w (F0 + F1), w (F1 - F0)/2, A n
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int tid = threadIdx.x;
  const int c0 = p.blk_cell0[b], nown = p.blk_cell0[b + 1] - c0;
  const int h0 = p.blk_halo0[b], nhalo = p.blk_halo0[b + 1] - h0;
  const int s0 = p.blk_slot0[b], nslot = p.blk_slot0[b + 1] - s0;
  const int nc = p.nc;
  bool bad = false;
  const int e = c0 + tid;
  // Loads that later phases need, issued before the first barrier so that
  // their latency overlaps phase 0 (the LDS sets the occupancy, two
  // workgroups per CU, so these registers cost none): the cell's incidence
  // range, first incidences, geometry and (stage 2) Pi(U^n) row; the halo
  // cell's first neighbours; this thread's slots of the first flux pass.
  int i0 = 0, i1 = 0;
  T cg[8], ua[12];
  IncPre ipre;
  HaloPre hpre;
  int f0 = 0, f1 = 0;  // stage 2's CFL bound: the cell's global incidence range
  if (tid < nown) {
    i0 = p.cell_inc0[e];
    i1 = p.cell_inc0[e + 1];
#pragma unroll
    for (int k = 0; k < 8; ++k) cg[k] = p.cell_geo[8 * (size_t)e + k];
    if (MODE == kStage2) {
      load12(p.ua, nc, e, ua);
      if (p.dtpart) {
        f0 = p.lim_inc0[e];
        f1 = p.lim_inc0[e + 1];
      }
    }
  }
  int hg = 0;
  if (LIM && tid < nhalo) {
    hg = p.halo_cell[h0 + tid];
    load_halo_pre(p, hg, hpre);
  }
  if (LIM && tid < nown) load_inc_pre(p, i0, i1, ipre);
  constexpr int kSP = kHalf / kBlock;  // slots per thread and flux pass
  int slr[kSP];
  T sgeo[kSP][7];
#pragma unroll
  for (int j = 0; j < kSP; ++j) {
    const int sl = tid + j * kBlock;
    if (sl < min(nslot, kHalf)) {
      slr[j] = p.slot_lr[s0 + sl];
#pragma unroll
      for (int k = 0; k < 7; ++k) sgeo[j][k] = p.slot_geo[8 * (size_t)(s0 + sl) + k];
    }
  }
  // 0. raw coefficients of the block's cells and its halo
  for (int i = tid; i < nown + nhalo; i += kBlock) {
    const int g = i < nown ? c0 + i : p.halo_cell[h0 + i - nown];
#pragma unroll
    for (int k = 0; k < 12; ++k) cU[k][i] = p.in[k * nc + g];
  }
  __syncthreads();
  // 1. limit on read (the limiter reads only means; only gradients change)
  T q[12];
  if (tid < nown) {
#pragma unroll
    for (int k = 0; k < 12; ++k) q[k] = cU[k][tid];
  }
  if (LIM) {
    T qh[12];
    if (tid < nhalo) {
#pragma unroll
      for (int k = 0; k < 12; ++k) qh[k] = cU[k][nown + tid];
      limit_global_cell(p, p.in, hg, qh, hpre);
    }
    if (tid < nown) {
      limit_block_cell(p, i0, i1, tid, cU, q, ipre);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        cU[3 * v + 1][tid] = q[3 * v + 1];
        cU[3 * v + 2][tid] = q[3 * v + 2];
      }
      // stage 1 hands Pi(U^n) of its cells to stage 2's combination
      if (MODE == kStage1 && p.lim_out) {
#pragma unroll
        for (int k = 0; k < 12; ++k) p.lim_out[k * nc + e] = q[k];
      }
    }
    if (tid < nhalo) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        cU[3 * v + 1][nown + tid] = qh[3 * v + 1];
        cU[3 * v + 2][nown + tid] = qh[3 * v + 2];
      }
    }
    __syncthreads();
  }
  // 2-3. slot fluxes into LDS, half the slots at a time; each cell gathers its
  // incidences of the half (they are sorted by slot)
  T rm[4] = {T(0), T(0), T(0), T(0)};
  T rx[4] = {T(0), T(0), T(0), T(0)};
  T ry[4] = {T(0), T(0), T(0), T(0)};
  const T is3 = T(0.57735026918962576451);  // 1/sqrt(3)
  int ii = i0;
  for (int sa = 0; sa < nslot; sa += kHalf) {
    const int sb = min(nslot, sa + kHalf);
#pragma unroll
    for (int j = 0; j < kSP; ++j) {
      const int sl = sa + tid + j * kBlock;
      if (sl >= sb) break;
      int lr;
      T g[7];
      if (sa == 0) {
        lr = slr[j];
#pragma unroll
        for (int k = 0; k < 7; ++k) g[k] = sgeo[j][k];
      } else {
        lr = p.slot_lr[s0 + sl];
#pragma unroll
        for (int k = 0; k < 7; ++k) g[k] = p.slot_geo[8 * (size_t)(s0 + sl) + k];
      }
      const int L = lr & 0xffff, R = lr >> 16;
      const T nx = g[0], ny = g[1], A = g[2], fx = g[3], fy = g[4], dx = g[5], dy = g[6];
      // Gauss points x_f -+ A/(2 sqrt 3) t, t = (-n_y, n_x), from L's centroid
      const T o = T(0.5) * A * is3;
      const T tx = -ny * o, ty = nx * o;
      T uL[4], uR[4], F0[4], F1[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T gLx = cU[3 * v + 1][L], gLy = cU[3 * v + 2][L];
        const T gRx = cU[3 * v + 1][R], gRy = cU[3 * v + 2][R];
        uL[v] = cU[3 * v][L] + gLx * (fx - tx) + gLy * (fy - ty);
        uR[v] = cU[3 * v][R] + gRx * (fx - tx - dx) + gRy * (fy - ty - dy);
      }
      hll_n(uL, uR, nx, ny, p.gamma, F0, bad);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T gLx = cU[3 * v + 1][L], gLy = cU[3 * v + 2][L];
        const T gRx = cU[3 * v + 1][R], gRy = cU[3 * v + 2][R];
        uL[v] = cU[3 * v][L] + gLx * (fx + tx) + gLy * (fy + ty);
        uR[v] = cU[3 * v][R] + gRx * (fx + tx - dx) + gRy * (fy + ty - dy);
      }
      hll_n(uL, uR, nx, ny, p.gamma, F1, bad);
      const T w = T(0.5) * A;
      const int ls = sl - sa;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sF[v][ls] = w * (F0[v] + F1[v]);
        sF[4 + v][ls] = T(0.5) * w * (F1[v] - F0[v]);
      }
      sF[8][ls] = A * nx;
      sF[9][ls] = A * ny;
    }
    __syncthreads();
    if (tid < nown) {
      // side 0 (L) takes -flux, side 1 (R) +flux; the Gauss-point offsets
      // from the cell's centroid are r_f -+ delta/2, delta = (A/sqrt3) t.
      // The half's incidences (sorted by slot) kInc at a time, loads first;
      // the first incidence of a later half ends the pass.
      bool stop = false;
      while (!stop && ii < i1) {
        int inc[kInc];
        T fx[kInc], fy[kInc];
#pragma unroll
        for (int u = 0; u < kInc; ++u) {
          const int i = ii + u < i1 ? ii + u : ii;
          inc[u] = p.cell_inc[i];
          fx[u] = p.inc_rf[2 * (size_t)i];
          fy[u] = p.inc_rf[2 * (size_t)i + 1];
        }
        int done = 0;
#pragma unroll
        for (int u = 0; u < kInc; ++u) {
          const int ls = ((inc[u] & 0xffff) >> 1) - sa;
          if (stop || ii + u >= i1 || ls >= kHalf) {
            stop = true;
            continue;
          }
          const T sg = (inc[u] & 1) ? T(1) : T(-1);
          const T Anx = sF[8][ls], Any = sF[9][ls];
          const T ddx = -Any * is3, ddy = Anx * is3;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const T G = sg * sF[v][ls], K = sg * sF[4 + v][ls];
            rm[v] += G;
            rx[v] += fma(G, fx[u], K * ddx);
            ry[v] += fma(G, fy[u], K * ddy);
          }
          ++done;
        }
        ii += done;
      }
    }
    if (sb < nslot) __syncthreads();  // the next half overwrites the table
  }
  // 4. volume term, M^-1, RK combination
  double dtmin = 1e300;
  if (tid < nown) {
    const T iV = cg[0];
    const T m00 = cg[1], m01 = cg[2], m11 = cg[3];
    // volume term: 4 principal-axis points, weights V/4 (the 1/V of the
    // inverse mass matrix is folded in)
    T vx[4] = {T(0), T(0), T(0), T(0)}, vy[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const T sgn = (k & 1) ? T(1) : T(-1);
      const T ox = sgn * ((k & 2) ? cg[6] : cg[4]);
      const T oy = sgn * ((k & 2) ? cg[7] : cg[5]);
      T u[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) u[v] = fma(q[3 * v + 1], ox, fma(q[3 * v + 2], oy, q[3 * v]));
      const T ir = rcp(u[0]);
      const T ux = u[1] * ir, uy = u[2] * ir;
      const T pr = (p.gamma - T(1)) * (u[3] - T(0.5) * (u[1] * ux + u[2] * uy));
      bad |= !(u[0] > T(0)) || !(pr > T(0));
      vx[0] += u[1];
      vx[1] += u[1] * ux + pr;
      vx[2] += u[2] * ux;
      vx[3] += (u[3] + pr) * ux;
      vy[0] += u[2];
      vy[1] += u[1] * uy;
      vy[2] += u[2] * uy + pr;
      vy[3] += (u[3] + pr) * uy;
    }
    T d[12];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const T gx = rx[v] * iV + T(0.25) * vx[v];
      const T gy = ry[v] * iV + T(0.25) * vy[v];
      d[3 * v] = rm[v] * iV;
      d[3 * v + 1] = m00 * gx + m01 * gy;
      d[3 * v + 2] = m01 * gx + m11 * gy;
    }
    T o[12];
    if (MODE == kRhs) {
#pragma unroll
      for (int k = 0; k < 12; ++k) o[k] = d[k];
    } else {
      const T dt = (T)(p.dt_dev ? *p.dt_dev : p.dt_host);
#pragma unroll
      for (int k = 0; k < 12; ++k) o[k] = fma(dt, d[k], q[k]);
      if (MODE == kStage2) {
        // ua: Pi(U^n) (written by stage 1 of the same U^n, or by the
        // stand-alone limiter), U^n itself without a limiter
#pragma unroll
        for (int k = 0; k < 12; ++k) o[k] = T(0.5) * (ua[k] + o[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) p.out[k * nc + e] = o[k];
    if (MODE == kStage2 && p.dtpart) {
      // CFL bound 2V / sum_f A (|v.n| + c) from the new means
      const double r = o[0], ir = 1.0 / r, ux = o[3] * ir, uy = o[6] * ir;
      const double pr = ((double)p.gamma - 1.0) * (o[9] - 0.5 * r * (ux * ux + uy * uy));
      const double cs = sqrt((double)p.gamma * pr * ir);
      double s = cs * (double)p.perim[e];
      for (int i = f0; i < f1; ++i)
        s += fabs(ux * (double)p.lim_an[2 * i] + uy * (double)p.lim_an[2 * i + 1]);
      dtmin = 2.0 / ((double)iV * s);
    }
  }
  if (bad) atomicOr(p.status, 1);
  if (MODE == kStage2 && p.dtpart) {
    dtmin = wave_min(dtmin);
    __shared__ double sd[kBlock / 64];
    if ((tid & 63) == 0) sd[tid >> 6] = dtmin;
    __syncthreads();
    if (tid == 0) {
      double m = sd[0];
      for (int w = 1; w < kBlock / 64; ++w) m = fmin(m, sd[w]);
      p.dtpart[b] = m;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_fl_cfl(PF<T> p) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  double d = 1e300;
  if (e < p.ncells) {
    const double r = p.in[e], ir = 1.0 / r, ux = p.in[3 * p.nc + e] * ir,
                 uy = p.in[6 * p.nc + e] * ir;
    const double pr =
        ((double)p.gamma - 1.0) * (p.in[9 * p.nc + e] - 0.5 * r * (ux * ux + uy * uy));
    const double cs = sqrt((double)p.gamma * pr * ir);
    double s = cs * (double)p.perim[e];
    for (int i = p.lim_inc0[e]; i < p.lim_inc0[e + 1]; ++i)
      s += fabs(ux * (double)p.lim_an[2 * i] + uy * (double)p.lim_an[2 * i + 1]);
    d = 2.0 / ((double)p.cell_geo[8 * (size_t)e] * s);
  }
  d = wave_min(d);
  if ((threadIdx.x & 63) == 0) p.dtpart[e >> 6] = d;
}

template <typename T>
PF<T> make_params(const dg_mesh* m, const void* in, const void* ua, void* out,
                  const double* dt_dev, double dt_host) {
  const FLDev& f = *m->fld;
  PF<T> p;
  p.in = static_cast<const T*>(in);
  p.ua = static_cast<const T*>(ua);
  p.out = static_cast<T*>(out);
  p.lim_out = nullptr;
  p.dt_dev = dt_dev;
  p.dt_host = dt_host;
  p.status = m->status;
  p.dtpart = nullptr;
  p.ncells = f.ncells;
  p.nc = f.ncells;
  p.gamma = (T)m->cfg.gamma;
  p.blk_cell0 = f.blk_cell0;
  p.blk_slot0 = f.blk_slot0;
  p.blk_halo0 = f.blk_halo0;
  p.halo_cell = f.halo_cell;
  p.slot_lr = f.slot_lr;
  p.slot_geo = static_cast<const T*>(f.slot_geo);
  p.cell_inc0 = f.cell_inc0;
  p.cell_inc = f.cell_inc;
  p.inc_rf = static_cast<const T*>(f.inc_rf);
  p.cell_geo = static_cast<const T*>(f.cell_geo);
  p.lim_inc0 = f.lim_inc0;
  p.lim_nbr = f.lim_nbr;
  p.lim_geo = static_cast<const T*>(f.lim_geo);
  p.lim_an = p.lim_geo + 2 * f.ninc;
  p.perim = static_cast<const T*>(f.cell_perim);
  return p;
}

template <typename T>
hipError_t lim_t(const dg_mesh* m, const void* in, void* out, hipStream_t s) {
  PF<T> p = make_params<T>(m, in, nullptr, out, nullptr, 0.0);
  hipLaunchKernelGGL((k_fl_lim<T>), dim3((p.ncells + 255) / 256), dim3(256), 0, s, p);
  return hipGetLastError();
}

template <typename T>
hipError_t step_t(const dg_mesh* m, int mode, const void* in, const void* ua, void* out,
                  void* lim_out, const double* dt_dev, double dt_host, bool want_dt,
                  hipStream_t s) {
  PF<T> p = make_params<T>(m, in, ua, out, dt_dev, dt_host);
  p.lim_out = static_cast<T*>(lim_out);
  if (want_dt) p.dtpart = m->dtpart;
  const dim3 g(m->fld->nblocks), b(kBlock);
  const bool lim = m->cfg.limiter == DG_LIMITER_MINMOD;
  switch (mode) {
    case kRhs:
      hipLaunchKernelGGL((k_fl_step<T, kRhs, false>), g, b, 0, s, p);
      break;
    case kStage1:
      if (lim)
        hipLaunchKernelGGL((k_fl_step<T, kStage1, true>), g, b, 0, s, p);
      else
        hipLaunchKernelGGL((k_fl_step<T, kStage1, false>), g, b, 0, s, p);
      break;
    case kStage2:
      if (lim)
        hipLaunchKernelGGL((k_fl_step<T, kStage2, true>), g, b, 0, s, p);
      else
        hipLaunchKernelGGL((k_fl_step<T, kStage2, false>), g, b, 0, s, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t cfl_t(const dg_mesh* m, const void* U, hipStream_t s) {
  PF<T> p = make_params<T>(m, U, nullptr, nullptr, nullptr, 0.0);
  p.dtpart = m->dtpart;
  hipLaunchKernelGGL((k_fl_cfl<T>), dim3((p.ncells + 255) / 256), dim3(256), 0, s, p);
  return hipGetLastError();
}

// ------------------------------------------------------- discrete adjoint --
// Adjoint of a stage (as for the Cartesian meshes):
//   out = Pi_P^T lamW,   lamW = c_id lam + c_L (dL/dW)^T lam + c_extra extra,
// W = Pi(P), the branch the forward step takes (dt frozen).  k_adjfl_L computes
// lamW block by block from the faces and the cells' volume points, applies the
// transpose of each cell's own limiter and leaves a message for the one neighbour
// whose mean set a bound; k_adjfl_msg adds each cell's messages.  No atomics; the
// flux Jacobians come from one reverse sweep per Gauss point (hll_n_vjp), the linear
// parts (Gauss-point extrapolation, residual weights, M^-1) are transposed by hand.
// Measured (262144 cells, FP64, one adjoint stage): k_adjfl_L 0.100 ms, bound by the
// latency of its loads, and k_adjfl_msg 0.017 ms (gathers).  With the limiter's part
// as a kernel of its own 0.076 + 0.046 ms (0.034 with four incidences in flight,
// which fit two waves per SIMD, instead of eight); the sweep as one workgroup per CU
// with separate tables 0.093 in place of 0.076, as a thread per cell that sweeps its
// faces from gathered neighbours 0.134 (0.107 in XCD order with two waves per SIMD).
// The adjoint step 0.42 -> 0.28 ms.
template <typename T>
struct PFA {
  const T* W;      // Pi(P)
  const T* P;      // the stage input (limit_transpose)
  const T* lam;    // adjoint of the stage output
  const T* extra;  // added to lamW with weight c_extra (may be NULL)
  T* out;
  T* msg;          // limiter messages: 4 values a cell
  int* to;         // and the incidences they go through
  const double* dt_dev;
  double dt_host;
  double c_id, c_L_over_dt, c_extra;
  int nc;
  T gamma;
  const int* inc0;
  const int* nbr;
  const int* inc_face;
  const T* lim_geo;
  const T* cell_geo;
  // the blocks (k_adjfl_L)
  const int* blk_cell0;
  const int* blk_slot0;
  const int* blk_halo0;
  const int* halo_cell;
  const int* slot_lr;
  const T* slot_geo;
  const int* cell_inc0;
  const int* cell_inc;
};

// Cotangents of a cell's residual sums from the adjoint of its time
// derivative: d mean = rm / V, d grad = (V M^-1) (r / V + vol / 4), with r the
// face moments sum_g w F_g (x_g - c) and vol the sums of the volume fluxes.
template <typename T>
struct Cot {
  T rm[4], rx[4], ry[4], vx[4], vy[4];
};

template <typename T>
__device__ __forceinline__ void cotangents(const T* lam, const T* cg, Cot<T>& c) {
  const T iV = cg[0], m00 = cg[1], m01 = cg[2], m11 = cg[3];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const T gx = fma(m00, lam[3 * v + 1], m01 * lam[3 * v + 2]);
    const T gy = fma(m01, lam[3 * v + 1], m11 * lam[3 * v + 2]);
    c.rm[v] = iV * lam[3 * v];
    c.rx[v] = iV * gx;
    c.ry[v] = iV * gy;
    c.vx[v] = T(0.25) * gx;
    c.vy[v] = T(0.25) * gy;
  }
}

// Vector-Jacobian product of hll_n: uLb and uRb are the cotangents of the two
// states from the flux cotangent Fb, in one reverse sweep.  S_L and S_R take the
// left state on ties, as hll_n's min and max do.
template <typename T>
__device__ __forceinline__ void hll_n_vjp(const T* uL, const T* uR, T nx, T ny, T gamma,
                                          const T* Fb, T* uLb, T* uRb) {
  const T gm1 = gamma - T(1);
  T ir[2], vx[2], vy[2], p[2], c[2], vn[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const T* u = s == 0 ? uL : uR;
    ir[s] = rcp(u[0]);
    vx[s] = u[1] * ir[s];
    vy[s] = u[2] * ir[s];
    p[s] = gm1 * (u[3] - T(0.5) * (u[1] * vx[s] + u[2] * vy[s]));
    c[s] = sqrt_pos(gamma * p[s] * ir[s]);
    vn[s] = vx[s] * nx + vy[s] * ny;
  }
  const T l0 = vn[0] - c[0], l1 = vn[1] - c[1], r0 = vn[0] + c[0], r1 = vn[1] + c[1];
  const bool loR = l1 < l0, hiR = r1 > r0;
  const T SL = loR ? l1 : l0, SR = hiR ? r1 : r0;
  const T inv = rcp(SR - SL);
  const bool left = SL >= T(0), right = SR <= T(0), fan = !left && !right;
  // Fb . F_L, Fb . F_R, Fb . (u_R - u_L)
  const T g0 = Fb[1] * nx + Fb[2] * ny;
  T dot[2], D = T(0);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const T* u = s == 0 ? uL : uR;
    dot[s] = vn[s] * (Fb[0] * u[0] + Fb[1] * u[1] + Fb[2] * u[2] + Fb[3] * (u[3] + p[s])) +
             g0 * p[s];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) D = fma(Fb[k], uR[k] - uL[k], D);
  const T Q = (SR * dot[0] - SL * dot[1] + SL * SR * D) * inv;
  const T SLb = fan ? (Q - dot[1] + SR * D) * inv : T(0);
  const T SRb = fan ? (dot[0] - Q + SL * D) * inv : T(0);
  const T cu = fan ? SL * SR * inv : T(0);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    // this side's weight of its own flux, of u_R - u_L, and its wave speeds
    const T a = fan ? (s ? -SL : SR) * inv : ((s ? right : left) ? T(1) : T(0));
    const T cs = s ? cu : -cu;
    const T lb = (loR == (s == 1)) ? SLb : T(0), rb = (hiR == (s == 1)) ? SRb : T(0);
    const T* u = s == 0 ? uL : uR;
    T* ub = s == 0 ? uLb : uRb;
    const T ics = rcp(c[s]);
    const T G0 = a * Fb[0], G1 = a * Fb[1], G2 = a * Fb[2], G3 = a * Fb[3];
    const T vnb = G0 * u[0] + G1 * u[1] + G2 * u[2] + G3 * (u[3] + p[s]) + lb + rb;
    const T cb = T(0.5) * gamma * (rb - lb) * ics;  // c = sqrt(gamma p / rho)
    const T pb = gm1 * (a * g0 + G3 * vn[s] + cb * ir[s]);
    const T irb = cb * p[s];
    const T vxb = vnb * nx - T(0.5) * pb * u[1], vyb = vnb * ny - T(0.5) * pb * u[2];
    ub[0] = G0 * vn[s] - ir[s] * (vxb * vx[s] + vyb * vy[s] + ir[s] * irb) + cs * Fb[0];
    ub[1] = G1 * vn[s] + vxb * ir[s] - T(0.5) * pb * vx[s] + cs * Fb[1];
    ub[2] = G2 * vn[s] + vyb * ir[s] - T(0.5) * pb * vy[s] + cs * Fb[2];
    ub[3] = G3 * vn[s] + pb + cs * Fb[3];
  }
}

// Volume term at one point: cotangent of the state u from those of its fluxes
// along x and y (Fxb, Fyb).
template <typename T>
__device__ __forceinline__ void euler_xy_vjp(const T* u, T gamma, const T* Fxb, const T* Fyb,
                                             T* ub) {
  const T gm1 = gamma - T(1);
  const T ir = rcp(u[0]);
  const T vx = u[1] * ir, vy = u[2] * ir;
  const T Ep = u[3] + gm1 * (u[3] - T(0.5) * (u[1] * vx + u[2] * vy));
  const T pb = gm1 * (Fxb[1] + Fyb[2] + Fxb[3] * vx + Fyb[3] * vy);
  const T vxb = Fxb[1] * u[1] + Fxb[2] * u[2] + Fxb[3] * Ep - T(0.5) * pb * u[1];
  const T vyb = Fyb[1] * u[1] + Fyb[2] * u[2] + Fyb[3] * Ep - T(0.5) * pb * u[2];
  ub[0] = -ir * (vxb * vx + vyb * vy);
  ub[1] = Fxb[0] + Fxb[1] * vx + Fyb[1] * vy + vxb * ir - T(0.5) * pb * vx;
  ub[2] = Fyb[0] + Fxb[2] * vx + Fyb[2] * vy + vyb * ir - T(0.5) * pb * vy;
  ub[3] = Fxb[3] * vx + Fyb[3] * vy + pb;
}

// The limiter transpose Pi_P^T lamW of one cell's own limiter (that of k_fl_lim:
// bounds over the cell and its neighbours in the incidence order, alpha = min
// over the incidences of psi at the face centroid, the first on ties): writes
// the adjoint of its gradients and the part its own mean takes, and per variable
// a message for the neighbour whose mean set the bound.  msg[v * nc + e] holds
// the value, to[v * nc + e] the incidence code (face << 1 | side) through which
// the cell sees that neighbour, -1 for no message.
template <typename T>
__device__ __forceinline__ void limit_transpose(const PFA<T>& p, int e, const T* lw) {
  T q[12];
  load12(p.P, p.nc, e, q);
  T hi[4], lo[4];
  int ihi[4], ilo[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    hi[v] = lo[v] = q[3 * v];
    ihi[v] = ilo[v] = -1;
  }
  // incidences kBatch at a time with their loads in flight (eight spill 100 B a lane:
  // 0.112 against 0.100 ms)
  constexpr int kBatch = 4;
  const int i0 = p.inc0[e], i1 = p.inc0[e + 1];
  for (int b0 = i0; b0 < i1; b0 += kBatch) {
    int nb[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) nb[u] = b0 + u < i1 ? p.nbr[b0 + u] : e;
    T m[kBatch][4];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[u][v] = p.P[(3 * v) * p.nc + nb[u]];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        ihi[v] = m[u][v] > hi[v] ? b0 + u : ihi[v];
        ilo[v] = m[u][v] < lo[v] ? b0 + u : ilo[v];
        hi[v] = fmax(hi[v], m[u][v]);
        lo[v] = fmin(lo[v], m[u][v]);
      }
  }
  // alpha and the increment d = g . r of the face that sets it (d = 0: none)
  T al[4], da[4], rx[4], ry[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    al[v] = T(1);
    da[v] = rx[v] = ry[v] = T(0);
  }
  for (int b0 = i0; b0 < i1; b0 += kBatch) {
    T ox[kBatch], oy[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = b0 + u < i1 ? b0 + u : b0;
      ox[u] = p.lim_geo[2 * (size_t)i];
      oy[u] = p.lim_geo[2 * (size_t)i + 1];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T d = q[3 * v + 1] * ox[u] + q[3 * v + 2] * oy[u];
        const T psi = psi_of(d, q[3 * v], hi[v], lo[v]);
        const bool set = psi < al[v];
        al[v] = set ? psi : al[v];
        da[v] = set ? d : da[v];
        rx[v] = set ? ox[u] : rx[v];
        ry[v] = set ? oy[u] : ry[v];
      }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    // psi = (bound - phi) / d: bound with cotangent ab / d, d with -psi ab / d
    const bool act = da[v] != T(0), up = da[v] > T(0);
    const T ab = lw[3 * v + 1] * q[3 * v + 1] + lw[3 * v + 2] * q[3 * v + 2];
    const T ad = fabs(da[v]);
    const T w = act ? div_small(up ? ab : -ab, ad) : T(0);
    const int to = up ? ihi[v] : ilo[v];
    const bool send = act && to >= 0;
    p.out[(size_t)(3 * v) * p.nc + e] = lw[3 * v] - (send ? w : T(0));
    p.out[(size_t)(3 * v + 1) * p.nc + e] = al[v] * (lw[3 * v + 1] - w * rx[v]);
    p.out[(size_t)(3 * v + 2) * p.nc + e] = al[v] * (lw[3 * v + 2] - w * ry[v]);
    p.msg[(size_t)v * p.nc + e] = w;
    p.to[(size_t)v * p.nc + e] = send ? p.inc_face[to] : -1;
  }
}

// lamW of a block of cells (the blocks of k_fl_step).  The face sweep of a block's
// faces runs once for both sides and leaves per face and side the sum and the
// difference of the two Gauss points; each cell then gathers its incidences.  The
// LDS decides how many workgroups overlap their loads with another's sweep: two per
// CU in FP64 (80 KB each), because the residual cotangents of the cells and Pi(P)
// take turns in one table (each thread folds the cotangents of its up to four faces
// into eight values a face first) and a pass sweeps kBlock faces.
template <typename T, bool LIM>
__global__ __launch_bounds__(kBlock, 2) void k_adjfl_L(PFA<T> p) {
  __shared__ T cT[12][kLocal];   // rm, rx, ry of each variable, then Pi(P)
  __shared__ T sB[22][kBlock];   // per slot: each side's ub0 + ub1 and ub1 - ub0, the
                                 // points' offset, the face centroid from L and from R
  constexpr int kPasses = kMaxSlots / kBlock;
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int tid = threadIdx.x;
  const int c0 = p.blk_cell0[b], nown = p.blk_cell0[b + 1] - c0;
  const int h0 = p.blk_halo0[b], nhalo = p.blk_halo0[b + 1] - h0;
  const int s0 = p.blk_slot0[b], nslot = p.blk_slot0[b + 1] - s0;
  const int nc = p.nc;
  const T is3 = T(0.57735026918962576451);  // 1/sqrt(3)
  const int e = c0 + tid;
  const bool own = tid < nown;
  // the last two waves take a halo cell each beside their own
  const int hi = tid - (kBlock - kMaxHalo);
  const bool halo = hi >= 0 && hi < nhalo;
  int ii = 0, i1 = 0;
  T g[12], we[12], wh[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) g[k] = T(0);
  auto put_cot = [&](const Cot<T>& c, int i) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      cT[3 * v][i] = c.rm[v];
      cT[3 * v + 1][i] = c.rx[v];
      cT[3 * v + 2][i] = c.ry[v];
    }
  };
  if (halo) {
    const int ge = p.halo_cell[h0 + hi];
    T le[12];
    load12(p.W, nc, ge, wh);
    load12(p.lam, nc, ge, le);
    Cot<T> c;
    cotangents(le, p.cell_geo + 8 * (size_t)ge, c);
    put_cot(c, nown + hi);
  }
  if (own) {
    ii = p.cell_inc0[e];
    i1 = p.cell_inc0[e + 1];
    T le[12], cg[8];
    load12(p.W, nc, e, we);
    load12(p.lam, nc, e, le);
#pragma unroll
    for (int k = 0; k < 8; ++k) cg[k] = p.cell_geo[8 * (size_t)e + k];
    Cot<T> c;
    cotangents(le, cg, c);
    put_cot(c, tid);
    // volume term: the 4 principal-axis points c -+ a_k
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      const T sgn = (q & 1) ? T(1) : T(-1);
      const T ox = sgn * ((q & 2) ? cg[6] : cg[4]);
      const T oy = sgn * ((q & 2) ? cg[7] : cg[5]);
      T u[4], ub[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) u[v] = fma(we[3 * v + 1], ox, fma(we[3 * v + 2], oy, we[3 * v]));
      euler_xy_vjp(u, p.gamma, c.vx, c.vy, ub);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        g[3 * v] += ub[v];
        g[3 * v + 1] = fma(ox, ub[v], g[3 * v + 1]);
        g[3 * v + 2] = fma(oy, ub[v], g[3 * v + 2]);
      }
    }
  }
  __syncthreads();
  // Gauss points x_f -+ A/(2 sqrt 3) t, t = (-n_y, n_x); weights A/2; the L cell
  // takes -w F, the R cell +w F (mean and the moments about its centroid): the flux
  // cotangent at the face centroid and its change to a point
  T aF[kPasses][4], bF[kPasses][4];
#pragma unroll
  for (int j = 0; j < kPasses; ++j) {
    const int sl = j * kBlock + tid;
    if (sl < nslot) {
      const int lr = p.slot_lr[s0 + sl], L = lr & 0xffff, R = lr >> 16;
      const T* sg = p.slot_geo + 8 * (size_t)(s0 + sl);
      const T w = T(0.5) * sg[2], o = w * is3;
      const T tx = -sg[1] * o, ty = sg[0] * o, fx = sg[3], fy = sg[4];
      const T gx = fx - sg[5], gy = fy - sg[6];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        T qx = cT[3 * v + 1][R], qy = cT[3 * v + 2][R];
        const T a = cT[3 * v][R] + qx * gx + qy * gy, d = qx * tx + qy * ty;
        qx = cT[3 * v + 1][L], qy = cT[3 * v + 2][L];
        aF[j][v] = w * (a - (cT[3 * v][L] + qx * fx + qy * fy));
        bF[j][v] = w * (d - (qx * tx + qy * ty));
      }
    }
  }
  __syncthreads();
  if (halo) {
#pragma unroll
    for (int k = 0; k < 12; ++k) cT[k][nown + hi] = wh[k];
  }
  if (own) {
#pragma unroll
    for (int k = 0; k < 12; ++k) cT[k][tid] = we[k];
  }
  // the cell's incidences (sorted by slot), loaded ahead
  int inc = ii < i1 ? p.cell_inc[ii] : 0, inc1 = ii + 1 < i1 ? p.cell_inc[ii + 1] : 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPasses; ++j) {
    const int sa = j * kBlock;
    if (sa >= nslot) break;
    if (sa + tid < nslot) {
      const int lr = p.slot_lr[s0 + sa + tid], L = lr & 0xffff, R = lr >> 16;
      const T* sg = p.slot_geo + 8 * (size_t)(s0 + sa + tid);
      const T nx = sg[0], ny = sg[1], o = T(0.5) * sg[2] * is3;
      const T tx = -ny * o, ty = nx * o, fx = sg[3], fy = sg[4];
      const T gx = fx - sg[5], gy = fy - sg[6];
      T aL[4], bL[4], aR[4], bR[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        T qx = cT[3 * v + 1][L], qy = cT[3 * v + 2][L];
        aL[v] = cT[3 * v][L] + qx * fx + qy * fy;
        bL[v] = qx * tx + qy * ty;
        qx = cT[3 * v + 1][R], qy = cT[3 * v + 2][R];
        aR[v] = cT[3 * v][R] + qx * gx + qy * gy;
        bR[v] = qx * tx + qy * ty;
      }
      T S[8], D[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) S[k] = D[k] = T(0);
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) {
        const T sgn = gp ? T(1) : T(-1);
        T uL[4], uR[4], Fb[4], ub[8];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          uL[v] = fma(sgn, bL[v], aL[v]);
          uR[v] = fma(sgn, bR[v], aR[v]);
          Fb[v] = fma(sgn, bF[j][v], aF[j][v]);
        }
        hll_n_vjp(uL, uR, nx, ny, p.gamma, Fb, ub, ub + 4);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          S[k] += ub[k];
          D[k] = fma(sgn, ub[k], D[k]);
        }
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          sB[8 * s + v][tid] = S[4 * s + v];
          sB[8 * s + 4 + v][tid] = D[4 * s + v];
        }
      sB[16][tid] = tx;
      sB[17][tid] = ty;
      sB[18][tid] = fx;
      sB[19][tid] = fy;
      sB[20][tid] = gx;
      sB[21][tid] = gy;
    }
    __syncthreads();
    // this pass's incidences
    while (ii < i1 && ((inc & 0xffff) >> 1) < sa + kBlock) {
      const int ls = ((inc & 0xffff) >> 1) - sa, side = inc & 1;
      inc = inc1;
      inc1 = ii + 2 < i1 ? p.cell_inc[ii + 2] : 0;
      ++ii;
      const T tx = sB[16][ls], ty = sB[17][ls];
      const T fx = sB[18 + 2 * side][ls], fy = sB[19 + 2 * side][ls];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T S = sB[8 * side + v][ls], D = sB[8 * side + 4 + v][ls];
        g[3 * v] += S;
        g[3 * v + 1] += fma(S, fx, D * tx);
        g[3 * v + 2] += fma(S, fy, D * ty);
      }
    }
    if (sa + kBlock < nslot) __syncthreads();  // the next pass overwrites the table
  }
  if (!own) return;
  const double dt = p.dt_dev ? *p.dt_dev : p.dt_host;
  const T cid = (T)p.c_id, cL = (T)(p.c_L_over_dt * dt), cx = (T)p.c_extra;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    g[k] = fma(cL, g[k], cid * p.lam[(size_t)k * nc + e]);
    if (p.extra) g[k] = fma(cx, p.extra[(size_t)k * nc + e], g[k]);
  }
  if (LIM) {
    limit_transpose(p, e, g);
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) p.out[(size_t)k * nc + e] = g[k];
  }
}

// Adds to each mean adjoint the messages of its face neighbours: the neighbour
// across incidence (face << 1 | side) sees this cell through that code with the
// side flipped (also where a cell is its own neighbour or shares two faces).
template <typename T>
__global__ __launch_bounds__(256) void k_adjfl_msg(PFA<T> p) {
  const int e = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (e >= p.nc) return;
  T add[4] = {T(0), T(0), T(0), T(0)};
  constexpr int kBatch = 4;
  const int i0 = p.inc0[e], i1 = p.inc0[e + 1];
  for (int b0 = i0; b0 < i1; b0 += kBatch) {
    int nb[kBatch], c[kBatch], to[kBatch][4];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = b0 + u < i1 ? b0 + u : i0;
      nb[u] = p.nbr[i];
      c[u] = b0 + u < i1 ? (p.inc_face[i] ^ 1) : -2;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) to[u][v] = p.to[(size_t)v * p.nc + nb[u]];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (to[u][v] == c[u]) add[v] += p.msg[(size_t)v * p.nc + nb[u]];
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) p.out[(size_t)(3 * v) * p.nc + e] += add[v];
}

template <typename T>
hipError_t adjoint_t(const dg_mesh* m, const void* U, const void* V1, const double* dt_dev,
                     double dt, const void* lam_np1, void* lam_n, void* ws1, void* ws2,
                     void* scratch, hipStream_t s) {
  const FLDev& f = *m->fld;
  const bool lim = m->cfg.limiter == DG_LIMITER_MINMOD;
  const dim3 grid((unsigned)((f.ncells + 255) / 256)), block(256);
  PFA<T> p{};
  p.dt_dev = dt_dev;
  p.dt_host = dt;
  p.nc = f.ncells;
  p.gamma = (T)m->cfg.gamma;
  p.inc0 = f.lim_inc0;
  p.nbr = f.lim_nbr;
  p.inc_face = f.inc_face;
  p.blk_cell0 = f.blk_cell0;
  p.blk_slot0 = f.blk_slot0;
  p.blk_halo0 = f.blk_halo0;
  p.halo_cell = f.halo_cell;
  p.slot_lr = f.slot_lr;
  p.slot_geo = static_cast<const T*>(f.slot_geo);
  p.cell_inc0 = f.cell_inc0;
  p.cell_inc = f.cell_inc;
  p.lim_geo = static_cast<const T*>(f.lim_geo);
  p.cell_geo = static_cast<const T*>(f.cell_geo);
  auto adj_stage = [&](const void* P, const void* lam, const void* extra, double c_id,
                       double c_L_over_dt, double c_extra, void* out) -> hipError_t {
    // W = Pi(P) into ws1; out = Pi_P^T lamW (lamW itself without a limiter)
    const void* W = P;
    if (lim) {
      hipError_t r = lim_t<T>(m, P, ws1, s);
      if (r != hipSuccess) return r;
      W = ws1;
    }
    PFA<T> a = p;
    a.W = static_cast<const T*>(W);
    a.P = static_cast<const T*>(P);
    a.lam = static_cast<const T*>(lam);
    a.extra = static_cast<const T*>(extra);
    a.c_id = c_id;
    a.c_L_over_dt = c_L_over_dt;
    a.c_extra = c_extra;
    a.out = static_cast<T*>(out);
    a.msg = static_cast<T*>(scratch);
    a.to = reinterpret_cast<int*>(a.msg + (size_t)4 * f.ncells);
    const dim3 blocks((unsigned)f.nblocks);
    if (!lim) {
      hipLaunchKernelGGL((k_adjfl_L<T, false>), blocks, dim3(kBlock), 0, s, a);
    } else {
      hipLaunchKernelGGL((k_adjfl_L<T, true>), blocks, dim3(kBlock), 0, s, a);
      hipLaunchKernelGGL((k_adjfl_msg<T>), grid, block, 0, s, a);
    }
    return hipGetLastError();
  };
  // stage 2: lam_V1 = Pi_V1^T [lam'/2 + (dt/2) L^T lam'] (in ws2: blocks write their
  // cells of lam_n while others still read their halo of lam_V1); stage 1:
  // lam_n = Pi_U^T [lam_V1 + dt L^T lam_V1 + lam'/2]
  hipError_t e = adj_stage(V1, lam_np1, nullptr, 0.5, 0.5, 0.0, ws2);
  if (e != hipSuccess) return e;
  return adj_stage(U, ws2, lam_np1, 1.0, 1.0, 0.5, lam_n);
}

// ------------------------------------------------------------ host setup --
template <typename T>
hipError_t upload(const std::vector<double>& h, void** d) {
  std::vector<T> t(h.begin(), h.end());
  hipError_t e = hipMalloc(d, sizeof(T) * std::max<size_t>(t.size(), 1));
  if (e == hipSuccess && !t.empty())
    e = hipMemcpy(*d, t.data(), sizeof(T) * t.size(), hipMemcpyHostToDevice);
  return e;
}

hipError_t upload_i(const std::vector<int>& h, int** d) {
  hipError_t e = hipMalloc((void**)d, sizeof(int) * std::max<size_t>(h.size(), 1));
  if (e == hipSuccess && !h.empty())
    e = hipMemcpy(*d, h.data(), sizeof(int) * h.size(), hipMemcpyHostToDevice);
  return e;
}

}  // namespace

void facelist_destroy(dg_mesh* m);

dg_status facelist_create(dg_mesh* m, const dg_mesh_desc* d) {
  const int64_t nc = d->ncells, nf = d->nfaces;
  if (nc < 1 || nf < 1) {
    set_error("dg_mesh_create: face list needs ncells >= 1 and nfaces >= 1");
    return DG_EINVAL;
  }
  if (!d->cell_volume || !d->cell_centroid || !d->cell_moments || !d->face_cells ||
      !d->face_area || !d->face_normal || !d->face_centroid || !d->face_shift) {
    set_error("dg_mesh_create: face list with a NULL array");
    return DG_EINVAL;
  }
  if (!(d->box[0] > 0) || !(d->box[1] > 0)) {
    set_error("dg_mesh_create: face list box must be positive");
    return DG_EINVAL;
  }
  const double bx[2] = {d->box[0], d->box[1]};
  // validation: indices, positive sizes, unit normals, closure
  std::vector<double> closure(2 * nc, 0.0), perim(nc, 0.0);
  for (int64_t f = 0; f < nf; ++f) {
    const int L = d->face_cells[2 * f], R = d->face_cells[2 * f + 1];
    if (L < 0 || L >= nc || R < 0 || R >= nc) {
      set_error("dg_mesh_create: face " + std::to_string(f) + " has a cell index out of range");
      return DG_EINVAL;
    }
    const double A = d->face_area[f], nx = d->face_normal[2 * f], ny = d->face_normal[2 * f + 1];
    if (!(A > 0) || std::fabs(nx * nx + ny * ny - 1.0) > 1e-10) {
      set_error("dg_mesh_create: face " + std::to_string(f) + " needs A > 0 and a unit normal");
      return DG_EINVAL;
    }
    for (int k = 0; k < 2; ++k) {
      const int s = d->face_shift[2 * f + k];
      if (s < -1 || s > 1) {
        set_error("dg_mesh_create: face shifts must be -1, 0 or 1");
        return DG_EINVAL;
      }
    }
    closure[2 * L] += A * nx;
    closure[2 * L + 1] += A * ny;
    closure[2 * R] -= A * nx;
    closure[2 * R + 1] -= A * ny;
    perim[L] += A;
    perim[R] += A;
  }
  for (int64_t e = 0; e < nc; ++e) {
    const double V = d->cell_volume[e];
    const double a = d->cell_moments[3 * e], b = d->cell_moments[3 * e + 1],
                 c = d->cell_moments[3 * e + 2];
    if (!(V > 0) || !(a > 0) || !(c > 0) || !(a * c - b * b > 0)) {
      set_error("dg_mesh_create: cell " + std::to_string(e) +
                " needs V > 0 and positive-definite moments");
      return DG_EINVAL;
    }
    if (!(perim[e] > 0)) {
      set_error("dg_mesh_create: cell " + std::to_string(e) + " has no faces");
      return DG_EINVAL;
    }
    if (std::hypot(closure[2 * e], closure[2 * e + 1]) > 1e-9 * perim[e]) {
      set_error("dg_mesh_create: cell " + std::to_string(e) + " is not closed (sum A n != 0)");
      return DG_EINVAL;
    }
  }
  // per-cell geometry: 1/V, M^-1, scaled principal axes
  std::vector<double> cgeo(8 * nc);
  for (int64_t e = 0; e < nc; ++e) {
    const double V = d->cell_volume[e];
    const double a = d->cell_moments[3 * e], b = d->cell_moments[3 * e + 1],
                 c = d->cell_moments[3 * e + 2];
    const double det = a * c - b * b;
    // inverse mass matrix per unit volume: V * M^-1
    cgeo[8 * e] = 1.0 / V;
    cgeo[8 * e + 1] = V * c / det;
    cgeo[8 * e + 2] = -V * b / det;
    cgeo[8 * e + 3] = V * a / det;
    const double tr = 0.5 * (a + c), disc = std::sqrt(0.25 * (a - c) * (a - c) + b * b);
    const double lam[2] = {tr + disc, tr - disc};
    double ev[2][2];
    if (b == 0.0) {
      if (a >= c) {
        ev[0][0] = 1; ev[0][1] = 0; ev[1][0] = 0; ev[1][1] = 1;
      } else {
        ev[0][0] = 0; ev[0][1] = 1; ev[1][0] = 1; ev[1][1] = 0;
      }
    } else {
      for (int k = 0; k < 2; ++k) {
        const double vx = b, vy = lam[k] - a, nn = std::hypot(vx, vy);
        ev[k][0] = vx / nn;
        ev[k][1] = vy / nn;
      }
    }
    for (int k = 0; k < 2; ++k) {
      const double r = std::sqrt(2.0 * lam[k] / V);
      cgeo[8 * e + 4 + 2 * k] = r * ev[k][0];
      cgeo[8 * e + 5 + 2 * k] = r * ev[k][1];
    }
  }
  // global incidence CSR (limiter, CFL): per cell its faces as seen from it
  std::vector<int> inc0(nc + 1, 0);
  for (int64_t f = 0; f < nf; ++f) {
    inc0[d->face_cells[2 * f] + 1]++;
    inc0[d->face_cells[2 * f + 1] + 1]++;
  }
  for (int64_t e = 0; e < nc; ++e) inc0[e + 1] += inc0[e];
  std::vector<int> fill(inc0.begin(), inc0.end() - 1), nbr(inc0[nc]);
  // offsets of all incidences, then their A n (the limiter reads only the first block)
  const size_t ninc = (size_t)inc0[nc];
  std::vector<double> lgeo(4 * ninc);
  // face geometry offsets (from each side's centroid)
  auto offsets = [&](int64_t f, double* rc, double* dLR) {
    const int L = d->face_cells[2 * f], R = d->face_cells[2 * f + 1];
    for (int k = 0; k < 2; ++k) {
      rc[k] = d->face_centroid[2 * f + k] - d->cell_centroid[2 * L + k];
      dLR[k] = d->cell_centroid[2 * R + k] + d->face_shift[2 * f + k] * bx[k] -
               d->cell_centroid[2 * L + k];
    }
  };
  for (int64_t f = 0; f < nf; ++f) {
    const int L = d->face_cells[2 * f], R = d->face_cells[2 * f + 1];
    double rc[2], dLR[2];
    offsets(f, rc, dLR);
    const double A = d->face_area[f], nx = d->face_normal[2 * f], ny = d->face_normal[2 * f + 1];
    int i = fill[L]++;
    nbr[i] = R;
    lgeo[2 * i] = rc[0];
    lgeo[2 * i + 1] = rc[1];
    lgeo[2 * ninc + 2 * i] = A * nx;
    lgeo[2 * ninc + 2 * i + 1] = A * ny;
    i = fill[R]++;
    nbr[i] = L;
    lgeo[2 * i] = rc[0] - dLR[0];
    lgeo[2 * i + 1] = rc[1] - dLR[1];
    lgeo[2 * ninc + 2 * i] = -A * nx;
    lgeo[2 * ninc + 2 * i + 1] = -A * ny;
  }
  // face ids per cell (same order as the global CSR)
  std::vector<int> cface(inc0[nc]), cside(inc0[nc]);
  {
    std::vector<int> fl2(inc0.begin(), inc0.end() - 1);
    for (int64_t f = 0; f < nf; ++f) {
      const int L = d->face_cells[2 * f], R = d->face_cells[2 * f + 1];
      int i = fl2[L]++;
      cface[i] = (int)f;
      cside[i] = 0;
      i = fl2[R]++;
      cface[i] = (int)f;
      cside[i] = 1;
    }
  }
  // the adjoint's incidence codes
  std::vector<int> inc_face(inc0[nc]);
  for (int64_t i = 0; i < (int64_t)inc0[nc]; ++i) inc_face[i] = (cface[i] << 1) | cside[i];
  // blocks of up to kBlock consecutive cells; a block is halved until its
  // distinct incident faces fit the slot table and its outside neighbours the
  // halo table
  std::vector<int> blk_cell0{0};
  {
    std::vector<int64_t> fmark(nf, -1), cmark(nc, -1);
    int64_t stamp = 0, e = 0;
    while (e < nc) {
      int64_t e1 = std::min<int64_t>(e + kBlock, nc);
      for (;;) {
        ++stamp;
        int ns = 0, nh = 0;
        for (int64_t c = e; c < e1; ++c)
          for (int i = inc0[c]; i < inc0[c + 1]; ++i) {
            const int f = cface[i];
            if (fmark[f] != stamp) {
              fmark[f] = stamp;
              ++ns;
            }
            const int o = cside[i] ? d->face_cells[2 * f] : d->face_cells[2 * f + 1];
            if ((o < e || o >= e1) && cmark[o] != stamp) {
              cmark[o] = stamp;
              ++nh;
            }
          }
        if ((ns <= kMaxSlots && nh <= kMaxHalo) || e1 - e <= 1) break;
        e1 = e + (e1 - e) / 2;
      }
      blk_cell0.push_back((int)e1);
      e = e1;
    }
  }
  const int nblocks = (int)blk_cell0.size() - 1;
  std::vector<int> blk_slot0{0}, blk_halo0{0}, halo_cell, slot_lr, cell_inc0(nc + 1, 0), cell_inc;
  std::vector<double> sgeo, irf;
  std::vector<int> slot_of_face(nf, -1), local_of(nc, -1);
  int max_slots = 0;
  for (int b = 0; b < nblocks; ++b) {
    const int ca = blk_cell0[b], cb = blk_cell0[b + 1], nown = cb - ca;
    // block-local indices: own cells first, then the halo in first-seen order
    std::vector<int> halo;
    for (int c = ca; c < cb; ++c) local_of[c] = c - ca;
    for (int c = ca; c < cb; ++c)
      for (int i = inc0[c]; i < inc0[c + 1]; ++i) {
        const int f = cface[i];
        const int o = cside[i] ? d->face_cells[2 * f] : d->face_cells[2 * f + 1];
        if (local_of[o] < 0) {
          local_of[o] = nown + (int)halo.size();
          halo.push_back(o);
        }
      }
    if ((int)halo.size() > kMaxHalo) {
      set_error("dg_mesh_create: a cell block has too many outside neighbours");
      return DG_EINVAL;
    }
    // slots in first-seen order; each cell's incidences sorted by slot
    std::vector<int> touched;
    int ns = 0;
    for (int c = ca; c < cb; ++c) {
      std::vector<std::pair<int, int>> mine;  // (slot, incidence index in the global CSR)
      for (int i = inc0[c]; i < inc0[c + 1]; ++i) {
        const int f = cface[i];
        if (slot_of_face[f] < 0) {
          slot_of_face[f] = ns++;
          touched.push_back(f);
          const int L = d->face_cells[2 * f], R = d->face_cells[2 * f + 1];
          slot_lr.push_back(local_of[L] | (local_of[R] << 16));
          double rc[2], dLR[2];
          offsets(f, rc, dLR);
          const double g[8] = {d->face_normal[2 * f], d->face_normal[2 * f + 1], d->face_area[f],
                               rc[0], rc[1], dLR[0], dLR[1], 0.0};
          sgeo.insert(sgeo.end(), g, g + 8);
        }
        mine.emplace_back(slot_of_face[f], i);
      }
      std::sort(mine.begin(), mine.end());
      for (const auto& si : mine) {
        const int i = si.second, f = cface[i];
        const int o = cside[i] ? d->face_cells[2 * f] : d->face_cells[2 * f + 1];
        cell_inc.push_back((si.first * 2 + cside[i]) | (local_of[o] << 16));
        double rc[2], dLR[2];
        offsets(f, rc, dLR);
        // face centroid from this side's centroid (R: its image next to L)
        irf.push_back(cside[i] ? rc[0] - dLR[0] : rc[0]);
        irf.push_back(cside[i] ? rc[1] - dLR[1] : rc[1]);
      }
      cell_inc0[c + 1] = (int)cell_inc.size();
    }
    for (int f : touched) slot_of_face[f] = -1;
    for (int c = ca; c < cb; ++c) local_of[c] = -1;
    for (int o : halo) local_of[o] = -1;
    if (ns > kMaxSlots) {
      set_error("dg_mesh_create: a cell block has too many incident faces");
      return DG_EINVAL;
    }
    max_slots = std::max(max_slots, ns);
    blk_slot0.push_back(blk_slot0.back() + ns);
    halo_cell.insert(halo_cell.end(), halo.begin(), halo.end());
    blk_halo0.push_back((int)halo_cell.size());
  }
  FLDev* fd = new FLDev();
  std::memset(fd, 0, sizeof(FLDev));
  fd->ncells = (int)nc;
  fd->nblocks = nblocks;
  fd->max_slots = max_slots;
  fd->ninc = (int64_t)ninc;
  m->fld = fd;
  m->fl.nblocks = nblocks;
  m->ncells = nc;
  const bool f64 = m->cfg.precision == DG_FP64;
  hipError_t err = upload_i(blk_cell0, &fd->blk_cell0);
  if (err == hipSuccess) err = upload_i(blk_slot0, &fd->blk_slot0);
  if (err == hipSuccess) err = upload_i(blk_halo0, &fd->blk_halo0);
  if (err == hipSuccess) err = upload_i(halo_cell, &fd->halo_cell);
  if (err == hipSuccess) err = upload_i(slot_lr, &fd->slot_lr);
  if (err == hipSuccess) err = upload_i(cell_inc0, &fd->cell_inc0);
  if (err == hipSuccess) err = upload_i(cell_inc, &fd->cell_inc);
  if (err == hipSuccess) err = upload_i(inc0, &fd->lim_inc0);
  if (err == hipSuccess) err = upload_i(nbr, &fd->lim_nbr);
  auto up = [&](const std::vector<double>& h, void** dst) {
    return f64 ? upload<double>(h, dst) : upload<float>(h, dst);
  };
  if (err == hipSuccess) err = up(sgeo, &fd->slot_geo);
  if (err == hipSuccess) err = up(irf, &fd->inc_rf);
  if (err == hipSuccess) err = up(cgeo, &fd->cell_geo);
  if (err == hipSuccess) err = up(lgeo, &fd->lim_geo);
  if (err == hipSuccess) err = up(perim, &fd->cell_perim);
  if (err == hipSuccess) err = upload_i(inc_face, &fd->inc_face);
  if (err != hipSuccess) {
    facelist_destroy(m);
    return hip_fail(err, "dg_mesh_create: face-list upload");
  }
  return DG_OK;
}

void facelist_destroy(dg_mesh* m) {
  FLDev* f = m->fld;
  if (!f) return;
  (void)hipFree(f->blk_cell0);
  (void)hipFree(f->blk_slot0);
  (void)hipFree(f->blk_halo0);
  (void)hipFree(f->halo_cell);
  (void)hipFree(f->slot_lr);
  (void)hipFree(f->slot_geo);
  (void)hipFree(f->cell_inc0);
  (void)hipFree(f->cell_inc);
  (void)hipFree(f->inc_rf);
  (void)hipFree(f->cell_geo);
  (void)hipFree(f->lim_inc0);
  (void)hipFree(f->lim_nbr);
  (void)hipFree(f->lim_geo);
  (void)hipFree(f->cell_perim);
  (void)hipFree(f->inc_face);
  delete f;
  m->fld = nullptr;
}

hipError_t launch_min_finalize(const double* part, int n, double cfl, double* dt, hipStream_t s);

hipError_t launch_facelist(const dg_mesh* m, int mode, const void* in, const void* u0, void* out,
                           const double* dt_dev, double dt_host, double cfl, double* dt_next,
                           hipStream_t s) {
  const bool f64 = m->cfg.precision == DG_FP64;
  const bool lim = m->cfg.limiter == DG_LIMITER_MINMOD;
  auto limit = [&](const void* a, void* b) {
    return f64 ? lim_t<double>(m, a, b, s) : lim_t<float>(m, a, b, s);
  };
  auto step = [&](int md, const void* ua, void* lim_out, bool want_dt) {
    return f64 ? step_t<double>(m, md, in, ua, out, lim_out, dt_dev, dt_host, want_dt, s)
               : step_t<float>(m, md, in, ua, out, lim_out, dt_dev, dt_host, want_dt, s);
  };
  hipError_t e = hipSuccess;
  switch (mode) {
    case kLimit:
      return limit(in, out);
    case kRhs:
      return step(kRhs, nullptr, nullptr, false);
    case kStage1:
      // keeps Pi(U) of every cell in ws_a for the stage 2 of the same U
      return step(kStage1, nullptr, lim ? m->ws_a : nullptr, false);
    case kStage2: {
      const void* ua = u0;
      if (lim) {
        if (!(m->ws_a_fresh && m->ws_a_src == u0)) e = limit(u0, m->ws_a);
        ua = m->ws_a;
      }
      if (e == hipSuccess) e = step(kStage2, ua, nullptr, dt_next != nullptr);
      if (e == hipSuccess && dt_next)
        e = launch_min_finalize(m->dtpart, m->fld->nblocks, cfl, dt_next, s);
      return e;
    }
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_adjoint_facelist(const dg_mesh* m, const void* U, const void* V1,
                                   const double* dt_dev, double dt, const void* lam_np1,
                                   void* lam_n, void* ws1, void* ws2, void* scratch,
                                   hipStream_t s) {
  if (m->cfg.precision == DG_FP64)
    return adjoint_t<double>(m, U, V1, dt_dev, dt, lam_np1, lam_n, ws1, ws2, scratch, s);
  return adjoint_t<float>(m, U, V1, dt_dev, dt, lam_np1, lam_n, ws1, ws2, scratch, s);
}

// Bytes of the limiter messages: four values and four incidence codes a cell.
size_t adjoint_facelist_scratch(const dg_mesh* m) {
  return (size_t)m->ncells * 4 * ((size_t)m->elem + sizeof(int));
}

hipError_t launch_facelist_cfl(const dg_mesh* m, const void* U, double cfl, double* dt_dev,
                               hipStream_t s) {
  hipError_t e = m->cfg.precision == DG_FP64 ? cfl_t<double>(m, U, s) : cfl_t<float>(m, U, s);
  if (e != hipSuccess) return e;
  return launch_min_finalize(m->dtpart, (m->fld->ncells + 63) / 64, cfl, dt_dev, s);
}

}  // namespace dg
