// Discrete adjoint of the 2D ideal-MHD Cartesian SSP-RK2 step: the HLLD flux of
// Sec. 2.3 on the face-averaged normal field, the 2D divergence-free field
// basis of Sec. 2.2 and the limiter of Sec. 2.5 with one alpha for B; dt is
// frozen and every branch (limiter, HLLD wave region) is the one the forward
// step takes.  Ties follow the first argument of min and max, in the order
// self, -x, +x, -y, +y, and |x| takes +x at 0, as the CPU oracle's dual
// numbers do.
//
// As for 2D Euler, the two stages are two "adjoint stages"
//   out = Pi_P^T lamW,   lamW = c_id lam + c_L (dL/dW)^T lam + c_extra extra,
//   W = Pi(P),
// stage 2: P = V1, lam = lam', c_id = 1/2, c_L = dt/2; stage 1: P = U,
// lam = lam_V1, c_id = 1, c_L = dt, extra = lam' with c_extra = 1/2.  Each
// runs the forward limiter (k_lim2m) into a workspace, then, chunk of rows by
// chunk of rows, without atomics:
//   k_adj2m_face one thread per face, each face once, both Gauss points.  The
//                cotangent of its flux is the transpose of the linear residual
//                weights (the same algebra as the forward accumulation) applied to
//                the adjoints of both adjacent cells; one reverse sweep through
//                the HLLD flux (hlld_vjp) gives the cotangents of both sides'
//                point states, which go to a face table (64 values a cell);
//   k_adj2m_cell lamW of a cell from its four faces' entries (the extrapolation
//                to the Gauss points is linear, transposed by hand) and its volume
//                points, then the transpose of its own limiter: all it hands back
//                to its own coefficients, and a message per limited variable (a
//                value and a direction) for the neighbour whose mean set the bound;
// and at last
//   k_adj2m_msg  each cell adds the messages of its four neighbours.
// One wave per SIMD bounds k_adj2m_face (about 1,050 vector instructions a sweep in
// 38% of the issue slots, 17% of a wave's cycles waiting for data and 29% for an
// instruction to issue; waves of their own workgroup, since four to a workgroup wait
// for the slowest: 0.080 against 0.099 ms; a two-wave budget spills 300 B a lane, 0.15
// ms); memory traffic bounds k_adj2m_cell (400 MB at 5.8 TB/s).  Measured (512^2, FP64,
// one adjoint stage): faces 0.086, cells 0.069, messages 0.014 ms; one thread per cell solving each
// face from both sides 0.168 + 0.030 + 0.011 ms; with a forward-mode solve per
// state component and every limiter that reads a cell differentiated, component
// by component, 0.901 + 0.410 ms.  The adjoint step 2.59 -> 0.38 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dg_internal.h"
#include "dg_math.h"
#include "limiter_vjp.h"
#include "mhd_hlld_vjp.h"

namespace dg {

hipError_t launch_mhd2d(const dg_mesh* m, int mode, const void* in, const void* u0, void* out,
                        const double* dt_dev, double dt_host, double cfl, double* dt_next,
                        hipStream_t s);

namespace {

// Coefficient layout of a cell (23 values): 3v, 3v+1, 3v+2 the mean and x, y
// gradient of rho, mx, my, mz, E (v = 0..4); 15..17 the means of Bx, By, Bz;
// 18..22 a1, a2, a3, dBz/dx, dBz/dy.  The gradient of B_c along axis d is
// sgn(c, d) a[j(c, d)]: grad Bx = (a3, a1), grad By = (a2, -a3), grad Bz =
// (dBz/dx, dBz/dy).
__device__ __forceinline__ int bj(int c, int d) {
  return c == 0 ? (d == 0 ? 2 : 0) : (c == 1 ? (d == 0 ? 1 : 2) : (d == 0 ? 3 : 4));
}
__device__ __forceinline__ int bs(int c, int d) { return (c == 1 && d == 1) ? -1 : 1; }

constexpr size_t kFaceVals = 64;  // face table: 2 axes, 2 sides, 2 Gauss points, 8 variables

// Coefficient index of conserved mean k (rho, mx, my, mz, E, Bx, By, Bz).
__device__ __forceinline__ int mean_index(int k) { return k < 5 ? 3 * k : 10 + k; }

template <typename T>
struct PJ {
  const T* W;      // Pi(P), the state the stage's operator sees
  const T* P;      // the stage input (limiter transpose)
  const T* lam;    // adjoint of the stage output
  const T* extra;  // added to lamW with weight c_extra (may be NULL)
  T* out;
  T* F;            // face table of the rows at hand: [64][nF]
  T* msg;          // limiter messages: 6 values a cell
  unsigned* code;  // and their directions
  const double* dt_dev;
  double dt_host;
  double c_id, c_L_over_dt, c_extra;
  int nx, ny, nc;
  int row0, rows, nF;  // rows at hand, nF = nx (rows + 1)
  T gamma, eps;
  T c2h[2], c3[2], cs, pt[2], half[2], q[2], imu[3];
};

template <typename T>
__device__ __forceinline__ void load23(const T* __restrict__ U, int nc, int e, T* c) {
#pragma unroll
  for (int k = 0; k < 23; ++k) c[k] = U[(size_t)k * nc + e];
}

// The four face neighbours -x, +x, -y, +y of cell e (periodic).
__device__ __forceinline__ void neighbours(int e, int nx, int ny, int* nb) {
  const int i = e % nx, j = e / nx;
  nb[0] = j * nx + (i == 0 ? nx - 1 : i - 1);
  nb[1] = j * nx + (i == nx - 1 ? 0 : i + 1);
  nb[2] = (j == 0 ? ny - 1 : j - 1) * nx + i;
  nb[3] = (j == ny - 1 ? 0 : j + 1) * nx + i;
}

// Adjoint of the residual accumulators of a cell (means of the 8 conserved
// variables, hydro gradients, the field moments P[c][d]) from the adjoint of
// its time derivative: the transpose of the map from accumulators to
// coefficients (identity, and a1 = P[x][y]/mu_y, a2 = P[y][x]/mu_x,
// a3 = (P[x][x] - P[y][y])/(mu_x + mu_y), dBz/dx = P[z][x]/mu_x,
// dBz/dy = P[z][y]/mu_y).
template <typename T>
struct AccBar {
  T m[8], g[5][2], P[3][2];
};

template <typename T>
__device__ __forceinline__ void acc_bar(const T* lam, const PJ<T>& p, AccBar<T>& a) {
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    a.m[v] = lam[3 * v];
    a.g[v][0] = lam[3 * v + 1];
    a.g[v][1] = lam[3 * v + 2];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) a.m[5 + c] = lam[15 + c];
  a.P[0][1] = lam[18] * p.imu[1];
  a.P[1][0] = lam[19] * p.imu[0];
  a.P[0][0] = lam[20] * p.imu[2];
  a.P[1][1] = -lam[20] * p.imu[2];
  a.P[2][0] = lam[21] * p.imu[0];
  a.P[2][1] = lam[22] * p.imu[1];
}

// State of a cell's polynomial at the point (hn along axis D, ht along the
// other axis) from its centroid: hydro Taylor terms and the field basis.
template <typename T, int D>
__device__ __forceinline__ void point_state(const T* c, T hn, T ht, T* u) {
  constexpr int t = 1 - D;
#pragma unroll
  for (int v = 0; v < 5; ++v) u[v] = fma(c[3 * v + 1 + t], ht, fma(c[3 * v + 1 + D], hn, c[3 * v]));
#pragma unroll
  for (int k = 0; k < 3; ++k)
    u[5 + k] = fma(T(bs(k, t)) * c[18 + bj(k, t)], ht,
                   fma(T(bs(k, D)) * c[18 + bj(k, D)], hn, c[15 + k]));
}

// Transpose of point_state: the cotangent ub of the point state added to the
// coefficient adjoint g.
template <typename T, int D>
__device__ __forceinline__ void point_state_bar(const T* ub, T hn, T ht, T* g) {
  constexpr int t = 1 - D;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    g[3 * v] += ub[v];
    g[3 * v + 1 + D] = fma(hn, ub[v], g[3 * v + 1 + D]);
    g[3 * v + 1 + t] = fma(ht, ub[v], g[3 * v + 1 + t]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    g[15 + k] += ub[5 + k];
    g[18 + bj(k, D)] = fma(T(bs(k, D)) * hn, ub[5 + k], g[18 + bj(k, D)]);
    g[18 + bj(k, t)] = fma(T(bs(k, t)) * ht, ub[5 + k], g[18 + bj(k, t)]);
  }
}

// The -D face of cell eR, both Gauss points (offsets -+ q_t along the face): the
// cotangents of both sides' point states, to the face table.  The cotangent of a flux F is
// the transpose of the forward accumulation, for the R cell (sigma = +1) and the
// L cell (sigma = -1):
//   mean_k += sigma F_k/(2 h_D)           (k other than the normal field)
//   grad_v[D] -= 3 F_v / h_D^2,  grad_v[t] += s sigma sqrt3 F_v / (h_D h_t)
//   P[c][D] -= F_Bc / 4,  P[c][t] += s sigma h_t F_Bc / (4 sqrt3 h_D)  (c != D),
// F0 its part common to both points and F1 the part that changes sign.
template <typename T, int D>
__device__ __forceinline__ void face_adjoint(const PJ<T>& p, int eL, int eR, int le) {
  constexpr int t = 1 - D;
  // every load first: one latency for the thread's two solves
  T cL[23], cR[23];
  load23(p.W, p.nc, eL, cL);
  load23(p.W, p.nc, eR, cR);
  T F0[8], F1[8];
  {
    T lam[23];
    AccBar<T> a;
    load23(p.lam, p.nc, eR, lam);
    acc_bar(lam, p, a);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      F0[k] = p.c2h[D] * a.m[k];
      F1[k] = T(0);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      F0[v] = fma(-p.c3[D], a.g[v][D], F0[v]);
      F1[v] = p.cs * a.g[v][t];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c == D) continue;
      F0[5 + c] = fma(T(-0.25), a.P[c][D], F0[5 + c]);
      F1[5 + c] = p.pt[D] * a.P[c][t];
    }
    load23(p.lam, p.nc, eL, lam);
    acc_bar(lam, p, a);
#pragma unroll
    for (int k = 0; k < 8; ++k) F0[k] = fma(-p.c2h[D], a.m[k], F0[k]);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      F0[v] = fma(-p.c3[D], a.g[v][D], F0[v]);
      F1[v] = fma(-p.cs, a.g[v][t], F1[v]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c == D) continue;
      F0[5 + c] = fma(T(-0.25), a.P[c][D], F0[5 + c]);
      F1[5 + c] = fma(-p.pt[D], a.P[c][t], F1[5 + c]);
    }
  }
#pragma unroll 1
  for (int gp = 0; gp < 2; ++gp) {
    const T s = gp ? T(1) : T(-1);
    const T ht = s * p.q[t];
    T uL[8], uR[8], Fb[8], bL[8], bR[8];
    point_state<T, D>(cL, p.half[D], ht, uL);
    point_state<T, D>(cR, -p.half[D], ht, uR);
    const T bn = T(0.5) * (uL[5 + D] + uR[5 + D]);
    uL[5 + D] = uR[5 + D] = bn;
#pragma unroll
    for (int k = 0; k < 8; ++k) Fb[k] = fma(s, F1[k], F0[k]);
    hlld_vjp<T, D>(uL, uR, p.gamma, p.eps, Fb, bL, bR);
    T* F = p.F + (size_t)(32 * D + 8 * gp) * p.nF + le;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      F[(size_t)k * p.nF] = bL[k];
      F[(size_t)(16 + k) * p.nF] = bR[k];
    }
  }
}

// Both lower faces of the cells of rows [row0, row0 + rows), and the -y faces of
// the row above them.
template <typename T>
__global__ __launch_bounds__(64) void k_adj2m_face(PJ<T> p) {
  const int nb = gridDim.x >> 1;
  const int b = blockIdx.x;
  const int le = (b < nb ? b : b - nb) * 64 + threadIdx.x;
  if (le >= p.nF) return;
  const int lr = le / p.nx, i = le - lr * p.nx;
  int j = p.row0 + lr;
  if (j >= p.ny) j -= p.ny;
  const int e = j * p.nx + i;
  if (b < nb) {
    if (lr == p.rows) return;
    face_adjoint<T, 0>(p, j * p.nx + (i == 0 ? p.nx - 1 : i - 1), e, le);
  } else {
    face_adjoint<T, 1>(p, (j == 0 ? p.ny - 1 : j - 1) * p.nx + i, e, le);
  }
}

// Adds one face's entry of the face table to the coefficient adjoint g: side 0
// (the cell is L, its normal offset +h_D/2) or 1 (R, -h_D/2).
template <typename T, int D, int SIDE>
__device__ __forceinline__ void add_face(const PJ<T>& p, int le, T* g) {
  constexpr int t = 1 - D;
  const T hn = SIDE == 0 ? p.half[D] : -p.half[D];
  T S[8], Tt[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const T u0 = p.F[(size_t)(32 * D + 16 * SIDE + k) * p.nF + le];
    const T u1 = p.F[(size_t)(32 * D + 16 * SIDE + 8 + k) * p.nF + le];
    S[k] = u0 + u1;
    Tt[k] = u1 - u0;
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    g[3 * v] += S[v];
    g[3 * v + 1 + D] = fma(hn, S[v], g[3 * v + 1 + D]);
    g[3 * v + 1 + t] = fma(p.q[t], Tt[v], g[3 * v + 1 + t]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    g[15 + k] += S[5 + k];
    g[18 + bj(k, D)] = fma(T(bs(k, D)) * hn, S[5 + k], g[18 + bj(k, D)]);
    g[18 + bj(k, t)] = fma(T(bs(k, t)) * p.q[t], Tt[5 + k], g[18 + bj(k, t)]);
  }
}

// Volume term of cell e over the 2x2 Gauss points: adds its contribution to
// (dL/dW_e)^T lam to g.  Forward: grad_v[e] += 3 fe[e][v] / h_e^2,
// P[x][y] += F_y(Bx)/4, P[y][x] -= F_y(Bx)/4, P[z][x] += F_x(Bz)/4,
// P[z][y] += F_y(Bz)/4.
template <typename T>
__device__ void volume_adjoint(const T* ce, const AccBar<T>& ae, const PJ<T>& p, T* g) {
  T feb[2][5], indb[3];
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int v = 0; v < 5; ++v) feb[e][v] = p.c3[e] * ae.g[v][e];
  indb[0] = T(0.25) * (ae.P[0][1] - ae.P[1][0]);
  indb[1] = T(0.25) * ae.P[2][0];
  indb[2] = T(0.25) * ae.P[2][1];
#pragma unroll 1
  for (int gp = 0; gp < 4; ++gp) {
    const T o0 = (gp & 2) ? p.q[0] : -p.q[0];
    const T o1 = (gp & 1) ? p.q[1] : -p.q[1];
    T u[8], ub[8];
    point_state<T, 0>(ce, o0, o1, u);
    mhd_flux_vjp<T, 2>(u, p.gamma, feb, indb[0], -indb[1], -indb[2], ub);
    point_state_bar<T, 0>(ub, o0, o1, g);
  }
}

// lamW of one cell from the face table, its volume term and its own lam, then the
// transpose of the cell's own limiter: the adjoint of its gradients, field
// coefficients and the part its own mean takes are written out, and, for the six
// limited variables (rho .. E, the field), a message to the neighbour whose mean
// set the bound: a value and the neighbour's direction.  msg[s * nc + e] holds
// slot s, the codes of a cell 4 bits a slot (0: none, 1 + direction), the field
// component of slot 5 in bits 24 and 25.  Without a limiter lamW is the result.
template <typename T, bool LIM>
__global__ __launch_bounds__(256) void k_adj2m_cell(PJ<T> p) {
  const int le = blockIdx.x * 256 + threadIdx.x;
  if (le >= p.nx * p.rows) return;
  const int e = p.row0 * p.nx + le;
  const int lr = le / p.nx, i = le - lr * p.nx;
  T lw[23];
  {
    T ce[23], le_[23], g[23];
    load23(p.W, p.nc, e, ce);
    load23(p.lam, p.nc, e, le_);
#pragma unroll
    for (int k = 0; k < 23; ++k) g[k] = T(0);
    add_face<T, 0, 1>(p, le, g);
    add_face<T, 0, 0>(p, i == p.nx - 1 ? le - i : le + 1, g);
    add_face<T, 1, 1>(p, le, g);
    add_face<T, 1, 0>(p, le + p.nx, g);
    AccBar<T> ae;
    acc_bar(le_, p, ae);
    volume_adjoint(ce, ae, p, g);
    const double dt = p.dt_dev ? *p.dt_dev : p.dt_host;
    const T cid = (T)p.c_id, cL = (T)(p.c_L_over_dt * dt), cx = (T)p.c_extra;
#pragma unroll
    for (int k = 0; k < 23; ++k) {
      T o = fma(cL, g[k], cid * le_[k]);
      if (p.extra) o = fma(cx, p.extra[(size_t)k * p.nc + e], o);
      lw[k] = o;
    }
  }
  auto put = [&](int k, T x) { p.out[(size_t)k * p.nc + e] = x; };
  if (!LIM) {
#pragma unroll
    for (int k = 0; k < 23; ++k) put(k, lw[k]);
    return;
  }
  int nb[4];
  neighbours(e, p.nx, p.ny, nb);
  T c[23];
  load23(p.P, p.nc, e, c);
  unsigned code = 0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    T m[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) m[f] = p.P[(size_t)(3 * v) * p.nc + nb[f]];
    const T* g = c + 3 * v + 1;
    const auto r = limiter_decide<T, 2>(c[3 * v], m, g, p.half);
    T gb[2] = {r.alpha * lw[3 * v + 1], r.alpha * lw[3 * v + 2]};
    const T b = limiter_bar<T, 2>(r, lw[3 * v + 1] * g[0] + lw[3 * v + 2] * g[1], g, p.half, gb);
    const bool send = r.act && r.nbr != 0;
    put(3 * v, lw[3 * v] - (send ? b : T(0)));
    put(3 * v + 1, gb[0]);
    put(3 * v + 2, gb[1]);
    if (send) {
      code |= (unsigned)r.nbr << (4 * v);
      p.msg[(size_t)v * p.nc + e] = b;
    }
  }
  // the field: one alpha, the smallest of the components' (the first on ties)
  LimDecision<T> rB{};
  rB.alpha = T(1);
  T gB[2] = {T(0), T(0)};
  int cB = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T m[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) m[f] = p.P[(size_t)(15 + k) * p.nc + nb[f]];
    const T g[2] = {T(bs(k, 0)) * c[18 + bj(k, 0)], T(bs(k, 1)) * c[18 + bj(k, 1)]};
    const auto r = limiter_decide<T, 2>(c[15 + k], m, g, p.half);
    if (r.alpha < rB.alpha) {
      rB = r;
      gB[0] = g[0];
      gB[1] = g[1];
      cB = k;
    }
  }
  T ab = T(0), fb[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    ab = fma(lw[18 + j], c[18 + j], ab);
    fb[j] = rB.alpha * lw[18 + j];
  }
  T gb[2] = {T(0), T(0)};
  const T b = limiter_bar<T, 2>(rB, ab, gB, p.half, gb);
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int d = 0; d < 2; ++d) fb[bj(k, d)] += k == cB ? T(bs(k, d)) * gb[d] : T(0);
  const bool send = rB.act && rB.nbr != 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) put(15 + k, lw[15 + k] - (send && k == cB ? b : T(0)));
#pragma unroll
  for (int j = 0; j < 5; ++j) put(18 + j, fb[j]);
  if (send) {
    code |= ((unsigned)rB.nbr << 20) | ((unsigned)cB << 24);
    p.msg[(size_t)5 * p.nc + e] = b;
  }
  p.code[e] = code;
}

// Adds to each mean adjoint the messages its face neighbours sent it.  A
// message of cell n in direction g arrives at n's neighbour there, which sees n
// in the opposite direction g ^ 1 (also where a cell is its own neighbour).
template <typename T>
__global__ __launch_bounds__(256) void k_adj2m_msg(PJ<T> p) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= p.nc) return;
  int nb[4];
  neighbours(e, p.nx, p.ny, nb);
  unsigned code[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) code[f] = p.code[nb[f]];
  T add[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) add[k] = T(0);
  unsigned hit = 0;
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int s = 0; s < 6; ++s)
      if (((code[f] >> (4 * s)) & 15u) == (unsigned)((f ^ 1) + 1)) {
        const T x = p.msg[(size_t)s * p.nc + nb[f]];
        const int cB = (int)(code[f] >> 24);
        if (s < 5) {
          add[s] += x;
          hit |= 1u << s;
        } else {
#pragma unroll
          for (int k = 0; k < 3; ++k) add[5 + k] += k == cB ? x : T(0);
          hit |= 32u << cB;
        }
      }
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (hit >> k & 1u) p.out[(size_t)mean_index(k) * p.nc + e] += add[k];
}

template <typename T>
PJ<T> make_adj_params(const dg_mesh* m, const double* dt_dev, double dt) {
  PJ<T> p{};
  p.dt_dev = dt_dev;
  p.dt_host = dt;
  p.nx = m->c2.nx;
  p.ny = m->c2.ny;
  p.nc = (int)m->ncells;
  p.gamma = (T)m->cfg.gamma;
  p.eps = (T)(m->cfg.precision == DG_FP64 ? 1e-12 : 1e-6);  // as the forward HLLD
  const double h[2] = {m->c2.hx, m->c2.hy};
  const double s3 = 1.7320508075688772;
  for (int d = 0; d < 2; ++d) {
    p.c2h[d] = (T)(0.5 / h[d]);
    p.c3[d] = (T)(3.0 / (h[d] * h[d]));
    p.pt[d] = (T)(h[1 - d] / (4.0 * s3 * h[d]));
    p.half[d] = (T)(0.5 * h[d]);
    p.q[d] = (T)(0.5 * h[d] / s3);
  }
  p.cs = (T)(s3 / (h[0] * h[1]));
  const double mx = h[0] * h[0] / 12.0, my = h[1] * h[1] / 12.0;
  p.imu[0] = (T)(1.0 / mx);
  p.imu[1] = (T)(1.0 / my);
  p.imu[2] = (T)(1.0 / (mx + my));
  return p;
}

// Rows whose face table fits the budget (at least one), shared evenly.
int chunk_rows(const dg_mesh* m) {
  const int ny = m->c2.ny;
  const size_t row = kFaceVals * m->elem * (size_t)m->c2.nx;
  const int most = (int)std::min<size_t>((size_t)ny, std::max<size_t>(kAdjFaceBudget / row, 2) - 1);
  const int chunks = (ny + most - 1) / most;
  return (ny + chunks - 1) / chunks;
}

template <typename T>
hipError_t adjoint_t(const dg_mesh* m, const void* U, const void* V1, const double* dt_dev,
                     double dt, const void* lam_np1, void* lam_n, void* ws1, void* ws2,
                     void* scratch, hipStream_t s) {
  const bool lim = m->cfg.limiter == DG_LIMITER_MINMOD;
  const dim3 block(256);
  const PJ<T> p = make_adj_params<T>(m, dt_dev, dt);
  const int chunk = chunk_rows(m);
  hipError_t e = hipSuccess;
  auto adj_stage = [&](const void* P, const void* lam, const void* extra, double c_id,
                       double c_L_over_dt, double c_extra, void* out) -> hipError_t {
    // W = Pi(P) into ws1; out = Pi_P^T lamW
    const void* W = P;
    if (lim) {
      hipError_t r = launch_mhd2d(m, kLimit, P, nullptr, ws1, nullptr, 0.0, 0.0, nullptr, s);
      if (r != hipSuccess) return r;
      W = ws1;
    }
    PJ<T> a = p;
    a.W = static_cast<const T*>(W);
    a.P = static_cast<const T*>(P);
    a.lam = static_cast<const T*>(lam);
    a.extra = static_cast<const T*>(extra);
    a.c_id = c_id;
    a.c_L_over_dt = c_L_over_dt;
    a.c_extra = c_extra;
    a.out = static_cast<T*>(out);
    a.msg = static_cast<T*>(scratch);
    a.code = reinterpret_cast<unsigned*>(a.msg + (size_t)6 * m->ncells);
    a.F = a.msg + (size_t)7 * m->ncells;
    for (a.row0 = 0; a.row0 < p.ny; a.row0 += chunk) {
      a.rows = std::min(chunk, p.ny - a.row0);
      a.nF = p.nx * (a.rows + 1);
      hipLaunchKernelGGL((k_adj2m_face<T>), dim3(2 * ((a.nF + 63) / 64)), dim3(64), 0, s, a);
      const dim3 cells((p.nx * a.rows + 255) / 256);
      if (lim)
        hipLaunchKernelGGL((k_adj2m_cell<T, true>), cells, block, 0, s, a);
      else
        hipLaunchKernelGGL((k_adj2m_cell<T, false>), cells, block, 0, s, a);
    }
    if (lim)
      hipLaunchKernelGGL((k_adj2m_msg<T>), dim3((p.nc + 255) / 256), block, 0, s, a);
    return hipGetLastError();
  };
  // stage 2: ws2 = lam_V1 = Pi_V1^T [lam'/2 + (dt/2) L^T lam']
  e = adj_stage(V1, lam_np1, nullptr, 0.5, 0.5, 0.0, ws2);
  if (e != hipSuccess) return e;
  // stage 1: lam_n = Pi_U^T [lam_V1 + dt L^T lam_V1 + lam'/2]
  return adj_stage(U, ws2, lam_np1, 1.0, 1.0, 0.5, lam_n);
}

}  // namespace

size_t adjoint_mhd2d_scratch(const dg_mesh* m) {
  return (7 * (size_t)m->ncells + kFaceVals * (size_t)m->c2.nx * (chunk_rows(m) + 1)) * m->elem;
}

hipError_t launch_adjoint_mhd2d(const dg_mesh* m, const void* U, const void* V1,
                                const double* dt_dev, double dt, const void* lam_np1,
                                void* lam_n, void* ws1, void* ws2, void* scratch, hipStream_t s) {
  if (m->cfg.precision == DG_FP64)
    return adjoint_t<double>(m, U, V1, dt_dev, dt, lam_np1, lam_n, ws1, ws2, scratch, s);
  return adjoint_t<float>(m, U, V1, dt_dev, dt, lam_np1, lam_n, ws1, ws2, scratch, s);
}

}  // namespace dg
