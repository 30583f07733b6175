// Discrete adjoint of the 3D ideal-MHD Cartesian SSP-RK2 step: the HLLD flux of
// Sec. 2.3 at 2x2 Gauss points per face on the face-averaged normal field, the
// locally divergence-free field basis V1..V11 of Sec. 2.2 and the limiter of
// Sec. 2.5 with one alpha for B; dt frozen, the branch the forward step takes,
// ties to the first argument of min and max in the order self, -x, +x, -y,
// +y, -z, +z (the CPU oracle's dual-number conventions).
//
// The same two adjoint stages as in two dimensions (stage 2: P = V1,
// lam = lam', c_id = 1/2, c_L = dt/2; stage 1: P = U, lam = lam_V1, c_id = 1,
// c_L = dt, extra = lam' with weight 1/2), each the forward limiter (k_lim3d)
// into a workspace, then chunk by chunk of planes (of rows where two planes are too
// many for the face table), without atomics:
//   k_adj3m_face one thread per half face (two of the four Gauss points), each
//                face once: flux cotangents from the transposed residual weights
//                of both adjacent cells, one reverse sweep through the HLLD flux
//                per Gauss point (hlld_vjp), both sides' point cotangents to a
//                face table (192 values a cell);
//   k_adj3m_cell lamW of a cell from its six faces' entries (the Gauss-point
//                extrapolation and the map from residual moments to a4..a11
//                transposed by hand) and its eight volume points, then the
//                transpose of its own limiter, with a message per limited variable
//                for the neighbour whose mean set the bound;
// and at last k_adj3m_msg, in which each cell adds its neighbours' messages.
// One wave per SIMD bounds k_adj3m_face (39% of the issue slots), the traffic of
// the face table k_adj3m_cell (two waves per SIMD at 84 B spilled a lane: 0.144
// against 0.162 ms without).  The chunks' tables take 256 MiB (64^3, one stage:
// two chunks 0.45 ms; five of 96 MiB 0.49; one of 600 MiB 0.46).  Measured (64^3,
// FP64, one adjoint stage): faces 0.28, cells 0.14, messages 0.013 ms; one thread
// per cell solving each face from both sides 0.98 + 0.05 ms; with a forward-mode
// solve per state component and every limiter that reads a cell differentiated
// 3.55 + 0.77 ms.  The adjoint step 8.77 -> 0.90 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dg_internal.h"
#include "dg_math.h"
#include "limiter_vjp.h"
#include "mhd_hlld_vjp.h"

namespace dg {

hipError_t launch_cart3d(const dg_mesh* m, int mode, const void* in, const void* u0, void* out,
                         const double* dt_dev, double dt_host, double cfl, double* dt_next,
                         hipStream_t s);

namespace {

constexpr int kNC3 = 31;
constexpr size_t kFaceVals3 = 192;  // face table: 3 axes, 4 Gauss points, 2 sides, 8 variables

// Coefficient layout (31 values): 4v the mean and 4v+1+d the gradient along d
// of rho, mx, my, mz, E (v = 0..4); 20..22 the means of Bx, By, Bz; 23..30
// a4..a11.  Mean index of conserved variable k (rho .. E, Bx, By, Bz).
__device__ __forceinline__ int mean3(int k) { return k < 5 ? 4 * k : 15 + k; }

// The gradient of B_c along d in a4..a11 (offsets 0..7):
//   grad Bx = (a10 + a11, a4, a5), grad By = (a6, -a10, a7), grad Bz = (a8, a9, -a11).
template <typename S>
__device__ __forceinline__ S dB3(const S* a, int c, int d) {
  if (c == 0) return d == 0 ? a[6] + a[7] : (d == 1 ? a[0] : a[1]);
  if (c == 1) return d == 0 ? a[2] : (d == 1 ? -a[6] : a[3]);
  return d == 0 ? a[4] : (d == 1 ? a[5] : -a[7]);
}

// Transpose of dB3: adds w times d(dB3(a, c, d))/da to abar.
template <typename T>
__device__ __forceinline__ void dB3_bar(int c, int d, T w, T* abar) {
  if (c == 0) {
    if (d == 0) {
      abar[6] += w;
      abar[7] += w;
    } else {
      abar[d == 1 ? 0 : 1] += w;
    }
  } else if (c == 1) {
    if (d == 1)
      abar[6] -= w;
    else
      abar[d == 0 ? 2 : 3] += w;
  } else {
    if (d == 2)
      abar[7] -= w;
    else
      abar[d == 0 ? 4 : 5] += w;
  }
}

template <typename T>
struct PJ3 {
  const T* W;
  const T* P;
  const T* lam;
  const T* extra;
  T* out;
  T* F;            // face table of the chunk at hand: [192][nF]
  T* msg;          // limiter messages: 6 values a cell
  unsigned* code;  // and their directions
  const double* dt_dev;
  double dt_host;
  double c_id, c_L_over_dt, c_extra;
  int nx, ny, nz, nc;
  int plane0, planes, cell0, nr;  // chunk at hand: nr cells (whole rows) from cell0 of these planes
  T gamma, eps;
  T c4h[3], c15[3], cs[3][3], pt[3][3], half[3], q[3], imu[3], ib[4];

  // cells of a plane in the table (one row more where the chunk has not all rows) and
  // of the table (computed: the FP64 arguments just fill seven cache lines, and an eighth
  // cost 0.5 us a launch)
  __host__ __device__ __forceinline__ int nt() const { return nr < nx * ny ? nr + nx : nr; }
  __host__ __device__ __forceinline__ int nF() const { return nt() * (planes + 1); }
};

template <typename T>
__device__ __forceinline__ void load31(const T* __restrict__ U, int nc, int e, T* c) {
#pragma unroll
  for (int k = 0; k < kNC3; ++k) c[k] = U[(size_t)k * nc + e];
}

// Face neighbours -x, +x, -y, +y, -z, +z of cell e (periodic).
__device__ __forceinline__ void neighbours3(int e, int nx, int ny, int nz, int* nb) {
  const int i = e % nx, j = (e / nx) % ny, k = e / (nx * ny);
  nb[0] = e - i + (i == 0 ? nx - 1 : i - 1);
  nb[1] = e - i + (i == nx - 1 ? 0 : i + 1);
  nb[2] = e + ((j == 0 ? ny - 1 : j - 1) - j) * nx;
  nb[3] = e + ((j == ny - 1 ? 0 : j + 1) - j) * nx;
  nb[4] = e + ((k == 0 ? nz - 1 : k - 1) - k) * nx * ny;
  nb[5] = e + ((k == nz - 1 ? 0 : k + 1) - k) * nx * ny;
}

// Adjoint of the residual accumulators from the adjoint of the time derivative
// (transpose of: identity for means and hydro gradients; a4 = P[x][y]/mu_y,
// a5 = P[x][z]/mu_z, a6 = P[y][x]/mu_x, a7 = P[y][z]/mu_z, a8 = P[z][x]/mu_x,
// a9 = P[z][y]/mu_y, (a10, a11) = ib (P[x][x] - P[y][y], P[x][x] - P[z][z])).
template <typename T>
struct AccBar3 {
  T m[8], g[5][3], P[3][3];
};

template <typename T>
__device__ __forceinline__ void acc_bar3(const T* lam, const PJ3<T>& p, AccBar3<T>& a) {
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    a.m[v] = lam[4 * v];
#pragma unroll
    for (int d = 0; d < 3; ++d) a.g[v][d] = lam[4 * v + 1 + d];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) a.m[5 + c] = lam[20 + c];
  a.P[0][1] = lam[23] * p.imu[1];
  a.P[0][2] = lam[24] * p.imu[2];
  a.P[1][0] = lam[25] * p.imu[0];
  a.P[1][2] = lam[26] * p.imu[2];
  a.P[2][0] = lam[27] * p.imu[0];
  a.P[2][1] = lam[28] * p.imu[1];
  const T r10 = p.ib[0] * lam[29] + p.ib[2] * lam[30];
  const T r11 = p.ib[1] * lam[29] + p.ib[3] * lam[30];
  a.P[0][0] = r10 + r11;
  a.P[1][1] = -r10;
  a.P[2][2] = -r11;
}

// State of a cell's polynomial at offset o from its centroid, and the
// transpose (the cotangent ub of the state added to the coefficient adjoint g).
template <typename T>
__device__ __forceinline__ void point3(const T* c, const T* o, T* u) {
#pragma unroll
  for (int v = 0; v < 5; ++v)
    u[v] = fma(c[4 * v + 3], o[2], fma(c[4 * v + 2], o[1], fma(c[4 * v + 1], o[0], c[4 * v])));
#pragma unroll
  for (int k = 0; k < 3; ++k)
    u[5 + k] = fma(dB3(c + 23, k, 2), o[2],
                   fma(dB3(c + 23, k, 1), o[1], fma(dB3(c + 23, k, 0), o[0], c[20 + k])));
}

template <typename T>
__device__ __forceinline__ void point3_bar(const T* ub, const T* o, T* g) {
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    g[4 * v] += ub[v];
#pragma unroll
    for (int d = 0; d < 3; ++d) g[4 * v + 1 + d] = fma(o[d], ub[v], g[4 * v + 1 + d]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    g[20 + k] += ub[5 + k];
#pragma unroll
    for (int d = 0; d < 3; ++d) dB3_bar(k, d, o[d] * ub[5 + k], g + 23);
  }
}

// Half of the -D face of cell eR: the two Gauss points at tangential offset
// s1 q_t1, s2 = -+ along t2 (t1 < t2 the other two axes): the cotangents of both
// sides' point states, to the face table.  The cotangent of a flux is the
// transpose of the forward accumulation, for the R cell (sigma +1) and L (-1):
//   mean_k += sigma F_k/(4 h_D)  (k not the normal field),
//   grad_v[D] -= 1.5 F_v/h_D^2,  grad_v[t_i] += sigma s_i (sqrt3/2) F_v/(h_D h_ti),
//   P[c][D] -= F_Bc/8 (c != D),  P[c][t_i] += sigma s_i h_ti F_Bc/(8 sqrt3 h_D),
// F0 its part common to both points and F1 the part that changes sign with s2.
template <typename T, int D>
__device__ __forceinline__ void face_adjoint3(const PJ3<T>& p, int eL, int eR, int half1, int le) {
  constexpr int t1 = D == 0 ? 1 : 0, t2 = D == 2 ? 1 : 2;
  const T s1 = half1 ? T(1) : T(-1);
  T F0[8], F1[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) F0[k] = F1[k] = T(0);
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const T sg = side == 0 ? T(-1) : T(1);
    T lam[kNC3];
    AccBar3<T> a;
    load31(p.lam, p.nc, side == 0 ? eL : eR, lam);
    acc_bar3(lam, p, a);
    const T g1 = sg * s1 * p.cs[D][t1], g2 = sg * p.cs[D][t2];
    const T b1 = sg * s1 * p.pt[D][t1], b2 = sg * p.pt[D][t2];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k != 5 + D) F0[k] = fma(sg * p.c4h[D], a.m[k], F0[k]);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      F0[v] = fma(-p.c15[D], a.g[v][D], fma(g1, a.g[v][t1], F0[v]));
      F1[v] = fma(g2, a.g[v][t2], F1[v]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c == D) continue;
      F0[5 + c] = fma(T(-0.125), a.P[c][D], fma(b1, a.P[c][t1], F0[5 + c]));
      F1[5 + c] = fma(b2, a.P[c][t2], F1[5 + c]);
    }
  }
  T cL[kNC3], cR[kNC3];
  load31(p.W, p.nc, eL, cL);
  load31(p.W, p.nc, eR, cR);
#pragma unroll 1
  for (int half2 = 0; half2 < 2; ++half2) {
    const T s2 = half2 ? T(1) : T(-1);
    T oL[3], oR[3];
    oL[D] = p.half[D];
    oR[D] = -p.half[D];
    oL[t1] = oR[t1] = s1 * p.q[t1];
    oL[t2] = oR[t2] = s2 * p.q[t2];
    T uL[8], uR[8], Fb[8], bL[8], bR[8];
    point3(cL, oL, uL);
    point3(cR, oR, uR);
    const T bn = T(0.5) * (uL[5 + D] + uR[5 + D]);
    uL[5 + D] = uR[5 + D] = bn;
#pragma unroll
    for (int k = 0; k < 8; ++k) Fb[k] = fma(s2, F1[k], F0[k]);
    hlld_vjp<T, D>(uL, uR, p.gamma, p.eps, Fb, bL, bR);
    T* F = p.F + (size_t)(64 * D + 32 * half1 + 8 * half2) * p.nF() + le;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      F[(size_t)k * p.nF()] = bL[k];
      F[(size_t)(16 + k) * p.nF()] = bR[k];
    }
  }
}

// The lower faces of the chunk's cells, the -z faces of the plane above them and,
// where the chunk has not all rows, the -y faces of the row above them.  One thread per
// half face; six half faces of 64 consecutive cells are neighbouring workgroups (they
// share the cells' rows).
template <typename T>
__global__ __launch_bounds__(64) void k_adj3m_face(PJ3<T> p) {
  const int b = blockIdx.x, part = b % 6;
  const int le = (b / 6) * 64 + threadIdx.x;
  if (le >= p.nF()) return;
  const int nxy = p.nx * p.ny;
  const int lp = le / p.nt(), r = le - lp * p.nt(), i = r % p.nx;
  int k = p.plane0 + lp, c = p.cell0 + r;  // plane, cell within it
  if (k >= p.nz) k -= p.nz;
  if (c >= nxy) c -= nxy;
  const int e = k * nxy + c;
  const int axis = part >> 1, half1 = part & 1;
  if ((axis < 2 && lp == p.planes) || (axis != 1 && r >= p.nr)) return;
  if (axis == 0)
    face_adjoint3<T, 0>(p, i == 0 ? e + p.nx - 1 : e - 1, e, half1, le);
  else if (axis == 1)
    face_adjoint3<T, 1>(p, c < p.nx ? e + nxy - p.nx : e - p.nx, e, half1, le);
  else
    face_adjoint3<T, 2>(p, k == 0 ? e + (p.nz - 1) * nxy : e - nxy, e, half1, le);
}

// Adds one face's entry of the face table to the coefficient adjoint g: side 0
// (the cell is L, its normal offset +h_D/2) or 1 (R, -h_D/2).
template <typename T, int D, int SIDE>
__device__ __forceinline__ void add_face3(const PJ3<T>& p, int le, T* g) {
  constexpr int t1 = D == 0 ? 1 : 0, t2 = D == 2 ? 1 : 2;
  const T hn = SIDE == 0 ? p.half[D] : -p.half[D];
  const T* F = p.F + (size_t)(64 * D + 16 * SIDE) * p.nF() + le;
  T S[8], A[8], B[8];  // sums over the four points, weighted 1, s1, s2
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const T f00 = F[(size_t)k * p.nF()], f01 = F[(size_t)(8 + k) * p.nF()];
    const T f10 = F[(size_t)(32 + k) * p.nF()], f11 = F[(size_t)(40 + k) * p.nF()];
    const T lo = f00 + f01, hi = f10 + f11;
    S[k] = lo + hi;
    A[k] = hi - lo;
    B[k] = (f01 - f00) + (f11 - f10);
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    g[4 * v] += S[v];
    g[4 * v + 1 + D] = fma(hn, S[v], g[4 * v + 1 + D]);
    g[4 * v + 1 + t1] = fma(p.q[t1], A[v], g[4 * v + 1 + t1]);
    g[4 * v + 1 + t2] = fma(p.q[t2], B[v], g[4 * v + 1 + t2]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    g[20 + k] += S[5 + k];
    dB3_bar(k, D, hn * S[5 + k], g + 23);
    dB3_bar(k, t1, p.q[t1] * A[5 + k], g + 23);
    dB3_bar(k, t2, p.q[t2] * B[5 + k], g + 23);
  }
}

// Volume term over the 2x2x2 Gauss points (forward: grad_v[e] += 1.5 fe/h_e^2,
// P[x][y] += F_y(Bx)/8, P[y][x] -= F_y(Bx)/8, P[x][z] += F_z(Bx)/8,
// P[z][x] -= F_z(Bx)/8, P[y][z] += F_z(By)/8, P[z][y] -= F_z(By)/8).
template <typename T>
__device__ void volume_adjoint3(const T* ce, const AccBar3<T>& ae, const PJ3<T>& p, T* g) {
  T feb[3][5], indb[3];
#pragma unroll
  for (int e = 0; e < 3; ++e)
#pragma unroll
    for (int v = 0; v < 5; ++v) feb[e][v] = p.c15[e] * ae.g[v][e];
  indb[0] = T(0.125) * (ae.P[0][1] - ae.P[1][0]);
  indb[1] = T(0.125) * (ae.P[0][2] - ae.P[2][0]);
  indb[2] = T(0.125) * (ae.P[1][2] - ae.P[2][1]);
#pragma unroll 1
  for (int gp = 0; gp < 8; ++gp) {
    const T o[3] = {(gp & 4) ? p.q[0] : -p.q[0], (gp & 2) ? p.q[1] : -p.q[1],
                    (gp & 1) ? p.q[2] : -p.q[2]};
    T u[8], ub[8];
    point3(ce, o, u);
    mhd_flux_vjp<T, 3>(u, p.gamma, feb, indb[0], indb[1], indb[2], ub);
    point3_bar(ub, o, g);
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
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_adj3m_cell(PJ3<T> p) {
  const int lc = blockIdx.x * 256 + threadIdx.x;
  if (lc >= p.nr * p.planes) return;
  const int lp = lc / p.nr, r = lc - lp * p.nr;
  const int e = (p.plane0 + lp) * (p.nx * p.ny) + p.cell0 + r;
  T lw[kNC3];
  {
    const int lr = r / p.nx, i = r - lr * p.nx;
    const int le = lp * p.nt() + r;
    T g[kNC3];
#pragma unroll
    for (int k = 0; k < kNC3; ++k) g[k] = T(0);
    add_face3<T, 0, 1>(p, le, g);
    add_face3<T, 0, 0>(p, i == p.nx - 1 ? le - i : le + 1, g);
    add_face3<T, 1, 1>(p, le, g);
    add_face3<T, 1, 0>(p, lr == p.ny - 1 ? le - lr * p.nx : le + p.nx, g);
    add_face3<T, 2, 1>(p, le, g);
    add_face3<T, 2, 0>(p, le + p.nt(), g);
    T ce[kNC3], la[kNC3];
    load31(p.W, p.nc, e, ce);
    load31(p.lam, p.nc, e, la);
    AccBar3<T> ae;
    acc_bar3(la, p, ae);
    volume_adjoint3(ce, ae, p, g);
    const double dt = p.dt_dev ? *p.dt_dev : p.dt_host;
    const T cid = (T)p.c_id, cL = (T)(p.c_L_over_dt * dt), cx = (T)p.c_extra;
#pragma unroll
    for (int k = 0; k < kNC3; ++k) {
      T o = fma(cL, g[k], cid * la[k]);
      if (p.extra) o = fma(cx, p.extra[(size_t)k * p.nc + e], o);
      lw[k] = o;
    }
  }
  auto put = [&](int k, T x) { p.out[(size_t)k * p.nc + e] = x; };
  if (!LIM) {
#pragma unroll
    for (int k = 0; k < kNC3; ++k) put(k, lw[k]);
    return;
  }
  int nb[6];
  neighbours3(e, p.nx, p.ny, p.nz, nb);
  T c[kNC3];
  load31(p.P, p.nc, e, c);
  unsigned code = 0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    T m[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) m[f] = p.P[(size_t)(4 * v) * p.nc + nb[f]];
    const T* g = c + 4 * v + 1;
    const auto r = limiter_decide<T, 3>(c[4 * v], m, g, p.half);
    T gb[3] = {r.alpha * lw[4 * v + 1], r.alpha * lw[4 * v + 2], r.alpha * lw[4 * v + 3]};
    const T b = limiter_bar<T, 3>(r, lw[4 * v + 1] * g[0] + lw[4 * v + 2] * g[1] + lw[4 * v + 3] * g[2], g, p.half, gb);
    const bool send = r.act && r.nbr != 0;
    put(4 * v, lw[4 * v] - (send ? b : T(0)));
    put(4 * v + 1, gb[0]);
    put(4 * v + 2, gb[1]);
    put(4 * v + 3, gb[2]);
    if (send) {
      code |= (unsigned)r.nbr << (4 * v);
      p.msg[(size_t)v * p.nc + e] = b;
    }
  }
  // the field: one alpha, the smallest of the components' (the first on ties)
  LimDecision<T> rB{};
  rB.alpha = T(1);
  T gB[3] = {T(0), T(0), T(0)};
  int cB = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T m[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) m[f] = p.P[(size_t)(20 + k) * p.nc + nb[f]];
    const T g[3] = {dB3(c + 23, k, 0), dB3(c + 23, k, 1), dB3(c + 23, k, 2)};
    const auto r = limiter_decide<T, 3>(c[20 + k], m, g, p.half);
    if (r.alpha < rB.alpha) {
      rB = r;
      gB[0] = g[0];
      gB[1] = g[1];
      gB[2] = g[2];
      cB = k;
    }
  }
  T ab = T(0), fb[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    ab = fma(lw[23 + j], c[23 + j], ab);
    fb[j] = rB.alpha * lw[23 + j];
  }
  T gb[3] = {T(0), T(0), T(0)};
  const T b = limiter_bar<T, 3>(rB, ab, gB, p.half, gb);
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int d = 0; d < 3; ++d) dB3_bar(k, d, k == cB ? gb[d] : T(0), fb);
  const bool send = rB.act && rB.nbr != 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) put(20 + k, lw[20 + k] - (send && k == cB ? b : T(0)));
#pragma unroll
  for (int j = 0; j < 8; ++j) put(23 + j, fb[j]);
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
__global__ __launch_bounds__(256) void k_adj3m_msg(PJ3<T> p) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= p.nc) return;
  int nb[6];
  neighbours3(e, p.nx, p.ny, p.nz, nb);
  unsigned code[6];
#pragma unroll
  for (int f = 0; f < 6; ++f) code[f] = p.code[nb[f]];
  T add[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) add[k] = T(0);
  unsigned hit = 0;
#pragma unroll
  for (int f = 0; f < 6; ++f)
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
    if (hit >> k & 1u) p.out[(size_t)mean3(k) * p.nc + e] += add[k];
}

template <typename T>
PJ3<T> make_adj3_params(const dg_mesh* m, const double* dt_dev, double dt) {
  PJ3<T> p{};
  p.dt_dev = dt_dev;
  p.dt_host = dt;
  p.nx = m->c3.nx;
  p.ny = m->c3.ny;
  p.nz = m->c3.nz;
  p.nc = (int)m->ncells;
  p.gamma = (T)m->cfg.gamma;
  p.eps = (T)(m->cfg.precision == DG_FP64 ? 1e-12 : 1e-6);  // as the forward HLLD
  const double h[3] = {m->c3.hx, m->c3.hy, m->c3.hz};
  const double s3 = 1.7320508075688772;
  for (int d = 0; d < 3; ++d) {
    p.c4h[d] = (T)(0.25 / h[d]);
    p.c15[d] = (T)(1.5 / (h[d] * h[d]));
    p.half[d] = (T)(0.5 * h[d]);
    p.q[d] = (T)(0.5 * h[d] / s3);
    p.imu[d] = (T)(12.0 / (h[d] * h[d]));
    for (int t = 0; t < 3; ++t) {
      p.cs[d][t] = (T)(0.5 * s3 / (h[d] * h[t]));
      p.pt[d][t] = (T)(h[t] / (8.0 * s3 * h[d]));
    }
  }
  const double mx = h[0] * h[0] / 12.0, my = h[1] * h[1] / 12.0, mz = h[2] * h[2] / 12.0;
  const double det = (mx + my) * (mx + mz) - mx * mx;
  p.ib[0] = (T)((mx + mz) / det);
  p.ib[1] = (T)(-mx / det);
  p.ib[2] = (T)(-mx / det);
  p.ib[3] = (T)((mx + my) / det);
  return p;
}

// Planes, and rows of them, whose face table fits the budget, shared evenly: whole
// planes, at least one, or where two planes are over it at least one row of one.
struct Chunk3 {
  int planes, rows, rt;
};

Chunk3 chunk3(const dg_mesh* m) {
  const int ny = m->c3.ny, nz = m->c3.nz;
  const size_t row = kFaceVals3 * m->elem * (size_t)m->c3.nx;
  auto share = [](int n, size_t most) {
    const int chunks = (int)((n + most - 1) / most);
    return (n + chunks - 1) / chunks;
  };
  const size_t planes = kAdjFaceBudget / (row * ny);
  if (planes >= 2) return {share(nz, planes - 1), ny, ny};
  const int rows = share(ny, std::max<size_t>(kAdjFaceBudget / (2 * row), 2) - 1);
  return {1, rows, rows < ny ? rows + 1 : ny};
}

template <typename T>
hipError_t adjoint3_t(const dg_mesh* m, const void* U, const void* V1, const double* dt_dev,
                      double dt, const void* lam_np1, void* lam_n, void* ws1, void* ws2,
                      void* scratch, hipStream_t s) {
  const bool lim = m->cfg.limiter == DG_LIMITER_MINMOD;
  const PJ3<T> p = make_adj3_params<T>(m, dt_dev, dt);
  const Chunk3 chunk = chunk3(m);
  auto adj_stage = [&](const void* P, const void* lam, const void* extra, double c_id,
                       double c_L_over_dt, double c_extra, void* out) -> hipError_t {
    // W = Pi(P) into ws1; out = Pi_P^T lamW
    const void* W = P;
    if (lim) {
      hipError_t r = launch_cart3d(m, kLimit, P, nullptr, ws1, nullptr, 0.0, 0.0, nullptr, s);
      if (r != hipSuccess) return r;
      W = ws1;
    }
    PJ3<T> a = p;
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
    for (int c = 0, nr = (p.ny + chunk.rows - 1) / chunk.rows; (c / nr) * chunk.planes < p.nz; ++c) {
      a.plane0 = (c / nr) * chunk.planes;
      a.planes = std::min(chunk.planes, p.nz - a.plane0);
      const int row0 = (c % nr) * chunk.rows, rows = std::min(chunk.rows, p.ny - row0);
      a.cell0 = p.nx * row0;
      a.nr = p.nx * rows;
      hipLaunchKernelGGL((k_adj3m_face<T>), dim3(6 * ((a.nF() + 63) / 64)), dim3(64), 0, s, a);
      const dim3 cells((a.nr * a.planes + 255) / 256);
      if (lim)
        hipLaunchKernelGGL((k_adj3m_cell<T, true>), cells, dim3(256), 0, s, a);
      else
        hipLaunchKernelGGL((k_adj3m_cell<T, false>), cells, dim3(256), 0, s, a);
    }
    if (lim)
      hipLaunchKernelGGL((k_adj3m_msg<T>), dim3((p.nc + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
  };
  // stage 2: ws2 = lam_V1, then stage 1: lam_n
  hipError_t e = adj_stage(V1, lam_np1, nullptr, 0.5, 0.5, 0.0, ws2);
  if (e != hipSuccess) return e;
  return adj_stage(U, ws2, lam_np1, 1.0, 1.0, 0.5, lam_n);
}

}  // namespace

size_t adjoint_mhd3d_scratch(const dg_mesh* m) {
  const Chunk3 c = chunk3(m);
  return (7 * (size_t)m->ncells + kFaceVals3 * (size_t)m->c3.nx * c.rt * (c.planes + 1)) * m->elem;
}

hipError_t launch_adjoint_mhd3d(const dg_mesh* m, const void* U, const void* V1,
                                const double* dt_dev, double dt, const void* lam_np1,
                                void* lam_n, void* ws1, void* ws2, void* scratch, hipStream_t s) {
  if (m->cfg.precision == DG_FP64)
    return adjoint3_t<double>(m, U, V1, dt_dev, dt, lam_np1, lam_n, ws1, ws2, scratch, s);
  return adjoint3_t<float>(m, U, V1, dt_dev, dt, lam_np1, lam_n, ws1, ws2, scratch, s);
}

}  // namespace dg
