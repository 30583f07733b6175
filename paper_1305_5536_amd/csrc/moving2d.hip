// 2D Euler DG on a moving periodic Voronoi mesh (Sec. 2.3) with the
// MUSCL-Hancock step (Sec. 2.4), on gfx950.
//
// The mesh is the Voronoi tessellation of generators that move with their
// cell's fluid velocity (mean momentum over mean density, constant over a
// step).  Every step rebuilds it on the GPU, cell by cell, with no global
// triangulation; the one atomic counts the cells whose ring is not kept (the order in
// which they are listed varies from run to run, no result depends on it):
//   * the cell of generator i is the intersection of the half-planes closer to
//     i than to each candidate j; the candidates are i's neighbours and their
//     neighbours in the previous mesh (a cell's new neighbours over one CFL
//     step were among them).  Over one step most cells keep their neighbours:
//     the previous ring is kept where its vertices lie in the half-plane of every
//     candidate.  The faces of the other cells are found by walking around the
//     cell counter-clockwise from the nearest candidate: the next face is the
//     candidate whose bisector first cuts the current face's bisector (no
//     polygon is stored, only the ring of neighbours);
//   * each Voronoi vertex is then recomputed as the circumcentre of its three
//     generators, in the frame of the smallest of the three indices, so that
//     every cell that shares a vertex or a face derives it from the same
//     operands (a face between two workgroups of the update is solved by both; the
//     canonical operands make the two results agree);
//   * faces shorter than 1e-10 times their generators' distance (four nearly
//     cocircular generators) are dropped by both cells;
//   * areas, centroids and second moments (the mass matrix of Sec. 2.2, which
//     a moving mesh recomputes every step) are the exact polygon moments.
// A cell whose candidates do not bound it, a polygon beyond the capacities
// below, or a neighbour that does not list the cell back, latches status bit 2
// (reported by dg_check).  The kernels over all cells map their blocks XCD by XCD
// (xcd_remap): with cells numbered along a space-filling curve each XCD's L2
// then holds the positions, rings and states of one compact region, which the
// neighbour gathers reuse.
//
// One step, n -> n+1 (sets: t^n, the half step, t^{n+1}):
//   k_mv_lim   limiter on the mesh of t^n (none, the Arepo limiter on the
//              conserved coefficients, or the WENO-type limiter on primitive
//              variables with a least-squares stencil slope), and the
//              generator positions at t^{n+1/2} and t^{n+1};
//   k_mv_check, k_mv_walk, k_mv_geom  the mesh of the half-step generators;
//   k_mv_upd   the half-step mesh: for each face (once) and Gauss point,
//              both cells' half-step primitive predictions (centred at the
//              t^n centroids) at the point, boosted into the frame of the face
//              there (the bisector's velocity), the Riemann flux (HLL or
//              exact) in that frame carried back to the lab frame
//              (F_m = F - U w^T); the volume flux F - U w_e^T on the half-step
//              cell's 4-point rule; out: the conserved totals V^n ubar +
//              dt (...) and the first moments about the cell's origin carried
//              along with w_e (c^n + t w_e);
//   k_mv_check, k_mv_walk, k_mv_geom  the mesh of t^{n+1}, then the new state: means = totals /
//              V^{n+1}, gradients = (M^{n+1})^-1 (moments - (c^{n+1} - c^n -
//              dt w_e) totals), and the cell's CFL bound.
// Geometry is FP64 (absolute positions in a box); the state is T.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "dg_internal.h"
#include "dg_math.h"
#include "euler_exact.h"

namespace dg {

constexpr int kRing = 16;  // neighbours a cell may have
constexpr int kFast = 8;   // neighbours of a cell whose ring k_mv_check can keep
constexpr int kGeo = 6;    // V, centroid - generator (2), Mxx, Mxy, Myy
constexpr int kWalkBlocks = 2048;  // most workgroups of the walk
constexpr int kCand = 40;  // distinct candidates of a cell that a thread can walk

struct MVDev {
  int n = 0;
  double box[2] = {1.0, 1.0};
  int motion = 1;
  int cur = 0, nxt = 2;  // sets holding t^n and t^{n+1}; set 1 is the half step
  // [4][n]: x block, y block, then the same positions interleaved (x, y) per
  // generator, which the walk gathers with one 16-byte load per candidate
  double* pos[3] = {nullptr, nullptr, nullptr};
  int* ring[3] = {nullptr, nullptr, nullptr};    // [n][kRing], counter-clockwise
  int* deg[3] = {nullptr, nullptr, nullptr};     // [n]
  double* geo[3] = {nullptr, nullptr, nullptr};  // [kGeo][n]
  void* ua = nullptr;                            // limited state
  double2* mid = nullptr;                        // [kRing][n]: face midpoints of t^n
  void* pred = nullptr;                          // [14][n]: predictions and velocities
  double2* shift = nullptr;                      // [n]: half-step generator - t^n centroid
  int* list = nullptr;                           // [n + 1]: cells to walk, their count last
  bool timing = false;                           // record events around each kernel
  std::vector<hipEvent_t> ev;                    // 5 per timed step
};

namespace {

// One set of mesh arrays as kernels see it.
struct MSet {
  const double* x;  // x block of the positions (y = x + n, interleaved pairs from x + 2n)
  const int* ring;
  const int* deg;
  const double* geo;
};
struct MOut {
  double* x;
  int* ring;
  int* deg;
  double* geo;
};

template <typename T>
struct PM {
  const T* __restrict__ in;
  const T* __restrict__ ua;
  T* __restrict__ ua_out;
  T* __restrict__ out;
  const double* dt_dev;
  double dt_host;
  int* status;
  double* dtpart;
  int n;
  double Lx, Ly;
  T gamma;
  int motion;
  int* list;      // cells whose ring k_mv_check could not keep
  int* count;     // and their number
  int write_pos;  // k_mv_lim: write the half-step and next positions
  MSet s0;        // t^n
  MSet sh;        // half step
  const double2* mid;    // [kRing][n] face midpoints of t^n from the generators
  double2* mid_out;      // k_mv_geom: those of the mesh it finishes (NULL: not kept)
  const T* pred;         // [14][n] half-step prediction (12) and velocity of each cell
  T* pred_out;
  const double2* shift;  // [n] half-step generator - t^n centroid
  double2* shift_out;
  double* xh;     // positions written by k_mv_lim
  double* x1;
};

// The periodic box and its inverse sides.
struct PM_box {
  double Lx, Ly, iLx, iLy;
};

// Minimum image.  1 / L is loop-invariant (a division here was a quarter of the
// instructions of k_mv_geom; the step 0.465 -> 0.451 ms at 512^2) and taken a rounding
// low, so that d = L/2 stays unwrapped, as with d / L.
__device__ __forceinline__ double mimg(double d, double L) {
  return d - L * rint(d * (0x1.fffffffffffffp-1 / L));
}

// x + s w wrapped into [0, L), rounded as (s w) then the sum.
__device__ __forceinline__ double advance(double x, double s, double w, double L) {
#pragma clang fp contract(off)
  const double y = x + s * w;
  if (y < 0.0) return y + L;
  if (y >= L) return y - L;
  return y;
}

// Voronoi vertex of generators a, b, c (their circumcentre) as an offset from
// the smallest of the three indices, which is returned in f.  Worked from
// minimum-image offsets in that frame, without contraction, so that every cell
// sharing the vertex gets the same bits.
struct Vertex {
  double x, y;
  double2 origin;  // position of generator f
  int f;
};

__device__ __forceinline__ Vertex vertex(const double2* __restrict__ P, double Lx, double Ly,
                                         int a, int b, int c) {
#pragma clang fp contract(off)
  int t;
  if (a > b) { t = a; a = b; b = t; }
  if (b > c) { t = b; b = c; c = t; }
  if (a > b) { t = a; a = b; b = t; }
  const double2 pa = P[a], pb = P[b], pc = P[c];
  const double px = mimg(pb.x - pa.x, Lx), py = mimg(pb.y - pa.y, Ly);
  const double qx = mimg(pc.x - pa.x, Lx), qy = mimg(pc.y - pa.y, Ly);
  const double D = 2.0 * (px * qy - py * qx);
  const double pp = px * px + py * py, qq = qx * qx + qy * qy;
  return Vertex{(qy * pp - py * qq) / D, (px * qq - qx * pp) / D, pa, a};
}

// The vertex as an offset from generator g at position pg.
__device__ __forceinline__ void vertex_from(const Vertex& v, double Lx, double Ly, int g, double2 pg,
                                            double& ox, double& oy) {
#pragma clang fp contract(off)
  ox = v.x;
  oy = v.y;
  if (v.f != g) {
    ox += mimg(v.origin.x - pg.x, Lx);
    oy += mimg(v.origin.y - pg.y, Ly);
  }
}

// Circumcentre of generators a, b, c as an offset from generator f.
__device__ __forceinline__ void circumcentre(const double* __restrict__ X, int n, double Lx,
                                          double Ly, int a, int b, int c, int f, double& ox,
                                          double& oy) {
  // the interleaved copy of the positions: one 16-byte load per generator
  const double2* P = reinterpret_cast<const double2*>(X + 2 * (size_t)n);
  vertex_from(vertex(P, Lx, Ly, a, b, c), Lx, Ly, f, P[f], ox, oy);
}

// Face between cells L < R whose Voronoi edge ends at the vertices va and vb:
// endpoints (from L's generator) ordered so that the normal (e_y, -e_x)/|e|
// points from L towards R, the generator offset dLR, and the length.  Every
// argument order gives the same bits.
struct FaceG {
  double ax, ay, bx, by;  // endpoints
  double dx, dy;          // R's generator - L's generator
  double A, nx, ny;
};

__device__ __forceinline__ void face_geometry(double Lx, double Ly, int L, double2 pL, double2 pR,
                                              const Vertex& va, const Vertex& vb, FaceG& g) {
#pragma clang fp contract(off)
  double ax, ay, bx, by;
  vertex_from(va, Lx, Ly, L, pL, ax, ay);
  vertex_from(vb, Lx, Ly, L, pL, bx, by);
  const double dx = mimg(pR.x - pL.x, Lx), dy = mimg(pR.y - pL.y, Ly);
  double ex = bx - ax, ey = by - ay;
  if (ey * dx - ex * dy < 0.0) {
    double t = ax; ax = bx; bx = t;
    t = ay; ay = by; by = t;
    ex = -ex;
    ey = -ey;
  }
  g.ax = ax;
  g.ay = ay;
  g.bx = bx;
  g.by = by;
  g.dx = dx;
  g.dy = dy;
  g.A = sqrt(ex * ex + ey * ey);
  g.nx = ey / g.A;
  g.ny = -ex / g.A;
}

// Polygon moments about the generator, one edge of the polygon at a time: area,
// first and second moments of the fan triangles from the generator.
struct Moments {
  double V = 0, m1x = 0, m1y = 0, mxx = 0, mxy = 0, myy = 0;
  __device__ __forceinline__ void add(double e0x, double e0y, double e1x, double e1y) {
    const double ar = 0.5 * (e0x * e1y - e0y * e1x);
    const double sx = e0x + e1x, sy = e0y + e1y;
    V += ar;
    m1x += ar * sx / 3.0;
    m1y += ar * sy / 3.0;
    const double w = ar / 12.0;
    mxx += w * (e0x * e0x + e1x * e1x + sx * sx);
    mxy += w * (e0x * e0y + e1x * e1y + sx * sy);
    myy += w * (e0y * e0y + e1y * e1y + sy * sy);
  }
  __device__ __forceinline__ void geometry(double* geo) const {
    const double cx = m1x / V, cy = m1y / V;
    geo[0] = V;
    geo[1] = cx;
    geo[2] = cy;
    geo[3] = mxx - V * cx * cx;
    geo[4] = mxy - V * cx * cy;
    geo[5] = myy - V * cy * cy;
  }
};

// Vertices of cell e of a mesh set (offsets from its generator): vertex k is
// the circumcentre of (e, ring[k-1], ring[k]).
__device__ __forceinline__ int cell_polygon(const MSet& s, int n, double Lx, double Ly, int e,
                                            double* vx, double* vy, int* nb) {
  const int d = min(s.deg[e], kRing);
  for (int k = 0; k < d; ++k) nb[k] = s.ring[e * kRing + k];
  for (int k = 0; k < d; ++k)
    circumcentre(s.x, n, Lx, Ly, e, nb[k == 0 ? d - 1 : k - 1], nb[k], e, vx[k], vy[k]);
  return d;
}

template <typename T>
__device__ __forceinline__ void load12(const T* __restrict__ U, int n, int e, T* q) {
#pragma unroll
  for (int k = 0; k < 12; ++k) q[k] = U[(size_t)k * n + e];
}

template <typename T>
__device__ __forceinline__ double step_size(const PM<T>& p) {
  return p.dt_dev ? *p.dt_dev : p.dt_host;
}

// Primitive (rho, v_x, v_y, p) of conserved means.
template <typename T>
__device__ __forceinline__ void prim4(const T* m, T gm1, T* w) {
  const T ir = rcp(m[0]);
  w[0] = m[0];
  w[1] = m[1] * ir;
  w[2] = m[2] * ir;
  w[3] = gm1 * (m[3] - T(0.5) * (m[1] * w[1] + m[2] * w[2]));
}

// Half-step primitive prediction of a limited cell (Sec. 2.4): values at
// the centroid advanced by h in w[0..3], primitive gradients in gx, gy.
template <typename T>
struct Pred {
  T w[4], gx[4], gy[4];
};

template <typename T>
__device__ __forceinline__ Pred<T> predict(const T* q, T gamma, T h) {
  const T gm1 = gamma - T(1);
  const T rho = q[0], ir = rcp(rho);
  const T vx = q[3] * ir, vy = q[6] * ir;
  const T v2 = vx * vx + vy * vy;
  const T pr = gm1 * (q[9] - T(0.5) * rho * v2);
  Pred<T> o;
  o.gx[0] = q[1];
  o.gy[0] = q[2];
  o.gx[1] = (q[4] - vx * q[1]) * ir;
  o.gy[1] = (q[5] - vx * q[2]) * ir;
  o.gx[2] = (q[7] - vy * q[1]) * ir;
  o.gy[2] = (q[8] - vy * q[2]) * ir;
  o.gx[3] = gm1 * (q[10] - T(0.5) * v2 * q[1] - rho * (vx * o.gx[1] + vy * o.gx[2]));
  o.gy[3] = gm1 * (q[11] - T(0.5) * v2 * q[2] - rho * (vx * o.gy[1] + vy * o.gy[2]));
  const T div = o.gx[1] + o.gy[2];
  const T rho_t = -(vx * o.gx[0] + vy * o.gy[0] + rho * div);
  const T vx_t = -(vx * o.gx[1] + vy * o.gy[1] + o.gx[3] * ir);
  const T vy_t = -(vx * o.gx[2] + vy * o.gy[2] + o.gy[3] * ir);
  const T p_t = -(gamma * pr * div + vx * o.gx[3] + vy * o.gy[3]);
  o.w[0] = rho + h * rho_t;
  o.w[1] = vx + h * vx_t;
  o.w[2] = vy + h * vy_t;
  o.w[3] = pr + h * p_t;
  return o;
}

// ------------------------------------------------------------- limiter --
// Per cell of the mesh of t^n.  LIM 0 copies, 1 the Arepo limiter on the
// conserved coefficients, 2 the WENO-type limiter on (rho, v, p) with the
// least-squares stencil slope over the face neighbours.  Also moves the
// generators (when write_pos) and checks that every neighbour lists the
// cell back.
template <typename T, int LIM>
__global__ __launch_bounds__(256) void k_mv_lim(PM<T> p) {
  const int e = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (e >= p.n) return;
  const int n = p.n;
  T q[12];
  load12(p.in, n, e, q);
  const MSet& s = p.s0;
  const int* re = s.ring + e * kRing;
  const int d = min(s.deg[e], kRing);
  bool meshbad = s.deg[e] > kRing || s.deg[e] < 3;
  const int4* R4 = reinterpret_cast<const int4*>(s.ring);
  for (int k = 0; k < d; ++k) {
    // (entries beyond a ring's degree are -1)
    const int j = re[k];
    const int4 a = R4[4 * (size_t)j], b = R4[4 * (size_t)j + 1];
    bool back = a.x == e || a.y == e || a.z == e || a.w == e || b.x == e || b.y == e ||
                b.z == e || b.w == e;
    if (!back && s.deg[j] > 8) {
      const int4 c = R4[4 * (size_t)j + 2], f = R4[4 * (size_t)j + 3];
      back = c.x == e || c.y == e || c.z == e || c.w == e || f.x == e || f.y == e || f.z == e ||
             f.w == e;
    }
    meshbad |= !back;
  }
  if (meshbad) atomicOr(p.status, 2);
  const double dcx = s.geo[1 * n + e], dcy = s.geo[2 * n + e];
  // The faces are visited in passes that read the face midpoints k_mv_geom left
  // and the neighbours' means, instead of keeping per-face arrays, which would
  // live in per-lane scratch memory.
  auto faces = [&](auto&& f) {
    for (int k = 0; k < d; ++k) {
      const double2 m = p.mid[(size_t)k * n + e];
      f(k, re[k], (T)(m.x - dcx), (T)(m.y - dcy));
    }
  };
  if (LIM != 0) {
    const T gm1 = p.gamma - T(1);
    if (LIM == 1) {
      T hi[4], lo[4], alpha[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        hi[v] = lo[v] = q[3 * v];
        alpha[v] = T(1);
      }
      for (int k = 0; k < d; ++k) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T m = p.in[(size_t)(3 * v) * n + re[k]];
          hi[v] = fmax(hi[v], m);
          lo[v] = fmin(lo[v], m);
        }
      }
      faces([&](int, int, T rx, T ry) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T dd = q[3 * v + 1] * rx + q[3 * v + 2] * ry;
          const T num = dd > T(0) ? hi[v] - q[3 * v] : lo[v] - q[3 * v];
          const T psi = dd > T(0) ? div_small(num, dd) : (dd < T(0) ? div_small(-num, -dd) : T(1));
          alpha[v] = fmin(alpha[v], psi);
        }
      });
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        q[3 * v + 1] *= alpha[v];
        q[3 * v + 2] *= alpha[v];
      }
    } else {
      const T eps = sizeof(T) == 8 ? T(2.220446049250313e-16) : T(1.1920929e-7);
      T mi[4] = {q[0], q[3], q[6], q[9]};
      T wi[4];
      prim4(mi, gm1, wi);
      auto nbr_prim = [&](int j, T* w) {
        T mj[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) mj[v] = p.in[(size_t)(3 * v) * n + j];
        prim4(mj, gm1, w);
      };
      const T rho = wi[0], ir = rcp(rho), ux = wi[1], uy = wi[2];
      const T v2 = ux * ux + uy * uy;
      // DG primitive slopes (chain rule at the centroid)
      T gx[4], gy[4];
      gx[0] = q[1];
      gy[0] = q[2];
      gx[1] = (q[4] - ux * gx[0]) * ir;
      gy[1] = (q[5] - ux * gy[0]) * ir;
      gx[2] = (q[7] - uy * gx[0]) * ir;
      gy[2] = (q[8] - uy * gy[0]) * ir;
      gx[3] = gm1 * (q[10] - T(0.5) * v2 * gx[0] - rho * (ux * gx[1] + uy * gx[2]));
      gy[3] = gm1 * (q[11] - T(0.5) * v2 * gy[0] - rho * (ux * gy[1] + uy * gy[2]));
      // pass 1: least-squares normal equations of the stencil, bounds
      T a00 = T(0), a01 = T(0), a11 = T(0), b0[4], b1[4], hi[4], lo[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        b0[v] = b1[v] = T(0);
        hi[v] = lo[v] = wi[v];
      }
      const double2* P = reinterpret_cast<const double2*>(s.x + 2 * (size_t)n);
      const double2 pe = P[e];
      for (int k = 0; k < d; ++k) {
        const int j = re[k];
        const double2 pj = P[j];
        const T dnx = (T)(mimg(pj.x - pe.x, p.Lx) + s.geo[1 * n + j] - dcx);
        const T dny = (T)(mimg(pj.y - pe.y, p.Ly) + s.geo[2 * n + j] - dcy);
        a00 += dnx * dnx;
        a01 += dnx * dny;
        a11 += dny * dny;
        T wj[4];
        nbr_prim(j, wj);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T dw = wj[v] - wi[v];
          b0[v] += dnx * dw;
          b1[v] += dny * dw;
          hi[v] = fmax(hi[v], wj[v]);
          lo[v] = fmin(lo[v], wj[v]);
        }
      }
      const T idet = rcp(a00 * a11 - a01 * a01);
      T sx[4], sy[4], alpha[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sx[v] = (a11 * b0[v] - a01 * b1[v]) * idet;
        sy[v] = (a00 * b1[v] - a01 * b0[v]) * idet;
        alpha[v] = T(1);
      }
      // pass 2: the stencil slope limited as in the Arepo limiter
      faces([&](int, int, T rx, T ry) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T dd = sx[v] * rx + sy[v] * ry;
          // the clamp absorbs rounding of hi - w (w a product): D >= 0
          const T num = dd > T(0) ? fmax(hi[v] - wi[v], T(0)) : fmin(lo[v] - wi[v], T(0));
          const T psi = dd > T(0) ? div_small(num, dd) : (dd < T(0) ? div_small(-num, -dd) : T(1));
          alpha[v] = fmin(alpha[v], psi);
        }
      });
      // pass 3: oscillation factors of the two candidates
      T os[4], od[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sx[v] *= alpha[v];
        sy[v] *= alpha[v];
        os[v] = od[v] = T(0);
      }
      faces([&](int, int j, T rx, T ry) {
        T wj[4];
        nbr_prim(j, wj);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T ds = sx[v] * rx + sy[v] * ry;
          const T dg = gx[v] * rx + gy[v] * ry;
          os[v] += fabs(ds) + fabs(wj[v] - (wi[v] + ds));
          od[v] += fabs(dg) + fabs(wj[v] - (wi[v] + dg));
        }
      });
      T ngx[4], ngy[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T ws = rcp(sqrt_pos(eps + os[v])), wd = rcp(sqrt_pos(eps + od[v]));
        const T iw = rcp(ws + wd);
        ngx[v] = (ws * sx[v] + wd * gx[v]) * iw;
        ngy[v] = (ws * sy[v] + wd * gy[v]) * iw;
      }
      q[1] = ngx[0];
      q[2] = ngy[0];
      q[4] = ux * ngx[0] + rho * ngx[1];
      q[5] = ux * ngy[0] + rho * ngy[1];
      q[7] = uy * ngx[0] + rho * ngx[2];
      q[8] = uy * ngy[0] + rho * ngy[2];
      const T igm1 = rcp(gm1);
      q[10] = ngx[3] * igm1 + T(0.5) * v2 * ngx[0] + rho * (ux * ngx[1] + uy * ngx[2]);
      q[11] = ngy[3] * igm1 + T(0.5) * v2 * ngy[0] + rho * (ux * ngy[1] + uy * ngy[2]);
    }
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) p.ua_out[(size_t)k * n + e] = q[k];
  if (p.write_pos) {
    const double dt = step_size(p);
    double wx = 0.0, wy = 0.0;
    if (p.motion) {
      wx = (double)q[3] / (double)q[0];
      wy = (double)q[6] / (double)q[0];
    }
    const double x = s.x[e], y = s.x[n + e];
    const double hx = advance(x, 0.5 * dt, wx, p.Lx), hy = advance(y, 0.5 * dt, wy, p.Ly);
    // what both cells of every face need of this one in the update: its half-step
    // prediction, its velocity and where its t^n centroid lies from its half-step
    // generator
    const Pred<T> w = predict(q, p.gamma, T(0.5 * dt));
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p.pred_out[(size_t)v * n + e] = w.w[v];
      p.pred_out[(size_t)(4 + v) * n + e] = w.gx[v];
      p.pred_out[(size_t)(8 + v) * n + e] = w.gy[v];
    }
    p.pred_out[(size_t)12 * n + e] = p.motion ? q[3] / q[0] : T(0);
    p.pred_out[(size_t)13 * n + e] = p.motion ? q[6] / q[0] : T(0);
    p.shift_out[e] = make_double2(mimg(hx - x, p.Lx) - dcx, mimg(hy - y, p.Ly) - dcy);
    const double nx1 = advance(x, dt, wx, p.Lx), ny1 = advance(y, dt, wy, p.Ly);
    p.xh[e] = hx;
    p.xh[n + e] = hy;
    reinterpret_cast<double2*>(p.xh + 2 * (size_t)n)[e] = make_double2(hx, hy);
    p.x1[e] = nx1;
    p.x1[n + e] = ny1;
    reinterpret_cast<double2*>(p.x1 + 2 * (size_t)n)[e] = make_double2(nx1, ny1);
  }
}

// ----------------------------------------------------------------- mesh --
// The mesh of the positions dst.x from the mesh `src`, in three launches.
// k_mv_check keeps the ring of every cell whose neighbours did not change and
// lists the others; k_mv_walk finds the rings of the listed cells from the 2-ring
// of `src`; k_mv_geom computes the cell geometry from the ring (canonical
// vertices, polygon moments); with FINISH also the new state from the totals and
// moments in p.out (the mesh of t^n in p.s0, the limited state p.ua for w_e) and
// the cell's CFL bound in the per-wave minima when p.dtpart is set.  The
// candidates of a cell are its previous neighbours and the entries of their rings.

__device__ __forceinline__ void nearest_image(const PM_box& b, double& dx, double& dy) {
  dx -= b.Lx * rint(dx * b.iLx);
  dy -= b.Ly * rint(dy * b.iLy);
}

// One thread per cell.  The previous ring is still the cell's ring exactly when
// the vertices it gives at the new positions (circumcentres of the cell and two
// neighbours that follow each other) lie in the half-plane of every candidate:
// then each is a vertex of the cell, and the walk from the nearest neighbour
// would visit the same faces in the same order.  The test keeps a distance from
// rounding (sine of the angle between neighbours above 1e-2, vertices inside by
// 1e-9 of the candidate's distance).  Nearer candidates (four cells that meet in a
// point, as on a lattice) are looked at one by one (`settled`): one that is inside
// beyond rounding, or whose face k_mv_geom would drop, leaves the ring as it is (the
// walk of such a cell gives the same ring once that face is dropped; a step on a
// square lattice of 512^2 cells takes 0.29 ms, 2.76 ms with every such cell on the
// list).  Cells that miss the test, that have more than kFast neighbours, or whose ring
// changed, go to the list.
// The vertices and neighbours stay in registers; a candidate costs kFast comparisons
// of its index and kFast products, no list and no dependent scan.  The latency of its
// three gathers (ring, neighbours' rings, positions) bounds it.  Measured (262144
// cells, FP64): 0.064 ms, and 0.015 ms for the walk of the listed cells; walking
// every cell, one thread each over a list of its candidates in LDS, took 0.177
// ms, its dependent scans (one of all candidates per face) bound by latency.
template <typename T>
__global__ __launch_bounds__(256) void k_mv_check(PM<T> p, MSet src, MOut dst) {
  const int e = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  const bool live = e < p.n;
  bool ok = false;
  if (live) {
    const int n = p.n;
    const double2* XY = reinterpret_cast<const double2*>(dst.x + 2 * (size_t)n);
    const PM_box box{p.Lx, p.Ly, 1.0 / p.Lx, 1.0 / p.Ly};
    const double2 pe = XY[e];
    const int d = src.deg[e];
    ok = d >= 3 && d <= kFast;
    const int4* R4 = reinterpret_cast<const int4*>(src.ring);
    int r[kFast];
    {
      const int4 lo = R4[4 * (size_t)e], hi = R4[4 * (size_t)e + 1];
      r[0] = lo.x, r[1] = lo.y, r[2] = lo.z, r[3] = lo.w;
      r[4] = hi.x, r[5] = hi.y, r[6] = hi.z, r[7] = hi.w;
    }
    double dx[kFast], dy[kFast], n2[kFast], vx[kFast], vy[kFast];
#pragma unroll
    for (int k = 0; k < kFast; ++k) {
      r[k] = ok && k < d ? r[k] : e;
      const double2 q = XY[r[k]];
      dx[k] = q.x - pe.x;
      dy[k] = q.y - pe.y;
      nearest_image(box, dx[k], dy[k]);
      n2[k] = dx[k] * dx[k] + dy[k] * dy[k];
    }
    constexpr double kIn = 1.0 - 1e-9;
#pragma unroll
    for (int k = 0; k < kFast; ++k) {
      const bool wrap = k + 1 == kFast || k + 1 >= d;
      const double x1 = wrap ? dx[0] : dx[(k + 1) % kFast], y1 = wrap ? dy[0] : dy[(k + 1) % kFast];
      const double m1 = wrap ? n2[0] : n2[(k + 1) % kFast];
      const double den = dx[k] * y1 - dy[k] * x1;
      if (k < d) ok &= den > 0.0 && den * den > 1e-4 * n2[k] * m1;
      // 2 x the vertex: d_k + t perp(d_k), t = (|d_k1|^2 - d_k . d_k1) / den
      const double t = (m1 - (dx[k] * x1 + dy[k] * y1)) * rcp(den);
      vx[k] = k < d ? dx[k] - t * dy[k] : 0.0;
      vy[k] = k < d ? dy[k] + t * dx[k] : 0.0;
    }
    // Candidates that come within 1e-9 of a vertex: c, the neighbour `own` of the cell
    // or (own < 0) one further out.  Where the vertex is well conditioned (sines above
    // 0.1, distances within a factor of 4) 1e-12 of the distance is far from rounding.
    // A candidate further out may also touch or cut one vertex, between its two
    // neighbours, if the cut, its depth times (cot + cot) of its angles to them, is
    // shorter than half of the length (1e-10 of its distance) below which k_mv_geom
    // drops a face.  (Rare; the positions are read again, since the offsets would cost
    // registers in the loop over the candidates.)
    auto settled = [&](int c, int own) {
      auto offset = [&](int i, double& x, double& y) {
        const double2 q = XY[i];
        x = q.x - pe.x;
        y = q.y - pe.y;
        nearest_image(box, x, y);
      };
      double cx, cy;
      offset(c, cx, cy);
      const double m = cx * cx + cy * cy;
      int cuts = 0;
      bool good = true;
#pragma unroll
      for (int k = 0; k < kFast; ++k) {
        const int next = k + 1 < d ? k + 1 : 0;
        const double cut = vx[k] * cx + vy[k] * cy - m;
        if (k < d && own != k && own != next && !(cut < (kIn - 1.0) * m)) {
          double ax, ay, bx, by;
          offset(r[k], ax, ay);
          offset(k + 1 < kFast && k + 1 < d ? r[(k + 1) % kFast] : r[0], bx, by);
          const double sa = ax * cy - ay * cx, sb = cx * by - cy * bx, sab = ax * by - ay * bx;
          const double ma = ax * ax + ay * ay, mb = bx * bx + by * by;
          good &= sa * sa > 0.01 * ma * m && sb * sb > 0.01 * mb * m && sab * sab > 0.01 * ma * mb &&
                  fmax(ma, mb) < 16.0 * m;
          if (!(cut < -1e-12 * m)) {
            good &= sa > 0.0 && sb > 0.0 &&
                    (fmax(cut, 0.0) + 1e-12 * m) *
                            ((ax * cx + ay * cy) * sb + (bx * cx + by * cy) * sa) <
                        1e-10 * m * (sa * sb);
            ++cuts;
          }
        }
      }
      return good && cuts <= (own < 0 ? 1 : 0);
    };
    // the cell's other neighbours, then every candidate further out
    unsigned open = 0;
#pragma unroll
    for (int c = 0; c < kFast; ++c)
#pragma unroll
      for (int k = 0; k < kFast; ++k) {
        const bool own = c == k || c == (k + 1 < d ? k + 1 : 0);
        if (c < d && k < d && !own && !(vx[k] * dx[c] + vy[k] * dy[c] < kIn * n2[c])) open |= 1u << c;
      }
    for (; open && ok; open &= open - 1) {
      const int c = __ffs(open) - 1;
      ok = settled(src.ring[(size_t)e * kRing + c], c);
    }
    if (ok) {
      for (int a = 0; a < d && ok; ++a) {
        const int j = src.ring[(size_t)e * kRing + a];
        const int dj = min(src.deg[j], kRing);
        for (int b = 0; b < dj; b += 8) {
          const int4 lo = R4[4 * (size_t)j + (b >> 2)], hi = R4[4 * (size_t)j + (b >> 2) + 1];
          const int c[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          double2 q[8];
          bool out[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            out[u] = b + u < dj && c[u] != e;
#pragma unroll
            for (int k = 0; k < kFast; ++k) out[u] &= c[u] != r[k];
            q[u] = XY[out[u] ? c[u] : e];
          }
          open = 0;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            double cx = q[u].x - pe.x, cy = q[u].y - pe.y;
            nearest_image(box, cx, cy);
            const double m = cx * cx + cy * cy;
            double most = vx[0] * cx + vy[0] * cy;
#pragma unroll
            for (int k = 1; k < kFast; ++k) most = fmax(most, vx[k] * cx + vy[k] * cy);
            ok &= !out[u] || most < (2.0 - kIn) * m;
            open |= out[u] && !(most < kIn * m) ? 1u << u : 0u;
          }
          for (; open && ok; open &= open - 1)
            ok = settled(src.ring[(size_t)j * kRing + b + __ffs(open) - 1], -1);
        }
      }
    }
    if (ok) {
      // the ring from the nearest neighbour on, as the walk gives it
      int s = 0;
#pragma unroll
      for (int k = 1; k < kFast; ++k) {
        double best = n2[0];
        int rb = r[0];
#pragma unroll
        for (int q = 1; q < k; ++q) {
          best = q == s ? n2[q] : best;
          rb = q == s ? r[q] : rb;
        }
        if (k < d && (n2[k] < best || (n2[k] == best && r[k] < rb))) s = k;
      }
      int* out = dst.ring + (size_t)e * kRing;
#pragma unroll
      for (int k = 0; k < kFast; ++k)
        if (k < d) out[k >= s ? k - s : k - s + d] = r[k];
      for (int k = d; k < kRing; ++k) out[k] = -1;
      dst.deg[e] = d;
    }
  }
  // list the others, one counter update per wave
  const unsigned long long todo = __ballot(live && !ok);
  if (todo) {
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == __ffsll((long long)todo) - 1) base = atomicAdd(p.count, __popcll(todo));
    base = __shfl(base, __ffsll((long long)todo) - 1);
    if (live && !ok) p.list[base + __popcll(todo & ((1ull << lane) - 1))] = e;
  }
}

// The walk of a listed cell.  The cell is walked counter-clockwise, one face at a
// time.  The nearest candidate is a neighbour (the midpoint of the two generators lies
// on their common face).  The face of neighbour j lies on the bisector
// x(t) = d_j/2 + t perp(d_j), perp(d) = (-d_y, d_x); candidate k bounds it from the
// counter-clockwise side at t_k = (|d_k|^2 - d_j . d_k) / (2 perp(d_j) . d_k) when
// perp(d_j) . d_k > 0, and the next neighbour is the candidate with the smallest t_k
// (compared by cross-multiplication; ties to the smaller index).  The walk ends back at
// the first neighbour; nothing but the ring is stored.  The next face depends on the
// current one alone, so a walk that meets a neighbour again before the first one has
// run into a circle and the cell is not bounded: no ring holds a neighbour twice (the
// rings given at creation, those k_mv_check keeps and those that lose short faces
// are distinct too).
struct WalkMin {  // the smallest t_k so far, as num / den
  double num = 1.0, den = 0.0, x = 0.0, y = 0.0;
  int k = -1;
  __device__ __forceinline__ void take(int id, double nu, double de, double dx, double dy) {
    const double l = nu * den, r = num * de;
    if (k < 0 || l < r || (l == r && id < k)) {
      num = nu;
      den = de;
      k = id;
      x = dx;
      y = dy;
    }
  }
};

// By a wave, the candidates spread over its lanes (an entry that several neighbours
// list appears several times: equal values, harmless).
template <typename T>
__device__ __forceinline__ void walk_by_wave(const PM<T>& p, const MSet& src, const MOut& dst,
                                             const PM_box& box, int e) {
  const int lane = threadIdx.x & 63;
  const double2* XY = reinterpret_cast<const double2*>(dst.x + 2 * (size_t)p.n);
  constexpr int kSlots = (kRing * (kRing + 1) + 63) / 64;
  const double2 pe = XY[e];
  const int d0 = min(src.deg[e], kRing);
  int id[kSlots];
  double kx[kSlots], ky[kSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const int t = lane + 64 * q, a = t / (kRing + 1), b = t - a * (kRing + 1) - 1;
    id[q] = -1;
    kx[q] = ky[q] = 0.0;
    if (a < d0) {
      const int j = src.ring[(size_t)e * kRing + a];
      const int k = b < 0 ? j : (b < min(src.deg[j], kRing) ? src.ring[(size_t)j * kRing + b] : e);
      if (k != e) {
        const double2 pk = XY[k];
        id[q] = k;
        kx[q] = pk.x - pe.x;
        ky[q] = pk.y - pe.y;
        nearest_image(box, kx[q], ky[q]);
      }
    }
  }
  // the nearest candidate
  double best = 1e300, bx = 0.0, by = 0.0;
  int j0 = -1;
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const double dd = kx[q] * kx[q] + ky[q] * ky[q];
    if (id[q] >= 0 && (j0 < 0 || dd < best || (dd == best && id[q] < j0))) {
      best = dd;
      j0 = id[q];
      bx = kx[q];
      by = ky[q];
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o), ox = __shfl_xor(bx, o), oy = __shfl_xor(by, o);
    const int oj = __shfl_xor(j0, o);
    if (oj >= 0 && (j0 < 0 || ob < best || (ob == best && oj < j0))) {
      best = ob;
      j0 = oj;
      bx = ox;
      by = oy;
    }
  }
  // (one lane's winner for all: near ties may round differently across lanes)
  j0 = __builtin_amdgcn_readfirstlane(j0);
  bool bad = j0 < 0;
  int mine = -1;  // ring entry `lane`
  int d = 0, cur = j0;
  double cx = __shfl(bx, 0), cy = __shfl(by, 0);
  while (!bad) {
    if (d > kRing || __any(mine == cur)) {
      bad = true;
      break;
    }
    mine = lane == d ? cur : mine;
    ++d;
    WalkMin w;
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      const double den = cx * ky[q] - cy * kx[q];  // perp(d_cur) . d_k
      if (id[q] >= 0 && id[q] != cur && den > 0.0)
        w.take(id[q], kx[q] * kx[q] + ky[q] * ky[q] - (cx * kx[q] + cy * ky[q]), den, kx[q], ky[q]);
    }
    for (int o = 32; o > 0; o >>= 1) {
      const int ok = __shfl_xor(w.k, o);
      const double on = __shfl_xor(w.num, o), od = __shfl_xor(w.den, o);
      const double ox = __shfl_xor(w.x, o), oy = __shfl_xor(w.y, o);
      if (ok >= 0) w.take(ok, on, od, ox, oy);
    }
    const int nxt = __builtin_amdgcn_readfirstlane(w.k);
    if (nxt < 0) {
      bad = true;
      break;
    }
    if (nxt == j0) break;
    cur = nxt;
    cx = __shfl(w.x, 0);
    cy = __shfl(w.y, 0);
  }
  bad |= d > kRing;
  if (lane < kRing) dst.ring[(size_t)e * kRing + lane] = !bad && lane < d ? mine : -1;
  if (lane == 0) {
    dst.deg[e] = bad ? 0 : d;
    if (bad) atomicOr(p.status, 2);
  }
}

// By a thread, over the list of its distinct candidates in a column of LDS (no
// barrier), kChunk of their positions loaded together.  False, and nothing written,
// where they are more than kCand.
template <typename T>
__device__ __forceinline__ bool walk_by_thread(const PM<T>& p, const MSet& src, const MOut& dst,
                                               const PM_box& box, int e, int* cl) {
  constexpr int kChunk = 4;
  const double2* XY = reinterpret_cast<const double2*>(dst.x + 2 * (size_t)p.n);
  const double2 pe = XY[e];
  const int d0 = min(src.deg[e], kRing);
  int nc = 0;
  for (int a = 0; a < d0; ++a) {
    const int j = src.ring[(size_t)e * kRing + a];
    const int dj = min(src.deg[j], kRing);
    for (int b = -1; b < dj; ++b) {
      const int k = b < 0 ? j : src.ring[(size_t)j * kRing + b];
      bool seen = k == e;
      for (int c = 0; c < nc && !seen; ++c) seen = cl[c * 256] == k;
      if (seen) continue;
      if (nc == kCand) return false;
      cl[nc++ * 256] = k;
    }
  }
  auto visit = [&](auto&& f) {
    for (int c0 = 0; c0 < nc; c0 += kChunk) {
      int k[kChunk];
      double2 q[kChunk];
#pragma unroll
      for (int u = 0; u < kChunk; ++u) k[u] = c0 + u < nc ? cl[(c0 + u) * 256] : e;
#pragma unroll
      for (int u = 0; u < kChunk; ++u) q[u] = XY[k[u]];
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        if (k[u] == e) continue;
        double dx = q[u].x - pe.x, dy = q[u].y - pe.y;
        nearest_image(box, dx, dy);
        f(k[u], dx, dy);
      }
    }
  };
  int j0 = -1, cur, d = 0;
  double best = 1e300, cx = 0.0, cy = 0.0;
  visit([&](int k, double dx, double dy) {
    const double dd = dx * dx + dy * dy;
    if (j0 < 0 || dd < best || (dd == best && k < j0)) {
      best = dd;
      j0 = k;
      cx = dx;
      cy = dy;
    }
  });
  int* ring = dst.ring + (size_t)e * kRing;
  bool bad = j0 < 0;
  cur = j0;
  while (!bad) {
    if (d == kRing) {  // (a circle that misses the first neighbour ends here too)
      bad = true;
      break;
    }
    ring[d++] = cur;
    WalkMin w;
    visit([&](int k, double dx, double dy) {
      const double den = cx * dy - cy * dx;  // perp(d_cur) . d_k
      if (k != cur && den > 0.0) w.take(k, dx * dx + dy * dy - (cx * dx + cy * dy), den, dx, dy);
    });
    bad = w.k < 0;
    if (w.k == j0) break;
    cur = w.k;
    cx = w.x;
    cy = w.y;
  }
  for (int k = bad ? 0 : d; k < kRing; ++k) ring[k] = -1;
  dst.deg[e] = bad ? 0 : d;
  if (bad) atomicOr(p.status, 2);
  return true;
}

// A short list is walked by a wave a cell, for the shortest chain; a list of more than a
// tenth of the cells by a thread a cell, for the least work.  Measured (262144 cells,
// FP64; check, walk and geometry): 5% and 8% of the cells on the list 0.21 ms by waves
// and 0.40 and 0.23 by threads, 12% 0.34 against 0.29, all 1.3 against 0.4.
template <typename T>
__global__ __launch_bounds__(256) void k_mv_walk(PM<T> p, MSet src, MOut dst) {
  __shared__ int cl[kCand * 256];
  const int count = *p.count, tid = threadIdx.x;
  const PM_box box{p.Lx, p.Ly, 1.0 / p.Lx, 1.0 / p.Ly};
  if (count > p.n / 10) {
    for (int i0 = blockIdx.x * 256 + (tid & ~63); i0 < count; i0 += gridDim.x * 256) {
      const int i = i0 + (tid & 63);
      const int e = i < count ? p.list[i] : -1;
      const bool more = e >= 0 && !walk_by_thread(p, src, dst, box, e, cl + tid);
      for (unsigned long long m = __ballot(more); m; m &= m - 1)
        walk_by_wave(p, src, dst, box, __builtin_amdgcn_readlane(e, __ffsll((long long)m) - 1));
    }
  } else {
    for (int i = blockIdx.x * 4 + (tid >> 6); i < count; i += gridDim.x * 4)
      walk_by_wave(p, src, dst, box, __builtin_amdgcn_readfirstlane(p.list[i]));
  }
}

template <typename T, bool FINISH>
__global__ __launch_bounds__(256) void k_mv_geom(PM<T> p, MOut dst) {
  const int e = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  double dtb = 1e300;
  if (e == 0) *p.count = 0;  // the walk that read it is done; the next check counts from zero
  if (e < p.n) {
    const int n = p.n;
    const double2* P = reinterpret_cast<const double2*>(dst.x + 2 * (size_t)n);
    const double2 pe = P[e];
    const double xe = pe.x, ye = pe.y;
    int* ring = dst.ring + (size_t)e * kRing;
    int d = dst.deg[e];
    bool look = false;
    bool bad = d < 3 || d > kRing;
    Moments mom;
    // f(k, a, b) for every edge of the polygon: face k runs from vertex k, the one
    // of (e, ring[k-1], ring[k]), to vertex k + 1
    auto edges = [&](auto&& f) {
      const int last = ring[d - 1], first = ring[0];
      double ax, ay;
      vertex_from(vertex(P, p.Lx, p.Ly, e, last, first), p.Lx, p.Ly, e, pe, ax, ay);
      const double a0x = ax, a0y = ay;
      int j = first;
      for (int k = 0; k < d; ++k) {
        double bx = a0x, by = a0y;
        int jn = first;
        if (k + 1 < d) {
          jn = ring[k + 1];
          vertex_from(vertex(P, p.Lx, p.Ly, e, j, jn), p.Lx, p.Ly, e, pe, bx, by);
        }
        f(k, j, ax, ay, bx, by);
        ax = bx;
        ay = by;
        j = jn;
      }
    };
    double perim = 0.0;
    auto measure = [&]() {
      mom = Moments();
      perim = 0.0;
      edges([&](int k, int j, double ax, double ay, double bx, double by) {
        const double ex = bx - ax, ey = by - ay, l2 = ex * ex + ey * ey;
        const double2 pj = P[j];
        const double gx = mimg(pj.x - xe, p.Lx), gy = mimg(pj.y - ye, p.Ly);
        look |= !(l2 > 1e-16 * (gx * gx + gy * gy));
        mom.add(ax, ay, bx, by);
        if (FINISH) perim += sqrt(l2);
        if (p.mid_out) p.mid_out[(size_t)k * n + e] = make_double2(0.5 * (ax + bx), 0.5 * (ay + by));
      });
    };
    if (!bad) measure();
    if (!bad && look) {
      // drop the faces shorter than 1e-10 of their generators' distance (their
      // existence is decided by rounding); both cells of such a face decide it
      // from the same canonical operands.  Only a cell with a face near that
      // length comes here.
      const int first = ring[0];
      int prev = ring[d - 1], dk = 0;
      for (int k = 0; k < d; ++k) {
        const int j = ring[k], next = k + 1 == d ? first : ring[k + 1];
        const int L = min(e, j), Rr = max(e, j);
        FaceG g;
        face_geometry(p.Lx, p.Ly, L, P[L], P[Rr], vertex(P, p.Lx, p.Ly, L, Rr, prev),
                      vertex(P, p.Lx, p.Ly, L, Rr, next), g);
        if (g.A >= 1e-10 * sqrt(g.dx * g.dx + g.dy * g.dy)) ring[dk++] = j;
        prev = j;
      }
      bad |= dk < 3;
      for (int k = dk; k < kRing; ++k) ring[k] = -1;
      dst.deg[e] = bad ? 0 : dk;
      if (bad) atomicOr(p.status, 2);
      const bool fewer = dk != d;
      d = dk;
      if (!bad && fewer) measure();
    }
    double geo[kGeo] = {0, 0, 0, 0, 0, 0};
    if (!bad) {
      mom.geometry(geo);
      bad |= !(geo[0] > 0.0) || !(geo[3] * geo[5] - geo[4] * geo[4] > 0.0);
      if (bad) atomicOr(p.status, 2);
    }
    if (bad) {
      d = 0;
      geo[0] = 1.0;
      geo[1] = geo[2] = geo[4] = 0.0;
      geo[3] = geo[5] = 1.0;
    }
    for (int k = 0; k < kGeo; ++k) dst.geo[(size_t)k * n + e] = geo[k];
    if (FINISH) {
      const double dt = step_size(p);
      T Q[12];
      load12(p.out, n, e, Q);
      const T r0 = p.ua[e], wxT = p.ua[(size_t)3 * n + e], wyT = p.ua[(size_t)6 * n + e];
      double wx = 0.0, wy = 0.0;
      if (p.motion) {
        wx = (double)wxT / (double)r0;
        wy = (double)wyT / (double)r0;
      }
      const MSet& s0 = p.s0;
      const double delx = mimg(xe - s0.x[e], p.Lx) + geo[1] - s0.geo[1 * n + e] - dt * wx;
      const double dely = mimg(ye - s0.x[n + e], p.Ly) + geo[2] - s0.geo[2 * n + e] - dt * wy;
      const double V = geo[0], Mxx = geo[3], Mxy = geo[4], Myy = geo[5];
      const double idet = 1.0 / (Mxx * Myy - Mxy * Mxy);
      T u[12];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double q0 = (double)Q[3 * v];
        const double qx = (double)Q[3 * v + 1] - delx * q0;
        const double qy = (double)Q[3 * v + 2] - dely * q0;
        u[3 * v] = (T)(q0 / V);
        u[3 * v + 1] = (T)((Myy * qx - Mxy * qy) * idet);
        u[3 * v + 2] = (T)((Mxx * qy - Mxy * qx) * idet);
      }
#pragma unroll
      for (int k = 0; k < 12; ++k) p.out[(size_t)k * n + e] = u[k];
      if (p.dtpart && !bad) {
        // CFL bound 2 V / sum_f A_f (|(v - w) . n_f| + c): w = v when the
        // generators move with the flow, w = 0 when they are held still
        const double rho = (double)u[0], ir = 1.0 / rho;
        const double ux = (double)u[3] * ir, uy = (double)u[6] * ir;
        const double pr =
            ((double)p.gamma - 1.0) * ((double)u[9] - 0.5 * rho * (ux * ux + uy * uy));
        const double cs = sqrt((double)p.gamma * pr * ir);
        double s = cs * perim;
        if (!p.motion)  // A |v . n|, n = (e_y, -e_x) / A
          edges([&](int, int, double ax, double ay, double bx, double by) {
            s += fabs(ux * (by - ay) - uy * (bx - ax));
          });
        dtb = 2.0 * V / s;
      }
    }
  }
  if (FINISH && p.dtpart) {
    dtb = wave_min(dtb);
    if ((threadIdx.x & 63) == 0) p.dtpart[e >> 6] = dtb;
  }
}

// ------------------------------------------------------------- update --
// Conserved state, boosted into the frame moving with (wx, wy), of the
// predicted primitive polynomial at offset (rx, ry) from the centroid.
template <typename T>
__device__ __forceinline__ void boosted_state(const Pred<T>& c, T rx, T ry, T wx, T wy, T igm1,
                                              T* u) {
  const T rho = c.w[0] + c.gx[0] * rx + c.gy[0] * ry;
  const T vx = c.w[1] + c.gx[1] * rx + c.gy[1] * ry - wx;
  const T vy = c.w[2] + c.gx[2] * rx + c.gy[2] * ry - wy;
  const T pr = c.w[3] + c.gx[3] * rx + c.gy[3] * ry;
  u[0] = rho;
  u[1] = rho * vx;
  u[2] = rho * vy;
  u[3] = pr * igm1 + T(0.5) * rho * (vx * vx + vy * vy);
}

// Lab-frame flux F - U w^T from the flux Fb of the same state in the frame
// moving with w.
template <typename T>
__device__ __forceinline__ void unboost(T* F, T wx, T wy) {
  const T f0 = F[0], f1 = F[1], f2 = F[2];
  F[1] = f1 + f0 * wx;
  F[2] = f2 + f0 * wy;
  F[3] = F[3] + wx * f1 + wy * f2 + T(0.5) * (wx * wx + wy * wy) * f0;
}

// HLL flux along x (Davis speeds).
template <typename T>
__device__ __forceinline__ void hll_x(const T* uL, const T* uR, T gamma, T* F, bool& bad) {
  const T gm1 = gamma - T(1);
  const T irL = rcp(uL[0]), irR = rcp(uR[0]);
  const T vL = uL[1] * irL, vR = uR[1] * irR;
  const T pL = gm1 * (uL[3] - T(0.5) * (uL[1] * vL + uL[2] * uL[2] * irL));
  const T pR = gm1 * (uR[3] - T(0.5) * (uR[1] * vR + uR[2] * uR[2] * irR));
  bad |= !(uL[0] > T(0)) || !(uR[0] > T(0)) || !(pL > T(0)) || !(pR > T(0));
  const T cL = sqrt_pos(gamma * pL * irL), cR = sqrt_pos(gamma * pR * irR);
  const T SL = fmin(vL - cL, vR - cR), SR = fmax(vL + cL, vR + cR);
  T FL[4] = {uL[1], uL[1] * vL + pL, uL[2] * vL, (uL[3] + pL) * vL};
  T FR[4] = {uR[1], uR[1] * vR + pR, uR[2] * vR, (uR[3] + pR) * vR};
  const T inv = rcp(SR - SL);
  T a = SR * inv, b = -SL * inv, c = SL * SR * inv;
  const bool left = SL >= T(0), right = SR <= T(0);
  a = left ? T(1) : (right ? T(0) : a);
  b = left ? T(0) : (right ? T(1) : b);
  c = (left || right) ? T(0) : c;
#pragma unroll
  for (int k = 0; k < 4; ++k) F[k] = fma(a, FL[k], fma(b, FR[k], c * (uR[k] - uL[k])));
}

// Riemann flux along the unit normal (nx, ny): rotate into (normal,
// tangential) components, solve along x, rotate back.
template <typename T, int RS>
__device__ __forceinline__ void riemann_n(const T* uL, const T* uR, T nx, T ny, T gamma, T* F,
                                          bool& bad) {
  T a[4] = {uL[0], uL[1] * nx + uL[2] * ny, uL[2] * nx - uL[1] * ny, uL[3]};
  T b[4] = {uR[0], uR[1] * nx + uR[2] * ny, uR[2] * nx - uR[1] * ny, uR[3]};
  T G[4];
  if (RS == 1)
    exact_flux<T, 0>(a, b, gamma, G, bad);
  else
    hll_x(a, b, gamma, G, bad);
  F[0] = G[0];
  F[1] = G[1] * nx - G[2] * ny;
  F[2] = G[1] * ny + G[2] * nx;
  F[3] = G[3];
}

template <typename T>
__device__ __forceinline__ void load_pred(const PM<T>& p, int e, Pred<T>& w, T& vx, T& vy) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    w.w[v] = p.pred[(size_t)v * p.n + e];
    w.gx[v] = p.pred[(size_t)(4 + v) * p.n + e];
    w.gy[v] = p.pred[(size_t)(8 + v) * p.n + e];
  }
  vx = p.pred[(size_t)12 * p.n + e];
  vy = p.pred[(size_t)13 * p.n + e];
}

// A workgroup updates kUpd consecutive cells (a compact region).  A face between two
// of them is solved once, by the lower cell of the pair; a face to a cell outside
// is solved by the cell itself.  The faces of the workgroup are listed in LDS, so
// that a pass gives every thread a face whatever the cells' numbers of neighbours
// are (a thread per cell that walks its ring waits for the longest ring of its wave,
// and solves every face twice); after each pass the cells gather from the pass's
// table.  A face that only one of its cells has (degenerate vertices), or that is
// one of several between the same pair (small periodic meshes), is solved by the
// cells that have it.  Two waves per SIMD, which is what the exact solver's 253
// registers in FP64 allow: with one the gathers are not hidden behind the divergent
// Newton loops.  Measured (262144 cells, FP64, exact solver): 0.149 ms, 11.7
// thousand vector instructions a wave (80 us of issue; the rest is the latency of
// each pass's gathers and its slowest Newton solve), against 0.236 ms and 21.7
// thousand with a thread per cell that walks its ring.
constexpr int kUpd = 256;

template <typename T, int RS>
__global__ __launch_bounds__(kUpd) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_mv_upd(PM<T> p) {
  __shared__ int nbr[kRing][kUpd];              // the cells' rings
  __shared__ unsigned short face[kRing][kUpd];  // of each: cell << 5 | ring index << 1 | side
  __shared__ unsigned short slot[kRing * kUpd]; // faces to solve: cell << 4 | ring index
  __shared__ unsigned own[kUpd];                // a cell's first slot << 16 | the faces it solves
  __shared__ unsigned char deg[kUpd];
  __shared__ int wsum[kUpd / 64];
  __shared__ T fl[8][kUpd];        // A/2 (F0 + F1), A/2 (F1 - F0)
  __shared__ double off[6][kUpd];  // face midpoint from each side's centroid, Gauss offset
  const int c0 = xcd_remap(blockIdx.x, gridDim.x) * kUpd;
  const int tid = threadIdx.x, e = c0 + tid;
  const int n = p.n;
  const bool live = e < n;
  const double dt = step_size(p);
  const T half = T(0.5 * dt);
  const T gamma = p.gamma, igm1 = rcp(gamma - T(1));
  const MSet& s0 = p.s0;
  const MSet& sh = p.sh;
  // interleaved (x, y) positions of the half step
  const double2* PH = reinterpret_cast<const double2*>(sh.x + 2 * (size_t)n);
  bool bad = false;
  const int d = live ? min(sh.deg[e], kRing) : 0;
  T wex = T(0), wey = T(0);
  if (live) {
    wex = p.pred[(size_t)12 * n + e];
    wey = p.pred[(size_t)13 * n + e];
  }
  deg[tid] = (unsigned char)d;
  for (int k = 0; k < d; ++k) nbr[k][tid] = sh.ring[(size_t)e * kRing + k];
  __syncthreads();
  unsigned mask = 0;
  for (int k = 0; k < d; ++k) {
    const int j = nbr[k][tid], side = j < e;
    unsigned code = (unsigned)tid << 5 | (unsigned)k << 1 | side;
    bool mine = true;
    if (side && j >= c0) {
      const int jl = j - c0, dj = deg[jl];
      int at = 0, times = 0, here = 0;
      for (int q = 0; q < dj; ++q)
        if (nbr[q][jl] == e) at = q, ++times;
      for (int q = 0; q < d; ++q) here += nbr[q][tid] == j;
      if (times == 1 && here == 1) {
        mine = false;
        code = (unsigned)jl << 5 | (unsigned)at << 1 | 1u;
      }
    }
    if (mine) mask |= 1u << k;
    face[k][tid] = (unsigned short)code;
  }
  int first = __popc(mask);
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(first, o);
    if ((tid & 63) >= o) first += up;
  }
  if ((tid & 63) == 63) wsum[tid >> 6] = first;
  __syncthreads();
  int nslot = 0;
  for (int w = 0; w < kUpd / 64; ++w) {
    if (w < (tid >> 6)) first += wsum[w];
    nslot += wsum[w];
  }
  first -= __popc(mask);
  own[tid] = (unsigned)first << 16 | mask;
  for (unsigned m = mask; m; m &= m - 1)
    slot[first++] = (unsigned short)(tid << 4 | (__ffs(m) - 1));
  __syncthreads();
  constexpr double kG = 0.28867513459481288225;  // 1/(2 sqrt 3)
  T S0[4] = {T(0), T(0), T(0), T(0)}, Sx[4] = {T(0), T(0), T(0), T(0)},
    Sy[4] = {T(0), T(0), T(0), T(0)};
  for (int sa = 0; sa < nslot; sa += kUpd) {
    if (sa + tid < nslot) {
      const int l = slot[sa + tid] >> 4, k = slot[sa + tid] & 15, dl = deg[l];
      const int a = c0 + l, j = nbr[k][l];
      const int L = min(a, j), R = max(a, j);
      const Vertex va = vertex(PH, p.Lx, p.Ly, a, nbr[k == 0 ? dl - 1 : k - 1][l], j);
      const Vertex vb = vertex(PH, p.Lx, p.Ly, a, j, nbr[k + 1 == dl ? 0 : k + 1][l]);
      FaceG g;
      face_geometry(p.Lx, p.Ly, L, PH[L], PH[R], va, vb, g);
      // both cells' half-step predictions; offsets from their t^n centroids
      // (R's generator lies at g.d from L's)
      Pred<T> pL, pR;
      T wLx, wLy, wRx, wRy;
      load_pred(p, L, pL, wLx, wLy);
      load_pred(p, R, pR, wRx, wRy);
      const double2 oL = p.shift[L];
      double2 oR = p.shift[R];
      oR.x -= g.dx;
      oR.y -= g.dy;
      const double dd = g.dx * g.dx + g.dy * g.dy;
      const T nx = (T)g.nx, ny = (T)g.ny, wq = (T)(0.5 * g.A);
      const double mx = 0.5 * (g.ax + g.bx), my = 0.5 * (g.ay + g.by);
      const double tx = kG * (g.bx - g.ax), ty = kG * (g.by - g.ay);
      T F[2][4];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const double gx = q == 0 ? mx - tx : mx + tx, gy = q == 0 ? my - ty : my + ty;
        // face velocity at the Gauss point: the mean of the generator velocities
        // plus the bisector's normal motion there
        const double sw = ((double)(wLx - wRx) * (gx - 0.5 * g.dx) +
                           (double)(wLy - wRy) * (gy - 0.5 * g.dy)) / dd;
        const T fwx = (T)(0.5 * (double)(wLx + wRx) + sw * g.dx);
        const T fwy = (T)(0.5 * (double)(wLy + wRy) + sw * g.dy);
        T uL[4], uR[4];
        boosted_state(pL, (T)(gx + oL.x), (T)(gy + oL.y), fwx, fwy, igm1, uL);
        boosted_state(pR, (T)(gx + oR.x), (T)(gy + oR.y), fwx, fwy, igm1, uR);
        riemann_n<T, RS>(uL, uR, nx, ny, gamma, F[q], bad);
        unboost(F[q], fwx, fwy);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        fl[v][tid] = wq * (F[0][v] + F[1][v]);
        fl[4 + v][tid] = wq * (F[1][v] - F[0][v]);
      }
      off[0][tid] = mx + oL.x;
      off[1][tid] = my + oL.y;
      off[2][tid] = mx + oR.x;
      off[3][tid] = my + oR.y;
      off[4][tid] = tx;
      off[5][tid] = ty;
    }
    __syncthreads();
    for (int k = 0; k < d; ++k) {
      const unsigned f = face[k][tid], o = own[f >> 5];
      const int i = (int)(o >> 16) + __popc(o & ((1u << ((f >> 1) & 15)) - 1u)) - sa;
      if (i < 0 || i >= kUpd) continue;
      const int side = f & 1;
      const T sg = side ? T(1) : T(-1);
      const T rx = (T)off[2 * side][i] - half * wex, ry = (T)off[2 * side + 1][i] - half * wey;
      const T tx = (T)off[4][i], ty = (T)off[5][i];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const T S = sg * fl[v][i], D = sg * fl[4 + v][i];
        S0[v] += S;
        Sx[v] += S * rx + D * tx;
        Sy[v] += S * ry + D * ty;
      }
    }
    if (sa + kUpd < nslot) __syncthreads();  // the next pass overwrites the table
  }
  if (bad) atomicOr(p.status, 1);
  if (!live) return;
  bad = false;
  Pred<T> pe;
  load_pred(p, e, pe, wex, wey);
  const double2 oe = p.shift[e];
  // volume term on the half-step cell's principal-axis rule
  {
    const double Vh = sh.geo[e], a = sh.geo[3 * n + e], b = sh.geo[4 * n + e],
                 c = sh.geo[5 * n + e];
    const double ox = oe.x + sh.geo[1 * n + e], oy = oe.y + sh.geo[2 * n + e];
    const double tr = 0.5 * (a + c), disc = sqrt(0.25 * (a - c) * (a - c) + b * b);
    const double lam[2] = {tr + disc, tr - disc};
    double ev[2][2];
    if (b == 0.0) {
      const bool xfirst = a >= c;
      ev[0][0] = xfirst ? 1.0 : 0.0;
      ev[0][1] = xfirst ? 0.0 : 1.0;
      ev[1][0] = xfirst ? 0.0 : 1.0;
      ev[1][1] = xfirst ? 1.0 : 0.0;
    } else {
      for (int k = 0; k < 2; ++k) {
        const double vx = b, vy = lam[k] - a, nn = sqrt(vx * vx + vy * vy);
        ev[k][0] = vx / nn;
        ev[k][1] = vy / nn;
      }
    }
    const T wv = (T)(0.25 * Vh);
    for (int k = 0; k < 2; ++k) {
      const double r = sqrt(2.0 * fmax(lam[k], 0.0) / Vh);
      for (int sgn = -1; sgn <= 1; sgn += 2) {
        const T rx = (T)(ox + sgn * r * ev[k][0]), ry = (T)(oy + sgn * r * ev[k][1]);
        T u[4];
        boosted_state(pe, rx, ry, wex, wey, igm1, u);
        const T ir = rcp(u[0]), vx = u[1] * ir, vy = u[2] * ir;
        const T pr = (gamma - T(1)) * (u[3] - T(0.5) * (u[1] * vx + u[2] * vy));
        bad |= !(u[0] > T(0)) || !(pr > T(0));
        T Fx[4] = {u[1], u[1] * vx + pr, u[2] * vx, (u[3] + pr) * vx};
        T Fy[4] = {u[2], u[1] * vy, u[2] * vy + pr, (u[3] + pr) * vy};
        unboost(Fx, wex, wey);
        unboost(Fy, wex, wey);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          Sx[v] += wv * Fx[v];
          Sy[v] += wv * Fy[v];
        }
      }
    }
  }
  // totals and moments about the carried origin
  const T V0 = (T)s0.geo[e], Mxx = (T)s0.geo[3 * n + e], Mxy = (T)s0.geo[4 * n + e],
          Myy = (T)s0.geo[5 * n + e];
  const T tdt = (T)dt;
  T qe[12];
  load12(p.ua, n, e, qe);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    p.out[(size_t)(3 * v) * n + e] = V0 * qe[3 * v] + tdt * S0[v];
    p.out[(size_t)(3 * v + 1) * n + e] = Mxx * qe[3 * v + 1] + Mxy * qe[3 * v + 2] + tdt * Sx[v];
    p.out[(size_t)(3 * v + 2) * n + e] = Mxy * qe[3 * v + 1] + Myy * qe[3 * v + 2] + tdt * Sy[v];
  }
  if (bad || !(qe[0] > T(0))) atomicOr(p.status, 1);
}

// CFL bound on the mesh of t^n (dg_cfl_dt).
template <typename T>
__global__ __launch_bounds__(256) void k_mv_cfl(PM<T> p) {
  const int e = xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  double dtb = 1e300;
  if (e < p.n) {
    const int n = p.n;
    int nb[kRing];
    double vx[kRing], vy[kRing];
    const int d = cell_polygon(p.s0, n, p.Lx, p.Ly, e, vx, vy, nb);
    const double rho = (double)p.in[e], ir = 1.0 / rho;
    const double ux = (double)p.in[(size_t)3 * n + e] * ir, uy = (double)p.in[(size_t)6 * n + e] * ir;
    const double pr =
        ((double)p.gamma - 1.0) * ((double)p.in[(size_t)9 * n + e] - 0.5 * rho * (ux * ux + uy * uy));
    const double cs = sqrt((double)p.gamma * pr * ir);
    double s = 0.0;
    for (int k = 0; k < d; ++k) {
      const int k1 = k + 1 == d ? 0 : k + 1;
      const double ex = vx[k1] - vx[k], ey = vy[k1] - vy[k];
      s += cs * sqrt(ex * ex + ey * ey);
      if (!p.motion) s += fabs(ux * ey - uy * ex);
    }
    dtb = 2.0 * p.s0.geo[e] / s;
  }
  dtb = wave_min(dtb);
  if ((threadIdx.x & 63) == 0) p.dtpart[e >> 6] = dtb;
}

template <typename T>
PM<T> make_params(const dg_mesh* m, const void* in, void* out) {
  const MVDev& v = *m->mvd;
  PM<T> p;
  std::memset(&p, 0, sizeof(p));
  p.in = static_cast<const T*>(in);
  p.ua = static_cast<const T*>(v.ua);
  p.ua_out = static_cast<T*>(v.ua);
  p.out = static_cast<T*>(out);
  p.status = m->status;
  p.n = v.n;
  p.Lx = v.box[0];
  p.Ly = v.box[1];
  p.gamma = (T)m->cfg.gamma;
  p.motion = v.motion;
  p.list = v.list;
  p.count = v.list + v.n;
  p.mid = v.mid;
  p.pred = static_cast<const T*>(v.pred);
  p.pred_out = static_cast<T*>(v.pred);
  p.shift = p.shift_out = v.shift;
  p.s0 = MSet{v.pos[v.cur], v.ring[v.cur], v.deg[v.cur], v.geo[v.cur]};
  p.sh = MSet{v.pos[1], v.ring[1], v.deg[1], v.geo[1]};
  p.xh = v.pos[1];
  p.x1 = v.pos[v.nxt];
  return p;
}

template <typename T>
hipError_t lim_launch(const PM<T>& p, int lim, hipStream_t s) {
  const dim3 g((p.n + 255) / 256), b(256);
  if (lim == DG_LIMITER_WENO)
    hipLaunchKernelGGL((k_mv_lim<T, 2>), g, b, 0, s, p);
  else if (lim == DG_LIMITER_MINMOD)
    hipLaunchKernelGGL((k_mv_lim<T, 1>), g, b, 0, s, p);
  else
    hipLaunchKernelGGL((k_mv_lim<T, 0>), g, b, 0, s, p);
  return hipGetLastError();
}

template <typename T>
hipError_t step_t(dg_mesh* m, const void* in, void* out, const double* dt_dev, double dt_host,
                  bool want_dt, hipStream_t s) {
  MVDev& v = *m->mvd;
  PM<T> p = make_params<T>(m, in, out);
  p.dt_dev = dt_dev;
  p.dt_host = dt_host;
  p.write_pos = 1;
  const dim3 g((p.n + 255) / 256), b(256);
  // per-phase events go straight into the record (launch_moving drops the
  // ones of a step that fails)
  auto mark = [&]() {
    if (!v.timing) return hipSuccess;
    hipEvent_t ev;
    hipError_t r = hipEventCreate(&ev);
    if (r != hipSuccess) return r;
    v.ev.push_back(ev);
    return hipEventRecord(ev, s);
  };
  hipError_t e = mark();
  if (e == hipSuccess) e = lim_launch(p, m->cfg.limiter, s);
  if (e == hipSuccess) e = mark();
  if (e != hipSuccess) return e;
  // mesh of the half-step generators (candidates from t^n)
  const MOut half{v.pos[1], v.ring[1], v.deg[1], v.geo[1]};
  const dim3 gw(std::min((p.n + 3) / 4, kWalkBlocks));
  hipLaunchKernelGGL((k_mv_check<T>), g, b, 0, s, p, p.s0, half);
  hipLaunchKernelGGL((k_mv_walk<T>), gw, b, 0, s, p, p.s0, half);
  hipLaunchKernelGGL((k_mv_geom<T, false>), g, b, 0, s, p, half);
  e = mark();
  if (e != hipSuccess) return e;
  if (m->cfg.flux == DG_FLUX_EXACT)
    hipLaunchKernelGGL((k_mv_upd<T, 1>), g, b, 0, s, p);
  else
    hipLaunchKernelGGL((k_mv_upd<T, 0>), g, b, 0, s, p);
  e = mark();
  if (e != hipSuccess) return e;
  // mesh of t^{n+1} (candidates from the half step) and the new state
  if (want_dt) p.dtpart = m->dtpart;
  p.mid_out = v.mid;
  const MOut next{v.pos[v.nxt], v.ring[v.nxt], v.deg[v.nxt], v.geo[v.nxt]};
  hipLaunchKernelGGL((k_mv_check<T>), g, b, 0, s, p, p.sh, next);
  hipLaunchKernelGGL((k_mv_walk<T>), gw, b, 0, s, p, p.sh, next);
  hipLaunchKernelGGL((k_mv_geom<T, true>), g, b, 0, s, p, next);
  e = hipGetLastError();
  if (e == hipSuccess) std::swap(v.cur, v.nxt);
  return e;
}

}  // namespace

hipError_t launch_min_finalize(const double* part, int n, double cfl, double* dt, hipStream_t s);

hipError_t launch_moving(dg_mesh* m, int mode, const void* in, void* out, const double* dt_dev,
                         double dt_host, double cfl, double* dt_next, hipStream_t s) {
  const bool f64 = m->cfg.precision == DG_FP64;
  if (mode == kLimit) {
    if (f64) {
      PM<double> p = make_params<double>(m, in, nullptr);
      p.ua_out = static_cast<double*>(out);
      return lim_launch(p, m->cfg.limiter, s);
    }
    PM<float> p = make_params<float>(m, in, nullptr);
    p.ua_out = static_cast<float*>(out);
    return lim_launch(p, m->cfg.limiter, s);
  }
  if (mode != kMH) return hipErrorInvalidValue;
  MVDev& v = *m->mvd;
  const size_t ev0 = v.ev.size();
  hipError_t e = f64 ? step_t<double>(m, in, out, dt_dev, dt_host, dt_next != nullptr, s)
                     : step_t<float>(m, in, out, dt_dev, dt_host, dt_next != nullptr, s);
  if (e == hipSuccess && dt_next)
    e = launch_min_finalize(m->dtpart, (int)((m->ncells + 63) / 64), cfl, dt_next, s);
  if (e == hipSuccess && v.timing) {
    // the fifth event closes the new-mesh kernel and the dt reduction
    hipEvent_t last;
    e = hipEventCreate(&last);
    if (e == hipSuccess) {
      v.ev.push_back(last);
      e = hipEventRecord(last, s);
    }
  }
  if (e != hipSuccess) {
    // a failed step leaves no partial record: the timings stay in groups of five
    for (size_t k = ev0; k < v.ev.size(); ++k) (void)hipEventDestroy(v.ev[k]);
    v.ev.resize(ev0);
  }
  return e;
}

hipError_t launch_moving_cfl(const dg_mesh* m, const void* U, double cfl, double* dt_dev,
                             hipStream_t s) {
  const dim3 g((m->ncells + 255) / 256), b(256);
  if (m->cfg.precision == DG_FP64) {
    PM<double> p = make_params<double>(m, U, nullptr);
    p.dtpart = m->dtpart;
    hipLaunchKernelGGL((k_mv_cfl<double>), g, b, 0, s, p);
  } else {
    PM<float> p = make_params<float>(m, U, nullptr);
    p.dtpart = m->dtpart;
    hipLaunchKernelGGL((k_mv_cfl<float>), g, b, 0, s, p);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_min_finalize(m->dtpart, (int)((m->ncells + 63) / 64), cfl, dt_dev, s);
}

// ------------------------------------------------------------ host setup --
void moving_destroy(dg_mesh* m) {
  if (!m->mvd) return;
  MVDev& v = *m->mvd;
  for (hipEvent_t e : v.ev) (void)hipEventDestroy(e);
  for (int k = 0; k < 3; ++k) {
    (void)hipFree(v.pos[k]);
    (void)hipFree(v.ring[k]);
    (void)hipFree(v.deg[k]);
    (void)hipFree(v.geo[k]);
  }
  (void)hipFree(v.ua);
  (void)hipFree(v.list);
  (void)hipFree(v.mid);
  (void)hipFree(v.pred);
  (void)hipFree(v.shift);
  delete m->mvd;
  m->mvd = nullptr;
}

dg_status moving_create(dg_mesh* m, const dg_mesh_desc* d) {
  const int64_t n = d->ncells, nf = d->nfaces;
  if (n < 64 || n > (1 << 26) || nf < 1) {
    set_error("dg_mesh_create: a moving mesh needs 64 <= ncells <= 2^26 and its initial faces");
    return DG_EINVAL;
  }
  if (!d->generators || !d->face_cells || !d->face_shift) {
    set_error("dg_mesh_create: a moving mesh needs generators, face_cells and face_shift");
    return DG_EINVAL;
  }
  const double Lx = d->box[0], Ly = d->box[1];
  if (!(Lx > 0) || !(Ly > 0) || !std::isfinite(Lx) || !std::isfinite(Ly)) {
    set_error("dg_mesh_create: moving mesh box must be positive");
    return DG_EINVAL;
  }
  std::vector<double> pos(4 * n);
  for (int64_t i = 0; i < n; ++i) {
    const double x = d->generators[2 * i], y = d->generators[2 * i + 1];
    if (!std::isfinite(x) || !std::isfinite(y) || x < 0 || x >= Lx || y < 0 || y >= Ly) {
      set_error("dg_mesh_create: generator " + std::to_string(i) + " is not inside [0, box)");
      return DG_EINVAL;
    }
    pos[i] = x;
    pos[n + i] = y;
    pos[2 * n + 2 * i] = x;
    pos[2 * n + 2 * i + 1] = y;
  }
  // initial rings: each cell's face neighbours sorted by angle
  std::vector<std::vector<std::pair<double, int>>> nbr(n);
  for (int64_t f = 0; f < nf; ++f) {
    const int L = d->face_cells[2 * f], R = d->face_cells[2 * f + 1];
    if (L < 0 || L >= n || R < 0 || R >= n || L == R) {
      set_error("dg_mesh_create: initial face " + std::to_string(f) + " has bad cells");
      return DG_EINVAL;
    }
    const double dx = pos[R] + d->face_shift[2 * f] * Lx - pos[L];
    const double dy = pos[n + R] + d->face_shift[2 * f + 1] * Ly - pos[n + L];
    nbr[L].push_back({std::atan2(dy, dx), R});
    nbr[R].push_back({std::atan2(-dy, -dx), L});
  }
  std::vector<int> ring((size_t)n * kRing, -1), deg(n);
  for (int64_t i = 0; i < n; ++i) {
    auto& v = nbr[i];
    std::sort(v.begin(), v.end());
    if (v.size() < 3 || v.size() > (size_t)kRing) {
      set_error("dg_mesh_create: cell " + std::to_string(i) + " has " + std::to_string(v.size()) +
                " faces (3 to 16 supported)");
      return DG_EINVAL;
    }
    for (size_t k = 0; k < v.size(); ++k) {
      for (size_t k2 = 0; k2 < k; ++k2)
        if (v[k2].second == v[k].second) {
          set_error("dg_mesh_create: cells " + std::to_string(i) + " and " +
                    std::to_string(v[k].second) + " share two faces (mesh too coarse)");
          return DG_EINVAL;
        }
      ring[i * kRing + k] = v[k].second;
    }
    deg[i] = (int)v.size();
  }
  m->mvd = new (std::nothrow) MVDev();
  if (!m->mvd) {
    set_error("dg_mesh_create: out of host memory");
    return DG_ENOMEM;
  }
  MVDev& v = *m->mvd;
  v.n = (int)n;
  v.box[0] = Lx;
  v.box[1] = Ly;
  v.motion = 1;
  v.cur = 0;
  v.nxt = 2;
  hipError_t e = hipSuccess;
  for (int k = 0; k < 3 && e == hipSuccess; ++k) {
    e = hipMalloc((void**)&v.pos[k], sizeof(double) * 4 * n);
    if (e == hipSuccess) e = hipMalloc((void**)&v.ring[k], sizeof(int) * kRing * n);
    if (e == hipSuccess) e = hipMalloc((void**)&v.deg[k], sizeof(int) * n);
    if (e == hipSuccess) e = hipMalloc((void**)&v.geo[k], sizeof(double) * kGeo * n);
  }
  if (e == hipSuccess) e = hipMalloc(&v.ua, m->elem * 12 * n);
  if (e == hipSuccess) e = hipMalloc((void**)&v.mid, sizeof(double2) * kRing * n);
  if (e == hipSuccess) e = hipMalloc(&v.pred, m->elem * 14 * n);
  if (e == hipSuccess) e = hipMalloc((void**)&v.shift, sizeof(double2) * n);
  if (e == hipSuccess) e = hipMalloc((void**)&v.list, sizeof(int) * (n + 1));
  if (e == hipSuccess) e = hipMemset(v.list + n, 0, sizeof(int));
  if (e == hipSuccess)
    e = hipMemcpy(v.pos[0], pos.data(), sizeof(double) * 4 * n, hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(v.ring[1], ring.data(), sizeof(int) * kRing * n, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(v.deg[1], deg.data(), sizeof(int) * n, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    moving_destroy(m);
    return hip_fail(e, "dg_mesh_create: moving mesh upload");
  }
  return DG_OK;
}

// Build the mesh of t^0 from the uploaded rings (set 1) and positions (set 0);
// the caller checks the status word afterwards.
hipError_t moving_init(dg_mesh* m) {
  MVDev& v = *m->mvd;
  PM<double> p;
  std::memset(&p, 0, sizeof(p));
  p.status = m->status;
  p.list = v.list;
  p.count = v.list + v.n;
  p.mid_out = v.mid;
  p.n = v.n;
  p.Lx = v.box[0];
  p.Ly = v.box[1];
  p.gamma = m->cfg.gamma;
  const dim3 g((v.n + 255) / 256), b(256);
  const MOut first{v.pos[0], v.ring[0], v.deg[0], v.geo[0]};
  const dim3 gw(std::min((v.n + 3) / 4, kWalkBlocks));
  const MSet given{v.pos[0], v.ring[1], v.deg[1], v.geo[1]};
  hipLaunchKernelGGL((k_mv_check<double>), g, b, 0, nullptr, p, given, first);
  hipLaunchKernelGGL((k_mv_walk<double>), gw, b, 0, nullptr, p, given, first);
  hipLaunchKernelGGL((k_mv_geom<double, false>), g, b, 0, nullptr, p, first);
  return hipGetLastError();
}

}  // namespace dg

namespace dg {

// Host copy of the current mesh (synchronous).  Any output may be NULL.
int moving_read(const dg_mesh* m, double* gen, double* vol, double* cen, int32_t* ring,
                int32_t* deg) {
  const MVDev& v = *m->mvd;
  const int n = v.n;
  std::vector<double> pos(2 * (size_t)n), geo((size_t)kGeo * n);
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess)
    e = hipMemcpy(pos.data(), v.pos[v.cur], sizeof(double) * 2 * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess)
    e = hipMemcpy(geo.data(), v.geo[v.cur], sizeof(double) * kGeo * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess && ring)
    e = hipMemcpy(ring, v.ring[v.cur], sizeof(int) * kRing * n, hipMemcpyDeviceToHost);
  if (e == hipSuccess && deg)
    e = hipMemcpy(deg, v.deg[v.cur], sizeof(int) * n, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return (int)e;
  for (int i = 0; i < n; ++i) {
    if (gen) {
      gen[2 * i] = pos[i];
      gen[2 * i + 1] = pos[n + i];
    }
    if (vol) vol[i] = geo[i];
    if (cen) {
      cen[2 * i] = pos[i] + geo[(size_t)n + i];
      cen[2 * i + 1] = pos[n + i] + geo[2 * (size_t)n + i];
    }
  }
  return 0;
}

void moving_set_motion(dg_mesh* m, int motion) { m->mvd->motion = motion ? 1 : 0; }

static void drop_events(MVDev& v) {
  for (hipEvent_t e : v.ev) (void)hipEventDestroy(e);
  v.ev.clear();
}

void moving_set_timing(dg_mesh* m, int on) {
  drop_events(*m->mvd);
  m->mvd->timing = on != 0;
}

// Average durations (ms) of the four phases of the timed steps since the
// last call, then a fresh record.
int moving_timing(dg_mesh* m, double* avg_ms, int* nsteps) {
  MVDev& v = *m->mvd;
  hipError_t e = hipDeviceSynchronize();
  const int ns = (int)(v.ev.size() / 5);
  double acc[4] = {0, 0, 0, 0};
  for (int k = 0; k < ns && e == hipSuccess; ++k)
    for (int j = 0; j < 4 && e == hipSuccess; ++j) {
      float ms = 0.0f;
      e = hipEventElapsedTime(&ms, v.ev[5 * k + j], v.ev[5 * k + j + 1]);
      acc[j] += ms;
    }
  drop_events(v);
  if (e != hipSuccess) return (int)e;
  for (int j = 0; j < 4; ++j) avg_ms[j] = ns ? acc[j] / ns : 0.0;
  if (nsteps) *nsteps = ns;
  return 0;
}

}  // namespace dg
