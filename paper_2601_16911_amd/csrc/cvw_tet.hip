// DG on tetrahedra (P_1, P_2 at the equispaced lattice points; affine cells):
//
//  * tet_vertex_kernel -- eight lanes per mesh vertex: the Hermite data
//    D^k u^e(x_i), 1 <= |k| <= p, of every cell of the vertex patch (eq.
//    taylorsol) from reference derivatives of the basis at the reference
//    vertex and the chain rule with the cell's inverse Jacobian, the pointwise
//    smoothness indicators and Jiang-Shu weights, and the vertex candidate
//    (eq. taylorcand), Sec. 3.2.  Float64.
//  * tet_sensor_kernel -- one thread per cell: the cell-vertex WENO sensor
//    (eq. finalweno, eq. gamma) in float64 with the element semi-norms (eq.
//    snorm, h_e^{2|k|-3}) in closed form from the cell's volume and central
//    second moments (every polynomial involved has degree <= 2).
//  * tet_eval_kernel -- one thread per cell, float32: the viscosity (eq.
//    lostab), the shock-capturing weights (eqs. dissrateorig to alphaq), the
//    volume and interface terms of the DG residual and optionally the
//    Runge-Kutta stage update with the exact element mass; scalar laws and
//    the Euler equations (HLL at the faces; the sensor field and the SC
//    weights from the density).
//
// A face's points are Radon's symmetric rule; the neighbour's trace at the
// cell's own points comes from its nodes in the order of the own face's
// (fmap, by the neighbour's face and the permutation between the two cells'
// orders of the face's vertices, packed with its id by the mesh build).
#include "cvw_device.h"
#include "cvw_cells3d.h"

namespace cvw {

constexpr int TET_THREADS = 64;
constexpr int TET_VLANES = 8;      // lanes per vertex in the vertex pass

// sum over the eight lanes of the own half row (quad butterflies, then the
// mirrored lane of the other quad); every lane receives bitwise the same value
__device__ __forceinline__ double oct_sumd(double x) {
#pragma clang fp contract(off)
  x = x + dppd<(1 | (0 << 2) | (3 << 4) | (2 << 6))>(x);
  x = x + dppd<(2 | (3 << 2) | (0 << 4) | (1 << 6))>(x);
  x = x + dppd<0x141>(x);
  return x;
}

template <int P>
struct TetShape {
  static constexpr int NLOC = (P + 1) * (P + 2) * (P + 3) / 6, NK = NLOC - 1, NQ = (P + 1) * (P + 1) * (P + 1);
};

struct TetGeo {
  double x0[3];
  double J[3][3];   // J[a][b] = d x_a / d xi_b
  double A[3][3];   // J^{-1}: A[b][a] = d xi_b / d x_a
  double det, h;
};

__device__ __forceinline__ TetGeo load_tetgeo(const double* __restrict__ g, int64_t e) {
  TetGeo G;
  const double* p = g + e * 16;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    G.x0[a] = p[a];
#pragma unroll
    for (int b = 0; b < 3; ++b) G.J[a][b] = p[3 + 3 * a + b];
  }
  G.h = p[12];
  const double (&J)[3][3] = G.J;
  const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1], c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2],
               c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  G.det = J[0][0] * c00 + J[0][1] * c01 + J[0][2] * c02;
  const double inv = 1.0 / G.det;
  G.A[0][0] = c00 * inv;
  G.A[1][0] = c01 * inv;
  G.A[2][0] = c02 * inv;
  G.A[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * inv;
  G.A[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * inv;
  G.A[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * inv;
  G.A[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * inv;
  G.A[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * inv;
  G.A[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * inv;
  return G;
}

// physical derivatives (multi-index order (1,0,0),(0,1,0),(0,0,1),(2,0,0),
// (1,1,0),(1,0,1),(0,2,0),(0,1,1),(0,0,2)) from reference derivatives in the
// same order: d/dx_a = sum_b A[b][a] d/dxi_b
template <int P>
__device__ __forceinline__ void tet_phys(const double (&A)[3][3], const double* R, double* D) {
#pragma unroll
  for (int a = 0; a < 3; ++a) D[a] = A[0][a] * R[0] + A[1][a] * R[1] + A[2][a] * R[2];
  if constexpr (P >= 2) {
    double H[3][3];
    H[0][0] = R[3]; H[0][1] = H[1][0] = R[4]; H[0][2] = H[2][0] = R[5];
    H[1][1] = R[6]; H[1][2] = H[2][1] = R[7]; H[2][2] = R[8];
    const int ia[6] = {0, 0, 0, 1, 1, 2}, ic[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      double s = 0.0;
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int d = 0; d < 3; ++d) s = fma(A[b][ia[t]] * A[d][ic[t]], H[b][d], s);
      D[3 + t] = s;
    }
  }
}

// first derivatives at the offset dx of a Taylor polynomial t about its point (P = 2: plus
// the constant second derivatives, already in t[3..8])
template <int P>
__device__ __forceinline__ void taylor_first(const double* t, const double (&dx)[3], double (&D)[3]) {
  D[0] = t[0];
  D[1] = t[1];
  D[2] = t[2];
  if constexpr (P >= 2) {
    D[0] += t[3] * dx[0] + t[4] * dx[1] + t[5] * dx[2];
    D[1] += t[4] * dx[0] + t[6] * dx[1] + t[7] * dx[2];
    D[2] += t[5] * dx[0] + t[7] * dx[1] + t[8] * dx[2];
  }
}

// ---------------------------------------------------------------------------
// vertex pass
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void tet_vertex_kernel(const float* __restrict__ u, float* __restrict__ cand,
                                                         const int32_t* __restrict__ vptr,
                                                         const int32_t* __restrict__ vent,
                                                         const double* __restrict__ geot,
                                                         const TetTables* __restrict__ tab, int64_t Nv,
                                                         MethodScalars ms) {
  using S = TetShape<P>;
  constexpr int NLOC = S::NLOC, NK = S::NK;
  __shared__ double sTV[4][NK][NLOC];
  for (int i = threadIdx.x; i < 4 * NK * NLOC; i += blockDim.x) {
    const int l = i / (NK * NLOC), r = i % (NK * NLOC);
    sTV[l][r / NLOC][r % NLOC] = tab->TV[l][r / NLOC][r % NLOC];
  }
  __syncthreads();
  // TET_VLANES lanes per vertex, each taking every TET_VLANES-th cell of the patch
  const int64_t v = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / TET_VLANES;
  const int sub = threadIdx.x % TET_VLANES;
  const bool on = v < Nv;
  double acc[NK], wsum = 0.0;
#pragma unroll
  for (int k = 0; k < NK; ++k) acc[k] = 0.0;
  const int32_t i0 = on ? vptr[v] + sub : 0, i1 = on ? vptr[v + 1] : 0;
  for (int32_t i = i0; i < i1; i += TET_VLANES) {
    const int32_t ent = vent[i];
    const int64_t ce = ent >> 2;
    const int lv = ent & 3;
    const TetGeo G = load_tetgeo(geot, ce);
    const float* uc = u + ce * NLOC;
    const double u0 = static_cast<double>(uc[0]);
    double R[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) R[k] = 0.0;
#pragma unroll
    for (int j = 1; j < NLOC; ++j) {
      const double dj = static_cast<double>(uc[j]) - u0;
#pragma unroll
      for (int k = 0; k < NK; ++k) R[k] = fma(sTV[lv][k][j], dj, R[k]);
    }
    double D[NK];
    tet_phys<P>(G.A, R, D);
    // pointwise semi-norm with h_e^{2|k|} of this cell
    const double h2 = G.h * G.h;
    double b2 = 0.0;
#pragma unroll
    for (int k = 0; k < NK; ++k) b2 = fma((k < 3 ? h2 : h2 * h2) * D[k], D[k], b2);
    double beta = sqrt(b2);
    double w;
    if (ms.fast_exp) {
      const double t = ms.eps_vd + beta;
      w = 1.0 / (t * t);
    } else {
      beta = pow(beta, static_cast<double>(ms.q_beta));
      w = pow(ms.eps_vd + beta, -static_cast<double>(ms.r));
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) acc[k] = fma(w, D[k], acc[k]);
    wsum += w;
  }
  // sums over the vertex's lanes (all lanes of the wavefront take part)
#pragma unroll
  for (int k = 0; k < NK; ++k) acc[k] = oct_sumd(acc[k]);
  wsum = oct_sumd(wsum);
  if (!on || sub != 0) return;
  const double iw = 1.0 / wsum;
#pragma unroll
  for (int k = 0; k < NK; ++k) cand[v * NK + k] = static_cast<float>(acc[k] * iw);
}

// ---------------------------------------------------------------------------
// cell pass
// ---------------------------------------------------------------------------
template <int FLUX>
__device__ __forceinline__ float tet_fn(const MethodScalars& ms, float u, const float (&n)[3]) {
  const float vn = ms.fp[0] * n[0] + ms.fp[1] * n[1] + ms.fp[2] * n[2];
  if constexpr (FLUX == CVW_BURGERS) return 0.5f * u * u * vn;
  else return vn * u;
}

// Element semi-norm (eq. snorm, weights h_e^{2|k|-3}) of a polynomial of
// degree <= 2 on an affine cell, in closed form: its gradient is affine,
// g + H (x - x_c) with g the gradient at the centroid x_c and H the constant
// Hessian (xx, xy, xz, yy, yz, zz), so that
//   int_K |grad p|^2 = vol |g|^2 + tr(M H H),  M = int_K (x - x_c)(x - x_c)^T,
//   int_K |D^k p|^2 = vol H_k^2 for |k| = 2.
template <int P>
__device__ __forceinline__ double tet_snorm(const double (&g)[3], const double (&H)[6], const double (&M)[6], double vol,
                                            double hw1, double hw2) {
  double s1 = vol * (g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
  if constexpr (P >= 2) {
    const double Hf[3][3] = {{H[0], H[1], H[2]}, {H[1], H[3], H[4]}, {H[2], H[4], H[5]}};
    const double Mf[3][3] = {{M[0], M[1], M[2]}, {M[1], M[3], M[4]}, {M[2], M[4], M[5]}};
    // tr(M H H) = sum_{a,c} (M H)_{ac} H_{ca}
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double mh = Mf[a][0] * Hf[0][c] + Mf[a][1] * Hf[1][c] + Mf[a][2] * Hf[2][c];
        s1 = fma(mh, Hf[c][a], s1);
      }
    double s2 = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) s2 = fma(H[t], H[t], s2);
    return fma(hw1, s1, hw2 * vol * s2);
  } else {
    return hw1 * s1;
  }
}

// Sensor pass: one thread per cell, float64 (the weights, square roots and
// the ratio of gamma_e in float32).  u_h, the four vertex candidates (Taylor
// polynomials about the vertices, eq. taylorcand) and u_h - u_h^{e,*} are
// polynomials of degree <= p, each semi-norm the closed form above.
template <int P>
__global__ __launch_bounds__(TET_THREADS) void tet_sensor_kernel(const float* __restrict__ u, float* __restrict__ gamma,
                                                                 const float* __restrict__ cand,
                                                                 const int32_t* __restrict__ cell_vtx,
                                                                 const double* __restrict__ geot,
                                                                 const TetTables* __restrict__ tab, int64_t E,
                                                                 MethodScalars ms) {
  using S = TetShape<P>;
  constexpr int NLOC = S::NLOC, NK = S::NK;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * TET_THREADS + threadIdx.x;
  if (e >= E) return;
  const int4 vid = *reinterpret_cast<const int4*>(cell_vtx + e * 4);
  const TetGeo G = load_tetgeo(geot, e);
  float uv[NLOC];
#pragma unroll
  for (int j = 0; j < NLOC; ++j) uv[j] = u[e * NLOC + j];
  const double vol = G.det / 6.0;
  const double hw1 = 1.0 / G.h, hw2 = G.h;          // h_e^{2|k|-3}: |k| = 1, 2
  // centroid offset from vertex 0 and the central second moments
  // M = vol / 20 sum_i y_i y_i^T (y_i the vertices about the centroid)
  double cc[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) cc[a] = 0.25 * (G.J[a][0] + G.J[a][1] + G.J[a][2]);
  double M[6];
  {
    const int ia[6] = {0, 0, 0, 1, 1, 2}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int a = ia[t], b = ib[t];
      const double s = G.J[a][0] * G.J[b][0] + G.J[a][1] * G.J[b][1] + G.J[a][2] * G.J[b][2] - 4.0 * cc[a] * cc[b];
      M[t] = vol / 20.0 * s;
    }
  }
  // u_h: the gradient at the centroid and the Hessian, from the nodal values
  // less the first one
  double du[NLOC];
  const double u00 = static_cast<double>(uv[0]);
#pragma unroll
  for (int j = 0; j < NLOC; ++j) du[j] = static_cast<double>(uv[j]) - u00;
  double R[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) R[k] = 0.0;
#pragma unroll
  for (int j = 1; j < NLOC; ++j) {
#pragma unroll
    for (int b = 0; b < 3; ++b) R[b] = fma(tab->Gc[b][j], du[j], R[b]);
    if constexpr (P >= 2) {
#pragma unroll
      for (int t = 0; t < 6; ++t) R[3 + t] = fma(tab->H2[t][j], du[j], R[3 + t]);
    }
  }
  double D[NK];
  tet_phys<P>(G.A, R, D);
  double gu[3] = {D[0], D[1], D[2]}, Hu[6] = {0, 0, 0, 0, 0, 0};
  if constexpr (P >= 2) {
#pragma unroll
    for (int t = 0; t < 6; ++t) Hu[t] = D[3 + t];
  }
  const double n02 = tet_snorm<P>(gu, Hu, M, vol, hw1, hw2);
  // the candidates: Taylor data about vertex l; gradient at the centroid
  // t_grad + H (x_c - x_l)
  double gl[4][3], Hl[4][6], b2[4];
  const int32_t vv[4] = {vid.x, vid.y, vid.z, vid.w};
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    const float* cv = cand + static_cast<int64_t>(vv[l]) * NK;
    double t[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) t[k] = static_cast<double>(cv[k]);
    double dx[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) dx[a] = l == 0 ? cc[a] : cc[a] - G.J[a][l - 1];
#pragma unroll
    for (int a = 0; a < 3; ++a) gl[l][a] = t[a];
#pragma unroll
    for (int q = 0; q < 6; ++q) Hl[l][q] = 0.0;
    if constexpr (P >= 2) {
#pragma unroll
      for (int q = 0; q < 6; ++q) Hl[l][q] = t[3 + q];
      gl[l][0] += t[3] * dx[0] + t[4] * dx[1] + t[5] * dx[2];
      gl[l][1] += t[4] * dx[0] + t[6] * dx[1] + t[7] * dx[2];
      gl[l][2] += t[5] * dx[0] + t[7] * dx[1] + t[8] * dx[2];
    }
    b2[l] = tet_snorm<P>(gl[l], Hl[l], M, vol, hw1, hw2);
  }
  // weights of the cell candidate and the four vertex candidates
  const float n0 = fsqrt(static_cast<float>(fmax(n02, 0.0)));
  double om[5];
  {
    float wf[5], wsum = 0.0f;
#pragma unroll
    for (int l = 0; l < 5; ++l) {
      const float b = l == 0 ? n0 : fsqrt(static_cast<float>(fmax(b2[l - 1], 0.0)));
      const float lin = l == 0 ? 1.0f - 4.0f * ms.lin_w : ms.lin_w;
      if (ms.fast_exp) {
        const float tt = ms.eps_c + b;
        wf[l] = lin / (tt * tt);
      } else {
        wf[l] = lin * powf(ms.eps_c + powf(b, ms.q_beta), -ms.r);
      }
      wsum += wf[l];
    }
#pragma unroll
    for (int l = 0; l < 5; ++l) om[l] = static_cast<double>(wf[l] / wsum);
  }
  double osum = 0.0;
#pragma unroll
  for (int l = 1; l < 5; ++l) osum += om[l];
  // u_h - u_h^{e,*} = sum_{l >= 1} omega_l (u_h - s_l)
  double gd[3], Hd[6];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double v = osum * gu[a];
#pragma unroll
    for (int l = 0; l < 4; ++l) v = fma(-om[l + 1], gl[l][a], v);
    gd[a] = v;
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    double v = osum * Hu[q];
#pragma unroll
    for (int l = 0; l < 4; ++l) v = fma(-om[l + 1], Hl[l][q], v);
    Hd[q] = v;
  }
  const double d2 = tet_snorm<P>(gd, Hd, M, vol, hw1, hw2);
  float gam = 1.0f;
  if (n02 > 0.0) {
    float ratio = fminf(1.0f, fsqrt(static_cast<float>(fmax(d2, 0.0))) / n0);
    if (!ms.fast_exp) ratio = powf(ratio, ms.q_sensor);
    gam = 1.0f - ratio;
  }
  gamma[e] = gam;
}

// Variables per node (the Euler equations: rho, m_x, m_y, m_z, E)
template <int FLUX>
struct TetNV {
  static constexpr int value = FLUX == CVW_EULER ? 5 : 1;
};

// Euler: velocity and pressure of a state
__device__ __forceinline__ float tet_prim(const MethodScalars& ms, const float* u, float (&v)[3]) {
  const float inv = frcp(u[0]);
  v[0] = u[1] * inv;
  v[1] = u[2] * inv;
  v[2] = u[3] * inv;
  return (ms.fp[0] - 1.0f) * (u[4] - 0.5f * u[0] * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]));
}

// HLL with Davis wave-speed estimates for the Euler equations, normal n
__device__ __forceinline__ void tet_hll(const MethodScalars& ms, const float* um, const float* up, const float (&n)[3],
                                        float* fs) {
  const float g = ms.fp[0];
  float vm3[3], vp3[3];
  const float pm = tet_prim(ms, um, vm3), pp = tet_prim(ms, up, vp3);
  const float vm = vm3[0] * n[0] + vm3[1] * n[1] + vm3[2] * n[2];
  const float vp = vp3[0] * n[0] + vp3[1] * n[1] + vp3[2] * n[2];
  const float cm = fsqrt(fmaxf(g * pm * frcp(um[0]), 0.0f)), cp = fsqrt(fmaxf(g * pp * frcp(up[0]), 0.0f));
  const float SL = fminf(vm - cm, vp - cp);
  const float SR = fmaxf(vm + cm, vp + cp);
  float Fm[5], Fp[5];
  Fm[0] = um[0] * vm;
  Fp[0] = up[0] * vp;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    Fm[1 + a] = um[1 + a] * vm + pm * n[a];
    Fp[1 + a] = up[1 + a] * vp + pp * n[a];
  }
  Fm[4] = (um[4] + pm) * vm;
  Fp[4] = (up[4] + pp) * vp;
  const float inv = frcp(SR - SL);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const float mid = (SR * Fm[v] - SL * Fp[v] + SL * SR * (up[v] - um[v])) * inv;
    fs[v] = (SL >= 0.0f) ? Fm[v] : ((SR <= 0.0f) ? Fp[v] : mid);
  }
}

// the nodes of face f: its vertices a < b < c, for P = 2 then the midpoints ab, ac, bc
template <int P>
struct TetFace {
  static constexpr int NF = (P + 1) * (P + 2) / 2;
  int n[4][NF];
  constexpr TetFace() : n{} {
    const int V[4][3] = {{1, 2, 3}, {0, 2, 3}, {0, 1, 3}, {0, 1, 2}};
    const int vert[4] = {0, P == 1 ? 1 : 2, P == 1 ? 2 : 5, P == 1 ? 3 : 9};
    const int mid[4][4] = {{0, 1, 3, 6}, {1, 0, 4, 7}, {3, 4, 0, 8}, {6, 7, 8, 0}};
    for (int f = 0; f < 4; ++f)
      for (int i = 0; i < 3; ++i) {
        n[f][i] = vert[V[f][i]];
        if (P == 2) n[f][NF - 3 + i] = mid[V[f][i == 2 ? 1 : 0]][V[f][i == 0 ? 1 : 2]];
      }
  }
};
template <int P>
inline constexpr TetFace<P> tet_face{};

// Cell pass, one thread per cell.  A polynomial of the cell is kept as its
// monomial coefficients about the centroid (c[0]; x, y, z; for P = 2 xx, xy,
// xz, yy, yz, zz, the squares' doubled; from differences, so that constants
// have zero gradients; about a vertex the residual's error is 1.4 times as
// large).  The volume points lie on lines along x, on which a variable is one
// polynomial in x: values and gradients cost a few multiply-adds per point,
// and the test functions' gradients, affine too, need only the moments of the
// flux in 1, x, y, z.  A face's trace depends on its nodes alone; the
// neighbour's are read in the order of the own face.  VALU bound: 13,000
// instructions per wavefront of P_2 Euler cells, two wavefronts per SIMD at
// 226 registers (three would spill: 209 us).  300,366 cells, residual: 171 us
// against 273 with the basis and its gradients applied node by node at every
// point (24,900 instructions).
template <int P, int FLUX>
__global__ __launch_bounds__(TET_THREADS) void tet_eval_kernel(
    const float* __restrict__ u, const float* __restrict__ u0, float* __restrict__ out, float* __restrict__ gamma_out,
    float* __restrict__ alpha_out, const float* __restrict__ gamma_in, const int32_t* __restrict__ nbrt, const double* __restrict__ geot, const TetTables* __restrict__ tab, int64_t E,
    MethodScalars ms, int mode, float dt, float a0, float b0, uint32_t* __restrict__ status) {
  using S = TetShape<P>;
  constexpr int NLOC = S::NLOC, NQ = S::NQ, NV = TetNV<FLUX>::value, N1 = P + 1, NF = TetFace<P>::NF;
  const int tid = threadIdx.x;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * TET_THREADS + tid;
  if (e >= E) return;
  const TetGeo G = load_tetgeo(geot, e);
  // variable v of cell e at (v E + e) NLOC
  float uv[NV][NLOC];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int j = 0; j < NLOC; ++j) uv[v][j] = u[(v * E + e) * NLOC + j];
  const int4 nb4 = reinterpret_cast<const int4*>(nbrt)[e];

  // ---- gamma_e: from the sensor pass, or the fixed value
  const float gam = ms.sensor_kind != CVW_SENSOR_FIXED ? gamma_in[e] : ms.fixed_gamma;

  // ---- residual (float32)
  float A[3][3];
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a) A[b][a] = static_cast<float>(G.A[b][a]);
  float n0[3];                                 // -grad lambda_0
#pragma unroll
  for (int a = 0; a < 3; ++a) n0[a] = static_cast<float>(G.A[0][a] + G.A[1][a] + G.A[2][a]);
  const float fdet = static_cast<float>(G.det);
  // monomial coefficients about the centroid
  float c[NV][NLOC];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const float* w = uv[v];
    if constexpr (P == 1) {
#pragma unroll
      for (int j = 1; j < 4; ++j) c[v][j] = w[j] - w[0];
      c[v][0] = fmaf(0.25f, c[v][1] + c[v][2] + c[v][3], w[0]);
    } else {
      // at the centroid the vertex functions have value -1/8 and gradient 0,
      // the midpoint functions 1/4 and the sum of their two grad lambda
      const float x1 = 4.0f * (w[1] - w[0]), x2 = w[2] - w[0], y1 = 4.0f * (w[3] - w[0]), y2 = w[5] - w[0];
      const float z1 = 4.0f * (w[6] - w[0]), z2 = w[9] - w[0];
      const float xy = 4.0f * (w[4] - w[0]), xz = 4.0f * (w[7] - w[0]), yz = 4.0f * (w[8] - w[0]);
      c[v][0] = w[0] + (0.0625f * ((x1 + y1 + z1) + (xy + xz + yz)) - 0.125f * (x2 + y2 + z2));
      c[v][1] = (w[4] - w[3]) + (w[7] - w[6]);
      c[v][2] = (w[4] - w[1]) + (w[8] - w[6]);
      c[v][3] = (w[7] - w[1]) + (w[8] - w[3]);
      c[v][4] = 2.0f * (2.0f * x2 - x1);
      c[v][5] = xy - x1 - y1;
      c[v][6] = xz - x1 - z1;
      c[v][7] = 2.0f * (2.0f * y2 - y1);
      c[v][8] = yz - y1 - z1;
      c[v][9] = 2.0f * (2.0f * z2 - z1);
    }
  }
  // a variable on the line t: l[0] + l[1] x (+ l[2] x^2 / 2), and the physical
  // gradient there: p + q x
  auto line_val = [&](int v, const float* t, float (&l)[3]) {
    const float y = t[0], z = t[1], yh = t[2], zh = t[3];
    if constexpr (P == 1) {
      l[0] = fmaf(c[v][2], y, fmaf(c[v][3], z, c[v][0]));
      l[1] = c[v][1];
      l[2] = 0.0f;
    } else {
      const float ty = fmaf(c[v][8], z, fmaf(c[v][7], yh, c[v][2]));
      const float tz = fmaf(c[v][9], zh, c[v][3]);
      l[0] = fmaf(ty, y, fmaf(tz, z, c[v][0]));
      l[1] = fmaf(c[v][5], y, fmaf(c[v][6], z, c[v][1]));
      l[2] = c[v][4];
    }
  };
  auto line_grad = [&](int v, const float* t, float (&p)[3], float (&q)[3]) {
    const float y = t[0], z = t[1];
    float gx = c[v][1], gy = c[v][2], gz = c[v][3];
    if constexpr (P == 2) {
      gx = fmaf(c[v][5], y, fmaf(c[v][6], z, gx));
      gy = fmaf(c[v][8], z, fmaf(c[v][7], y, gy));
      gz = fmaf(c[v][8], y, fmaf(c[v][9], z, gz));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      p[a] = fmaf(A[0][a], gx, fmaf(A[1][a], gy, A[2][a] * gz));
      q[a] = P == 1 ? 0.0f : fmaf(A[1][a], c[v][P == 1 ? 0 : 5], fmaf(A[2][a], c[v][P == 1 ? 0 : 6], A[0][a] * c[v][P == 1 ? 0 : 4]));
    }
  };
  auto line_at = [&](const float (&l)[3], const float* t, int i) {
    return P == 1 ? fmaf(l[1], t[4 + i], l[0]) : fmaf(fmaf(l[2], t[7 + i], l[1]), t[4 + i], l[0]);
  };

  // second derivatives of the sensor field (P = 2; constant), for alpha~
  float hs2 = 0.0f;
  if constexpr (P >= 2) {
    double R[S::NK] = {}, D[S::NK], w[NLOC];
#pragma unroll
    for (int j = 0; j < NLOC; ++j) w[j] = static_cast<double>(uv[0][j]);
    R[3] = 4.0 * ((w[2] - w[1]) - (w[1] - w[0]));
    R[4] = 4.0 * ((w[4] - w[3]) - (w[1] - w[0]));
    R[5] = 4.0 * ((w[7] - w[6]) - (w[1] - w[0]));
    R[6] = 4.0 * ((w[5] - w[3]) - (w[3] - w[0]));
    R[7] = 4.0 * ((w[8] - w[6]) - (w[3] - w[0]));
    R[8] = 4.0 * ((w[9] - w[6]) - (w[6] - w[0]));
    tet_phys<P>(G.A, R, D);
#pragma unroll
    for (int t = 0; t < 6; ++t) hs2 += static_cast<float>(D[3 + t] * D[3 + t]);
  }
  float lam = ms.lam_g;
  if (!(lam > 0.0f)) {
    const float vn = fsqrt(ms.fp[0] * ms.fp[0] + ms.fp[1] * ms.fp[1] + ms.fp[2] * ms.fp[2]);
    lam = 0.0f;
#pragma unroll 1
    for (int k = 0; k < N1 * N1; ++k) {
      const float* t = tab->line[k];
      float l[NV][3];
#pragma unroll
      for (int v = 0; v < NV; ++v) line_val(v, t, l[v]);
#pragma unroll
      for (int i = 0; i < N1; ++i) {
        float uq[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) uq[v] = line_at(l[v], t, i);
        float sp;
        if constexpr (FLUX == CVW_EULER) {
          float vel[3];
          const float pq = tet_prim(ms, uq, vel);
          sp = fsqrt(vel[0] * vel[0] + vel[1] * vel[1] + vel[2] * vel[2]) + fsqrt(fmaxf(ms.fp[0] * pq * frcp(uq[0]), 0.0f));
        } else {
          sp = FLUX == CVW_BURGERS ? fabsf(uq[0]) * vn : vn;
        }
        lam = fmaxf(lam, sp);
      }
    }
  }
  const float nu = lam * static_cast<float>(G.h) / (2.0f * P);
  // SC weights (sensor field): S = sum W f, T = sum W alpha~ f over the volume points
  const bool sc_active = ms.sc_on && gam < ms.c_gamma;
  float Sv = 0.0f, Tv = 0.0f;
  const float fh2 = static_cast<float>(G.h * G.h);
  const float ah2 = fh2 * fh2 * hs2;
  if (sc_active) {
#pragma unroll 1
    for (int k = 0; k < N1 * N1; ++k) {
      const float* t = tab->line[k];
      float p[3], q[3];
      line_grad(0, t, p, q);
#pragma unroll
      for (int i = 0; i < N1; ++i) {
        float g2 = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const float d = fmaf(q[a], t[4 + i], p[a]);
          g2 = fmaf(d, d, g2);
        }
        const float W = t[10 + i] * fdet;
        const float f = (1.0f - gam) * g2;
        Sv = fmaf(W, f, Sv);
        Tv = fmaf(W * fsqrt(fmaf(fh2, g2, ah2)), f, Tv);
      }
    }
  }
  const bool use_alpha = sc_active && Sv > 0.0f && Tv > 0.0f;
  const float ratioST = use_alpha ? Sv / Tv : 0.0f;
  const float nug = nu * (1.0f - gam);

  // ---- volume terms: the moments of V = w (nu alpha (1 - gamma) grad u - f(u))
  // in reference components, M[v]: V_x, V_y, V_z; for P = 2 also x V_x,
  // y V_x + x V_y, z V_x + x V_z, y V_y, z V_y + y V_z, z V_z
  float M[NV][NLOC - 1];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int k = 0; k < NLOC - 1; ++k) M[v][k] = 0.0f;
#pragma unroll 1
  for (int k = 0; k < N1 * N1; ++k) {
    const float* t = tab->line[k];
    const float y = t[0], z = t[1];
    float uq[NV][N1], gs[N1];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float l[3];
      line_val(v, t, l);
#pragma unroll
      for (int i = 0; i < N1; ++i) uq[v][i] = line_at(l, t, i);
    }
#pragma unroll
    for (int i = 0; i < N1; ++i) gs[i] = 1.0f;
    if (use_alpha) {
      float p[3], q[3];
      line_grad(0, t, p, q);
#pragma unroll
      for (int i = 0; i < N1; ++i) {
        float g2 = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const float d = fmaf(q[a], t[4 + i], p[a]);
          g2 = fmaf(d, d, g2);
        }
        gs[i] = fsqrt(fmaf(fh2, g2, ah2)) * ratioST;
      }
    }
    if (mode == MODE_SENSOR) {
      if (alpha_out)
#pragma unroll
        for (int i = 0; i < N1; ++i) alpha_out[e * NQ + N1 * k + i] = gs[i];
      continue;
    }
    float inv[N1], pres[N1];                 // 1 / rho and pressure (Euler)
#pragma unroll
    for (int i = 0; i < N1; ++i) {
      gs[i] *= nug;
      pres[i] = inv[i] = 0.0f;
      if constexpr (FLUX == CVW_EULER) {
        inv[i] = frcp(uq[0][i]);
        const float m2 = uq[1][i] * uq[1][i] + uq[2][i] * uq[2][i] + uq[3][i] * uq[3][i];
        pres[i] = (ms.fp[0] - 1.0f) * (uq[4][i] - 0.5f * m2 * inv[i]);
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float p[3], q[3], S0[3] = {0.0f, 0.0f, 0.0f}, S1[3] = {0.0f, 0.0f, 0.0f};
      line_grad(v, t, p, q);
#pragma unroll
      for (int i = 0; i < N1; ++i) {
        const float w = t[10 + i], wx = t[13 + i];
        // Euler: f_a of variable v: m_a, m_c v_a + p delta_ca, (E + p) v_a = h m_a (+ p delta_ca)
        float h = 0.0f;
        if constexpr (FLUX == CVW_EULER) h = (v < 4 ? uq[v][i] : uq[4][i] + pres[i]) * inv[i];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          float fa;
          if constexpr (FLUX == CVW_EULER)
            fa = v == 0 ? uq[1 + a][i] : h * uq[1 + a][i] + (v - 1 == a ? pres[i] : 0.0f);
          else
            fa = FLUX == CVW_BURGERS ? 0.5f * uq[0][i] * uq[0][i] * ms.fp[a] : ms.fp[a] * uq[0][i];
          const float V = gs[i] * (P == 1 ? p[a] : fmaf(q[a], t[4 + i], p[a])) - fa;
          S0[a] = fmaf(w, V, S0[a]);
          if constexpr (P == 2) S1[a] = fmaf(wx, V, S1[a]);
        }
      }
      float r0[3], r1[3];
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        r0[b] = A[b][0] * S0[0] + A[b][1] * S0[1] + A[b][2] * S0[2];
        r1[b] = P == 1 ? 0.0f : A[b][0] * S1[0] + A[b][1] * S1[1] + A[b][2] * S1[2];
        M[v][b] += r0[b];
      }
      if constexpr (P == 2) {
        M[v][3] += r1[0];
        M[v][4] += fmaf(y, r0[0], r1[1]);
        M[v][5] += fmaf(z, r0[0], r1[2]);
        M[v][6] = fmaf(y, r0[1], M[v][6]);
        M[v][7] = fmaf(z, r0[1], fmaf(y, r0[2], M[v][7]));
        M[v][8] = fmaf(z, r0[2], M[v][8]);
      }
    }
  }
  if (mode == MODE_SENSOR) {
    if (gamma_out) gamma_out[e] = gam;
    return;
  }
  // sum_q V . grad phi_j from the moments: the transpose of the coefficients
  float r[NV][NLOC];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    float m[NLOC - 1];
#pragma unroll
    for (int k = 0; k < NLOC - 1; ++k) m[k] = M[v][k] * fdet;
    if constexpr (P == 1) {
      r[v][0] = -(m[0] + m[1] + m[2]);
      r[v][1] = m[0];
      r[v][2] = m[1];
      r[v][3] = m[2];
    } else {
      r[v][0] = 4.0f * ((m[3] + m[6] + m[8]) + (m[4] + m[5] + m[7]));
      r[v][1] = -(m[1] + m[2]) - 4.0f * (2.0f * m[3] + m[4] + m[5]);
      r[v][2] = 4.0f * m[3];
      r[v][3] = -(m[0] + m[2]) - 4.0f * (2.0f * m[6] + m[4] + m[7]);
      r[v][4] = (m[0] + m[1]) + 4.0f * m[4];
      r[v][5] = 4.0f * m[6];
      r[v][6] = -(m[0] + m[1]) - 4.0f * (2.0f * m[8] + m[5] + m[7]);
      r[v][7] = (m[0] + m[2]) + 4.0f * m[5];
      r[v][8] = (m[1] + m[2]) + 4.0f * m[7];
      r[v][9] = 4.0f * m[8];
    }
  }

  // ---- interface terms (face f opposite vertex f): the outward normal is
  // -grad lambda_f / |grad lambda_f|, the face Jacobian |det J| |grad lambda_f|
  // The cell's values are read again: their registers are needed meanwhile.
  int64_t er = e;
  asm volatile("" : "+v"(er));
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int j = 0; j < NLOC; ++j) uv[v][j] = u[(v * E + er) * NLOC + j];
  // one face per copy of the code (its nodes are registers), its points rolled
  const int32_t codes[4] = {nb4.x, nb4.y, nb4.z, nb4.w};
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int64_t e2 = codes[f] >> 5;
    const uint32_t pk = tab->fmap[codes[f] & 31];
    float un[NV][NF];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int i = 0; i < NF; ++i) un[v][i] = u[(v * E + e2) * NLOC + ((pk >> (4 * i)) & 15)];
    float n[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) n[a] = f == 0 ? n0[a] : -A[f == 0 ? 0 : f - 1][a];
    const float na = fsqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]), ina = 1.0f / na;
    const float jf = fabsf(fdet) * na;
#pragma unroll
    for (int a = 0; a < 3; ++a) n[a] *= ina;
    const float bn = fabsf(ms.fp[0] * n[0] + ms.fp[1] * n[1] + ms.fp[2] * n[2]);
#pragma unroll 1
    for (int g = 0; g < TET_NFP; ++g) {
      const float* B = tab->Bt[g];
      float um[NV], up[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        um[v] = B[0] * uv[v][tet_face<P>.n[f][0]];
        up[v] = B[0] * un[v][0];
#pragma unroll
        for (int i = 1; i < NF; ++i) {
          um[v] = fmaf(B[i], uv[v][tet_face<P>.n[f][i]], um[v]);
          up[v] = fmaf(B[i], un[v][i], up[v]);
        }
      }
      float fs[NV];
      if constexpr (FLUX == CVW_EULER) {
        tet_hll(ms, um, up, n, fs);
      } else {
        float lf = ms.lam_g;
        if (!(lf > 0.0f)) lf = FLUX == CVW_BURGERS ? fmaxf(fabsf(um[0]), fabsf(up[0])) * bn : bn;
        fs[0] = 0.5f * (tet_fn<FLUX>(ms, um[0], n) + tet_fn<FLUX>(ms, up[0], n)) - 0.5f * lf * (up[0] - um[0]);
      }
      const float wj = tab->wf[g] * jf;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const float w = wj * fs[v];
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          float& x = r[v][tet_face<P>.n[f][i]];
          x = fmaf(B[i], w, x);
        }
      }
    }
  }

  // ---- output: r, or u_out = a0 u_n + b0 (u - dt M_e^{-1} r), M_e = det J M_ref
  bool nonfinite = false;
  const float scl = dt / fdet;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int64_t idx = (v * E + e) * NLOC;
    float o[NLOC];
    if (mode == MODE_RESIDUAL) {
#pragma unroll
      for (int j = 0; j < NLOC; ++j) o[j] = r[v][j];
    } else {
      float base[NLOC];
#pragma unroll
      for (int j = 0; j < NLOC; ++j) base[j] = 0.0f;
      if (a0 != 0.0f)
#pragma unroll
        for (int j = 0; j < NLOC; ++j) base[j] = a0 * u0[idx + j];
#pragma unroll
      for (int j = 0; j < NLOC; ++j) {
        float x = 0.0f;
#pragma unroll
        for (int i = 0; i < NLOC; ++i) x = fmaf(tab->Minv[j][i], r[v][i], x);
        o[j] = base[j] + b0 * (uv[v][j] - scl * x);
      }
    }
#pragma unroll
    for (int j = 0; j < NLOC; ++j) {
      nonfinite |= !isfinite(o[j]);
      out[idx + j] = o[j];
    }
  }
  if (gamma_out) gamma_out[e] = gam;
  if (nonfinite) atomicOr(status, ST_NONFINITE);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
cvw_status tet_candidates(const cvw_mesh* m, const cvw_params* prm, const float* u, float* cand, hipStream_t s) {
  const MethodScalars ms = make_scalars(prm);
  const dim3 g(static_cast<unsigned>((m->Nv * TET_VLANES + 255) / 256)), b(256);
  switch (m->degree) {
    case 1: hipLaunchKernelGGL(tet_vertex_kernel<1>, g, b, 0, s, u, cand, m->d_vtx_ptr, m->d_vtx_ent, m->d_geoth, m->d_tett, m->Nv, ms); break;
    case 2: hipLaunchKernelGGL(tet_vertex_kernel<2>, g, b, 0, s, u, cand, m->d_vtx_ptr, m->d_vtx_ent, m->d_geoth, m->d_tett, m->Nv, ms); break;
    default: set_error("tetrahedra: degree 1 or 2"); return CVW_EUNSUPPORTED;
  }
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

template <int P, int FLUX>
static void launch_tet_eval(const cvw_mesh* m, const MethodScalars& ms, int mode, const float* u, const float* u0,
                            float* out, float* gamma, float* alpha, const float* cand, float* gbuf, uint32_t* status,
                            float dt, float a0, float b0, hipStream_t s) {
  const dim3 g(static_cast<unsigned>((m->E + TET_THREADS - 1) / TET_THREADS)), b(TET_THREADS);
  // the sensor pass writes gamma_e into the caller's array when there is one, else into the scratch
  float* gs = gamma ? gamma : gbuf;
  const bool plain = ms.sensor_kind != CVW_SENSOR_FIXED;
  if (plain)
    hipLaunchKernelGGL((tet_sensor_kernel<P>), g, b, 0, s, u, gs, cand, m->d_cell_vtx, m->d_geoth, m->d_tett, m->E, ms);
  float* gout = (plain && gamma) ? nullptr : gamma;
  hipLaunchKernelGGL((tet_eval_kernel<P, FLUX>), g, b, 0, s, u, u0, out, gout, alpha, gs, m->d_nbrt, m->d_geoth,
                     m->d_tett, m->E, ms, mode, dt, a0, b0, status);
}

cvw_status tet_eval(const cvw_mesh* m, const cvw_params* prm, int mode, const float* u, const float* u0, float* out,
                    float* gamma, float* alpha, const float* cand, float* gbuf, uint32_t* status, float dt, float a0,
                    float b0, hipStream_t s) {
  const MethodScalars ms = make_scalars(prm);
  const bool burgers = prm->flux == CVW_BURGERS;
  const bool euler = prm->flux == CVW_EULER;
  switch (m->degree) {
    case 1:
      if (burgers) launch_tet_eval<1, CVW_BURGERS>(m, ms, mode, u, u0, out, gamma, alpha, cand, gbuf, status, dt, a0, b0, s);
      else if (euler) launch_tet_eval<1, CVW_EULER>(m, ms, mode, u, u0, out, gamma, alpha, cand, gbuf, status, dt, a0, b0, s);
      else launch_tet_eval<1, CVW_ADVECT_CONST>(m, ms, mode, u, u0, out, gamma, alpha, cand, gbuf, status, dt, a0, b0, s);
      break;
    case 2:
      if (burgers) launch_tet_eval<2, CVW_BURGERS>(m, ms, mode, u, u0, out, gamma, alpha, cand, gbuf, status, dt, a0, b0, s);
      else if (euler) launch_tet_eval<2, CVW_EULER>(m, ms, mode, u, u0, out, gamma, alpha, cand, gbuf, status, dt, a0, b0, s);
      else launch_tet_eval<2, CVW_ADVECT_CONST>(m, ms, mode, u, u0, out, gamma, alpha, cand, gbuf, status, dt, a0, b0, s);
      break;
    default: set_error("tetrahedra: degree 1 or 2"); return CVW_EUNSUPPORTED;
  }
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

}  // namespace cvw
