// Time stepping for the CG paths (the DG paths update the state in their cell
// kernels).
//
// The stage needs L = -M^{-1} R with the consistent global mass matrix M (Sec.
// 2.1, eq. sdstab).
//
// Quadrilaterals: a preconditioned conjugate gradient iteration that stays on
// the device.  Its scalars live in a small device array or are formed by every
// block from the block partials, and once the preconditioned residual has dropped
// below the tolerance every later kernel of the launch sequence returns at once;
// the sequence is as long as the mesh's spectrum allows an iteration to last.  No
// host synchronisation, so a stage can be captured in a graph.  Preconditioner:
// the inverse row sums of M (the integrals of the nodal basis functions; positive
// for Gauss-Lobatto nodes).  Dot products are reduced in float64 in a fixed order
// (deterministic).
//
// Lines: a direct solve at low degree, the same iteration inside one workgroup
// per variable at high degree.
#include "cvw_device.h"
#include "cvw_pcg.h"

#include <algorithm>
#include <cmath>

namespace cvw {

constexpr int PCG_THREADS = 256;

__device__ __forceinline__ bool pcg_writer() { return blockIdx.x == 0 && threadIdx.x == 0; }

// sum of one double per thread over N threads in the order of a halving tree
// (s = N / 2, ..., 1: thread t adds t + s); the last six levels lie inside the
// first wave.  Result valid in every thread.
template <int N>
__device__ __forceinline__ double tree_sum(double v, double* sh) {
  __syncthreads();
  sh[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = N / 2; s > 64; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < 64) {
    v = sh[threadIdx.x] + sh[threadIdx.x + 64];
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s, 64);
    if (threadIdx.x == 0) sh[0] = v;
  }
  __syncthreads();
  return sh[0];
}
// sum of the nb block partials (fixed order)
__device__ __forceinline__ double partial_sum(const double* __restrict__ part, int nb, double* sh) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < nb; i += PCG_THREADS) acc += part[i];
  return tree_sum<PCG_THREADS>(acc, sh);
}

// ---------------------------------------------------------------------------
// Conjugate gradients on bilinear quadrilaterals.  The work is small (65 k cells,
// 262 k DOFs at 256 x 256 Q2: 20 MB and 20 MFLOP per iteration), the time is
// launches (3-4 us each on the host) and dependent reads.  So there are no launches
// for the direction and the scalars (every block sums the partials itself), and
// the sequence is as long as the mesh's spectrum allows an iteration to last (25
// instead of always 64).  An iteration is
//   cells:  beta from the partials of r.z; y_e = M_e p with the new direction
//           p = z + beta p formed at the cell's nodes on the way in;
//   gather: p at the DOF, Ap = sum of the y_e, partials of p.Ap;
//   update: alpha from those partials, x, r, z, partials of r.z;
// or, up to PCG_APPLY_PARTIALS partials, two launches:
//   apply:  cells and gather in one, every DOF evaluating its rows of its cells;
//   update.
// Apply has four times the vector memory instructions (12.7 us at 262 k DOFs against
// 4.4 + 3.3 us for cells and gather) and one launch less, which counts twice: the
// iterations after the last active one are launches alone (a step of nothing but
// those 690 us against 950).  A Q2 step, apply against cells + gather: 128^2 cells
// 753 and 755 us, 181^2 892 and 859, 222^2 1053 and 980, 300^2 1514 and 1274, 512^2
// 3959 and 2614; Q1 from 181^2 to 512^2 within 3 %.  The line is at 262,144 DOFs:
// there (256^2 Q2) steps one after another, which hide the launches, take 1002 us
// with apply and 964 without, a step that is waited for 1032 and 1120; above, the
// kernels decide, below, the launches.  Above PCG_FUSED_PARTIALS partials summing
// them in every block would cost more than a launch of its own.  Every sum keeps
// its order: all variants give the same bits.  A step (three stages) at 256 x 256
// Q2: 3371 us with six launches per iteration, 997 us now; at 31 x 27: 3591 us and
// 697 us; at 500 x 400: 3832 us and 2088 us.
// ---------------------------------------------------------------------------
constexpr int PCG_APPLY_PARTIALS = 1024, PCG_FUSED_PARTIALS = 4096;

// R_I = sum of the element rows sharing I (ascending (cell, node) order), r = R,
// z = D R; block partial of r . z
__global__ __launch_bounds__(PCG_THREADS) void pcg_init_kernel(const float* __restrict__ rcell,
                                                               const float* __restrict__ dinv, float* __restrict__ r,
                                                               float2* __restrict__ pz, double* __restrict__ part,
                                                               const int32_t* __restrict__ dptr,
                                                               const int32_t* __restrict__ dent, int64_t n,
                                                               double* __restrict__ S, double tol2) {
  __shared__ double sh[PCG_THREADS];
  const int64_t i = blockIdx.x * static_cast<int64_t>(PCG_THREADS) + threadIdx.x;
  if (pcg_writer()) pcg_setup(S, tol2);
  double d = 0.0;
  if (i < n) {
    float bi = 0.0f;
    for (int it = dptr[i]; it < dptr[i + 1]; ++it) bi += rcell[dent[it]];   // ent = cell * nloc + local node
    const float zi = dinv[i] * bi;
    r[i] = bi;
    pz[i] = make_float2(0.0f, zi);
    d = static_cast<double>(bi) * static_cast<double>(zi);
  }
  const double s = tree_sum<PCG_THREADS>(d, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// p = z + beta p (FIRST: p = z) at the cell's nodes and y = M_e p; the (p+1)^2 Gauss
// rule integrates phi_i phi_j |det J| exactly (degree 2p + 1 per direction).
// FUSED: this launch begins the iteration (r.z from its partials).
template <int P, bool FIRST, bool FUSED>
__global__ __launch_bounds__(PCG_THREADS) void pcg_cells_kernel(const float2* __restrict__ pz, float* __restrict__ ycell,
                                                                const double* __restrict__ rz_part, int nb,
                                                                const int32_t* __restrict__ cdof,
                                                                const float* __restrict__ geo,
                                                                const CGTables* __restrict__ tab, int64_t E, double* S,
                                                                int it) {
  constexpr int N1 = P + 1, NLOC = N1 * N1;
  __shared__ double sh[PCG_THREADS];
  if (FUSED ? !pcg_enter(S, it, pcg_writer()) : !pcg_runs(S, it)) return;
  const int64_t e = blockIdx.x * static_cast<int64_t>(PCG_THREADS) + threadIdx.x, ec = e < E ? e : E - 1;
  int I[NLOC];
  float2 v[NLOC];
#pragma unroll
  for (int j = 0; j < NLOC; ++j) I[j] = cdof[j * E + ec];
#pragma unroll
  for (int j = 0; j < NLOC; ++j) v[j] = pz[I[j]];
  const Geo G = load_geo(geo, ec);
  float beta = 0.0f;
  if constexpr (FUSED) {
    const double rz = partial_sum(rz_part, nb, sh);
    if (!pcg_begin<FIRST>(rz, S, it, pcg_writer(), beta)) return;
  } else if constexpr (!FIRST) {
    beta = static_cast<float>(S[S_BETA]);
  }
  if (e >= E) return;
  float xe[NLOC], y[NLOC];
#pragma unroll
  for (int j = 0; j < NLOC; ++j) {
    xe[j] = FIRST ? v[j].y : fmaf(beta, v[j].x, v[j].y);
    y[j] = 0.0f;
  }
#pragma unroll
  for (int qy = 0; qy < N1; ++qy)
#pragma unroll
    for (int qx = 0; qx < N1; ++qx) {
      float px, py, J[2][2];
      geo_eval(G, tab->xv[qx], tab->xv[qy], px, py, J);
      const float W = tab->wv[qx] * tab->wv[qy] * fabsf(J[0][0] * J[1][1] - J[0][1] * J[1][0]);
      float xq = 0.0f;
#pragma unroll
      for (int b = 0; b < N1; ++b)
#pragma unroll
        for (int a = 0; a < N1; ++a) xq = fmaf(tab->Dv[0][qx][a] * tab->Dv[0][qy][b], xe[a + N1 * b], xq);
      const float Wx = W * xq;
#pragma unroll
      for (int b = 0; b < N1; ++b)
#pragma unroll
        for (int a = 0; a < N1; ++a) y[a + N1 * b] = fmaf(tab->Dv[0][qx][a] * tab->Dv[0][qy][b], Wx, y[a + N1 * b]);
    }
#pragma unroll
  for (int j = 0; j < NLOC; ++j) ycell[j * E + e] = y[j];
}

// p = z + beta p (FIRST: p = z), Ap_I = sum of the element entries sharing I
// (ascending (cell, node) order); block partial of p . Ap
template <int NLOC, bool FIRST>
__global__ __launch_bounds__(PCG_THREADS) void pcg_gather_kernel(const float* __restrict__ ycell, float2* __restrict__ pz,
                                                                 float* __restrict__ Ap, double* __restrict__ part,
                                                                 const int4* __restrict__ ent4,
                                                                 const int32_t* __restrict__ dptr,
                                                                 const int32_t* __restrict__ dent, int64_t E, int64_t n,
                                                                 const double* __restrict__ S, int it) {
  __shared__ double sh[PCG_THREADS];
  if (!pcg_runs(S, it)) return;
  const int64_t I = blockIdx.x * static_cast<int64_t>(PCG_THREADS) + threadIdx.x;
  double d = 0.0;
  if (I < n) {
    const int4 k = ent4[I];
    const float2 o = pz[I];
    const float y0 = ycell[k.x < 0 ? 0 : k.x], y1 = ycell[k.y < 0 ? 0 : k.y], y2 = ycell[k.z < 0 ? 0 : k.z],
                y3 = ycell[k.w < 0 ? 0 : k.w];
    float s = 0.0f;
    if (k.x == -2) {
      for (int c = dptr[I]; c < dptr[I + 1]; ++c) {
        const int64_t e = dent[c] / NLOC;
        s += ycell[(dent[c] - e * NLOC) * E + e];
      }
    } else {
      s += y0;
      if (k.y >= 0) s += y1;
      if (k.z >= 0) s += y2;
      if (k.w >= 0) s += y3;
    }
    const float p = FIRST ? o.y : fmaf(static_cast<float>(S[S_BETA]), o.x, o.y);
    pz[I].x = p;
    Ap[I] = s;
    d = static_cast<double>(p) * static_cast<double>(s);
  }
  const double b = tree_sum<PCG_THREADS>(d, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

// W[e][q] = w_q |det J| of the volume rule, for the apply kernel
template <int P>
__global__ __launch_bounds__(256) void cgq_mass_weights_kernel(float* __restrict__ W, const float* __restrict__ geo,
                                                               const CGTables* __restrict__ tab, int64_t E) {
  constexpr int N1 = P + 1, NLOC = N1 * N1;
  const int64_t e = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (e >= E) return;
  const Geo G = load_geo(geo, e);
#pragma unroll
  for (int qy = 0; qy < N1; ++qy)
#pragma unroll
    for (int qx = 0; qx < N1; ++qx) {
      float px, py, J[2][2];
      geo_eval(G, tab->xv[qx], tab->xv[qy], px, py, J);
      W[e * NLOC + qx + N1 * qy] = tab->wv[qx] * tab->wv[qy] * fabsf(J[0][0] * J[1][1] - J[0][1] * J[1][0]);
    }
}

// basis products phi_j(x_q) of the tensor rule, [q][j] (kernel argument: read
// through the scalar unit)
template <int NLOC>
struct MassBasis {
  float phi[NLOC][NLOC];
};

// cells and gather in one (begins the iteration): Ap_I = sum over
// the cells sharing I of the row sum_q phi_I(x_q) W_q p_h(x_q); the directions
// alternate between pz and pz_new, as other DOFs still read the old one
template <int P, bool FIRST>
__global__ __launch_bounds__(PCG_THREADS) void pcg_apply_kernel(
    const float2* __restrict__ pz, float2* __restrict__ pz_new, float* __restrict__ Ap,
    const double* __restrict__ rz_part, double* __restrict__ pap_part, int nb, const float* __restrict__ W,
    const int32_t* __restrict__ cdof, const int32_t* __restrict__ dptr, const int32_t* __restrict__ dent,
    MassBasis<(P + 1) * (P + 1)> B, int64_t n, double* S, int it) {
  constexpr int NLOC = (P + 1) * (P + 1);
  __shared__ double sh[PCG_THREADS];
  __shared__ float sphi[NLOC][NLOC];      // [j][q]
  if (!pcg_enter(S, it, pcg_writer())) return;
  const double rz = partial_sum(rz_part, nb, sh);
  float beta;
  if (!pcg_begin<FIRST>(rz, S, it, pcg_writer(), beta)) return;
  if (threadIdx.x < NLOC * NLOC) sphi[threadIdx.x % NLOC][threadIdx.x / NLOC] = (&B.phi[0][0])[threadIdx.x];
  __syncthreads();
  const int64_t I = blockIdx.x * static_cast<int64_t>(PCG_THREADS) + threadIdx.x;
  double d = 0.0;
  if (I < n) {
    float s = 0.0f;
    const int beg = dptr[I], end = dptr[I + 1];
    for (int k = beg; k < end; ++k) {
      const int ent = dent[k];
      const int64_t e = ent / NLOC;
      const int i = ent - static_cast<int>(e) * NLOC;
      float xe[NLOC], Wq[NLOC];
#pragma unroll
      for (int j = 0; j < NLOC; ++j) {
        const float2 v = pz[cdof[e * NLOC + j]];
        xe[j] = FIRST ? v.y : fmaf(beta, v.x, v.y);
        Wq[j] = W[e * NLOC + j];
      }
      float y = 0.0f;
#pragma unroll
      for (int q = 0; q < NLOC; ++q) {
        float xq = 0.0f;
#pragma unroll
        for (int j = 0; j < NLOC; ++j) xq = fmaf(B.phi[q][j], xe[j], xq);
        const float Wx = Wq[q] * xq;
        y = fmaf(sphi[i][q], Wx, y);
      }
      s += y;
    }
    const float2 o = pz[I];
    const float p = FIRST ? o.y : fmaf(beta, o.x, o.y);
    pz_new[I].x = p;
    Ap[I] = s;
    d = static_cast<double>(p) * static_cast<double>(s);
  }
  const double b = tree_sum<PCG_THREADS>(d, sh);
  if (threadIdx.x == 0) pap_part[blockIdx.x] = b;
}

// x += alpha p (FIRST: x = alpha p), r -= alpha Ap, z = D r; block partial of r . z
template <bool FIRST, bool FUSED>
__global__ __launch_bounds__(PCG_THREADS) void pcg_update_kernel(float* __restrict__ x, float* __restrict__ r,
                                                                 float2* __restrict__ pz, const float* __restrict__ Ap,
                                                                 const float* __restrict__ dinv,
                                                                 const double* __restrict__ pap_part,
                                                                 double* __restrict__ rz_part, int nb, int64_t n,
                                                                 const double* __restrict__ S, int it) {
  __shared__ double sh[PCG_THREADS];
  if (!pcg_runs(S, it)) return;
  const int64_t i = blockIdx.x * static_cast<int64_t>(PCG_THREADS) + threadIdx.x, ic = i < n ? i : n - 1;
  const float p = pz[ic].x, xo = FIRST ? 0.0f : x[ic], ro = r[ic], ap = Ap[ic], di = dinv[ic];
  float al;
  if constexpr (FUSED) al = static_cast<float>(S[pcg_rz_word(it)] / partial_sum(pap_part, nb, sh));
  else al = static_cast<float>(S[S_ALPHA]);
  double d = 0.0;
  if (i < n) {
    x[i] = fmaf(al, p, xo);
    const float ri = fmaf(-al, ap, ro);
    const float zi = di * ri;
    r[i] = ri;
    pz[i].y = zi;
    d = static_cast<double>(ri) * static_cast<double>(zi);
  }
  const double s = tree_sum<PCG_THREADS>(d, sh);
  if (threadIdx.x == 0) rz_part[blockIdx.x] = s;
}

// Large meshes, one block: the beginning of iteration `it` (which its other
// launches then only read), or its alpha = rz / (p . Ap), from the block partials.
enum { SCALAR_BEGIN, SCALAR_ALPHA };
__global__ __launch_bounds__(PCG_THREADS) void pcg_scalar_kernel(const double* __restrict__ part, int nb,
                                                                 double* __restrict__ S, int op, int it) {
  __shared__ double sh[PCG_THREADS];
  if (op == SCALAR_BEGIN ? !pcg_enter(S, it, pcg_writer()) : !pcg_runs(S, it)) return;
  const double v = partial_sum(part, nb, sh);
  float beta;
  if (op == SCALAR_ALPHA) {
    if (pcg_writer()) S[S_ALPHA] = S[pcg_rz_word(it)] / v;
  } else if (it == 0) {
    pcg_begin<true>(v, S, it, pcg_writer(), beta);
  } else {
    pcg_begin<false>(v, S, it, pcg_writer(), beta);
  }
}

// u_out = a0 u_n + b0 (u_s - dt x) (no iteration: x = 0).  A solve that has not met
// its tolerance (nor broken down) when the launch sequence ends sets
// ST_PCG_STALL in the workspace status word.  it: the last iteration begun; part:
// the partials of r.z after it (null: a scalar launch has begun it, so they are
// judged).
__global__ __launch_bounds__(PCG_THREADS) void pcg_finish_kernel(const float* __restrict__ us,
                                                                 const float* __restrict__ un,
                                                                 const float* __restrict__ x, float* __restrict__ uo,
                                                                 float a0, float b0, float dt, int64_t n,
                                                                 const double* __restrict__ S, int it,
                                                                 const double* __restrict__ part, int nb,
                                                                 uint32_t* __restrict__ status) {
  __shared__ double sh[PCG_THREADS];
  if (blockIdx.x == 0 && pcg_runs(S, it)) {
    const bool ok = part && !(partial_sum(part, nb, sh) > S[S_TOL2] * S[S_RZ0]);
    if (threadIdx.x == 0 && !ok) atomicOr(status, ST_PCG_STALL);
  }
  const int64_t i = blockIdx.x * static_cast<int64_t>(PCG_THREADS) + threadIdx.x;
  if (i >= n) return;
  const float xi = S[pcg_state_word(it)] == PCG_NO_RHS ? 0.0f : x[i];
  const float base = (a0 != 0.0f) ? a0 * un[i] : 0.0f;
  uo[i] = base + b0 * (us[i] - dt * xi);
}

// u_out = a0 u_n + b0 (u_s - dt x), x = M^{-1} R; a0 = 0: u_n is not read
template <typename Real>
__global__ __launch_bounds__(256) void stage_update_kernel(const Real* __restrict__ us, const Real* __restrict__ un,
                                                           const Real* __restrict__ x, Real* __restrict__ uo, Real a0,
                                                           Real b0, Real dt, int64_t n) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i >= n) return;
  const Real base = (a0 != Real(0)) ? a0 * un[i] : Real(0);
  uo[i] = base + b0 * (us[i] - dt * x[i]);
}

// The whole PCG solve of a line (segments) in one workgroup per variable
// (workgroup v: variable v; every vector is [n_var][ndof]): the same
// iteration, tolerance and cap as the launch sequence above, with the phases
// separated by workgroup barriers instead of kernel launches (a 1D mesh has
// at most a few thousand DOFs, where the launch sequence costs ~3 us per
// launch and the arithmetic well under that).  The element mass is
// (h_e / 2) M_ref with M_ref = sum_q w_q l_i(x_q) l_j(x_q), formed in LDS from
// the tables of any degree.  Dot products: per-thread partials in a fixed
// stride order, then a fixed tree.
constexpr int SMALL_THREADS = 1024;

__device__ __forceinline__ double wg_sum(double v, double* sh) {
  __syncthreads();
  sh[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = SMALL_THREADS / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  return sh[0];
}

template <typename Real>
__global__ __launch_bounds__(SMALL_THREADS) void pcg_line_kernel(
    const Real* __restrict__ b, Real* __restrict__ x, Real* __restrict__ r, Real* __restrict__ z,
    Real* __restrict__ p, Real* __restrict__ Ap, Real* __restrict__ ycell, const Real* __restrict__ dinv,
    const double* __restrict__ tab, const double* __restrict__ hcell, const int32_t* __restrict__ cdof,
    const int32_t* __restrict__ dptr, const int32_t* __restrict__ dent, int deg, int64_t E, int64_t n, double tol2,
    int maxit, uint32_t* __restrict__ status) {
  __shared__ double sh[SMALL_THREADS];
  __shared__ double Mref[(HP_MAXP + 1) * (HP_MAXP + 1)];
  const int tid = threadIdx.x;
  {
    const int64_t off = static_cast<int64_t>(blockIdx.x) * n;   // this workgroup's variable
    b += off; x += off; r += off; z += off; p += off; Ap += off;
    ycell += static_cast<int64_t>(blockIdx.x) * E * (deg + 1);
  }
  const int n1 = deg + 1;
  const HPOff o = hp_off(deg);
  for (int w = tid; w < n1 * n1; w += SMALL_THREADS) {
    const int i = w / n1, j = w - i * n1;
    double s = 0.0;
    for (int q = 0; q < n1; ++q) s += tab[o.wq + q] * tab[o.DQ + i * n1 + q] * tab[o.DQ + j * n1 + q];
    Mref[w] = s;
  }
  double d = 0.0;
  for (int64_t i = tid; i < n; i += SMALL_THREADS) {
    const Real bi = b[i];
    const Real zi = dinv[i] * bi;
    x[i] = Real(0);
    r[i] = bi;
    z[i] = zi;
    p[i] = zi;
    d += static_cast<double>(bi) * static_cast<double>(zi);
  }
  double rz = wg_sum(d, sh);
  const double rz0 = rz;
  bool done = !(rz > 0.0);
  for (int it = 0; it < maxit && !done; ++it) {
    for (int64_t w = tid; w < E * n1; w += SMALL_THREADS) {
      const int64_t e = w / n1;
      const int i = static_cast<int>(w - e * n1);
      double y = 0.0;
      for (int j = 0; j < n1; ++j) y += Mref[i * n1 + j] * static_cast<double>(p[cdof[e * n1 + j]]);
      ycell[w] = static_cast<Real>(0.5 * hcell[e] * y);
    }
    __syncthreads();
    d = 0.0;
    for (int64_t I = tid; I < n; I += SMALL_THREADS) {
      Real s = Real(0);
      for (int k = dptr[I]; k < dptr[I + 1]; ++k) s += ycell[dent[k]];
      Ap[I] = s;
      d += static_cast<double>(p[I]) * static_cast<double>(s);
    }
    const double al = rz / wg_sum(d, sh);
    d = 0.0;
    for (int64_t i = tid; i < n; i += SMALL_THREADS) {
      x[i] = fma(static_cast<Real>(al), p[i], x[i]);
      const Real ri = fma(static_cast<Real>(-al), Ap[i], r[i]);
      const Real zi = dinv[i] * ri;
      r[i] = ri;
      z[i] = zi;
      d += static_cast<double>(ri) * static_cast<double>(zi);
    }
    const double rzn = wg_sum(d, sh);
    const double be = rzn / rz;
    rz = rzn;
    if (!(rzn > tol2 * rz0)) { done = true; break; }
    for (int64_t i = tid; i < n; i += SMALL_THREADS) p[i] = fma(static_cast<Real>(be), p[i], z[i]);
    __syncthreads();
  }
  if (tid == 0 && !done) atomicOr(status, ST_PCG_STALL);
}

// ---------------------------------------------------------------------------
// Direct solve on lines (tables: line_mass_operator on the host).  A block takes
// `own` consecutive vertices of the chain with 2^levels - 1 more on either side,
// which is as far as `levels` steps of cyclic reduction reach: blocks need nothing
// from each other and the whole solve with the stage update is one launch.
// Float64 throughout.  A NaN in a variable's assembled right-hand side leaves its
// x = 0, an infinity makes it NaN everywhere, as in the conjugate gradient
// iteration.  A single block sees every entry; several take the cell kernel's
// word on the element rows (rows), and where those hold infinities look for
// vertices at which two of them meet to a NaN.
// 128 cells, P2: 4.0 us against 65.3 us for the conjugate gradients (and their
// assembly and update launches); a step of P1 advection on 1500 cells 37.8 against
// 563 us, of P4 Euler on 1000 cells 90.6 against 867 us.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t row_bits(double v) {
  return isfinite(v) ? 0u : (isnan(v) ? CG_ROWS_NAN : CG_ROWS_INF);
}
__global__ void line_clear_rows_kernel(uint32_t* status) {
  if (threadIdx.x < 3) status[WS_CG_ROWS + threadIdx.x] = 0;
}

template <typename Real, int T>
__global__ __launch_bounds__(T) void line_mass_kernel(
    const Real* __restrict__ rcell, const Real* __restrict__ us, const Real* __restrict__ un, Real* __restrict__ uo,
    const double* __restrict__ red, const double* __restrict__ tab, const double* __restrict__ hcell,
    const int32_t* __restrict__ chain, const int32_t* __restrict__ cdof, int deg, int64_t E, int64_t nv, int64_t ndof,
    int loop, int levels, int own, const uint32_t* __restrict__ rows, Real a0, Real b0, Real dt) {
  constexpr int ML = 7;
  __shared__ double sh[2][T];
  const int t = threadIdx.x, n1 = deg + 1, ni = deg - 1, H = (1 << levels) - 1;
  const int64_t k0 = static_cast<int64_t>(blockIdx.x) * own;
  const int64_t off = blockIdx.y * ndof;
  rcell += blockIdx.y * E * n1;
  us += off;
  un += off;
  uo += off;
  int64_t k = k0 - H + t;
  if (loop) k = ((k % nv) + nv) % nv;
  const bool in = k >= 0 && k < nv;
  uint32_t fl = gridDim.x > 1 ? rows[blockIdx.y] : 0;
  if (fl == CG_ROWS_INF) {                // the same in every block and thread
    for (int64_t v = t; v < nv; v += T) {
      const int64_t l = v > 0 ? v - 1 : (loop ? nv - 1 : -1);
      Real b = Real(0);
      if (v < E) b += rcell[static_cast<int64_t>(chain[v]) * n1];
      if (l >= 0) b += rcell[static_cast<int64_t>(chain[l]) * n1 + deg];
      if (isnan(b)) fl |= CG_ROWS_NAN;
    }
  }
  double al[ML], ga[ML], g = 0.0, ib = 0.0;
#pragma unroll
  for (int l = 0; l < ML; ++l) {
    al[l] = ga[l] = 0.0;
    if (in && l < levels) {
      al[l] = red[(2 * l) * nv + k];
      ga[l] = red[(2 * l + 1) * nv + k];
    }
  }
  if (in) {
    ib = red[2 * levels * nv + k];
    const int64_t kl = k > 0 ? k - 1 : (loop ? nv - 1 : -1);
    Real b = Real(0);                     // the vertex's assembled entry
    if (k < E) {                          // the cell on the right: its node 0
      const Real* r = rcell + static_cast<int64_t>(chain[k]) * n1;
      double s = r[0];
      b += r[0];
      for (int i = 0; i < ni; ++i) {
        const double v = r[i + 1];
        fl |= row_bits(v);
        s -= tab[i] * v;
      }
      g += s;
    }
    if (kl >= 0) {                        // the cell on the left: its node p
      const Real* r = rcell + static_cast<int64_t>(chain[kl]) * n1;
      double s = r[deg];
      b += r[deg];
      for (int i = 0; i < ni; ++i) s -= tab[ni + i] * static_cast<double>(r[i + 1]);
      g += s;
    }
    fl |= row_bits(b);
  }
  sh[0][t] = g;
  fl = (__syncthreads_or(fl & CG_ROWS_NAN) ? CG_ROWS_NAN : 0) | (__syncthreads_or(fl & CG_ROWS_INF) ? CG_ROWS_INF : 0);
  int cur = 0;
#pragma unroll
  for (int l = 0; l < ML; ++l) {
    if (l >= levels) break;
    const int s = 1 << l;
    const double lo = t >= s ? sh[cur][t - s] : 0.0, hi = t + s < T ? sh[cur][t + s] : 0.0;
    g = fma(al[l], lo, fma(ga[l], hi, g));
    sh[cur ^ 1][t] = g;
    cur ^= 1;
    __syncthreads();
  }
  double xv = g * ib;
  if (fl) xv = (fl & CG_ROWS_NAN) ? 0.0 : __builtin_nan("");
  sh[cur ^ 1][t] = xv;
  __syncthreads();
  const double* xs = sh[cur ^ 1] + H;     // vertex k0 + j at xs[j]
  auto update = [&](int64_t I, double x) {
    const Real base = (a0 != Real(0)) ? a0 * un[I] : Real(0);
    uo[I] = base + b0 * (us[I] - dt * static_cast<Real>(x));
  };
  const int64_t nown = nv - k0 < own ? nv - k0 : own;
  for (int j = t; j < nown; j += T) {
    const int64_t kk = k0 + j;
    update(kk < E ? cdof[static_cast<int64_t>(chain[kk]) * n1] : cdof[static_cast<int64_t>(chain[E - 1]) * n1 + deg],
           xs[j]);
  }
  const int64_t ncell = E - k0 < own ? E - k0 : own;
  for (int w = t; w < ncell * ni; w += T) {
    const int j = w / ni, i = w - j * ni;
    const int64_t e = chain[k0 + j];
    const Real* r = rcell + e * n1 + 1;
    const double* Mi = tab + 2 * ni + i * ni;
    double s = 0.0;
    for (int q = 0; q < ni; ++q) s = fma(Mi[q], static_cast<double>(r[q]), s);
    double x = s * (2.0 / hcell[e]) - tab[i] * xs[j] - tab[ni + i] * xs[j + 1];
    if (fl) x = (fl & CG_ROWS_NAN) ? 0.0 : __builtin_nan("");
    update(cdof[e * n1 + i + 1], x);
  }
}

static unsigned nbk(int64_t n, int t) { return static_cast<unsigned>((n + t - 1) / t); }

size_t pcg_partials(int64_t n) { return nbk(n, PCG_THREADS); }

template <typename Real>
cvw_status line_pcg(const cvw_mesh* m, const Real* b, Real* x, Real* r, Real* z, Real* p, Real* Ap, Real* ycell,
                    const Real* dinv, double tol, int maxit, uint32_t* status, hipStream_t s, int nvar) {
  hipLaunchKernelGGL((pcg_line_kernel<Real>), dim3(nvar), dim3(SMALL_THREADS), 0, s, b, x, r, z, p, Ap, ycell, dinv,
                     m->d_hp, m->d_hcell, m->d_cell_dof, m->d_dof_ptr, m->d_dof_ent, m->degree, m->E, m->ndof,
                     tol * tol, maxit, status);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

// Iterations after which conjugate gradients must have met the tolerance: in
// the energy norm they reduce the error by 2 ((sqrt(c) - 1) / (sqrt(c) + 1))^k, and
// the preconditioned residual norm differs from it by a factor sqrt(c) at most
// (c: the condition number); a tenth and two more for rounding.  In float32, over
// jitters to 0.45, aspects to 1000 and rough right-hand sides, 11 to 23 were needed
// of 30 and more (Q1), 15 to 19 of 25 and more (Q2).
static int pcg_iterations(double cond, double tol, int maxit) {
  if (!(cond > 1.0)) return maxit;
  const double q = std::sqrt(cond), k = std::log(2.0 * q / tol) / std::log((q + 1.0) / (q - 1.0));
  return std::min(maxit, static_cast<int>(std::ceil(1.1 * k)) + 2);
}

template <int P>
static cvw_status quad_pcg(const cvw_mesh* m, const float* rcell, const QuadSolve& q, double tol, int maxit,
                           const float* us, const float* un, float* uo, double a0, double b0, double dt,
                           uint32_t* status, hipStream_t s) {
  constexpr int N1 = P + 1, NLOC = N1 * N1;
  const int64_t n = m->ndof;
  const int nb = static_cast<int>(nbk(n, PCG_THREADS));
  const bool fused = nb <= PCG_FUSED_PARTIALS && static_cast<size_t>(nb) <= q.part_cap;
  double* rz = q.part[0];
  double* pap = fused ? q.part[1] : q.part[0];
  const dim3 g(nb), t(PCG_THREADS);
  hipLaunchKernelGGL(pcg_init_kernel, g, t, 0, s, rcell, m->d_dinv_f, q.r, q.pz, rz, m->d_dof_ptr, m->d_dof_ent, n,
                     q.S, tol * tol);
  if (!fused) hipLaunchKernelGGL(pcg_scalar_kernel, dim3(1), t, 0, s, rz, nb, q.S, SCALAR_BEGIN, 0);
  const int iters = pcg_iterations(m->mass_cond, tol, maxit);
  const bool one = fused && nb <= PCG_APPLY_PARTIALS;
  MassBasis<NLOC> B;
  if (one) {
    for (int k = 0; k < NLOC; ++k)
      for (int j = 0; j < NLOC; ++j) B.phi[k][j] = m->cgt.Dv[0][k % N1][j % N1] * m->cgt.Dv[0][k / N1][j / N1];
    hipLaunchKernelGGL(cgq_mass_weights_kernel<P>, dim3(nbk(m->E, 256)), dim3(256), 0, s, q.y, m->d_geo, m->d_cgt,
                       m->E);
  }
  float* x = one ? q.x2 : q.x;
  for (int it = 0; it < iters; ++it) {
    float2* pz = one && !(it & 1) ? q.pz2 : q.pz;        // holds p and, after the update, z
    auto update = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, g, t, 0, s, x, q.r, pz, q.Ap, m->d_dinv_f, pap, rz, nb, n, q.S, it);
    };
    if (one) {
      auto apply = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, t, 0, s, (it & 1) ? q.pz2 : q.pz, pz, q.Ap, rz, pap, nb, q.y, m->d_cell_dof,
                           m->d_dof_ptr, m->d_dof_ent, B, n, q.S, it);
      };
      if (it == 0) apply(pcg_apply_kernel<P, true>); else apply(pcg_apply_kernel<P, false>);
      if (it == 0) update(pcg_update_kernel<true, true>); else update(pcg_update_kernel<false, true>);
      continue;
    }
    auto cells = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(nbk(m->E, PCG_THREADS)), t, 0, s, q.pz, q.y, rz, nb, m->d_cell_dof_t, m->d_geo,
                         m->d_cgt, m->E, q.S, it);
    };
    auto gather = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, g, t, 0, s, q.y, q.pz, q.Ap, pap, m->d_dof_ent4, m->d_dof_ptr, m->d_dof_ent, m->E, n,
                         q.S, it);
    };
    if (fused) {
      if (it == 0) cells(pcg_cells_kernel<P, true, true>); else cells(pcg_cells_kernel<P, false, true>);
    } else {
      if (it == 0) cells(pcg_cells_kernel<P, true, false>); else cells(pcg_cells_kernel<P, false, false>);
    }
    if (it == 0) gather(pcg_gather_kernel<NLOC, true>); else gather(pcg_gather_kernel<NLOC, false>);
    if (fused) {
      if (it == 0) update(pcg_update_kernel<true, true>); else update(pcg_update_kernel<false, true>);
    } else {
      hipLaunchKernelGGL(pcg_scalar_kernel, dim3(1), t, 0, s, pap, nb, q.S, SCALAR_ALPHA, it);
      if (it == 0) update(pcg_update_kernel<true, false>); else update(pcg_update_kernel<false, false>);
      hipLaunchKernelGGL(pcg_scalar_kernel, dim3(1), t, 0, s, rz, nb, q.S, SCALAR_BEGIN, it + 1);
    }
  }
  hipLaunchKernelGGL(pcg_finish_kernel, g, t, 0, s, us, un, x, uo, static_cast<float>(a0), static_cast<float>(b0),
                     static_cast<float>(dt), n, q.S, fused ? iters - 1 : iters, fused ? rz : nullptr, nb,
                     status);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

cvw_status cgquad_mass_stage(const cvw_mesh* m, const float* rcell, const QuadSolve& q, double tol, int maxit,
                             const float* us, const float* un, float* uo, double a0, double b0, double dt,
                             uint32_t* status, hipStream_t s) {
  return m->degree == 1 ? quad_pcg<1>(m, rcell, q, tol, maxit, us, un, uo, a0, b0, dt, status, s)
                        : quad_pcg<2>(m, rcell, q, tol, maxit, us, un, uo, a0, b0, dt, status, s);
}

template <typename Real>
cvw_status stage_update(const Real* us, const Real* un, const Real* x, Real* uo, double a0, double b0, double dt,
                        int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((stage_update_kernel<Real>), dim3(nbk(n, 256)), dim3(256), 0, s, us, un, x, uo,
                     static_cast<Real>(a0), static_cast<Real>(b0), static_cast<Real>(dt), n);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

// Threads per block of the direct line solve: they cover the block's vertices,
// the reach of the reduction on both sides and the right vertex of its last
// cell.  The smallest block that holds the whole chain (one block needs no
// clearing launch), else many small ones (512 threads at seven levels, whose
// reach is 127).
static int line_own(const cvw_mesh* m, int T) { return T - 2 * ((1 << m->line_levels) - 1) - 1; }
static int line_threads(const cvw_mesh* m) {
  for (int T = 256; T <= 1024; T *= 2)
    if (line_own(m, T) >= m->chain_nv) return T;
  return m->line_levels <= 6 ? 256 : 512;
}

cvw_status line_clear_rows(const cvw_mesh* m, uint32_t* status, hipStream_t s) {
  if (line_own(m, line_threads(m)) >= m->chain_nv) return CVW_OK;
  hipLaunchKernelGGL(line_clear_rows_kernel, dim3(1), dim3(64), 0, s, status);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

template <typename Real>
cvw_status line_mass_stage(const cvw_mesh* m, int nvar, const Real* rcell, const Real* us, const Real* un, Real* uo,
                           double a0, double b0, double dt, const uint32_t* rows_flag, hipStream_t s) {
  const int T = line_threads(m), own = line_own(m, T);
  const dim3 g(nbk(m->chain_nv, own), nvar);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, g, dim3(T), 0, s, rcell, us, un, uo, m->d_line_red, m->d_line_int, m->d_hcell,
                       m->d_chain, m->d_cell_dof, m->degree, m->E, m->chain_nv, m->ndof, m->chain_loop,
                       m->line_levels, own, rows_flag, static_cast<Real>(a0), static_cast<Real>(b0),
                       static_cast<Real>(dt));
  };
  if (T == 256) launch(line_mass_kernel<Real, 256>);
  else if (T == 512) launch(line_mass_kernel<Real, 512>);
  else launch(line_mass_kernel<Real, 1024>);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

template cvw_status line_mass_stage<float>(const cvw_mesh*, int, const float*, const float*, const float*, float*,
                                           double, double, double, const uint32_t*, hipStream_t);
template cvw_status line_mass_stage<double>(const cvw_mesh*, int, const double*, const double*, const double*,
                                            double*, double, double, double, const uint32_t*, hipStream_t);
template cvw_status line_pcg<float>(const cvw_mesh*, const float*, float*, float*, float*, float*, float*, float*,
                                    const float*, double, int, uint32_t*, hipStream_t, int);
template cvw_status line_pcg<double>(const cvw_mesh*, const double*, double*, double*, double*, double*, double*,
                                     double*, const double*, double, int, uint32_t*, hipStream_t, int);
template cvw_status stage_update<float>(const float*, const float*, const float*, float*, double, double, double,
                                        int64_t, hipStream_t);
template cvw_status stage_update<double>(const double*, const double*, const double*, double*, double, double, double,
                                         int64_t, hipStream_t);

}  // namespace cvw
