// Learned smoothness sensor: a 48 -> 64 -> 64 -> 1 network (GELU, sigmoid
// output) that predicts gamma_e from the cell features (see dgq_feat_kernel),
// on bfloat16 matrix cores (v_mfma_f32_32x32x16_bf16, float32 accumulation).
//
// Products are formed transposed, Z^T = W^T X^T, so that a wave's 32x32 tile
// holds one cell (or training sample) per lane column: lane l holds column
// l % 32 and, in accumulator v, row 8 (v / 4) + 4 (l / 32) + v % 4.  The
// second layer takes its B operand straight from the first layer's
// accumulators: the reduction index k of operand element i of lane group
// g = l / 32 is chosen as the row that group already holds (any k order
// gives the same sum, as long as A and B agree), so the A operand (W2^T)
// is read in two 4-element chunks.  No LDS round trip between the layers.
//
// Inference rounds inputs, weights and both hidden activations to bfloat16.
// Training keeps activations and back-propagated errors near float32 by
// splitting them into two bfloat16 terms (x = hi + lo, hi = bf16(x),
// lo = bf16(x - hi)) and summing the partial products on the matrix cores;
// weights and inputs are exact bfloat16 values.
#include "cvw_device.h"

namespace cvw {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {    // 16-byte aligned
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ bf16x8 load4x2(const uint16_t* p0, const uint16_t* p1) {   // 8-byte aligned chunks
  const u32x2 a = *reinterpret_cast<const u32x2*>(p0), b = *reinterpret_cast<const u32x2*>(p1);
  u32x4 w;
  w[0] = a[0];
  w[1] = a[1];
  w[2] = b[0];
  w[3] = b[1];
  return __builtin_bit_cast(bf16x8, w);
}
__device__ __forceinline__ bf16x8 pack8(const uint16_t* h) {
  u32x4 w;
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = static_cast<uint32_t>(h[2 * q]) | (static_cast<uint32_t>(h[2 * q + 1]) << 16);
  return __builtin_bit_cast(bf16x8, w);
}
__device__ __forceinline__ bf16x8 zero8() {
  u32x4 w = {0u, 0u, 0u, 0u};
  return __builtin_bit_cast(bf16x8, w);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 c;
#pragma unroll
  for (int v = 0; v < 16; ++v) c[v] = 0.0f;
  return c;
}
__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// row of accumulator v for lane group g within a 32-row tile
__device__ __forceinline__ int acc_row(int v, int g) { return 8 * (v >> 2) + 4 * g + (v & 3); }

// erf(z) by the rational-exponential approximation of Abramowitz and Stegun,
// formula 7.1.26 (after Hastings): erf(z) = 1 - t (a1 + a2 t + ... + a5 t^4)
// exp(-z^2), t = 1 / (1 + p z), z >= 0, |error| <= 1.5e-7 (far below the
// bfloat16 rounding of the activations).  Also returns exp(-z^2).
__device__ __forceinline__ float erf_as(float z, float& ez) {
  const float az = fabsf(z);
  const float t = frcp(fmaf(0.3275911f, az, 1.0f));
  float q = fmaf(1.061405429f, t, -1.453152027f);
  q = fmaf(q, t, 1.421413741f);
  q = fmaf(q, t, -0.284496736f);
  q = fmaf(q, t, 0.254829592f);
  ez = __builtin_amdgcn_exp2f(-1.44269504088896341f * az * az);      // exp(-z^2) = 2^(-z^2 log2 e)
  const float y = fmaf(-q * t, ez, 1.0f);
  return z < 0.0f ? -y : y;
}
__device__ __forceinline__ float gelu(float x) {
  float e;
  return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752f, e));
}
__device__ __forceinline__ float gelu_prime(float x) {
  float e;                                                            // e = exp(-x^2 / 2)
  const float ef = erf_as(x * 0.70710678118654752f, e);
  return fmaf(x * 0.39894228040143268f, e, 0.5f * (1.0f + ef));
}

// ---------------------------------------------------------------------------
// inference: 256 threads (4 waves), each wave one 32-cell tile per iteration
// ---------------------------------------------------------------------------
// With a guard G (learned sensor on a mesh): a cell whose features leave the
// network's validity box [lo, hi] (NaN included) or whose output is not
// finite, or every cell once the audit latch is set, gets gamma = NaN, its
// tile flag and a count: the plain sensor takes those cells over.
__global__ __launch_bounds__(256) void mlp_infer_kernel(const uint16_t* __restrict__ feat, int64_t n, MlpDev W,
                                                        float* __restrict__ gamma, MlpGuard G) {
  __shared__ float sb1[MLP_HID], sb2[MLP_HID], sw3[MLP_HID];
  __shared__ float slo[MLP_IN], shi[MLP_IN];
  // the weight operands of every lane, fragment-major (14 fragments x 64 lanes):
  // read per tile from LDS rather than held in registers
  __shared__ u32x4 sA[14][64];
  for (int t = threadIdx.x; t < MLP_HID; t += blockDim.x) {
    sb1[t] = W.b1[t];
    sb2[t] = W.b2[t];
    sw3[t] = bf16_value(W.w3[t]);
  }
  const bool guard = G.lo != nullptr;
  for (int t = threadIdx.x; t < MLP_IN; t += blockDim.x) {
    slo[t] = guard ? G.lo[t] : 0.0f;
    shi[t] = guard ? G.hi[t] : 0.0f;
  }
  const bool off = guard && G.status[WS_LEARNED_OFF] != 0u;
  for (int i = threadIdx.x; i < 14 * 64; i += blockDim.x) {
    const int f = i >> 6, l = i & 63, cl = l & 31, gl = l >> 5;
    bf16x8 a;
    if (f < 6) {
      const int ht = f / 3, kb = f % 3;
      a = load8(W.W1t + (32 * ht + cl) * MLP_IN + 16 * kb + 8 * gl);
    } else {
      const int ht = (f - 6) >> 2, st = ((f - 6) >> 1) & 1, kb = (f - 6) & 1;
      const uint16_t* row = W.W2t + (32 * ht + cl) * MLP_HID + 32 * st + 16 * kb + 4 * gl;
      a = load4x2(row, row + 8);
    }
    sA[f][l] = __builtin_bit_cast(u32x4, a);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 31, g = lane >> 5;
  const float b3 = W.b3[0];
  const int64_t ntiles = (n + 31) / 32;
  for (int64_t t = blockIdx.x * 4LL + wave; t < ntiles; t += static_cast<int64_t>(gridDim.x) * 4) {
    asm volatile("" ::: "memory");              // keeps the LDS weight reads in the loop
    const int64_t cell = t * 32 + c;
    const bool ok = cell < n;
    bf16x8 B1[3];
#pragma unroll
    for (int kb = 0; kb < 3; ++kb) B1[kb] = ok ? load8(feat + cell * MLP_IN + 16 * kb + 8 * g) : zero8();
    // the lane's 24 features against the validity box (lane group g holds k = 16 kb + 8 g + i)
    bool outside = false;
    if (guard) {
#pragma unroll
      for (int kb = 0; kb < 3; ++kb) {
        const u32x4 w = __builtin_bit_cast(u32x4, B1[kb]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint16_t h = static_cast<uint16_t>((w[i >> 1] >> (16 * (i & 1))) & 0xFFFFu);
          const float x = bf16_value(h);
          const int k = 16 * kb + 8 * g + i;
          outside |= !((x >= slo[k]) & (x <= shi[k]));
        }
      }
    }
    f32x16 C1[2];
#pragma unroll
    for (int ht = 0; ht < 2; ++ht) {
      C1[ht] = zero16();
#pragma unroll
      for (int kb = 0; kb < 3; ++kb) C1[ht] = mma(__builtin_bit_cast(bf16x8, sA[3 * ht + kb][lane]), B1[kb], C1[ht]);
    }
    bf16x8 B2[2][2];
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        u32x4 h;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 8 * kb + 2 * i;
          h[i] = bf16_pair(gelu(C1[st][v] + sb1[32 * st + acc_row(v, g)]),
                           gelu(C1[st][v + 1] + sb1[32 * st + acc_row(v + 1, g)]));
        }
        B2[st][kb] = __builtin_bit_cast(bf16x8, h);
      }
    float z = 0.0f;
#pragma unroll
    for (int ht = 0; ht < 2; ++ht) {
      f32x16 C2 = zero16();
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          C2 = mma(__builtin_bit_cast(bf16x8, sA[6 + 4 * ht + 2 * st + kb][lane]), B2[st][kb], C2);
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const int r = 32 * ht + acc_row(v, g);
        const uint32_t h = bf16_pair(gelu(C2[v] + sb2[r]), gelu(C2[v + 1] + sb2[r + 1]));
        z = fmaf(sw3[r], __uint_as_float(h << 16), z);
        z = fmaf(sw3[r + 1], __uint_as_float(h & 0xFFFF0000u), z);
      }
    }
    z += __shfl_xor(z, 32);
    float gv = 1.0f / (1.0f + expf(-(z + b3)));
    if (guard) {
      const bool other = __shfl_xor(static_cast<int>(outside), 32) != 0;
      const bool bad = ok && (off || outside || other || !isfinite(gv));
      if (bad) gv = __builtin_nanf("");
      if (bad && g == 0) {
        const int64_t i = cell % G.nx, j = cell / G.nx;
        G.tile_flag[(i / 16) + G.tiles_x * (j / 16)] = 1;
      }
      const unsigned long long m = __ballot(bad && g == 0);
      if (m && (threadIdx.x & 63) == __builtin_ctzll(m)) {
        atomicAdd(G.status + WS_FALLBACK_COUNT, static_cast<uint32_t>(__popcll(m)));
        atomicOr(G.status + WS_STATUS, ST_LEARNED_FALLBACK);
      }
    }
    if (g == 0 && ok) gamma[cell] = gv;
  }
}

// ---------------------------------------------------------------------------
// training: four waves per block, 32 samples; writes the block's gradient
// ---------------------------------------------------------------------------
__device__ __forceinline__ void split(float x, uint16_t& hi, uint16_t& lo) {
  hi = bf16_bits(x);
  lo = bf16_bits(x - bf16_value(hi));
}

// Wave (t, kb) takes the eight accumulators v = 8 kb .. 8 kb + 7 of tile t of each
// layer: that is the operand fragment (t, kb) of the next product, which it leaves
// in LDS for all four (split into two bfloat16 terms).  The 32 x 32 products
// themselves are formed by both waves of a tile; of the weight gradients' tiles
// each wave has one of either layer.  A batch has few blocks (128 at 4096 samples),
// so a block's chain of products, GELUs and LDS exchanges sets the time: one wave
// per block took 17.1 us, four take 12.5 us (4096 samples).
constexpr int SROW = 40;               // row stride of the bfloat16 copies: 16-byte aligned, spread over the banks
__global__ __launch_bounds__(256) void mlp_train_kernel(const uint16_t* __restrict__ feat,
                                                        const float* __restrict__ target,
                                                        const int32_t* __restrict__ idx, int batch, MlpDev W,
                                                        float* __restrict__ part) {
  __shared__ __align__(16) uint16_t sX[MLP_IN][SROW];
  __shared__ __align__(16) uint16_t sH1[2][MLP_HID][SROW];
  __shared__ __align__(16) uint16_t sD2[2][MLP_HID][SROW];
  __shared__ __align__(16) uint16_t sD1[2][MLP_HID][SROW];
  __shared__ float sD1f[MLP_HID][33], sD2f[MLP_HID][33], sH2f[MLP_HID][33], sd3[32], sz[4][32];
  __shared__ u32x4 sB[2][2][2][64];      // operand fragments [hi / lo][t][kb][lane]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int ti = wave & 1, kq = wave >> 1;
  const int sglob = blockIdx.x * 32 + c;
  const bool ok = sglob < batch;
  const int64_t row = ok ? idx[sglob] : 0;
  float* out = part + static_cast<int64_t>(blockIdx.x) * MLP_NPARAM;
  auto unit = [&](int i) { return 32 * ti + 16 * kq + 8 * (i >> 2) + 4 * g + (i & 3); };   // acc_row(8 kq + i, g) of tile ti
  auto share = [&](const float* x) {
    uint16_t hi[8], lo[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) split(x[i], hi[i], lo[i]);
    sB[0][ti][kq][lane] = __builtin_bit_cast(u32x4, pack8(hi));
    sB[1][ti][kq][lane] = __builtin_bit_cast(u32x4, pack8(lo));
  };
  auto pick = [&](const f32x16& C, float* x) {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = kq ? C[8 + i] : C[i];
  };
  // tile ti of the product of the rows R with the shared operand
  auto product = [&](const uint16_t* R) {
    f32x16 C = zero16();
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const uint16_t* r = R + (32 * ti + c) * MLP_HID + 32 * st + 16 * kb + 4 * g;
        const bf16x8 A = load4x2(r, r + 8);
        C = mma(A, __builtin_bit_cast(bf16x8, sB[0][st][kb][lane]), C);
        C = mma(A, __builtin_bit_cast(bf16x8, sB[1][st][kb][lane]), C);
      }
    return C;
  };

  // ---- forward ----
  bf16x8 B1[3];
#pragma unroll
  for (int kb = 0; kb < 3; ++kb) {
    B1[kb] = ok ? load8(feat + row * MLP_IN + 16 * kb + 8 * g) : zero8();
    if (wave == kb) {
      const u32x4 w = __builtin_bit_cast(u32x4, B1[kb]);
#pragma unroll
      for (int i = 0; i < 8; ++i) sX[16 * kb + 8 * g + i][c] = static_cast<uint16_t>(w[i >> 1] >> (16 * (i & 1)));
    }
  }
  float h1[8], gp1[8];
  {
    f32x16 C = zero16();
#pragma unroll
    for (int kb = 0; kb < 3; ++kb) C = mma(load8(W.W1t + (32 * ti + c) * MLP_IN + 16 * kb + 8 * g), B1[kb], C);
    float x[8];
    pick(C, x);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float z = x[i] + W.b1[unit(i)];
      h1[i] = gelu(z);
      gp1[i] = gelu_prime(z);
    }
  }
  share(h1);
  __syncthreads();
  float h2[8], gp2[8], w3[8], z3 = 0.0f;
  {
    float x[8];
    pick(product(W.W2t), x);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int n2 = unit(i);
      const float z = x[i] + W.b2[n2];
      h2[i] = gelu(z);
      gp2[i] = gelu_prime(z);
      w3[i] = bf16_value(W.w3[n2]);
      z3 = fmaf(w3[i], h2[i], z3);
    }
  }
  z3 += __shfl_xor(z3, 32);
  if (g == 0) sz[wave][c] = z3;
  __syncthreads();
  z3 = (sz[0][c] + sz[2][c]) + (sz[1][c] + sz[3][c]);      // the same in every wave
  const float gam = 1.0f / (1.0f + expf(-(z3 + W.b3[0])));
  const float d3 = ok ? 2.0f * (gam - target[row]) / static_cast<float>(batch) * gam * (1.0f - gam) : 0.0f;

  // ---- backward ----
  float d2[8], d1[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) d2[i] = d3 * w3[i] * gp2[i];
  share(d2);                             // every wave has passed its second product: the fragments are free
  __syncthreads();
  {
    // d1 = (W2 d2) * gelu'(z1): rows of W2, reduction over n in the held-row order
    float x[8];
    pick(product(W.W2r), x);
#pragma unroll
    for (int i = 0; i < 8; ++i) d1[i] = x[i] * gp1[i];
  }
  // transposed copies (row = unit, column = sample) for the weight gradients
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = unit(i);
    uint16_t hi, lo;
    split(h1[i], hi, lo);
    sH1[0][r][c] = hi;
    sH1[1][r][c] = lo;
    split(d2[i], hi, lo);
    sD2[0][r][c] = hi;
    sD2[1][r][c] = lo;
    split(d1[i], hi, lo);
    sD1[0][r][c] = hi;
    sD1[1][r][c] = lo;
    sD1f[r][c] = d1[i];
    sD2f[r][c] = d2[i];
    sH2f[r][c] = h2[i];
  }
  if (threadIdx.x < 32) sd3[c] = d3;
  __syncthreads();
  {
    // dW2[k][n] = sum_s h1[k][s] d2[n][s], tile (ti, kq)
    f32x16 C = zero16();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8 Ah = load8(&sH1[0][32 * ti + c][16 * ks + 8 * g]), Al = load8(&sH1[1][32 * ti + c][16 * ks + 8 * g]);
      const bf16x8 Bh = load8(&sD2[0][32 * kq + c][16 * ks + 8 * g]), Bl = load8(&sD2[1][32 * kq + c][16 * ks + 8 * g]);
      C = mma(Ah, Bh, C);
      C = mma(Ah, Bl, C);
      C = mma(Al, Bh, C);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) out[MLP_OFF_W2 + (32 * ti + acc_row(v, g)) * MLP_HID + 32 * kq + c] = C[v];
  }
  {
    // dW1[f][k] = sum_s x[s][f] d1[k][s], tile (ti, kq)
    f32x16 C = zero16();
    const int fr = 32 * ti + c;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8 A = (fr < MLP_IN) ? load8(&sX[fr][16 * ks + 8 * g]) : zero8();
      C = mma(A, load8(&sD1[0][32 * kq + c][16 * ks + 8 * g]), C);
      C = mma(A, load8(&sD1[1][32 * kq + c][16 * ks + 8 * g]), C);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int f = 32 * ti + acc_row(v, g);
      if (f < MLP_IN) out[MLP_OFF_W1 + f * MLP_HID + 32 * kq + c] = C[v];
    }
  }
  // bias and output-weight gradients, fixed order over the 32 samples
  if (wave == 0) {
    float s1 = 0.0f;
    for (int s = 0; s < 32; ++s) s1 += sD1f[lane][s];
    out[MLP_OFF_B1 + lane] = s1;
  } else if (wave == 1) {
    float s2 = 0.0f;
    for (int s = 0; s < 32; ++s) s2 += sD2f[lane][s];
    out[MLP_OFF_B2 + lane] = s2;
  } else if (wave == 2) {
    float s3 = 0.0f;
    for (int s = 0; s < 32; ++s) s3 = fmaf(sH2f[lane][s], sd3[s], s3);
    out[MLP_OFF_W3 + lane] = s3;
  } else if (lane == 0) {
    float s3 = 0.0f;
    for (int s = 0; s < 32; ++s) s3 += sd3[s];
    out[MLP_OFF_B3] = s3;
  }
}

// ---------------------------------------------------------------------------
// sum of the block gradients (float64), Adam on the float32 master weights
// (lr = 0: no update), and the compute copies.  A workgroup takes 64 parameters;
// its waves take every UPD_WAVES-th block gradient and their sums meet in wave order
// (one thread per parameter walking all 128 blocks: 31.3 us, so 4.0 us).
// ---------------------------------------------------------------------------
constexpr int UPD_WAVES = 16;
__global__ __launch_bounds__(64 * UPD_WAVES) void mlp_update_kernel(const float* __restrict__ part, int nblk,
                                                                    float* __restrict__ master, float* __restrict__ m1,
                                                                    float* __restrict__ m2, float lr, float beta1,
                                                                    float beta2, float omb1, float omb2, float eps,
                                                                    float bc1, float bc2, float* __restrict__ grad_out,
                                                                    MlpDevMut W) {
  __shared__ double sg[UPD_WAVES][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
  double gs = 0.0;
  if (j < MLP_NPARAM) {
#pragma unroll 8
    for (int b = wave; b < nblk; b += UPD_WAVES) gs += static_cast<double>(part[static_cast<int64_t>(b) * MLP_NPARAM + j]);
  }
  sg[wave][lane] = gs;
  __syncthreads();
  if (wave != 0 || j >= MLP_NPARAM) return;
#pragma unroll
  for (int w = 1; w < UPD_WAVES; ++w) gs += sg[w][lane];
  const float gr = static_cast<float>(gs);
  if (grad_out) grad_out[j] = gr;
  float w = master[j];
  if (lr > 0.0f) {
    const float a = beta1 * m1[j] + omb1 * gr;          // omb = 1 - beta, formed in float64
    const float b = beta2 * m2[j] + omb2 * gr * gr;
    m1[j] = a;
    m2[j] = b;
    w -= lr * (a / bc1) / (sqrtf(b / bc2) + eps);
    master[j] = w;
  }
  if (j < MLP_OFF_B1) {                      // W1[f][k]
    const int f = j / MLP_HID, k = j % MLP_HID;
    W.W1t[k * MLP_IN + f] = bf16_bits(w);
  } else if (j < MLP_OFF_W2) {
    W.b1[j - MLP_OFF_B1] = w;
  } else if (j < MLP_OFF_B2) {               // W2[k][n]
    const int q = j - MLP_OFF_W2, k = q / MLP_HID, n = q % MLP_HID;
    const uint16_t h = bf16_bits(w);
    W.W2t[n * MLP_HID + k] = h;
    W.W2r[k * MLP_HID + n] = h;
  } else if (j < MLP_OFF_W3) {
    W.b2[j - MLP_OFF_B2] = w;
  } else if (j < MLP_OFF_B3) {
    W.w3[j - MLP_OFF_W3] = bf16_bits(w);
  } else {
    W.b3[0] = w;
  }
}

// ---------------------------------------------------------------------------
cvw_status mlp_infer(const MlpDev& W, const uint16_t* feat, int64_t n, float* gamma, hipStream_t s,
                     const MlpGuard* guard) {
  if (n <= 0) return CVW_OK;
  const int64_t tiles = (n + 31) / 32;
  const unsigned grid = static_cast<unsigned>(std::min<int64_t>((tiles + 3) / 4, 4096));
  const MlpGuard G = guard ? *guard : MlpGuard{};
  hipLaunchKernelGGL(mlp_infer_kernel, dim3(grid), dim3(256), 0, s, feat, n, W, gamma, G);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

cvw_status mlp_train(const MlpDev& W, const uint16_t* feat, const float* target, const int32_t* idx, int batch,
                     float* part, hipStream_t s) {
  const int nblk = (batch + 31) / 32;
  hipLaunchKernelGGL(mlp_train_kernel, dim3(nblk), dim3(256), 0, s, feat, target, idx, batch, W, part);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

cvw_status mlp_update(const float* part, int nblk, float* master, float* m1, float* m2, float lr, double beta1,
                      double beta2, float eps, double bc1, double bc2, float* grad_out, const MlpDevMut& W,
                      hipStream_t s) {
  hipLaunchKernelGGL(mlp_update_kernel, dim3((MLP_NPARAM + 63) / 64), dim3(64 * UPD_WAVES), 0, s, part, nblk, master, m1, m2,
                     lr, static_cast<float>(beta1), static_cast<float>(beta2), static_cast<float>(1.0 - beta1),
                     static_cast<float>(1.0 - beta2), eps, static_cast<float>(bc1), static_cast<float>(bc2), grad_out,
                     W);
  return hipGetLastError() == hipSuccess ? CVW_OK : CVW_EDEVICE;
}

}  // namespace cvw
