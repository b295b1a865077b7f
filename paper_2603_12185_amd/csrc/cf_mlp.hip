// cf_mlp.hip - training and batch inference of the learned per-contact
// impedance network (layout in cf_mlp.h): bf16 MFMA with float32
// accumulation, mean-squared-error gradient with deterministic partial sums
// per block, Adam.
#include <hip/hip_runtime.h>

#include <mutex>
#include <string>

#include "../../include/cfsim.h"
#include "cf_mlp.h"

namespace cf {
cf_status api_error(cf_status st, const std::string &msg);  // cf_api.hip
}

namespace cf {
namespace mlp {

constexpr int BS = 256;  // four waves per block
constexpr int NWAVE = BS / 64;

// Weight fragments of the 16x16x16 products in the order the lanes read them:
// entry [f][l] is lane l's four K values of operand f (q = l / 16, c = l % 16),
// so a wave's read of a fragment is one conflict-free 8-byte LDS access (the
// row-major bf16 weights put all sixteen rows of a fragment on the same banks).
// Forward operands (rows = output units of the layer, K = input units):
//   w1[m]:      W1[4 q + t][16 m + c] (features >= 8: 0)
//   w2[4 o + m]: W2[16 m + 4 q + t][16 o + c]
//   w3[m]:      W3[16 m + 4 q + t][c]
struct Frags {
  bf16x4 w1[4][64], w2[16][64], w3[4][64];
  float4 b1[16], b2[16], b3[4];  // biases of units 4 i .. 4 i + 3
  float4 mean[2], istd[2];
};
// Operands of the reverse products (rows = input units, K = output units):
//   w2r[4 i + k]: W2[16 i + c][16 k + 4 q + t], w3r[m]: W3[16 m + c][4 q + t]
struct RevFrags {
  bf16x4 w2r[16][64], w3r[4][64];
};

// Four floats rounded to bf16 (nearest even), two per v_cvt_pk_bf16_f32.
__device__ inline bf16x4 pack4(float a, float b, float c, float d) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const f2 lo = {a, b}, hi = {c, d};
  const u2 v = {__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2)),
                __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2))};
  return __builtin_bit_cast(bf16x4, v);
}
__device__ inline bf16x4 pack4(f32x4 v) { return pack4(v[0], v[1], v[2], v[3]); }

// Fill the fragments from the float32 parameters (all threads; a wave's loads
// of one K value are four runs of 64 bytes).  The caller puts the barrier.
__device__ inline void stage_frags(const float *p, Frags &F) {
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6, q = l >> 4, c = l & 15;
#pragma unroll
  for (int i = wave; i < 16; i += NWAVE) {
    const float *w = p + OFF_W2 + (16 * (i & 3) + 4 * q) * NH + 16 * (i >> 2) + c;
    F.w2[i][l] = pack4(w[0], w[NH], w[2 * NH], w[3 * NH]);
  }
  {
    const int m = wave;
    const float *w = p + OFF_W1 + (4 * (q & 1)) * NH + 16 * m + c, *u = p + OFF_W3 + (16 * m + 4 * q) * NOUT + c;
    const bf16x4 a = pack4(w[0], w[NH], w[2 * NH], w[3 * NH]), z = {0, 0, 0, 0};
    F.w1[m][l] = q < 2 ? a : z;
    F.w3[m][l] = pack4(u[0], u[NOUT], u[2 * NOUT], u[3 * NOUT]);
  }
  const int i = threadIdx.x;
  auto f4 = [&](int at) { return *reinterpret_cast<const float4 *>(p + at); };
  if (i < 16) F.b1[i] = f4(OFF_B1 + 4 * i);
  else if (i < 32) F.b2[i - 16] = f4(OFF_B2 + 4 * (i - 16));
  else if (i < 36) F.b3[i - 32] = f4(OFF_B3 + 4 * (i - 32));
  else if (i < 38) F.mean[i - 36] = f4(OFF_MEAN + 4 * (i - 36));
  else if (i < 40) {
    const float4 s = f4(OFF_STD + 4 * (i - 38));
    F.istd[i - 38] = make_float4(1.0f / s.x, 1.0f / s.y, 1.0f / s.z, 1.0f / s.w);
  }
}
__device__ inline void stage_rev_frags(const float *p, RevFrags &F) {
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6, q = l >> 4, c = l & 15;
  auto f4 = [&](int at) {
    const float4 v = *reinterpret_cast<const float4 *>(p + at);
    return pack4(v.x, v.y, v.z, v.w);
  };
#pragma unroll
  for (int i = wave; i < 16; i += NWAVE) F.w2r[i][l] = f4(OFF_W2 + (16 * (i >> 2) + c) * NH + 16 * (i & 3) + 4 * q);
  F.w3r[wave][l] = f4(OFF_W3 + (16 * wave + c) * NOUT + 4 * q);
}

// The lane's raw features 4 q .. 4 q + 3 of contact ci (the lanes of q >= 2
// and of contacts past n hold zeros they never use).
__device__ inline float4 load_feats(const float *feats, int ci, int n, int q) {
  return (ci < n && q < 2) ? *reinterpret_cast<const float4 *>(feats + (size_t)ci * NIN + 4 * q)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
}
// The lane's input operand: normalised features in bf16, zero past the seventh.
__device__ inline bf16x4 input_operand(float4 f, float4 mean, float4 istd, int q) {
  const float x0 = (f.x - mean.x) * istd.x, x1 = (f.y - mean.y) * istd.y, x2 = (f.z - mean.z) * istd.z,
              x3 = q == 0 ? (f.w - mean.w) * istd.w : 0.f;
  const bf16x4 v = pack4(x0, x1, x2, x3), z = {0, 0, 0, 0};
  return q < 2 ? v : z;
}
__device__ inline f32x4 add_bias(f32x4 z, float4 b) {
  z[0] += b.x; z[1] += b.y; z[2] += b.z; z[3] += b.w;
  return z;
}

// Batch inference, 16 contacts per wave and pass.  Bound: vector issue of the
// 128 SiLUs per contact (an exponential and a reciprocal each) beside 96 bytes
// of HBM traffic per contact.  Each wave keeps the 24 weight fragments in
// registers over its passes (they fit beside one tile's activations at four
// waves per SIMD) and loads the next tile's features during the current one.
// 954367 contacts on MI355X: 42 us (2.2 TB/s), against 95 us when every block
// of two waves converted the weights for its few tiles and re-read them, rows
// on the same banks, from LDS.
__global__ __launch_bounds__(BS, 4) void forward_kernel(const float *p, const float *feats, int n, float *out) {
  __shared__ Frags F;
  stage_frags(p, F);
  const int l = threadIdx.x & 63, q = l >> 4, c = l & 15;
  const int wave = blockIdx.x * NWAVE + (threadIdx.x >> 6), nwaves = gridDim.x * NWAVE;
  const int ntile = (n + 15) / 16;
  float4 f = load_feats(feats, wave * 16 + c, n, q);
  __syncthreads();
  bf16x4 w1[4], w2[16], w3[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    w1[i] = F.w1[i][l];
    w3[i] = F.w3[i][l];
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) w2[i] = F.w2[i][l];
  const float4 mean = F.mean[q & 1], istd = F.istd[q & 1];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  for (int tile = wave; tile < ntile; tile += nwaves) {
    const int ci = tile * 16 + c;
    const bf16x4 x = input_operand(f, mean, istd, q);
    const int next = tile + nwaves;
    if (next < ntile) f = load_feats(feats, next * 16 + c, n, q);
    bf16x4 a1[4], a2[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const f32x4 z = add_bias(mfma(w1[m], x, zero), F.b1[4 * m + q]);
      a1[m] = pack4(silu(z[0]), silu(z[1]), silu(z[2]), silu(z[3]));
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      f32x4 z = zero;
#pragma unroll
      for (int m = 0; m < 4; ++m) z = mfma(w2[4 * o + m], a1[m], z);
      z = add_bias(z, F.b2[4 * o + q]);
      a2[o] = pack4(silu(z[0]), silu(z[1]), silu(z[2]), silu(z[3]));
    }
    f32x4 y = zero;
#pragma unroll
    for (int m = 0; m < 4; ++m) y = mfma(w3[m], a2[m], y);
    y = add_bias(y, F.b3[q]);
    if (ci < n) *reinterpret_cast<float4 *>(out + (size_t)ci * NOUT + 4 * q) = make_float4(y[0], y[1], y[2], y[3]);
  }
}

// ---- gradient of L = sum over contacts and the first nout outputs of
// (y - target)^2 / (n nout)
//
// A lane's share of the sums: GREG registers in the matrix accumulator layout
// (lane l = (q, c), r = 0..3):
//   [4 j + r]             dL/dW1[4 q + r][16 j + c]
//   [16 + 16 i + 4 j + r] dL/dW2[16 i + 4 q + r][16 j + c]
//   [80 + 4 m + r]        dL/dW3[16 m + 4 q + r][c]
//   [96], [97]            dL/db1, dL/db2 of unit 16 (c / 4) + 4 q + c % 4
//   [98]                  dL/db3 of output 4 q + c (c < 4)
//   [99]                  the loss (lane 0)
// A block's partial sums are one row of GREG x 64 floats in that order.
constexpr int GREG = 100, GROW = GREG * 64;
// One wave per SIMD of the whole device: 65536 rows took 23.4 us at 256 blocks,
// 24.0 at 512 and 34.6 at 1024 (more partial rows to write and to sum).
constexpr int MAX_GRAD_BLOCKS = 256;

// Index in the gradient of register i of lane l (NPARAM: the loss), or -1.
__device__ inline int grad_index(int i, int l) {
  const int q = l >> 4, c = l & 15, r = i & 3;
  if (i < 16) return q < 2 ? OFF_W1 + (4 * q + r) * NH + 16 * (i >> 2) + c : -1;
  if (i < 80) return OFF_W2 + (16 * ((i - 16) >> 4) + 4 * q + r) * NH + 16 * ((i >> 2) & 3) + c;
  if (i < 96) return OFF_W3 + (16 * ((i - 80) >> 2) + 4 * q + r) * NOUT + c;
  const int u = 16 * (c >> 2) + 4 * q + (c & 3);
  if (i == 96) return OFF_B1 + u;
  if (i == 97) return OFF_B2 + u;
  if (i == 98) return c < 4 ? OFF_B3 + 4 * q + c : -1;
  return l == 0 ? NPARAM : -1;
}

// Sum over the sixteen lanes of a row (every lane gets it).
__device__ inline float row_sum(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, false));  // row_ror:8
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, false));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, false));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, false));
  return x;
}

// silu(z) and its derivative from one sigmoid.
__device__ inline float silu_both(float z, float &d) {
  const float s = sigmoid(z);
  d = s * (1.0f + z * (1.0f - s));
  return z * s;
}

// Each wave walks tiles of 16 contacts; the block's waves add their sums in
// LDS in a fixed order and the block writes one row of `partial`.
//
// The weight gradients contract over contacts, so both operands are needed
// with contacts along K while the forward products hold them along columns.
// A 16 x 16 block V (lane (q, c): V[4 q + r][c]) read as an A operand is V^T;
// its product with the identity gives V^T in the accumulator layout, which read
// as an operand again holds V's rows along the lanes and contacts along K:
// the transpose is one more MFMA, exact on bf16 values, and nothing passes
// through LDS (a layout change through 2-byte LDS accesses took most of the
// earlier kernel's time).  dL/dy alone goes through LDS, so that a non-finite
// output adjoint stays in its own column.  65536 rows on MI355X: the gradient
// and its sum take 23 us; they took 64 + 481 us with 2048 rows of partials,
// summed by 23 blocks.
union GradLds {
  struct {
    Frags f;
    RevFrags b;
    float dys[NWAVE][16 * 16];
  } s;
  float red[NWAVE / 2][GROW];
};
__global__ __launch_bounds__(BS, 1) void grad_kernel(const float *p, const float *feats, const float *tgt, int n,
                                                     int nout, float *partial) {
  __shared__ GradLds G;
  Frags &F = G.s.f;
  RevFrags &R = G.s.b;
  stage_frags(p, F);
  stage_rev_frags(p, R);
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, q = l >> 4, c = l & 15;
  const int wave = blockIdx.x * NWAVE + wv, nwaves = gridDim.x * NWAVE;
  float *dys = G.s.dys[wv];
  __syncthreads();
  const int ntile = (n + 15) / 16;
  const float sc = 2.0f / ((float)n * (float)nout);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const bf16x4 eye = pack4(4 * q == c ? 1.f : 0.f, 4 * q + 1 == c ? 1.f : 0.f, 4 * q + 2 == c ? 1.f : 0.f,
                           4 * q + 3 == c ? 1.f : 0.f);
  auto turn = [&](bf16x4 v) { return pack4(mfma(v, eye, zero)); };
  f32x4 gW1[4], gW2[4][4], gW3[4], gb1[4], gb2[4], gb3 = zero;
  float lossp = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    gW1[i] = gW3[i] = gb1[i] = gb2[i] = zero;
#pragma unroll
    for (int j = 0; j < 4; ++j) gW2[i][j] = zero;
  }
  for (int tile = wave; tile < ntile; tile += nwaves) {
    const int ci = tile * 16 + c;
    const bool valid = ci < n;
    const float4 f = load_feats(feats, ci, n, q);
    const float4 tg = valid ? *reinterpret_cast<const float4 *>(tgt + (size_t)ci * NOUT + 4 * q)
                            : make_float4(0.f, 0.f, 0.f, 0.f);
    // forward pass, keeping the activations (bf16) and the SiLU derivatives
    const bf16x4 x = input_operand(f, F.mean[q & 1], F.istd[q & 1], q);
    bf16x4 a1[4], a2[4];
    f32x4 d1[4], d2[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const f32x4 z = add_bias(mfma(F.w1[m][l], x, zero), F.b1[4 * m + q]);
      f32x4 s;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float d;
        s[r] = silu_both(z[r], d);
        d1[m][r] = d;
      }
      a1[m] = pack4(s);
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      f32x4 z = zero;
#pragma unroll
      for (int m = 0; m < 4; ++m) z = mfma(F.w2[4 * o + m][l], a1[m], z);
      z = add_bias(z, F.b2[4 * o + q]);
      f32x4 s;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float d;
        s[r] = silu_both(z[r], d);
        d2[o][r] = d;
      }
      a2[o] = pack4(s);
    }
    f32x4 y = zero;
#pragma unroll
    for (int m = 0; m < 4; ++m) y = mfma(F.w3[m][l], a2[m], y);
    y = add_bias(y, F.b3[q]);
    // dL/dy, transposed: lane holds outputs 4 q + r of contact c
    f32x4 dy;
    const float t4[4] = {tg.x, tg.y, tg.z, tg.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 4 * q + r;
      const float d = (valid && o < nout) ? y[r] - t4[r] : 0.f;
      lossp += d * d;
      dy[r] = sc * d;
      dys[o * 16 + c] = dy[r];
      gb3[r] += dy[r];
    }
    const bf16x4 dyb = pack4(dy);
    // dz2^T = (W3 dy^T) * silu'(z2)
    bf16x4 z2b[4], z1b[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f32x4 dz = mfma(R.w3r[m][l], dyb, zero);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dz[r] *= d2[m][r];
        gb2[m][r] += dz[r];
      }
      z2b[m] = pack4(dz);
    }
    // dz1^T = (W2 dz2^T) * silu'(z1)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f32x4 dz = zero;
#pragma unroll
      for (int k = 0; k < 4; ++k) dz = mfma(R.w2r[4 * m + k][l], z2b[k], dz);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dz[r] *= d1[m][r];
        gb1[m][r] += dz[r];
      }
      z1b[m] = pack4(dz);
    }
    // weight gradients over the tile's 16 contacts (K = contacts)
    __builtin_amdgcn_wave_barrier();
    const float4 dyt = *reinterpret_cast<const float4 *>(dys + c * 16 + 4 * q);
    const bf16x4 bdy = pack4(dyt.x, dyt.y, dyt.z, dyt.w), ax = turn(x);
    bf16x4 bz[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      gW3[m] = mfma(turn(a2[m]), bdy, gW3[m]);
      gW1[m] = mfma(ax, turn(z1b[m]), gW1[m]);
      bz[m] = turn(z2b[m]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16x4 at = turn(a1[i]);
#pragma unroll
      for (int j = 0; j < 4; ++j) gW2[i][j] = mfma(at, bz[j], gW2[i][j]);
    }
    __builtin_amdgcn_wave_barrier();
  }
  // the lane's registers in the row's order
  float g[GREG];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      g[4 * j + r] = gW1[j][r];
      g[80 + 4 * j + r] = gW3[j][r];
#pragma unroll
      for (int i = 0; i < 4; ++i) g[16 + 16 * i + 4 * j + r] = gW2[i][j][r];
    }
  g[96] = g[97] = g[98] = 0.f;
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float s1 = row_sum(gb1[m][r]), s2 = row_sum(gb2[m][r]);
      if (c == 4 * m + r) {
        g[96] = s1;
        g[97] = s2;
      }
      if (m == 0) {
        const float s3 = row_sum(gb3[r]);
        if (c == r) g[98] = s3;
      }
    }
  for (int off = 32; off > 0; off >>= 1) lossp += __shfl_xor(lossp, off);
  g[99] = lossp / ((float)n * (float)nout);
  // waves 2, 3 into 0, 1, then 1 into 0, through LDS
#pragma unroll
  for (int h = NWAVE / 2; h > 0; h >>= 1) {
    __syncthreads();
    if (wv >= h && wv < 2 * h) {
#pragma unroll
      for (int i = 0; i < GREG; ++i) G.red[wv - h][i * 64 + l] = g[i];
    }
    __syncthreads();
    if (wv < h) {
#pragma unroll
      for (int i = 0; i < GREG; ++i) g[i] += G.red[wv][i * 64 + l];
    }
  }
  if (wv == 0) {
    float *P = partial + (size_t)blockIdx.x * GROW;
#pragma unroll
    for (int i = 0; i < GREG; ++i) P[i * 64 + l] = g[i];
  }
}

// Sum of the partial rows: block i takes register i of the rows (256 bytes of
// each), its sixteen waves every sixteenth row; their sums are added in wave
// order.  A hundred blocks of independent loads keep the sum at the latency of
// one pass over at most 6.6 MB, where one thread per parameter walked all rows
// in turn.
constexpr int RED_WAVES = 16;
__global__ __launch_bounds__(64 * RED_WAVES) void reduce_kernel(const float *partial, int rows, float *grad,
                                                                float *loss) {
  __shared__ float part[RED_WAVES][64];
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, i = blockIdx.x;
  const float *P = partial + i * 64 + l;
  float acc = 0.f;
#pragma unroll 8
  for (int r = wv; r < rows; r += RED_WAVES) acc += P[(size_t)r * GROW];
  part[wv][l] = acc;
  __syncthreads();
  if (wv == 0) {
    float s = part[0][l];
#pragma unroll
    for (int k = 1; k < RED_WAVES; ++k) s += part[k][l];
    const int at = grad_index(i, l);
    if (at >= 0 && at < NPARAM) grad[at] = s;
    else if (at == NPARAM && loss) *loss = s;
  } else if (wv == 1 && i == 0 && l < TRAIN_FROM) {
    grad[l] = 0.f;  // the normalisation is not trained
  }
}

__global__ void adam_kernel(float *p, float *m, float *v, const float *g, float lr, float bc1, float bc2) {
  const int i = TRAIN_FROM + blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= NPARAM) return;
  const float gi = g[i];
  const float mi = 0.9f * m[i] + 0.1f * gi;
  const float vi = 0.999f * v[i] + 0.001f * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + 1e-8f);
}

// Partial rows (blocks) of a gradient over n contacts: a tile per wave until
// the device holds one wave per SIMD, then more tiles per wave, which costs no
// further partial sums.
static int grad_rows(int n) {
  const int rows = ((n + 15) / 16 + NWAVE - 1) / NWAVE;
  return rows < MAX_GRAD_BLOCKS ? rows : MAX_GRAD_BLOCKS;
}

// Floats of the caller's workspace: room for one row of NPARAM + 1 floats per
// two tiles, at most 2048, which covers the partial rows of every n (grad_rows(n)
// of GROW floats) and is what callers of this ABI have allocated.
static int64_t work_floats_of(int n) {
  int64_t w = ((n + 15) / 16 + 1) / 2;
  w = w > 2048 ? 2048 : w < 2 ? 2 : (w + 1) / 2 * 2;
  return w * (NPARAM + 1);
}

// The network's LDS image (layout of Weights: bf16 transposed weights, float32
// biases and normalisation) written once per step from the float32 parameters,
// so each workgroup of the resolution copies it instead of converting.
__global__ __launch_bounds__(256) void pack_kernel(const float *p, Weights *img) { stage_weights<256>(p, img); }

}  // namespace mlp

size_t mlp_image_bytes() { return sizeof(mlp::Weights); }
size_t mlp_image_k32_bytes() { return sizeof(mlp::WeightsK32); }

hipError_t launch_mlp_pack(const float *params, void *img, hipStream_t s) {
  hipLaunchKernelGGL(mlp::pack_kernel, dim3(1), dim3(256), 0, s, params, reinterpret_cast<mlp::Weights *>(img));
  return hipGetLastError();
}

}  // namespace cf

using namespace cf::mlp;

static bool al16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

extern "C" int32_t cf_mlp_nparam(void) { return NPARAM; }

extern "C" int64_t cf_mlp_work_floats(int32_t n) {
  if (n < 1) return 0;
  return work_floats_of(n);
}

extern "C" cf_status cf_mlp_forward(void *stream, const float *params, const float *feats, int32_t n, float *out) {
  if (!params || !feats || !out || n < 0) return cf::api_error(CF_E_INVALID_ARG, "cf_mlp_forward: bad argument");
  if (!al16(params) || !al16(feats) || !al16(out)) return cf::api_error(CF_E_INVALID_ARG, "buffers must be 16-byte aligned");
  if (n == 0) return CF_OK;
  // a tile per wave until the device is full (four blocks of four waves per CU)
  int blocks = ((n + 15) / 16 + NWAVE - 1) / NWAVE;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(forward_kernel, dim3(blocks), dim3(BS), 0, (hipStream_t)stream, params, feats, n, out);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? CF_OK : cf::api_error(CF_E_DEVICE, std::string("mlp forward: ") + hipGetErrorString(e));
}

// The gradient's two launches: one partial row per block into `work` (every
// entry written), then their sum.
static cf_status launch_gradient(hipStream_t s, const float *params, const float *feats, const float *targets, int n,
                                 int nout, float *work, float *grad, float *loss) {
  const int rows = grad_rows(n);
  hipLaunchKernelGGL(grad_kernel, dim3(rows), dim3(BS), 0, s, params, feats, targets, n, nout, work);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(reduce_kernel, dim3(GREG), dim3(64 * RED_WAVES), 0, s, work, rows, grad, loss);
    e = hipGetLastError();
  }
  return e == hipSuccess ? CF_OK : cf::api_error(CF_E_DEVICE, std::string("mlp gradient: ") + hipGetErrorString(e));
}

extern "C" cf_status cf_mlp_gradient(void *stream, const float *params, const float *feats, const float *targets,
                                     int32_t n, int32_t nout, float *work, int64_t work_floats, float *grad,
                                     float *loss) {
  if (!params || !feats || !targets || !work || !grad || n < 1 || nout < 1 || nout > NOUT)
    return cf::api_error(CF_E_INVALID_ARG, "cf_mlp_gradient: bad argument");
  if (!al16(params) || !al16(feats) || !al16(targets) || !al16(work) || !al16(grad))
    return cf::api_error(CF_E_INVALID_ARG, "buffers must be 16-byte aligned");
  if (work_floats < work_floats_of(n))
    return cf::api_error(CF_E_INVALID_ARG, "work buffer smaller than cf_mlp_work_floats(n)");
  return launch_gradient((hipStream_t)stream, params, feats, targets, n, nout, work, grad, loss);
}

// ---- cf_mlp_gradient without a caller workspace
// The partial rows live in `scratch`: room for the most blocks the gradient
// launches (MAX_GRAD_BLOCKS rows of GROW floats, 6.6 MB), so every n fits.
// Each GPU the library runs on holds its own copy until the process ends.  The
// kernel writes every entry of each row it uses before the sum reads it, so
// nothing is cleared between calls; calls that overlap on one GPU share the
// array and race.
constexpr size_t kScratchFloats = (size_t)MAX_GRAD_BLOCKS * GROW;
static __device__ __align__(256) float scratch[kScratchFloats];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch[kMaxDevices] = {};  // device address of each GPU's `scratch`, taken once per device

// Device address of the current GPU's `scratch` (the array's name is a host
// stand-in: only this address may reach a kernel).
cf_status scratch_address(float **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return cf::api_error(CF_E_DEVICE, "cf_mlp_gradient_noalloc: no current HIP device");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return cf::api_error(CF_E_DEVICE, std::string("cf_mlp_gradient_noalloc: address of the static scratch: ") +
                                            hipGetErrorString(e));
    g_scratch[dev] = static_cast<float *>(p);
  }
  *out = g_scratch[dev];
  return CF_OK;
}
}  // namespace

extern "C" cf_status cf_mlp_gradient_noalloc(void *stream, const float *params, const float *feats,
                                             const float *targets, int32_t n, int32_t nout, float *grad,
                                             float *loss) {
  if (!params || !feats || !targets || !grad || n < 1 || nout < 1 || nout > NOUT)
    return cf::api_error(CF_E_INVALID_ARG, "cf_mlp_gradient_noalloc: bad argument");
  if (!al16(params) || !al16(feats) || !al16(targets) || !al16(grad))
    return cf::api_error(CF_E_INVALID_ARG, "buffers must be 16-byte aligned");
  float *work = nullptr;
  const cf_status st = scratch_address(&work);
  if (st != CF_OK) return st;
  return launch_gradient((hipStream_t)stream, params, feats, targets, n, nout, work, grad, loss);
}

extern "C" cf_status cf_mlp_adam(void *stream, float *params, float *m, float *v, const float *grad, int32_t step,
                                 float lr) {
  if (!params || !m || !v || !grad || step < 1) return cf::api_error(CF_E_INVALID_ARG, "cf_mlp_adam: bad argument");
  const float bc1 = 1.0f - powf(0.9f, (float)step), bc2 = 1.0f - powf(0.999f, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3((NPARAM - TRAIN_FROM + 255) / 256), dim3(256), 0, (hipStream_t)stream, params,
                     m, v, grad, lr, bc1, bc2);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? CF_OK : cf::api_error(CF_E_DEVICE, std::string("mlp adam: ") + hipGetErrorString(e));
}
