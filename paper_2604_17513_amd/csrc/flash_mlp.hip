// Learned warm start: a 16 -> 128 -> 128 -> 128 -> 3 ReLU MLP that predicts the
// contact multipliers of a step from local features.  Every product runs on the
// CDNA matrix cores (v_mfma_f32_32x32x16_bf16): operands are rounded to
// bfloat16 (round to nearest even), products accumulate in FP32.  Training
// keeps FP32 master weights and Adam moments; bias gradients and losses use
// fixed-order reductions, so a training run is deterministic.
#include <algorithm>

#include "flash_device.h"
#include "flash_launch.h"
#include "flash_mlp.h"

namespace flash {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// Fused forward pass on v_mfma_f32_32x32x16_bf16.  Lane layout of that
// instruction: A(m, k) from lane m + 32 (k / 8), element k % 8; B(k, n) from
// lane n + 32 (k / 8), element k % 8; D(i, j) in lane j + 32 ((i / 4) % 2),
// register 4 (i / 8) + i % 4.  The network runs transposed (H^T = W X^T):
// rows of a D tile are neurons, columns are 32 samples, so the registers a
// lane holds for one output tile are exactly the B operand of the next layer
// once the 16 inputs of each K step are visited in the order neuron(k) =
// 8 ((k % 8) / 4) + 4 (k / 8) + k % 4.  The weights are staged in LDS as
// bf16 with the columns of each 16-block permuted to that order (bits 2 and
// 3 of the input index swapped), so every A operand is one 16-byte read.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kLd1 = 24;    // LDS row stride of W1 (bf16): 48 B keeps 16-byte reads conflict-free
constexpr int kLdH = 136;   // LDS row stride of W2, W3, W4 (bf16): 272 B
constexpr int kWaves = 4;

struct FusedSmem {
  __bf16 w1[kHidden * kLd1];
  __bf16 w2[kHidden * kLdH];
  __bf16 w3[kHidden * kLdH];
  __bf16 w4[kOut * kLdH];
  alignas(16) float b[3 * kHidden + 4];
  float nrm[kNorm + 1];
};
constexpr size_t kFusedSmem = sizeof(FusedSmem);

__device__ __forceinline__ int perm16(int c) { return (c & ~12) | ((c & 4) << 1) | ((c & 8) >> 1); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// Two floats to bf16 (nearest even) in one instruction.
__device__ __forceinline__ bf16x2 to_bf2(float a, float b) {
  const floatx2 v = {a, b};
  return __builtin_convertvector(v, bf16x2);
}

// Rounded weights [rows x cols] (row-major floats at W, 16-byte groups) to LDS rows of stride ld, columns
// permuted by perm16 with PERM: each group of 4 columns stays together.  U groups per thread in flight.
template <bool PERM, int U>
__device__ __forceinline__ void stage_weights(const float* W, int rows, int cols, __bf16* dst, int ld) {
  const int n4 = rows * cols / 4;
#pragma unroll 1
  for (int i0 = threadIdx.x; i0 < n4; i0 += U * blockDim.x) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float* src = W + 4 * (size_t)min(i0 + u * (int)blockDim.x, n4 - 1);
      v[u] = make_float4(src[0], src[1], src[2], src[3]);   // the caller's weights may be 4-byte aligned only
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * (int)blockDim.x;
      if (i >= n4) continue;
      const int r = 4 * i / cols, c = 4 * i - r * cols;
      bf16x2* d = reinterpret_cast<bf16x2*>(dst + r * ld + (PERM ? perm16(c) : c));
      d[0] = to_bf2(v[u].x, v[u].y);
      d[1] = to_bf2(v[u].z, v[u].w);
    }
  }
}

// Tiles (of 32 rows) a wave of the forward pass takes together: they share every A operand read from LDS.
constexpr int kPair = 2;

// The 16 values a lane holds of a tile, rounded to the next product's operands.
__device__ __forceinline__ void round_tile(const float (&v)[16], bf16x8 (&out)[2]) {
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf16x2 c = to_bf2(v[8 * p + 2 * t], v[8 * p + 2 * t + 1]);
      out[p][2 * t] = c[0];
      out[p][2 * t + 1] = c[1];
    }
}

// Bias, ReLU and rounding of one 32-neuron output tile mt: the next layer's operands, and bit r of
// the result set where register r's value is positive.
__device__ __forceinline__ unsigned hidden_epilogue(const floatx16& acc, const float* bias, int mt, int l,
                                                    bf16x8 (&out)[2]) {
  float v[16];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 b = *reinterpret_cast<const float4*>(bias + 32 * mt + 8 * q + 4 * (l >> 5));
    v[4 * q] = fmaxf(acc[4 * q] + b.x, 0.f);
    v[4 * q + 1] = fmaxf(acc[4 * q + 1] + b.y, 0.f);
    v[4 * q + 2] = fmaxf(acc[4 * q + 2] + b.z, 0.f);
    v[4 * q + 3] = fmaxf(acc[4 * q + 3] + b.w, 0.f);
  }
  unsigned mask = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) mask |= v[r] > 0.f ? 1u << r : 0u;
  round_tile(v, out);
  return mask;
}

// One hidden layer of a wave's G tiles: out = relu(W in + b), in and out as operands.
template <int G>
__device__ __forceinline__ void fused_hidden(const __bf16* w, const float* bias, const bf16x8 (&in)[G][4][2],
                                             bf16x8 (&out)[G][4][2], int l, unsigned (&mask)[G][4]) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const __bf16* wrow = w + (32 * mt + (l & 31)) * kLdH + 8 * (l >> 5);
    floatx16 acc[G] = {};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(wrow + 32 * q + 16 * p);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, in[g][q][p], acc[g], 0, 0, 0);
      }
#pragma unroll
    for (int g = 0; g < G; ++g) mask[g][mt] = hidden_epilogue(acc[g], bias, mt, l, out[g][mt]);
  }
}

// First and last layer's weights, biases and feature scales to LDS.
template <class S>
__device__ __forceinline__ void stage_small(S& sm, const float* W, const float* norm) {
  const MlpLayout L;
  const int tid = threadIdx.x;
  stage_weights<false, 2>(W + L.w1, kHidden, kFeat, sm.w1, kLd1);
  stage_weights<true, 1>(W + L.w4, kOut, kHidden, sm.w4, kLdH);
  for (int i = tid; i < kHidden; i += blockDim.x) {
    sm.b[i] = W[L.b1 + i];
    sm.b[kHidden + i] = W[L.b2 + i];
    sm.b[2 * kHidden + i] = W[L.b3 + i];
  }
  if (tid < kOut) sm.b[3 * kHidden + tid] = W[L.b4 + tid];
  if (tid < kNorm) sm.nrm[tid] = norm ? norm[tid] : (tid < kFeat ? 0.f : 1.f);
}

// The 8 features a lane holds of one sample, normalised and rounded.
template <class S>
__device__ __forceinline__ bf16x8 feature_operand(const S& sm, const float* x, int h) {
  float v[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = x[8 * h + t];
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = (v[t] - sm.nrm[8 * h + t]) * sm.nrm[kFeat + 8 * h + t];
  bf16x8 out;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const bf16x2 c = to_bf2(v[2 * t], v[2 * t + 1]);
    out[2 * t] = c[0];
    out[2 * t + 1] = c[1];
  }
  return out;
}

// The four layers on a wave's G tiles: the operands of the hidden layers in h1..h3 (two of them may be the
// same array), positive-value masks, and the output tile (rows 0..2; the others repeat row 2).
template <int G, class S>
__device__ __forceinline__ void network(const S& sm, const bf16x8 (&xb)[G], int l, bf16x8 (&h1)[G][4][2],
                                        bf16x8 (&h2)[G][4][2], bf16x8 (&h3)[G][4][2], unsigned (&m1)[G][4],
                                        unsigned (&m2)[G][4], unsigned (&m3)[G][4], floatx16 (&y)[G]) {
  const int h = l >> 5;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(sm.w1 + (32 * mt + (l & 31)) * kLd1 + 8 * h);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      floatx16 acc = {};
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xb[g], acc, 0, 0, 0);
      m1[g][mt] = hidden_epilogue(acc, sm.b, mt, l, h1[g][mt]);
    }
  }
  fused_hidden<G>(sm.w2, sm.b + kHidden, h1, h2, l, m2);
  fused_hidden<G>(sm.w3, sm.b + 2 * kHidden, h2, h3, l, m3);
  const __bf16* wrow = sm.w4 + min(l & 31, kOut - 1) * kLdH + 8 * h;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(wrow + 32 * q + 16 * p);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (q + p == 0) y[g] = floatx16{};
        y[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, h3[g][q][p], y[g], 0, 0, 0);
      }
    }
}

// Y = network(X) for `rows` rows.  norm != nullptr: X holds raw features, normalised on load.
// need != nullptr: 32-row tiles without a flagged row are skipped (their Y is left as is).
// What bounds it: the matrix cores (76 MFMA of 32 cycles per tile) against about 500 vector instructions of
// bias, ReLU and rounding; two tiles per wave share the weights' LDS reads and hide each other's chains,
// and rounding takes half an instruction per value (v_cvt_pk_bf16_f32) instead of six.  One million rows:
// 81 us a call (0.91 PFLOP/s of network arithmetic), 277 us with one tile per wave and rounding in integer code.
__global__ void __launch_bounds__(64 * kWaves, 2) k_mlp_fused(const float* W, const float* norm, const float* X,
                                                              long rows, const int* need, float* Y) {
  extern __shared__ __align__(16) unsigned char fsm_raw[];
  FusedSmem& S = *reinterpret_cast<FusedSmem*>(fsm_raw);
  const MlpLayout L;
  stage_weights<true, 8>(W + L.w2, kHidden, kHidden, S.w2, kLdH);
  stage_weights<true, 8>(W + L.w3, kHidden, kHidden, S.w3, kLdH);
  stage_small(S, W, norm);
  __syncthreads();

  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = l >> 5;
  const long npairs = ((rows + 31) / 32 + kPair - 1) / kPair;
  for (long pair = (long)blockIdx.x * kWaves + wave; pair < npairs; pair += (long)gridDim.x * kWaves) {
    long row[kPair];
    bool on[kPair];
    bool any = false;
#pragma unroll
    for (int g = 0; g < kPair; ++g) {
      row[g] = (pair * kPair + g) * 32 + (l & 31);
      on[g] = true;
      if (need) on[g] = __ballot(row[g] < rows && need[row[g]] != 0) != 0;
      any |= on[g];
    }
    if (!any) continue;
    bf16x8 xb[kPair];
#pragma unroll
    for (int g = 0; g < kPair; ++g)   // rows past the end repeat the last one, unused
      xb[g] = feature_operand(S, X + (row[g] < rows ? row[g] : rows - 1) * kFeat, h);
    bf16x8 ha[kPair][4][2], hb[kPair][4][2];
    unsigned mask[kPair][4];
    floatx16 acc[kPair];
    network<kPair>(S, xb, l, ha, hb, ha, mask, mask, mask, acc);
#pragma unroll
    for (int g = 0; g < kPair; ++g)
      if (h == 0 && on[g] && row[g] < rows)
        for (int k = 0; k < kOut; ++k) Y[row[g] * kOut + k] = acc[g][k] + S.b[3 * kHidden + k];
  }
}

void launch_mlp_fused(const float* W, const float* norm, const float* X, long rows, const int* need, float* Y,
                      hipStream_t s) {
  if (rows <= 0) return;
  const long npairs = ((rows + 31) / 32 + kPair - 1) / kPair;
  // two workgroups per CU (their LDS); more would stage the weights again
  const long blocks = std::min<long>((npairs + kWaves - 1) / kWaves, 512);
  hipLaunchKernelGGL(k_mlp_fused, dim3((unsigned)blocks), dim3(64 * kWaves), kFusedSmem, s, W, norm, X, rows, need, Y);
}

// ---------------------------------------------------------------------------
// Loss and gradient of a minibatch in two launches: k_mlp_grad takes up to 128 rows per workgroup (32 per wave)
// through the forward pass, the loss and the whole backward pass, and leaves the block's share of every
// weight gradient in the workgroup's slab and the rows' dz in memory; k_mlp_reduce adds the slabs in order, sums
// dz over the rows for the biases and, in training, applies Adam.  A wave's activations stay in its registers as
// bf16 operands; the weight gradients, which contract over rows, take their operands from LDS copies
// [neuron][row] of one layer at a time.  The backward products add their terms in natural order, 16 at a time
// (the bits of two products of 8), and rows are split as the weight gradients' sums always were, so training keeps
// its bits.
// ---------------------------------------------------------------------------
struct GradSmem {
  __bf16 w1[kHidden * kLd1];
  __bf16 w2[kHidden * kLdH];    // W2, then its transpose
  __bf16 w3[kHidden * kLdH];    // W3, then its transpose
  __bf16 w4[kOut * kLdH];
  alignas(16) float b[3 * kHidden + 4];
  float nrm[kNorm + 1];
  __bf16 dz[kHidden * kLdH];    // loss gradient of a layer's pre-activations [neuron][row]
  __bf16 hin[kHidden * kLdH];   // that layer's inputs [neuron][row]
  double e2[kWaves];
};
constexpr size_t kGradSmem = sizeof(GradSmem);
static_assert(kGradSmem <= 160 * 1024, "one workgroup's LDS");
static_assert(kWaves * 32 == kGradRows, "a wave takes 32 of a block's rows");

// A thread's 2 x 4 blocks of a 128 x 128 weight matrix.  A wave spans 8 block rows and 8 block columns, so that
// the loads are whole 128-byte lines and both LDS forms, rows and transposed rows, are free of bank conflicts.
constexpr int kBlocks = kHidden * kHidden / 8 / (64 * kWaves);
__device__ __forceinline__ int block_row(int u) {
  const int i = threadIdx.x + u * 64 * kWaves;
  return 2 * (((i >> 3) & 7) + 8 * (i >> 8));
}
__device__ __forceinline__ int block_col(int u) {
  const int i = threadIdx.x + u * 64 * kWaves;
  return 4 * ((i & 7) + 8 * ((i >> 6) & 3));
}
static_assert(kWaves == 4 && kBlocks == 8, "the block maps");

__device__ __forceinline__ void load_blocks(const float* W, float (&f)[kBlocks][8]) {
#pragma unroll
  for (int u = 0; u < kBlocks; ++u) {
    const float* src = W + block_row(u) * kHidden + block_col(u);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f[u][t] = src[t];
      f[u][4 + t] = src[kHidden + t];
    }
  }
}

// Rounded rows of W to LDS (columns permuted by perm16).
__device__ __forceinline__ void put_blocks(const float (&f)[kBlocks][8], __bf16* dst) {
#pragma unroll
  for (int u = 0; u < kBlocks; ++u)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      bf16x2* d = reinterpret_cast<bf16x2*>(dst + (block_row(u) + i) * kLdH + perm16(block_col(u)));
      d[0] = to_bf2(f[u][4 * i], f[u][4 * i + 1]);
      d[1] = to_bf2(f[u][4 * i + 2], f[u][4 * i + 3]);
    }
}

// From those rows to registers, and back as rows of the transpose.
__device__ __forceinline__ void read_blocks(const __bf16* src, bf16x4 (&w)[kBlocks][2]) {
#pragma unroll
  for (int u = 0; u < kBlocks; ++u)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      w[u][i] = *reinterpret_cast<const bf16x4*>(src + (block_row(u) + i) * kLdH + perm16(block_col(u)));
}
__device__ __forceinline__ void put_transposed(const bf16x4 (&w)[kBlocks][2], __bf16* dst) {
#pragma unroll
  for (int u = 0; u < kBlocks; ++u)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf16x2 c = {w[u][0][t], w[u][1][t]};
      *reinterpret_cast<bf16x2*>(dst + (block_col(u) + t) * kLdH + block_row(u)) = c;
    }
}

// A wave's operands of one layer to [neuron][row] form, rows past the end as zeros.
__device__ __forceinline__ void put_rows(__bf16* dst, const bf16x8 (&op)[4][2], int col, int h, bool valid) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int t = 0; t < 8; ++t)
        dst[(32 * mt + 16 * p + 8 * (t >> 2) + 4 * h + (t & 3)) * kLdH + col] = valid ? op[mt][p][t] : (__bf16)0.f;
}

typedef short shortx4 __attribute__((ext_vector_type(4)));

// acc + A B for 8 terms, lane l holding the terms 4 (l / 32) + t of its row of A and its column of B.
__device__ __forceinline__ floatx16 mfma8(bf16x4 a, bf16x4 b, floatx16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(shortx4, a), __builtin_bit_cast(shortx4, b), acc, 0,
                                                  0, 0);
}

// ReLU mask, store (at d, when there is a row, in the layout [column / 4][rows][4]) and rounding of one tile of dz.
__device__ __forceinline__ void dz_tile(const floatx16& acc, unsigned mask, int mt, int h, float* d, long rows,
                                        bf16x8 (&out)[2]) {
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = (mask >> r) & 1u ? acc[r] : 0.f;
  if (d) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(d + (8 * mt + 2 * q + h) * rows * 4) =
          make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  }
  round_tile(v, out);
}

// dz of the layer below from this layer's (operands din) through the transposed weights wt.
__device__ __forceinline__ void dz_below(const __bf16* wt, const bf16x8 (&din)[4][2], const unsigned (&mask)[4], int l,
                                         float* d, long rows, bf16x8 (&dout)[4][2]) {
  // The operands with k = 8 (l / 32) + t natural, from 4 (l / 32) + t of either 8: the upper lanes' first halves
  // change places with the lower lanes' second.  Products of 16 in natural order have the bits of two of 8.
  bf16x8 nat[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const uint4 u = __builtin_bit_cast(uint4, din[q][p]);
      const auto a = __builtin_amdgcn_permlane32_swap(u.x, u.z, false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(u.y, u.w, false, false);
      nat[q][p] = __builtin_bit_cast(bf16x8, make_uint4(a[0], b[0], a[1], b[1]));
    }
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const __bf16* wrow = wt + (32 * mt + (l & 31)) * kLdH + 8 * (l >> 5);
    floatx16 acc = {};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(wrow + 32 * q + 16 * p),
                                                      nat[q][p], acc, 0, 0, 0);
    dz_tile(acc, mask[mt], mt, l >> 5, d, rows, dout[mt]);
    __builtin_amdgcn_sched_barrier(0);   // one tile's operands in flight, not all four's
  }
}

// acc plus one 32 x 32 tile of dz hin^T over the block's rows; mrow, nrow: this lane's rows of the two operands.
__device__ __forceinline__ floatx16 row_product(const __bf16* mrow, const __bf16* nrow, floatx16 acc) {
#pragma unroll
  for (int k = 0; k < kGradRows; k += 16)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(mrow + k), *reinterpret_cast<const bf16x8*>(nrow + k), acc, 0, 0, 0);
  return acc;
}

// A lane's 16 values of a 32 x 32 tile of G (row stride ld), column c: zeros for a slab's first block of rows,
// else what the earlier blocks left; and back.
__device__ __forceinline__ floatx16 get_tile(const float* G, int ld, int row0, int c, int h, bool first) {
  const float* p = G + (row0 + 4 * h) * ld + c;
  floatx16 v = {};
  if (!first)
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = p[(8 * (r >> 2) + (r & 3)) * ld];
  return v;
}
__device__ __forceinline__ void put_tile(float* G, int ld, int row0, int c, int h, const floatx16& v) {
  float* p = G + (row0 + 4 * h) * ld + c;
#pragma unroll
  for (int r = 0; r < 16; ++r) p[(8 * (r >> 2) + (r & 3)) * ld] = v[r];
}

// The 128 x 128 weight gradient of a hidden layer: wave w takes the 32 inputs 32 w .. and all outputs.
__device__ __forceinline__ void hidden_wgrad(const GradSmem& S, float* G, int l, int wave, bool first) {
  const int h = l >> 5, c = 32 * wave + (l & 31);
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    put_tile(G, kHidden, 32 * mt, c, h,
             row_product(S.dz + (32 * mt + (l & 31)) * kLdH + 8 * h, S.hin + c * kLdH + 8 * h,
                         get_tile(G, kHidden, 32 * mt, c, h, first)));
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Rows idx[r] (or r) of feat and lab, normalised with norm (or as they are).  Workgroup b takes the blocks of
// `span` rows (at most kGradRows) b, b + gridDim.x, ...; its sums go to slab[b][MlpLayout] and partial[b] (squared
// errors), the rows' dz to dz[layer 1..3][kHidden / 4][rows][4] and dy[rows][kOut].
// What bounds it: latency of one wave per SIMD through ten dependent products, then LDS traffic of the
// [neuron][row] copies; activations never reach memory.  A minibatch of 4096 (32
// workgroups): 28 us and 7 us for the reduction; separate kernels per product, mask, sum and layer (21 launches,
// activations through memory) took 300 us.
__global__ void __launch_bounds__(64 * kWaves, 1) k_mlp_grad(const float* W, const float* norm, const float* feat,
                                                             const float* lab, const int* idx, long rows, int span,
                                                             float* slab, double* partial, float* dz, float* dy_out) {
  extern __shared__ __align__(16) unsigned char gsm_raw[];
  GradSmem& S = *reinterpret_cast<GradSmem*>(gsm_raw);
  const MlpLayout L;
  const int wave = threadIdx.x >> 6;
  const long nblk = (rows + span - 1) / span;
  float* G = slab + (size_t)blockIdx.x * kSlab;
  for (long blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const bool first = blk == blockIdx.x;
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));   // addresses are formed where they are used, not kept through the loop
    const int h = l >> 5;
    const int col = 32 * wave + (l & 31);   // this lane's row within the block
    {
      float f2[kBlocks][8], f3[kBlocks][8];
      load_blocks(W + L.w2, f2);
      load_blocks(W + L.w3, f3);
      stage_small(S, W, norm);
      put_blocks(f2, S.w2);
      put_blocks(f3, S.w3);
    }
    const long row = blk * span + col;
    const bool valid = row < rows && col < span;
    const long at = valid ? row : rows - 1;
    float* drow = valid ? dz + row * 4 : nullptr;
    const long layer = rows * kHidden;
    const long src = idx ? idx[at] : at;
    float target[kOut];
    for (int k = 0; k < kOut; ++k) target[k] = lab[src * kOut + k];
    __syncthreads();
    bf16x8 xb[1] = {feature_operand(S, feat + src * kFeat, h)};
    bf16x8 h1[1][4][2], h2[1][4][2], h3[1][4][2];
    unsigned m1[1][4], m2[1][4], m3[1][4];
    floatx16 y[1];
    network<1>(S, xb, l, h1, h2, h3, m1, m2, m3, y);
    if (!valid)
      for (int mt = 0; mt < 4; ++mt) m1[0][mt] = m2[0][mt] = m3[0][mt] = 0;
    // loss: the lower half of the lanes holds the outputs
    float dy[kOut];
    double e2 = 0.0;
#pragma unroll
    for (int k = 0; k < kOut; ++k) {
      const float d = (y[0][k] + S.b[3 * kHidden + k]) - target[k] * S.nrm[2 * kFeat + k];
      const bool on = valid & (h == 0);
      dy[k] = on ? 2.f * d / (float)(rows * kOut) : 0.f;
      e2 += on ? (double)d * d : 0.0;
    }
    for (int s = 32; s > 0; s >>= 1) e2 += __shfl_xor(e2, s);
    if (l == 0) S.e2[wave] = e2;
    // output layer: its inputs and dy to LDS; dz3 (= W4^T dy) needs no transposed copy
    const bf16x2 d01 = to_bf2(dy[0], dy[1]), d2 = to_bf2(dy[2], 0.f);
    const bf16x4 dyb = {d01[0], d01[1], d2[0], (__bf16)0.f};
    if (h == 0)
#pragma unroll
      for (int k = 0; k < kOut; ++k) S.dz[k * kLdH + col] = dyb[k];
    put_rows(S.hin, h3[0], col, h, valid);
    if (valid && h == 0)
#pragma unroll
      for (int k = 0; k < kOut; ++k) dy_out[row * kOut + k] = dy[k];
    __syncthreads();   // forward weights free, dy and h3 written
    {
      floatx16 acc = {};
      if (!first && h == 0)
#pragma unroll
        for (int k = 0; k < kOut; ++k) acc[k] = G[L.w4 + k * kHidden + col];
      acc = row_product(S.dz + min(l & 31, kOut - 1) * kLdH + 8 * h, S.hin + col * kLdH + 8 * h, acc);
      if (h == 0)
#pragma unroll
        for (int k = 0; k < kOut; ++k) G[L.w4 + k * kHidden + col] = acc[k];
      if (threadIdx.x == 0) partial[blockIdx.x] = (first ? 0.0 : partial[blockIdx.x]) + ((S.e2[0] + S.e2[1]) + (S.e2[2] + S.e2[3]));
    }
    bf16x4 w2[kBlocks][2], w3[kBlocks][2];
    read_blocks(S.w3, w3);
    read_blocks(S.w2, w2);
    bf16x4 w4t[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        w4t[mt][t] = t < kOut && h == 0 ? S.w4[t * kLdH + perm16(32 * mt + (l & 31))] : (__bf16)0.f;
    __syncthreads();   // dy, h3 and the weights' rows read
    put_transposed(w3, S.w3);
    put_transposed(w2, S.w2);
    bf16x8 dz3[4][2], dz2[4][2], dz1[4][2];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      floatx16 acc = {};
      acc = mfma8(w4t[mt], dyb, acc);
      dz_tile(acc, m3[0][mt], mt, h, drow ? drow + 2 * layer : nullptr, rows, dz3[mt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    put_rows(S.dz, dz3, col, h, true);
    put_rows(S.hin, h2[0], col, h, valid);
    __syncthreads();
    hidden_wgrad(S, G + L.w3, l, wave, first);
    __syncthreads();
    dz_below(S.w3, dz3, m2[0], l, drow ? drow + layer : nullptr, rows, dz2);
    put_rows(S.dz, dz2, col, h, true);
    put_rows(S.hin, h1[0], col, h, valid);
    __syncthreads();
    hidden_wgrad(S, G + L.w2, l, wave, first);
    __syncthreads();
    dz_below(S.w2, dz2, m1[0], l, drow, rows, dz1);
    put_rows(S.dz, dz1, col, h, true);
#pragma unroll
    for (int t = 0; t < 8; ++t) S.hin[(8 * h + t) * kLdH + col] = valid ? xb[0][t] : (__bf16)0.f;
    __syncthreads();
    const int feature = min(l & 31, kFeat - 1);
    const floatx16 acc = row_product(S.dz + col * kLdH + 8 * h, S.hin + feature * kLdH + 8 * h,
                                     get_tile(G + L.w1, kFeat, 32 * wave, feature, h, first));
    if ((l & 31) < kFeat) put_tile(G + L.w1, kFeat, 32 * wave, l & 31, h, acc);
    __syncthreads();
  }
}

// Weight gradients = sums of the slabs in order (kReduceGrid blocks), bias gradients = sums of dz over the rows, in
// the order of 256 strided sums and a tree (kBiasGrid blocks of 4 columns): to grad, or (p != nullptr) straight
// into an Adam step on p, m, v.  The first wave adds the squared errors: loss = sum / n.
constexpr unsigned kReduceGrid = (unsigned)((MlpLayout::total + 255) / 256);
constexpr unsigned kBiasGrid = 3 * kHidden / 4 + 1;   // the last block: the output layer's kOut columns
__global__ void __launch_bounds__(256) k_mlp_reduce(const float* slab, int slabs, const double* partial,
                                                    const float* dz, const float* dy, long rows, float* loss, float* grad,
                                                    float* p, float* m, float* v, float lr, float b1, float b2,
                                                    float eps, float c1, float c2) {
  __shared__ float sh[4][256];
  const MlpLayout L;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid < 64) {
    double s = 0.0;
    for (int b = tid; b < slabs; b += 64) s += partial[b];
    for (int k = 32; k > 0; k >>= 1) s += __shfl_xor(s, k);
    if (tid == 0) *loss = (float)(s / (double)(rows * kOut));
  }
  int i = -1;
  float gi = 0.f;
  if (blockIdx.x < kReduceGrid) {
    i = blockIdx.x * 256 + tid;
    const bool bias = (i >= L.b1 && i < L.w2) || (i >= L.b2 && i < L.w3) || (i >= L.b3 && i < L.w4) || i >= L.b4;
    if (bias) return;
#pragma unroll 16
    for (int b = 0; b < slabs; ++b) gi += slab[(size_t)b * kSlab + i];
  } else {
    const int g = blockIdx.x - kReduceGrid, layer = g / (kHidden / 4), c0 = 4 * (g % (kHidden / 4));
    const bool last = layer == 3;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (last) {
      for (long r = tid; r < rows; r += 256)
#pragma unroll
        for (int k = 0; k < kOut; ++k) s[k] += dy[r * kOut + k];
    } else {
      const float* d = dz + layer * rows * kHidden + c0 * rows;
#pragma unroll 16
      for (long r = tid; r < rows; r += 256) {
        const float4 q = *reinterpret_cast<const float4*>(d + r * 4);
        s[0] += q.x; s[1] += q.y; s[2] += q.z; s[3] += q.w;
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sh[k][tid] = s[k];
    __syncthreads();
    // a wave per column: the tree t + 128, t + 64, ..., t + 1
    const int c = tid >> 6, l = tid & 63;
    gi = (sh[c][l] + sh[c][l + 128]) + (sh[c][l + 64] + sh[c][l + 192]);
    for (int k = 32; k > 0; k >>= 1) gi += __shfl_down(gi, k);
    if (l != 0 || (last && c >= kOut)) return;
    i = (int)(layer == 0 ? L.b1 : layer == 1 ? L.b2 : layer == 2 ? L.b3 : L.b4) + (last ? 0 : c0) + c;
  }
  if (!p) {
    grad[i] = gi;
    return;
  }
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

void prepare_mlp() {
  (void)hipFuncSetAttribute((const void*)k_mlp_fused, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFusedSmem);
  (void)hipFuncSetAttribute((const void*)k_mlp_grad, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGradSmem);
}

static void launch_grad_blocks(const float* W, const float* norm, const float* feat, const float* lab, const int* idx,
                               long rows, const GradScratch& g, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)grad_slabs(rows)), dim3(64 * kWaves), kGradSmem, s, W, norm, feat, lab,
                     idx, rows, grad_span(rows), g.slab, g.partial, g.dz, g.dy);
}

void launch_mlp_grad(const float* W, const float* X, const float* Lab, long rows, float* grad, float* loss,
                     const GradScratch& g, hipStream_t s) {
  launch_grad_blocks(W, nullptr, X, Lab, nullptr, rows, g, s);
  hipLaunchKernelGGL(k_mlp_reduce, dim3(kReduceGrid + kBiasGrid), dim3(256), 0, s, g.slab, (int)grad_slabs(rows),
                     g.partial, g.dz, g.dy, rows, loss, grad, nullptr, nullptr, nullptr, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f);
}

void launch_mlp_train(float* W, const float* norm, const float* feat, const float* lab, const int* idx, long rows,
                      float* m, float* v, float lr, int t, float* loss, const GradScratch& g, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  launch_grad_blocks(W, norm, feat, lab, idx, rows, g, s);
  hipLaunchKernelGGL(k_mlp_reduce, dim3(kReduceGrid + kBiasGrid), dim3(256), 0, s, g.slab, (int)grad_slabs(rows),
                     g.partial, g.dz, g.dy, rows, loss, nullptr, W, m, v, lr, b1, b2, 1e-8f, c1, c2);
}

// per-block partial sums of (Y - L)^2 in fixed order
__global__ void k_mse(const float* Y, const float* L, long n, double* partial) {
  __shared__ double sh[256];
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  double e2 = 0.0;
  if (i < n) {
    const float d = Y[i] - L[i];
    e2 = (double)d * d;
  }
  sh[threadIdx.x] = e2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

__global__ void k_sum_partials(const double* partial, int nb, long n, float* loss) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int b = 0; b < nb; ++b) s += partial[b];
    *loss = (float)(s / (double)n);
  }
}

// rows idx of the data with feature / label normalisation
__global__ void k_gather_batch(const float* feat, const float* lab, const int* idx, int B, const float* norm,
                               float* X, float* Y) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= B) return;
  const long s = idx[r];
  for (int k = 0; k < kFeat; ++k) X[r * kFeat + k] = (feat[s * kFeat + k] - norm[k]) * norm[kFeat + k];
  for (int k = 0; k < 3; ++k) Y[r * 3 + k] = lab[s * 3 + k] * norm[2 * kFeat + k];
}

void mlp_loss(const float* Y, const float* Lab, long n, double* partial, float* loss, hipStream_t s) {
  const long m = 3 * n;
  const int nb = (int)((m + 255) / 256);
  hipLaunchKernelGGL(k_mse, dim3(nb), dim3(256), 0, s, Y, Lab, m, partial);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(1), 0, s, partial, nb, m, loss);
}

void launch_gather_batch(const float* feat, const float* lab, const int* idx, int B, const float* norm, float* X,
                         float* Y, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_batch, dim3((B + 255) / 256), dim3(256), 0, s, feat, lab, idx, B, norm, X, Y);
}

// ---------------------------------------------------------------------------
// per-contact features and labels (one thread per contact slot of every env)
// features: d0/dc, n.u~/dc, (h v - dobs).{n,t1,t2}/dc, s lambda0/dc (3), had-warm-start,
// mu, log10(Gbar_vv m_v), log10(m_v / 1 g), contacts on the vertex, (g.n) h^2/dc,
// (dobs.n)/dc, 1.
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_ws_features(DevBatch<T> B, const T* mu_env, float* feat, int* need) {
  const long slot = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= (long)B.n_envs * B.cap) return;
  const int e = (int)(slot / B.cap), jj = (int)(slot - (long)e * B.cap);
  float* f = feat + slot * kFeat;
  // empty slots and attachment rows (bilateral, no prediction) get no features
  if (jj >= B.ccount[e] || B.cobs[slot] >= kMaxObs) {
    for (int k = 0; k < kFeat; ++k) f[k] = 0.f;
    if (need) need[slot] = 0;
    return;
  }
  if (need) need[slot] = B.cnew[slot];
  const double dc = B.margin > 0 ? B.margin : 1e-3;
  const int vloc = B.cvert[slot];
  const int vi = B.voff[e] + vloc;
  const T* F = B.cframe + 9 * slot;
  const int o = e * kMaxObs + B.cobs[slot];
  double dob[3];
  for (int k = 0; k < 3; ++k) dob[k] = B.obs_move[o] != 0 ? B.h * B.obs_vel[3 * o + k] : 0.0;
  double ut[3], hv[3];
  for (int k = 0; k < 3; ++k) {
    ut[k] = (double)B.ut[(size_t)k * B.NV + vi];
    hv[k] = B.h * (double)B.v[(size_t)k * B.NV + vi] - dob[k];
  }
  const double m = (double)B.mass[vi];
  const double s = B.h * B.h / m;
  const T* G = B.G + B.goff[e];
  const double gvv = (double)G[(size_t)vloc * B.gld[e] + vloc];
  auto dotF = [&](int a, const double* w) {
    return (double)F[3 * a] * w[0] + (double)F[3 * a + 1] * w[1] + (double)F[3 * a + 2] * w[2];
  };
  int nc = 1;
  if (jj > 0 && B.cvert[slot - 1] == vloc) ++nc;
  if (jj + 1 < B.ccount[e] && B.cvert[slot + 1] == vloc) ++nc;
  const double g[3] = {B.g[0], B.g[1], B.g[2]};
  f[0] = (float)(B.cd0d[slot] / dc);
  f[1] = (float)(dotF(0, ut) / dc);
  f[2] = (float)(dotF(0, hv) / dc);
  f[3] = (float)(dotF(1, hv) / dc);
  f[4] = (float)(dotF(2, hv) / dc);
  f[5] = (float)(s * B.clam[3 * slot] / dc);
  f[6] = (float)(s * B.clam[3 * slot + 1] / dc);
  f[7] = (float)(s * B.clam[3 * slot + 2] / dc);
  f[8] = B.cnew[slot] ? 0.f : 1.f;
  f[9] = (float)mu_env[e];
  f[10] = (float)log10(fmax(gvv * m, 1e-30));
  f[11] = (float)log10(m / 1e-3);
  f[12] = (float)nc;
  f[13] = (float)(dotF(0, g) * B.h * B.h / dc);
  f[14] = (float)(dotF(0, dob) / dc);
  f[15] = 1.f;
}

// label: s (lambda - lambda_ws) / dc, the first contact solve's change of each
// contact's multipliers from its previous-step warm start (features 5..7 hold s lambda_ws / dc)
template <class T>
__global__ void k_ws_labels(DevBatch<T> B, const float* feat, float* lab) {
  const long slot = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= (long)B.n_envs * B.cap) return;
  const int e = (int)(slot / B.cap), jj = (int)(slot - (long)e * B.cap);
  float* y = lab + slot * 3;
  if (jj >= B.ccount[e] || B.cobs[slot] >= kMaxObs) { y[0] = y[1] = y[2] = 0.f; return; }
  const double dc = B.margin > 0 ? B.margin : 1e-3;
  const int vi = B.voff[e] + B.cvert[slot];
  const double s = B.h * B.h / (double)B.mass[vi];
  for (int k = 0; k < 3; ++k) y[k] = (float)(s * B.clam[3 * slot + k] / dc - (double)feat[slot * kFeat + 5 + k]);
}

// network output -> candidate multipliers (cone-projected) for the contact solve
template <class T>
__global__ void k_ws_candidates(DevBatch<T> B, const T* mu_env, const float* feat, const float* Y, const float* norm,
                                double* lam_ml) {
  const long slot = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= (long)B.n_envs * B.cap) return;
  const int e = (int)(slot / B.cap), jj = (int)(slot - (long)e * B.cap);
  if (jj >= B.ccount[e]) return;
  if (B.cobs[slot] >= kMaxObs) {   // attachment rows keep the plain start
    for (int k = 0; k < 3; ++k) lam_ml[3 * slot + k] = B.clam[3 * slot + k];
    return;
  }
  const double dc = B.margin > 0 ? B.margin : 1e-3;
  const int vi = B.voff[e] + B.cvert[slot];
  const double s = B.h * B.h / (double)B.mass[vi];
  double l[3];
  for (int k = 0; k < 3; ++k)
    l[k] = ((double)feat[slot * kFeat + 5 + k] + (double)Y[slot * 3 + k] / (double)norm[2 * kFeat + k]) * dc / s;
  // a non-finite prediction stays non-finite: the solve's merit test then rejects it
  l[0] = l[0] > 0.0 ? l[0] : (l[0] == l[0] ? 0.0 : l[0]);
  const double lt = sqrt(l[1] * l[1] + l[2] * l[2]), rho = (double)mu_env[e] * l[0];
  if (lt > rho) { const double f = lt > 0 ? rho / lt : 0.0; l[1] *= f; l[2] *= f; }
  for (int k = 0; k < 3; ++k) lam_ml[3 * slot + k] = l[k];
}

// per-column sum and sum of squares (FP64, fixed order), one block per column
__global__ void k_col_moments(const float* X, long rows, int cols, double* out) {
  __shared__ double s1[256], s2[256];
  const int c = blockIdx.x;
  double a = 0.0, q = 0.0;
  for (long r = threadIdx.x; r < rows; r += 256) {
    const double v = X[r * cols + c];
    a += v;
    q += v * v;
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = q;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) { s1[threadIdx.x] += s1[threadIdx.x + k]; s2[threadIdx.x] += s2[threadIdx.x + k]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) { out[2 * c] = s1[0]; out[2 * c + 1] = s2[0]; }
}

void launch_col_moments(const float* X, long rows, int cols, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_col_moments, dim3(cols), dim3(256), 0, s, X, rows, cols, out);
}

// coff[e] = number of active contacts in envs before e (coff[n_envs] = total)
__global__ void k_count_offsets(const int* ccount, int n_envs, int cap, int* coff) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    int s = 0;
    for (int e = 0; e < n_envs; ++e) {
      coff[e] = s;
      const int c = ccount[e];
      s += c < cap ? c : cap;
    }
    coff[n_envs] = s;
  }
}

template <class T>
__global__ void k_ws_compact(DevBatch<T> B, const int* coff, const float* feat, const float* lab, float* out_feat,
                             float* out_lab, long base) {
  const long slot = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= (long)B.n_envs * B.cap) return;
  const int e = (int)(slot / B.cap), jj = (int)(slot - (long)e * B.cap);
  if (jj >= B.ccount[e]) return;
  const long row = base + coff[e] + jj;
  for (int k = 0; k < kFeat; ++k) out_feat[row * kFeat + k] = feat[slot * kFeat + k];
  for (int k = 0; k < kOut; ++k) out_lab[row * kOut + k] = lab[slot * kOut + k];
}

template <class T>
void launch_ws_features(const DevBatch<T>& B, const T* mu_env, float* feat, int* need, hipStream_t s) {
  const long n = (long)B.n_envs * B.cap;
  hipLaunchKernelGGL(k_ws_features<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, B, mu_env, feat, need);
}
template <class T>
void launch_ws_labels(const DevBatch<T>& B, const float* feat, float* lab, hipStream_t s) {
  const long n = (long)B.n_envs * B.cap;
  hipLaunchKernelGGL(k_ws_labels<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, B, feat, lab);
}
template <class T>
void launch_ws_infer(const DevBatch<T>& B, const T* mu_env, const MlpBuffers& M, hipStream_t s) {
  const long n = (long)B.n_envs * B.cap;
  launch_mlp_fused(M.W, M.norm, M.feat, n, M.need, M.Y, s);
  hipLaunchKernelGGL(k_ws_candidates<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, B, mu_env, M.feat, M.Y,
                     M.norm, M.lam_ml);
}

template <class T>
void launch_ws_compact(const DevBatch<T>& B, const float* feat, const float* lab, float* out_feat, float* out_lab,
                       long base, int* coff, hipStream_t s) {
  const long n = (long)B.n_envs * B.cap;
  hipLaunchKernelGGL(k_count_offsets, dim3(1), dim3(64), 0, s, B.ccount, B.n_envs, B.cap, coff);
  hipLaunchKernelGGL(k_ws_compact<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, B, coff, feat, lab,
                     out_feat, out_lab, base);
}

#define INSTW(T)                                                                           \
  template void launch_ws_features<T>(const DevBatch<T>&, const T*, float*, int*, hipStream_t); \
  template void launch_ws_labels<T>(const DevBatch<T>&, const float*, float*, hipStream_t);             \
  template void launch_ws_infer<T>(const DevBatch<T>&, const T*, const MlpBuffers&, hipStream_t); \
  template void launch_ws_compact<T>(const DevBatch<T>&, const float*, const float*, float*, float*, long, int*, \
                                     hipStream_t);
INSTW(float)
INSTW(double)

}  // namespace flash
