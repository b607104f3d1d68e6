// Learned coarse closure: a per-node network on stencil-gathered fields that
// corrects a coarse Navier-Stokes right-hand side (trained on fine runs of
// the same method restricted to the coarse nodes).
//
// Network: x (148 gathered values + 1 node value, padded to 160) ->
// h1 = tanh(W1 x + b1) (128) -> h2 = tanh(W2 h1 + b2) (128) -> y = W3 h2 + b3
// (4, padded to 16). BF16 weights and activations, FP32 accumulation on the
// matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Two kernels, both from the state to their result in one launch: the forward
// pass, and a training pass that keeps the activations of a tile of samples in
// LDS and the parameter gradient in registers.
// Lane layout of the 16x16x32 instruction: lane l holds A[l%16][8(l/16)..+7],
// B[8(l/16)..+7][l%16] (so row l%16 of B^T) and D[4(l/16)..+3][l%16].
#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "model.hpp"

namespace {

constexpr int HID = 128, KIN = 160, NOUT = 16, NSLOT_MAX = 37;
constexpr int OW1 = 0, OB1 = OW1 + HID * KIN, OW2 = OB1 + HID, OB2 = OW2 + HID * HID, OW3 = OB2 + HID,
              OB3 = OW3 + NOUT * HID, NPARAM = OB3 + NOUT;
static_assert(NPARAM == RBFFD_CLOSURE_NPARAMS, "parameter layout");

typedef __attribute__((ext_vector_type(4))) float f4v;
typedef f4v f4u __attribute__((aligned(4)));  // a caller's rows of four floats, aligned as floats
typedef __attribute__((ext_vector_type(8))) __bf16 bf8v;

// ---- fused forward pass -------------------------------------------------
// One kernel from the state to the normalised correction. The products are
// computed transposed, H^T = W X^T: the weights are the A operand (packed in
// LDS as per-lane fragments, shared by every sample tile of the block) and
// the samples the B operand, so lane l always holds sample l%16 of its tile:
// the input fragment is gathered straight from the state, and a layer's
// accumulators (outputs 16t + 4(l/16) + i) become the next layer's B
// fragment without moving data between lanes, once the contraction index of
// the next weight matrix is permuted to that order (mlp_perm). The biases
// enter as the accumulator input of each output tile's first product.
constexpr int FR1 = 8 * 5, FR2 = 8 * 4, FR3 = 4, NFRAG = FR1 + FR2 + FR3;  // 16 B x 64 lanes each
constexpr int NBIAS = HID + HID + NOUT;
constexpr size_t MLP_LDS = static_cast<size_t>(NFRAG) * 64 * 16 + NBIAS * sizeof(float);

// Position p of a 32-wide contraction block j of layers 2 and 3 -> hidden unit.
__host__ __device__ constexpr int mlp_perm(int j, int p) {
  return 32 * j + ((p & 7) < 4 ? 4 * (p >> 3) + (p & 7) : 16 + 4 * (p >> 3) + (p & 7) - 4);
}

// frag[f][lane][q], f < FR1: W1 tile (t = f / 5, k-block j = f % 5); then W2
// tiles (t = f' / 4, j = f' % 4) and W3 (j) with permuted contraction index.
__global__ void frag_pack_kernel(const float *__restrict__ p, __bf16 *__restrict__ frag) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= NFRAG * 512) return;
  const int f = t >> 9, l = (t >> 3) & 63, q = t & 7;
  const int row = l & 15, pos = 8 * (l >> 4) + q;
  float v;
  if (f < FR1) {
    v = p[OW1 + (16 * (f / 5) + row) * KIN + 32 * (f % 5) + pos];
  } else if (f < FR1 + FR2) {
    const int g = f - FR1;
    v = p[OW2 + (16 * (g / 4) + row) * HID + mlp_perm(g % 4, pos)];
  } else {
    v = p[OW3 + row * HID + mlp_perm(f - FR1 - FR2, pos)];
  }
  frag[t] = static_cast<__bf16>(v);
}

// The activation; relu propagates NaN (IEEE maximum, one instruction).
template <int ACT> __device__ __forceinline__ float act_fn(float v) {
  if constexpr (ACT == RBFFD_ACT_RELU) {
    return __builtin_elementwise_maximum(v, 0.0f);
  } else {
    return tanhf(v);
  }
}

// Input fragment of contraction block j for one sample: slots 8j + 2g and
// 8j + 2g + 1 (four fields each). Branch-free: a slot past the stencil
// re-reads the node itself (difference 0); slot 37 carries the node value.
// `rows`: the sample's entry of row 2g of the neighbour table (place 0 of each
// node's members), `ye`: the state at this member.
__device__ __forceinline__ bf8v gather_block(const float4 *__restrict__ ye, const unsigned *__restrict__ rows, int64_t Na,
                                             float nodev, float4 inv, float4 own, int j, int slot0) {
  bf8v x;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float4 f = ye[rows[(8 * j + h) * Na]];
    const float4 b = j == 0 && slot0 + h == 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : own;
    float v0 = (f.x - b.x) * inv.x, v1 = (f.y - b.y) * inv.y, v2 = (f.z - b.z) * inv.z, v3 = (f.w - b.w) * inv.w;
    if (j == 4 && slot0 + 32 + h == NSLOT_MAX) v0 = nodev;
    x[4 * h + 0] = static_cast<__bf16>(v0);
    x[4 * h + 1] = static_cast<__bf16>(v1);
    x[4 * h + 2] = static_cast<__bf16>(v2);
    x[4 * h + 3] = static_cast<__bf16>(v3);
  }
  return x;
}

// Y[s][0..3] times out_scale for S samples (and bad[e] = stamp for members with a value that
// is not finite, unless bad is NULL), T tiles of 16 samples per wavefront; blocks of
// W wavefronts share one LDS copy of the weights; each XCD has a contiguous
// range of the units (tiles), which its blocks take in turns; OCC wavefronts
// per SIMD bound the registers. The launch shapes (T, W, OCC) rbffd_closure_tune chooses from
// are kMlpShapes; a sample's arithmetic is the same in every shape. Measured
// on 557,056 samples: one 16-wavefront block per compute unit at four
// wavefronts per SIMD and T = 1 is fastest (more wavefronts hide the gather
// latency better than larger tiles save LDS reads of the weight fragments).
// Bound by the chain gather - products - activations of each tile at four
// wavefronts per SIMD: of this launch's 50 us the matrix pipe is busy 37%, the
// vector unit 43% and LDS 46%, without bank conflicts (50%, 57% and 62% of the
// cycles in which a compute unit has a wavefront).
template <int T, int MLP_WAVES, int MLP_OCC, int ACT>
__global__ __launch_bounds__(64 * MLP_WAVES) __attribute__((amdgpu_waves_per_eu(MLP_OCC, MLP_OCC))) void
mlp_forward_kernel(
    const float *__restrict__ y, const unsigned *__restrict__ idx_t, int64_t Na, int E,
    const float *__restrict__ nodef, float4 inv, const __bf16 *__restrict__ frag_g, const float *__restrict__ params,
    float *__restrict__ Y, float4 out_scale, int64_t S, int *__restrict__ bad, int stamp) {
  extern __shared__ __attribute__((aligned(16))) unsigned char mlp_lds[];
  const bf8v *s_frag = reinterpret_cast<const bf8v *>(mlp_lds);
  float *s_bias = reinterpret_cast<float *>(mlp_lds + static_cast<size_t>(NFRAG) * 64 * 16);
  {
    const f4v *src = reinterpret_cast<const f4v *>(frag_g);
    f4v *dst = reinterpret_cast<f4v *>(mlp_lds);
    for (int k = threadIdx.x; k < NFRAG * 64; k += 64 * MLP_WAVES) dst[k] = src[k];
    for (int k = threadIdx.x; k < NBIAS; k += 64 * MLP_WAVES)
      s_bias[k] = k < HID ? params[OB1 + k] : (k < 2 * HID ? params[OB2 + k - HID] : params[OB3 + k - 2 * HID]);
  }
  __syncthreads();
  const f4v *s_b4 = reinterpret_cast<const f4v *>(s_bias);   // 4 consecutive biases per lane group
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int64_t units = (S + 16 * T - 1) / (16 * T);
  // XCD x = b % 8 takes a contiguous range of units, its blocks in turns, so
  // that they gather the same neighbours at the same time from its L2
  // (557,056 samples, 256 members: 58.0 -> 56.7 us against a range per block)
  const int64_t nb = gridDim.x, b = blockIdx.x, ng = nb < 8 ? 1 : 8, x = b % ng;
  const int64_t per = (units + ng - 1) / ng, nbx = (nb - x + ng - 1) / ng;
  const int64_t u_end = min(units, (x + 1) * per);
  for (int64_t u = x * per + (b / ng) * MLP_WAVES + wave; u < u_end; u += nbx * MLP_WAVES) {
    const int64_t base = u * 16 * T;
    // keeps the weight fragments' LDS reads inside the loop: hoisted out of
    // it as loop-invariant they would need 304 registers
    asm volatile("" ::: "memory");
    unsigned si[T], se[T];
    float4 own[T];
    float nodev[T];
#pragma unroll
    for (int tl = 0; tl < T; ++tl) {
      // (S < 2^28: 32-bit division)
      const unsigned s = static_cast<unsigned>(min(base + 16 * tl + r, S - 1));  // rows past S compute a copy, never stored
      si[tl] = s / static_cast<unsigned>(E);
      se[tl] = s - si[tl] * static_cast<unsigned>(E);
      own[tl] = reinterpret_cast<const float4 *>(y)[s];
      nodev[tl] = nodef[si[tl]];
    }
    // output tile outermost: only one tile's accumulators are live, so the
    // whole input (5 blocks) and both hidden fragments fit in 128 registers
    // and four wavefronts run per SIMD
    bf8v x[5][T];
#pragma unroll
    for (int j = 0; j < 5; ++j)
#pragma unroll
      for (int tl = 0; tl < T; ++tl)
        x[j][tl] = gather_block(reinterpret_cast<const float4 *>(y) + se[tl], idx_t + 2 * g * Na + si[tl], Na, nodev[tl],
                                inv, own[tl], j, 2 * g);
    bf8v hb[4][T];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      f4v acc[T];
      const f4v c0 = s_b4[4 * t + g];
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const bf8v a = s_frag[(t * 5 + j) * 64 + lane];
#pragma unroll
        for (int tl = 0; tl < T; ++tl)
          acc[tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x[j][tl], j == 0 ? c0 : acc[tl], 0, 0, 0);
      }
#pragma unroll
      for (int tl = 0; tl < T; ++tl)
#pragma unroll
        for (int i = 0; i < 4; ++i) hb[t >> 1][tl][4 * (t & 1) + i] = static_cast<__bf16>(act_fn<ACT>(acc[tl][i]));
    }
    bf8v hb2[4][T];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      f4v acc[T];
      const f4v c0 = s_b4[32 + 4 * t + g];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf8v a = s_frag[FR1 * 64 + (t * 4 + j) * 64 + lane];
#pragma unroll
        for (int tl = 0; tl < T; ++tl)
          acc[tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hb[j][tl], j == 0 ? c0 : acc[tl], 0, 0, 0);
      }
#pragma unroll
      for (int tl = 0; tl < T; ++tl)
#pragma unroll
        for (int i = 0; i < 4; ++i) hb2[t >> 1][tl][4 * (t & 1) + i] = static_cast<__bf16>(act_fn<ACT>(acc[tl][i]));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int tl = 0; tl < T; ++tl) hb[j][tl] = hb2[j][tl];
    // layer 3: one output tile, outputs 0..3 in the lanes of group 0
    f4v out[T];
    const f4v c3 = s_b4[64 + g];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bf8v a = s_frag[(FR1 + FR2 + j) * 64 + lane];
#pragma unroll
      for (int tl = 0; tl < T; ++tl)
        out[tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hb[j][tl], j == 0 ? c3 : out[tl], 0, 0, 0);
    }
    if (g == 0) {
#pragma unroll
      for (int tl = 0; tl < T; ++tl) {
        const int64_t s = base + 16 * tl + r;
        if (s < S) {
          *reinterpret_cast<f4u *>(Y + s * 4) = f4v{out[tl][0] * out_scale.x, out[tl][1] * out_scale.y,
                                                    out[tl][2] * out_scale.z, out[tl][3] * out_scale.w};
          if (bad && !(isfinite(out[tl][0]) && isfinite(out[tl][1]) && isfinite(out[tl][2]) && isfinite(out[tl][3])))
            bad[se[tl]] = stamp;  // (any such sample of the member writes the same)
        }
      }
    }
  }
}

// Matrix-core throughput probe: every wavefront runs `iters` rounds of four
// independent BF16 products on register operands (no memory traffic), of
// shape 16x16x32 (SHAPE 0) or 32x32x16 (SHAPE 1); each lane stores one sum so
// that none of them is dead.
template <int SHAPE> __global__ __launch_bounds__(256) void mfma_probe_kernel(float *__restrict__ out, int iters) {
  typedef __attribute__((ext_vector_type(16))) float f16v;
  const int tid = threadIdx.x;
  bf8v a, b;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    a[q] = static_cast<__bf16>(1.0f + 0.001f * static_cast<float>((tid + q) & 7));
    b[q] = static_cast<__bf16>(0.5f - 0.001f * static_cast<float>((tid * 3 + q) & 7));
  }
  float v = 0.0f;
  if constexpr (SHAPE == 0) {
    f4v acc[4] = {};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[u], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) v += acc[u][0] + acc[u][1] + acc[u][2] + acc[u][3];
  } else {
    f16v acc[4] = {};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[u], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) v += acc[u][0] + acc[u][5] + acc[u][10] + acc[u][15];
  }
  out[static_cast<int64_t>(blockIdx.x) * 256 + tid] = v;
}

// ---- fused training pass -----------------------------------------------
// Loss and parameter gradient in one persistent kernel: blocks of eight
// wavefronts (one block per compute unit) take tiles of 64 samples through
// gather, forward, loss, backward and the weight gradients without leaving
// LDS, and hold the whole gradient in matrix-core accumulators (at most 80
// registers per lane) over all their tiles. One partial gradient per block
// goes to memory; grad_reduce_kernel adds them in a fixed order.
//
// Products use v_mfma_f32_32x32x16_bf16 (twice the rate of 16x16x32): lane l
// holds A[l%32][8(l/32)..+7], B[8(l/32)..+7][l%32] and, in register i,
// D[8(i/4) + 4(l/32) + i%4][l%32]. Wavefront w owns hidden units
// 32 (w%4)..+31 and samples 32 (w/4)..+31 of each layer's output, and in the
// weight gradients the same hidden units and every second half of the
// columns. The layer outputs lie in LDS as [sample][unit], so the next layer
// reads rows (16 bytes a lane) and the weight gradients, which contract over
// the samples, read columns with the transposing LDS load; so do the
// products with W2 transposed, from the one copy of W2. Rows are 256 bytes;
// their 16-byte chunks are permuted by row (tr_sw) so that the reads of rows
// and of columns touch every bank once. The 8-byte stores of the activations,
// the 8-byte accesses of the back-propagation and the columns of dY meet
// others in a bank (two-way): 15% of the cycles in which LDS is active. Most of
// W1 stays in registers.
//
// Feature 150 (padding of the input row, where the network's W1 sees 0) is
// set to 1: its column of the W1 gradient is the gradient of b1. Likewise
// output 4 (padding) of dY in LDS is 1, and its row of a product with dH2 the
// gradient of b2.
//
// Bound by the matrix and LDS pipes at two wavefronts per SIMD. 417,792
// samples (192 members x 2,176 nodes): 164 us per call (150 us this kernel,
// 9 us the sum of the blocks' gradients), against 1,471 us with one launch per
// product and the activations, their transposes and atomic weight gradients in
// HBM. The matrix pipe is busy 27% of the launch, the vector unit 35%, LDS 38%
// (32%, 40% and 44% of the cycles in which a compute unit has a wavefront):
// what is left is the latency of the four phases between barriers.
constexpr int TR_S = 64, TR_WAVES = 8, TR_ONE = 150, TR_ONE_DY = 4;
constexpr int TR_W1_REG = 6;                          // W1 fragments in registers (of 10); the others in LDS
constexpr unsigned TR_ROWS = TR_S * 256;              // one [64][128] array
// arrays with 256-byte rows: inputs 0-127 of two tiles, H1, H2 (within the
// 64 KB that an LDS instruction's offset reaches), dH2, dH1, W2 (the next)
constexpr unsigned TR_XA = 0, TR_H1 = 2 * TR_ROWS, TR_H2 = 3 * TR_ROWS, TR_HI = 65536, TR_D2 = TR_HI,
                   TR_D1 = TR_D2 + TR_ROWS, TR_W2 = TR_D1 + TR_ROWS, TR_XB = TR_W2 + HID * 256,
                   TR_XB_TILE = TR_S * 64, TR_DY = TR_XB + 2 * TR_XB_TILE, TR_W3 = TR_DY + TR_S * 32,
                   TR_W1 = TR_W3 + 1024, TR_B = TR_W1 + 4 * (10 - TR_W1_REG) * 1024,
                   TR_LDS = TR_B + (2 * HID + 4) * 4;
static_assert(TR_H2 + TR_ROWS <= TR_HI, "arrays below the second base");
static_assert(TR_LDS <= 160 * 1024, "LDS of the training kernel");

typedef __attribute__((ext_vector_type(16))) float f16v;
typedef __attribute__((ext_vector_type(4))) __bf16 bf4v;
typedef __attribute__((ext_vector_type(4))) short s4v;
typedef __attribute__((ext_vector_type(2))) unsigned short u2s;

// LDS by byte address
template <typename T> __device__ __forceinline__ T lds_get(unsigned at) {
  return *(const __attribute__((address_space(3))) T *)(at);
}
template <typename T> __device__ __forceinline__ void lds_put(unsigned at, T v) {
  *(__attribute__((address_space(3))) T *)(at) = v;
}
// Byte offset of 16-byte chunk c of row `row`: of a 256-byte-row array, and of
// the inputs' last 32 features (64-byte rows). The permutation touches bits
// 4-7 (4-5), so (at ^ 16 c') is chunk c ^ c'.
__device__ __forceinline__ unsigned tr_at(int row, int c) {
  return row * 256 + ((c ^ (((row & 3) << 2) | ((row >> 2) & 3))) << 4);
}
__device__ __forceinline__ unsigned tr_at_x(int row, int c) { return row * 64 + ((c ^ ((row >> 2) & 3)) << 4); }

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// Eight 16-bit values of one column, from the four rows at p0 and the four at
// p1: in each group of 16 lanes, lane i gives the address of row i/4, columns
// 4 (i%4)..+3 and receives column i.
__device__ __forceinline__ bf8v read_tr2(unsigned p0, unsigned p1) {
  const s4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)(p0));
  const s4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)(p1));
  return __builtin_bit_cast(bf8v, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Back through the activation: d a'(h), rounded to BF16, from the BF16 values
// h. relu: h is 0 or above, or NaN, and the value is kept where h > 0: where
// h's bits lie in 1 .. 0x7f80, so that both h and 0x7f81 - h (saturating) are
// at least 1. (A NaN activation has derivative 0, as in a comparison.)
template <int ACT> __device__ __forceinline__ bf4v act_back(f4v d, bf4v h) {
  bf4v o;
  if constexpr (ACT == RBFFD_ACT_RELU) {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = static_cast<__bf16>(d[i]);
    typedef __attribute__((ext_vector_type(4))) unsigned short u4s;
    const u4s hb = __builtin_bit_cast(u4s, h), top = {0x7f81, 0x7f81, 0x7f81, 0x7f81};
    const u4s keep = __builtin_elementwise_min(__builtin_elementwise_min(hb, __builtin_elementwise_sub_sat(top, hb)),
                                               u4s{1, 1, 1, 1});
    return __builtin_bit_cast(bf4v, static_cast<u4s>(__builtin_bit_cast(u4s, o) * keep));
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = static_cast<float>(h[i]);
      o[i] = static_cast<__bf16>(d[i] * (1.0f - f * f));
    }
    return o;
  }
}

// Sum over the 32 lanes that share l/32.
template <typename T> __device__ __forceinline__ T half_sum(T v) {
  for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <int ACT>
__global__ __launch_bounds__(64 * TR_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void train_kernel(
    const float *__restrict__ y, const unsigned *__restrict__ idx_t, int Na, int E, const float *__restrict__ nodef,
    float4 inv, const __bf16 *__restrict__ w1, const __bf16 *__restrict__ w2, const __bf16 *__restrict__ w3,
    const float *__restrict__ params, const float *__restrict__ target, int S, float *__restrict__ part,
    double *__restrict__ part_loss) {
  extern __shared__ __attribute__((aligned(256))) unsigned char lds[];
  const unsigned L0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char *)lds));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), hg = wave & 3, sg = wave >> 2;
  const int lc = lane & 31, lh = lane >> 5;            // column and half of the 32x32 products
  // weights: W1 fragments in registers and LDS, W2, W3's four rows
  // ([16-byte chunk][row]) and the biases in LDS
  bf8v fw1[TR_W1_REG];
  const unsigned w1_at = L0 + TR_W1 + hg * (10 - TR_W1_REG) * 1024 + lane * 16;
#pragma unroll
  for (int kk = 0; kk < 10; ++kk) {
    bf8v v = *reinterpret_cast<const bf8v *>(w1 + (32 * hg + lc) * KIN + 16 * kk + 8 * lh);
    if (kk == TR_ONE / 16 && lh == (TR_ONE % 16) / 8) v[TR_ONE % 8] = static_cast<__bf16>(0.0f);
    if (kk < TR_W1_REG)
      fw1[kk < TR_W1_REG ? kk : 0] = v;
    else if (sg == 0)
      lds_put(w1_at + (kk - TR_W1_REG) * 1024, v);
  }
  bf8v fw3t;                                           // W3 transposed, contraction over the four outputs
#pragma unroll
  for (int q = 0; q < 8; ++q)
    fw3t[q] = q < 4 && lh == 0 ? w3[q * HID + 32 * hg + lc] : static_cast<__bf16>(0.0f);
  for (int t = tid; t < HID * 16; t += 64 * TR_WAVES)
    lds_put(L0 + TR_W2 + tr_at(t >> 4, t & 15), *reinterpret_cast<const bf8v *>(w2 + (t >> 4) * HID + 8 * (t & 15)));
  if (tid < 64) lds_put(L0 + TR_W3 + tid * 16, *reinterpret_cast<const bf8v *>(w3 + (tid & 3) * HID + 8 * (tid >> 2)));
  for (int t = tid; t < 2 * HID + 4; t += 64 * TR_WAVES)
    lds_put(L0 + TR_B + t * 4, t < HID ? params[OB1 + t] : (t < 2 * HID ? params[OB2 + t - HID] : params[OB3 + t - 2 * HID]));
  for (int t = tid; t < TR_S * 16; t += 64 * TR_WAVES)
    lds_put(L0 + TR_DY + t * 2, static_cast<__bf16>(t % 16 == TR_ONE_DY ? 1.0f : 0.0f));
  // the first tile has no predecessor: zeros stand in for its dH1 and inputs
  for (int t = tid; t < static_cast<int>(TR_ROWS / 16); t += 64 * TR_WAVES) {
    lds_put(L0 + TR_XA + TR_ROWS + t * 16, f4v{});
    lds_put(L0 + TR_D1 + t * 16, f4v{});
  }
  for (int t = tid; t < static_cast<int>(TR_XB_TILE / 16); t += 64 * TR_WAVES)
    lds_put(L0 + TR_XB + TR_XB_TILE + t * 16, f4v{});

  // tiles in XCD order: block b takes tiles of XCD b % 8's range, strided
  const int tiles = (S + TR_S - 1) / TR_S;
  const int nb = gridDim.x, ng = nb < 8 ? 1 : 8, xcd = blockIdx.x % ng;
  const int per = (tiles + ng - 1) / ng, step = (nb - xcd + ng - 1) / ng;
  const int t_end = min(tiles, (xcd + 1) * per);
  const float scale = 1.0f / static_cast<float>(4 * static_cast<int64_t>(S));

  // input gather: eight threads per sample, thread g8 the groups g8 + 8 j of
  // four features (group 0: the node, 37: its feature and the constant, others:
  // slot differences, 0 past the stencil). Samples past S repeat the last one;
  // their dY is 0.
  const int gs = tid >> 3, g8 = tid & 7;
  unsigned gj[5], gi = 0, ge = 0;
  auto gather_index = [&](int tile) {
    const unsigned s = min(tile * TR_S + gs, S - 1);
    gi = s / static_cast<unsigned>(E);
    ge = s - gi * E;
#pragma unroll
    for (int j = 0; j < 5; ++j) gj[j] = idx_t[static_cast<int64_t>(8 * j + g8) * Na + gi];
  };
  float4 gf[5], gown;
  float gnode;
  auto gather_load = [&]() {
    const float4 *ye = reinterpret_cast<const float4 *>(y) + ge;
    gown = ye[gi * static_cast<unsigned>(E)];
#pragma unroll
    for (int j = 0; j < 5; ++j) gf[j] = ye[gj[j]];
    gnode = nodef[gi];
  };
  unsigned xa_at = L0 + TR_XA + tr_at(gs, g8 >> 1) + 8 * (g8 & 1);      // group g8 + 8 j: chunk g8 / 2 + 4 j
  unsigned xb_at = L0 + TR_XB + tr_at_x(gs, g8 >> 1) + 8 * (g8 & 1);
  auto gather_store = [&](unsigned buf) {
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const float4 f = gf[j];
      const float4 b = j == 0 && g8 == 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : gown;
      bf4v x;
      x[0] = static_cast<__bf16>((f.x - b.x) * inv.x);
      x[1] = static_cast<__bf16>((f.y - b.y) * inv.y);
      x[2] = static_cast<__bf16>((f.z - b.z) * inv.z);
      x[3] = static_cast<__bf16>((f.w - b.w) * inv.w);
      if (j == 4) {
        x[0] = g8 == NSLOT_MAX - 32 ? static_cast<__bf16>(gnode) : x[0];
        x[TR_ONE - 4 * NSLOT_MAX] = static_cast<__bf16>(g8 == NSLOT_MAX - 32 ? 1.0f : static_cast<float>(x[TR_ONE - 4 * NSLOT_MAX]));
        lds_put(xb_at + buf * TR_XB_TILE, x);
      } else {
        lds_put((xa_at ^ (64 * j)) + buf * TR_ROWS, x);
      }
    }
  };

  // lane parts of the LDS addresses: this lane's row (sample, W2 row), chunk
  // lh + 2 kk = (at ^ 32 kk); its four units of a layer output, chunk 4 hg +
  // i4 = (at ^ 16 i4); its part of a column read of 16 rows, column tile
  // ct = (at ^ 64 ct), rows 16 kk on = at + 4096 kk
  const int srow = 32 * sg + lc, i16 = lane & 15, gq = lane >> 4;
  unsigned a_row = L0 + tr_at(srow, lh), a_rowx = L0 + TR_XB + tr_at_x(srow, lh), a_w2 = L0 + TR_W2 + tr_at(32 * hg + lc, lh);
  unsigned a_out = L0 + tr_at(srow, 4 * hg) + 8 * lh;
  const int r0 = 8 * (gq >> 1) + (i16 >> 2), c0 = 2 * (gq & 1) + ((i16 & 3) >> 1);
  unsigned a_c0 = L0 + tr_at(r0, c0) + 8 * (i16 & 1), a_c1 = L0 + tr_at(r0 + 4, c0) + 8 * (i16 & 1);
  unsigned a_x0 = L0 + TR_XB + tr_at_x(r0, c0) + 8 * (i16 & 1), a_x1 = L0 + TR_XB + tr_at_x(r0 + 4, c0) + 8 * (i16 & 1);
  // keeps the address arithmetic inside the tile loop: hoisted out of it, the
  // addresses of every read would be held in registers
  auto opaque = [&]() {
    asm volatile("" : "+v"(a_row), "+v"(a_rowx), "+v"(a_w2), "+v"(a_out), "+v"(a_c0), "+v"(a_c1));
  };
  auto bias16 = [&](unsigned at) {
    f16v a;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f4v v = lds_get<f4v>(L0 + at + 4 * (32 * hg + 8 * i4 + 4 * lh));
#pragma unroll
      for (int i = 0; i < 4; ++i) a[4 * i4 + i] = v[i];
    }
    return a;
  };
  auto store_act = [&](unsigned M, const f16v &acc) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      bf4v h;
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = static_cast<__bf16>(act_fn<ACT>(acc[4 * i4 + i]));
      lds_put((a_out ^ (16 * i4)) + M, h);
    }
  };
  // back through the activation whose values are in H
  auto store_back = [&](unsigned M, unsigned H, const f16v &d) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const unsigned at = a_out ^ (16 * i4);
      const bf4v h = lds_get<bf4v>(at + H);
      const f4v v = {d[4 * i4], d[4 * i4 + 1], d[4 * i4 + 2], d[4 * i4 + 3]};
      lds_put(at + M, act_back<ACT>(v, h));
    }
  };

  f16v dw1[3] = {}, dw2[2] = {};
  f4v dw3 = {}, db2 = {};
  float db3[4] = {};
  double loss = 0.0;
  // W1 gradient of one tile: column tiles 0, 1, 2 (sg = 0) or 3, 4 (sg = 1)
  auto grad_w1 = [&](unsigned buf) {
    const unsigned d0 = a_c0 ^ (64 * hg), d1 = a_c1 ^ (64 * hg);
    const unsigned p0 = (a_c0 ^ (sg ? 192 : 0)) + buf * TR_ROWS, p1 = (a_c1 ^ (sg ? 192 : 0)) + buf * TR_ROWS;
    const unsigned q0 = sg ? a_x0 + buf * TR_XB_TILE : (a_c0 ^ 64) + buf * TR_ROWS,
                   q1 = sg ? a_x1 + buf * TR_XB_TILE : (a_c1 ^ 64) + buf * TR_ROWS;
    const unsigned qs = sg ? 1024 : 4096;
    bf8v a[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      a[kk] = read_tr2(d0 + TR_D1 + kk * 4096, d1 + TR_D1 + kk * 4096);
      dw1[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], read_tr2(p0 + kk * 4096, p1 + kk * 4096), dw1[0], 0, 0, 0);
      dw1[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], read_tr2(q0 + kk * qs, q1 + kk * qs), dw1[1], 0, 0, 0);
    }
    if (sg == 0) {
      const unsigned t0 = (a_c0 ^ 128) + buf * TR_ROWS, t1 = (a_c1 ^ 128) + buf * TR_ROWS;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        dw1[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], read_tr2(t0 + kk * 4096, t1 + kk * 4096), dw1[2], 0, 0, 0);
    }
  };

  int tile = xcd * per + static_cast<int>(blockIdx.x) / ng;
  unsigned cur = 0;
  if (tile < t_end) {
    gather_index(tile);
    gather_load();
    gather_store(0);
    if (tile + step < t_end) gather_index(tile + step);
  }
  lds_barrier();
  for (; tile < t_end; tile += step) {
    const int next = tile + step;
    const bool more = next < t_end;
    opaque();
    // layer 1, and the previous tile's W1 gradient
    {
      f16v acc = bias16(TR_B);
#pragma unroll
      for (int kk = 0; kk < 10; ++kk) {
        const bf8v a = kk < TR_W1_REG ? fw1[kk < TR_W1_REG ? kk : 0] : lds_get<bf8v>(w1_at + (kk - TR_W1_REG) * 1024);
        const bf8v x = kk < 8 ? lds_get<bf8v>((a_row ^ (32 * kk)) + cur * TR_ROWS)
                              : lds_get<bf8v>((a_rowx ^ (32 * (kk - 8))) + cur * TR_XB_TILE);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, x, acc, 0, 0, 0);
      }
      store_act(TR_H1, acc);
    }
    if (more) gather_load();
    grad_w1(cur ^ 1);
    lds_barrier();
    const int s_own = tile * TR_S + srow;
    const f4v t_own = *reinterpret_cast<const f4u *>(target + static_cast<int64_t>(min(s_own, S - 1)) * 4);
    opaque();
    // layer 2
    {
      f16v acc = bias16(TR_B + HID * 4);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_get<bf8v>(a_w2 ^ (32 * kk)),
                                                      lds_get<bf8v>((a_row ^ (32 * kk)) + TR_H1), acc, 0, 0, 0);
      store_act(TR_H2, acc);
    }
    if (more) gather_store(cur ^ 1);
    if (next + step < t_end) gather_index(next + step);
    lds_barrier();
    opaque();
    // output layer (each wavefront for its samples), loss, and dH2
    {
      f16v acc = {};
      const unsigned a_w3 = L0 + TR_W3 + lh * 64 + (lane & 3) * 16;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_get<bf8v>(a_w3 + kk * 128),
                                                      lds_get<bf8v>((a_row ^ (32 * kk)) + TR_H2), acc, 0, 0, 0);
      bf8v dy = {};
      if (lh == 0 && s_own < S) {  // outputs 0-3: registers 0-3 of lanes 0-31
        const f4v b3 = lds_get<f4v>(L0 + TR_B + 2 * HID * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float d = acc[i] + b3[i] - t_own[i];
          const float g = 2.0f * d * scale;
          dy[i] = static_cast<__bf16>(g);
          if (hg == 0) {
            db3[i] += g;
            loss += static_cast<double>(d) * d;
          }
        }
      }
      if (hg == 0 && lh == 0) lds_put(L0 + TR_DY + srow * 32, __builtin_shufflevector(dy, dy, 0, 1, 2, 3));
      f16v d2 = {};
      d2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw3t, dy, d2, 0, 0, 0);
      store_back(TR_D2, TR_H2, d2);
    }
    lds_barrier();
    opaque();
    // dH1, and the W2, W3 and b2 gradients
    {
      f16v d1 = {};
      const unsigned w0 = (a_c0 ^ (64 * hg)) + TR_W2, w1c = (a_c1 ^ (64 * hg)) + TR_W2;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_tr2(w0 + kk * 4096, w1c + kk * 4096),
                                                     lds_get<bf8v>((a_row ^ (32 * kk)) + TR_D2), d1, 0, 0, 0);
      store_back(TR_D1, TR_H1, d1);
      const unsigned d0 = (a_c0 ^ (64 * hg)) + TR_D2, d1c = (a_c1 ^ (64 * hg)) + TR_D2;
      const unsigned h0 = (a_c0 ^ (128 * sg)) + TR_H1, h1 = (a_c1 ^ (128 * sg)) + TR_H1;
      const unsigned g0 = (a_c0 ^ (128 * sg + 64)) + TR_H1, g1 = (a_c1 ^ (128 * sg + 64)) + TR_H1;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bf8v a = read_tr2(d0 + kk * 4096, d1c + kk * 4096);
        dw2[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, read_tr2(h0 + kk * 4096, h1 + kk * 4096), dw2[0], 0, 0, 0);
        dw2[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, read_tr2(g0 + kk * 4096, g1 + kk * 4096), dw2[1], 0, 0, 0);
      }
    }
    // 16x16x32 products: lane l holds rows 8(l/16)..+7 of column l%16; this
    // wavefront's 16 hidden units
    {
      const int r = 8 * gq + (i16 >> 2), c = 2 * wave + ((i16 & 3) >> 1);
      const unsigned pd = L0 + TR_DY + r * 32 + 8 * (i16 & 3);
      const unsigned p0 = L0 + tr_at(r, c) + 8 * (i16 & 1), p1 = L0 + tr_at(r + 4, c) + 8 * (i16 & 1);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf8v a = read_tr2(pd + kk * 1024, pd + kk * 1024 + 128);
        const unsigned o = kk * 8192;
        dw3 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, read_tr2(p0 + o + TR_H2, p1 + o + TR_H2), dw3, 0, 0, 0);
        db2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, read_tr2(p0 + o + TR_D2, p1 + o + TR_D2), db2, 0, 0, 0);
      }
    }
    lds_barrier();
    cur ^= 1;
  }
  grad_w1(cur ^ 1);

  // this block's partial gradient, in the parameters' layout
  float *p = part + static_cast<int64_t>(blockIdx.x) * NPARAM;
  const int n1 = sg == 0 ? 3 : 2;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (c >= n1) break;
    const int f = 32 * (3 * sg + c) + lc;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int h = 32 * hg + 8 * (i / 4) + 4 * lh + i % 4;
      p[f == TR_ONE ? OB1 + h : OW1 + h * KIN + f] = dw1[c][i];
      if (f == TR_ONE) p[OW1 + h * KIN + f] = 0.0f;
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      p[OW2 + (32 * hg + 8 * (i / 4) + 4 * lh + i % 4) * HID + 32 * (2 * sg + c) + lc] = dw2[c][i];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = 4 * gq + i;
    p[OW3 + o * HID + 16 * wave + i16] = o < 4 ? dw3[i] : 0.0f;
    if (o == TR_ONE_DY) p[OB2 + 16 * wave + i16] = db2[i];
  }
  // b3 and the loss: lanes hold samples; the two sample halves meet in LDS
  lds_barrier();
  float *red = reinterpret_cast<float *>(lds);            // [2][4]
  double *redl = reinterpret_cast<double *>(lds + 64);    // [2]
  if (hg == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = half_sum(db3[i]);
      if (lane == 0) red[sg * 4 + i] = v;
    }
    loss = half_sum(loss);
    if (lane == 0) redl[sg] = loss;
  }
  lds_barrier();
  if (tid < NOUT) p[OB3 + tid] = tid < 4 ? red[tid] + red[4 + tid] : 0.0f;
  if (tid == 0) part_loss[blockIdx.x] = redl[0] + redl[1];
}

// grad = sum of the nb blocks' partial gradients (four interleaved slices per
// parameter, added in LDS), and the loss.
constexpr int GR_PARAMS = 64, GR_SLICES = 4;
__global__ __launch_bounds__(GR_PARAMS *GR_SLICES) void grad_reduce_kernel(const float *__restrict__ part,
                                                                          const double *__restrict__ part_loss, int nb,
                                                                          int64_t S, float *__restrict__ grad,
                                                                          double *__restrict__ loss) {
  __shared__ float s[GR_SLICES][GR_PARAMS];
  const int c = threadIdx.x % GR_PARAMS, sl = threadIdx.x / GR_PARAMS;
  const int q = blockIdx.x * GR_PARAMS + c;
  float v = 0.0f;
  if (q < NPARAM) {
#pragma unroll 8
    for (int b = sl; b < nb; b += GR_SLICES) v += part[static_cast<int64_t>(b) * NPARAM + q];
  }
  s[sl][c] = v;
  __syncthreads();
  if (sl == 0 && q < NPARAM) grad[q] = (s[0][c] + s[1][c]) + (s[2][c] + s[3][c]);
  if (blockIdx.x == 0) {  // one wavefront: nb / 64 values a lane, then across the lanes
    if (threadIdx.x < 64) {
      double l = 0.0;
      for (int b = threadIdx.x; b < nb; b += 64) l += part_loss[b];
      for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
      if (threadIdx.x == 0) *loss = l / (4.0 * static_cast<double>(S));
    }
  }
}

// BF16 copies of the weights for the training kernel.
__global__ void pack_kernel(const float *__restrict__ p, __bf16 *__restrict__ w1, __bf16 *__restrict__ w2,
                            __bf16 *__restrict__ w3) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < HID * KIN) w1[t] = static_cast<__bf16>(p[OW1 + t]);
  if (t < HID * HID) w2[t] = static_cast<__bf16>(p[OW2 + t]);
  if (t < NOUT * HID) w3[t] = static_cast<__bf16>(p[OW3 + t]);
}

__global__ void adam_kernel(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m1,
                            float *__restrict__ m2, int n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const float gt = g[t];
  const float a = b1 * m1[t] + (1.0f - b1) * gt;
  const float v = b2 * m2[t] + (1.0f - b2) * gt * gt;
  m1[t] = a;
  m2[t] = v;
  p[t] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
}

// y_active += dt * Y * out_scale, except for members whose correction is not
// finite (bad[e] = stamp); each of those counts once in `fallback`.
__global__ void apply_kernel(float *__restrict__ y, const float *__restrict__ Y, int64_t Na, int E,
                             const int *__restrict__ bad, int stamp, unsigned long long *__restrict__ fallback,
                             float4 out_scale, float dt) {
  const int64_t s = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= Na * E) return;
  const int e = static_cast<int>(s % E);
  if (bad[e] == stamp) {
    if (s < E) atomicAdd(fallback, 1ull);
    return;
  }
  float4 o = *reinterpret_cast<const float4 *>(y + s * 4);
  const float4 q = *reinterpret_cast<const float4 *>(Y + s * 4);
  o.x += dt * q.x * out_scale.x;
  o.y += dt * q.y * out_scale.y;
  o.z += dt * q.z * out_scale.z;
  o.w += dt * q.w * out_scale.w;
  *reinterpret_cast<float4 *>(y + s * 4) = o;
}

// The gather's neighbours, one row per group of four input features: row k the
// node of slot k (1 <= k < n), the node itself in every other row, so that a
// slot past the stencil gives the difference 0; as the place of the node's
// first member in the state (node E, below 2^32 for n_active E <= 2^28).
constexpr int NGROUP = KIN / 4;
__global__ void gather_rows_fill_kernel(const int *__restrict__ idx_t, int64_t Na, int n, unsigned E,
                                        unsigned *__restrict__ out) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= Na * NGROUP) return;
  const int64_t k = t / Na;
  out[t] = E * static_cast<unsigned>(k >= 1 && k < n ? idx_t[t] : static_cast<int>(t - k * Na));
}

__global__ void f64_to_f32_kernel(const double *__restrict__ a, int64_t n, float *__restrict__ b) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t < n) b[t] = static_cast<float>(a[t]);
}

}  // namespace

struct rbffd_closure {
  rbffd_model *model = nullptr;
  int64_t max_s = 0;
  float4 inv_in{}, out_sc{};
  DevBuf params, grad, m1, m2, nodef, idx;
  DevBuf w1, w2, w3;                                 // BF16 weights
  DevBuf part, part_loss;                            // training: each block's partial gradient and loss
  DevBuf frag, Yc;                                   // fused forward: packed weights, Y [S][4]
  DevBuf loss, bad, fallback;                        // bad: per member, the step (from 1) of the last bad correction
  int64_t step = 0;
  int act = RBFFD_ACT_TANH;
  int shape = 0;  // fused forward launch shape (rbffd_closure_tune)
};

namespace {

// Loss and parameter gradient (into cl->grad) for targets T [S][4]: one block
// per compute unit, fewer when there are fewer tiles.
int gradient(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, const float *T, int64_t S) {
  hipStream_t s = ctx->stream;
  rbffd_model *m = cl->model;
  const int nb = static_cast<int>(std::min<int64_t>(ctx->n_cu, (S + TR_S - 1) / TR_S));
  auto kern = cl->act == RBFFD_ACT_RELU ? train_kernel<RBFFD_ACT_RELU> : train_kernel<RBFFD_ACT_TANH>;
  kern<<<nb, 64 * TR_WAVES, TR_LDS, s>>>(static_cast<const float *>(state), cl->idx.as<unsigned>(), static_cast<int>(m->Na),
                                         m->E, cl->nodef.as<float>(), cl->inv_in, cl->w1.as<__bf16>(),
                                         cl->w2.as<__bf16>(), cl->w3.as<__bf16>(), cl->params.as<float>(), T,
                                         static_cast<int>(S), cl->part.as<float>(), cl->part_loss.as<double>());
  grad_reduce_kernel<<<grid_for(NPARAM, GR_PARAMS), GR_PARAMS * GR_SLICES, 0, s>>>(
      cl->part.as<float>(), cl->part_loss.as<double>(), nb, S, cl->grad.as<float>(), cl->loss.as<double>());
  RBFFD_HIP(ctx, hipGetLastError());
  return RBFFD_OK;
}

void repack(rbffd_closure *cl, hipStream_t s) {
  pack_kernel<<<grid_for(HID * KIN, 256), 256, 0, s>>>(cl->params.as<float>(), cl->w1.as<__bf16>(), cl->w2.as<__bf16>(),
                                                        cl->w3.as<__bf16>());
  frag_pack_kernel<<<grid_for(NFRAG * 512, 256), 256, 0, s>>>(cl->params.as<float>(), cl->frag.as<__bf16>());
}

struct MlpShape {
  int T, waves, occ;
};
constexpr MlpShape kMlpShapes[] = {{1, 16, 4}, {1, 8, 4}, {1, 4, 4}, {2, 8, 2}, {2, 4, 2}};
constexpr int kNumMlpShapes = sizeof(kMlpShapes) / sizeof(kMlpShapes[0]);

template <int S, int ACT> auto mlp_kernel() {
  return mlp_forward_kernel<kMlpShapes[S].T, kMlpShapes[S].waves, kMlpShapes[S].occ, ACT>;
}

template <int S> void set_mlp_lds_shape(bool &ok) {
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void *>(mlp_kernel<S, RBFFD_ACT_RELU>()),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(MLP_LDS)) == hipSuccess;
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void *>(mlp_kernel<S, RBFFD_ACT_TANH>()),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(MLP_LDS)) == hipSuccess;
}

void set_mlp_lds(bool &ok) {
  set_mlp_lds_shape<0>(ok);
  set_mlp_lds_shape<1>(ok);
  set_mlp_lds_shape<2>(ok);
  set_mlp_lds_shape<3>(ok);
  set_mlp_lds_shape<4>(ok);
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void *>(train_kernel<RBFFD_ACT_RELU>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, TR_LDS) == hipSuccess;
  ok = ok && hipFuncSetAttribute(reinterpret_cast<const void *>(train_kernel<RBFFD_ACT_TANH>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, TR_LDS) == hipSuccess;
}

// Fused forward pass into Y [S][4], times sc, in launch shape SH. Resident blocks per
// compute unit: as many as LDS (160 KB, 77 KB of packed weights each) and the
// SIMDs' wavefront slots allow; the grid is one wave of them.
template <int SH>
void launch_forward(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, int64_t S, float *Y, float4 sc, int *bad,
                    int stamp) {
  constexpr MlpShape sh = kMlpShapes[SH];
  rbffd_model *m = cl->model;
  constexpr int per_cu = std::min<int>(static_cast<int>((160 * 1024) / MLP_LDS), 4 * sh.occ / sh.waves);
  static_assert(per_cu >= 1, "fused forward launch shape");
  const int64_t units = (S + 16 * sh.T - 1) / (16 * sh.T);
  const unsigned nb = static_cast<unsigned>(
      std::max<int64_t>(1, std::min<int64_t>(static_cast<int64_t>(ctx->n_cu) * per_cu, (units + sh.waves - 1) / sh.waves)));
  auto kern = cl->act == RBFFD_ACT_RELU ? mlp_kernel<SH, RBFFD_ACT_RELU>() : mlp_kernel<SH, RBFFD_ACT_TANH>();
  kern<<<nb, 64 * sh.waves, MLP_LDS, ctx->stream>>>(static_cast<const float *>(state), cl->idx.as<unsigned>(), m->Na,
                                                    m->E, cl->nodef.as<float>(), cl->inv_in, cl->frag.as<__bf16>(),
                                                    cl->params.as<float>(), Y, sc, S, bad, stamp);
}

const float4 kOne = make_float4(1.0f, 1.0f, 1.0f, 1.0f);

int forward_fused(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, int64_t S, float *Y, float4 sc,
                  int *bad = nullptr, int stamp = 0) {
  switch (cl->shape) {
    case 1: launch_forward<1>(ctx, cl, state, S, Y, sc, bad, stamp); break;
    case 2: launch_forward<2>(ctx, cl, state, S, Y, sc, bad, stamp); break;
    case 3: launch_forward<3>(ctx, cl, state, S, Y, sc, bad, stamp); break;
    case 4: launch_forward<4>(ctx, cl, state, S, Y, sc, bad, stamp); break;
    default: launch_forward<0>(ctx, cl, state, S, Y, sc, bad, stamp); break;
  }
  RBFFD_HIP(ctx, hipGetLastError());
  return RBFFD_OK;
}

}  // namespace

int closure_create(rbffd_ctx *ctx, rbffd_model *m, const rbffd_closure_desc *d, rbffd_closure **out) {
  if (m->physics != RBFFD_PHYS_NS || m->fdt != RBFFD_F32)
    return rbffd_fail(ctx, RBFFD_EINVAL, "the closure needs a Navier-Stokes model with FP32 fields");
  if (m->n > NSLOT_MAX) return rbffd_fail(ctx, RBFFD_EINVAL, "the closure takes stencils of at most 37 nodes");
  if (!d->init_params || !d->node_feature) return rbffd_fail(ctx, RBFFD_EINVAL, "null closure input");
  if (d->activation != RBFFD_ACT_TANH && d->activation != RBFFD_ACT_RELU)
    return rbffd_fail(ctx, RBFFD_EINVAL, "activation must be RBFFD_ACT_TANH or RBFFD_ACT_RELU");
  const int64_t S = m->Na * m->E;
  if (d->max_samples < S || d->max_samples > (int64_t(1) << 28))
    return rbffd_fail(ctx, RBFFD_EINVAL, "max_samples must cover n_active * E (%lld)", (long long)S);
  for (int c = 0; c < 4; ++c)
    if (!(d->in_scale[c] > 0.0f) || !(d->out_scale[c] > 0.0f))
      return rbffd_fail(ctx, RBFFD_EINVAL, "scales must be positive");
  auto *cl = new (std::nothrow) rbffd_closure();
  if (!cl) return rbffd_fail(ctx, RBFFD_ENOMEM, "host allocation");
  cl->model = m;
  cl->act = d->activation;
  cl->max_s = d->max_samples;
  cl->inv_in = make_float4(1.0f / d->in_scale[0], 1.0f / d->in_scale[1], 1.0f / d->in_scale[2], 1.0f / d->in_scale[3]);
  cl->out_sc = make_float4(d->out_scale[0], d->out_scale[1], d->out_scale[2], d->out_scale[3]);
  const size_t Sx = static_cast<size_t>(cl->max_s), b2 = 2, n_cu = static_cast<size_t>(ctx->n_cu);
  bool ok = cl->params.alloc(4 * NPARAM) == hipSuccess && cl->grad.alloc(4 * NPARAM) == hipSuccess &&
            cl->m1.alloc(4 * NPARAM) == hipSuccess && cl->m2.alloc(4 * NPARAM) == hipSuccess &&
            cl->nodef.alloc(4 * m->Na) == hipSuccess && cl->idx.alloc(4 * m->Na * NGROUP) == hipSuccess &&
            cl->w1.alloc(b2 * HID * KIN) == hipSuccess && cl->w2.alloc(b2 * HID * HID) == hipSuccess &&
            cl->w3.alloc(b2 * NOUT * HID) == hipSuccess && cl->part.alloc(4 * NPARAM * n_cu) == hipSuccess &&
            cl->part_loss.alloc(8 * n_cu) == hipSuccess && cl->loss.alloc(8) == hipSuccess &&
            cl->bad.alloc(4 * m->E) == hipSuccess && cl->fallback.alloc(8) == hipSuccess && cl->frag.alloc(b2 * NFRAG * 512) == hipSuccess &&
            cl->Yc.alloc(4 * Sx * 4) == hipSuccess;
  if (!ok) {
    delete cl;
    return rbffd_fail(ctx, RBFFD_ENOMEM, "device allocation (closure)");
  }
  bool lds_ok = true;
  set_mlp_lds(lds_ok);
  if (!lds_ok) {
    delete cl;
    return rbffd_fail(ctx, RBFFD_EDEVICE, "closure: LDS size of the fused kernels");
  }
  hipStream_t s = ctx->stream;
  bool cp_ok = hipMemcpyAsync(cl->params.p, d->init_params, 4 * NPARAM, hipMemcpyDeviceToDevice, s) == hipSuccess &&
               hipMemsetAsync(cl->m1.p, 0, 4 * NPARAM, s) == hipSuccess &&
               hipMemsetAsync(cl->m2.p, 0, 4 * NPARAM, s) == hipSuccess;
  if (!cp_ok) {
    delete cl;
    return rbffd_fail(ctx, RBFFD_EDEVICE, "closure set-up copies");
  }
  f64_to_f32_kernel<<<grid_for(m->Na, 256), 256, 0, s>>>(d->node_feature, m->Na, cl->nodef.as<float>());
  gather_rows_fill_kernel<<<grid_for(m->Na * NGROUP, 256), 256, 0, s>>>(m->idx_t.as<int>(), m->Na, m->n,
                                                                      static_cast<unsigned>(m->E), cl->idx.as<unsigned>());
  repack(cl, s);
  const hipError_t e_launch = hipGetLastError();
  const hipError_t e_sync = hipStreamSynchronize(s);
  if (e_launch != hipSuccess || e_sync != hipSuccess) {
    delete cl;
    return rbffd_fail(ctx, RBFFD_EDEVICE, "closure set-up: launches %s, synchronisation %s",
                      hipGetErrorString(e_launch), hipGetErrorString(e_sync));
  }
  *out = cl;
  return RBFFD_OK;
}

int closure_destroy(rbffd_closure *cl) {
  delete cl;
  return RBFFD_OK;
}

float *closure_params(rbffd_closure *cl) { return cl->params.as<float>(); }

int closure_forward(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, float *out) {
  const int64_t S = cl->model->Na * cl->model->E;
  return forward_fused(ctx, cl, state, S, out, cl->out_sc);
}

// Time every launch shape of the fused forward kernel on `state` (one
// untimed call, then three timed ones each) and keep the fastest; with
// *chosen >= 0 on entry, time and keep that shape only.
int closure_tune(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, int *chosen, double *best_us) {
  const int64_t S = cl->model->Na * cl->model->E;
  if (*chosen >= kNumMlpShapes) return rbffd_fail(ctx, RBFFD_EINVAL, "closure shape %d outside -1..%d", *chosen,
                                                  kNumMlpShapes - 1);
  const int first = *chosen >= 0 ? *chosen : 0, last = *chosen >= 0 ? *chosen : kNumMlpShapes - 1;
  hipEvent_t e0, e1;
  RBFFD_HIP(ctx, hipEventCreate(&e0));
  RBFFD_HIP(ctx, hipEventCreate(&e1));
  int best = first;
  double best_t = -1.0;
  int rc = RBFFD_OK;
  for (int sh = first; sh <= last && rc == RBFFD_OK; ++sh) {
    cl->shape = sh;
    rc = forward_fused(ctx, cl, state, S, cl->Yc.as<float>(), kOne);
    if (rc) break;
    if (hipEventRecord(e0, ctx->stream) != hipSuccess) rc = RBFFD_EDEVICE;
    for (int r = 0; r < 3 && rc == RBFFD_OK; ++r) rc = forward_fused(ctx, cl, state, S, cl->Yc.as<float>(), kOne);
    float ms = 0.0f;
    if (rc == RBFFD_OK && (hipEventRecord(e1, ctx->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                           hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
      rc = rbffd_fail(ctx, RBFFD_EDEVICE, "closure tuning: event timing");
    const double us = 1e3 * ms / 3.0;
    if (rc == RBFFD_OK && (best_t < 0.0 || us < best_t)) {
      best_t = us;
      best = sh;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  cl->shape = best;
  if (rc) return rc;
  *chosen = best;
  *best_us = best_t;
  return RBFFD_OK;
}

int closure_gradient(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, const float *target, float *grad,
                     double *loss) {
  const int64_t S = cl->model->Na * cl->model->E;
  int rc = gradient(ctx, cl, state, target, S);
  if (rc) return rc;
  if (grad) RBFFD_HIP(ctx, hipMemcpyAsync(grad, cl->grad.p, 4 * NPARAM, hipMemcpyDeviceToDevice, ctx->stream));
  RBFFD_HIP(ctx, hipMemcpyAsync(loss, cl->loss.p, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
  RBFFD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return RBFFD_OK;
}

int closure_train_step(rbffd_ctx *ctx, rbffd_closure *cl, const void *state, const float *target, double lr,
                       double *loss) {
  int rc = closure_gradient(ctx, cl, state, target, nullptr, loss);
  if (rc) return rc;
  cl->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - powf(b1, static_cast<float>(cl->step)), c2 = 1.0f - powf(b2, static_cast<float>(cl->step));
  adam_kernel<<<grid_for(NPARAM, 256), 256, 0, ctx->stream>>>(cl->params.as<float>(), cl->grad.as<float>(),
                                                              cl->m1.as<float>(), cl->m2.as<float>(), NPARAM,
                                                              static_cast<float>(lr), b1, b2, 1e-8f, c1, c2);
  repack(cl, ctx->stream);
  RBFFD_HIP(ctx, hipGetLastError());
  return RBFFD_OK;
}

int closure_step(rbffd_ctx *ctx, rbffd_closure *cl, void *state, double *t, double dt, int64_t n_steps, int tableau,
                 int64_t *n_fallback) {
  rbffd_model *m = cl->model;
  const int64_t S = m->Na * m->E;
  hipStream_t s = ctx->stream;
  RBFFD_HIP(ctx, hipMemsetAsync(cl->bad.p, 0, cl->bad.bytes, s));
  RBFFD_HIP(ctx, hipMemsetAsync(cl->fallback.p, 0, 8, s));
  for (int64_t k = 0; k < n_steps; ++k) {
    const int stamp = static_cast<int>(k % INT32_MAX) + 1;
    int rc = model_ghost(ctx, m, state);
    if (!rc) rc = forward_fused(ctx, cl, state, S, cl->Yc.as<float>(), kOne, cl->bad.as<int>(), stamp);  // correction of the state before the step
    if (!rc) rc = model_step(ctx, m, state, t, dt, 1, tableau, true);
    if (rc) return rc;
    apply_kernel<<<grid_for(S, 256), 256, 0, s>>>(static_cast<float *>(state), cl->Yc.as<float>(), m->Na, m->E,
                                                  cl->bad.as<int>(), stamp, cl->fallback.as<unsigned long long>(),
                                                  cl->out_sc, static_cast<float>(dt));
    RBFFD_HIP(ctx, hipGetLastError());
  }
  if (n_fallback) {
    unsigned long long fb = 0;
    RBFFD_HIP(ctx, hipMemcpyAsync(&fb, cl->fallback.p, 8, hipMemcpyDeviceToHost, s));
    RBFFD_HIP(ctx, hipStreamSynchronize(s));
    *n_fallback = static_cast<int64_t>(fb);
  }
  return RBFFD_OK;
}

// Launch the matrix-core probe: four 256-thread blocks per compute unit.
int mfma_probe(rbffd_ctx *ctx, int shape, float *out, int64_t n_out, int iters, int64_t *flops) {
  const int64_t blocks = 4 * static_cast<int64_t>(ctx->n_cu);
  if (!out || iters < 1 || (shape != 0 && shape != 1) || n_out < blocks * 256)
    return rbffd_fail(ctx, RBFFD_EINVAL, "mfma probe: needs shape 0 or 1, iters >= 1 and %lld output floats",
                      static_cast<long long>(blocks * 256));
  if (shape == 0)
    mfma_probe_kernel<0><<<static_cast<unsigned>(blocks), 256, 0, ctx->stream>>>(out, iters);
  else
    mfma_probe_kernel<1><<<static_cast<unsigned>(blocks), 256, 0, ctx->stream>>>(out, iters);
  RBFFD_HIP(ctx, hipGetLastError());
  // 4 wavefronts per block, 4 products per round of 16 x 16 x 32 or 32 x 32 x 16 multiply-adds
  const int64_t per = shape == 0 ? 2 * 16 * 16 * 32 : 2 * 32 * 32 * 16;
  *flops = blocks * 4 * static_cast<int64_t>(iters) * 4 * per;
  return RBFFD_OK;
}
