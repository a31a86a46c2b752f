// aa_mlp.hip -- the mixing-weight network of the learned-guarded AA step.
//
// 230 -> 256 -> 256 -> 256 -> 21 (padded to 256 in / 64 out), GELU (erf form),
// BF16 operands on the matrix cores (gfx950's v_mfma_f32_16x16x32_bf16) with
// FP32 accumulation, FP32 master weights, Adam.  The network is small and its
// layers depend on each other, so what bounds it is launches and the latency
// of each, not the matrix cores: a forward pass is one launch (k_mlp_forward,
// 16 rows per workgroup, activations in LDS, weights straight from the L2 in
// operand order), a backward pass two (k_mlp_backward: the chain of dZ;
// k_mlp_grads: every weight and bias gradient).
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <new>
#include <vector>

#include "aa_device.h"

namespace aa {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Operand and result layout of v_mfma_f32_16x16x32_bf16: lane l supplies
// A[l % 16][8 (l / 16) + e] and B[8 (l / 16) + e][l % 16], e < 8, and
// register r of its result holds D[mfma_row(l, r)][l % 16].
__device__ __forceinline__ int mfma_row(int lane, int r) { return 4 * (lane >> 4) + r; }

constexpr int kIn = 256, kH = 256, kOutP = 64;
constexpr int kNF = AA_MLP_FEATURES, kNO = AA_MLP_OUTPUTS;
constexpr int kLayers = 4;

// Packed parameters: layer l is W_l (din 256 x dout, row-major) then b_l.
__host__ __device__ constexpr int layer_out(int l) { return l == kLayers - 1 ? kOutP : kH; }
__host__ __device__ constexpr int layer_w(int l) { return l * (kH * kH + kH); }
__host__ __device__ constexpr int layer_b(int l) { return layer_w(l) + kH * layer_out(l); }
constexpr int kParams = layer_b(kLayers - 1) + kOutP;

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.f + erff(z * 0.70710678118654752f)) +
         z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// Rows per workgroup (one MFMA row block), threads (eight waves; wave w owns
// output columns 32 w .. 32 w + 31 of a hidden layer) and LDS row stride of an
// activation tile (528 bytes: 16-byte aligned, rows four banks apart).
constexpr int kRows = 16, kChainWG = 512, kActS = kH + 8;

// Eight consecutive reduction indices of one output column, from a matrix
// stored with the reduction index fastest (ld elements a column).
__device__ __forceinline__ v8bf ld_op(const uint16_t* w, int ld, int n, int k) {
  return *reinterpret_cast<const v8bf*>(w + (size_t)n * ld + k);
}

// acc[nb] = tile (16 x 32 STEPS, LDS) times this wave's operands
template <int STEPS, int NB>
__device__ __forceinline__ void mma_tile(const uint16_t (*act)[kActS], const v8bf (&b)[NB][8],
                                         v4f (&acc)[NB]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const v8bf af = *reinterpret_cast<const v8bf*>(&act[lane & 15][32 * s + 8 * (lane >> 4)]);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, b[nb][s], acc[nb], 0, 0, 0);
  }
}

struct FwdArgs {
  const float* x;        // [batch x 230]
  float* out;            // [batch x 21] or null
  const uint16_t* wt;    // transposed BF16 weights: W_l^T at layer_w(l)
  const float* p;        // packed FP32 parameters (biases)
  uint16_t* h[kLayers];  // layer inputs, kept for the backward pass
  float* z[kLayers - 1]; // hidden pre-activations, kept
  int batch;
};

// The whole forward pass of 16 rows.  Latency bound (16 workgroups at 256
// rows): a layer is 16 operand loads per lane in flight from the L2, the next
// layer's issued before this one's activation function, so a layer costs about
// one L2 round trip plus the GELU.  At 256 rows: 17 us (23 with the features read
// and stored one after another and each layer's bias read behind the next
// layer's weights; two layers of weights in flight: 17.6), where the 64 x 64 GEMM
// tiles and elementwise kernels before it took nine launches and 120 us.
// (Rolling the layer loop, a third of the code, changed nothing: the weights
// Adam has just rewritten come from beyond the L2.)
__global__ __launch_bounds__(kChainWG) void k_mlp_forward(FwdArgs a) {
  __shared__ __align__(16) uint16_t act[2][kRows][kActS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = blockIdx.x * kRows, li = lane & 15, lk = 8 * (lane >> 4);
  v8bf b[2][8];
  auto load = [&](int l) {
    if (l == kLayers - 1 && w >= 4) return;
    const int n0 = l == kLayers - 1 ? 16 * w : 32 * w;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
      if (nb == 0 || l < kLayers - 1)
#pragma unroll
        for (int s = 0; s < 8; ++s)
          b[nb][s] = ld_op(a.wt + layer_w(l), kH, n0 + 16 * nb + li, 32 * s + lk);
  };
  // (every feature in flight before the first store, which may alias them for
  // all the compiler knows)
  static_assert(kRows * kIn % kChainWG == 0, "whole turns");
  float xv[kRows * kIn / kChainWG];
#pragma unroll
  for (int u = 0; u < kRows * kIn / kChainWG; ++u) {
    const int e = tid + u * kChainWG, r = e / kIn, c = e % kIn, row = r0 + r;
    const bool in = row < a.batch && c < kNF;
    const float v = a.x[in ? (size_t)row * kNF + c : 0];
    xv[u] = in ? v : 0.f;
  }
  // (the biases too: loads return in order, and one issued in its layer would
  // wait for the next layer's weights)
  float bias[kLayers][2];
#pragma unroll
  for (int l = 0; l < kLayers - 1; ++l)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) bias[l][nb] = a.p[layer_b(l) + 32 * w + 16 * nb + li];
  bias[kLayers - 1][0] = w < 4 ? a.p[layer_b(kLayers - 1) + 16 * w + li] : 0.f;
  load(0);
#pragma unroll
  for (int u = 0; u < kRows * kIn / kChainWG; ++u) {
    const int e = tid + u * kChainWG, r = e / kIn, c = e % kIn, row = r0 + r;
    const uint16_t v = f2bf(xv[u]);
    act[0][r][c] = v;
    if (row < a.batch) a.h[0][(size_t)row * kIn + c] = v;
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < kLayers - 1; ++l) {
    v4f acc[2];
    mma_tile<8, 2>(act[l & 1], b, acc);
    load(l + 1);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int n = 32 * w + 16 * nb + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = mfma_row(lane, r), row = r0 + rr;
        const float z = acc[nb][r] + bias[l][nb];
        const uint16_t hv = f2bf(gelu_f(z));
        act[(l + 1) & 1][rr][n] = hv;
        if (row < a.batch) {
          a.z[l][(size_t)row * kH + n] = z;
          a.h[l + 1][(size_t)row * kH + n] = hv;
        }
      }
    }
    __syncthreads();
  }
  if (w >= 4 || !a.out) return;
  v4f acc[1];
  v8bf bl[1][8];
#pragma unroll
  for (int s = 0; s < 8; ++s) bl[0][s] = b[0][s];
  mma_tile<8, 1>(act[(kLayers - 1) & 1], bl, acc);
  const int n = 16 * w + li;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = r0 + mfma_row(lane, r);
    if (row < a.batch && n < kNO)
      a.out[(size_t)row * kNO + n] = acc[0][r] + bias[kLayers - 1][0];
  }
}

struct BwdArgs {
  const float* dout;           // [batch x 21]
  const uint16_t* wb;          // BF16 weights, packed as the parameters
  const float* z[kLayers - 1]; // hidden pre-activations
  float* dz[kLayers];          // FP32 gradients of the pre-activations (bias sums)
  uint16_t* dzb[kLayers];      // their BF16 copies (weight gradients)
  int batch;
};

// The chain dZ_3 -> dZ_0 of 16 rows: dH = dZ_l W_l^T (W_l's rows have the
// reduction index fastest), dZ_{l-1} = dH gelu'(z_{l-1}).  As the forward pass;
// 14.7 us at 256 rows, 86 us as seven launches.
__global__ __launch_bounds__(kChainWG) void k_mlp_backward(BwdArgs a) {
  __shared__ __align__(16) uint16_t act[2][kRows][kActS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = blockIdx.x * kRows, li = lane & 15, lk = 8 * (lane >> 4);
  v8bf b[2][8];
  auto load = [&](int l) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (s < layer_out(l) / 32)
          b[nb][s] = ld_op(a.wb + layer_w(l), layer_out(l), 32 * w + 16 * nb + li, 32 * s + lk);
  };
  float dv[kRows * kOutP / kChainWG];
#pragma unroll
  for (int u = 0; u < kRows * kOutP / kChainWG; ++u) {
    const int e = tid + u * kChainWG, r = e / kOutP, c = e % kOutP, row = r0 + r;
    const bool in = row < a.batch && c < kNO;
    const float v = a.dout[in ? (size_t)row * kNO + c : 0];
    dv[u] = in ? v : 0.f;
  }
  load(kLayers - 1);
  float zv[kLayers - 1][2][4];  // every layer's, in flight at once
#pragma unroll
  for (int l = kLayers - 1; l >= 1; --l)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + mfma_row(lane, r), n = 32 * w + 16 * nb + li;
        const float z = a.z[l - 1][row < a.batch ? (size_t)row * kH + n : 0];
        zv[l - 1][nb][r] = row < a.batch ? z : 0.f;
      }
#pragma unroll
  for (int u = 0; u < kRows * kOutP / kChainWG; ++u) {
    const int e = tid + u * kChainWG, r = e / kOutP, c = e % kOutP, row = r0 + r;
    act[1][r][c] = f2bf(dv[u]);
    if (row < a.batch) {
      a.dz[kLayers - 1][(size_t)row * kOutP + c] = dv[u];
      a.dzb[kLayers - 1][(size_t)row * kOutP + c] = f2bf(dv[u]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int l = kLayers - 1; l >= 1; --l) {
    v4f acc[2];
    if (l == kLayers - 1)
      mma_tile<kOutP / 32, 2>(act[l & 1], b, acc);
    else
      mma_tile<kH / 32, 2>(act[l & 1], b, acc);
    if (l > 1) load(l - 1);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = mfma_row(lane, r), row = r0 + rr, n = 32 * w + 16 * nb + li;
        const float v = acc[nb][r] * gelu_grad_f(zv[l - 1][nb][r]);
        const uint16_t vb = f2bf(v);
        act[(l - 1) & 1][rr][n] = vb;
        if (row < a.batch) {
          a.dz[l - 1][(size_t)row * kH + n] = v;
          a.dzb[l - 1][(size_t)row * kH + n] = vb;
        }
      }
    __syncthreads();
  }
}

// Every gradient in one launch: dW_l += H_l^T dZ_l as 32 x 32 tiles (64 per
// hidden layer: 208 workgroups, where 64 x 64 tiles gave 16 a layer), one
// 16 x 16 block per wave, the batch in steps of 64 rows staged transposed in
// LDS with the next step's 16-byte loads in flight; then the bias gradients,
// 16 columns a workgroup.  The batch index runs in order in every sum.  At 256
// rows 8.3 us; twelve launches took 130 us.
constexpr int kGT = 32, kGK = 64, kGS = kGK + 8;
constexpr int kHidTiles = (kH / kGT) * (kH / kGT);
constexpr int kOutTiles = (kH / kGT) * (kOutP / kGT);
constexpr int kWTiles = (kLayers - 1) * kHidTiles + kOutTiles;
constexpr int kBiasCols = 16;
constexpr int kBTiles = ((kLayers - 1) * kH + kOutP) / kBiasCols;
constexpr int kColSplit = 32;  // row slices of a bias sum, four row phases each

struct GradArgs {
  const uint16_t* h[kLayers];
  const uint16_t* dzb[kLayers];
  const float* dz[kLayers];
  float* g;
  int batch;
};

// db[j] += sum_r dz[r][j]: slice sums (four phases combined as a tree), then
// the slices in order.
__device__ void bias_tile(const GradArgs& a, int t) {
  __shared__ float part[kColSplit][4][kBiasCols];
  const int per_l = kH / kBiasCols;
  const int l = t / per_l < kLayers - 1 ? t / per_l : kLayers - 1;
  const int j0 = (t - l * per_l) * kBiasCols, cols = layer_out(l);
  const int per = (a.batch + kColSplit - 1) / kColSplit;
  const int c = threadIdx.x % kBiasCols;
  for (int i = threadIdx.x / kBiasCols; i < 4 * kColSplit; i += 256 / kBiasCols) {
    const int y = i >> 2, ph = i & 3;
    const int b0 = y * per, b1 = b0 + per < a.batch ? b0 + per : a.batch;
    float s = 0.f;
    for (int r = b0 + ph; r < b1; r += 4) s += a.dz[l][(size_t)r * cols + j0 + c];
    part[y][ph][c] = s;
  }
  __syncthreads();
  if (threadIdx.x < kBiasCols) {
    float s = 0.f;
    for (int y = 0; y < kColSplit; ++y)
      s += (part[y][0][c] + part[y][1][c]) + (part[y][2][c] + part[y][3][c]);
    a.g[layer_b(l) + j0 + c] += s;
  }
}

__global__ __launch_bounds__(256) void k_mlp_grads(GradArgs a) {
  if (blockIdx.x >= kWTiles) {
    bias_tile(a, blockIdx.x - kWTiles);
    return;
  }
  __shared__ __align__(16) uint16_t As[kGT][kGS], Bs[kGT][kGS];  // [column][batch row]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l = blockIdx.x / kHidTiles, t = blockIdx.x % kHidTiles;
  const int N = layer_out(l), nt = N / kGT;
  const int m0 = t / nt * kGT, n0 = t % nt * kGT;
  // this thread's 16 bytes of a step: row tid / 4, columns 8 (tid % 4) ...
  const int sr = tid >> 2, sc = 8 * (tid & 3);
  uint4 va, vb;
  auto fetch = [&](int k0) {
    const int r = k0 + sr;
    va = vb = uint4{0u, 0u, 0u, 0u};
    if (r < a.batch) {
      va = *reinterpret_cast<const uint4*>(a.h[l] + (size_t)r * kH + m0 + sc);
      vb = *reinterpret_cast<const uint4*>(a.dzb[l] + (size_t)r * N + n0 + sc);
    }
  };
  v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
  const int mb = 16 * (w >> 1), nb = 16 * (w & 1), li = lane & 15, lk = 8 * (lane >> 4);
  fetch(0);
  for (int k0 = 0; k0 < a.batch; k0 += kGK) {
    const uint32_t pa[4] = {va.x, va.y, va.z, va.w}, pv[4] = {vb.x, vb.y, vb.z, vb.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      As[sc + e][sr] = (uint16_t)(pa[e >> 1] >> (16 * (e & 1)));
      Bs[sc + e][sr] = (uint16_t)(pv[e >> 1] >> (16 * (e & 1)));
    }
    __syncthreads();
    if (k0 + kGK < a.batch) fetch(k0 + kGK);
#pragma unroll
    for (int s = 0; s < kGK; s += 32) {
      const v8bf af = *reinterpret_cast<const v8bf*>(&As[mb + li][s + lk]);
      const v8bf bf = *reinterpret_cast<const v8bf*>(&Bs[nb + li][s + lk]);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc, 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    a.g[layer_w(l) + (size_t)(m0 + mb + mfma_row(lane, r)) * N + n0 + nb + li] += acc[r];
}

// BF16 copies of parameter i: packed, and (weights) transposed for the
// forward operands.
__device__ __forceinline__ void put_bf16(uint16_t* pb, uint16_t* wt, int i, float v) {
  const uint16_t q = f2bf(v);
  pb[i] = q;
  const int l = i / layer_w(1) < kLayers - 1 ? i / layer_w(1) : kLayers - 1;
  const int e = i - layer_w(l), N = layer_out(l);
  if (e < kH * N) wt[layer_w(l) + (e % N) * kH + e / N] = q;
}

// Adam on FP32 master weights; clears the gradient; refreshes the BF16 copies.
__global__ void k_adam(float* p, float* g, float* m, float* v, uint16_t* pb, uint16_t* wt,
                       float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kParams) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float upd = lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  const float pi = p[i] - upd;
  p[i] = pi;
  put_bf16(pb, wt, i, pi);
  g[i] = 0.f;
}

// Gradients and moments cleared, BF16 copies refreshed.
__global__ void k_reset(const float* p, float* g, float* m, float* v, uint16_t* pb,
                        uint16_t* wt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kParams) return;
  g[i] = m[i] = v[i] = 0.f;
  put_bf16(pb, wt, i, p[i]);
}

__global__ void k_fillf(float* p, int64_t n, float v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// W (din x dout, row-major): N(0,1) * scale on the live block (rows < fin,
// cols < fout), element (r, c) from counter r * dout + c of the stream.
__global__ void k_init_layer(float* W, int din, int dout, int fin, int fout, uint64_t base,
                             float scale) {
  const int64_t tot = (int64_t)din * dout;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < tot;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(i / dout), c = (int)(i % dout);
    W[i] = (r < fin && c < fout) ? (float)normal_at(base, (uint64_t)i) * scale : 0.f;
  }
}

static int eltgrid(int64_t n) {
  int64_t g = (n + 255) / 256;
  return (int)(g < 1 ? 1 : g > 8192 ? 8192 : g);
}

}  // namespace aa

using namespace aa;

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {
size_t al(size_t x) { return (x + 255) / 256 * 256; }
}  // namespace

struct aa_mlp;
static aa_status mlp_reset_state(aa_mlp* n);

struct aa_mlp {
  int max_batch = 0;
  hipStream_t stream = nullptr;
  float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;  // packed W0 b0 W1 b1 ...
  uint16_t *pb = nullptr, *wt = nullptr;  // BF16 copies: as packed, weights transposed
  uint16_t* h[kLayers] = {};      // h[l] = BF16 input of layer l [B x 256]
  float* z[kLayers - 1] = {};     // hidden pre-activations
  float* dz[kLayers] = {};        // their gradients, and the outputs'
  uint16_t* dzb[kLayers] = {};
  int last_batch = 0;
  int64_t t = 0;  // Adam steps taken
};

// Zero gradients and Adam moments, refresh the BF16 weights (after an
// initialization or a load of the master weights).
static aa_status mlp_reset_state(aa_mlp* n) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  hipLaunchKernelGGL(k_reset, dim3((kParams + 255) / 256), dim3(256), 0, n->stream, n->p, n->g,
                     n->m, n->v, n->pb, n->wt);
  n->t = 0;
  return hipGetLastError() == hipSuccess ? AA_OK : AA_EHIP;
}

namespace aa {
hipStream_t mlp_stream(const aa_mlp* n) { return n->stream; }
int mlp_max_batch(const aa_mlp* n) { return n->max_batch; }
}  // namespace aa

extern "C" {

aa_status aa_mlp_workspace_size(int max_batch, size_t* bytes) {
  if (max_batch < 1 || max_batch > (1 << 20) || !bytes) return AA_EINVAL;
  const size_t B = (size_t)max_batch;
  size_t s = 4 * al(sizeof(float) * kParams) + 2 * al(sizeof(uint16_t) * kParams);
  s += kLayers * al(sizeof(uint16_t) * B * kH);            // h
  s += (kLayers - 1) * al(sizeof(float) * B * kH);         // z
  for (int l = 0; l < kLayers; ++l)                        // dz, dzb
    s += al(sizeof(float) * B * layer_out(l)) + al(sizeof(uint16_t) * B * layer_out(l));
  *bytes = s;
  return AA_OK;
}

aa_status aa_mlp_init(aa_mlp** out, int max_batch, uint64_t seed, void* d_ws, size_t bytes,
                      void* stream) {
  if (!out) return AA_EINVAL;
  *out = nullptr;
  size_t need = 0;
  if (aa_mlp_workspace_size(max_batch, &need) != AA_OK) return AA_EINVAL;
  if (!d_ws || ((uintptr_t)d_ws % 256) != 0) return AA_EINVAL;
  if (bytes < need) return AA_ENOSPACE;
  aa_mlp* n = new (std::nothrow) aa_mlp();
  if (!n) return AA_EINVAL;
  n->max_batch = max_batch;
  n->stream = (hipStream_t)stream;
  char* base = (char*)d_ws;
  size_t o = 0;
  const size_t B = (size_t)max_batch;
  auto take = [&](size_t sz) {
    char* r = base + o;
    o += al(sz);
    return r;
  };
  n->p = (float*)take(sizeof(float) * kParams);
  n->g = (float*)take(sizeof(float) * kParams);
  n->m = (float*)take(sizeof(float) * kParams);
  n->v = (float*)take(sizeof(float) * kParams);
  n->pb = (uint16_t*)take(sizeof(uint16_t) * kParams);
  n->wt = (uint16_t*)take(sizeof(uint16_t) * kParams);
  for (int l = 0; l < kLayers; ++l) n->h[l] = (uint16_t*)take(sizeof(uint16_t) * B * kH);
  for (int l = 0; l < kLayers - 1; ++l) n->z[l] = (float*)take(sizeof(float) * B * kH);
  for (int l = 0; l < kLayers; ++l) {
    n->dz[l] = (float*)take(sizeof(float) * B * layer_out(l));
    n->dzb[l] = (uint16_t*)take(sizeof(uint16_t) * B * layer_out(l));
  }
  aa_status s = aa_mlp_reseed(n, seed);
  if (s != AA_OK) {
    delete n;
    return s;
  }
  *out = n;
  return AA_OK;
}

aa_status aa_mlp_reseed(aa_mlp* n, uint64_t seed) {
  if (!n) return AA_EINVAL;
  const hipStream_t st = n->stream;
  hipLaunchKernelGGL(k_fillf, dim3(eltgrid(kParams)), dim3(256), 0, st, n->p,
                     (int64_t)kParams, 0.f);
  for (int l = 0; l < kLayers - 1; ++l) {
    const int fin = l == 0 ? kNF : kH;
    const uint64_t sb = sm64_mix_host(sm64_mix_host(seed) + (uint64_t)l);
    hipLaunchKernelGGL(k_init_layer, dim3(eltgrid((int64_t)kH * kH)), dim3(256), 0,
                       st, n->p + layer_w(l), kH, kH, fin, kH, sb,
                       sqrtf(2.0f / (float)fin));
  }
  // last layer: zero weights, beta-logit bias +4
  hipLaunchKernelGGL(k_fillf, dim3(1), dim3(64), 0, st, n->p + layer_b(kLayers - 1) + (kNO - 1),
                     (int64_t)1, 4.0f);
  return mlp_reset_state(n);
}

aa_status aa_mlp_set_params(aa_mlp* n, const float* h) {
  if (!n || !h) return AA_EINVAL;
  if (hipMemcpyAsync(n->p, h, sizeof(float) * kParams, hipMemcpyHostToDevice, n->stream) !=
          hipSuccess ||
      hipStreamSynchronize(n->stream) != hipSuccess)
    return AA_EHIP;
  return mlp_reset_state(n);
}

aa_status aa_mlp_get_params(aa_mlp* n, float* h) {
  if (!n || !h) return AA_EINVAL;
  if (hipMemcpyAsync(h, n->p, sizeof(float) * kParams, hipMemcpyDeviceToHost, n->stream) !=
          hipSuccess ||
      hipStreamSynchronize(n->stream) != hipSuccess)
    return AA_EHIP;
  return AA_OK;
}

aa_status aa_mlp_get_grads(aa_mlp* n, float* h) {
  if (!n || !h) return AA_EINVAL;
  if (hipMemcpyAsync(h, n->g, sizeof(float) * kParams, hipMemcpyDeviceToHost, n->stream) !=
          hipSuccess ||
      hipStreamSynchronize(n->stream) != hipSuccess)
    return AA_EHIP;
  return AA_OK;
}

int64_t aa_mlp_param_count(void) { return kParams; }

aa_status aa_mlp_forward(aa_mlp* n, int batch, const float* x, float* out) {
  if (!n || !x || batch < 1 || batch > n->max_batch) return AA_EINVAL;
  const hipStream_t st = n->stream;
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  FwdArgs a{};
  a.x = x;
  a.out = out;
  a.wt = n->wt;
  a.p = n->p;
  for (int l = 0; l < kLayers; ++l) a.h[l] = n->h[l];
  for (int l = 0; l < kLayers - 1; ++l) a.z[l] = n->z[l];
  a.batch = batch;
  hipLaunchKernelGGL(k_mlp_forward, dim3((batch + kRows - 1) / kRows), dim3(kChainWG), 0, st, a);
  n->last_batch = batch;
  return hipGetLastError() == hipSuccess ? AA_OK : AA_EHIP;
}

aa_status aa_mlp_backward(aa_mlp* n, int batch, const float* dout) {
  if (!n || !dout || batch < 1 || batch != n->last_batch) return AA_EINVAL;
  const hipStream_t st = n->stream;
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  BwdArgs a{};
  GradArgs ga{};
  a.dout = dout;
  a.wb = n->pb;
  for (int l = 0; l < kLayers - 1; ++l) a.z[l] = n->z[l];
  for (int l = 0; l < kLayers; ++l) {
    a.dz[l] = n->dz[l];
    a.dzb[l] = n->dzb[l];
    ga.h[l] = n->h[l];
    ga.dz[l] = n->dz[l];
    ga.dzb[l] = n->dzb[l];
  }
  a.batch = ga.batch = batch;
  ga.g = n->g;
  hipLaunchKernelGGL(k_mlp_backward, dim3((batch + kRows - 1) / kRows), dim3(kChainWG), 0, st, a);
  hipLaunchKernelGGL(k_mlp_grads, dim3(kWTiles + kBTiles), dim3(256), 0, st, ga);
  return hipGetLastError() == hipSuccess ? AA_OK : AA_EHIP;
}

aa_status aa_mlp_adam(aa_mlp* n, float lr, float b1, float b2, float eps) {
  if (!n || !(lr >= 0.f) || !(b1 >= 0.f && b1 < 1.f) || !(b2 >= 0.f && b2 < 1.f) || !(eps > 0.f))
    return AA_EINVAL;
  n->t += 1;
  const float c1 = 1.f - powf(b1, (float)n->t), c2 = 1.f - powf(b2, (float)n->t);
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  hipLaunchKernelGGL(k_adam, dim3((kParams + 255) / 256), dim3(256), 0, n->stream, n->p, n->g,
                     n->m, n->v, n->pb, n->wt, lr, b1, b2, eps, c1, c2);
  return hipGetLastError() == hipSuccess ? AA_OK : AA_EHIP;
}

aa_status aa_mlp_destroy(aa_mlp* n) {
  delete n;
  return AA_OK;
}

}  // extern "C"
