// Learned initial guess network on gfx950, FP32 on the matrix cores.  Small
// batches, and wide or deep networks, take one launch per layer and direction
// (k_layer, k_layer_tile), large batches a kernel that runs a tile of samples
// through the whole network (k_net); in training k_net_grad then forms all
// weight gradients and applies Adam.  See mlp.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <type_traits>
#include <vector>

#include "mlp.hpp"

namespace mlfma {
namespace {

#define MLP_TRY(expr)                                                     \
  do {                                                                    \
    hipError_t e_ = (expr);                                               \
    if (e_ != hipSuccess) {                                               \
      err = std::string(#expr " failed: ") + hipGetErrorString(e_);       \
      return -3;                                                          \
    }                                                                     \
  } while (0)

constexpr int kT = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// All products contract over k in steps of 16 with a k-permutation inside each
// step: of v_mfma_f32_16x16x4f32 (A[i][k] from lane i + 16k, B[k][j] from lane
// j + 16k, result row 4*(lane/16) + v, column lane % 16) lane (i, kq) holds the
// consecutive values 4 kq .. 4 kq + 3 of its row and column, and MFMA q
// contracts over kq, so that operands come in 16-byte loads.
__device__ __forceinline__ int pad16(int v) { return (v + 15) & ~15; }
// Elements k .. k + 3 of row r of a row-major [rows][K] matrix (row stride ld),
// zero past its end.
__device__ __forceinline__ f32x4 row4(const float* __restrict__ A, int rows, int K, long ld, int r, int k) {
  f32x4 o;
  const long at = (long)min(r, rows - 1) * ld;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float v = A[at + min(k + q, K - 1)];
    o[q] = r < rows && k + q < K ? v : 0.f;
  }
  return o;
}
// The same by one 16-byte load (any 4-byte alignment), of memory that may be read
// up to 3 elements past a row: its padding, or what follows.  Four loads in its
// place, as rows of other than a multiple of 4 elements took, cost 65,536 samples
// of the 43-301-303-77 network 543 us.
__device__ __forceinline__ f32x4 row4_over(const float* __restrict__ A, int rows, int K, long ld, int r, int k) {
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  const f32x4 v = *reinterpret_cast<const f32x4u*>(A + (long)min(r, rows - 1) * ld + min(k, (K - 1) & ~3));
  f32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = r < rows && k + q < K ? v[q] : 0.f;
  return o;
}
// Column r of a [K][rows] matrix.
__device__ __forceinline__ f32x4 col4(const float* __restrict__ A, int rows, int K, int r, int k) {
  f32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float v = A[(long)min(k + q, K - 1) * rows + min(r, rows - 1)];
    o[q] = r < rows && k + q < K ? v : 0.f;
  }
  return o;
}

// ------------------------------------------------------ one layer a launch --
// out[sample][m] = sum_k W(m, k) in[sample][k], W the layer's matrix or (back)
// its transpose, with the layer's epilogue.
struct LayerArgs {
  const float* W;     // [M][K], back: [K][M]
  const float* bias;  // forward
  const float* in;    // [n][ldi]
  const float* T;     // last layer in training: targets [n][M]
  const float* mask;  // back: the layer's inputs, feature-major [M][ldn]
  float* out;         // [n][ldo], sample-major (may be null)
  float* outT;        // training: feature-major [M][ldn]
  float* inT;         // first layer in training: its inputs, feature-major [K][ldn]
  double* part;       // last layer in training: squared error of each block
  int M, K, n, ldi, ldo, ldn, relu, back;
  int over;           // rows of `in` may be read past their end (row4_over; those of W always, what follows is
                      // the biases and the parameters' padding)
  int over_out;       // rows of `out` may be written up to a multiple of 4, and are 16-byte aligned
};
// The epilogue of outputs m .. m + 3 (m < M) of sample s (below max(n, ldn)) and
// their stores.
__device__ __forceinline__ void layer_store(const LayerArgs& a, int m, int s, f32x4 c, double& s2) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (m + v >= a.M) break;
    if (a.back) {
      c[v] = a.mask[(long)(m + v) * a.ldn + s] > 0.f ? c[v] : 0.f;
    } else {
      c[v] += a.bias[m + v];
      if (a.relu) c[v] = fmaxf(c[v], 0.f);
      if (a.T) {  // the delta of 0.5 / n sum (Y - T)^2
        const float d = s < a.n ? c[v] - a.T[(long)s * a.M + m + v] : 0.f;
        s2 += (double)d * d;
        c[v] = d / (float)a.n;
      }
    }
    if (a.outT) a.outT[(long)(m + v) * a.ldn + s] = c[v];
  }
  if (!a.out || s >= a.n) return;
  float* o = a.out + (long)s * a.ldo + m;
  if (a.over_out) {
    *reinterpret_cast<f32x4*>(o) = c;
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (m + v < a.M) o[v] = c[v];
  }
}
// The first layer's inputs of `ns` samples from n0 on, feature-major.
__device__ __forceinline__ void layer_inputs(const LayerArgs& a, int n0, int ns) {
  for (int e = threadIdx.x; e < ns * a.K; e += 256) {
    const int s = n0 + e % ns, k = e / ns;
    if (s < a.ldn) a.inT[(long)k * a.ldn + s] = s < a.n ? a.in[(long)s * a.ldi + k] : 0.f;
  }
}

// Small launches: a block takes 16 features x 16 samples, its four waves a
// quarter of k each, all of a wave's loads for K up to 256 in flight at once:
// 256 samples of the 256-wide layers make 256 blocks of one memory latency.
// Bound by that latency and the launch: a training step of 256 samples took
// 412 us with a 64 x 64 LDS GEMM per product (16 chunks of k, one at a time)
// and takes 80 us now; about 125 us with k_net, whose 16 blocks leave most of
// the chip idle.
__global__ __launch_bounds__(256) void k_layer(LayerArgs a) {
  __shared__ f32x4 red[3][64];
  const int tm = (a.M + 15) / 16, m0 = (blockIdx.x % tm) * 16, n0 = (blockIdx.x / tm) * 16;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int nk = pad16(a.K) / 16, k0 = wave * nk / 4, k1 = (wave + 1) * nk / 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;
  for (int s = k0; s < k1; s += U) {
    f32x4 x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = s + u < k1 ? 16 * (s + u) + 4 * kq : a.K;  // past the wave's range: zeros
      x[u] = a.back ? col4(a.W, a.M, a.K, m0 + i, k) : row4_over(a.W, a.M, a.K, a.K, m0 + i, k);
      y[u] = a.over ? row4_over(a.in, a.n, a.K, a.ldi, n0 + i, k) : row4(a.in, a.n, a.K, a.ldi, n0 + i, k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][q], y[u][q], acc, 0, 0, 0);
  }
  if (a.inT && m0 == 0) layer_inputs(a, n0, 16);
  if (wave > 0) red[wave - 1][lane] = acc;
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int w = 0; w < 3; ++w) acc += red[w][lane];
  double s2 = 0;
  if (m0 + 4 * kq < a.M) layer_store(a, m0 + 4 * kq, n0 + i, acc, s2);
  if (a.T) {
    for (int o = 32; o > 0; o >>= 1) s2 += __shfl_xor(s2, o);
    if (lane == 0) a.part[blockIdx.x] = s2;
  }
}

// Large launches (kTileFrom): a block takes 32 RT features x 32 CT samples, its
// four waves 2 x 2 shares of 16 RT x 16 CT, whose operands come from L1 and L2
// with the next k-step's in flight.  The 16 x 16 blocks read 16 bytes of L2 for
// 64 products, this one RT CT / (RT + CT) times less.  Sums are set aside every
// 256 k, so that a chain is no longer than a wave's quarter of a 1024-wide layer
// above.
// OVER: as LayerArgs::over.
template <int RT, int CT, bool BACK, bool OVER>
__global__ __launch_bounds__(256) void k_layer_tile(LayerArgs a) {
  __shared__ double red[4];
  const int tm = (a.M + 32 * RT - 1) / (32 * RT);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int b0 = (int)(blockIdx.x / tm) * 32 * CT;
  const int m0 = (int)(blockIdx.x % tm) * 32 * RT + (wave & 1) * 16 * RT, n0 = b0 + (wave >> 1) * 16 * CT;
  const int nk = pad16(a.K) / 16;
  f32x4 acc[RT][CT], sum[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = sum[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int st, f32x4(&x)[RT], f32x4(&y)[CT]) {  // (past the last step: zeros)
    const int k = 16 * st + 4 * kq;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      x[rt] = BACK ? col4(a.W, a.M, a.K, m0 + 16 * rt + i, k) : row4_over(a.W, a.M, a.K, a.K, m0 + 16 * rt + i, k);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      y[ct] = OVER ? row4_over(a.in, a.n, a.K, a.ldi, n0 + 16 * ct + i, k)
                   : row4(a.in, a.n, a.K, a.ldi, n0 + 16 * ct + i, k);
  };
  auto multiply = [&](const f32x4(&x)[RT], const f32x4(&y)[CT]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[rt][q], y[ct][q], acc[rt][ct], 0, 0, 0);
  };
  f32x4 x0[RT], y0[CT], x1[RT], y1[CT];
  load(0, x0, y0);
  for (int st = 0; st < nk; st += 2) {
    load(st + 1, x1, y1);
    multiply(x0, y0);
    load(st + 2, x0, y0);
    multiply(x1, y1);
    if ((st & 14) == 14)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          sum[rt][ct] += acc[rt][ct];
          acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
  }
  if (a.inT && blockIdx.x % tm == 0) layer_inputs(a, b0, 32 * CT);
  double s2 = 0;
  const int ns = max(a.n, a.ldn);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int m = m0 + 16 * rt + 4 * kq, s = n0 + 16 * ct + i;
      if (m < a.M && s < ns) layer_store(a, m, s, sum[rt][ct] + acc[rt][ct], s2);
    }
  if (a.T) {
    for (int o = 32; o > 0; o >>= 1) s2 += __shfl_xor(s2, o);
    if (lane == 0) red[wave] = s2;
    __syncthreads();
    if (threadIdx.x == 0) a.part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}
// Features and samples per block of a layer's launch: 16 x 16 below kTileFrom
// blocks (back: twice that, as the transposed weights come in 4-byte loads) of
// 128 x 64 or, where that pads the features less, 64 x 128.  Times in us, 16 x 16
// against the tiles, of 2048, 4096 and 32,768 samples of the 43-1024-1024-120
// network (256, 512 and 4096 blocks a layer): forward 176 and 100, 335 and 158,
// 2558 and 986 (a 64 x 64 LDS GEMM: 378, -, 1489); training 444 and 368, 831 and
// 611, 6621 and 4689.  With 128 blocks the tiles lose: 97 and 142 (1024 samples).
constexpr long kTileFrom = 256;
struct LayerTile {
  int m, n;
  long blocks(int M, int S) const { return (long)((M + m - 1) / m) * ((S + n - 1) / n); }
};
inline LayerTile layer_tile(int M, int n, bool back) {
  const LayerTile t = (M + 127) / 128 * 128 == (M + 63) / 64 * 64 ? LayerTile{128, 64} : LayerTile{64, 128};
  return t.blocks(M, n) >= (back ? 2 : 1) * kTileFrom ? t : LayerTile{16, 16};
}
template <bool BACK>
void launch_layer(const LayerArgs& a, hipStream_t st) {
  const LayerTile t = layer_tile(a.M, a.n, BACK);
  const dim3 grid((unsigned)t.blocks(a.M, a.n)), block(256);
  if (t.m == 16) hipLaunchKernelGGL(k_layer, grid, block, 0, st, a);
  else if (t.m == 128 && a.over) hipLaunchKernelGGL((k_layer_tile<4, 2, BACK, true>), grid, block, 0, st, a);
  else if (t.m == 128) hipLaunchKernelGGL((k_layer_tile<4, 2, BACK, false>), grid, block, 0, st, a);
  else if (a.over) hipLaunchKernelGGL((k_layer_tile<2, 4, BACK, true>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_layer_tile<2, 4, BACK, false>), grid, block, 0, st, a);
}

// ------------------------------------------------------ fused network --
// One block takes 16 CT samples through the network: the activations stay in
// LDS (sample-major, one buffer: a layer's outputs are held in registers until
// every wave has read its inputs), the weights stream from L2.  W waves share
// the output features, wave w taking the 16-feature tiles w, w + W, ... (RT at
// most); the samples are the columns.  The weights of the next U steps are in
// flight during the current U.  Training (MODE 1) goes on to the deltas of
// every layer (W^T as the operand) and writes activations and deltas
// feature-major, the layout in which the weight gradients contract over
// samples.  102,400 samples of the 43-256-256-256-120 network take 0.45 ms,
// features and phases included (2.6 ms with a GEMM per layer and the features
// formed on the host): the matrix cores are busy 63% of it, with 42.8 GFLOP for
// the network's 35.4 (the 120 outputs fill one of a wave's two tiles, the 43
// inputs 43 of 48 k); the rest goes to barriers and epilogues.  Two blocks of 8
// waves share a CU, so that one's inputs, phases and barriers hide behind the
// other's products: two steps of weights in flight and 124 registers, where four
// steps took 162, one block per CU and 0.62 ms.
//
// Used from kNetFrom samples on, where its blocks of 16 (CT = 1, 16 waves)
// cover half of the chip (training step: 106 against 89 us by layers at 1024
// samples, 115 against 131 at 2048, 144 against 217 at 4096).  From kNetWide
// on (twice that in training, whose blocks do three times the work) CT = 4 and
// 8 waves read the weights a quarter as often (forward 75 against 83 us at
// 8192 samples, 76 against 162 at 16384; training 308 against 262 and 390 against
// 523).  Networks wider than kNetWidth or deeper than kNetLayers take a launch
// per layer for every batch.
constexpr int kNetLayers = 8, kNetWidth = 512, kNetFrom = 2048, kNetWide = 8192;
struct NetArgs {
  const float* P;                                       // parameters
  const float* X;                                       // [n][in]
  const float* T;                                       // training: targets [n][out]
  float* Y;                                             // forward: [n][out]
  float *H[kNetLayers], *G[kNetLayers];                 // training: inputs, deltas of each layer [width][ldn]
  double* part;                                         // training: squared error of each block
  long woff[kNetLayers], boff[kNetLayers];
  int size[kNetLayers + 1];
  int L, n, ldn, stride;                                // layers, samples, padded samples, floats per LDS row
};
// Inputs and outputs of the learned guess (MODE 2: complex float, 3: complex
// double): sample s = r * P + p, features as mlfma_guess_features forms them,
// outputs times the incident phase exp(-j k khat . r_p).
struct GuessArgs {
  const int *cls, *box_of, *part_of_box;
  const double *cen, *khat;
  const float* param;  // [classes] class parameter / scale
  void* x;
  double k;
  int P, C, nx, ny, edge_cap;
};
__device__ __forceinline__ float guess_feature(const GuessArgs& q, int s, int f) {
  const int r = s / q.P, p = s - r * q.P;
  if (f < q.C) return q.cls[p] == f ? 1.f : 0.f;
  f -= q.C;
  const int box = q.box_of[p], ix = box % q.nx, iy = box / q.nx;
  if (f < 8) {
    const int o = f + (f >= 4), jx = ix + o % 3 - 1, jy = iy + o / 3 - 1;
    const int nb = jx >= 0 && jy >= 0 && jx < q.nx && jy < q.ny ? q.part_of_box[jy * q.nx + jx] : -1;
    return nb >= 0 ? q.param[q.cls[nb]] : 0.f;
  }
  if (f < 10) return (float)q.khat[3 * r + f - 8];
  const int edge = min(min(ix, iy), min(q.nx - 1 - ix, q.ny - 1 - iy));
  return (float)min(edge, q.edge_cap) / q.edge_cap;
}

// acc = sum_k A(m, k) h[sample][k] for this wave's feature tiles: A = W [M][K]
// row-major, or its transpose (W [K][M]).  Rows and k past the end are zero.
template <int CT, int W, int RT, int U, bool TRANS>
__device__ __forceinline__ void net_product(f32x4 (&acc)[RT][CT], const float* __restrict__ Wl, int M, int K,
                                            const float* h, int stride, int wave, int i, int kq) {
  const int nk = pad16(K) / 16;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int k0, f32x4(&a)[U][RT]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int m = 16 * (wave + W * rt) + i, k = 16 * (k0 + u) + 4 * kq;
        a[u][rt] = TRANS ? col4(Wl, M, K, m, k) : row4_over(Wl, M, K, K, m, k);
      }
  };
  auto multiply = [&](int k0, const f32x4(&a)[U][RT]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u >= nk) break;
      f32x4 b[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        b[ct] = *reinterpret_cast<const f32x4*>(h + (16 * ct + i) * stride + 16 * (k0 + u) + 4 * kq);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][rt][q], b[ct][q], acc[rt][ct], 0, 0, 0);
    }
  };
  if (16 * wave >= pad16(M)) return;  // no tile of this layer is this wave's
  f32x4 a0[U][RT], a1[U][RT];
  load(0, a0);
  if constexpr (CT == 4 && RT == 2) {
    // steps past the end load clamped: a load that a branch may skip makes the
    // compiler wait for every load in flight where the branches meet.  With the
    // long strides of the narrow blocks the loads past the end cost more (8192
    // samples in training: 266 us, 313 so)
    for (int k0 = 0; k0 < nk; k0 += 2 * U) {
      load(k0 + U, a1);
      multiply(k0, a0);
      load(k0 + 2 * U, a0);
      multiply(k0 + U, a1);
    }
  } else {
    for (int k0 = 0; k0 < nk; k0 += 2 * U) {
      if (k0 + U < nk) load(k0 + U, a1);
      multiply(k0, a0);
      if (k0 + U >= nk) break;
      if (k0 + 2 * U < nk) load(k0 + 2 * U, a0);
      multiply(k0 + U, a1);
    }
  }
}

// MODE 0: Y = net(X); 1: activations, deltas and squared error of a training
// batch; 2, 3: the learned guess in complex float, double.
template <int CT, int W, int RT, int U, int MODE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(CT == 4 && RT == 2 && MODE != 1 ? 4 : 1))) void k_net(
    NetArgs a, GuessArgs q) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* h = reinterpret_cast<float*>(smem_raw);  // [S][stride]
  __shared__ double red[W];
  constexpr int S = 16 * CT, NT = 64 * W;
  const int s0 = blockIdx.x * S, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, kq = lane >> 4;
  {
    const int in = a.size[0], inp = pad16(in);
    for (int e = tid; e < S * inp; e += NT) {
      const int s = e / inp, f = e - s * inp;
      float v = 0.f;
      if (MODE < 2 && f < in && s0 + s < a.n) v = a.X[(long)(s0 + s) * in + f];
      h[s * a.stride + f] = v;
    }
    __syncthreads();
    if (MODE >= 2) {  // (all of a sample's chains of dependent reads at once, one per thread)
      for (int e = tid; e < S * 9; e += NT) {
        const int s = e / 9, o = e - 9 * s;
        if (s0 + s >= a.n) continue;
        float* hs = h + s * a.stride;
        if (o < 8) {
          hs[q.C + o] = guess_feature(q, s0 + s, q.C + o);
        } else {
          hs[q.cls[(s0 + s) % q.P]] = 1.f;
          for (int f = q.C + 8; f < q.C + 11; ++f) hs[f] = guess_feature(q, s0 + s, f);
        }
      }
      __syncthreads();
    }
    if (MODE == 1)
      for (int e = tid; e < S * in; e += NT) a.H[0][(long)(e / S) * a.ldn + s0 + e % S] = h[(e % S) * a.stride + e / S];
  }
  f32x4 acc[RT][CT];
  double s2 = 0;
  // h <- value(m, sample) of this wave's tiles, and to dst feature-major
  auto store = [&](int M, float* dst, auto value) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int m0 = 16 * (wave + W * rt) + 4 * kq;
      if (m0 >= pad16(M)) continue;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int s = 16 * ct + i;
        f32x4 o;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          o[v] = m0 + v < M ? value(m0 + v, s0 + s, acc[rt][ct][v]) : 0.f;
          if (MODE == 1 && m0 + v < M) dst[(long)(m0 + v) * a.ldn + s0 + s] = o[v];
        }
        *reinterpret_cast<f32x4*>(h + s * a.stride + m0) = o;
      }
    }
  };
  for (int l = 0; l < a.L; ++l) {
    const int K = a.size[l], M = a.size[l + 1];
    const bool last = l + 1 == a.L;
    net_product<CT, W, RT, U, false>(acc, a.P + a.woff[l], M, K, h, a.stride, wave, i, kq);
    const float* __restrict__ bias = a.P + a.boff[l];
    __syncthreads();  // every wave has read the layer's inputs
    store(M, MODE != 1 ? nullptr : last ? a.G[l] : a.H[l + 1], [&](int m, int s, float c) {
      c += bias[m];
      if (!last) return fmaxf(c, 0.f);
      if (MODE != 1) return c;
      const float d = s < a.n ? c - a.T[(long)s * M + m] : 0.f;  // the delta of 0.5 / n sum (Y - T)^2
      s2 += (double)d * d;
      return d / (float)a.n;
    });
    __syncthreads();
  }
  if constexpr (MODE == 1) {
    for (int l = a.L - 1; l > 0; --l) {
      const int K = a.size[l + 1], M = a.size[l];
      net_product<CT, W, RT, U, true>(acc, a.P + a.woff[l], M, K, h, a.stride, wave, i, kq);
      const float* H = a.H[l];  // written by this thread in the forward pass
      __syncthreads();
      store(M, a.G[l - 1], [&](int m, int s, float c) { return H[(long)m * a.ldn + s] > 0.f ? c : 0.f; });
      __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1) s2 += __shfl_xor(s2, o);
    if (lane == 0) red[wave] = s2;
    __syncthreads();
    if (tid == 0) {
      double t = 0;
      for (int w = 0; w < W; ++w) t += red[w];
      a.part[blockIdx.x] = t;
    }
  } else if constexpr (MODE == 0) {
    const int out = a.size[a.L], ns = min(S, a.n - s0);
    for (int e = tid; e < ns * out; e += NT) a.Y[(long)s0 * out + e] = h[(e / out) * a.stride + e % out];
  } else {
    using T = typename std::conditional<MODE == 2, float, double>::type;
    const int nc = a.size[a.L] / 2, ns = min(S, a.n - s0);
    double* ph = reinterpret_cast<double*>(h + S * a.stride);  // [S][2]
    for (int s = tid; s < ns; s += NT) {
      const int r = (s0 + s) / q.P, p = (s0 + s) - r * q.P;
      const double t = -q.k * (q.khat[3 * r] * q.cen[3 * p] + q.khat[3 * r + 1] * q.cen[3 * p + 1] +
                               q.khat[3 * r + 2] * q.cen[3 * p + 2]);
      sincos(t, &ph[2 * s + 1], &ph[2 * s]);
    }
    __syncthreads();
    T* x = static_cast<T*>(q.x) + 2 * (long)s0 * nc;
    for (int e = tid; e < ns * nc; e += NT) {
      const int s = e / nc, j = e - s * nc;
      const double re = h[s * a.stride + 2 * j], im = h[s * a.stride + 2 * j + 1], pr = ph[2 * s], pi = ph[2 * s + 1];
      x[2 * e] = (T)(re * pr - im * pi);
      x[2 * e + 1] = (T)(re * pi + im * pr);
    }
  }
}

// Adam's scalars (c1, c2: bias corrections 1 - beta^t)
struct Adam {
  float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ void adam_update(const Adam& A, float gg, float* p, float* m, float* v) {
  const float mm = A.b1 * *m + (1.f - A.b1) * gg;
  const float vv = A.b2 * *v + (1.f - A.b2) * gg * gg;
  *m = mm;
  *v = vv;
  *p -= A.lr * (mm / A.c1) / (sqrtf(vv / A.c2) + A.eps);
}

// Weight and bias gradients of up to kNetLayers layers in one launch: a block
// takes a 32 x 32 tile of one layer's dW = G H^T, its four waves a quarter of
// the samples each (both operands feature-major, so that a lane's 16-byte loads
// run along the samples), adds their sums through LDS in a fixed order and
// finishes one of its 16 x 16 tiles per wave.  The tiles of the first input
// columns also sum the rows of G, the bias gradients.  With `adam` the
// parameters are updated in place, else the gradients are written.  Small
// batches are bound by latency: four steps of loads are in flight.
struct NetGradArgs {
  const float *H[kNetLayers], *G[kNetLayers];
  float *p, *m, *v, *g;
  long woff[kNetLayers], boff[kNetLayers];
  int size[kNetLayers + 1], first[kNetLayers + 1];  // first block of each layer
  int L, ldn, adam;
  Adam A;
};
__global__ __launch_bounds__(256) void k_net_grad(NetGradArgs a) {
  __shared__ f32x4 red[4][4][64];
  __shared__ float rsum[4][32];
  int l = 0;
  while (l + 1 < a.L && (int)blockIdx.x >= a.first[l + 1]) ++l;
  const int M = a.size[l + 1], N = a.size[l], tn = (N + 31) / 32, t = blockIdx.x - a.first[l];
  const int m0 = (t / tn) * 32, n0 = (t % tn) * 32;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const float *__restrict__ G = a.G[l], *__restrict__ H = a.H[l];
  const int nk = a.ldn / 16, k0 = wave * nk / 4, k1 = (wave + 1) * nk / 4;
  const float *pa[2], *pb[2];
  bool oka[2], okb[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int m = m0 + 16 * u + i, n = n0 + 16 * u + i;
    oka[u] = m < M;
    okb[u] = n < N;
    pa[u] = G + (long)min(m, M - 1) * a.ldn + 4 * kq;
    pb[u] = H + (long)min(n, N - 1) * a.ldn + 4 * kq;
  }
  f32x4 acc[2][2];
  float rs[2] = {0.f, 0.f};
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) acc[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int k = k0; k < k1; ++k) {
    f32x4 x[2], y[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      x[u] = *reinterpret_cast<const f32x4*>(pa[u] + 16 * (long)k);
      y[u] = *reinterpret_cast<const f32x4*>(pb[u] + 16 * (long)k);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][q], y[v][q], acc[u][v], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 2; ++u) rs[u] += (x[u][0] + x[u][1]) + (x[u][2] + x[u][3]);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    rs[u] += __shfl_xor(rs[u], 16);
    rs[u] += __shfl_xor(rs[u], 32);
    if (kq == 0) rsum[wave][16 * u + i] = rs[u];
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) red[wave][2 * u + v][lane] = acc[u][v];
  __syncthreads();
  auto put = [&](long o, float g) {
    if (a.adam) adam_update(a.A, g, a.p + o, a.m + o, a.v + o);
    else a.g[o] = g;
  };
  f32x4 sum = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < 4; ++w) sum += red[w][wave][lane];
  const int n = n0 + 16 * (wave & 1) + i;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int m = m0 + 16 * (wave >> 1) + 4 * kq + e;
    if (m < M && n < N) put(a.woff[l] + (long)m * N + n, sum[e]);
  }
  if (wave == 0 && n0 == 0 && lane < 32 && m0 + lane < M)
    put(a.boff[l] + m0 + lane, (rsum[0][lane] + rsum[1][lane]) + (rsum[2][lane] + rsum[3][lane]));
}

// The features of a learned guess, and x[s][j] = (Y[s][2j] + i Y[s][2j+1]) *
// phase[s], for the batches k_net does not take.
template <typename T>
__global__ __launch_bounds__(kT) void k_guess(GuessArgs q, int S, int n, const float* __restrict__ Y, T* __restrict__ x) {
  const long cnt = (long)S * n;
  for (long e = (long)blockIdx.x * kT + threadIdx.x; e < cnt; e += (long)gridDim.x * kT) {
    const int s = (int)(e / n), j = (int)(e % n), r = s / q.P, p = s - r * q.P;
    const double t = -q.k * (q.khat[3 * r] * q.cen[3 * p] + q.khat[3 * r + 1] * q.cen[3 * p + 1] +
                             q.khat[3 * r + 2] * q.cen[3 * p + 2]);
    double pr, pi;
    sincos(t, &pi, &pr);
    const double re = Y[(long)s * 2 * n + 2 * j], im = Y[(long)s * 2 * n + 2 * j + 1];
    x[2 * e] = (T)(re * pr - im * pi);
    x[2 * e + 1] = (T)(re * pi + im * pr);
  }
}
__global__ __launch_bounds__(kT) void k_features(GuessArgs q, int S, int nf, float* __restrict__ X) {
  const long cnt = (long)S * nf;
  for (long e = (long)blockIdx.x * kT + threadIdx.x; e < cnt; e += (long)gridDim.x * kT)
    X[e] = guess_feature(q, (int)(e / nf), (int)(e % nf));
}

struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  DevBuf() = default;
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  DevBuf(DevBuf&& o) noexcept : p(o.p), bytes(o.bytes) {
    o.p = nullptr;
    o.bytes = 0;
  }
  DevBuf& operator=(DevBuf&& o) noexcept {
    std::swap(p, o.p);
    std::swap(bytes, o.bytes);
    return *this;
  }
  ~DevBuf() {
    if (p) (void)hipFree(p);
  }
  hipError_t ensure(size_t b) {
    if (b <= bytes) return hipSuccess;
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
    hipError_t e = hipMalloc(&p, b);
    if (e == hipSuccess) bytes = b;
    return e;
  }
  float* f() const { return static_cast<float*>(p); }
  double* d() const { return static_cast<double*>(p); }
};

int grid(long work) { return (int)std::max<long>(1, std::min<long>((work + kT - 1) / kT, 4096)); }

uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

}  // namespace

class Mlp {
 public:
  std::vector<int> sizes;
  std::vector<long> woff, boff;  // offsets of each layer's W [out][in] and b [out] in the parameter vector
  long nparam = 0;
  DevBuf params, grads, m1, m2;
  long step = 0;
  // training: inputs and deltas of the layers, feature-major, and the blocks'
  // squared errors, written to host memory by the kernels; activations between
  // k_layer launches; the guess's class parameters, directions, features and
  // outputs
  std::vector<DevBuf> fin, fdel;
  int f_cap = 0, h_cap = 0;
  double* hpart = nullptr;
  DevBuf act[2], gtab, gx, gy;
  int layers() const { return (int)sizes.size() - 1; }
  ~Mlp() {
    if (hpart) (void)hipHostFree(hpart);
  }

  int widest() const { return *std::max_element(sizes.begin(), sizes.end()); }
  bool fused(int n) const { return n >= kNetFrom && layers() <= kNetLayers && widest() <= kNetWidth; }
  static int tile(int n, bool train) { return n >= (train ? 2 : 1) * kNetWide ? 64 : 16; }  // samples per block of k_net
  NetArgs net_args(int n, bool train) const {
    NetArgs a{};
    a.P = params.f();
    for (int l = 0; l < layers(); ++l) {
      a.woff[l] = woff[l];
      a.boff[l] = boff[l];
    }
    for (size_t l = 0; l < sizes.size(); ++l) a.size[l] = sizes[l];
    a.L = layers();
    a.n = n;
    const int S = tile(n, train);
    a.ldn = (n + S - 1) / S * S;
    a.stride = (widest() + 15) / 16 * 16 + 4;  // (4 more: columns of a step fall on different banks)
    return a;
  }
  template <int MODE>
  int launch_net(const NetArgs& a, const GuessArgs& q, hipStream_t st, std::string& err) {
    const int S = tile(a.n, MODE == 1);
    const dim3 grid((a.n + S - 1) / S);
    const uint32_t sh = (uint32_t)(S * a.stride * sizeof(float) + (MODE >= 2 ? 2 * S * sizeof(double) : 0));
    auto run = [&](auto kernel, int W) -> int {
      if (sh > 64 * 1024)
        MLP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)sh));
      hipLaunchKernelGGL(kernel, grid, dim3(64 * W), sh, st, a, q);
      return 0;
    };
    const bool narrow = widest() <= 256;
    constexpr int U = MODE == 1 ? 6 : 8;  // (training keeps more in registers)
    if (S == 16) return narrow ? run(k_net<1, 16, 1, U, MODE>, 16) : run(k_net<1, 16, 2, U / 2, MODE>, 16);
    return narrow ? run(k_net<4, 8, 2, 2, MODE>, 8) : run(k_net<4, 8, 4, 2, MODE>, 8);
  }
  // The layers one launch each, forward: outputs to Y (inference), or the last
  // layer's deltas and squared errors (training: fin, fdel, part).
  int forward_layers(const float* X, const float* T, int n, int ldn, float* Y, double* part, hipStream_t st,
                     std::string& err) {
    const int L = layers(), ld = (widest() + 15) / 16 * 16;
    for (auto& b : act) MLP_TRY(b.ensure((size_t)n * ld * sizeof(float)));
    for (int l = 0; l < L; ++l) {
      LayerArgs a{};
      const bool last = l + 1 == L;
      a.W = params.f() + woff[l];
      a.bias = params.f() + boff[l];
      a.in = l ? act[(l - 1) % 2].f() : X;
      a.ldi = l ? ld : sizes[0];
      a.M = sizes[l + 1];
      a.K = sizes[l];
      a.n = n;
      a.ldn = ldn;
      a.relu = !last;
      a.over = l > 0 || a.K % 4 == 0;
      a.out = last && !T ? Y : act[l % 2].f();
      a.over_out = !last || T || (a.M % 4 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0);
      a.ldo = last && !T ? a.M : ld;
      if (T) {
        a.inT = l ? nullptr : fin[0].f();
        a.outT = last ? fdel[l].f() : fin[l + 1].f();
        if (last) {
          a.T = T;
          a.part = part;
        }
      }
      launch_layer<false>(a, st);
    }
    MLP_TRY(hipGetLastError());
    return 0;
  }
  // ... and back: the deltas of every layer but the last
  int backward_layers(int n, int ldn, hipStream_t st, std::string& err) {
    const int L = layers(), ld = (widest() + 15) / 16 * 16;
    for (int l = L - 1; l > 0; --l) {
      LayerArgs a{};
      a.W = params.f() + woff[l];
      a.in = act[l % 2].f();  // this layer's deltas
      a.ldi = ld;
      a.M = sizes[l];
      a.K = sizes[l + 1];
      a.n = n;
      a.ldn = ldn;
      a.back = 1;
      a.over = a.over_out = 1;
      a.mask = fin[l].f();
      a.out = act[(l - 1) % 2].f();
      a.ldo = ld;
      a.outT = fdel[l - 1].f();
      launch_layer<true>(a, st);
    }
    MLP_TRY(hipGetLastError());
    return 0;
  }
  // Activations and deltas of a batch, then the gradients into `grads` or,
  // with an Adam step, straight into the parameters.  Returns when they are
  // written: the callers read parameters and gradients by copies that no stream
  // orders after this one, and use the workspaces on other streams.
  int train_batch(const float* X, const float* T, int n, const Adam* A, double* loss, hipStream_t st, std::string& err) {
    const int L = layers();
    const bool net = fused(n);
    const int ldn = net ? net_args(n, true).ldn : (n + 15) / 16 * 16;
    const int nb = net ? ldn / tile(n, true) : (int)layer_tile(sizes[L], n, false).blocks(sizes[L], n);
    if (ldn > f_cap) {
      f_cap = 0;
      fin.resize(L);
      fdel.resize(L);
      for (int l = 0; l < L; ++l) {
        MLP_TRY(fin[l].ensure((size_t)sizes[l] * ldn * sizeof(float)));
        MLP_TRY(fdel[l].ensure((size_t)sizes[l + 1] * ldn * sizeof(float)));
      }
      f_cap = ldn;
    }
    if (nb > h_cap) {
      if (hpart) (void)hipHostFree(hpart);
      hpart = nullptr;
      h_cap = 0;
      MLP_TRY(hipHostMalloc(reinterpret_cast<void**>(&hpart), nb * sizeof(double), hipHostMallocDefault));
      h_cap = nb;
    }
    void* dpart = nullptr;
    MLP_TRY(hipHostGetDevicePointer(&dpart, hpart, 0));
    if (net) {
      NetArgs a = net_args(n, true);
      a.X = X;
      a.T = T;
      a.part = static_cast<double*>(dpart);
      for (int l = 0; l < L; ++l) {
        a.H[l] = fin[l].f();
        a.G[l] = fdel[l].f();
      }
      if (int rc = launch_net<1>(a, GuessArgs{}, st, err)) return rc;
      MLP_TRY(hipGetLastError());
    } else if (int rc = forward_layers(X, T, n, ldn, nullptr, static_cast<double*>(dpart), st, err)) {
      return rc;
    }
    if (!net)
      if (int rc = backward_layers(n, ldn, st, err)) return rc;
    for (int l0 = 0; l0 < L; l0 += kNetLayers) {
      NetGradArgs g{};
      g.L = std::min(L - l0, kNetLayers);
      for (int l = 0; l < g.L; ++l) {
        g.H[l] = fin[l0 + l].f();
        g.G[l] = fdel[l0 + l].f();
        g.woff[l] = woff[l0 + l];
        g.boff[l] = boff[l0 + l];
        g.first[l + 1] = g.first[l] + ((sizes[l0 + l + 1] + 31) / 32) * ((sizes[l0 + l] + 31) / 32);
      }
      for (int l = 0; l <= g.L; ++l) g.size[l] = sizes[l0 + l];
      g.p = params.f();
      g.m = m1.f();
      g.v = m2.f();
      g.g = grads.f();
      g.ldn = ldn;
      g.adam = A ? 1 : 0;
      if (A) g.A = *A;
      hipLaunchKernelGGL(k_net_grad, dim3(g.first[g.L]), dim3(256), 0, st, g);
    }
    MLP_TRY(hipGetLastError());
    MLP_TRY(hipStreamSynchronize(st));
    double s2 = 0;
    for (int b = 0; b < nb; ++b) s2 += hpart[b];
    if (loss) *loss = 0.5 * s2 / n;
    return 0;
  }
};

Mlp* mlp_create(const std::vector<int>& sizes, uint64_t seed, std::string& err) {
  if (sizes.size() < 2) {
    err = "a network needs at least an input and an output size";
    return nullptr;
  }
  for (int v : sizes)
    if (v < 1 || v > 65536) {
      err = "layer sizes must be in [1, 65536]";
      return nullptr;
    }
  auto* m = new Mlp();
  m->sizes = sizes;
  long off = 0;
  for (size_t l = 0; l + 1 < sizes.size(); ++l) {
    m->woff.push_back(off);
    off += (long)sizes[l] * sizes[l + 1];
    m->boff.push_back(off);
    off += sizes[l + 1];
  }
  m->nparam = off;
  // He-normal weights (Box-Muller on a splitmix64 stream), zero biases
  std::vector<float> h(off, 0.f);
  uint64_t st = seed;
  for (size_t l = 0; l + 1 < sizes.size(); ++l) {
    const double sd = std::sqrt(2.0 / sizes[l]);
    for (long e = 0; e < (long)sizes[l] * sizes[l + 1]; ++e) {
      const double u1 = ((splitmix64(st) >> 11) + 0.5) * (1.0 / 9007199254740992.0);
      const double u2 = ((splitmix64(st) >> 11) + 0.5) * (1.0 / 9007199254740992.0);
      h[m->woff[l] + e] = (float)(sd * std::sqrt(-2.0 * std::log(u1)) * std::cos(2.0 * 3.14159265358979323846 * u2));
    }
  }
  if (mlp_set_params(m, h.data(), err)) {
    delete m;
    return nullptr;
  }
  return m;
}

void mlp_destroy(Mlp* m) { delete m; }
int64_t mlp_num_params(const Mlp* m) { return m->nparam; }
int mlp_inputs(const Mlp* m) { return m->sizes.front(); }
int mlp_outputs(const Mlp* m) { return m->sizes.back(); }

int mlp_get_params(const Mlp* m, float* host, std::string& err) {
  MLP_TRY(hipMemcpy(host, m->params.p, m->nparam * sizeof(float), hipMemcpyDeviceToHost));
  return 0;
}

int mlp_set_params(Mlp* m, const float* host, std::string& err) {
  const size_t b = m->nparam * sizeof(float);
  MLP_TRY(m->params.ensure(b + 3 * sizeof(float)));  // (row4_over of the last weights)
  MLP_TRY(m->grads.ensure(b));
  MLP_TRY(m->m1.ensure(b));
  MLP_TRY(m->m2.ensure(b));
  MLP_TRY(hipMemcpy(m->params.p, host, b, hipMemcpyHostToDevice));
  MLP_TRY(hipMemset(m->m1.p, 0, b));
  MLP_TRY(hipMemset(m->m2.p, 0, b));
  m->step = 0;
  return 0;
}

int mlp_forward(Mlp* m, const float* X, int n, float* Y, void* stream, std::string& err) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (!m->fused(n)) return m->forward_layers(X, nullptr, n, 0, Y, nullptr, st, err);
  NetArgs a = m->net_args(n, false);
  a.X = X;
  a.Y = Y;
  if (int rc = m->launch_net<0>(a, GuessArgs{}, st, err)) return rc;
  MLP_TRY(hipGetLastError());
  return 0;
}

int mlp_loss_grad(Mlp* m, const float* X, const float* T, int n, double* loss, float* grads, void* stream,
                  std::string& err) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (int rc = m->train_batch(X, T, n, nullptr, loss, st, err)) return rc;
  if (grads) MLP_TRY(hipMemcpy(grads, m->grads.p, m->nparam * sizeof(float), hipMemcpyDeviceToHost));
  return 0;
}

int mlp_train_step(Mlp* m, const float* X, const float* T, int n, float lr, double* loss, void* stream,
                   std::string& err) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const double t = (double)(m->step + 1);
  const Adam A{lr, 0.9f, 0.999f, 1e-8f, (float)(1.0 - std::pow(0.9, t)), (float)(1.0 - std::pow(0.999, t))};
  if (int rc = m->train_batch(X, T, n, &A, loss, st, err)) return rc;
  m->step++;
  return 0;
}

int mlp_guess(Mlp* m, const GuessInput& in, int R, int n, int precision, void* x_dev, void* stream, std::string& err) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int S = R * in.P, nf = m->sizes.front();
  if (nf != in.C + 11 || m->sizes.back() != 2 * n) {
    err = "network inputs/outputs do not match the features / unknowns per particle";
    return -1;
  }
  // the call's small tables: directions, then class parameters over scale
  const size_t kb = (size_t)3 * R * sizeof(double), tb = kb + in.C * sizeof(float);
  std::vector<unsigned char> tab(tb);
  std::memcpy(tab.data(), in.khat, kb);
  for (int c = 0; c < in.C; ++c) {
    const float v = (float)(in.class_param[c] / in.scale);
    std::memcpy(tab.data() + kb + c * sizeof(float), &v, sizeof(float));
  }
  MLP_TRY(m->gtab.ensure(tb));
  MLP_TRY(hipMemcpyAsync(m->gtab.p, tab.data(), tb, hipMemcpyHostToDevice, st));
  GuessArgs q{};
  q.cls = in.cls;
  q.box_of = in.box_of;
  q.part_of_box = in.part_of_box;
  q.cen = in.centers;
  q.khat = m->gtab.d();
  q.param = reinterpret_cast<const float*>(static_cast<const char*>(m->gtab.p) + kb);
  q.x = x_dev;
  q.k = in.k;
  q.P = in.P;
  q.C = in.C;
  q.nx = in.nx;
  q.ny = in.ny;
  q.edge_cap = in.edge_cap;
  if (m->fused(S)) {
    const NetArgs a = m->net_args(S, false);
    if (int rc = precision == 1 ? m->launch_net<3>(a, q, st, err) : m->launch_net<2>(a, q, st, err)) return rc;
  } else {
    MLP_TRY(m->gx.ensure((size_t)S * nf * sizeof(float)));
    MLP_TRY(m->gy.ensure((size_t)S * 2 * n * sizeof(float)));
    hipLaunchKernelGGL(k_features, dim3(grid((long)S * nf)), dim3(kT), 0, st, q, S, nf, m->gx.f());
    if (int rc = mlp_forward(m, m->gx.f(), S, m->gy.f(), stream, err)) return rc;
    const dim3 g(grid((long)S * n));
    if (precision == 1)
      hipLaunchKernelGGL(k_guess<double>, g, dim3(kT), 0, st, q, S, n, (const float*)m->gy.f(), static_cast<double*>(x_dev));
    else
      hipLaunchKernelGGL(k_guess<float>, g, dim3(kT), 0, st, q, S, n, (const float*)m->gy.f(), static_cast<float*>(x_dev));
  }
  MLP_TRY(hipGetLastError());
  MLP_TRY(hipStreamSynchronize(st));  // the caller's tables may be released on return
  return 0;
}

// Device copies of the particle tables the guess reads.
struct GuessTables {
  DevBuf mem;
  int device = -1;
};
GuessTables* guess_tables_create() { return new GuessTables(); }
void guess_tables_destroy(GuessTables* t) { delete t; }
int guess_tables_fill(GuessTables* t, const std::vector<int>& cls, const std::vector<int>& box_of,
                      const std::vector<int>& part_of_box, const std::vector<double>& centers, GuessInput& in,
                      std::string& err) {
  int dev = 0;
  MLP_TRY(hipGetDevice(&dev));
  const size_t nc = centers.size() * sizeof(double), ni = cls.size() * sizeof(int), nb = part_of_box.size() * sizeof(int);
  if (t->device != dev) {  // first use, or another device than the copies are on
    t->device = -1;
    t->mem = DevBuf();
    MLP_TRY(t->mem.ensure(nc + 2 * ni + nb));
    char* p = static_cast<char*>(t->mem.p);
    MLP_TRY(hipMemcpy(p, centers.data(), nc, hipMemcpyHostToDevice));
    MLP_TRY(hipMemcpy(p + nc, cls.data(), ni, hipMemcpyHostToDevice));
    MLP_TRY(hipMemcpy(p + nc + ni, box_of.data(), ni, hipMemcpyHostToDevice));
    MLP_TRY(hipMemcpy(p + nc + 2 * ni, part_of_box.data(), nb, hipMemcpyHostToDevice));
    t->device = dev;
  }
  const char* p = static_cast<const char*>(t->mem.p);
  in.centers = reinterpret_cast<const double*>(p);
  in.cls = reinterpret_cast<const int*>(p + nc);
  in.box_of = reinterpret_cast<const int*>(p + nc + ni);
  in.part_of_box = reinterpret_cast<const int*>(p + nc + 2 * ni);
  return 0;
}

}  // namespace mlfma
