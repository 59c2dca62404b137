// Length head (Section 4.3) and shortest-job-first order (Section 5.4).
//
//   W1 h                          mlp_partial_kernel (matrix cores, split over the depth)
//   a = act(W1 h + b1), o = W2 a + b2
//                                 head_out_kernel: one workgroup per prompt
//   K == 1: yhat = o_0;  K > 1: p = softmax(o), yhat = sum_k p_k c_k (Eq. 7), bin = argmax p
//   order: stable ascending argsort of yhat (rank counting, exact and deterministic)
//
// One training step of the K-bin head (Eq. 6 - Eq. 8, AdamW as in Section 5.1):
//   W1 h as above                                    mlp_partial_kernel
//   forward, Eq. 6 soft labels, Eq. 8 loss, dL/do and dL/dz = (dL/do W2) act'(z) of one sample
//                                                    train_sample_kernel (one workgroup per sample)
//   every gradient and its AdamW update, batch loss  train_update_kernel
// Every batch sum runs in a fixed order: the step is bitwise reproducible.
#include <algorithm>
#include <cmath>

#include "estp_common.h"

namespace estp {
namespace detail {

constexpr int kKChunk = 256;  // the depth of the first layer is never split finer over workgroups than this
constexpr int kMaxDepth = 65536 * kKChunk;
static_assert(size_t(kMaxDepth) * 32 * 4 < kPastEnd, "byte offsets within the narrow tile's rows");

__device__ __forceinline__ float act_fn(float x, int act) {
  if (act == ESTP_ACT_RELU) return fmaxf(x, 0.f);
  // tanh-form GELU: 0.5 x (1 + tanh(sqrt(2/pi) (x + 0.044715 x^3)))
  const float u = 0.7978845608028654f * fmaf(0.044715f * x, x * x, x);
  return 0.5f * x * (1.f + tanhf(u));
}

// Partial products of the first layer: part[z, b, j] = sum over the k of depth share z of P[b, k] W1[j, k].
// A workgroup forms a 16 NB x 16 NB (prompt x hidden) tile; its kDW waves take consecutive depth ranges of
// kw and their tiles are added in wave order through LDS.  Both operands are contiguous along the depth, so
// a lane loads 16 bytes of its row and the four floats feed four matrix-core steps (step i multiplies depths
// k + i, k + 4 + i, k + 8 + i and k + 12 + i): no LDS staging and no transposition, and the next 16 or 32
// depths load while the current ones multiply.  The fp32 matrix cores have the
// rate of the fp32 vector FMAs but read each operand once per 16 products; the vector form (32 x 32 tiles
// through LDS, five 4-byte LDS reads per four FMAs) was bound by LDS: us per estp_predict call on MI355X,
// 4096 -> 1024 -> 16, that form and this: one prompt 31 and 12, 64 prompts 46 and 19, 256 prompts 116 and 33,
// 2048 prompts 695 and 173 (109 of it fp32 arithmetic at the peak rate).
template <int NB, int kDW, bool kVec>
__global__ __launch_bounds__(64 * kDW) void mlp_partial_kernel(const float* __restrict__ P,
                                                               const float* __restrict__ W1, int B, int d, int Hd,
                                                               int kw, float* __restrict__ part) {
  constexpr int kT = 16 * NB, kPitch = kT + 4;  // the four row groups of a tile store land in distinct banks
  __shared__ float red[kDW][kT * kPitch];
  const int th = blockIdx.x * kT, tb = blockIdx.y * kT, z = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, grp = lane >> 4;
  const int k_lo = min(d, (z * kDW + wave) * kw), k_hi = min(d, k_lo + kw);
  // this lane's rows: prompts tb + row + 16 i, hidden units th + row + 16 i.  Through buffer resources that
  // end with the tile's last live row, so that rows past it, and depths past the wave's range (sent to an
  // offset past the end), read as zero without a branch around the load.
  const buf_rsrc_t rp = make_rsrc(P + size_t(tb) * d, uint32_t(min(kT, B - tb)) * uint32_t(d) * 4u);
  const buf_rsrc_t rw = make_rsrc(W1 + size_t(th) * d, uint32_t(min(kT, Hd - th)) * uint32_t(d) * 4u);
  auto load4 = [&](buf_rsrc_t r, int i, int k) {  // depths k .. k + 3 of row 16 i + row, zero past the range
    const uint32_t off = (uint32_t(16 * i + row) * uint32_t(d) + uint32_t(k)) * 4u;
    if (kVec) return buf_load4(r, k < k_hi ? off : kPastEnd);  // k_hi and k are multiples of 4
    f32x4_t v;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = buf_load1(r, k + c < k_hi ? off + 4 * c : kPastEnd);
    return v;
  };
  constexpr int kHalves = NB == 4 ? 1 : 2;  // NB = 4: two whole-line steps would spill
  struct Step {
    f32x4_t a[kHalves][NB], b[kHalves][NB];
  };
  auto load_step = [&](Step& f, int k) {
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        f.a[h][i] = load4(rp, i, k + 16 * h + 4 * grp);
        f.b[h][i] = load4(rw, i, k + 16 * h + 4 * grp);
      }
  };
  f32x4_t acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const Step& f) {
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[i][j] = mfma16_f32(f.a[h][i][c], f.b[h][j][c], acc[i][j]);
  };
  constexpr int kStep = 16 * kHalves;
  Step f0, f1;
  load_step(f0, k_lo);
  for (int k = k_lo; k < k_hi; k += 2 * kStep) {  // steps past the range: zeros, no access
    load_step(f1, k + kStep);
    __builtin_amdgcn_sched_barrier(0);  // the loads go out before the products, not behind them
    multiply(f0);
    __builtin_amdgcn_sched_barrier(0);
    if (k + kStep >= k_hi) break;
    load_step(f0, k + 2 * kStep);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f1);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(16 * i + 4 * grp + r) * kPitch + 16 * j + row] = acc[i][j][r];
  __syncthreads();
#pragma unroll
  for (int e = threadIdx.x; e < kT * kT; e += 64 * kDW) {
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < kDW; ++q) v += red[q][e / kT * kPitch + e % kT];
    const int b = tb + e / kT, j = th + e % kT;
    if (b < B && j < Hd) part[(size_t(z) * B + b) * Hd + j] = v;
  }
}

// Depth shares of the first layer: the number that makes rounds of 256 workgroups, each over its share of
// the depth, shortest; every share costs its partial sums as well (B / 30000 of the time of an unsplit tile).
int mlp_shares(size_t tiles, int B, int d) {
  const int most = (d + kKChunk - 1) / kKChunk;
  int best = 1;
  float best_cost = INFINITY;
  for (int z = 1; z <= most && z <= 64; ++z) {
    const float cost = float((tiles * z + 255) / 256) / float(z) + float(z) * float(B) / 30000.f;
    if (cost < best_cost) {
      best = z;
      best_cost = cost;
    }
  }
  return best;
}

// Launch of the partial products; returns the number of depth shares written.  16-byte loads when
// every row starts 16-byte aligned.
template <int NB, int kDW>
int launch_mlp_tiles(const float* P, const float* W1, int B, int d, int Hd, float* part, hipStream_t s) {
  constexpr int kT = 16 * NB;
  const int nh = (Hd + kT - 1) / kT, nb = (B + kT - 1) / kT;
  const int nz = mlp_shares(size_t(nh) * nb, B, d);
  const int waves = nz * kDW;
  const int kw = ((d + waves - 1) / waves + 31) / 32 * 32;  // depth range of one wave: whole steps
  const dim3 grid(nh, nb, nz), block(64 * kDW);
  if (d % 4 == 0 && aligned(P, 16) && aligned(W1, 16))
    mlp_partial_kernel<NB, kDW, true><<<grid, block, 0, s>>>(P, W1, B, d, Hd, kw, part);
  else
    mlp_partial_kernel<NB, kDW, false><<<grid, block, 0, s>>>(P, W1, B, d, Hd, kw, part);
  return nz;
}
// Tiles of 64 x 64, which read half as much per product, where there are at least 64 of them; else of 32 x 32,
// which spread over more CUs (us per estp_predict call on MI355X with 32 and with 64: 4096 -> 1024, 2048
// prompts 281 and 173, 256 prompts 42 and 33, one prompt 12 and 16; 1536 -> 256, 256 prompts 17 and 20).  A
// tile's rows have to end below kPastEnd, in bytes: the deepest inputs take the narrow tile.
int launch_mlp_partial(const float* P, const float* W1, int B, int d, int Hd, float* part, hipStream_t s) {
  const bool wide = ((size_t(B) + 63) / 64) * ((size_t(Hd) + 63) / 64) >= 64 && size_t(d) * 256 <= kPastEnd;
  return wide ? launch_mlp_tiles<4, 8>(P, W1, B, d, Hd, part, s) : launch_mlp_tiles<2, 16>(P, W1, B, d, Hd, part, s);
}

// z_j = sum_z part[z, b, j] + b1[j], shares added in order.
__device__ __forceinline__ float hidden_sum(const float* __restrict__ part, const float* __restrict__ b1, int b, int B,
                                            int Hd, int nz, int j) {
  const float* p = part + size_t(b) * Hd + j;
  float v = 0.f;
#pragma unroll 8
  for (int z = 0; z < nz; ++z) v += p[size_t(z) * B * Hd];
  return v + (b1 ? b1[j] : 0.f);
}

// o[k] = W2[k] . a + b2[k] of one prompt, by a workgroup of kHeadWaves waves; a is its own global scratch
// row.  A wave takes outputs k, k + 16, ... (kQ of them together) and its lanes run over the hidden units
// eight steps at a time, so that enough loads are in flight.  With four waves, one output and one step at a
// time, the 16 x 1024 products of a prompt were 64 load latencies in a row: 23 us for 256 prompts on MI355X, 6.2
// so, and 32 us for one prompt, 7 so.
constexpr int kHeadWaves = 16;
constexpr int kHeadThreads = 64 * kHeadWaves;
template <int kQ>
__device__ __forceinline__ void head_logits(const float* a, const float* __restrict__ W2,
                                            const float* __restrict__ b2, int Hd, int K, float* o) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int k0 = wave; k0 < K; k0 += kHeadWaves * kQ) {
    float v[kQ];
    const float* w[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      v[q] = 0.f;
      w[q] = W2 + size_t(min(k0 + kHeadWaves * q, K - 1)) * Hd;
    }
#pragma unroll 8
    for (int j = lane; j < Hd; j += 64) {
      const float aj = a[j];
#pragma unroll
      for (int q = 0; q < kQ; ++q) v[q] = fmaf(w[q][j], aj, v[q]);
    }
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const float t = wave_sum(v[q]);
      const int k = k0 + kHeadWaves * q;
      if (lane == 0 && k < K) o[k] = t + (b2 ? b2[k] : 0.f);
    }
  }
}
__device__ __forceinline__ void head_logits(const float* a, const float* __restrict__ W2,
                                            const float* __restrict__ b2, int Hd, int K, float* o) {
  if (K <= kHeadWaves)
    head_logits<1>(a, W2, b2, Hd, K, o);
  else
    head_logits<4>(a, W2, b2, Hd, K, o);
}

// One workgroup per prompt: a = act(z), o = W2 a + b2, then y-hat and bin.
__global__ __launch_bounds__(kHeadThreads) void head_out_kernel(const float* __restrict__ part, const float* __restrict__ b1,
                                                       const float* __restrict__ W2, const float* __restrict__ b2,
                                                       const float* __restrict__ centres, int B, int Hd, int nz, int K,
                                                       int act, float* a_ws, float* o_ws, float* __restrict__ yhat,
                                                       int* __restrict__ bin) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* a = a_ws + size_t(b) * Hd;
  float* o = o_ws + size_t(b) * K;
  for (int j = threadIdx.x; j < Hd; j += kHeadThreads) a[j] = act_fn(hidden_sum(part, b1, b, B, Hd, nz, j), act);
  __syncthreads();
  head_logits(a, W2, b2, Hd, K, o);
  __syncthreads();
  if (K == 1) {
    if (threadIdx.x == 0) yhat[b] = o[0];
    return;
  }
  if (wave != 0) return;
  // softmax over K bins, expectation over the centres, argmax (lowest index)
  float mx = -INFINITY;
  int mi = 0x7fffffff;
  for (int k = lane; k < K; k += 64)
    if (o[k] > mx) {
      mx = o[k];
      mi = k;
    }
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(mx, off, 64);
    const int oi = __shfl_xor(mi, off, 64);
    if (ov > mx || (ov == mx && oi < mi)) {
      mx = ov;
      mi = oi;
    }
  }
  float z = 0.f, zc = 0.f;
  for (int k = lane; k < K; k += 64) {
    const float p = fast_exp2((o[k] - mx) * kLog2e);
    z += p;
    zc = fmaf(p, centres[k], zc);
  }
  z = wave_sum(z);
  zc = wave_sum(zc);
  if (lane == 0) {
    yhat[b] = zc / z;
    if (bin) bin[b] = mi;
  }
}

// order[rank(i)] = i with rank(i) = #{j : y_j < y_i or (y_j == y_i and j < i)}.  A workgroup ranks 64
// prompts; its 16 waves count over a sixteenth of each 1024 staged values and add their counts through LDS
// (256 prompts in one workgroup of one thread each, the counting loop was the call's longest chain: 7.6 us
// of 56 on MI355X, 3.9 so).
constexpr int kOrderWaves = 16;
__global__ __launch_bounds__(64 * kOrderWaves) void sjf_order_kernel(const float* __restrict__ y, int B,
                                                                     int* __restrict__ order) {
  __shared__ __attribute__((aligned(16))) float sy[1024];
  __shared__ int cnt[kOrderWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const float yi = i < B ? y[i] : 0.f;
  int rank = 0;
  for (int j0 = 0; j0 < B; j0 += 1024) {
    __syncthreads();
    // slots past the batch hold a value that no comparison counts
    sy[threadIdx.x] = j0 + int(threadIdx.x) < B ? y[j0 + threadIdx.x] : __builtin_nanf("");
    __syncthreads();
    const int n4 = (min(1024, B - j0) + 3) / 4;
#pragma unroll 4
    for (int t = wave; t < n4; t += kOrderWaves) {
      const float4 v = reinterpret_cast<const float4*>(sy)[t];
      const int j = j0 + 4 * t;
      rank += int(v.x < yi) | (int(v.x == yi) & int(j < i));
      rank += int(v.y < yi) | (int(v.y == yi) & int(j + 1 < i));
      rank += int(v.z < yi) | (int(v.z == yi) & int(j + 2 < i));
      rank += int(v.w < yi) | (int(v.w == yi) & int(j + 3 < i));
    }
  }
  cnt[wave][lane] = rank;
  __syncthreads();
  if (wave != 0 || i >= B) return;
#pragma unroll
  for (int w = 1; w < kOrderWaves; ++w) rank += cnt[w][lane];
  order[rank] = i;
}
static_assert(64 * kOrderWaves == 1024, "one staged value per thread");

// ---------------------------------------------------------------- training step

__device__ __forceinline__ float act_grad(float z, int act) {
  if (act == ESTP_ACT_RELU) return z > 0.f ? 1.f : 0.f;
  const float k = 0.7978845608028654f;  // sqrt(2 / pi)
  const float t = tanhf(k * fmaf(0.044715f * z, z * z, z));
  return 0.5f * (1.f + t) + 0.5f * z * (1.f - t * t) * k * fmaf(3.f * 0.044715f, z * z, 1.f);
}

struct AdamW {
  float lr, beta1, beta2, eps, decay;  // decay = 1 - lr * weight_decay
  float bc1, bc2;                      // 1 / (1 - beta1^t), 1 / (1 - beta2^t)
};

__device__ __forceinline__ void adamw_update(float& th, float& m, float& v, float g, const AdamW& a) {
  m = fmaf(a.beta1, m, (1.f - a.beta1) * g);
  v = fmaf(a.beta2, v, (1.f - a.beta2) * g * g);
  th = th * a.decay - a.lr * (m * a.bc1) / (sqrtf(v * a.bc2) + a.eps);
}

// One workgroup per sample b: z = W1 h + b1, a = act(z), o = W2 a + b2, p-hat = softmax(o),
// y-hat = sum_k p-hat_k c_k (Eq. 7); the true bin i of y (edges, Eq. 6), the soft
// labels p_j = exp(-|j - i|) / sum_k exp(-|k - i|); the sample's loss
// lambda3 CE(p, p-hat) + (1 - lambda3) (y - y-hat)^2 (Eq. 8),
// dL/do_k = (lambda3 (p-hat_k - p_k) - 2 (1 - lambda3) (y - y-hat) p-hat_k (c_k - y-hat)) / B and
// dL/dz_j = (sum_k dL/do_k W2[k, j]) act'(z_j).
__global__ __launch_bounds__(kHeadThreads) void train_sample_kernel(
    const float* __restrict__ part, const float* __restrict__ b1, const float* __restrict__ W2,
    const float* __restrict__ b2, const float* __restrict__ edges, const float* __restrict__ centres,
    const float* __restrict__ y, int B, int Hd, int nz, int K, int act, float lambda3, float* z_ws, float* a_ws,
    float* o_ws, float* __restrict__ dO, float* __restrict__ dZ, float* __restrict__ loss_b) {
  __shared__ float sg[1024];  // dL/do of the sample
  const int b = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* zr = z_ws + size_t(b) * Hd;
  float* a = a_ws + size_t(b) * Hd;
  float* o = o_ws + size_t(b) * K;
  for (int j = threadIdx.x; j < Hd; j += kHeadThreads) {
    const float z = hidden_sum(part, b1, b, B, Hd, nz, j);
    zr[j] = z;
    a[j] = act_fn(z, act);
  }
  __syncthreads();
  head_logits(a, W2, b2, Hd, K, o);
  __syncthreads();
  if (wave == 0) {
    const float yb = y[b];
    float mx = -INFINITY;
    int below = 0;  // edges 1 .. K-1 at or below y: the bin index
    for (int k = lane; k < K; k += 64) {
      mx = fmaxf(mx, o[k]);
      if (k >= 1 && edges[k] <= yb) ++below;
    }
    mx = wave_max(mx);
    const int i = int(wave_sum(float(below)));
    float z = 0.f, zc = 0.f, zs = 0.f;
    for (int k = lane; k < K; k += 64) {
      const float q = fast_exp2((o[k] - mx) * kLog2e);
      z += q;
      zc = fmaf(q, centres[k], zc);
      zs += expf(-fabsf(float(k - i)));
    }
    z = wave_sum(z);
    zc = wave_sum(zc);
    zs = wave_sum(zs);
    const float lse = mx + logf(z);
    const float yhat = zc / z;
    const float r = yb - yhat;
    float ce = 0.f;
    for (int k = lane; k < K; k += 64) {
      const float ph = fast_exp2((o[k] - lse) * kLog2e);
      const float pk = expf(-fabsf(float(k - i))) / zs;
      ce = fmaf(-pk, o[k] - lse, ce);
      const float g = lambda3 * (ph - pk) - 2.f * (1.f - lambda3) * r * ph * (centres[k] - yhat);
      sg[k] = g / float(B);
      dO[size_t(b) * K + k] = g / float(B);
    }
    ce = wave_sum(ce);
    if (lane == 0) loss_b[b] = lambda3 * ce + (1.f - lambda3) * r * r;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < Hd; j += kHeadThreads) {
    float g = 0.f;
#pragma unroll 8
    for (int k = 0; k < K; ++k) g = fmaf(sg[k], W2[size_t(k) * Hd + j], g);
    dZ[size_t(b) * Hd + j] = g * act_grad(zr[j], act);
  }
}

// A 32 x 128 tile of one weight matrix theta [M, N]: gradient G[i, c] = sum_b U[b, i] V[b, c] (U [B, M],
// V [B, N]) and its AdamW update.  Wave w forms columns 32 w .. + 31 on the matrix cores, two samples per
// step (lane half 0 the even one, both loads whole 128-byte runs); the tile goes through LDS so that the
// update reads and writes theta, m and v in rows.  Those are loaded before the products, which their
// latency then covers.  kVec: rows of N floats are 16-byte aligned.
constexpr int kURows = 32, kUCols = 128, kUPitch = kUCols + 4;
template <bool kVec>
__device__ __forceinline__ void update_tile(const float* __restrict__ U, const float* __restrict__ V, int B, int M,
                                            int N, int i0, int c0, float* __restrict__ th, float* __restrict__ m,
                                            float* __restrict__ v, const AdamW& opt, float (&g)[kURows][kUPitch]) {
  constexpr int kW = kVec ? 4 : 1;                          // floats per access
  constexpr int kAcc = kURows * kUCols / (256 * kW);        // accesses per thread
  constexpr int kPerRow = kUCols / kW, kRowStep = 256 / kPerRow;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int uc = int(threadIdx.x) % kPerRow * kW, ur = int(threadIdx.x) / kPerRow;
  float t[kAcc][kW], mm[kAcc][kW], vv[kAcc][kW];
  auto live = [&](int q) { return i0 + ur + kRowStep * q < M && c0 + uc < N; };
  auto at = [&](int q) { return size_t(i0 + ur + kRowStep * q) * N + c0 + uc; };
#pragma unroll
  for (int q = 0; q < kAcc; ++q)
    if (live(q)) {
      if (kVec) {
        *reinterpret_cast<float4*>(t[q]) = *reinterpret_cast<const float4*>(th + at(q));
        *reinterpret_cast<float4*>(mm[q]) = *reinterpret_cast<const float4*>(m + at(q));
        *reinterpret_cast<float4*>(vv[q]) = *reinterpret_cast<const float4*>(v + at(q));
      } else {
        t[q][0] = th[at(q)];
        mm[q][0] = m[at(q)];
        vv[q][0] = v[at(q)];
      }
    }
  {
    const int col = lane & 31, half = lane >> 5;
    const int i = i0 + col, c = c0 + 32 * wave + col;
    const float* up = U + (i < M ? i : 0);
    const float* vp = V + (c < N ? c : 0);
    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    if (c0 + 32 * wave < N) {  // this wave's columns
      constexpr int kAhead = 8;
      for (int b = 0; b < B; b += 2 * kAhead) {
        float x[kAhead], w[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
          const int bb = b + 2 * q + half;
          const bool in = bb < B;
          x[q] = in ? up[size_t(bb) * M] : 0.f;
          w[q] = in ? vp[size_t(bb) * N] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) acc = mfma32_f32(x[q], w[q], acc);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) g[mfma_row(r, half)][32 * wave + col] = acc[r];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kAcc; ++q)
    if (live(q)) {
      const float* gr = &g[ur + kRowStep * q][uc];
#pragma unroll
      for (int k = 0; k < kW; ++k) adamw_update(t[q][k], mm[q][k], vv[q][k], gr[k], opt);
      if (kVec) {
        *reinterpret_cast<float4*>(th + at(q)) = *reinterpret_cast<const float4*>(t[q]);
        *reinterpret_cast<float4*>(m + at(q)) = *reinterpret_cast<const float4*>(mm[q]);
        *reinterpret_cast<float4*>(v + at(q)) = *reinterpret_cast<const float4*>(vv[q]);
      } else {
        th[at(q)] = t[q][0];
        m[at(q)] = mm[q][0];
        v[at(q)] = vv[q][0];
      }
    }
}

// Every gradient with its AdamW update, and the batch loss, in one launch over the flat layout
// [W1 | b1 | W2 | b2]: workgroups take tiles of W1 (U = dZ, V = P), tiles of W2 (U = dO, V = A), then 32 of
// the Hd + K biases each (eight threads per bias on samples q, q + 8, ..., added in order), and the last one
// the loss (1/B) sum_b loss_b (strided per thread, then a fixed tree).  Bound by the 6 x 4 bytes per
// parameter of theta, m and v: 28 us for 64 samples, 4096 -> 1024 -> 16 on MI355X, 3.6 TB/s (the vector form,
// one row of W1 and 1024 features per workgroup, re-read every sample's features for each row: 48 us, and
// 18 us for the other parameters).
__global__ __launch_bounds__(256) void train_update_kernel(const float* __restrict__ P, const float* __restrict__ dZ,
                                                           const float* __restrict__ dO, const float* __restrict__ A,
                                                           const float* __restrict__ loss_b, int B, int d, int Hd,
                                                           int K, int n_w1, int n_w2, float* __restrict__ th,
                                                           float* __restrict__ m, float* __restrict__ v, AdamW opt,
                                                           float* __restrict__ loss) {
  __shared__ float g[kURows][kUPitch];
  int wg = blockIdx.x;
  if (wg < n_w1) {
    const int nc = (d + kUCols - 1) / kUCols;
    update_tile<true>(dZ, P, B, Hd, d, wg / nc * kURows, wg % nc * kUCols, th, m, v, opt, g);
    return;
  }
  wg -= n_w1;
  const size_t off_b1 = size_t(Hd) * d, off_w2 = off_b1 + Hd, off_b2 = off_w2 + size_t(K) * Hd;
  if (wg < n_w2) {
    const int nc = (Hd + kUCols - 1) / kUCols;
    update_tile<false>(dO, A, B, K, Hd, wg / nc * kURows, wg % nc * kUCols, th + off_w2, m + off_w2, v + off_w2, opt,
                       g);
    return;
  }
  wg -= n_w2;
  const int n_bias = (Hd + K + 31) / 32;
  float* sh = &g[0][0];
  if (wg < n_bias) {
    const int e = wg * 32 + int(threadIdx.x & 31), q = threadIdx.x >> 5;
    const bool first = e < Hd;
    float s = 0.f;
    if (e < Hd + K) {
      const float* src = first ? dZ + e : dO + (e - Hd);
      const size_t step = first ? Hd : K;
#pragma unroll 8
      for (int b = q; b < B; b += 8) s += src[size_t(b) * step];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    if (q == 0 && e < Hd + K) {
      s = 0.f;
      for (int k = 0; k < 8; ++k) s += sh[32 * k + e % 32];
      const size_t o = first ? off_b1 + e : off_b2 + (e - Hd);
      float t = th[o], mm = m[o], vv = v[o];
      adamw_update(t, mm, vv, s, opt);
      th[o] = t;
      m[o] = mm;
      v[o] = vv;
    }
    return;
  }
  float s = 0.f;
  for (int b = threadIdx.x; b < B; b += 256) s += loss_b[b];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *loss = (sh[0] + sh[1] + sh[2] + sh[3]) / float(B);
}

}  // namespace detail
}  // namespace estp

using namespace estp;
using namespace estp::detail;

extern "C" size_t estp_predict_workspace_size(int32_t B, int32_t d, int32_t hidden, int32_t K) {
  if (B < 1 || hidden < 1 || K < 1 || d < 1) return 0;
  const size_t nz = (size_t(d) + kKChunk - 1) / kKChunk;
  Carver c(nullptr);
  c.take<float>(nz * B * hidden);     // split-K partials of the first layer
  c.take<float>(size_t(B) * hidden);  // hidden activations
  c.take<float>(size_t(B) * K);       // head outputs
  return c.bytes();
}

extern "C" int estp_predict(const float* pooled, int32_t B, int32_t d, const float* W1, const float* b1,
                            int32_t hidden, int act, const float* W2, const float* b2, int32_t K,
                            const float* centres, float* yhat, int32_t* bin, int32_t* order, void* workspace,
                            size_t workspace_bytes, void* stream) {
  clear_error();
  ESTP_REQUIRE(pooled && W1 && W2 && yhat, ESTP_ERR_INVALID_ARG,
               "estp_predict: pooled, W1, W2 and yhat must be non-null");
  ESTP_REQUIRE(B >= 1 && B <= 65536 && d >= 1 && hidden >= 1 && K >= 1 && K <= 1024, ESTP_ERR_INVALID_ARG,
               "estp_predict: need 1 <= B <= 65536, d >= 1, hidden >= 1, 1 <= K <= 1024");
  ESTP_REQUIRE(d <= kMaxDepth, ESTP_ERR_UNSUPPORTED, "estp_predict: d %d exceeds %d", d, kMaxDepth);
  ESTP_REQUIRE(K == 1 || centres, ESTP_ERR_INVALID_ARG, "estp_predict: centres required when K > 1");
  ESTP_REQUIRE(act == ESTP_ACT_RELU || act == ESTP_ACT_GELU_TANH, ESTP_ERR_INVALID_ARG,
               "estp_predict: unknown activation %d", act);
  const size_t need = estp_predict_workspace_size(B, d, hidden, K);
  ESTP_REQUIRE(workspace_bytes >= need, ESTP_ERR_WORKSPACE, "estp_predict: workspace of %zu bytes, %zu needed",
               workspace_bytes, need);
  ESTP_REQUIRE(workspace && aligned(workspace, 256), ESTP_ERR_INVALID_ARG,
               "estp_predict: workspace must be non-null and 256-byte aligned");
  const int most = (d + kKChunk - 1) / kKChunk;  // of the depth shares launch_mlp_partial writes
  Carver c(workspace);
  float* part = c.take<float>(size_t(most) * B * hidden);
  float* A = c.take<float>(size_t(B) * hidden);
  float* o = c.take<float>(size_t(B) * K);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nz = launch_mlp_partial(pooled, W1, B, d, hidden, part, s);
  ESTP_CHECK_LAUNCH("mlp_partial_kernel");
  head_out_kernel<<<dim3(B), dim3(kHeadThreads), 0, s>>>(part, b1, W2, b2, centres, B, hidden, nz, K, act, A, o, yhat,
                                                K > 1 ? bin : nullptr);
  ESTP_CHECK_LAUNCH("head_out_kernel");
  if (order) {
    sjf_order_kernel<<<dim3((B + 63) / 64), dim3(64 * kOrderWaves), 0, s>>>(yhat, B, order);
    ESTP_CHECK_LAUNCH("sjf_order_kernel");
  }
  return ESTP_OK;
}

extern "C" size_t estp_head_train_step_workspace_size(int32_t B, int32_t d, int32_t hidden, int32_t K) {
  if (B < 1 || hidden < 1 || K < 1 || d < 1) return 0;
  const size_t nz = (size_t(d) + kKChunk - 1) / kKChunk;
  Carver c(nullptr);
  c.take<float>(nz * B * hidden);     // split-K partials of the first layer
  c.take<float>(size_t(B) * hidden);  // pre-activations Z
  c.take<float>(size_t(B) * hidden);  // activations A
  c.take<float>(size_t(B) * hidden);  // dL/dZ
  c.take<float>(size_t(B) * K);       // head outputs
  c.take<float>(size_t(B) * K);       // dL/do
  c.take<float>(size_t(B));           // per-sample losses
  c.take<float>(1);                   // batch loss when the caller passes none
  return c.bytes();
}

extern "C" int estp_head_train_step(const float* pooled, const float* y, int32_t B, int32_t d, int32_t hidden,
                                    int32_t K, int act, const float* edges, const float* centres, float* theta,
                                    float* m, float* v, int32_t step, float lambda3, float lr, float beta1,
                                    float beta2, float eps, float weight_decay, float* loss, void* workspace,
                                    size_t workspace_bytes, void* stream) {
  clear_error();
  ESTP_REQUIRE(pooled && y && edges && centres && theta && m && v, ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: pooled, y, edges, centres, theta, m and v must be non-null");
  ESTP_REQUIRE(B >= 1 && B <= 65536 && hidden >= 1 && K >= 2 && K <= 1024, ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: need 1 <= B <= 65536, hidden >= 1, 2 <= K <= 1024");
  ESTP_REQUIRE(d >= 4 && d % 4 == 0, ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: d must be a positive multiple of 4, got %d", d);
  ESTP_REQUIRE(d <= kMaxDepth, ESTP_ERR_UNSUPPORTED, "estp_head_train_step: d %d exceeds %d", d, kMaxDepth);
  ESTP_REQUIRE(act == ESTP_ACT_RELU || act == ESTP_ACT_GELU_TANH, ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: unknown activation %d", act);
  ESTP_REQUIRE(step >= 1, ESTP_ERR_INVALID_ARG, "estp_head_train_step: step counts from 1, got %d", step);
  ESTP_REQUIRE(lambda3 >= 0.f && lambda3 <= 1.f, ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: lambda3 must be in [0, 1]");
  ESTP_REQUIRE(lr >= 0.f && lr < INFINITY && weight_decay >= 0.f && weight_decay < INFINITY && eps > 0.f &&
                   eps < INFINITY,
               ESTP_ERR_INVALID_ARG, "estp_head_train_step: need finite lr >= 0, weight_decay >= 0, eps > 0");
  ESTP_REQUIRE(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f, ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: betas must be in [0, 1)");
  ESTP_REQUIRE(aligned(pooled, 16) && aligned(theta, 16) && aligned(m, 16) && aligned(v, 16), ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: pooled, theta, m and v must be 16-byte aligned");
  const size_t need = estp_head_train_step_workspace_size(B, d, hidden, K);
  ESTP_REQUIRE(workspace_bytes >= need, ESTP_ERR_WORKSPACE,
               "estp_head_train_step: workspace of %zu bytes, %zu needed", workspace_bytes, need);
  ESTP_REQUIRE(workspace && aligned(workspace, 256), ESTP_ERR_INVALID_ARG,
               "estp_head_train_step: workspace must be non-null and 256-byte aligned");

  const int most = (d + kKChunk - 1) / kKChunk;  // of the depth shares launch_mlp_partial writes
  Carver c(workspace);
  float* part = c.take<float>(size_t(most) * B * hidden);
  float* Z = c.take<float>(size_t(B) * hidden);
  float* A = c.take<float>(size_t(B) * hidden);
  float* dZ = c.take<float>(size_t(B) * hidden);
  float* o = c.take<float>(size_t(B) * K);
  float* dO = c.take<float>(size_t(B) * K);
  float* loss_b = c.take<float>(size_t(B));
  float* loss_ws = c.take<float>(1);
  float* W1 = theta;
  float* b1 = W1 + size_t(hidden) * d;
  float* W2 = b1 + hidden;
  float* b2 = W2 + size_t(K) * hidden;
  AdamW opt;
  opt.lr = lr;
  opt.beta1 = beta1;
  opt.beta2 = beta2;
  opt.eps = eps;
  opt.decay = float(1.0 - double(lr) * double(weight_decay));
  opt.bc1 = float(1.0 / (1.0 - std::pow(double(beta1), double(step))));
  opt.bc2 = float(1.0 / (1.0 - std::pow(double(beta2), double(step))));
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nz = launch_mlp_partial(pooled, W1, B, d, hidden, part, s);
  ESTP_CHECK_LAUNCH("mlp_partial_kernel");
  train_sample_kernel<<<dim3(B), dim3(kHeadThreads), 0, s>>>(part, b1, W2, b2, edges, centres, y, B, hidden, nz, K, act, lambda3,
                                                    Z, A, o, dO, dZ, loss_b);
  ESTP_CHECK_LAUNCH("train_sample_kernel");
  const size_t n_w1 = ((size_t(hidden) + kURows - 1) / kURows) * ((size_t(d) + kUCols - 1) / kUCols);
  const size_t n_w2 = ((size_t(K) + kURows - 1) / kURows) * ((size_t(hidden) + kUCols - 1) / kUCols);
  const size_t n_bias = (size_t(hidden) + K + 31) / 32;
  train_update_kernel<<<dim3(unsigned(n_w1 + n_w2 + n_bias + 1)), dim3(256), 0, s>>>(
      pooled, dZ, dO, A, loss_b, B, d, hidden, K, int(n_w1), int(n_w2), theta, m, v, opt, loss ? loss : loss_ws);
  ESTP_CHECK_LAUNCH("train_update_kernel");
  return ESTP_OK;
}
