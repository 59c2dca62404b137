// Token entropy (Eq. 2) for fp32 hidden states and LM-head weights, with fp32
// arithmetic throughout, on the fp32 matrix cores (v_mfma_f32_16x16x4_f32; the
// same rate as the vector FMAs, but an operand is read once per 16 products).
//
// A workgroup of 4 waves owns one token tile and, in turn, the vocabulary tiles
// of one vocabulary slice (tiles slice, slice + n_vsplit, ...).  Wave (wv, wt)
// forms 16 NB vocabulary rows x 16 NB tokens: vocabulary rows on the M side, so
// that a lane owns NB token columns and folds its rows in registers.  Both
// operands are contiguous along the hidden dimension: a lane loads 16 bytes of
// its row, which feed four matrix-core steps (step c multiplies depths k + c,
// k + 4 + c, k + 8 + c and k + 12 + c), straight from global memory, one
// 128-byte line of each row ahead of the products.  After the last depth of a
// tile a lane folds its logits into one online-softmax state per token column
// (Ent2, base 2; exact, with the tile's own max).  At the end the lanes and
// waves that share a token column merge their states in a fixed order and the
// slice writes the partial layout that entropy_merge_kernel reduces.  The kArg
// variant also keeps each token column's largest logit and its lowest
// vocabulary index through the same merges.
//
// NB = 4 (128 x 128 tiles) re-reads least; NB = 2 (64 x 64) spreads calls whose
// larger tiles would leave compute units idle.  Times on MI355X, of
// the vector form (8 x 8 logits per thread from k-major LDS tiles of 128 x 128,
// 16 slices) and this: 128 tokens, d 64, V 1000 34 and 22 us (launches and the
// merge included); 700 tokens, d 1536, V 32000 4.66 and 1.15 ms; 8192 tokens,
// d 4096, V 32768 31.4 and 18.5 ms (70 and 119 of 157 TFLOP/s).
#include <algorithm>

#include "estp_common.h"
#include "f32_paths.h"

namespace estp {
namespace detail {

// b replaces a when larger, or equal with a lower index.
__device__ __forceinline__ void arg_merge_f32(float& av, int& ai, float bv, int bi) {
  const bool take = bv > av || (bv == av && bi < ai);
  av = take ? bv : av;
  ai = take ? bi : ai;
}

template <int NB, bool kArg>
__global__ __launch_bounds__(256, NB == 4 ? 2 : 3) void entropy_f32_kernel(const float* __restrict__ X, const float* __restrict__ W,
                                                          int n_tok, int d, int V, int n_vsplit, int n_vt,
                                                          float* __restrict__ part_m, float* __restrict__ part_s,
                                                          float* __restrict__ part_t,
                                                          float* __restrict__ part_zmax,
                                                          int* __restrict__ part_arg) {
  constexpr int kWT = 16 * NB;  // rows of either operand per wave
  constexpr int kT = 2 * kWT;   // and per workgroup
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = wave & 1, wt = wave >> 1;
  const int row = lane & 15, grp = lane >> 4;
  const int slice = blockIdx.x % n_vsplit;
  const int t0 = (blockIdx.x / n_vsplit) * kT + wt * kWT;  // the wave's first token
  const int n_mine = (n_vt - slice + n_vsplit - 1) / n_vsplit;  // vocabulary tiles of this slice

  // Resources that end with the last live row: rows past V or n_tok read as zero (a wave with none
  // has an empty one), and so do depths past d, sent to an offset past the end.
  const buf_rsrc_t rx =
      make_rsrc(X + size_t(min(t0, n_tok)) * d, uint32_t(max(0, min(kWT, n_tok - t0))) * uint32_t(d) * 4u);
  constexpr int kHalves = NB == 4 ? 1 : 2, kStep = 16 * kHalves;  // two register sets of one step each
  struct Step {
    f32x4_t a[kHalves][NB], b[kHalves][NB];
  };
  auto load_step = [&](Step& f, const buf_rsrc_t& rw, int k0) {
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
      const int k = k0 + 16 * h + 4 * grp;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const uint32_t off = k < d ? (uint32_t(16 * i + row) * uint32_t(d) + uint32_t(k)) * 4u : kPastEnd;
        f.a[h][i] = buf_load4(rw, off);
        f.b[h][i] = buf_load4(rx, off);
      }
    }
  };

  Ent2 st[NB];
  float zmax[NB];  // kArg: largest logit per token column and its vocabulary index
  int zarg[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    st[j] = Ent2{-INFINITY, 0.f, 0.f};
    zmax[j] = -INFINITY;
    zarg[j] = INT32_MAX;
  }
  for (int tile = 0; tile < n_mine; ++tile) {
    const int v0 = (slice + tile * n_vsplit) * kT + wv * kWT;  // the wave's first vocabulary row
    const buf_rsrc_t rw =
        make_rsrc(W + size_t(min(v0, V)) * d, uint32_t(max(0, min(kWT, V - v0))) * uint32_t(d) * 4u);
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
    Step f0, f1;
    load_step(f0, rw, 0);
    for (int k = 0; k < d; k += 2 * kStep) {  // steps past d: zeros, no access
      load_step(f1, rw, k + kStep);
      __builtin_amdgcn_sched_barrier(0);  // the loads go out before the products, not behind them
      multiply(f0);
      __builtin_amdgcn_sched_barrier(0);
      if (k + kStep >= d) break;
      load_step(f0, rw, k + 2 * kStep);
      __builtin_amdgcn_sched_barrier(0);
      multiply(f1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // acc[i][j][r]: vocabulary row v0 + 16 i + 4 grp + r, token t0 + 16 j + row; rows past V left out
    const int lim = V - v0 - 4 * grp;  // live: 16 i + r < lim
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float mx = -INFINITY;
      int imx = 0;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // rows ascend: a strict compare keeps the lowest index among equal logits
          const bool up = (16 * i + r < lim) & (acc[i][j][r] > mx);
          imx = up ? 16 * i + r : imx;
          mx = up ? acc[i][j][r] : mx;
        }
      if (kArg && mx > zmax[j]) {
        zmax[j] = mx;
        zarg[j] = v0 + 4 * grp + imx;
      }
      if (lim > 0) {  // the lane's first row is its lowest; none live -> nothing to add
        const float m2 = mx * kLog2e;
        float s = 0.f, t = 0.f;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float z = fmaf(acc[i][j][r], kLog2e, -m2);
            const float p = fast_exp2(z);
            const bool in = 16 * i + r < lim;
            s += in ? p : 0.f;
            t = in ? fmaf(p, z, t) : t;
          }
        st[j] = ent2_merge(st[j], Ent2{m2, s, t});
      }
    }
  }

  // lanes row, row + 16, row + 32 and row + 48 share their token columns ...
#pragma unroll
  for (int j = 0; j < NB; ++j) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const Ent2 other{__shfl_xor(st[j].m, o, 64), __shfl_xor(st[j].s, o, 64), __shfl_xor(st[j].t, o, 64)};
      st[j] = ent2_merge(st[j], other);
      if (kArg) arg_merge_f32(zmax[j], zarg[j], __shfl_xor(zmax[j], o, 64), __shfl_xor(zarg[j], o, 64));
    }
  }
  // ... and so do the two waves of a token half: merged through LDS
  __shared__ float red[5][kT];
  if (wv == 1 && grp == 0) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int col = wt * kWT + 16 * j + row;
      red[0][col] = st[j].m;
      red[1][col] = st[j].s;
      red[2][col] = st[j].t;
      red[3][col] = zmax[j];
      red[4][col] = __int_as_float(zarg[j]);
    }
  }
  __syncthreads();
  if (wv == 0 && grp == 0) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int col = wt * kWT + 16 * j + row, tok = t0 + 16 * j + row;
      if (tok >= n_tok) continue;
      const Ent2 a = ent2_merge(st[j], Ent2{red[0][col], red[1][col], red[2][col]});
      const size_t o = size_t(slice) * n_tok + tok;
      part_m[o] = a.m;
      part_s[o] = a.s;
      part_t[o] = a.t;
      if (kArg) {
        arg_merge_f32(zmax[j], zarg[j], red[3][col], __float_as_int(red[4][col]));
        part_zmax[o] = zmax[j];
        part_arg[o] = zarg[j];
      }
    }
  }
}

namespace {
size_t tiles_of(int n, int t) { return (size_t(n) + t - 1) / t; }
// 64 x 64 tiles where 128 x 128 ones (of at most max_slices vocabulary slices) would not give every CU one
bool small_tiles(int n_tok, int V, int max_slices) {
  return tiles_of(n_tok, 128) * std::min<size_t>(tiles_of(V, 128), max_slices) < 256;
}
}  // namespace

int entropy_f32_slices(int n_tok, int V, int max_slices) {
  return int(std::min<size_t>(tiles_of(V, small_tiles(n_tok, V, max_slices) ? 64 : 128), max_slices));
}

size_t entropy_f32_workgroups(int n_tok, int V, int max_slices) {
  return size_t(entropy_f32_slices(n_tok, V, max_slices)) *
         tiles_of(n_tok, small_tiles(n_tok, V, max_slices) ? 64 : 128);
}

void launch_entropy_f32(const float* X, const float* W, int n_tok, int d, int V, int max_slices, float* part_m,
                        float* part_s, float* part_t, float* part_zmax, int* part_arg, hipStream_t s) {
  const bool small = small_tiles(n_tok, V, max_slices);
  const int n_vt = int(tiles_of(V, small ? 64 : 128)), slices = entropy_f32_slices(n_tok, V, max_slices);
  const dim3 grid(unsigned(entropy_f32_workgroups(n_tok, V, max_slices))), block(256);
  auto go = [&](auto kernel) {
    kernel<<<grid, block, 0, s>>>(X, W, n_tok, d, V, slices, n_vt, part_m, part_s, part_t, part_zmax, part_arg);
  };
  if (small) {
    if (part_arg)
      go(entropy_f32_kernel<2, true>);
    else
      go(entropy_f32_kernel<2, false>);
  } else {
    if (part_arg)
      go(entropy_f32_kernel<4, true>);
    else
      go(entropy_f32_kernel<4, false>);
  }
}

}  // namespace detail
}  // namespace estp
