// Attention importance, Eq. 1 (Section 4.1), in one pass for prompts of up to
// 2048 tokens (bf16): every score is formed and exponentiated once.
//
// The two-pass kernels (importance.hip) form each score twice, because a
// column sum needs the row normalisers of all later rows.  Here a workgroup
// keeps the exponentials of 32 whole rows in registers until their sums are
// known: wave w of W owns the 32-key blocks w, w + W, ... (at most 8, 128 fp32
// registers per lane), forms S = Q K^T for the row block against each of them
// (queries on the MFMA "M" side: a lane owns one key column and 16 rows),
// takes p = 2^(c s) in place and adds the rows' sums; the waves exchange those
// through LDS (one barrier per row block), and each adds p / Z to its own
// columns' masses, which stay in registers for the whole walk over the
// workgroup's heads and row blocks.
//
// Exponentials are taken without a row maximum: fp32 holds 2^(c s) for
// |c s| < 126 with the relative precision of the score itself.  A row block
// with a live row whose sum leaves [2^-30, 2^100] (or is not a number) is
// formed again, and those after it are formed so at once while their rows need
// it: each wave keeps the scores until it knows its own keys' row maxima, takes
// those off, and the waves' sums and weights are put on one scale as they are
// exchanged.  us per call on MI355X, ordinary scores, every row out of range, and
// the two passes on the latter: 16 x 512 tokens, 32/8 heads of 128 66, 80 and 95,
// 16 x 2048 581, 658 and 609; heads of 64 384, 490 and 427.  (Such a row block formed
// three more times, a key block at a time, took 351, 4450 and 2780.)
//
// Keys stream through per-wave LDS rings of 32-key x 64-feature pieces
// (buffer -> LDS transfers, no barrier: a wave reads only its own ring), across
// row-block boundaries; the 32 queries of the next row block arrive in a shared
// double buffer meanwhile.
//
// What bounds it: registers allow two waves per SIMD, and a row block costs a
// wave about 3500 cycles besides its key blocks (first products with nothing
// behind them, last exponentials, the exchange and its barrier) and about 1500
// per key block, half of it vector issue (one exponential, a multiply, an add
// and an FMA per score): 32 x 2048 tokens, 32/8 heads of 128 run at 50% vector
// and 21% matrix-core issue at 2.0 GHz.
//
// Work split.  A KV group's query heads go to hsplit workgroups and a prompt's
// row blocks, interleaved, to rsplit: workgroups that share keys run next to
// each other on one XCD.  Each writes a row of column masses (zero where it
// saw nothing), which attn_reduce_kernel adds in a fixed order.
#include <algorithm>
#include <type_traits>

#include "attn_tiles.h"

namespace estp {
namespace detail {
namespace {

constexpr int kBlocks = 8;  // most 32-key blocks per wave

// Sum (or maximum: op) of v[r] over the 32 lanes of a half-wave, for each r of 16: lane l ends with that of
// r = l % 16 (butterflies that halve the values each step, then the two 16-lane rows).
template <int kCtrl>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}
template <typename Op>
__device__ __forceinline__ float reduce16(const float (&v)[16], int lane, Op op) {
  float a[8], b[4], c[2];
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = op(b3 ? v[k + 8] : v[k], dpp_mov<0x140>(b3 ? v[k] : v[k + 8]));  // row mirror
#pragma unroll
  for (int k = 0; k < 4; ++k) b[k] = op(b2 ? a[k + 4] : a[k], dpp_mov<0x141>(b2 ? a[k] : a[k + 4]));  // half mirror
#pragma unroll
  for (int k = 0; k < 2; ++k) c[k] = op(b1 ? b[k + 2] : b[k], dpp_mov<0x4e>(b1 ? b[k] : b[k + 2]));  // lane ^ 2
  const float d = op(b0 ? c[1] : c[0], dpp_mov<0xb1>(b0 ? c[0] : c[1]));                             // lane ^ 1
  return op(d, __shfl_xor(d, 16, 64));
}

// A value the compiler cannot see through: keeps the 16 diagonal masks of a lane (32 scalar
// registers) from being formed once, ahead of the loops, and spilled.
__device__ __forceinline__ int opaque(int x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(x));
#endif
  return x;
}

// The same for a uniform value: the pieces' addresses are formed in each row block from it, not once ahead of the
// loops for all bodies, and spilled (128 scalar registers; 9 prompts of 45-1021 tokens 28.8 us, so 26.2).
__device__ __forceinline__ uint32_t opaque_uniform(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+s"(x));
#endif
  return x;
}

template <int DH, int W>
__global__ __launch_bounds__(64 * W, 2) void attn_onepass_kernel(const uint16_t* __restrict__ Q,
                                                                 const uint16_t* __restrict__ K,
                                                                 const int* __restrict__ cu, int B, int n_tok, int L,
                                                                 int Hq, int Hkv, float c2, int strict, int hsplit,
                                                                 int rsplit, float* __restrict__ part) {
  constexpr int PD = DH < 64 ? DH : 64;  // features of a key piece
  constexpr int NP = DH / PD;            // pieces per key block
  constexpr int KS = DH / 16, KP = PD / 16;
  using TK = RowTile<PD>;
  using TQ = RowTile<DH>;
  constexpr int kPiece = 32 * TK::kRowBytes;
  constexpr int PI = kPiece / 1024;  // transfers per piece
  constexpr int S = W == 8 ? 4 : 3;  // ring slots (two workgroups of 4 waves share a CU's LDS)
  constexpr int kQTile = 32 * TQ::kRowBytes;
  constexpr int QI = kQTile / 1024;  // transfers per query tile, dealt over the waves
  // One shared array: several would be told apart by alias scopes, and the compiler then guards every
  // read of any of them with a wait for all transfers into LDS in flight.
  constexpr int kRing = 0, kQ = W * S * kPiece, kZ = kQ + 2 * kQTile, kM = kZ + 2 * W * 32 * 4;
  constexpr int kWt = kM + 2 * W * 32 * 4;
  __shared__ __attribute__((aligned(16))) char lds[kWt + W * 32 * 4];
  auto ring = [&](int wave, int slot) { return lds + kRing + (wave * S + slot) * kPiece; };
  auto qbuf = [&](int buf) { return lds + kQ + buf * kQTile; };
  auto zsum = [&](int buf, int wave) { return reinterpret_cast<float*>(lds + kZ) + (buf * W + wave) * 32; };
  auto zmax = [&](int buf, int wave) { return reinterpret_cast<float*>(lds + kM) + (buf * W + wave) * 32; };
  auto wrow = [&](int wave) { return reinterpret_cast<float*>(lds + kWt) + wave * 32; };

  // workgroup -> (unit, share): an eighth of the units to each XCD, the shares of a unit (same keys)
  // next to each other there; units: prompt fastest, then KV head and layer
  const int shares = hsplit * rsplit;
  const int xcd = blockIdx.x & 7, jx = blockIdx.x >> 3;
  const int unit = (jx / shares) * 8 + xcd, share = jx % shares;
  if (unit >= B * L * Hkv) return;
  const int hs = share / rsplit, rs0 = share % rsplit;
  const int b = unit % B, lg = unit / B;
  const int l = lg / Hkv, g = lg % Hkv;
  const int base = cu[b];
  const int N = min(cu[b + 1] - base, 32 * kBlocks * W);  // the host guarantees N <= 256 W
  const int G = Hq / Hkv, hpw = G / hsplit;
  const int nrb = (N + 31) / 32;

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const uint32_t qrow = uint32_t(Hq) * DH * 2, krow = uint32_t(Hkv) * DH * 2;  // bytes
  const char* Qh = reinterpret_cast<const char*>(Q) + (size_t(l) * n_tok + base) * qrow +
                   size_t(g * G + hs * hpw) * DH * 2;
  const char* Kg = reinterpret_cast<const char*>(K) + (size_t(l) * n_tok + base) * krow + size_t(g) * DH * 2;
  const uint32_t k_bytes = uint32_t(N - 1) * krow + DH * 2;  // rows past the prompt's end read as zero

  // ---- key ring.  Every row block reads the wave's key blocks from the first on, so the pieces that
  // follow a row block's last are always pieces 0, 1, ... of the next: which piece to transfer is known
  // when the row block's body is compiled, and only the slot rotates.
  uint32_t k_off[PI];
#pragma unroll
  for (int q = 0; q < PI; ++q) {
    const int r = q * TK::kRowsPerInst + lane / TK::kChunks;
    k_off[q] = uint32_t(r) * krow + uint32_t(TK::swz(r, lane % TK::kChunks) * 16);
  }
  const uint32_t k_first = uint32_t(w) * 32u * krow, k_step = uint32_t(W) * 32u * krow;
  // piece idx (key block idx / NP of the wave, features PD (idx % NP) ...) into a slot
  auto issue_piece = [&](int idx, int to, uint32_t first, uint32_t step) {
    const uint32_t at = first + uint32_t(idx / NP) * step + uint32_t(idx % NP) * (PD * 2);
    const buf_rsrc_t r = make_rsrc(Kg + at, uint32_t(max(0, int(k_bytes) - int(at))));  // past the prompt: no access
#pragma unroll
    for (int q = 0; q < PI; ++q) lds_dma16_buf(r, k_off[q], 0, ring(w, to) + q * 1024);
  };
  // ---- query tile of row block i, head share hh.  Rows past the prompt take its last query again: zeros there
  // would meet an infinite key feature as NaN, which a row weight of 0 does not keep out of the key's mass.
  auto issue_q = [&](int hh, int i, int buf) {
    const int rows = min(32, N - 32 * i);
    const buf_rsrc_t rq = make_rsrc(Qh + size_t(32 * i) * qrow + size_t(hh) * DH * 2,
                                    uint32_t(rows - 1) * qrow + DH * 2);
#pragma unroll
    for (int q = w; q < QI; q += W) {
      const int r = q * TQ::kRowsPerInst + lane / TQ::kChunks;
      lds_dma16_buf(rq, uint32_t(min(r, rows - 1)) * qrow + uint32_t(TQ::swz(r, lane % TQ::kChunks) * 16), 0,
                    qbuf(buf) + q * 1024);
    }
  };

  float csum[kBlocks];
#pragma unroll
  for (int c = 0; c < kBlocks; ++c) csum[c] = 0.f;

  if (rs0 < nrb) {
    issue_q(0, rs0, 0);
#pragma unroll
    for (int q = 0; q < S - 1; ++q) issue_piece(q, q, k_first, k_step);
    wait_vm<0>();
    lds_barrier();
    int slot = 0, par = 0, i = rs0;  // slot: of the next piece to read; i: the row block
    bool far = false;                // the last row block's sums were out of the plain form's range
    // acc[r] of a block: query 32 i + 8 (r / 4) + 4 half + r % 4, key 32 (w + W c) + col

    // ---- one row block against this wave's CNT key blocks; one body per CNT, so that the scores stay in
    // the same registers from their products to their masses.  kMax: relative to the row maxima of the wave's
    // keys.  Returns whether a live row's sum is out of the plain form's range: only with kMax are the masses
    // added then.
    auto row_block = [&](auto cnt_c, auto max_c) {
      constexpr int CNT = decltype(cnt_c)::value;
      constexpr bool kMax = decltype(max_c)::value;
      const bool diag = CNT > 0 && w + W * (CNT - 1) == i;  // the last block holds the diagonal
      f32x16_t sc[CNT > 0 ? CNT : 1];
      float rs[16];  // row sums (kMax: at first the row maxima)
#pragma unroll
      for (int r = 0; r < 16; ++r) rs[r] = kMax && CNT > 0 ? -INFINITY : 0.f;
      // 16 values of a row of 32, those of this lane's accumulator rows
      auto rows_of = [&](const float* p, float (&v)[16]) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const float4 x = *reinterpret_cast<const float4*>(p + 8 * q4 + 4 * half);
          v[4 * q4] = x.x;
          v[4 * q4 + 1] = x.y;
          v[4 * q4 + 2] = x.z;
          v[4 * q4 + 3] = x.w;
        }
      };
      if constexpr (CNT > 0) {
        const uint32_t kf = opaque_uniform(k_first), k_st = opaque_uniform(k_step);
        bf16x8_t aq[KS];
        const int qc = opaque(col);  // its addresses formed here, not kept through the loops
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          aq[ks] = *reinterpret_cast<const bf16x8_t*>(qbuf(par) + TQ::off(qc, ks * 2 + half));
        auto exps = [&](f32x16_t& acc, int from, int to) {
#pragma unroll
          for (int r = from; r < to; ++r) {
            if constexpr (kMax) {
              rs[r] = fmaxf(rs[r], acc[r]);
            } else {
              acc[r] = fast_exp2(acc[r] * c2);
              rs[r] += acc[r];
            }
          }
        };
        // behind step q of the row block: the piece S - 1 further on, into the slot read last
        constexpr int kSteps = CNT * NP > S - 1 ? CNT * NP : S - 1;
        auto refill = [&](int q) {
          const int idx = q + S - 1 < kSteps ? q + S - 1 : q + S - 1 - kSteps;
          issue_piece(idx, slot == 0 ? S - 1 : slot - 1, kf, k_st);
        };
#pragma unroll
        for (int c = 0; c < CNT; ++c) {
          // the scores of block c, piece by piece (the transfers of the piece S - 1 ahead go into the slot
          // read last); behind each piece's reads, a share of the exponentials of the block before it,
          // which the matrix cores' work of the piece before covers
#pragma unroll
          for (int r = 0; r < 16; ++r) sc[c][r] = 0.f;
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            // the piece has landed, and the reads of the slot refilled next are done
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            wait_vm_lds<(S - 2) * PI>();
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            refill(c * NP + p);
            const char* kt = ring(w, slot);
            bf16x8_t bk[KP];
#pragma unroll
            for (int kk = 0; kk < KP; ++kk) bk[kk] = *reinterpret_cast<const bf16x8_t*>(kt + TK::off(col, kk * 2 + half));
            __builtin_amdgcn_sched_barrier(0);
            if (c > 0) exps(sc[c > 0 ? c - 1 : 0], 16 / NP * p, 16 / NP * (p + 1));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < KP; ++kk)
              sc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[p * KP + kk], bk[kk], sc[c], 0, 0, 0);
            slot = slot + 1 == S ? 0 : slot + 1;
          }
        }
        // a row block of fewer pieces than are kept ahead passes over the others
#pragma unroll
        for (int q = CNT * NP; q < kSteps; ++q) {
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          wait_vm_lds<(S - 2) * PI>();
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          refill(q);
          slot = slot + 1 == S ? 0 : slot + 1;
        }
        if (diag) {
          const int t = opaque(col - 4 * half);
#pragma unroll
          for (int r = 0; r < 16; ++r) sc[CNT - 1][r] = 8 * (r >> 2) + (r & 3) < t ? -INFINITY : sc[CNT - 1][r];
        }
        exps(sc[CNT - 1], 0, 16);
        if constexpr (kMax) {
          // the wave's row maxima in base-2 units; rows whose every score is -inf stay above them, and add 0
          const int ln = opaque(lane), out_row = 8 * ((ln & 15) >> 2) + 4 * half + (ln & 3);  // row of reduce16's value
          const float m = fmaxf(reduce16(rs, ln, [](float x, float y) { return fmaxf(x, y); }) * c2, -1e30f);
          if ((ln & 16) == 0) zmax(par, w)[out_row] = m;
          __builtin_amdgcn_wave_barrier();
          float ref[16];
          rows_of(zmax(par, w), ref);
#pragma unroll
          for (int r = 0; r < 16; ++r) rs[r] = 0.f;
#pragma unroll
          for (int c = 0; c < CNT; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              sc[c][r] = fast_exp2(fmaf(sc[c][r], c2, -ref[r]));
              rs[r] += sc[c][r];
            }
        }
      } else if constexpr (kMax) {
        if (lane < 32) zmax(par, w)[lane] = -1e30f;
      }

      // row sums over the workgroup: one barrier (double buffered), which also publishes the next row
      // block's queries (older than the S - 1 pieces that follow this row block's)
      {
        const int ln = opaque(lane), out_row = 8 * ((ln & 15) >> 2) + 4 * half + (ln & 3);
        const float z = reduce16(rs, ln, [](float x, float y) { return x + y; });
        if ((ln & 16) == 0) zsum(par, w)[out_row] = z;
      }
      if constexpr (CNT > 0)
        wait_vm<(S - 1) * PI>();
      else
        wait_vm<0>();
      lds_barrier();
      const bool live = 32 * i + col < N;
      float Z = 0.f, M = 0.f;  // the row's sum is Z 2^M
      bool out;
      if constexpr (kMax) {
        M = zmax(par, 0)[col];
#pragma unroll
        for (int q = 1; q < W; ++q) M = fmaxf(M, zmax(par, q)[col]);
#pragma unroll
        for (int q = 0; q < W; ++q) Z = fmaf(zsum(par, q)[col], fast_exp2(zmax(par, q)[col] - M), Z);
        const float z2 = M + fast_log2(Z);
        out = __any(live && !(z2 >= -30.f && z2 <= 100.f));
      } else {
#pragma unroll
        for (int q = 0; q < W; ++q) Z += zsum(par, q)[col];
        out = __any(live && !(Z >= 0x1p-30f && Z <= 0x1p100f));
        if (__builtin_expect(out, 0)) return true;
      }
      if constexpr (CNT > 0) {
        // this wave's copy of the row weights (0 past the prompt), 16 per lane
        const float scale = kMax ? fast_exp2(zmax(par, w)[col] - M) : 1.f;
        if (lane < 32) wrow(w)[col] = live ? scale / Z : 0.f;
        float wt[16];
        rows_of(wrow(w), wt);
#pragma unroll
        for (int c = 0; c < CNT - 1; ++c) {
          float s0 = csum[c], s1 = 0.f;
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            s0 = fmaf(sc[c][r], wt[r], s0);
            s1 = fmaf(sc[c][r + 1], wt[r + 1], s1);
          }
          csum[c] = s0 + s1;
        }
        // masked probabilities stay out also where a weight is not a number, and the diagonal itself when
        // self-attention is excluded
        const int t = diag ? opaque(col - 4 * half + strict) : -32;
        float s0 = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) s0 += 8 * (r >> 2) + (r & 3) < t ? 0.f : sc[CNT - 1][r] * wt[r];
        csum[CNT - 1] += s0;
      }
      return out;
    };
    for (int hh = 0; hh < hpw; ++hh)
      for (i = rs0; i < nrb; i += rsplit, par ^= 1) {
        if (i + rsplit < nrb)
          issue_q(hh, i + rsplit, par ^ 1);
        else if (hh + 1 < hpw)
          issue_q(hh + 1, rs0, par ^ 1);
        const int cnt = i >= w ? (i - w) / W + 1 : 0;  // key blocks of this wave up to the diagonal
        auto go = [&](auto max_c) {
          switch (cnt) {
            case 0: return row_block(std::integral_constant<int, 0>{}, max_c);
            case 1: return row_block(std::integral_constant<int, 1>{}, max_c);
            case 2: return row_block(std::integral_constant<int, 2>{}, max_c);
            case 3: return row_block(std::integral_constant<int, 3>{}, max_c);
            case 4: return row_block(std::integral_constant<int, 4>{}, max_c);
            case 5: return row_block(std::integral_constant<int, 5>{}, max_c);
            case 6: return row_block(std::integral_constant<int, 6>{}, max_c);
            case 7: return row_block(std::integral_constant<int, 7>{}, max_c);
            default: return row_block(std::integral_constant<int, 8>{}, max_c);
          }
        };
        // the same in every wave, which all read the same sums
        if (!far) {
          far = go(std::false_type{});
          // again: the pieces in flight are this wave's first ones and the queries are still there; every wave
          // has read the sums before they are written again
          if (__builtin_expect(far, 0)) __syncthreads();
        }
        if (__builtin_expect(far, 0)) far = go(std::true_type{});
      }
    wait_vm<0>();  // no transfer into LDS outlives the workgroup
  }
  // the two row halves (lane, lane + 32) of each key column
  float* out = part + (size_t(lg) * shares + share) * n_tok + base;
#pragma unroll
  for (int c = 0; c < kBlocks; ++c) {
    const float v = csum[c] + __shfl_xor(csum[c], 32, 64);
    const int j = 32 * (w + W * c) + col;
    if (half == 0 && j < N) out[j] = v;
  }
}

template <int DH>
void launch_dh(const OnepassPlan& p, unsigned grid, const uint16_t* Q, const uint16_t* K, const int* cu, int B,
               int n_tok, int L, int Hq, int Hkv, float c2, int strict, float* part, hipStream_t s) {
  if (p.waves == 8)
    attn_onepass_kernel<DH, 8><<<dim3(grid), dim3(512), 0, s>>>(Q, K, cu, B, n_tok, L, Hq, Hkv, c2, strict, p.hsplit,
                                                                p.rsplit, part);
  else
    attn_onepass_kernel<DH, 4><<<dim3(grid), dim3(256), 0, s>>>(Q, K, cu, B, n_tok, L, Hq, Hkv, c2, strict, p.hsplit,
                                                                p.rsplit, part);
}

size_t onepass_grid(const OnepassPlan& p, int B, int L, int Hkv) {
  const size_t units = size_t(B) * L * Hkv;
  return (units + 7) / 8 * 8 * size_t(p.hsplit) * p.rsplit;
}

}  // namespace

// Whether row shares of heads of 32 or 64, up to 1024 tokens and with few KV heads, end in so many workgroups of a row
// block or two that the two passes are faster: an estimate of both in us, fitted to 1200 calls of random shapes on
// MI355X (row blocks, key blocks of the busiest wave and workgroups over the 512 resident, and the column masses; each
// estimate within 20% of nearly every call).  Two passes and one, 166 prompts of up to 335 tokens, 7/1 heads of 64 65
// and 88, 170 of 230, 6/2 of 32 34.6 and 41, 61 of 171-342, 28/4 of 64 82 and 118.  With eight KV heads, and below
// 4096 tokens, the one pass was the faster one or within a few us.
bool shares_too_fine(const OnepassPlan& p, int64_t n_tok, int B, int L, int Hq, int Hkv, int dh) {
  if (dh == 128 || p.waves != 4 || Hkv > 4 || n_tok < 4096) return false;
  const float n = float(n_tok), heads = float(L) * float(Hq), scores = heads * n * (n / float(B));  // as if equal
  const float row_blocks = heads * (n / 32.f + float(B) / 2.f), key_blocks = scores / 8192.f + 0.4f * row_blocks;
  const float shares = float(L) * float(Hkv) * float(p.rsplit * p.hsplit);
  const float one = 8.5f + (1.25f * row_blocks + (dh == 32 ? 0.25f : 0.38f) * key_blocks + shares * float(B)) / 512.f +
                    6e-6f * shares * n;
  const float two = 27.f + 1.4f * scores / (8192.f * 768.f) + (dh == 32 ? 6e-6f : 25e-6f) * heads * n;
  return one > 0.95f * two;
}

// One pass for prompts of up to 2048 tokens where it is the faster one.  us per call on MI355X, two passes and
// one, 32/8 heads of 128, 1 layer: 1 x 500 tokens 45 and 20, 1 x 2048 128 and 70, 16 x 512 83 and 66, 600 x 64
// 217 and 166, 32 x 1024 380 and 335, 32 x 2048 1290 and 1150 (4 layers: 5422 and 4293).  Two passes stay
// - for batches of mixed lengths unless they are small: every workgroup walks whole rows of its prompt, so the
//   longest prompts decide (64 prompts of 32-2048 tokens 485 and 630, 16 of them 148 and 267; 9 prompts of
//   45-1021 tokens, 12/2 heads 67 and 27; 30 of 500-900 210 and 171);
// - for large calls with smaller heads, whose scores cost less to form again (heads of 64: 16 x 2048 438 and
//   402, 32 x 512 with 4 layers 310 and 316, 100 x 100 55 and 59; heads of 32: 20 x 1500 249 and 264);
// - past 1024 tokens, where workgroups of eight waves leave most of their last key blocks idle, for all but small
//   calls: with heads of 32 and 64 (1051 tokens, 16/4 heads of 64 166 and 206; 69 prompts of 593-1187 262 and 306;
//   1156 tokens, 8/1 of 32 72 and 96; equal prompts near 2048 gain with heads of 64, 27 x 1920, 24/8 486 and 448), and
//   with heads of 128 where lengths differ (8 prompts of 524-1048, 48/8 heads 136 and 158; equal, 24/8 at 1544 tokens
//   839 and 772);
// - where the shares get too fine.
// Shares: row blocks over up to 8 workgroups (they stream the same keys through one L2) of at least 16 row
// blocks each while there are enough workgroups, then more, then a group's heads, then single row blocks.  A group
// of a prime number of heads stays whole where its split would give more than twice the workgroups wanted and half of
// them are there (61 prompts of 171-342 tokens, 28/4 heads of 64: 118 split, 80 whole).
OnepassPlan plan_onepass(int64_t n_tok, int B, int max_seqlen, int L, int Hq, int Hkv, int dh, bool f32,
                         bool with_lse) {
  OnepassPlan p{0, 1, 1};
  if (f32 || with_lse || max_seqlen > 2048) return p;
  if (size_t(Hq) * dh * 2 * 2048 >= (size_t(1) << 31)) return p;  // 32-bit offsets inside a prompt
  const size_t n_cu = size_t(std::max(1, current_device_cu_count()));
  const size_t blocks = std::min<size_t>(size_t(n_tok) / 256 + B, (size_t(max_seqlen) + 255) / 256 * B);
  const size_t wgs = blocks * L * Hq;  // of the two-pass kernels' first pass
  const bool even = size_t(B) * max_seqlen * 4 <= size_t(n_tok) * 7;  // the longest within 1.75 of the mean
  if (!even && wgs * 2 > 3 * n_cu) return p;
  if (dh < 128 && wgs >= size_t(dh == 64 && max_seqlen > 256 ? 24 : 8) * n_cu) return p;
  const int G = Hq / Hkv, nrb = (max_seqlen + 31) / 32;
  const int waves = max_seqlen <= 1024 ? 4 : 8;
  const bool few = wgs * 2 < 7 * n_cu;
  if (waves == 8 && !few) {
    const bool differ = size_t(n_tok) * 20 < size_t(B) * max_seqlen * 19;  // the mean under 95% of the longest
    if (dh == 128 ? differ && max_seqlen <= 1408 : dh < 64 || differ || max_seqlen <= 1792) return p;
  }
  const size_t want = size_t(waves == 8 ? 4 : 8) * n_cu;
  const size_t units = size_t(B) * L * Hkv;
  p.rsplit = std::max(1, std::min(8, G * nrb / 16));
  while (p.rsplit < std::min(8, nrb) && units * p.rsplit < want) ++p.rsplit;
  for (int h = 2; h <= G && units * p.rsplit * p.hsplit < want; ++h)
    if (G % h == 0) {
      if (units * p.rsplit * h > 2 * want && units * p.rsplit * p.hsplit * 2 >= want) break;
      p.hsplit = h;
    }
  if (units * p.rsplit * p.hsplit < want)
    p.rsplit = int(std::min<size_t>(nrb, (want + units * p.hsplit - 1) / (units * p.hsplit)));
  if (!fits_launch(onepass_grid(p, B, L, Hkv), size_t(64) * waves)) return p;
  p.waves = waves;
  if (shares_too_fine(p, n_tok, B, L, Hq, Hkv, dh)) p.waves = 0;
  return p;
}

void launch_onepass(const OnepassPlan& p, int dh, const uint16_t* Q, const uint16_t* K, const int* cu, int B,
                    int n_tok, int L, int Hq, int Hkv, float c2, int strict, float* part, hipStream_t s) {
  const unsigned grid = unsigned(onepass_grid(p, B, L, Hkv));
  if (dh == 32)
    launch_dh<32>(p, grid, Q, K, cu, B, n_tok, L, Hq, Hkv, c2, strict, part, s);
  else if (dh == 64)
    launch_dh<64>(p, grid, Q, K, cu, B, n_tok, L, Hq, Hkv, c2, strict, part, s);
  else
    launch_dh<128>(p, grid, Q, K, cu, B, n_tok, L, Hq, Hkv, c2, strict, part, s);
}

}  // namespace detail
}  // namespace estp
