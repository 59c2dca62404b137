// Shared by the bf16 importance kernels: swizzled LDS row tiles, and the launcher of the one-pass
// kernel (importance_onepass.hip).
#pragma once

#include "estp_common.h"

namespace estp {
namespace detail {

// Rows of DH bf16 staged in LDS: 16-byte chunks XOR-swizzled so that 16
// consecutive rows read at one logical chunk hit 16 distinct bank groups.
template <int DH>
struct RowTile {
  static constexpr int kRowBytes = DH * 2;
  static constexpr int kChunks = kRowBytes / 16;
  static constexpr int kRowsPerInst = 64 / kChunks;  // rows one wave-wide 16-byte transfer fills
  static constexpr int kRowsPerWindow = kRowBytes >= 256 ? 1 : 256 / kRowBytes;
  __device__ static __forceinline__ int swz(int row, int chunk) {
    return chunk ^ ((row / kRowsPerWindow) & (kChunks - 1));
  }
  // byte offset of the fragment (row, logical chunk)
  __device__ static __forceinline__ int off(int row, int chunk) { return row * kRowBytes + swz(row, chunk) * 16; }
};

// How the one-pass kernel cuts a call into workgroups.
struct OnepassPlan {
  int waves;    // 0: the call is not for the one-pass kernel; else 4 or 8 waves per workgroup
  int hsplit;   // shares of a KV group's query heads
  int rsplit;   // shares of a prompt's 32-query row blocks
};
OnepassPlan plan_onepass(int64_t n_tok, int B, int max_seqlen, int L, int Hq, int Hkv, int dh, bool f32,
                         bool with_lse);

// Column masses part [L, Hkv * hsplit * rsplit, n_tok] of every prompt (each of at most 256 * waves tokens).
void launch_onepass(const OnepassPlan& p, int dh, const uint16_t* Q, const uint16_t* K, const int* cu, int B,
                    int n_tok, int L, int Hq, int Hkv, float c2, int strict, float* part, hipStream_t s);

}  // namespace detail
}  // namespace estp
