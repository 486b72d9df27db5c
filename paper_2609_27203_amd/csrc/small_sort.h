// Stable LSD radix sort of at most SS_MAX keys by one workgroup of SS_THREADS
// threads, in LDS: every 8-bit pass runs in one launch instead of two or three
// launches per pass.  Wavefront w owns positions [256w, 256w + 256), four
// 64-key runs; a pass ranks each key among the equal digits of its wavefront
// with the ballot match used by the scatter of the large sort, offsets each
// (digit, wavefront) count in digit-major order, and scatters the keys to
// their new positions in LDS.
#pragma once
#include "device_util.h"

namespace xlh {
namespace k {

constexpr int SS_THREADS = 1024;
constexpr int SS_WAVES = SS_THREADS / 64;
constexpr int SS_ITEMS = 4;
constexpr int SS_MAX = SS_THREADS * SS_ITEMS;

template <typename K, bool VALS>
struct SmallSort {
  K sk[SS_MAX];
  uint32_t sv[VALS ? SS_MAX : 1];
  uint32_t cnt[SS_WAVES][256];
  uint32_t s_w[SS_WAVES];
};

// Position of the calling thread's j-th key.
__device__ __forceinline__ int ss_place(int j) {
  return (int)(threadIdx.x >> 6) * 64 * SS_ITEMS + j * 64 + lane_id();
}

// key[j] (and val[j]) hold the key at ss_place(j) (positions from n on are
// ignored) before and after.
template <typename K, bool VALS>
__device__ __forceinline__ void small_sort(K (&key)[SS_ITEMS], uint32_t (&val)[SS_ITEMS], int n, int bits,
                                           SmallSort<K, VALS>& L) {
  const int lane = lane_id(), w = threadIdx.x >> 6;
  for (int shift = 0; shift < bits; shift += 8) {
    const int nbits = bits - shift < 8 ? bits - shift : 8;
    const uint32_t dmask = (1u << nbits) - 1u;
    for (int i = threadIdx.x; i < SS_WAVES * 256; i += SS_THREADS) (&L.cnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t rank[SS_ITEMS], dig[SS_ITEMS];
#pragma unroll
    for (int j = 0; j < SS_ITEMS; ++j) {
      const bool valid = ss_place(j) < n;
      const uint32_t d = (uint32_t)(key[j] >> shift) & dmask;
      u64 peers = __ballot(valid);
      for (int b = 0; b < nbits; ++b) {
        const bool bit = (d >> b) & 1u;
        const u64 bal = __ballot(bit);
        peers &= bit ? bal : ~bal;
      }
      if (!valid) peers = 0;
      const uint32_t lt = __popcll(peers & lanemask_lt());
      const uint32_t before = L.cnt[w][d];
      wave_lds_sync();
      rank[j] = before + lt;
      dig[j] = d;
      if (valid && lt == 0) L.cnt[w][d] = before + (uint32_t)__popcll(peers);
      wave_lds_sync();
    }
    __syncthreads();
    // digit d's total, then the digit-major offsets of every (digit, wavefront)
    uint32_t tot = 0;
    if (threadIdx.x < 256)
      for (int ww = 0; ww < SS_WAVES; ++ww) tot += L.cnt[ww][threadIdx.x];
    const uint32_t incl = wave_incl_scan_t<uint32_t>(tot);
    if (lane == 63) L.s_w[w] = incl;
    __syncthreads();
    uint32_t run = incl - tot;
    for (int ww = 0; ww < w; ++ww) run += L.s_w[ww];
    if (threadIdx.x < 256)
      for (int ww = 0; ww < SS_WAVES; ++ww) {
        const uint32_t c = L.cnt[ww][threadIdx.x];
        L.cnt[ww][threadIdx.x] = run;
        run += c;
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SS_ITEMS; ++j) {
      if (ss_place(j) < n) {
        const uint32_t pos = L.cnt[w][dig[j]] + rank[j];
        L.sk[pos] = key[j];
        if (VALS) L.sv[pos] = val[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SS_ITEMS; ++j) {
      const int p = ss_place(j);
      if (p < n) {
        key[j] = L.sk[p];
        if (VALS) val[j] = L.sv[p];
      }
    }
    __syncthreads();
  }
}

}  // namespace k
}  // namespace xlh
