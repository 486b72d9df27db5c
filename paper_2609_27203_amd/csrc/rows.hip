// Rows as sort keys: the columns of a relation packed into one 32- or 64-bit
// key of as many bits as their bounds need (order-preserving images, first
// column highest), so that putting rows into canonical order is one radix sort
// of few digits with no permutation and no gathers; a last column that does
// not fit travels as the payload.  The sorted keys hold the rows: they are
// unpacked (and deduplicated) straight into the columns.  Every kernel here is
// bound by its traffic.  Loading 8 M rows (i32, i32, f32: 40 key bits and a
// payload) takes 5 radix passes of 12-byte records instead of 12 passes of
// (key, row number) pairs and as many random gathers: 1.74 -> 0.60 ms of
// kernels (five passes 0.41, runs ordered 0.05, pack 0.04, count and unpack 0.06,
// bounds 0.03).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/xlh.h"
#include "device_util.h"
#include "kernels.h"
#include "small_sort.h"

namespace xlh {
namespace k {

namespace {

__device__ __forceinline__ uint32_t row_image(uint32_t x, int type) {
  if (type == T_F32) return x ^ ((x >> 31) ? 0xffffffffu : 0x80000000u);  // totalOrder
  return x ^ 0x80000000u;                                                  // signed int
}
__device__ __forceinline__ uint32_t row_value(uint32_t image, int type) {
  if (type == T_F32) return image ^ ((image >> 31) ? 0x80000000u : 0xffffffffu);
  return image ^ 0x80000000u;
}
__device__ __forceinline__ u64 value_of_key(u64 k, int ltype) {  // inverse of the dictionaries' total-order key
  constexpr u64 sign = 1ull << 63;
  if (ltype == XL_I64) return k ^ sign;
  if (ltype == XL_F64) return (k & sign) ? (k & ~sign) : ~k;
  return k;
}

}  // namespace

// Bounds of every column's images in one launch (blockIdx.y = column):
// out[2j] = max of the complements (so ~out[2j] is the minimum), out[2j + 1] =
// maximum; out starts at zero.  At most 256 workgroups of 8,192 values a step:
// the two atomics of each are on one address, and 2,048 workgroups' made a
// column of 8 M values take 50 us, three times its reading.
constexpr int RB_THREADS = 1024, RB_ITEMS = 8;
__global__ __launch_bounds__(RB_THREADS) void col_bounds_k(RowPack r, int64_t n, uint32_t* out) {
  __shared__ uint32_t s_lo[RB_THREADS / 64], s_hi[RB_THREADS / 64];
  const int j = blockIdx.y, type = r.type[j];
  const uint32_t* col = r.col[j];
  uint32_t lo = 0, hi = 0;  // lo: of the complement
  constexpr int64_t STEP = (int64_t)RB_THREADS * RB_ITEMS;
  for (int64_t b = (int64_t)blockIdx.x * STEP; b < n; b += (int64_t)gridDim.x * STEP) {
    uint32_t v[RB_ITEMS];
#pragma unroll
    for (int i = 0; i < RB_ITEMS; ++i) {
      const int64_t at = b + (int64_t)i * RB_THREADS + threadIdx.x;
      v[i] = row_image(col[at < n ? at : n - 1], type);
    }
#pragma unroll
    for (int i = 0; i < RB_ITEMS; ++i) {
      lo = max(lo, ~v[i]);
      hi = max(hi, v[i]);
    }
  }
  for (int d = 32; d > 0; d >>= 1) {
    lo = max(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
  }
  if (lane_id() == 0) {
    s_lo[threadIdx.x >> 6] = lo;
    s_hi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < RB_THREADS / 64; ++w) {
      lo = max(lo, s_lo[w]);
      hi = max(hi, s_hi[w]);
    }
    atomicMax(&out[2 * j], lo);
    atomicMax(&out[2 * j + 1], hi);
  }
}
hipError_t col_bounds(const RowPack& r, int ncols, int64_t n, uint32_t* out, hipStream_t s) {
  if (n <= 0 || ncols <= 0) return hipSuccess;
  const hipError_t e = hipMemsetAsync(out, 0, 8 * MAXC, s);
  if (e != hipSuccess) return e;
  col_bounds_k<<<dim3(grid_for(n, RB_THREADS * RB_ITEMS, 256), (unsigned)ncols), RB_THREADS, 0, s>>>(r, n, out);
  return hipGetLastError();
}

// key[i] = the first r.by columns packed; pay[i] = the image of column r.by.
template <typename K, bool PAY>
__global__ void pack_rows_k(RowPack r, int64_t n, K* key, uint32_t* pay) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    K k = 0;
#pragma unroll
    for (int j = 0; j < MAXC; ++j)
      if (j < r.by) k |= (K)(row_image(r.col[j][i], r.type[j]) - r.lo[j]) << r.shift[j];
    key[i] = k;
    if (PAY) pay[i] = row_image(r.col[r.by][i], r.type[r.by]);
  }
}
hipError_t pack_rows(const RowPack& r, int64_t n, void* key, bool wide, uint32_t* pay, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned g = grid_for(n, 256, 65536);
  if (wide && pay) pack_rows_k<u64, true><<<g, 256, 0, s>>>(r, n, (u64*)key, pay);
  else if (wide) pack_rows_k<u64, false><<<g, 256, 0, s>>>(r, n, (u64*)key, nullptr);
  else if (pay) pack_rows_k<uint32_t, true><<<g, 256, 0, s>>>(r, n, (uint32_t*)key, pay);
  else pack_rows_k<uint32_t, false><<<g, 256, 0, s>>>(r, n, (uint32_t*)key, nullptr);
  return hipGetLastError();
}

// Rows of equal keys (sorted by key only) put into payload order, in place.
// Every row finds its place in its run by counting the payloads before it that
// are not greater and those after it that are less.  A run belongs to the
// workgroup in whose tile it starts, which alone uses and writes its payloads
// (up to RW_RUN - 1 of them after the tile), from LDS; neighbouring lanes
// compare neighbouring words.  Bound by its traffic where runs are short (rows
// that agree in all columns but the last are few, and a row alone is not
// written), by the comparisons where they are long: a row takes as many steps as
// its run has rows.  Loads of 8 M rows (32 key bits, a float), us: no runs 418,
// runs of ten 480, of 30 576, of 60 720 (one thread a run, sorting by insertion:
// 408, 698, 1965 and 2997); 20,000 rows in runs of 40 141 (217).  512 rows a
// workgroup: with 1,024 60,000 rows take 131 us, with 512 or 256 128, and 8 M
// rows with 256 692, with more 684.
// Runs of more than RW_RUN rows raise *flag, and their tile is left to run_keys
// below; the keys ascend, so two equal ones RW_RUN apart tell.
constexpr int RW_RUN = 64, RO_THREADS = 256, RO_ITEMS = 2, RO_TILE = RO_THREADS * RO_ITEMS;
template <typename K>
__global__ __launch_bounds__(RO_THREADS) void order_runs_k(const K* key, uint32_t* pay, int64_t n, uint32_t* flag) {
  __shared__ K s_key[1 + RO_TILE + RW_RUN];  // from the row before the tile on
  __shared__ uint32_t s_p[RO_TILE + RW_RUN];
  K* s_k = s_key + 1;
  const int64_t first = (int64_t)blockIdx.x * RO_TILE;
  const int have = (int)min((int64_t)(RO_TILE + RW_RUN), n - first);  // rows in LDS
  for (int q = threadIdx.x; q < have; q += RO_THREADS) {
    s_k[q] = key[first + q];
    s_p[q] = pay[first + q];
  }
  if (threadIdx.x == 0) s_k[-1] = first > 0 ? key[first - 1] : 0;
  __syncthreads();
  bool over = false;
#pragma unroll
  for (int t = 0; t < RO_ITEMS; ++t) {
    const int q = t * RO_THREADS + (int)threadIdx.x;
    over = over || (q + RW_RUN < have && s_k[q] == s_k[q + RW_RUN]);
  }
  if (__syncthreads_or(over)) {
    // (read first: thousands of workgroups' atomics on one word are served one after another)
    if (threadIdx.x == 0 && !__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(flag, 1u);
    return;
  }
  for (int q = threadIdx.x; q < have; q += RO_THREADS) {
    const K k = s_k[q];
    const uint32_t x = s_p[q];
    int start = q, place = 0;
    for (; start > 0 && s_k[start - 1] == k; --start) place += s_p[start - 1] <= x ? 1 : 0;
    if (start >= RO_TILE || (start == 0 && first > 0 && s_k[-1] == k)) continue;  // another tile's run
    int end = q + 1;
    for (; end < have && s_k[end] == k; ++end) place += s_p[end] < x ? 1 : 0;
    if (end - start > 1) pay[first + start + place] = x;
  }
}
hipError_t order_runs(const void* key, bool wide, uint32_t* pay, int64_t n, uint32_t* flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned g = grid_for(n, RO_TILE, 1 << 30);
  if (wide) order_runs_k<u64><<<g, RO_THREADS, 0, s>>>((const u64*)key, pay, n, flag);
  else order_runs_k<uint32_t><<<g, RO_THREADS, 0, s>>>((const uint32_t*)key, pay, n, flag);
  return hipGetLastError();
}

// Tiles of 2,048 sorted rows per workgroup.  COUNT: cnt[tile] = rows that
// differ from the row before; else the rows are unpacked into the columns, at
// off[tile] + the differing rows before them in the tile (off null: every row
// at its own position).
constexpr int RW_THREADS = 256, RW_ITEMS = 8, RW_TILE = RW_THREADS * RW_ITEMS;

template <typename K, bool COUNT>
__global__ __launch_bounds__(RW_THREADS) void unpack_rows_k(RowPack r, const K* key, const uint32_t* pay, int64_t n,
                                                            uint32_t* cnt, const uint32_t* off) {
  __shared__ uint32_t s_c[RW_ITEMS * RW_THREADS / 64];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * RW_TILE;
  K k[RW_ITEMS];
  uint32_t p[RW_ITEMS];
  u64 m[RW_ITEMS];
#pragma unroll
  for (int q = 0; q < RW_ITEMS; ++q) {
    const int64_t i = base + q * RW_THREADS + threadIdx.x;
    k[q] = i < n ? key[i] : (K)0;
    p[q] = (pay && i < n) ? pay[i] : 0u;
    bool keep = i < n;
    if (keep && (COUNT || off) && i > 0) keep = key[i - 1] != k[q] || (pay && pay[i - 1] != p[q]);
    m[q] = __ballot(keep);
    if (lane == 0) s_c[q * (RW_THREADS / 64) + w] = (uint32_t)__popcll(m[q]);
  }
  __syncthreads();
  if (threadIdx.x < 64) {  // exclusive prefix of the 32 counts, in row order
    const uint32_t c = lane < RW_ITEMS * RW_THREADS / 64 ? s_c[lane] : 0u;
    const uint32_t incl = wave_incl_scan(c);
    if (lane < RW_ITEMS * RW_THREADS / 64) s_c[lane] = incl - c;
    if (COUNT && lane == 63) cnt[blockIdx.x] = incl;
  }
  if (COUNT) return;
  __syncthreads();
  const int64_t out0 = off ? (int64_t)off[blockIdx.x] : base;
#pragma unroll
  for (int q = 0; q < RW_ITEMS; ++q) {
    if (!((m[q] >> lane) & 1ull)) continue;
    const int64_t o = out0 + s_c[q * (RW_THREADS / 64) + w] + __popcll(m[q] & lanemask_lt());
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
      if (j > r.by || !r.dst[j]) continue;
      const uint32_t image = j < r.by ? (uint32_t)((k[q] >> r.shift[j]) & (K)r.mask[j]) + r.lo[j] : p[q];
      const uint32_t v = row_value(image, r.type[j]);
      switch (r.ltype[j]) {
        case XL_BOOL: ((uint8_t*)r.dst[j])[o] = (uint8_t)v; break;
        case XL_U32: ((uint32_t*)r.dst[j])[o] = v ^ 0x80000000u; break;
        case XL_I64:
        case XL_U64:
        case XL_F64: ((u64*)r.dst[j])[o] = value_of_key(r.dict[j][v], r.ltype[j]); break;
        default: ((uint32_t*)r.dst[j])[o] = v;
      }
    }
  }
}

int64_t row_tiles(int64_t n) { return (n + RW_TILE - 1) / RW_TILE; }

hipError_t count_rows(const void* key, bool wide, const uint32_t* pay, int64_t n, uint32_t* cnt, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned g = (unsigned)row_tiles(n);
  RowPack r{};
  if (wide) unpack_rows_k<u64, true><<<g, RW_THREADS, 0, s>>>(r, (const u64*)key, pay, n, cnt, nullptr);
  else unpack_rows_k<uint32_t, true><<<g, RW_THREADS, 0, s>>>(r, (const uint32_t*)key, pay, n, cnt, nullptr);
  return hipGetLastError();
}
hipError_t unpack_rows(const RowPack& r, const void* key, bool wide, const uint32_t* pay, int64_t n,
                       const uint32_t* off, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned g = (unsigned)row_tiles(n);
  if (wide) unpack_rows_k<u64, false><<<g, RW_THREADS, 0, s>>>(r, (const u64*)key, pay, n, nullptr, off);
  else unpack_rows_k<uint32_t, false><<<g, RW_THREADS, 0, s>>>(r, (const uint32_t*)key, pay, n, nullptr, off);
  return hipGetLastError();
}

// Long runs: every row as (number of its run) << bits | (payload - lo), whose
// sort leaves the runs where they are and orders each; off: the runs before
// each tile of RW_TILE rows (count_rows over the keys alone, scanned).
template <typename K>
__global__ __launch_bounds__(RW_THREADS) void run_keys_k(const K* key, const uint32_t* pay, int64_t n,
                                                         const uint32_t* off, int bits, uint32_t lo, u64* out) {
  __shared__ uint32_t s_c[RW_ITEMS * RW_THREADS / 64];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * RW_TILE;
  u64 m[RW_ITEMS];
#pragma unroll
  for (int q = 0; q < RW_ITEMS; ++q) {
    const int64_t i = base + q * RW_THREADS + threadIdx.x;
    m[q] = __ballot(i < n && (i == 0 || key[i - 1] != key[i]));
    if (lane == 0) s_c[q * (RW_THREADS / 64) + w] = (uint32_t)__popcll(m[q]);
  }
  __syncthreads();
  if (threadIdx.x < 64) {  // exclusive prefix of the 32 counts, in row order
    const uint32_t c = lane < RW_ITEMS * RW_THREADS / 64 ? s_c[lane] : 0u;
    const uint32_t incl = wave_incl_scan(c);
    if (lane < RW_ITEMS * RW_THREADS / 64) s_c[lane] = incl - c;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RW_ITEMS; ++q) {
    const int64_t i = base + q * RW_THREADS + threadIdx.x;
    if (i >= n) continue;
    // runs that start up to and with this row, less one (row 0 starts the first)
    const u64 upto = m[q] & (lanemask_lt() | (1ull << lane));
    const uint32_t run = off[blockIdx.x] + s_c[q * (RW_THREADS / 64) + w] + (uint32_t)__popcll(upto) - 1u;
    out[i] = ((u64)run << bits) | (u64)(pay[i] - lo);
  }
}
hipError_t run_keys(const void* key, bool wide, const uint32_t* pay, int64_t n, const uint32_t* off, int bits,
                    uint32_t lo, u64* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned g = (unsigned)row_tiles(n);
  if (wide) run_keys_k<u64><<<g, RW_THREADS, 0, s>>>((const u64*)key, pay, n, off, bits, lo, out);
  else run_keys_k<uint32_t><<<g, RW_THREADS, 0, s>>>((const uint32_t*)key, pay, n, off, bits, lo, out);
  return hipGetLastError();
}
__global__ void run_payloads_k(const u64* sorted, int64_t n, int bits, uint32_t lo, uint32_t* pay) {
  const u64 mask = (1ull << bits) - 1ull;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    pay[i] = (uint32_t)(sorted[i] & mask) + lo;
}
hipError_t run_payloads(const u64* sorted, int64_t n, int bits, uint32_t lo, uint32_t* pay, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  run_payloads_k<<<grid_for(n, 256, 65536), 256, 0, s>>>(sorted, n, bits, lo, pay);
  return hipGetLastError();
}

// A whole load of at most SS_MAX rows in one launch of one workgroup: bounds,
// packing, sort, deduplication and unpacking (r: columns, types, ltypes and
// dst, by = the column count; dst hold n values).  out[0] = distinct rows, or
// 0 when the packed rows need more than 64 bits (nothing is written then);
// out[1 + 2j], out[2 + 2j] = least and greatest image of column j.  Bound by
// its barriers; the separate kernels cost eight launches and a second host
// read (300 edges loaded, closed and read back: 251 -> 229 us).
__global__ __launch_bounds__(SS_THREADS) void load_small_k(RowPack r, int n, uint32_t* out) {
  __shared__ SmallSort<u64, false> L;
  __shared__ uint32_t s_lo[MAXC][SS_WAVES], s_hi[MAXC][SS_WAVES], s_c[SS_WAVES * SS_ITEMS];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  uint32_t img[MAXC][SS_ITEMS];
#pragma unroll
  for (int c = 0; c < MAXC; ++c) {
    if (c >= r.by) continue;
    uint32_t lo = 0xffffffffu, hi = 0;
#pragma unroll
    for (int j = 0; j < SS_ITEMS; ++j) {
      const int p = ss_place(j);
      img[c][j] = p < n ? row_image(r.col[c][p], r.type[c]) : 0u;
      if (p < n) {
        lo = min(lo, img[c][j]);
        hi = max(hi, img[c][j]);
      }
    }
    for (int d = 32; d > 0; d >>= 1) {
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
    }
    if (lane == 0) {
      s_lo[c][w] = lo;
      s_hi[c][w] = hi;
    }
  }
  __syncthreads();
  uint32_t lo[MAXC] = {}, width[MAXC] = {}, total = 0;
#pragma unroll
  for (int c = 0; c < MAXC; ++c) {
    if (c >= r.by) continue;
    uint32_t hi = 0;
    lo[c] = 0xffffffffu;
    for (int k = 0; k < SS_WAVES; ++k) {
      lo[c] = min(lo[c], s_lo[c][k]);
      hi = max(hi, s_hi[c][k]);
    }
    width[c] = 32u - (uint32_t)__clz((int)(hi - lo[c]));
    total += width[c];
    if (threadIdx.x == 0) {
      out[1 + 2 * c] = lo[c];
      out[2 + 2 * c] = hi;
    }
  }
  if (total > 64) {
    if (threadIdx.x == 0) out[0] = 0;
    return;
  }
  u64 key[SS_ITEMS];
  uint32_t none[SS_ITEMS] = {};
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) {
    key[j] = 0;
#pragma unroll
    for (int c = 0; c < MAXC; ++c)
      if (c < r.by && width[c]) key[j] = (width[c] < 64 ? key[j] << width[c] : 0) | (img[c][j] - lo[c]);
  }
  small_sort<u64, false>(key, none, n, (int)total, L);
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) L.sk[ss_place(j)] = key[j];
  __syncthreads();
  u64 keep[SS_ITEMS];
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) {
    const int p = ss_place(j);
    keep[j] = __ballot(p < n && (p == 0 || L.sk[p - 1] != key[j]));
    if (lane == 0) s_c[w * SS_ITEMS + j] = (uint32_t)__popcll(keep[j]);
  }
  __syncthreads();
  if (w == 0) {  // exclusive prefix of the 64 counts, in row order
    const uint32_t c = s_c[lane], incl = wave_incl_scan(c);
    s_c[lane] = incl - c;
    if (lane == 63) out[0] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) {
    if (!((keep[j] >> lane) & 1ull)) continue;
    const uint32_t o = s_c[w * SS_ITEMS + j] + (uint32_t)__popcll(keep[j] & lanemask_lt());
    u64 k = key[j];
#pragma unroll
    for (int c = MAXC - 1; c >= 0; --c) {
      if (c >= r.by) continue;
      const uint32_t image = (uint32_t)(k & (width[c] >= 32 ? 0xffffffffull : (1ull << width[c]) - 1ull)) + lo[c];
      k >>= width[c];
      ((uint32_t*)r.dst[c])[o] = row_value(image, r.type[c]);
    }
  }
}
static_assert(SS_WAVES * SS_ITEMS == 64, "one lane per count");

int64_t load_small_max() { return SS_MAX; }
hipError_t load_small(const RowPack& r, int64_t n, uint32_t* out, hipStream_t s) {
  if (n <= 0 || n > SS_MAX || r.by <= 0 || r.by > MAXC) return hipErrorInvalidValue;
  load_small_k<<<1, SS_THREADS, 0, s>>>(r, (int)n, out);
  return hipGetLastError();
}

}  // namespace k
}  // namespace xlh
