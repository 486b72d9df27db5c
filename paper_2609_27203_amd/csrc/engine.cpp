// Workspace arena, relation storage, index builds and the semi-naive
// fixpoint driver (host orchestration; every data-plane step is a kernel).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <memory>

#include "engine.h"
#include "kernels.h"

namespace xlh {

typedef unsigned long long u64;

// Grid cap (blocks of four wavefronts) of the insert-or-improve emission kernels.
constexpr int EMIT_GRID = 2048;
// Rows a wavefront may insert after the load limit is crossed before it
// learns so: its LDS staging buffer (512) plus one 64-item step.
constexpr int64_t WAVE_SLACK = 512 + 64;

// ================================================================== arena
void Arena::init(char* base, size_t size) {
  // every block starts on a 256-B boundary and spans a multiple of 256 B, so
  // kernels may read whole aligned vectors that hold a valid element
  const size_t skip = (256 - (uintptr_t)base % 256) % 256;
  base_ = base + skip;
  size_ = size > skip ? (size - skip) & ~(size_t)255 : 0;
  free_.clear();
  used_.clear();
  if (size_) free_[0] = size_;
  in_use_ = peak_ = 0;
}

void* Arena::alloc(size_t bytes) {
  bytes = (std::max<size_t>(bytes, 1) + 255) & ~(size_t)255;
  for (auto it = free_.begin(); it != free_.end(); ++it) {
    if (it->second < bytes) continue;
    size_t off = it->first, sz = it->second;
    free_.erase(it);
    if (sz > bytes) free_[off + bytes] = sz - bytes;
    used_[off] = bytes;
    in_use_ += bytes;
    peak_ = std::max(peak_, in_use_);
    return base_ + off;
  }
  return nullptr;
}

void Arena::release(void* p) {
  if (!p) return;
  size_t off = (size_t)((char*)p - base_);
  auto it = used_.find(off);
  if (it == used_.end()) return;
  size_t sz = it->second;
  used_.erase(it);
  in_use_ -= sz;
  auto nx = free_.lower_bound(off);
  if (nx != free_.end() && nx->first == off + sz) {
    sz += nx->second;
    free_.erase(nx);
  }
  auto pv = free_.lower_bound(off);
  if (pv != free_.begin()) {
    --pv;
    if (pv->first + pv->second == off) {
      pv->second += sz;
      return;
    }
  }
  free_[off] = sz;
}

size_t Arena::block_size(const void* p) const {
  if (!p) return 0;
  auto it = used_.find((size_t)((const char*)p - base_));
  return it == used_.end() ? 0 : it->second;
}

size_t Arena::largest_free() const {
  size_t m = 0;
  for (auto& kv : free_) m = std::max(m, kv.second);
  return m;
}

// ================================================================== helpers
#define XL_TRY(x)                        \
  do {                                   \
    xl_status _s = (x);                  \
    if (_s != XL_OK) return _s;          \
  } while (0)

#define HIP_TRY(ctx, x)                                                                  \
  do {                                                                                   \
    hipError_t _e = (x);                                                                 \
    if (_e != hipSuccess)                                                                \
      return (ctx)->fail(XL_DEVICE_ERROR, std::string(#x) + ": " + hipGetErrorString(_e)); \
  } while (0)

namespace {

// Arena block released on scope exit unless kept.
struct Buf {
  Context* c = nullptr;
  void* p = nullptr;
  Buf() = default;
  explicit Buf(Context* cc) : c(cc) {}
  Buf(const Buf&) = delete;
  Buf& operator=(const Buf&) = delete;
  ~Buf() { reset(); }
  void reset() {
    if (c && p) c->arena.release(p);
    p = nullptr;
  }
  void* keep() {
    void* q = p;
    p = nullptr;
    return q;
  }
  template <typename T>
  T* as() const {
    return (T*)p;
  }
};

xl_status dalloc(Context* c, size_t bytes, Buf* b, const char* what) {
  b->c = c;
  b->reset();
  b->p = c->arena.alloc(bytes);
  if (!b->p)
    return c->fail(XL_RESOURCE_EXHAUSTED,
                   std::string("workspace exhausted allocating ") + std::to_string(bytes) +
                       " bytes for " + what + " (in use " + std::to_string(c->arena.in_use()) +
                       " of " + std::to_string(c->arena.capacity()) + ", largest free block " +
                       std::to_string(c->arena.largest_free()) + ")");
  return XL_OK;
}

xl_status ctl_read(Context* c, const void* dev, size_t bytes, void* host) {
  if (bytes > CTL_CHECK_OFFSET) return c->fail(XL_DEVICE_ERROR, "control read larger than the control block (internal)");
  HIP_TRY(c, hipMemcpyAsync(c->pinned, dev, bytes, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  memcpy(host, c->pinned, bytes);
  c->control_bytes += (int64_t)bytes;
  return XL_OK;
}

constexpr int64_t BOUNDS_ONE_MAX = 65536;  // columns this short take one workgroup for their bounds

int bitlen(uint64_t x) {  // bits needed to represent values 0..x
  int b = 0;
  while (x) {
    ++b;
    x >>= 1;
  }
  return b;
}

uint64_t next_pow2(uint64_t x) {
  uint64_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

// Scratch of a lexicographic row sort.
struct LexScratch {
  Buf pa, pb, ka, kb, tmp;
};
xl_status lex_scratch(Context* c, int64_t n, LexScratch* x) {
  XL_TRY(dalloc(c, (size_t)n * 4, &x->pa, "sort permutation"));
  XL_TRY(dalloc(c, (size_t)n * 4, &x->pb, "sort permutation"));
  XL_TRY(dalloc(c, (size_t)n * 4, &x->ka, "sort keys"));
  XL_TRY(dalloc(c, (size_t)n * 4, &x->kb, "sort keys"));
  return dalloc(c, k::radix_temp_bytes(n), &x->tmp, "sort scratch");
}

// Permutation sorting the rows lexicographically (int32 signed, float32
// totalOrder), built as successive stable radix sorts from the last column.
xl_status lex_perm(Context* c, uint32_t* const* cols, const uint8_t* types, int arity, int64_t n,
                   Buf* perm_out) {
  LexScratch x;
  XL_TRY(lex_scratch(c, n, &x));
  HIP_TRY(c, k::iota_u32(x.pa.as<uint32_t>(), n, c->stream));
  for (int j = arity - 1; j >= 0; --j) {
    HIP_TRY(c, k::ordered_key(cols[j], types[j], x.pa.as<uint32_t>(), x.ka.as<uint32_t>(), n, c->stream));
    int alt = 0;
    HIP_TRY(c, k::radix_sort_u32(x.ka.as<uint32_t>(), x.pa.as<uint32_t>(), x.kb.as<uint32_t>(),
                                 x.pb.as<uint32_t>(), n, 32, x.tmp.p, c->stream, &alt));
    if (alt) std::swap(x.pa.p, x.pb.p);
  }
  std::swap(perm_out->p, x.pa.p);
  perm_out->c = c;
  return XL_OK;
}

// Rows sorted as packed keys (rows.hip): the key holds the first `by` columns,
// a payload the one after them, if any.
struct PackedRows {
  Buf key, pay, key2, pay2;
  k::RowPack r{};
  int bits = 0, pay_bits = 0;  // of the key, and of the payload less its least image
  bool wide = false, has_pay = false;
  void* skey() const { return key.p; }
  uint32_t* spay() const { return has_pay ? pay.as<uint32_t>() : nullptr; }
};

// Key layout of columns whose images lie in [lo, hi]: as many leading columns
// as 64 bits hold, at most one more as the payload.  keep (when positive) is a
// number of leading columns that are known to be distinct: no more are packed
// when the rest is one column.  False when the columns do not fit.
bool row_layout(const uint8_t* types, int arity, const uint32_t* lo, const uint32_t* hi, int64_t n, int keep,
                PackedRows* x) {
  int width[MAXC], by = 0, total = 0;
  for (int j = 0; j < arity; ++j) width[j] = bitlen((uint64_t)hi[j] - lo[j]);
  const int most = keep > 0 && keep == arity - 1 ? keep : arity;
  while (by < most && total + width[by] <= 64) total += width[by++];
  if (by < arity - 1) return false;
  // a last column that costs two passes or more is cheaper as the payload (1 M
  // edges with f32 weights: 34 + 26 bits), where the others tell most rows
  // apart (runs of equal keys are ordered one by one); up to 4,096 rows every
  // pass runs in one launch
  if (by == arity && arity > 1 && keep == 0 && n > 4096) {
    const int lead = total - width[arity - 1];
    if ((total + 7) / 8 - (lead + 7) / 8 >= 2 && lead >= bitlen((uint64_t)n) + 2) {
      total = lead;
      --by;
    }
  }
  x->has_pay = by < arity;
  x->pay_bits = x->has_pay ? width[by] : 0;
  x->bits = total;
  x->wide = total > 32;
  x->r.by = by;
  for (int j = 0, at = total; j < arity; ++j) {
    x->r.type[j] = types[j];
    x->r.lo[j] = lo[j];
    if (j < by) {
      at -= width[j];
      x->r.shift[j] = at >= (x->wide ? 64 : 32) ? 0 : at;  // (a constant column needs no bits)
      x->r.mask[j] = width[j] >= 32 ? 0xffffffffu : (1u << width[j]) - 1u;
    }
  }
  return true;
}

// Pack and sort n rows; the sorted keys and payloads end in x->key, x->pay.
// free_input (optional) runs once the columns have been read.
template <typename F>
xl_status sort_packed(Context* c, PackedRows* x, int64_t n, F free_input) {
  const size_t kb = x->wide ? 8 : 4;
  Buf tmp;
  XL_TRY(dalloc(c, (size_t)n * kb, &x->key, "sort keys"));
  if (x->has_pay) XL_TRY(dalloc(c, (size_t)n * 4, &x->pay, "sort payload"));
  HIP_TRY(c, k::pack_rows(x->r, n, x->key.p, x->wide, x->spay(), c->stream));
  free_input();
  XL_TRY(dalloc(c, (size_t)n * kb, &x->key2, "sort keys"));
  if (x->has_pay) XL_TRY(dalloc(c, (size_t)n * 4, &x->pay2, "sort payload"));
  XL_TRY(dalloc(c, k::radix_temp_bytes(n), &tmp, "sort scratch"));
  int alt = 0;
  uint32_t* pay2 = x->has_pay ? x->pay2.as<uint32_t>() : nullptr;
  if (x->wide)
    HIP_TRY(c, k::radix_sort_u64(x->key.as<u64>(), x->spay(), x->key2.as<u64>(), pay2, n, x->bits, tmp.p, c->stream,
                                 &alt));
  else
    HIP_TRY(c, k::radix_sort_u32(x->key.as<uint32_t>(), x->spay(), x->key2.as<uint32_t>(), pay2, n, x->bits, tmp.p,
                                 c->stream, &alt));
  if (alt) {
    std::swap(x->key.p, x->key2.p);
    std::swap(x->pay.p, x->pay2.p);
  }
  x->key2.reset();
  x->pay2.reset();
  return XL_OK;
}

// Least and greatest image of every column (n > 0 rows).
xl_status image_bounds(Context* c, const uint32_t* const* cols, const uint8_t* types, int arity, int64_t n,
                       uint32_t* lo, uint32_t* hi) {
  Buf b;
  XL_TRY(dalloc(c, 8 * MAXC, &b, "bounds"));
  k::RowPack r{};
  for (int j = 0; j < arity; ++j) {
    r.col[j] = cols[j];
    r.type[j] = types[j];
  }
  HIP_TRY(c, k::col_bounds(r, arity, n, b.as<uint32_t>(), c->stream));
  uint32_t out[2 * MAXC];
  XL_TRY(ctl_read(c, b.p, sizeof(out), out));
  for (int j = 0; j < arity; ++j) {
    lo[j] = ~out[2 * j];
    hi[j] = out[2 * j + 1];
  }
  return XL_OK;
}

inline int32_t image_i32(uint32_t image) { return (int32_t)(image ^ 0x80000000u); }

xl_status compute_bounds(Context* c, Relation* r) {
  if (r->nrows == 0) return XL_OK;
  uint32_t lo[MAXC], hi[MAXC];
  XL_TRY(image_bounds(c, r->col, r->types, r->arity, r->nrows, lo, hi));
  for (int j = 0; j < r->arity; ++j)
    if (r->types[j] == T_I32) {
      r->lo[j] = image_i32(lo[j]);
      r->hi[j] = image_i32(hi[j]);
    }
  return XL_OK;
}

// Images of n order keys (device) of the 8-byte type lt: their ranks in the
// context's dictionary after the keys new to it are added.  Adding keys
// renumbers the dictionary, so every stored column of type lt is remapped
// (old rank -> new rank, order kept) and its relation gets a new generation.
xl_status dict_encode(Context* c, int lt, const u64* keys, int64_t n, uint32_t* images) {
  if (n <= 0) return XL_OK;
  const int64_t nd = c->dict_n[lt], nt = nd + n;
  Buf cat, alt, tmp, flag, pos, stmp, tot;
  XL_TRY(dalloc(c, (size_t)nt * 8, &cat, "dictionary merge"));
  XL_TRY(dalloc(c, (size_t)nt * 8, &alt, "dictionary merge"));
  XL_TRY(dalloc(c, k::radix_temp_bytes(nt), &tmp, "sort scratch"));
  if (nd > 0)
    HIP_TRY(c, hipMemcpyAsync(cat.p, c->dict[lt], (size_t)nd * 8, hipMemcpyDeviceToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(cat.as<u64>() + nd, keys, (size_t)n * 8, hipMemcpyDeviceToDevice, c->stream));
  int a = 0;
  HIP_TRY(c, k::radix_sort_u64(cat.as<u64>(), nullptr, alt.as<u64>(), nullptr, nt, 64, tmp.p, c->stream, &a));
  const u64* sorted = a ? alt.as<u64>() : cat.as<u64>();
  XL_TRY(dalloc(c, (size_t)nt * 4, &flag, "dictionary flags"));
  XL_TRY(dalloc(c, (size_t)nt * 4, &pos, "dictionary positions"));
  XL_TRY(dalloc(c, k::scan_temp_bytes(nt), &stmp, "scan scratch"));
  XL_TRY(dalloc(c, 8, &tot, "count"));
  HIP_TRY(c, k::unique_flags64(sorted, nt, flag.as<uint32_t>(), c->stream));
  HIP_TRY(c, k::scan_exclusive_u32(flag.as<uint32_t>(), pos.as<uint32_t>(), nt, tot.as<uint32_t>(), stmp.p,
                                   c->stream));
  uint32_t m = 0;
  XL_TRY(ctl_read(c, tot.p, 4, &m));
  if (m > (uint32_t)nd) {
    if (m >= (1u << 31))
      return c->fail(XL_CAPACITY_EXCEEDED, std::string("more than 2^31 distinct ") + type_name(lt) + " values");
    Buf nd_keys;
    XL_TRY(dalloc(c, (size_t)m * 8, &nd_keys, "type dictionary"));
    HIP_TRY(c, k::compact64(sorted, flag.as<uint32_t>(), pos.as<uint32_t>(), nd_keys.as<u64>(), nt, c->stream));
    if (nd > 0) {
      Buf map;
      XL_TRY(dalloc(c, (size_t)nd * 4, &map, "dictionary renumbering"));
      HIP_TRY(c, k::rank64(nd_keys.as<u64>(), m, c->dict[lt], nd, map.as<uint32_t>(), c->stream));
      for (Relation* r : c->rels) {
        bool touched = false;
        for (int j = 0; j < r->arity; ++j)
          if (r->ltypes[j] == lt && r->nrows > 0 && r->col[j]) {
            HIP_TRY(c, k::remap_codes(r->col[j], r->nrows, map.as<uint32_t>(), c->stream));
            touched = true;
          }
        if (touched) {
          r->generation = ++c->generations;
          c->icache_drop(r, true);
          XL_TRY(compute_bounds(c, r));
        }
      }
    }
    c->arena.release(c->dict[lt]);
    c->dict[lt] = (unsigned long long*)nd_keys.keep();
    c->dict_n[lt] = m;
  }
  HIP_TRY(c, k::rank64(c->dict[lt], c->dict_n[lt], keys, n, images, c->stream));
  return XL_OK;
}

// Int32 images of the columns of r given to a load (n values each, in host or
// device memory, packed at each type's element size) written to img[j] for
// the columns of type u32, bool, i64, u64 or f64.  The columns of one 8-byte
// type go through one dictionary update together, so no image of this load
// is renumbered by a later one.
xl_status encode_columns(Context* c, const Relation* r, const void* const* cols, int64_t n, int on_device,
                         uint32_t* const* img) {
  const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
  for (int lt : {XL_U32, XL_BOOL}) {
    for (int j = 0; j < r->arity; ++j) {
      if (r->ltypes[j] != lt) continue;
      const size_t es = elem_bytes(lt);
      Buf in, bad;
      XL_TRY(dalloc(c, (size_t)n * es, &in, "loaded column"));
      XL_TRY(dalloc(c, 4, &bad, "check flag"));
      HIP_TRY(c, hipMemcpyAsync(in.p, cols[j], (size_t)n * es, kind, c->stream));
      HIP_TRY(c, hipMemsetAsync(bad.p, 0, 4, c->stream));
      HIP_TRY(c, k::encode_narrow(in.p, lt, n, img[j], bad.as<uint32_t>(), c->stream));
      uint32_t flag = 0;
      XL_TRY(ctl_read(c, bad.p, 4, &flag));
      if (flag)
        return c->fail(XL_INVALID_ARGUMENT,
                       "bool column " + std::to_string(j) + " of " + r->name + " holds a byte other than 0 or 1");
    }
  }
  for (int lt : {XL_I64, XL_U64, XL_F64}) {
    std::vector<int> js;
    for (int j = 0; j < r->arity; ++j)
      if (r->ltypes[j] == lt) js.push_back(j);
    if (js.empty()) continue;
    const int64_t m = n * (int64_t)js.size();
    Buf in, keys, imgs;
    XL_TRY(dalloc(c, (size_t)n * 8, &in, "loaded column"));
    XL_TRY(dalloc(c, (size_t)m * 8, &keys, "order keys"));
    XL_TRY(dalloc(c, (size_t)m * 4, &imgs, "column images"));
    for (size_t q = 0; q < js.size(); ++q) {
      HIP_TRY(c, hipMemcpyAsync(in.p, cols[js[q]], (size_t)n * 8, kind, c->stream));
      HIP_TRY(c, k::order_keys64(in.as<u64>(), lt, n, keys.as<u64>() + (int64_t)q * n, c->stream));
    }
    XL_TRY(dict_encode(c, lt, keys.as<u64>(), m, imgs.as<uint32_t>()));
    for (size_t q = 0; q < js.size(); ++q)
      HIP_TRY(c, hipMemcpyAsync(img[js[q]], imgs.as<uint32_t>() + (int64_t)q * n, (size_t)n * 4,
                                hipMemcpyDeviceToDevice, c->stream));
  }
  return XL_OK;
}

}  // namespace

// Give every constant of an 8-byte type in p's plans its current image,
// adding the values the dictionaries lack.
xl_status resolve_wide_constants(Program* p) {
  Context* c = p->ctx;
  for (int lt : {XL_I64, XL_U64, XL_F64}) {
    std::vector<u64> keys;
    std::vector<uint32_t*> dst;
    for (Stratum& st : p->strata)
      for (std::vector<RulePlan>* v : {&st.full, &st.variants})
        for (RulePlan& rp : *v)
          for (const WideConst& w : rp.wconsts) {
            if (w.ltype != lt) continue;
            keys.push_back(w.key);
            dst.push_back(w.where == 0   ? &rp.driver_act[w.a].cval
                          : w.where == 1 ? &rp.steps[w.a].act[w.b].cval
                                         : &rp.stage_consts[w.a][w.b]);
          }
    if (keys.empty()) continue;
    const int64_t n = (int64_t)keys.size();
    Buf dk, di;
    XL_TRY(dalloc(c, (size_t)n * 8, &dk, "constant keys"));
    XL_TRY(dalloc(c, (size_t)n * 4, &di, "constant images"));
    HIP_TRY(c, hipMemcpyAsync(dk.p, keys.data(), (size_t)n * 8, hipMemcpyHostToDevice, c->stream));
    XL_TRY(dict_encode(c, lt, dk.as<u64>(), n, di.as<uint32_t>()));
    std::vector<uint32_t> img((size_t)n);
    for (int64_t i0 = 0; i0 < n; i0 += 1024) {
      const int64_t m = std::min<int64_t>(1024, n - i0);
      XL_TRY(ctl_read(c, di.as<uint32_t>() + i0, (size_t)m * 4, img.data() + i0));
    }
    for (int64_t i = 0; i < n; ++i) *dst[(size_t)i] = img[(size_t)i];
  }
  return XL_OK;
}

// The gathered-round shape (see GatherShape).
bool gather_shape(const RulePlan& p, GatherShape* g) {
  if (!p.driver_delta || p.driver != p.head || p.driver->arity != 2 || p.steps.size() != 2 || p.nkey != 2 ||
      !p.negs.empty())
    return false;
  for (const auto& ops : p.stage_ops)
    if (!ops.empty()) return false;
  const ColAct &da = p.driver_act[0], &db = p.driver_act[1];
  if (da.kind != CA_BIND || db.kind != CA_BIND || da.slot == db.slot) return false;
  int ia = -1, ib = -1;
  for (int k = 0; k < 2; ++k) {
    if (p.steps[k].key_slot == da.slot) ia = k;
    else if (p.steps[k].key_slot == db.slot) ib = k;
  }
  if (ia < 0 || ib < 0) return false;
  auto other = [&](const StepPlan& st, int* col, int* slot) {
    if (st.rel == p.head || st.rel->arity != 2) return false;
    const int oc = 1 - st.key_col;
    if (st.act[oc].kind != CA_BIND) return false;
    *col = oc;
    *slot = st.act[oc].slot;
    return true;
  };
  int xs = -1, ys = -1;
  if (!other(p.steps[ia], &g->x_col, &xs) || !other(p.steps[ib], &g->y_col, &ys)) return false;
  if (xs != p.key_slot[0] || ys != p.key_slot[1] || xs == ys) return false;
  g->s1 = ia;
  g->s2 = ib;
  return true;
}

// h(X,Y) :- h(X,Z), h(Z,Y) with nothing else: its two delta variants (delta
// as the first atom, joined by column 0; delta as the second, by column 1).
static bool self_join_variant(const RulePlan& p, int key_col) {
  if (!p.driver_delta || p.driver != p.head || p.head->arity != 2 || p.nkey != 2 || p.steps.size() != 1 ||
      p.steps[0].rel != p.head || p.steps[0].key_col != key_col || !p.negs.empty())
    return false;
  for (const auto& ops : p.stage_ops)
    if (!ops.empty()) return false;
  const ColAct &d0 = p.driver_act[0], &d1 = p.driver_act[1], &e = p.steps[0].act[1 - key_col];
  if (d0.kind != CA_BIND || d1.kind != CA_BIND || e.kind != CA_BIND || d0.slot == d1.slot || e.slot == d0.slot ||
      e.slot == d1.slot || p.steps[0].act[key_col].kind != CA_NONE)
    return false;
  // delta first: d = (x, z), e = y; delta second: d = (z, y), e = x
  const int z = key_col == 0 ? d1.slot : d0.slot, x = key_col == 0 ? d0.slot : e.slot,
            y = key_col == 0 ? e.slot : d1.slot;
  return p.steps[0].key_slot == z && p.key_slot[0] == x && p.key_slot[1] == y;
}
bool self_join_shape(const std::vector<RulePlan>& variants) {
  return variants.size() == 2 && ((self_join_variant(variants[0], 0) && self_join_variant(variants[1], 1)) ||
                                  (self_join_variant(variants[0], 1) && self_join_variant(variants[1], 0)));
}

void relation_free_storage(Relation* r) {
  for (int j = 0; j < MAXC; ++j) {
    if (r->col[j]) r->ctx->arena.release(r->col[j]);
    r->col[j] = nullptr;
  }
  r->nrows = 0;
  r->sorted = false;
  r->key_cols = 0;
  r->generation = ++r->ctx->generations;  // cached indexes of the old rows no longer match
  r->ctx->icache_drop(r, true);
}

xl_status relation_clear(Relation* r) {
  relation_free_storage(r);
  return XL_OK;
}

// ================================================================== load / read
namespace {

// A load of few rows in one launch; *done stays false when the rows need more
// than 64 bits.
xl_status load_small(Context* c, const Relation* r, const uint32_t* const* rc, int64_t n, uint32_t* lo, uint32_t* hi,
                     Buf* fin, int64_t* m, bool* done) {
  k::RowPack p{};
  Buf out;
  p.by = r->arity;
  for (int j = 0; j < r->arity; ++j) {
    XL_TRY(dalloc(c, (size_t)n * 4, &fin[j], "relation column"));
    p.col[j] = rc[j];
    p.type[j] = r->types[j];
    p.dst[j] = fin[j].p;
  }
  XL_TRY(dalloc(c, 4 * (1 + 2 * MAXC), &out, "load result"));
  HIP_TRY(c, k::load_small(p, n, out.as<uint32_t>(), c->stream));
  uint32_t t[1 + 2 * MAXC];
  XL_TRY(ctl_read(c, out.p, sizeof(t), t));
  *done = t[0] > 0;
  *m = t[0];
  for (int j = 0; j < r->arity; ++j) {
    if (!*done) fin[j].reset();
    lo[j] = t[1 + 2 * j];
    hi[j] = t[2 + 2 * j];
  }
  return XL_OK;
}

// Payloads of sorted rows put in order within each run of equal keys, by one
// sort of (run, payload) keys, for runs of any length; at most `most` runs.
// cnt and off hold one word per row tile, scan and tot are scratch.
xl_status order_long_runs(Context* c, PackedRows* x, int64_t n, uint32_t most, uint32_t* cnt, uint32_t* off,
                          void* scan, uint32_t* tot) {
  Buf a, b, tmp;
  XL_TRY(dalloc(c, (size_t)n * 8, &a, "run keys"));
  XL_TRY(dalloc(c, (size_t)n * 8, &b, "run keys"));
  XL_TRY(dalloc(c, k::radix_temp_bytes(n), &tmp, "sort scratch"));
  HIP_TRY(c, k::count_rows(x->skey(), x->wide, nullptr, n, cnt, c->stream));
  HIP_TRY(c, k::scan_exclusive_u32(cnt, off, k::row_tiles(n), tot, scan, c->stream));
  const uint32_t lo = x->r.lo[x->r.by];
  HIP_TRY(c, k::run_keys(x->skey(), x->wide, x->spay(), n, off, x->pay_bits, lo, a.as<u64>(), c->stream));
  int alt = 0;
  HIP_TRY(c, k::radix_sort_u64(a.as<u64>(), nullptr, b.as<u64>(), nullptr, n, x->pay_bits + bitlen(most - 1), tmp.p,
                               c->stream, &alt));
  HIP_TRY(c, k::run_payloads(alt ? b.as<u64>() : a.as<u64>(), n, x->pay_bits, lo, x->spay(), c->stream));
  return XL_OK;
}

// The distinct rows of the loaded columns in canonical order, by one sort of
// packed keys; a last column that is the payload is then ordered within the
// runs of equal keys: by counting, or, where a run is too long for that, by a
// second sort (8 M rows in runs of 200: 888 us; 2,050 column by column).  *done
// stays false when the columns do not fit a key and a payload or when the
// workspace does not hold a sort: the caller then sorts column by column.  Raw
// columns released by then are all written again, in another row order.
xl_status load_packed(Context* c, const Relation* r, const uint32_t* const* rc, Buf* raw, int64_t n,
                      const uint32_t* lo, const uint32_t* hi, Buf* fin, int64_t* m, bool* done) {
  *done = false;
  PackedRows x;
  if (!row_layout(r->types, r->arity, lo, hi, n, 0, &x)) return XL_OK;
  for (int j = 0; j < r->arity; ++j) {
    x.r.col[j] = rc[j];
    x.r.ltype[j] = r->types[j] == T_F32 ? XL_F32 : XL_I32;  // images stay as they are
  }
  bool freed = false;
  auto give_back = [&](xl_status st) -> xl_status {  // every column from the keys (all in one row order)
    if (st != XL_RESOURCE_EXHAUSTED || !freed) return st == XL_RESOURCE_EXHAUSTED ? XL_OK : st;
    x.key2.reset();
    x.pay2.reset();
    for (int j = 0; j < r->arity; ++j) {
      XL_TRY(dalloc(c, (size_t)n * 4, &raw[j], "loaded column"));
      x.r.dst[j] = raw[j].p;
    }
    HIP_TRY(c, k::unpack_rows(x.r, x.skey(), x.wide, x.spay(), n, nullptr, c->stream));
    return XL_OK;
  };
  xl_status st = sort_packed(c, &x, n, [&]() {
    for (int j = 0; j < r->arity; ++j) {
      freed = freed || raw[j].p;
      raw[j].reset();
    }
  });
  if (st != XL_OK) return give_back(st);
  const int64_t nt = k::row_tiles(n);
  Buf cnt, off, tmp, tot;
  XL_TRY(dalloc(c, (size_t)nt * 4, &cnt, "dedup counts"));
  XL_TRY(dalloc(c, (size_t)nt * 4, &off, "dedup offsets"));
  XL_TRY(dalloc(c, k::scan_temp_bytes(nt), &tmp, "scan scratch"));
  XL_TRY(dalloc(c, 8, &tot, "count"));
  uint32_t t[2] = {0, 0};  // rows that differ from the one before; whether a run is too long
  auto count = [&]() -> xl_status {
    HIP_TRY(c, k::count_rows(x.skey(), x.wide, x.spay(), n, cnt.as<uint32_t>(), c->stream));
    HIP_TRY(c, k::scan_exclusive_u32(cnt.as<uint32_t>(), off.as<uint32_t>(), nt, tot.as<uint32_t>(), tmp.p, c->stream));
    return ctl_read(c, tot.p, x.has_pay ? 8 : 4, t);
  };
  if (x.has_pay) {
    HIP_TRY(c, hipMemsetAsync(tot.p, 0, 8, c->stream));
    HIP_TRY(c, k::order_runs(x.skey(), x.wide, x.spay(), n, tot.as<uint32_t>() + 1, c->stream));
  }
  XL_TRY(count());
  if (t[1]) {
    st = order_long_runs(c, &x, n, t[0], cnt.as<uint32_t>(), off.as<uint32_t>(), tmp.p, tot.as<uint32_t>());
    if (st != XL_OK) return give_back(st);
    XL_TRY(count());
  }
  *m = t[0];
  for (int j = 0; j < r->arity; ++j) {
    XL_TRY(dalloc(c, (size_t)*m * 4, &fin[j], "relation column"));
    x.r.dst[j] = fin[j].p;
  }
  HIP_TRY(c, k::unpack_rows(x.r, x.skey(), x.wide, x.spay(), n, off.as<uint32_t>(), c->stream));
  *done = true;
  return XL_OK;
}

// The same by successive stable sorts of single columns (any columns).
xl_status load_by_columns(Context* c, const Relation* r, uint32_t* const* rc, Buf* raw, int64_t n, Buf* fin,
                          int64_t* m) {
  Buf perm;
  XL_TRY(lex_perm(c, rc, r->types, r->arity, n, &perm));
  Buf sorted[MAXC];
  const uint32_t* sc[MAXC] = {};
  for (int j = 0; j < r->arity; ++j) {
    XL_TRY(dalloc(c, (size_t)n * 4, &sorted[j], "sorted column"));
    HIP_TRY(c, k::gather_u32(rc[j], perm.as<uint32_t>(), sorted[j].as<uint32_t>(), n, c->stream));
    sc[j] = sorted[j].as<uint32_t>();
    raw[j].reset();
  }
  Buf flag, pos, tmp, tot;
  XL_TRY(dalloc(c, (size_t)n * 4, &flag, "dedup flags"));
  XL_TRY(dalloc(c, (size_t)n * 4, &pos, "dedup positions"));
  XL_TRY(dalloc(c, k::scan_temp_bytes(n), &tmp, "scan scratch"));
  XL_TRY(dalloc(c, 8, &tot, "count"));
  HIP_TRY(c, k::row_change_flags(sc, r->arity, n, flag.as<uint32_t>(), c->stream));
  HIP_TRY(c, k::scan_exclusive_u32(flag.as<uint32_t>(), pos.as<uint32_t>(), n, tot.as<uint32_t>(), tmp.p,
                                   c->stream));
  uint32_t mm = 0;
  XL_TRY(ctl_read(c, tot.p, 4, &mm));
  *m = mm;
  for (int j = 0; j < r->arity; ++j) {
    XL_TRY(dalloc(c, (size_t)*m * 4, &fin[j], "relation column"));
    HIP_TRY(c, k::compact_u32(sc[j], flag.as<uint32_t>(), pos.as<uint32_t>(), fin[j].as<uint32_t>(), n, c->stream));
  }
  return XL_OK;
}

}  // namespace

xl_status relation_load(Relation* r, const void* const* cols, int64_t n, int on_device) {
  Context* c = r->ctx;
  if (c->device < 0) return c->fail(XL_INVALID_ARGUMENT, "planning-only context cannot hold data");
  if (n < 0 || (n > 0 && !cols)) return c->fail(XL_INVALID_ARGUMENT, "bad row count or column pointers");
  if (n >= (int64_t)1 << 31) return c->fail(XL_CAPACITY_EXCEEDED, "relations hold fewer than 2^31 rows");
  for (int j = 0; j < r->arity && n > 0; ++j)
    if (!cols[j]) return c->fail(XL_INVALID_ARGUMENT, "null column pointer");
  if (n == 0) {
    relation_free_storage(r);
    return XL_OK;
  }
  Buf raw[MAXC];
  uint32_t* img[MAXC] = {};
  const uint32_t* rc[MAXC] = {};  // columns as images; the caller's own where it is device memory that needs no coding
  for (int j = 0; j < r->arity; ++j) {
    const bool plain = r->ltypes[j] == XL_I32 || r->ltypes[j] == XL_F32;
    if (plain && on_device && (uintptr_t)cols[j] % 4 == 0) {
      rc[j] = (const uint32_t*)cols[j];
      continue;
    }
    XL_TRY(dalloc(c, (size_t)n * 4, &raw[j], "loaded column"));
    rc[j] = img[j] = raw[j].as<uint32_t>();
    if (plain)
      HIP_TRY(c, hipMemcpyAsync(raw[j].p, cols[j], (size_t)n * 4,
                                on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream));
  }
  XL_TRY(encode_columns(c, r, cols, n, on_device, img));
  // sets: sort the rows, keep those that differ from their predecessor
  Buf fin[MAXC];
  int64_t m = 0;
  uint32_t lo[MAXC], hi[MAXC];
  bool done = false;
  if (n <= k::load_small_max()) {
    XL_TRY(load_small(c, r, rc, n, lo, hi, fin, &m, &done));
  }
  if (!done) {
    XL_TRY(image_bounds(c, rc, r->types, r->arity, n, lo, hi));
    XL_TRY(load_packed(c, r, rc, raw, n, lo, hi, fin, &m, &done));
  }
  if (!done) {
    uint32_t* lc[MAXC] = {};
    for (int j = 0; j < r->arity; ++j) {
      if (!raw[j].p) {  // (not read yet, or handed back by the packed sort)
        XL_TRY(dalloc(c, (size_t)n * 4, &raw[j], "loaded column"));
        HIP_TRY(c, hipMemcpyAsync(raw[j].p, cols[j], (size_t)n * 4, hipMemcpyDeviceToDevice, c->stream));
      }
      lc[j] = raw[j].as<uint32_t>();
    }
    XL_TRY(load_by_columns(c, r, lc, raw, n, fin, &m));
  }
  if (r->max_rows > 0 && m > r->max_rows)
    return c->fail(XL_CAPACITY_EXCEEDED, "relation " + r->name + " holds at most " +
                                             std::to_string(r->max_rows) + " rows, load has " +
                                             std::to_string(m));
  relation_free_storage(r);
  for (int j = 0; j < r->arity; ++j) {
    r->col[j] = (uint32_t*)fin[j].keep();
    if (r->types[j] == T_I32) {
      r->lo[j] = image_i32(lo[j]);
      r->hi[j] = image_i32(hi[j]);
    }
  }
  r->nrows = m;
  r->sorted = true;  // the deduplication above leaves the rows in lexicographic order
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return XL_OK;
}

// Sorts the rows of a relation whose leading key_cols columns are distinct and
// bounded as packed keys; false when they do not fit, or the workspace does
// not hold the sort.
static bool sorted_for_read(Context* c, const Relation* r, int64_t n, PackedRows* x) {
  uint32_t lo[MAXC], hi[MAXC];
  for (int j = 0; j < r->arity; ++j) {
    const bool i32 = r->types[j] == T_I32;
    lo[j] = i32 ? (uint32_t)r->lo[j] ^ 0x80000000u : 0u;
    hi[j] = i32 ? (uint32_t)r->hi[j] ^ 0x80000000u : 0xffffffffu;
    x->r.col[j] = r->col[j];
  }
  if (r->key_cols == 0 || !row_layout(r->types, r->arity, lo, hi, n, r->key_cols, x)) return false;
  if (x->has_pay && x->r.by != r->key_cols) return false;
  if (sort_packed(c, x, n, []() {}) == XL_OK) return true;
  for (Buf* b : {&x->key, &x->pay, &x->key2, &x->pay2}) b->reset();
  return false;
}

xl_status relation_read(const Relation* r, void* const* cols, int64_t cap, int64_t* out_rows,
                        int on_device) {
  Context* c = r->ctx;
  if (cap < r->nrows) {
    if (out_rows) *out_rows = r->nrows;
    return c->fail(XL_CAPACITY_EXCEEDED, "output capacity " + std::to_string(cap) + " < " +
                                             std::to_string(r->nrows) + " rows of " + r->name);
  }
  const int64_t n = r->nrows;
  if (n > 0) {
    if (!cols) return c->fail(XL_INVALID_ARGUMENT, "null column pointers");
    for (int j = 0; j < r->arity; ++j)
      if (!cols[j]) return c->fail(XL_INVALID_ARGUMENT, "null column pointer");
    // decode straight into the caller's device buffer when it is aligned for
    // the element size, else through device staging
    auto direct = [&](int j) { return on_device && (uintptr_t)cols[j] % elem_bytes(r->ltypes[j]) == 0; };
    auto plain = [&](int j) { return r->ltypes[j] == XL_I32 || r->ltypes[j] == XL_F32; };
    auto copy_out = [&](int j, const void* from) -> xl_status {
      HIP_TRY(c, hipMemcpyAsync(cols[j], from, (size_t)n * elem_bytes(r->ltypes[j]),
                                on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(c, hipStreamSynchronize(c->stream));
      return XL_OK;
    };
    // the workspace a read asks for is the column sort's, whatever route it
    // takes (host bookkeeping only)
    {
      LexScratch reserve;
      XL_TRY(lex_scratch(c, n, &reserve));
    }
    Buf stage, img;
    if (r->sorted) {
      // rows already in canonical order (a load, a bitmap, a dense array or a
      // triangle join wrote them so): no sort, one pass over the columns
      // (reading the 129 M-row R-MAT closure to the device: 16.0 -> 0.4 ms).
      k::ReadCols rc{};
      int nc = 0;
      for (int j = 0; j < r->arity; ++j) {
        if (!direct(j)) continue;
        rc.src[nc] = r->col[j];
        rc.dst[nc] = cols[j];
        rc.dict[nc] = c->dict[r->ltypes[j]];
        rc.ltype[nc++] = r->ltypes[j];
      }
      HIP_TRY(c, k::read_columns(rc, nc, n, c->stream));
      for (int j = 0; j < r->arity; ++j) {
        if (direct(j)) continue;
        if (!stage.p) XL_TRY(dalloc(c, (size_t)n * 8, &stage, "readout staging"));
        if (plain(j)) {
          XL_TRY(copy_out(j, r->col[j]));
          continue;
        }
        HIP_TRY(c, k::decode_column(r->col[j], n, r->ltypes[j], c->dict[r->ltypes[j]], stage.p, c->stream));
        XL_TRY(copy_out(j, stage.p));
      }
    } else if (PackedRows x; sorted_for_read(c, r, n, &x)) {
      // the rows from their sorted keys: the columns written directly in one
      // launch, then the staged ones
      for (int j = 0; j < r->arity; ++j) {
        x.r.ltype[j] = r->ltypes[j];
        x.r.dict[j] = c->dict[r->ltypes[j]];
        x.r.dst[j] = direct(j) ? cols[j] : nullptr;
      }
      HIP_TRY(c, k::unpack_rows(x.r, x.skey(), x.wide, x.spay(), n, nullptr, c->stream));
      for (int j = 0; j < r->arity; ++j) {
        if (direct(j)) continue;
        if (!stage.p) XL_TRY(dalloc(c, (size_t)n * 8, &stage, "readout staging"));
        for (int q = 0; q < r->arity; ++q) x.r.dst[q] = q == j ? stage.p : nullptr;
        HIP_TRY(c, k::unpack_rows(x.r, x.skey(), x.wide, x.spay(), n, nullptr, c->stream));
        XL_TRY(copy_out(j, stage.p));
      }
    } else {
      Buf perm;
      XL_TRY(lex_perm(c, r->col, r->types, r->arity, n, &perm));
      for (int j = 0; j < r->arity; ++j) {
        const int lt = r->ltypes[j];
        if (!direct(j) && !stage.p) XL_TRY(dalloc(c, (size_t)n * 8, &stage, "readout staging"));
        void* dst = direct(j) ? cols[j] : stage.p;
        if (plain(j)) {
          HIP_TRY(c, k::gather_u32(r->col[j], perm.as<uint32_t>(), (uint32_t*)dst, n, c->stream));
        } else {
          if (!img.p) XL_TRY(dalloc(c, (size_t)n * 4, &img, "readout images"));
          HIP_TRY(c, k::gather_u32(r->col[j], perm.as<uint32_t>(), img.as<uint32_t>(), n, c->stream));
          HIP_TRY(c, k::decode_column(img.as<uint32_t>(), n, lt, c->dict[lt], dst, c->stream));
        }
        if (!direct(j)) XL_TRY(copy_out(j, dst));
      }
    }
    HIP_TRY(c, hipStreamSynchronize(c->stream));
  }
  if (out_rows) *out_rows = n;
  return XL_OK;
}

// ================================================================== fixpoint run
namespace {

struct Interval {
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  bool empty() const { return lo > hi; }
  void join(const Interval& o) {
    lo = std::min(lo, o.lo);
    hi = std::max(hi, o.hi);
  }
  static Interval full() { return {INT32_MIN, INT32_MAX}; }
};

struct DevIndex {
  Relation* rel = nullptr;
  int col = 0;
  int order_col = -1;  // >= 0: rows of one key ordered by this column (see order_kind)
  int order_kind = 0;  // 0: by the degree of the value, most first; 1: by the int32 value
  uint32_t* first = nullptr;  // with order_col: order_col value of each key's first row
  IndexProbe probe{};
  std::vector<std::unique_ptr<Buf>> owned;
};

// Sorted keys of a complete relation projected onto the columns a negated
// literal constrains.
struct DevNeg {
  Relation* rel = nullptr;
  int ncols = 0;
  int col[2] = {0, 0};
  Buf keys, bits;
  int64_t n = 0;
  uint32_t lo = 0, last = 0;
  NegTable table() const {
    return NegTable{keys.as<unsigned long long>(), n, bits.as<uint32_t>(), lo, last};
  }
};

struct HeadRun {
  Relation* rel = nullptr;
  Agg agg = Agg::NONE;
  int fold = k::FOLD_NONE;
  bool is_set = false, is_minmax = false, is_sortagg = false;
  int nkey = 1;
  bool once = false;  // head of a non-recursive stratum: no delta is kept
  bool lean = false;  // the same for dense values (unless the receipt counts listed slots)
  bool sorted_set = false;  // set head of a scan: candidate keys, sorted and deduplicated at the end
  bool in_order = false;    // the candidates ascend as they are
  int64_t sure_rows = 0;    // hash set head: rows of a rule that copies a finished relation
  double growth = 1;        // of the delta over the last round of a batch
  KeyPack kp{};
  int bits0 = 1;      // width of the first packed key component
  double domain = 0;  // number of possible keys
  Buf table;
  int64_t cap = 0, keys = 0;
  // set heads: append-only row list of every tuple; the delta is a range
  Buf rows[2];
  int64_t rows_cap = 0, nrows = 0, dbeg = 0, dend = 0, round_begin = 0;
  int64_t round_new = 0;  // dense heads: tuples added this round
  // aggregate heads: delta rows (k0[, k1], value)
  Buf drow[3];
  int64_t dcap = 0, dn = 0;
  Buf didx;
  int64_t didx_n = 0;
  Buf ckey, cval;
  int64_t ccap = 0, cn = 0;
  uint32_t round = 0;
  int64_t preloaded = 0;
  // dense set heads: one bit per key of the (range0 x range1) key domain,
  // rows of row_bits bits indexed by the first key component
  bool dense = false;
  Buf bits;
  Buf dbits;  // tuples new in this round (same layout as bits)
  u64 row_bits = 0;
  uint32_t row_words = 0;
  int64_t range0 = 0;
  // frontier form (closure-shaped stratum over a dense two-column head): the
  // delta is one bitmap row per first-key value that gained tuples
  bool frontier = false;
  bool resident = false;        // frontier form run by one resident launch, which reads
                                // the seed's delta straight from dbits
  bool frontier_ready = false;  // the current delta is in fcnt/fdiff[fcur] (or dbits)
  Buf fx, fcnt[2], fdiff[2];    // delta row slot sg belongs to first-key value fx[sg]
  // gathered form (h(X,Y) :- e1(X,A), delta h(A,B), e2(Y,B)): the delta is
  // bitmap rows in dbits / gbits (by gcur) with one flag per row in gflag
  bool gathered = false;
  bool gather_ready = false;
  Buf gbits, gflag[2];
  Buf gbound[2];  // word bounds of the delta rows of dbits / gbits: lo[range0] then hi[range0]
  Buf ghubs;      // nonzero: the rounds OR by atomics (GatherArgs::hubs)
  int gcur = 0;
  // self-joined form (h(X,Y) :- h(X,Z), h(Z,Y)): the delta stays a bitmap
  // (dbits / gbits by turns), with the set bits of every row counted
  bool selfjoin = false;
  bool sj_on = false;  // the delta is in dbits: row-OR rounds from here on
  Buf scnt, dcnt[2];
  Buf hasin;                    // Y values with an in-edge (pull direction)
  int fcur = 0;
  int64_t fn = 0, fnew = 0;
  // dense count heads: one counter per key of the domain
  bool dcount = false;
  bool vbounds = false;  // the value column's bounds were read with the rows
  Buf counts;
  int64_t range1 = 1;
  // dense value heads (min/max): value array over (rank of the first key in
  // a dictionary of its possible values) x (second key - lo1), presence and
  // listed-this-round bits, and the dictionary (dmap: value - lo0 -> rank)
  bool dv = false;
  Buf dmap, dict, dvals, dpres, dchg;
  int64_t n0 = 0, dmap_n = 0;
  int64_t nrank_d = 0;  // sum/logsumexp heads: rank stride of the target-major delta slots (n0 rounded up to 32)
  std::vector<std::pair<Relation*, int>> dict_src;
  // dense sum/logsumexp heads (one carried-value variant): the same slots;
  // dvals/dpres hold the full relation, dcur/dcur_pres this round's delta,
  // dnext/dnext_pres the next one, dchg the keys marked for the pull
  bool ds = false;
  Buf dcur, dcur_pres, dnext, dnext_pres;
  Buf ndrow[3];
  bool pulled = false;
  int64_t pull_n = 0;
  // dense min/max heads with one carried-value variant: tiled rounds, the
  // delta rows grouped by rank (roff: first row of each rank)
  bool tiled = false;
  Buf roff;
  // e's rows grouped by (Z, tile of Y), built at the first tiled round
  std::vector<std::unique_ptr<Buf>> tcols;
  Buf toff;
  IndexProbe tidx{};
  uint32_t tile = 0, ntiles = 0;
  // key-column domains (bounds recorded on the materialized relation)
  int64_t dom_lo[2] = {0, 0}, dom_hi[2] = {0, 0};
  // batched rounds: this head's counters and round boundaries on the device
  // (row counts of its row list, or positions of the batch's slot list), the
  // base its emissions append at and its load limit
  u64* b_cnt = nullptr;
  u64* b_bnd = nullptr;
  u64 b_base = 0, b_limit = 0;
};

struct Runner {
  Context* c;
  Program* prog;
  xl_fixpoint_stats* st;
  std::vector<std::unique_ptr<DevIndex>> indexes;
  std::vector<std::unique_ptr<DevIndex>> kept;  // ready indexes made while materializing
  std::vector<std::unique_ptr<DevNeg>> negtabs;  // negation tables over complete relations
  std::vector<std::unique_ptr<HeadRun>> heads;
  int64_t cands = 0;
  hipEvent_t ev[2] = {nullptr, nullptr};
  ~Runner() {
    for (hipEvent_t e : ev)
      if (e) (void)hipEventDestroy(e);
  }

  // Slots of a dense value head's full relation (rank-major; sum/logsumexp
  // heads target-major, nrank_d ranks per target).
  static int64_t full_slots(const HeadRun* h) {
    return h->ds ? h->nrank_d * h->range1 : std::max<int64_t>(h->n0, 1) * h->range1;
  }

  HeadRun* head_of(const Relation* r) {
    for (auto& h : heads)
      if (h->rel == r) return h.get();
    return nullptr;
  }

  void record(int64_t rows) {
    if (st->rounds_recorded < XL_STATS_ROUNDS) st->delta_rows[st->rounds_recorded] = rows;
    st->rounds_recorded++;
  }

  // ------------------------------------------------------------ indexes
  // Index of rel by column col.  With order_col >= 0 the rows of each key are
  // further ordered: order_kind 0 by how many rows of rel have the order_col
  // value in column order_col (its out-degree when rel is an edge relation
  // indexed by its target), most first by base-8 class -- the
  // frontier pull scans in-edges
  // in that order, so that edges from well-connected sources, the likeliest
  // to be in a delta, come first; order_kind 1 by the int32 value itself
  // (the triangle join intersects sorted lists).
  // first (when given, with order_col >= 0) receives an array holding, per
  // key, the order_col value of the key's first row.
  xl_status get_index(Relation* rel, int col, IndexProbe* out, int order_col = -1,
                      const uint32_t** first = nullptr, int order_kind = 0, bool dense_only = false) {
    for (auto& ix : indexes)
      if (ix->rel == rel && ix->col == col && ix->order_col == order_col &&
          (order_col < 0 || ix->order_kind == order_kind) && (!dense_only || !ix->probe.keys)) {
        *out = ix->probe;
        if (first) *first = ix->first;
        return XL_OK;
      }
    const bool cacheable = c->index_cache_bytes > 0 && !head_of(rel);
    if (cacheable)
      for (CachedIndex& ce : c->icache)
        if (ce.rel == rel && ce.generation == rel->generation && ce.col == col && ce.order_col == order_col &&
            (!dense_only || !ce.probe.keys) &&
            (order_col < 0 || ce.order_kind == order_kind)) {
          ce.last_run = c->runs;
          auto ix = std::make_unique<DevIndex>();
          ix->rel = rel;
          ix->col = col;
          ix->order_col = order_col;
          ix->order_kind = order_kind;
          ix->probe = ce.probe;
          ix->first = ce.first;
          *out = ix->probe;
          if (first) *first = ix->first;
          indexes.push_back(std::move(ix));
          st->index_reuses++;
          return XL_OK;
        }
    st->index_builds++;
    auto ix = std::make_unique<DevIndex>();
    ix->rel = rel;
    ix->col = col;
    ix->order_col = order_col;
    ix->order_kind = order_kind;
    IndexProbe& p = ix->probe;
    p.ncols = rel->arity;
    auto own = [&](size_t bytes, const char* what, void** ptr) -> xl_status {
      ix->owned.push_back(std::make_unique<Buf>());
      XL_TRY(dalloc(c, bytes, ix->owned.back().get(), what));
      *ptr = ix->owned.back()->p;
      return XL_OK;
    };
    // rows as this round sees them: a head of the running stratum (a
    // self-join) contributes its current full relation
    const uint32_t* rcol[MAXC] = {};
    int64_t n = rel->nrows;
    int32_t klo = rel->lo[col], khi = rel->hi[col];
    for (int j = 0; j < rel->arity; ++j) rcol[j] = rel->col[j];
    if (HeadRun* h = head_of(rel)) {
      if (h->frontier || h->dcount || h->is_sortagg || col >= h->nkey)
        return c->fail(XL_UNSUPPORTED, "relation " + rel->name + " cannot be joined inside its own stratum");
      klo = (int32_t)h->dom_lo[col];
      khi = (int32_t)h->dom_hi[col];
      if (h->dense) {  // rows of the current bitmap, in key order
        n = h->keys;
        void* snap[2] = {nullptr, nullptr};
        for (int j = 0; j < h->nkey; ++j) XL_TRY(own((size_t)std::max<int64_t>(n, 1) * 4, "head snapshot", &snap[j]));
        Buf tmp, tot;
        if (h->nkey == 2) {
          Buf cnt, off;
          XL_TRY(dalloc(c, (size_t)h->range0 * 4, &cnt, "row counts"));
          XL_TRY(dalloc(c, (size_t)(h->range0 + 1) * 4, &off, "row offsets"));
          XL_TRY(dalloc(c, k::scan_temp_bytes(h->range0), &tmp, "scan scratch"));
          HIP_TRY(c, k::row_popcount(h->bits.as<uint32_t>(), h->range0, h->row_words, cnt.as<uint32_t>(), c->stream));
          HIP_TRY(c, k::scan_exclusive_u32(cnt.as<uint32_t>(), off.as<uint32_t>(), h->range0,
                                           off.as<uint32_t>() + h->range0, tmp.p, c->stream));
          HIP_TRY(c, k::bits_to_rows(h->bits.as<uint32_t>(), h->range0, h->row_words, off.as<uint32_t>(),
                                     h->kp.lo[0], h->kp.lo[1], (uint32_t*)snap[0], (uint32_t*)snap[1], n,
                                     c->stream));
          HIP_TRY(c, k::check_eq(off.as<uint32_t>() + h->range0, (uint32_t)n, c->dcheck, CHECK_BITMAP_ROWS,
                                 c->stream));
        } else {
          const int64_t nbits = (h->range0 + 31) / 32 * 32;
          XL_TRY(dalloc(c, k::bits_list_temp_bytes(nbits), &tmp, "compaction scratch"));
          XL_TRY(dalloc(c, 8, &tot, "count"));
          for (int pass = 0; pass < 2; ++pass)
            HIP_TRY(c, k::bits_keys(h->bits.as<uint32_t>(), nbits, 1, h->kp.lo[0], 0, 1, false, (uint32_t*)snap[0],
                                    nullptr, tot.as<uint32_t>(), tmp.p, pass == 1, c->stream));
        }
        for (int j = 0; j < h->nkey; ++j) rcol[j] = (const uint32_t*)snap[j];
      } else if (h->is_set) {
        n = h->nrows;
        for (int j = 0; j < h->nkey; ++j) rcol[j] = h->rows[j].as<uint32_t>();
      } else {  // min/max: compact a snapshot of the current keys and values
        n = h->keys;
        void* snap[3];
        for (int j = 0; j <= h->nkey; ++j) XL_TRY(own((size_t)std::max<int64_t>(n, 1) * 4, "head snapshot", &snap[j]));
        Buf tmp, tot;
        const int64_t ns = h->dv ? full_slots(h) : h->cap;
        XL_TRY(dalloc(c, k::compact_temp_bytes(ns), &tmp, "compaction scratch"));
        XL_TRY(dalloc(c, 8, &tot, "count"));
        uint32_t* k1 = h->nkey == 2 ? (uint32_t*)snap[1] : nullptr;
        if (h->dv)
          HIP_TRY(c, k::dense_rows(h->dvals.as<uint32_t>(), h->dpres.as<uint32_t>(), h->dict.as<uint32_t>(), ns,
                                   h->range1, h->kp, rel->types[h->nkey], h->fold, (uint32_t*)snap[0], k1,
                                   (uint32_t*)snap[h->nkey], std::max<int64_t>(n, 1), tot.as<uint32_t>(), tmp.p,
                                   c->stream));
        else
          HIP_TRY(c, k::table16_compact(h->table.as<Slot16>(), h->cap, h->kp, rel->types[h->nkey], h->fold,
                                        (uint32_t*)snap[0], k1, (uint32_t*)snap[h->nkey], std::max<int64_t>(n, 1),
                                        tot.as<uint32_t>(), tmp.p, c->stream));
        for (int j = 0; j <= h->nkey; ++j) rcol[j] = (const uint32_t*)snap[j];
      }
    }
    if (n == 0) {
      void* off;
      XL_TRY(own(8, "index offsets", &off));
      HIP_TRY(c, hipMemsetAsync(off, 0, 8, c->stream));
      p.off = (uint32_t*)off;
      p.keys = nullptr;
      p.key_lo = 0;
      p.key_range = 0;
      if (order_col >= 0 && order_kind == 0) {  // (no key, so never read)
        void* fp;
        XL_TRY(own(4, "index first rows", &fp));
        ix->first = (uint32_t*)fp;
      }
    } else {
      if (rel->types[col] != T_I32) return c->fail(XL_UNSUPPORTED, "index key columns must be int32");
      const int64_t range = (int64_t)khi - klo + 1;
      const bool ordered = order_col >= 0 && order_col < rel->arity && rel->types[order_col] == T_I32;
      // Direct-address offsets over a dense key range; a compacted index
      // (distinct keys, found by binary search) over a wide or sparse one.
      // The kernels that address per-key arrays by key value (frontier,
      // tiled, pull and gathered rounds, index degrees, degree order) ask for
      // the direct form; it and ordered indexes keep at most 2^25 rows.
      const bool compact = !dense_only && (order_col < 0 || order_kind == 1) &&
                           (range > ((int64_t)1 << 30) || (range > ((int64_t)1 << 22) && range > 16 * n));
      if ((dense_only || ordered) && n > ((int64_t)1 << 25))
        return c->fail(XL_UNSUPPORTED, "indexed relation " + rel->name + " exceeds 2^25 rows for this join form");
      if (!compact && range > ((int64_t)1 << 30))
        return c->fail(XL_UNSUPPORTED, "key range of " + rel->name + " column " + std::to_string(col) +
                                           " exceeds 2^30 values for this join form");
      const int kbits = std::max(1, bitlen((uint64_t)range - 1));
      // offsets from ascending key images: direct over the range, or compacted
      auto offsets = [&](const uint32_t* sorted_keys) -> xl_status {
        void* off;
        if (!compact) {
          XL_TRY(own((size_t)(range + 1) * 4, "index offsets", &off));
          HIP_TRY(c, k::csr_offsets(sorted_keys, n, (uint32_t)range, (uint32_t*)off, c->stream));
          p.off = (uint32_t*)off;
          p.keys = nullptr;
          p.key_range = (uint32_t)range;
          return XL_OK;
        }
        void* uk;
        Buf tmp, cnt;
        XL_TRY(own((size_t)(n + 1) * 4, "index offsets", &off));
        XL_TRY(own((size_t)n * 4, "index keys", &uk));
        XL_TRY(dalloc(c, k::compact_offsets_temp_bytes(n), &tmp, "index compaction scratch"));
        XL_TRY(dalloc(c, 8, &cnt, "count"));
        HIP_TRY(c, k::compact_offsets(sorted_keys, n, (uint32_t*)uk, (uint32_t*)off, cnt.as<uint32_t>(), tmp.p,
                                      c->stream));
        uint32_t nk = 0;
        XL_TRY(ctl_read(c, cnt.p, 4, &nk));
        p.off = (uint32_t*)off;
        p.keys = (const uint32_t*)uk;
        p.key_range = nk;
        // first segments by the key's high bits, half a bucket to two per key: a
        // probe of evenly spread keys then searches a few of them instead of all
        // (200,000 distinct ids over 2^31, 262,144 buckets, reachability rounds:
        // 1098 -> 952 us).
        // Without room for the buckets every probe searches the whole list.
        const int bb = std::min(kbits, bitlen((uint64_t)nk));
        p.bshift = (uint32_t)(kbits - bb);
        p.buckets = (uint32_t)(((uint64_t)range - 1) >> p.bshift) + 1;
        ix->owned.push_back(std::make_unique<Buf>());
        if (dalloc(c, ((size_t)p.buckets + 1) * 4, ix->owned.back().get(), "index buckets") == XL_OK) {
          p.bucket = ix->owned.back()->as<uint32_t>();
          HIP_TRY(c, k::csr_offsets_high(uk, false, (int)p.bshift, nk, p.buckets, (uint32_t*)p.bucket, c->stream));
        } else {
          ix->owned.pop_back();
        }
        return XL_OK;
      };
      // A loaded relation keeps its rows in lexicographic order, so its index
      // by the first column -- plain, or ordered by the second column's
      // values -- is its rows as they are: only the offsets are built, and
      // the index reads the relation's own columns.
      const bool presorted = !head_of(rel) && rel->sorted && col == 0 &&
                             (order_col < 0 || (ordered && order_col == 1 && order_kind == 1));
      if (presorted) {
        Buf keys;
        XL_TRY(dalloc(c, (size_t)n * 4, &keys, "index keys"));
        HIP_TRY(c, k::sub_lo(rcol[col], klo, keys.as<uint32_t>(), n, c->stream));
        XL_TRY(offsets(keys.as<uint32_t>()));
        for (int j = 0; j < rel->arity; ++j) p.col[j] = rcol[j];
        p.key_lo = klo;
        *out = p;
        if (first) *first = ix->first;
        if (cacheable) cache_index(*ix);
        indexes.push_back(std::move(ix));
        return XL_OK;
      }
      Buf perm, perm2, tmp;
      XL_TRY(dalloc(c, (size_t)n * 4, &perm, "index permutation"));
      XL_TRY(dalloc(c, (size_t)n * 4, &perm2, "index permutation"));
      XL_TRY(dalloc(c, k::radix_temp_bytes(n), &tmp, "sort scratch"));
      uint32_t* sp = nullptr;
      if (ordered) {
        // one sort by (key, order value), of 32-bit composite keys when
        // both parts fit; the offsets come from the sorted keys' high bits.
        // Degree order reads each order value's degree from the plain
        // index of rel by the order column (its row count as a key there).
        IndexProbe dz{};
        if (order_kind == 0) XL_TRY(get_index(rel, order_col, &dz, -1, nullptr, 0, true));
        // value order: the order column's bounds when known (a finished
        // relation, or a key column of a head), else the whole int32 range
        int32_t vlo = INT32_MIN;
        int vbits = 32;
        if (order_kind == 1) {
          HeadRun* oh = head_of(rel);
          if (!oh && rel->nrows > 0) {
            vlo = rel->lo[order_col];
            vbits = std::max(1, bitlen((uint64_t)((int64_t)rel->hi[order_col] - rel->lo[order_col])));
          } else if (oh && order_col < oh->nkey) {
            vlo = (int32_t)oh->dom_lo[order_col];
            vbits = std::max(1, bitlen((uint64_t)(oh->dom_hi[order_col] - oh->dom_lo[order_col])));
          }
        }
        const int obits = order_kind == 1 ? vbits : 2;  // degree order: four base-8 classes
        const bool wide = obits + kbits > 32;
        const size_t kw = wide ? 8 : 4;
        Buf ka, kb;
        XL_TRY(dalloc(c, (size_t)n * kw, &ka, "index order keys"));
        XL_TRY(dalloc(c, (size_t)n * kw, &kb, "index order keys"));
        HIP_TRY(c, k::order_keys(rcol[col], klo, rcol[order_col], order_kind == 1 ? vlo : dz.key_lo, obits,
                                 order_kind == 1 ? nullptr : dz.off, dz.key_range, n, ka.p, wide,
                                 perm.as<uint32_t>(), c->stream));
        int alt = 0;
        if (wide)
          HIP_TRY(c, k::radix_sort_u64(ka.as<u64>(), perm.as<uint32_t>(), kb.as<u64>(), perm2.as<uint32_t>(), n,
                                       obits + kbits, tmp.p, c->stream, &alt));
        else
          HIP_TRY(c, k::radix_sort_u32(ka.as<uint32_t>(), perm.as<uint32_t>(), kb.as<uint32_t>(),
                                       perm2.as<uint32_t>(), n, obits + kbits, tmp.p, c->stream, &alt));
        sp = alt ? perm2.as<uint32_t>() : perm.as<uint32_t>();
        const void* sk = alt ? kb.p : ka.p;
        if (!compact) {
          void* off;
          XL_TRY(own((size_t)(range + 1) * 4, "index offsets", &off));
          HIP_TRY(c, k::csr_offsets_high(sk, wide, obits, n, (uint32_t)range, (uint32_t*)off, c->stream));
          p.off = (uint32_t*)off;
          p.keys = nullptr;
          p.key_range = (uint32_t)range;
        } else {
          Buf keys;
          XL_TRY(dalloc(c, (size_t)n * 4, &keys, "index keys"));
          HIP_TRY(c, k::high_bits(sk, wide, obits, n, keys.as<uint32_t>(), c->stream));
          XL_TRY(offsets(keys.as<uint32_t>()));
        }
      } else {
        Buf keys, keys2;
        XL_TRY(dalloc(c, (size_t)n * 4, &keys, "index keys"));
        XL_TRY(dalloc(c, (size_t)n * 4, &keys2, "index keys"));
        HIP_TRY(c, k::keys_perm(rcol[col], klo, n, keys.as<uint32_t>(), perm.as<uint32_t>(), c->stream));
        int alt = 0;
        HIP_TRY(c, k::radix_sort_u32(keys.as<uint32_t>(), perm.as<uint32_t>(), keys2.as<uint32_t>(),
                                     perm2.as<uint32_t>(), n, kbits, tmp.p, c->stream, &alt));
        const uint32_t* sk = alt ? keys2.as<uint32_t>() : keys.as<uint32_t>();
        sp = alt ? perm2.as<uint32_t>() : perm.as<uint32_t>();
        XL_TRY(offsets(sk));
      }
      uint32_t* cols[MAXC] = {};
      for (int j = 0; j < rel->arity; ++j) {
        void* cj;
        XL_TRY(own((size_t)n * 4, "index column", &cj));
        cols[j] = (uint32_t*)cj;
        p.col[j] = cols[j];
      }
      HIP_TRY(c, k::gather_cols(rcol, cols, rel->arity, sp, n, c->stream));
      if (ordered && order_kind == 0) {
        void* fp;
        XL_TRY(own((size_t)range * 4, "index first rows", &fp));
        HIP_TRY(c, k::segment_first(p.off, p.col[order_col], (uint32_t)range, (uint32_t*)fp, c->stream));
        ix->first = (uint32_t*)fp;
      }
      p.key_lo = klo;
    }
    *out = p;
    if (first) *first = ix->first;
    if (cacheable) cache_index(*ix);
    indexes.push_back(std::move(ix));
    return XL_OK;
  }

  // Hand a freshly built index of a relation that is not a head to the
  // context's cache (its blocks then outlive the run), and evict the least
  // recently used entries not used by this run while the cache is over its
  // budget.
  void cache_index(DevIndex& ix) {
    CachedIndex ce;
    ce.rel = ix.rel;
    ce.generation = ix.rel->generation;
    ce.col = ix.col;
    ce.order_col = ix.order_col;
    ce.order_kind = ix.order_kind;
    ce.probe = ix.probe;
    ce.first = ix.first;
    ce.last_run = c->runs;
    for (auto& b : ix.owned) {
      ce.bytes += c->arena.block_size(b->p);
      ce.blocks.push_back(b->keep());
    }
    ix.owned.clear();
    c->icache.push_back(std::move(ce));
    size_t total = 0;
    for (const CachedIndex& e : c->icache) total += e.bytes;
    while (total > c->index_cache_bytes) {
      int victim = -1;
      for (int i = 0; i < (int)c->icache.size(); ++i)
        if (c->icache[i].last_run != c->runs &&
            (victim < 0 || c->icache[i].last_run < c->icache[victim].last_run))
          victim = i;
      if (victim < 0) break;  // every entry serves the running program
      total -= c->icache[victim].bytes;
      for (void* b : c->icache[victim].blocks) c->arena.release(b);
      c->icache.erase(c->icache.begin() + victim);
    }
  }

  // ------------------------------------------------------------ domains / heads
  Interval col_interval(Relation* rel, int col, const std::map<Relation*, std::vector<Interval>>& dom) {
    auto it = dom.find(rel);
    if (it != dom.end()) {
      if (col < (int)it->second.size()) return it->second[col];
      return Interval::full();
    }
    if (rel->nrows == 0) return Interval{};
    if (rel->types[col] != T_I32) return Interval::full();
    return Interval{rel->lo[col], rel->hi[col]};
  }

  // A min/max head can use a dense value array when every rule binds its
  // first key from a finished relation's column (a superset of the values it
  // can take) or carries it over from the head's own first column.  The
  // dictionary is the union of those columns (and of rows already loaded
  // into the head).
  void plan_dense_values(const Stratum& s, HeadRun* hr) {
    Relation* h = hr->rel;
    const int64_t r0 = hr->dom_hi[0] - hr->dom_lo[0] + 1;
    const int64_t r1 = hr->nkey == 2 ? hr->dom_hi[1] - hr->dom_lo[1] + 1 : 1;
    if (r0 <= 0 || r0 > ((int64_t)1 << 28) || r1 <= 0 || r1 > ((int64_t)1 << 30)) return;
    // the dictionary build needs two arrays over the first key's range, and
    // the arrays one row per dictionary value over the second key's range:
    // with the budget init_dv applies to the arrays, skip the dense form
    // before building a dictionary that could not be used
    const double budget = std::min(8589934592.0, (double)c->arena.capacity() / 4);
    if ((double)r0 * 8 > budget || (double)r1 * 16.5 > budget) return;
    std::vector<std::pair<Relation*, int>> src;
    for (const RulePlan& p : s.full) {
      if (p.head != h) continue;
      const int sl = p.key_slot[0];
      if (p.var_is_arith[sl]) return;
      bool carried = false;
      std::pair<Relation*, int> best{nullptr, 0};
      for (const auto& vs : p.var_sources[sl]) {
        if (vs.first == h && vs.second == 0) carried = true;
        bool in_stratum = false;
        for (Relation* o : s.heads) in_stratum = in_stratum || o == vs.first;
        if (in_stratum || vs.first->types[vs.second] != T_I32) continue;
        if (!best.first || vs.first->nrows < best.first->nrows) best = vs;
      }
      if (carried) continue;
      if (!best.first) return;
      src.push_back(best);
    }
    if (hr->is_minmax && h->nrows > 0) src.push_back({h, 0});  // loaded rows
    hr->dv = true;
    hr->dmap_n = r0;
    // rank rows start on word boundaries; a head without a second key has one
    // slot per rank
    hr->range1 = hr->nkey == 2 ? (r1 + 31) / 32 * 32 : 1;
    hr->dict_src = src;
  }

  // Candidates follow the driver's rows: keys that are the leading columns of
  // a finished driver in canonical order ascend as they are.
  bool keys_lead(const RulePlan& p) {
    bool lead = p.driver->sorted && !p.driver_delta && !head_of(p.driver);
    for (int j = 0; j < p.nkey; ++j)
      lead = lead && p.driver_act[j].kind == CA_BIND && p.driver_act[j].slot == p.key_slot[j];
    return lead;
  }

  // Every driver column is a key (or fixed by a constant or another column), so
  // no two of its rows make the same candidate.
  static bool keys_cover_driver(const RulePlan& p) {
    for (int j = 0; j < p.driver->arity; ++j) {
      const ColAct& a = p.driver_act[j];
      bool kept = a.kind == CA_CHECK_CONST || a.kind == CA_CHECK_SLOT;
      for (int q = 0; q < p.nkey; ++q) kept = kept || (a.kind == CA_BIND && a.slot == p.key_slot[q]);
      if (!kept) return false;
    }
    return true;
  }

  // Every row of the driver, a finished relation, is a row of the head.
  static bool copies_driver(const Stratum& s, const RulePlan& p) {
    bool all = p.steps.empty() && p.negs.empty() && keys_cover_driver(p);
    for (const auto& ops : p.stage_ops) all = all && ops.empty();
    for (int j = 0; j < p.driver->arity; ++j) all = all && p.driver_act[j].kind == CA_BIND;
    for (const Relation* h : s.heads) all = all && h != p.driver;
    return all;
  }

  xl_status setup_heads(Stratum& s) {
    joined_rows = 0;
    for (const RulePlan& p : s.variants)
      for (const StepPlan& sp : p.steps) joined_rows = std::max(joined_rows, sp.rel->nrows);
    std::map<Relation*, std::vector<Interval>> dom;
    for (Relation* h : s.heads) {
      const Agg a = prog->head_agg(h);
      const int nkey = h->arity - (a != Agg::NONE ? 1 : 0);
      std::vector<Interval> d(nkey);
      const bool keep = a == Agg::NONE || a == Agg::MIN || a == Agg::MAX;
      if (keep && h->nrows > 0)
        for (int j = 0; j < nkey; ++j) d[j] = Interval{h->lo[j], h->hi[j]};
      dom[h] = d;
    }
    for (int iter = 0; iter < 64; ++iter) {
      bool changed = false;
      for (RulePlan& p : s.full) {
        std::vector<Interval>& d = dom[p.head];
        for (int j = 0; j < p.nkey; ++j) {
          const int sl = p.key_slot[j];
          Interval iv;
          if (p.var_is_arith[sl]) {
            iv = Interval::full();
          } else {
            iv = Interval::full();
            for (auto& src : p.var_sources[sl]) {
              Interval o = col_interval(src.first, src.second, dom);
              iv.lo = std::max(iv.lo, o.lo);
              iv.hi = std::min(iv.hi, o.hi);
            }
          }
          if (iv.empty()) continue;
          Interval before = d[j];
          d[j].join(iv);
          changed = changed || before.lo != d[j].lo || before.hi != d[j].hi;
        }
      }
      if (!changed) break;
    }
    for (Relation* h : s.heads) {
      auto hr = std::make_unique<HeadRun>();
      hr->rel = h;
      hr->agg = prog->head_agg(h);
      hr->nkey = h->arity - (hr->agg != Agg::NONE ? 1 : 0);
      hr->is_set = hr->agg == Agg::NONE;
      hr->is_minmax = hr->agg == Agg::MIN || hr->agg == Agg::MAX;
      hr->is_sortagg = !hr->is_set && !hr->is_minmax;
      hr->once = !s.recursive;
      hr->lean = hr->once && !c->profile;
      switch (hr->agg) {
        case Agg::COUNT: hr->fold = k::FOLD_COUNT; break;
        case Agg::SUM: hr->fold = k::FOLD_SUM; break;
        case Agg::MIN: hr->fold = k::FOLD_MIN; break;
        case Agg::MAX: hr->fold = k::FOLD_MAX; break;
        case Agg::LSE: hr->fold = k::FOLD_LSE; break;
        default: hr->fold = k::FOLD_NONE;
      }
      std::vector<Interval>& d = dom[h];
      KeyPack kp{};
      kp.nkey = hr->nkey;
      int bits0 = 1;
      double dsize = 1;
      int full = 0;  // key columns whose domain spans all 2^32 values
      for (int j = 0; j < hr->nkey; ++j) {
        Interval iv = d[j].empty() ? Interval{0, 0} : d[j];
        kp.lo[j] = (int32_t)iv.lo;
        const int b = std::max(1, bitlen((uint64_t)(iv.hi - iv.lo)));
        if (j == 0) bits0 = b; else kp.shift = b;
        dsize *= (double)(iv.hi - iv.lo + 1);
        full += iv.hi - iv.lo == 0xffffffffll;
      }
      // a packed key is all ones (the empty-slot marker of the hash tables)
      // only for the largest tuple of two key domains of 2^32 values each
      if (hr->nkey == 2 && full == 2)
        return c->fail(XL_UNSUPPORTED, "both key columns of " + h->name + " span all 2^32 values");
      hr->kp = kp;
      hr->bits0 = bits0;
      hr->domain = dsize;
      for (int j = 0; j < hr->nkey; ++j) {
        const Interval iv = d[j].empty() ? Interval{0, 0} : d[j];
        hr->dom_lo[j] = iv.lo;
        hr->dom_hi[j] = iv.hi;
      }
      if (hr->agg == Agg::COUNT && c->index_mode != 1) {
        const int64_t r0 = hr->dom_hi[0] - hr->dom_lo[0] + 1;
        const int64_t r1 = hr->nkey == 2 ? hr->dom_hi[1] - hr->dom_lo[1] + 1 : 1;
        if ((double)r0 * (double)r1 * 4 <= std::min(4294967296.0, (double)c->arena.capacity() / 8)) {
          hr->dcount = true;
          hr->range0 = r0;
          hr->range1 = r1;
        }
      }
      if (hr->is_minmax && c->index_mode != 1) {
        plan_dense_values(s, hr.get());
        hr->tiled = hr->dv && hr->nkey == 2 && c->dense_tiles >= 0 && s.recursive && s.heads.size() == 1 &&
                    s.variants.size() == 1 && s.variants[0].carried_val;
      }
      if ((hr->agg == Agg::SUM || hr->agg == Agg::LSE) && hr->nkey == 2 && c->index_mode != 1 && s.recursive &&
          s.heads.size() == 1 && s.variants.size() == 1 && s.variants[0].carried_val) {
        plan_dense_values(s, hr.get());
        hr->ds = hr->dv;
      }
      if (hr->is_set && c->index_mode != 1) {
        const Interval i0 = d[0].empty() ? Interval{0, 0} : d[0];
        const int64_t range0 = i0.hi - i0.lo + 1;
        int64_t range1 = 1;
        if (hr->nkey == 2) {
          const Interval i1 = d[1].empty() ? Interval{0, 0} : d[1];
          range1 = i1.hi - i1.lo + 1;
        }
        const u64 row_bits = hr->nkey == 2 ? (u64)((range1 + 31) / 32) * 32 : 1;
        const double total_bits = hr->nkey == 2 ? (double)range0 * (double)row_bits
                                                : (double)((range0 + 31) / 32) * 32.0;
        const double budget = c->index_mode == 2 ? (double)c->arena.capacity() / 2
                                                 : std::min(4294967296.0, (double)c->arena.capacity() / 4);
        // A set head whose rules only scan: at most as many candidates as
        // driver rows, so a sort of their keys replaces a bitmap that is far
        // larger than them (its clear, count and listing pass over every
        // word: 300 + 780 + 240 us for 1.25 GB holding 0.9 M rows, 80
        // as candidate keys), or a hash table whose rows every read would
        // sort.  The table stays where rows may repeat (a driver column that
        // is no key) and have to be sorted: it holds each once.  Rows turned
        // from 10 M candidates, evaluate and read, us (table / sorted): all
        // distinct 1035 / 812, a tenth of them 707 / 825, 1,000 rows 530 /
        // 986; from 100,000 candidates 200 / 210, 172 / 212 and 119 / 217; in
        // ascending order (no sort) 10 M take 250 and 219 sorted.  Up to 4,096
        // candidates are sorted in one launch.
        bool scans = hr->once && h->nrows == 0 && c->index_mode == 0, distinct = true;
        double rows = 0;
        for (const RulePlan& p : s.full) {
          scans = scans && p.head == h && p.steps.empty();
          distinct = distinct && keys_cover_driver(p);
          rows += (double)p.driver->nrows;
        }
        auto sorted_beats_table = [&]() {
          const bool lead = s.full.size() == 1 && keys_lead(s.full[0]);
          if ((lead ? 8 : 16) * rows > (double)(c->arena.capacity() - c->arena.in_use())) return false;  // no room
          // a table of distinct candidates grows to eight slots of 16 bytes per
          // row at most, or to 16 M slots, beside the one before it
          const double table = 160 * rows + (272 << 20) + 16.0 * (double)((int64_t)1 << c->hash_min_log2);
          return distinct || lead || rows <= 4096 || table > (double)c->arena.largest_free();
        };
        if (scans && rows < 2147483648.0 &&
            (total_bits / 8 > budget ? sorted_beats_table() : total_bits / 8 > 33554432.0 + 160.0 * rows)) {
          hr->sorted_set = true;
        } else if (total_bits / 8 <= budget) {
          hr->dense = true;
          hr->range0 = range0;
          hr->row_bits = row_bits;
          hr->row_words = (uint32_t)std::min<u64>(row_bits / 32, 0xffffffffull);
          // frontier form: the stratum is this head alone with one closure-shaped
          // variant; its kernel stages three rows of row_words words plus about
          // 19 KB in LDS, which must stay within a workgroup's 64 KB
          hr->frontier = s.recursive && s.heads.size() == 1 && s.variants.size() == 1 &&
                         s.variants[0].carried && hr->nkey == 2 && hr->row_words <= 3072 &&
                         total_bits / 8 * 3 <= budget;
          hr->resident = hr->frontier && c->frontier_resident;
          GatherShape gs;
          hr->gathered = !hr->frontier && c->gather_rounds && s.recursive && s.heads.size() == 1 &&
                         s.variants.size() == 1 && hr->nkey == 2 && hr->is_set && hr->row_words <= 3072 &&
                         total_bits / 8 * 2 <= budget && gather_shape(s.variants[0], &gs);
          // self-joined form, whole rows ORed: rows of at most 512 words;
          // fewer than 2^26 first keys, so no join key can reach the stage
          // kernel's limit of rows
          hr->selfjoin = s.recursive && s.heads.size() == 1 && hr->nkey == 2 && c->batched_rounds > 0 &&
                         hr->row_words <= k::SJ_MAX_WORDS && range0 < ((int64_t)1 << 26) &&
                         total_bits / 8 * 3 <= budget && self_join_shape(s.variants);
        }
      }
      if (hr->is_set && s.recursive)
        for (const RulePlan& p : s.full)
          if (p.head == h && copies_driver(s, p)) hr->sure_rows = std::max(hr->sure_rows, p.driver->nrows);
      hr->preloaded = (hr->is_set || hr->is_minmax) ? h->nrows : 0;
      XL_TRY(init_head(hr.get()));
      heads.push_back(std::move(hr));
    }
    return XL_OK;
  }

  size_t slot_bytes(const HeadRun* h) const { return h->is_set ? 8 : sizeof(Slot16); }

  xl_status alloc_table(HeadRun* h, int64_t cap, Buf* out) {
    XL_TRY(dalloc(c, (size_t)cap * slot_bytes(h), out, "hash table"));
    HIP_TRY(c, k::fill_bytes(out->p, 0xff, (size_t)cap * slot_bytes(h), c->stream));
    return XL_OK;
  }

  // Slots for a recursive set head that fills: eight per row of the largest
  // relation its rules join, within 64 times the smallest table and 1/32 of the
  // free workspace.
  int64_t filled_cap(const HeadRun* h) const {
    if (!h->is_set || h->once) return 0;
    return std::min({(int64_t)next_pow2((uint64_t)joined_rows * 8), (int64_t)64 << c->hash_min_log2,
                     (int64_t)next_pow2(c->arena.largest_free() / 32 / 16 + 1) / 2});
  }
  // First capacity of a head's hash table: 2^hash_min_log2 slots, or four per
  // expected row.  Batched rounds use as many wavefronts as a quarter of the
  // slots allows, and a growth inside a batch runs a round and inserts every row
  // again; but every slot is cleared, whatever the head ends with.  So a
  // recursive set head starts at filled_cap only within eight times the smallest
  // table or eight slots per row it is sure to get, and takes the rest where the
  // next batch would fill half of what it has (widen).  Evaluate and read, us, ids
  // over 2^31, from filled_cap / so: 39 rows from 12 M edges 795 / 640, from 30 M
  // 1250 / 907; 16 sources over 3 M edges (12 M rows) 3110 / 3170, over 12 M
  // (47 M rows) 11800 / 12200; 2 sources over 30 M (15 M rows) 4920 / 5710; chains
  // of four edges, 12 M (30 M rows) 6130 / 6180.  From 4 M slots with growths 16
  // sources over 0.8 M edges (3 M rows) take 2008 where these take 1200, over
  // 12 M 18300.
  int64_t initial_cap(const HeadRun* h, int64_t expect) {
    const int64_t cap = (int64_t)1 << c->hash_min_log2;
    const int64_t full = std::max(8 * cap, (int64_t)next_pow2((uint64_t)h->sure_rows * 8));
    return std::max({cap, std::min(full, filled_cap(h)),
                     (int64_t)next_pow2((uint64_t)std::max<int64_t>(expect, 1) * 4)});
  }
  // Before a batch of `rounds`: its rows as the last round's delta and growth
  // promise them, once there is a row per 64 slots (few rows multiply for a
  // round or two only).
  xl_status widen(HeadRun* h, int rounds) {
    if (h->keys * 64 < h->cap) return XL_OK;
    double rows = (double)h->keys, d = (double)(h->dend - h->dbeg);
    for (int r = 0; r < rounds; ++r) rows += d *= h->growth;
    const int64_t want = filled_cap(h);
    return rows > 0.5 * (double)h->cap && want > h->cap ? grow(h, 0, want) : XL_OK;
  }
  int64_t joined_rows = 0;  // rows of the largest relation outside the stratum that a variant joins

  xl_status init_dense(HeadRun* h) {
    Relation* r = h->rel;
    const double total_bits = h->nkey == 2 ? (double)h->range0 * (double)h->row_bits
                                           : (double)((h->range0 + 31) / 32) * 32.0;
    const size_t bytes = (size_t)(total_bits / 8);
    XL_TRY(dalloc(c, bytes, &h->bits, "dense key bitmap"));
    HIP_TRY(c, k::fill_bytes(h->bits.p, 0, bytes, c->stream));
    if (!h->once) {
      XL_TRY(dalloc(c, bytes, &h->dbits, "dense delta bitmap"));
      HIP_TRY(c, k::fill_bytes(h->dbits.p, 0, bytes, c->stream));
    }
    // the row list only holds loaded rows (the seed scans them); derived
    // tuples live in the bitmap and each round's delta in dbits
    h->rows_cap = std::max<int64_t>(h->preloaded, 1);
    for (int j = 0; j < h->nkey; ++j) {
      XL_TRY(dalloc(c, (size_t)h->rows_cap * 4, &h->rows[j], "relation rows"));
      if (h->preloaded)
        HIP_TRY(c, hipMemcpyAsync(h->rows[j].p, r->col[j], (size_t)h->preloaded * 4,
                                  hipMemcpyDeviceToDevice, c->stream));
    }
    HIP_TRY(c, k::bits_set_rows(h->bits.as<uint32_t>(), h->row_bits, h->rows[0].as<uint32_t>(),
                                h->nkey == 2 ? h->rows[1].as<uint32_t>() : nullptr, h->preloaded, h->kp,
                                c->stream));
    h->nrows = h->keys = h->preloaded;
    h->dbeg = h->dend = 0;
    if (h->selfjoin) {  // without room for its buffers the generic join takes the rounds
      const size_t cb = (size_t)std::max<int64_t>(h->range0, 1) * 4;
      h->selfjoin = dalloc(c, bytes, &h->gbits, "dense delta bitmap") == XL_OK &&
                    dalloc(c, cb, &h->scnt, "row counts") == XL_OK &&
                    dalloc(c, cb, &h->dcnt[0], "row counts") == XL_OK &&
                    dalloc(c, cb, &h->dcnt[1], "row counts") == XL_OK;
      if (!h->selfjoin)
        for (Buf* b : {&h->gbits, &h->scnt, &h->dcnt[0], &h->dcnt[1]}) b->reset();
    }
    if (h->gathered) {
      XL_TRY(dalloc(c, bytes, &h->gbits, "dense delta bitmap"));
      HIP_TRY(c, k::fill_bytes(h->gbits.p, 0, bytes, c->stream));
      for (int b = 0; b < 2; ++b) {
        XL_TRY(dalloc(c, (size_t)std::max<int64_t>(h->range0, 1) * 4, &h->gflag[b], "delta row flags"));
        HIP_TRY(c, hipMemsetAsync(h->gflag[b].p, 0, (size_t)std::max<int64_t>(h->range0, 1) * 4, c->stream));
        XL_TRY(dalloc(c, (size_t)std::max<int64_t>(h->range0, 1) * 8, &h->gbound[b], "delta row bounds"));
        HIP_TRY(c, k::fill_bounds(h->gbound[b].as<uint32_t>(), h->gbound[b].as<uint32_t>() + h->range0, h->range0,
                                  (uint32_t)h->row_words, 0u, c->stream));
      }
    }
    if (h->frontier && !h->resident) {
      XL_TRY(dalloc(c, (size_t)std::max<int64_t>(h->range0, 1) * 4, &h->fx, "delta row keys"));
      for (int b = 0; b < 2; ++b) {
        XL_TRY(dalloc(c, (size_t)std::max<int64_t>(h->range0, 1) * 4, &h->fcnt[b], "delta row counts"));
        XL_TRY(dalloc(c, (size_t)std::max<int64_t>(h->range0, 1) * h->row_words * 4, &h->fdiff[b],
                      "delta bitmap rows"));
      }
    }
    return XL_OK;
  }

  xl_status init_dcount(HeadRun* h) {
    const size_t bytes = (size_t)h->range0 * (size_t)h->range1 * 4;
    XL_TRY(dalloc(c, bytes, &h->counts, "dense counters"));
    HIP_TRY(c, k::fill_bytes(h->counts.p, 0, bytes, c->stream));
    return XL_OK;
  }



  // Build the first-key dictionary, then the dense arrays if they fit; a
  // head that does not fit falls back to the hash table (h->dv cleared).
  xl_status init_dv(HeadRun* h) {
    Relation* r = h->rel;
    const uint32_t range = (uint32_t)h->dmap_n;
    Buf pos, tmp, tot;
    XL_TRY(dalloc(c, (size_t)range * 4, &h->dmap, "key dictionary map"));
    HIP_TRY(c, hipMemsetAsync(h->dmap.p, 0, (size_t)range * 4, c->stream));
    for (const auto& sc : h->dict_src) {
      const int64_t n = sc.first == r ? h->preloaded : sc.first->nrows;
      HIP_TRY(c, k::dict_mark(sc.first->col[sc.second], n, h->kp.lo[0], range, h->dmap.as<uint32_t>(),
                              c->stream));
    }
    XL_TRY(dalloc(c, (size_t)range * 4, &pos, "key dictionary ranks"));
    XL_TRY(dalloc(c, k::scan_temp_bytes(range), &tmp, "scan scratch"));
    XL_TRY(dalloc(c, 8, &tot, "count"));
    HIP_TRY(c, k::scan_exclusive_u32(h->dmap.as<uint32_t>(), pos.as<uint32_t>(), range, tot.as<uint32_t>(),
                                     tmp.p, c->stream));
    uint32_t n0 = 0;
    XL_TRY(ctl_read(c, tot.p, 4, &n0));
    h->n0 = n0;
    const double slots = (double)std::max<uint32_t>(n0, 1) * (double)h->range1;
    // sum/logsumexp heads pad the ranks to whole words: their slot indices
    // (32-bit in the kernels) run up to the padded count
    const double padded = h->ds ? (double)((std::max<uint32_t>(n0, 1) + 31) / 32 * 32) * (double)h->range1 : slots;
    const double budget = std::min(8589934592.0, (double)c->arena.capacity() / 4);
    if (padded >= 4294967296.0 || padded * (h->ds ? 16.5 : 8.25) > budget) {
      h->dv = h->ds = h->tiled = false;
      h->dmap.reset();
      return XL_OK;
    }
    XL_TRY(dalloc(c, (size_t)std::max<uint32_t>(n0, 1) * 4, &h->dict, "key dictionary"));
    HIP_TRY(c, k::dict_finish(h->dmap.as<uint32_t>(), pos.as<uint32_t>(), range, h->kp.lo[0],
                              h->dict.as<uint32_t>(), c->stream));
    // sum/logsumexp heads lay the full relation out like their delta slots
    // (target-major, ranks padded to whole words)
    if (h->ds) h->nrank_d = (std::max<int64_t>(n0, 1) + 31) / 32 * 32;
    const size_t ns = h->ds ? (size_t)h->nrank_d * (size_t)h->range1 : (size_t)slots, nw = (ns + 31) / 32;
    XL_TRY(dalloc(c, ns * 4, &h->dvals, "dense values"));
    XL_TRY(dalloc(c, nw * 4, &h->dpres, "dense presence bits"));
    HIP_TRY(c, k::fill_bytes(h->dvals.p, 0xff, ns * 4, c->stream));
    HIP_TRY(c, k::fill_bytes(h->dpres.p, 0, nw * 4, c->stream));
    if (!h->lean) {
      XL_TRY(dalloc(c, nw * 4, &h->dchg, "dense delta bits"));
      HIP_TRY(c, k::fill_bytes(h->dchg.p, 0, nw * 4, c->stream));
    }
    if (h->tiled) XL_TRY(dalloc(c, (size_t)(n0 + 1) * 4, &h->roff, "delta rows per rank"));
    if (h->ds) {
      // target-major delta slots with whole words per target: y * nrank_d + rank
      const size_t nsd = (size_t)h->nrank_d * (size_t)h->range1, nwd = nsd / 32;
      XL_TRY(dalloc(c, nsd * 4, &h->dcur, "dense delta values"));
      XL_TRY(dalloc(c, nsd * 4, &h->dnext, "dense delta values"));
      XL_TRY(dalloc(c, nwd * 4, &h->dcur_pres, "dense delta bits"));
      XL_TRY(dalloc(c, nwd * 4, &h->dnext_pres, "dense delta bits"));
      XL_TRY(dalloc(c, nwd * 4, &h->dchg, "dense delta marks"));
      HIP_TRY(c, k::fill_bytes(h->dcur_pres.p, 0, nwd * 4, c->stream));
      HIP_TRY(c, k::fill_bytes(h->dnext_pres.p, 0, nwd * 4, c->stream));
      HIP_TRY(c, k::fill_bytes(h->dchg.p, 0, nwd * 4, c->stream));
    } else if (!h->lean) {
      XL_TRY(dalloc(c, ns * 4, &h->didx, "delta slot list"));
    }
    h->keys = 0;
    if (h->preloaded) {
      HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
      HIP_TRY(c, k::dense_insert_rows(h->dvals.as<uint32_t>(), h->dpres.as<uint32_t>(), h->dmap.as<uint32_t>(),
                                      range, (uint32_t)h->range1, r->col[0], h->nkey == 2 ? r->col[1] : nullptr,
                                      r->col[h->nkey], h->preloaded, h->kp, r->types[h->nkey],
                                      h->agg == Agg::MAX, c->dcounters, c->stream));
      u64 cnt[CNT_N];
      XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
      if (cnt[CNT_FATAL]) return c->fail(XL_DEVICE_ERROR, "loaded row outside the dense domain (internal)");
      h->keys = (int64_t)cnt[CNT_INSERTED];
    }
    return XL_OK;
  }

  xl_status init_head(HeadRun* h) {
    Relation* r = h->rel;
    if (h->dv) {
      XL_TRY(init_dv(h));
      if (h->dv) return XL_OK;
    }
    if (h->dense) return init_dense(h);
    if (h->dcount) return init_dcount(h);
    if (h->sorted_set || (h->is_sortagg && h->once)) return XL_OK;  // rows come from the sorted candidates
    h->cap = initial_cap(h, h->preloaded);
    XL_TRY(alloc_table(h, h->cap, &h->table));
    if (h->is_set) {
      h->rows_cap = h->cap;
      for (int j = 0; j < h->nkey; ++j) {
        XL_TRY(dalloc(c, (size_t)h->rows_cap * 4, &h->rows[j], "relation rows"));
        if (h->preloaded)
          HIP_TRY(c, hipMemcpyAsync(h->rows[j].p, r->col[j], (size_t)h->preloaded * 4,
                                    hipMemcpyDeviceToDevice, c->stream));
      }
      if (h->preloaded)
        HIP_TRY(c, k::set_insert_rows(h->table.as<u64>(), (u64)h->cap - 1, h->rows[0].as<uint32_t>(),
                                      h->nkey == 2 ? h->rows[1].as<uint32_t>() : nullptr, h->preloaded,
                                      h->kp, c->dcounters, c->stream));
      h->nrows = h->keys = h->preloaded;
      h->dbeg = h->dend = 0;
    } else {
      if (h->is_minmax) {
        XL_TRY(dalloc(c, (size_t)h->cap * 4, &h->didx, "delta slot list"));
        h->keys = 0;
        if (h->preloaded) {  // several loaded rows may share a key: count distinct keys
          HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
          HIP_TRY(c, k::table16_insert_rows(h->table.as<Slot16>(), (u64)h->cap - 1, r->col[0],
                                            h->nkey == 2 ? r->col[1] : nullptr, r->col[h->nkey],
                                            h->preloaded, h->kp, r->types[h->nkey],
                                            h->agg == Agg::MAX, c->dcounters, c->stream));
          u64 cnt[CNT_N];
          XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
          if (cnt[CNT_FATAL]) return c->fail(XL_DEVICE_ERROR, "hash table probe exhausted (internal)");
          h->keys = (int64_t)cnt[CNT_INSERTED];
        }
      }
    }
    return XL_OK;
  }

  // Grow the head's table (and row list) so it holds at least `need` keys, or to
  // `want` slots.
  xl_status grow(HeadRun* h, int64_t need, int64_t want = 0) {
    int64_t ncap = want ? want : h->cap * 4;
    while (!want && (ncap / 2 < need || ncap - need < WAVE_SLACK * 4 * EMIT_GRID + 1024)) ncap *= 2;
    Buf nt;
    XL_TRY(alloc_table(h, ncap, &nt));
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    if (h->is_set) {
      Buf nr[2];
      for (int j = 0; j < h->nkey; ++j) {
        XL_TRY(dalloc(c, (size_t)ncap * 4, &nr[j], "relation rows"));
        HIP_TRY(c, hipMemcpyAsync(nr[j].p, h->rows[j].p, (size_t)h->nrows * 4, hipMemcpyDeviceToDevice,
                                  c->stream));
      }
      HIP_TRY(c, k::set_insert_rows(nt.as<u64>(), (u64)ncap - 1, nr[0].as<uint32_t>(),
                                    h->nkey == 2 ? nr[1].as<uint32_t>() : nullptr, h->nrows, h->kp,
                                    c->dcounters, c->stream));
      for (int j = 0; j < h->nkey; ++j) std::swap(h->rows[j].p, nr[j].p);
      h->rows_cap = ncap;
    } else {
      HIP_TRY(c, k::table16_rehash(h->table.as<Slot16>(), h->cap, nt.as<Slot16>(), (u64)ncap - 1,
                                   c->dcounters, c->stream));
      if (h->is_minmax) {
        Buf nd;
        XL_TRY(dalloc(c, (size_t)ncap * 4, &nd, "delta slot list"));
        std::swap(h->didx.p, nd.p);
      }
    }
    std::swap(h->table.p, nt.p);
    h->cap = ncap;
    st->table_grows++;
    u64 cnt[CNT_N];
    XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
    if (cnt[CNT_FATAL]) return c->fail(XL_DEVICE_ERROR, "hash table rebuild failed");
    if (h->is_minmax && h->didx_n > 0) {
      // the slots listed for the current round moved: list the slots stamped
      // with the round again (in slot order)
      Buf tmp, tot;
      XL_TRY(dalloc(c, k::compact_temp_bytes(h->cap), &tmp, "compaction scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      HIP_TRY(c, k::table16_stamped(h->table.as<Slot16>(), h->cap, h->round, h->didx.as<uint32_t>(), h->cap,
                                    tot.as<uint32_t>(), tmp.p, c->stream));
      uint32_t n2 = 0;
      XL_TRY(ctl_read(c, tot.p, 4, &n2));
      h->didx_n = (int64_t)n2;
    }
    return XL_OK;
  }

  // ------------------------------------------------------------ rule evaluation
  struct Source {
    const uint32_t* col[MAXV];
    int64_t n;
  };

  Source resolve_driver(const RulePlan& p) {
    Source s{};
    HeadRun* h = head_of(p.driver);
    if (h && p.driver_delta) {
      if (h->is_set && !h->dense) {
        for (int j = 0; j < h->nkey; ++j) s.col[j] = h->rows[j].as<uint32_t>() + h->dbeg;
        s.n = h->dend - h->dbeg;
      } else {
        for (int j = 0; j < p.driver->arity; ++j) s.col[j] = h->drow[j].as<uint32_t>();
        s.n = h->dn;
      }
    } else if (h && h->is_set) {  // full scan of a head of this stratum (seed)
      for (int j = 0; j < h->nkey; ++j) s.col[j] = h->rows[j].as<uint32_t>();
      s.n = h->preloaded;
    } else {
      for (int j = 0; j < p.driver->arity; ++j) s.col[j] = p.driver->col[j];
      s.n = h ? h->preloaded : p.driver->nrows;
    }
    return s;
  }

  xl_status fill_ops(StageArgs& a, const RulePlan& p, int ks) {
    a.nops = (int)p.stage_ops[ks].size();
    for (int i = 0; i < a.nops; ++i) a.ops[i] = p.stage_ops[ks][i];
    for (size_t i = 0; i < p.stage_consts[ks].size(); ++i) a.consts[i] = p.stage_consts[ks][i];
    for (size_t q = 0; q < p.negs.size(); ++q) XL_TRY(get_neg(p.negs[q], &a.neg[q]));
    return XL_OK;
  }

  // The negation table of a negated literal over a complete relation (its
  // stratum ran before; stratification guarantees it): q's rows projected
  // onto the constrained columns, packed and radix sorted.
  xl_status get_neg(const NegPlan& np, NegTable* out) {
    for (auto& t : negtabs)
      if (t->rel == np.rel && t->ncols == np.ncols && (np.ncols < 1 || t->col[0] == np.col[0]) &&
          (np.ncols < 2 || t->col[1] == np.col[1])) {
        *out = t->table();
        return XL_OK;
      }
    if (head_of(np.rel)) return c->fail(XL_DEVICE_ERROR, "negated relation is not complete (internal)");
    auto t = std::make_unique<DevNeg>();
    t->rel = np.rel;
    t->ncols = np.ncols;
    t->col[0] = np.col[0];
    t->col[1] = np.col[1];
    t->n = np.rel->nrows;
    const Relation* q = np.rel;
    const int64_t range = np.ncols == 1 && t->n > 0 ? (int64_t)q->hi[np.col[0]] - q->lo[np.col[0]] + 1 : 0;
    if (range > 0 && range / 8 <= 16 * t->n) {
      // one bit per value of the column (no larger than the sorted keys and
      // their sort's buffer): filtering 1 M rows by 10,000 values, two passes
      // of 29 us searching the keys, 13 by bits, and no sort before
      const int64_t bytes = (range + 31) / 32 * 4;
      XL_TRY(dalloc(c, (size_t)bytes, &t->bits, "negation bits"));
      HIP_TRY(c, k::fill_bytes(t->bits.p, 0, (size_t)bytes, c->stream));
      KeyPack kp{};
      kp.nkey = 1;
      kp.lo[0] = q->lo[np.col[0]];
      HIP_TRY(c, k::bits_set_rows(t->bits.as<uint32_t>(), 1, q->col[np.col[0]], nullptr, t->n, kp, c->stream));
      t->lo = (uint32_t)kp.lo[0];
      t->last = (uint32_t)(range - 1);
    } else if (np.ncols > 0 && t->n > 0) {
      // (rows in canonical order without negative values project to ascending
      // unsigned keys on their leading columns)
      bool ascending = q->sorted;
      for (int j = 0; j < np.ncols; ++j) ascending = ascending && np.col[j] == j && q->lo[j] >= 0;
      XL_TRY(dalloc(c, (size_t)t->n * 8, &t->keys, "negation keys"));
      HIP_TRY(c, k::neg_keys(q->col[np.col[0]], np.ncols > 1 ? q->col[np.col[1]] : nullptr, t->n,
                             t->keys.as<u64>(), c->stream));
      if (!ascending) {
        Buf alt, tmp;
        XL_TRY(dalloc(c, (size_t)t->n * 8, &alt, "negation keys"));
        XL_TRY(dalloc(c, k::radix_temp_bytes(t->n), &tmp, "sort scratch"));
        int alt_used = 0;
        HIP_TRY(c, k::radix_sort_u64(t->keys.as<u64>(), nullptr, alt.as<u64>(), nullptr, t->n,
                                     np.ncols > 1 ? 64 : 32, tmp.p, c->stream, &alt_used));
        if (alt_used) std::swap(t->keys.p, alt.p);
      }
    }
    *out = t->table();
    negtabs.push_back(std::move(t));
    return XL_OK;
  }

  // Fatal flags of a stage launch: 32 is a join key with 2^26 or more rows
  // (the kernel's 32-bit match count per wavefront), anything else internal.
  xl_status stage_fatal(u64 flags, const char* internal) {
    if (flags & 32)
      return c->fail(XL_UNSUPPORTED, "a join key matches 2^26 or more rows of an indexed relation");
    return c->fail(XL_DEVICE_ERROR, internal);
  }

  xl_status counted_pass(StageArgs& a, int64_t* total, Buf* offs) {
    const int64_t nchunks = (a.src.n + 63) / 64;
    Buf cnt, tmp, tot;
    XL_TRY(dalloc(c, (size_t)nchunks * 8, &cnt, "chunk counts"));
    XL_TRY(dalloc(c, (size_t)nchunks * 8, offs, "chunk offsets"));
    XL_TRY(dalloc(c, k::scan_temp_bytes(nchunks), &tmp, "scan scratch"));
    XL_TRY(dalloc(c, 16, &tot, "count"));
    StageArgs ca = a;
    ca.emit.mode = EM_COUNT;
    ca.emit.chunk_cnt = cnt.as<u64>();
    ca.emit.counters = c->dcounters;
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    HIP_TRY(c, k::stage_launch(ca, c->stream, 1 << 16));
    HIP_TRY(c, k::scan_exclusive_u64(cnt.as<u64>(), offs->as<u64>(), nchunks, tot.as<u64>(), tmp.p,
                                     c->stream));
    // the total and the fatal flags in one read
    HIP_TRY(c, hipMemcpyAsync(tot.as<u64>() + 1, c->dcounters + CNT_FATAL, 8, hipMemcpyDeviceToDevice, c->stream));
    u64 t[2] = {0, 0};
    XL_TRY(ctl_read(c, tot.p, 16, t));
    if (t[1]) return stage_fatal(t[1], "stage count pass failed (internal)");
    *total = (int64_t)t[0];
    return XL_OK;
  }

  // Kernel arguments of the closure-shaped variant in frontier form, reading
  // the current delta rows.
  xl_status frontier_args(const RulePlan& p, HeadRun* h, FrontierArgs& f) {
    f.x = h->fx.as<uint32_t>();
    f.in_cnt = h->fcnt[h->fcur].as<uint32_t>();
    f.in_diff = h->fdiff[h->fcur].as<uint32_t>();
    f.nseg = h->fn;
    XL_TRY(get_index(p.steps[0].rel, p.steps[0].key_col, &f.idx, -1, nullptr, 0, true));
    f.ybind_col = p.carried_ycol;
    f.bits = h->bits.as<uint32_t>();
    f.lo0 = h->kp.lo[0];
    f.lo1 = h->kp.lo[1];
    f.row_words = h->row_words;
    f.out_cnt = h->fcnt[h->fcur ^ 1].as<uint32_t>();
    f.out_diff = h->fdiff[h->fcur ^ 1].as<uint32_t>();
    f.pull_ratio = (uint32_t)c->pull_ratio;
    if (c->pull_ratio) {
      XL_TRY(get_index(p.steps[0].rel, p.carried_ycol, &f.rev, p.steps[0].key_col, &f.rev_first, 0, true));
      if (!f.rev_first) return c->fail(XL_DEVICE_ERROR, "pull index without first rows (internal)");
      f.rev_zcol = p.steps[0].key_col;
      if (!h->hasin.p) {
        XL_TRY(dalloc(c, (size_t)h->row_words * 4, &h->hasin, "in-edge bitmap"));
        HIP_TRY(c, k::hasin_bits(f.rev, h->kp.lo[1], h->row_words, h->hasin.as<uint32_t>(), c->stream));
      }
      f.hasin = h->hasin.as<uint32_t>();
    }
    f.counters = c->dcounters;
    return XL_OK;
  }

  // One gathered round: reads the delta rows flagged in gflag[gcur] from
  // (gcur ? gbits : dbits), writes the next delta into the other pair, then
  // clears the rows it read.
  xl_status gather_args(const RulePlan& p, HeadRun* h, GatherArgs& a) {
    GatherShape g;
    if (!gather_shape(p, &g)) return c->fail(XL_DEVICE_ERROR, "gathered round of another rule shape (internal)");
    a.in_bits = (h->gcur ? h->gbits : h->dbits).as<uint32_t>();
    a.out_bits = (h->gcur ? h->dbits : h->gbits).as<uint32_t>();
    a.in_flag = h->gflag[h->gcur].as<uint32_t>();
    a.out_flag = h->gflag[h->gcur ^ 1].as<uint32_t>();
    a.bits = h->bits.as<uint32_t>();
    XL_TRY(get_index(p.steps[g.s1].rel, g.x_col, &a.e1, -1, nullptr, 0, true));
    a.e1_acol = p.steps[g.s1].key_col;
    a.by_a = c->gather_rounds == 1;
    if (a.by_a) {
      XL_TRY(get_index(p.steps[g.s1].rel, a.e1_acol, &a.e1a, -1, nullptr, 0, true));
      a.e1_xcol = g.x_col;
      // Rounds of two launches where the bitmap is larger than 8 MB.  Forests,
      // evaluate and read, us (one launch / two): 500 ids 184 / 239, 1,500
      // (0.3 MB) 232 / 330, 5,000 (3 MB) 354 / 371, 12,000 (18 MB) 601 / 529,
      // 20,000 (50 MB) 960 / 798.
      const bool two = h->range0 * (int64_t)h->row_words * 4 > (8 << 20);
      if (two && !h->ghubs.p) {  // once per run: the rounds all take the same form
        XL_TRY(dalloc(c, 4, &h->ghubs, "gathered round form"));
        HIP_TRY(c, k::gather_hubs(a.e1, h->ghubs.as<uint32_t>(), c->stream));
      }
      a.hubs = two ? h->ghubs.as<uint32_t>() : nullptr;
      a.in_lo = h->gbound[h->gcur].as<uint32_t>();
      a.in_hi = a.in_lo + h->range0;
      a.out_lo = h->gbound[h->gcur ^ 1].as<uint32_t>();
      a.out_hi = a.out_lo + h->range0;
    }
    XL_TRY(get_index(p.steps[g.s2].rel, p.steps[g.s2].key_col, &a.push.idx, -1, nullptr, 0, true));
    a.push.ybind_col = g.y_col;
    a.lo0 = a.push.lo0 = h->kp.lo[0];
    a.lo1 = a.push.lo1 = h->kp.lo[1];
    a.row_words = a.push.row_words = h->row_words;
    a.range0 = h->range0;
    return XL_OK;
  }

  xl_status eval_gathered(const RulePlan& p, HeadRun* h) {
    h->fnew = 0;
    GatherArgs a{};
    XL_TRY(gather_args(p, h, a));
    a.counters = c->dcounters;
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
    HIP_TRY(c, k::gather_round(a, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
    // the consumed delta becomes the next round's output buffer (the by-row
    // kernel empties each delta row it reads itself)
    if (!a.by_a)
      HIP_TRY(c, k::clear_flagged_rows((h->gcur ? h->gbits : h->dbits).as<uint32_t>(),
                                       h->gflag[h->gcur].as<uint32_t>(), h->range0, h->row_words, nullptr, nullptr,
                                       c->stream));
    u64 cnt[CNT_N];
    XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
    cands += (int64_t)cnt[CNT_CANDIDATES];
    if (c->profile) {
      float ms = 0;
      HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
      st->gather_ms += ms;
      st->gather_launches++;
      st->gather_candidates += (int64_t)cnt[CNT_CANDIDATES];
      st->gather_new += (int64_t)cnt[CNT_APPENDED];
    }
    h->fnew = (int64_t)cnt[CNT_APPENDED];
    h->keys += h->fnew;
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // One round of the closure-shaped variant in frontier form.
  xl_status eval_frontier(const RulePlan& p, HeadRun* h) {
    h->fnew = 0;
    if (h->fn == 0) return XL_OK;
    FrontierArgs f{};
    XL_TRY(frontier_args(p, h, f));
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
    HIP_TRY(c, k::frontier_round(f, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
    u64 cnt[CNT_N];
    XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
    cands += (int64_t)cnt[CNT_CANDIDATES];
    if (c->profile) {
      float ms = 0;
      HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
      st->front_ms += ms;
      st->front_launches++;
      st->front_candidates += (int64_t)cnt[CNT_CANDIDATES];
      st->front_new += (int64_t)cnt[CNT_APPENDED];
    }
    h->fnew = (int64_t)cnt[CNT_APPENDED];
    h->keys += h->fnew;
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // Every pass of a frontier stratum in one launch (resident form): each
  // first key runs its own rounds until its delta is empty.  The pass count
  // and per-pass delta sizes match the round-by-round loop, since a key's
  // rounds never read another key's rows: the i-th pass's delta is the union
  // of every key's i-th round.
  bool resident_frontier(const Stratum& s) {
    return heads.size() == 1 && heads[0]->resident && heads[0]->frontier_ready &&
           s.variants.size() == 1 && s.variants[0].driver_delta && head_of(s.variants[0].head) == heads[0].get();
  }

  xl_status run_frontier_resident(const RulePlan& p, HeadRun* h, int64_t max_iterations) {
    if (h->fn == 0) return XL_OK;
    FrontierArgs f{};
    XL_TRY(frontier_args(p, h, f));
    f.x = nullptr;  // delta row sg of first key lo0 + sg is dbits row sg
    f.in_cnt = nullptr;
    f.in_diff = h->dbits.as<uint32_t>();
    f.nseg = h->range0;
    f.out_cnt = f.out_diff = nullptr;
    // one block, one read: the work queue, largest round and cap overflow in
    // a 256-byte block of their own (every workgroup's atomic on the queue
    // word is on the path to its next key, so no other counter shares its
    // cache line), the kernel's counters, then the new tuples of each round
    constexpr size_t HDR = 256, CNTB = 256, BLOCK = HDR + CNTB + 8 * XL_STATS_ROUNDS;
    static_assert(8 * CNT_N <= CNTB, "counters fit their block");
    Buf rs;
    XL_TRY(dalloc(c, BLOCK, &rs, "round counters"));
    HIP_TRY(c, hipMemsetAsync(rs.p, 0, BLOCK, c->stream));
    f.queue = rs.as<uint32_t>();
    f.max_round = rs.as<uint32_t>() + 1;
    f.overflow = rs.as<uint32_t>() + 2;
    f.counters = (unsigned long long*)((char*)rs.p + HDR);
    f.round_new = (unsigned long long*)((char*)rs.p + HDR + CNTB);
    f.round_slots = XL_STATS_ROUNDS;
    f.max_rounds = (uint32_t)std::min<int64_t>(max_iterations, 0xffffffffll);
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
    HIP_TRY(c, k::frontier_resident(f, 0, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
    std::vector<unsigned char> blk(BLOCK);
    XL_TRY(ctl_read(c, rs.p, BLOCK, blk.data()));
    uint32_t hdr[4];
    u64 cnt[CNT_N];
    memcpy(hdr, blk.data(), sizeof(hdr));
    memcpy(cnt, blk.data() + HDR, sizeof(cnt));
    const uint32_t rounds = hdr[1];
    std::vector<u64> per((size_t)XL_STATS_ROUNDS, 0);
    memcpy(per.data(), blk.data() + HDR + CNTB, 8 * (size_t)XL_STATS_ROUNDS);
    cands += (int64_t)cnt[CNT_CANDIDATES];
    if (c->profile) {
      float ms = 0;
      HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
      st->front_ms += ms;
      st->front_launches++;
      st->front_candidates += (int64_t)cnt[CNT_CANDIDATES];
      st->front_new += (int64_t)cnt[CNT_APPENDED];
    }
    // one recorded round per pass (the last counter slot sums the passes from
    // there on, which the receipt does not list anyway)
    for (uint32_t r = 0; r < rounds; ++r) {
      st->iterations++;
      record(r < (uint32_t)XL_STATS_ROUNDS ? (int64_t)per[r] : 0);
    }
    st->new_tuples_total += (int64_t)cnt[CNT_APPENDED];
    h->keys += (int64_t)cnt[CNT_APPENDED];
    h->fn = 0;
    if (hdr[2])
      return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                 " reached before the fixpoint");
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // Turn the row-list delta [dbeg, dend) of a frontier head into delta bitmap
  // rows: sort by the first key, one delta row per distinct value.
  // First frontier: the seed round's new tuples are the delta bitmap; its
  // nonempty rows become the delta rows (no regrouping), then it is cleared.
  xl_status frontier_from_bits(HeadRun* h) {
    h->fn = 0;
    h->frontier_ready = true;
    if (h->round_new == 0) return XL_OK;
    Buf cnt, tmp, tot;
    XL_TRY(dalloc(c, (size_t)h->range0 * 4, &cnt, "row counts"));
    XL_TRY(dalloc(c, k::compact_temp_bytes(h->range0), &tmp, "compaction scratch"));
    XL_TRY(dalloc(c, 8, &tot, "count"));
    HIP_TRY(c, k::row_popcount(h->dbits.as<uint32_t>(), h->range0, h->row_words, cnt.as<uint32_t>(), c->stream));
    KeyPack kx{};
    kx.nkey = 1;
    kx.lo[0] = h->kp.lo[0];
    HIP_TRY(c, k::dcount_rows(cnt.as<uint32_t>(), h->range0, 1, kx, h->fx.as<uint32_t>(), nullptr,
                              h->fcnt[h->fcur].as<uint32_t>(), h->range0, tot.as<uint32_t>(), tmp.p, c->stream));
    uint32_t nseg = 0;
    XL_TRY(ctl_read(c, tot.p, 4, &nseg));
    HIP_TRY(c, k::gather_rows(h->dbits.as<uint32_t>(), h->row_words, h->fx.as<uint32_t>(), h->kp.lo[0], nseg,
                              h->fdiff[h->fcur].as<uint32_t>(), c->stream));
    HIP_TRY(c, k::fill_bytes(h->dbits.p, 0, (size_t)h->range0 * h->row_words * 4, c->stream));
    h->fn = nseg;
    return XL_OK;
  }



  // h(X, count(V)) :- r(..., X, ..., V, ...) with distinct variables, nothing
  // else in the body, over a finished relation that already has an index by
  // X's column: returns that index (the count per X is its degree), else null.
  const DevIndex* degree_index(const RulePlan& p) const {
    if (p.nkey != 1 || !p.steps.empty() || p.driver_delta) return nullptr;
    for (const auto& h : heads)
      if (h->rel == p.driver) return nullptr;
    for (const auto& ops : p.stage_ops)
      if (!ops.empty()) return nullptr;
    int kcol = -1;
    for (int j = 0; j < p.driver->arity; ++j) {
      const ColAct& a = p.driver_act[j];
      if (a.kind != CA_BIND && a.kind != CA_NONE) return nullptr;
      if (a.kind == CA_BIND && a.slot == p.key_slot[0]) {
        if (kcol >= 0) return nullptr;
        kcol = j;
      }
    }
    if (kcol < 0) return nullptr;
    for (const auto& ix : indexes)
      if (ix->rel == p.driver && ix->col == kcol && !ix->probe.keys) return ix.get();
    return nullptr;
  }

  // "value is P1 + W" / "P1 - W" with W bound by one column of e and nothing
  // else to check: returns 1 / 2 and the column, else 0.
  int affine_value(const RulePlan& p, int* col) const {
    const StepPlan& sp = p.steps[0];
    const auto& ops = p.stage_ops[0];
    if (p.cv_slot_p < 0 || ops.size() != 2) return 0;
    const MicroOp& m = ops[0];
    const MicroOp& o = ops[1];
    if (m.kind != OP_MOV || m.dst != p.val_slot || m.a != p.cv_slot_p || m.type != p.val_type) return 0;
    if ((o.kind != OP_ADD && o.kind != OP_SUB) || o.dst != p.val_slot || o.a != p.val_slot || o.b < 0 ||
        o.type != p.val_type)
      return 0;
    int wc = -1;
    for (int j = 0; j < sp.rel->arity; ++j) {
      const ColAct& ac = sp.act[j];
      if (ac.kind == CA_CHECK_SLOT || ac.kind == CA_CHECK_CONST) return 0;
      if (ac.kind == CA_BIND && ac.slot == o.b) wc = j;
    }
    if (wc < 0 || wc == sp.key_col || sp.rel->types[wc] != p.val_type) return 0;
    *col = wc;
    return o.kind == OP_ADD ? 1 : 2;
  }

  // One round of the carried-value variant over a dense sum/logsumexp head:
  // mark every key that receives a contribution (the stage kernel over the
  // delta rows), list the marked slots in order, then fold each key's
  // contributions by scanning e's rows for its Y value against the delta.
  // Arguments of the segmented pull of a carried-value rule over the current
  // delta (list, counts, row outputs and counters are set by the caller).
  xl_status pull_args(const RulePlan& p, HeadRun* h, int fast, int fcol, DensePullArgs& q) {
    const StepPlan& sp = p.steps[0];
    q.dict = h->dict.as<uint32_t>();
    q.range1 = (uint32_t)h->range1;
    q.nrank = (uint32_t)h->nrank_d;
    q.lo1 = h->kp.lo[1];
    XL_TRY(get_index(sp.rel, p.carried_ycol, &q.rev, -1, nullptr, 0, true));
    for (int j = 0; j < sp.rel->arity; ++j) q.rev.act[j] = sp.act[j];
    q.rev.act[p.carried_ycol].kind = CA_NONE;  // Y is bound from the key
    q.zcol = sp.key_col;
    q.slot_s = (int8_t)p.cv_slot_s;
    q.slot_z = (int8_t)p.cv_slot_z;
    q.slot_y = (int8_t)p.key_slot[1];
    q.slot_p = (int8_t)p.cv_slot_p;
    q.val_slot = (int8_t)p.val_slot;
    q.val_type = p.val_type;
    q.fold_kind = h->fold;
    q.fast = (int8_t)fast;
    q.fcol = (int8_t)fcol;
    q.nops = (int32_t)p.stage_ops[0].size();
    for (int i = 0; i < q.nops; ++i) q.ops[i] = p.stage_ops[0][i];
    for (size_t i = 0; i < p.stage_consts[0].size(); ++i) q.consts[i] = p.stage_consts[0][i];
    q.cval = h->dcur.as<uint32_t>();
    q.cpres = h->dcur_pres.as<uint32_t>();
    q.nval = h->dnext.as<uint32_t>();
    q.npres = h->dnext_pres.as<uint32_t>();
    q.fval = h->dvals.as<uint32_t>();
    q.fpres = h->dpres.as<uint32_t>();
    return XL_OK;
  }

  // Batched gathered rounds: each round gets its own counter block, so
  // `batched_rounds` rounds run per host read; rounds past the fixpoint find
  // no flagged delta row and change nothing.
  // ------------------------------------------------------------ batched set rounds
  // A recursive stratum with one set head held in a hash table (row list +
  // open-addressing set), whose delta variants each run in one stage-kernel
  // launch over the head's delta (one index step, or two fused into a
  // product) and join only relations outside the stratum, runs
  // batched_rounds rounds per host read: the head's row list is append-only,
  // so round j's delta is the rows between two boundaries that a one-thread
  // kernel records on the device after each round, and every launch reads
  // its driver range from there.  The batch shares one set of counters and
  // one load limit; a launch that crosses the limit (or refuses a product
  // row) sets the overflow flag, after which the rest of the batch does
  // nothing and the host re-runs that round the ordinary way (growing the
  // table; insert-if-absent keeps the partial round's rows valid).  Passes,
  // per-pass delta sizes and the iteration cap are those of the host loop.
  int batch_j = 0;              // round of the batch being enqueued (1-based; 0: not batching)
  // run by the next stage launch after the launch and before its count read
  std::function<xl_status()> before_count_read;
  int batch_grid = EMIT_GRID;  // workgroups of a batched launch (its waves bound the slack)
  // batched keyed value rounds: the batch's delta rows and slot list (one
  // position space: the first delta at [0, base), each round's slots and rows
  // after it), its capacity past the base, the round's stamp and the
  // accumulators of hashed folds
  uint32_t* batch_rows[3] = {nullptr, nullptr, nullptr};
  int64_t batch_rows_cap = 0;
  uint32_t* batch_idx = nullptr;
  u64 batch_delta_lim = 0;
  uint32_t batch_round = 0;
  u64* batch_acc = nullptr;

  // Batched rounds of set heads held in hash tables (row list + set): every
  // head of the stratum (one, or several in mutual recursion) is a hash set,
  // and each delta variant runs in one stage launch over its driver head's
  // delta and joins only relations outside the stratum.
  bool batched_sets(const Stratum& s) {
    if (c->batched_rounds <= 0 || heads.empty() || heads.size() > (size_t)k::MAX_BATCH_HEADS || s.variants.empty())
      return false;
    for (auto& hp : heads) {
      const HeadRun* h = hp.get();
      if (!h->is_set || h->dense || h->frontier || h->gathered || h->dv) return false;
    }
    for (const RulePlan& p : s.variants) {
      HeadRun* h = head_of(p.head);
      if (!p.driver_delta || !head_of(p.driver) || p.wcoj || !h) return false;
      for (const StepPlan& sp : p.steps)
        if (head_of(sp.rel)) return false;
      if (p.steps.size() > 2) return false;
      if (p.steps.size() == 2) {
        std::vector<MicroOp> pops;
        std::vector<uint32_t> pconsts;
        if (!c->product_joins || !product_plan(p, h, &pops, &pconsts)) return false;
      }
    }
    return true;
  }

  xl_status run_sets_batched(Stratum& s, int64_t max_iterations) {
    const int B = c->batched_rounds;
    const int nh = (int)heads.size();
    constexpr size_t CNTB = 256;
    static_assert(8 * CNT_N <= CNTB, "counters fit their block");
    const size_t per = CNTB + 8 * (size_t)(B + 2);  // one head's counters, then its round boundaries
    Buf blk;
    XL_TRY(dalloc(c, per * nh, &blk, "batch counters"));
    std::vector<unsigned char> host(per * nh);
    auto hcnt = [&](int q) { return (const u64*)(host.data() + per * q); };
    auto hbnd = [&](int q) { return (const u64*)(host.data() + per * q + CNTB); };
    for (int q = 0; q < nh; ++q) {
      heads[q]->b_cnt = (u64*)((char*)blk.p + per * q);
      heads[q]->b_bnd = (u64*)((char*)blk.p + per * q + CNTB);
    }
    auto any_delta = [&]() {
      for (auto& h : heads)
        if (h->dend > h->dbeg) return true;
      return false;
    };
    int64_t pass = 0;
    while (any_delta()) {
      if (pass >= max_iterations)
        return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                   " reached before the fixpoint");
      // every wavefront of a launch that crosses its head's limit may still
      // insert one batch: the grid takes at most a quarter of the smallest
      // table as slack (whatever the round's delta size, unknown here)
      int64_t waves = (int64_t)EMIT_GRID * 4;
      for (auto& h : heads) XL_TRY(widen(h.get(), B));
      for (auto& h : heads) waves = std::min<int64_t>(waves, h->cap / 4 / WAVE_SLACK);
      waves = std::max<int64_t>(256, waves) / 4 * 4;
      batch_grid = (int)(waves / 4);
      bool grown = false;
      for (auto& hp : heads) {
        HeadRun* h = hp.get();
        const int64_t max_keys = std::min<int64_t>(h->cap / 2, h->cap - WAVE_SLACK * waves - 1024);
        if (h->keys >= max_keys) {
          XL_TRY(grow(h, std::max<int64_t>(h->keys * 2, h->keys + WAVE_SLACK * waves + 1024)));
          grown = true;
        }
        h->b_limit = (u64)std::max<int64_t>(0, max_keys - h->keys);
      }
      if (grown) continue;
      const int K = (int)std::min<int64_t>(B, max_iterations - pass);
      HIP_TRY(c, hipMemsetAsync(blk.p, 0, per * nh, c->stream));
      k::BatchMarks marks{};
      marks.n = nh;
      for (int q = 0; q < nh; ++q) {
        HeadRun* h = heads[q].get();
        HIP_TRY(c, k::batch_init(h->b_bnd, B + 2, (u64)h->dbeg, (u64)h->dend, c->stream));
        h->b_base = (u64)h->nrows;
        marks.bnd[q] = h->b_bnd;
        marks.cnt[q] = h->b_cnt;
        marks.base[q] = h->b_base;
      }
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
      for (int j = 1; j <= K; ++j) {
        batch_j = j;
        for (RulePlan& p : s.variants) {
          const xl_status e = eval_plan(p);
          if (e != XL_OK) {
            batch_j = 0;
            return e;
          }
        }
        HIP_TRY(c, k::batch_mark_heads(marks, j, c->stream));
      }
      batch_j = 0;
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
      XL_TRY(ctl_read(c, blk.p, per * nh, host.data()));
      u64 emitted = 0, candidates = 0;
      for (int q = 0; q < nh; ++q) {
        HeadRun* h = heads[q].get();
        const u64* cnt = hcnt(q);
        if (cnt[CNT_FATAL] & ~16ull)
          return stage_fatal(cnt[CNT_FATAL], "hash table probe exhausted or row list overflow (internal)");
        candidates += cnt[CNT_CANDIDATES];
        emitted += cnt[CNT_APPENDED];
        h->nrows = (int64_t)h->b_base + (int64_t)cnt[CNT_APPENDED];
        h->keys += (int64_t)cnt[CNT_APPENDED];
        if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
          return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                                   std::to_string(h->rel->max_rows));
      }
      cands += (int64_t)candidates;
      if (c->profile) {
        float ms = 0;
        HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        st->emit_ms += ms;
        st->emit_launches += (int64_t)K * (int64_t)s.variants.size();
        st->emit_candidates += (int64_t)candidates;
        st->emit_new += (int64_t)emitted;
      }
      // the marks are all or nothing: a round is complete for every head or for none
      int done = 0;
      bool empty = false;
      for (int j = 1; j <= K && hbnd(0)[j + 1] != ~0ull; ++j) {
        ++done;
        ++pass;
        st->iterations++;
        int64_t d = 0;
        for (int q = 0; q < nh; ++q) d += (int64_t)(hbnd(q)[j + 1] - hbnd(q)[j]);
        record(d);
        st->new_tuples_total += d;
        if (d == 0) {
          empty = true;
          break;
        }
      }
      if (empty) {
        for (auto& h : heads) h->dbeg = h->dend = h->nrows;
        break;
      }
      if (done == K) {
        for (int q = 0; q < nh; ++q) {
          HeadRun* h = heads[q].get();
          const double before = (double)(hbnd(q)[K] - hbnd(q)[K - 1]);
          h->dbeg = (int64_t)hbnd(q)[K];
          h->dend = (int64_t)hbnd(q)[K + 1];
          h->growth = before > 0 ? (double)(h->dend - h->dbeg) / before : 1;
        }
        continue;
      }
      // round done + 1 stopped early: re-run it the ordinary way (each head's
      // driver is [b[done], b[done + 1]); the rows its stopped launches
      // appended are the start of its delta, and insert-if-absent keeps them)
      if (pass >= max_iterations)
        return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                   " reached before the fixpoint");
      std::vector<int64_t> rb(nh);
      for (int q = 0; q < nh; ++q) {
        HeadRun* h = heads[q].get();
        rb[q] = (int64_t)hbnd(q)[done + 1];
        h->dbeg = (int64_t)hbnd(q)[done];
        h->dend = rb[q];
        begin_round(h);
      }
      for (RulePlan& p : s.variants) XL_TRY(eval_plan(p));
      ++pass;
      st->iterations++;
      int64_t d = 0;
      for (int q = 0; q < nh; ++q) {
        HeadRun* h = heads[q].get();
        d += h->nrows - rb[q];
        h->dbeg = rb[q];
        h->dend = h->nrows;
      }
      record(d);
      st->new_tuples_total += d;
    }
    return XL_OK;
  }

  // Batched rounds of a min/max or sum/logsumexp head held in a keyed hash
  // table (index mode 1, or key domains too wide for the dense forms): the
  // stratum's delta variants each run in one stage launch and join only
  // relations outside the stratum.  Min/max candidates improve table values
  // (EM_MINMAX); sum/logsumexp candidates fold into one accumulator per slot
  // (EM_HAGG).  Either way the slots a round touches are listed once (round
  // stamps) after the batch's earlier rounds, and a range kernel turns them
  // into the next delta rows at the same positions (for hashed folds it also
  // merges the round into the full relation and resets the accumulators),
  // so every size stays on the device until the batch's one read.
  bool batched_values(const Stratum& s) {
    if (c->batched_rounds <= 0 || heads.size() != 1 || s.variants.empty()) return false;
    HeadRun* h = heads[0].get();
    if (h->is_set || h->dense || h->dv || h->ds || h->tiled || h->frontier || h->gathered || h->dcount) return false;
    const int vt = h->rel->types[h->nkey];
    const bool hashed = h->is_sortagg && (h->fold == k::FOLD_SUM || h->fold == k::FOLD_LSE) &&
                        (vt == T_I32 || vt == T_F32);
    if (!h->is_minmax && !hashed) return false;
    for (const RulePlan& p : s.variants) {
      if (!p.driver_delta || p.driver != h->rel || p.wcoj || head_of(p.head) != h) return false;
      for (const StepPlan& sp : p.steps)
        if (head_of(sp.rel)) return false;
      if (p.steps.size() > 2) return false;
      if (p.steps.size() == 2) {
        std::vector<MicroOp> pops;
        std::vector<uint32_t> pconsts;
        if (!c->product_joins || !product_plan(p, h, &pops, &pconsts)) return false;
      }
    }
    return true;
  }

  // Copy n delta rows (key columns and value) from position `from` of the
  // columns src into the head's delta rows.
  xl_status take_delta_rows(HeadRun* h, uint32_t* const* src, int64_t from, int64_t n) {
    XL_TRY(ensure_drow(h, std::max<int64_t>(n, 1)));
    for (int j = 0; j <= h->nkey && n > 0; ++j)
      HIP_TRY(c, hipMemcpyAsync(h->drow[j].p, src[j] + from, (size_t)n * 4, hipMemcpyDeviceToDevice, c->stream));
    h->dn = n;
    return XL_OK;
  }

  xl_status run_values_batched(Stratum& s, HeadRun* h, int64_t max_iterations) {
    const int B = c->batched_rounds;
    const bool hashed = !h->is_minmax;
    const int vt = h->rel->types[h->nkey];
    constexpr size_t CNTB = 256;
    static_assert(8 * CNT_N <= CNTB, "counters fit their block");
    Buf blk;  // the batch's counters, then the round boundaries
    XL_TRY(dalloc(c, CNTB + 8 * (size_t)(B + 2), &blk, "batch counters"));
    u64* counters = blk.as<u64>();
    u64* bnd = (u64*)((char*)blk.p + CNTB);
    std::vector<unsigned char> host(CNTB + 8 * (size_t)(B + 2));
    Buf acc, bidx, brow[3];
    int64_t acc_cap = 0, bcap = 0;
    int64_t pass = 0;
    while (h->dn > 0) {
      if (pass >= max_iterations)
        return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                   " reached before the fixpoint");
      const int64_t waves =
          std::max<int64_t>(256, std::min<int64_t>((int64_t)EMIT_GRID * 4, h->cap / 4 / WAVE_SLACK)) / 4 * 4;
      batch_grid = (int)(waves / 4);
      const int64_t max_keys = std::min<int64_t>(h->cap / 2, h->cap - WAVE_SLACK * waves - 1024);
      if (h->keys >= max_keys) {
        XL_TRY(grow(h, std::max<int64_t>(h->keys * 2, h->keys + WAVE_SLACK * waves + 1024)));
        continue;
      }
      if (hashed && acc_cap != h->cap) {  // accumulators follow the table's slots (all at identity here)
        acc.reset();
        XL_TRY(dalloc(c, (size_t)h->cap * 8, &acc, "fold accumulators"));
        HIP_TRY(c, k::acc_fill(acc.as<u64>(), h->cap, vt, h->fold, c->stream));
        acc_cap = h->cap;
      }
      // a round touches each key at most once: the table's capacity past the
      // first delta holds a batch of typical rounds; more overflows the batch
      const int64_t need = h->dn + std::max<int64_t>(h->cap, 4096);
      if (bcap < need) {
        bidx.reset();
        XL_TRY(dalloc(c, (size_t)need * 4, &bidx, "batch delta slots"));
        for (int j = 0; j <= h->nkey; ++j) {
          brow[j].reset();
          XL_TRY(dalloc(c, (size_t)need * 4, &brow[j], "batch delta rows"));
        }
        bcap = need;
      }
      uint32_t* rows[3] = {brow[0].as<uint32_t>(), h->nkey == 2 ? brow[1].as<uint32_t>() : nullptr,
                           brow[h->nkey].as<uint32_t>()};
      uint32_t* cols[3] = {brow[0].as<uint32_t>(), brow[1].as<uint32_t>(), brow[2].as<uint32_t>()};
      for (int j = 0; j <= h->nkey; ++j)
        HIP_TRY(c, hipMemcpyAsync(brow[j].p, h->drow[j].p, (size_t)h->dn * 4, hipMemcpyDeviceToDevice, c->stream));
      const int K = (int)std::min<int64_t>(B, max_iterations - pass);
      const int64_t dn0 = h->dn;
      HIP_TRY(c, hipMemsetAsync(counters, 0, CNTB, c->stream));
      HIP_TRY(c, k::batch_init(bnd, B + 2, 0ull, (u64)dn0, c->stream));
      h->b_cnt = counters;
      h->b_bnd = bnd;
      h->b_base = (u64)dn0;
      h->b_limit = (u64)(max_keys - h->keys);
      for (int j = 0; j <= h->nkey; ++j) batch_rows[j] = brow[j].as<uint32_t>();
      batch_rows_cap = bcap;
      batch_idx = bidx.as<uint32_t>();
      batch_delta_lim = (u64)(bcap - dn0);
      batch_acc = hashed ? acc.as<u64>() : nullptr;
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
      for (int j = 1; j <= K; ++j) {
        batch_j = j;
        batch_round = h->round + (uint32_t)j;
        for (RulePlan& p : s.variants) {
          const xl_status e = eval_plan(p);
          if (e != XL_OK) {
            batch_j = 0;
            return e;
          }
        }
        HIP_TRY(c, k::batch_mark(bnd, j, counters, (u64)dn0, c->stream));
        HIP_TRY(c, k::table16_rows_range(h->table.as<Slot16>(), batch_acc, bidx.as<uint32_t>(), bnd, j, bcap,
                                         h->kp, vt, h->fold, rows[0], rows[1], rows[2], c->stream));
      }
      batch_j = 0;
      batch_acc = nullptr;
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
      XL_TRY(ctl_read(c, blk.p, CNTB + 8 * (size_t)(K + 2), host.data()));
      u64 cnt[CNT_N];
      memcpy(cnt, host.data(), sizeof(cnt));
      const u64* b = (const u64*)(host.data() + CNTB);
      if (cnt[CNT_FATAL] & ~16ull) return stage_fatal(cnt[CNT_FATAL], "hash table probe exhausted (internal)");
      cands += (int64_t)cnt[CNT_CANDIDATES];
      if (c->profile) {
        float ms = 0;
        HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        st->emit_ms += ms;
        st->emit_launches += (int64_t)K * (int64_t)s.variants.size();
        st->emit_candidates += (int64_t)cnt[CNT_CANDIDATES];
        st->emit_new += (int64_t)cnt[CNT_INSERTED];
      }
      h->keys += (int64_t)cnt[CNT_INSERTED];
      if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
        return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                                 std::to_string(h->rel->max_rows));
      int done = 0;
      bool empty = false;
      for (int j = 1; j <= K && b[j + 1] != ~0ull; ++j) {
        ++done;
        ++pass;
        st->iterations++;
        const int64_t d = (int64_t)(b[j + 1] - b[j]);
        record(d);
        st->new_tuples_total += d;
        if (d == 0) {
          empty = true;
          break;
        }
      }
      h->round += (uint32_t)done;
      if (empty) {
        h->dn = 0;
        break;
      }
      if (done == K) {  // the last round's rows are the next delta
        XL_TRY(take_delta_rows(h, cols, (int64_t)b[K], (int64_t)(b[K + 1] - b[K])));
        continue;
      }
      // Round done + 1 stopped early (table load limit, slot list capacity
      // or a refused product row): re-run it the ordinary way from its driver
      // rows [b[done], b[done + 1]).
      if (pass >= max_iterations)
        return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                   " reached before the fixpoint");
      XL_TRY(take_delta_rows(h, cols, (int64_t)b[done], (int64_t)(b[done + 1] - b[done])));
      const uint32_t rid = h->round + 1;  // the stopped round's stamp
      if (hashed) {
        // its contributions so far are dropped (the run below folds them all
        // again, under a new stamp, by the sorted path); keys it inserted
        // hold the identity until that run's merge
        HIP_TRY(c, k::acc_fill(acc.as<u64>(), acc_cap, vt, h->fold, c->stream));
        h->round = rid;
        begin_round(h);
      } else {
        // its improvements stay in the table: list the slots it stamped and
        // let the run below add the rest
        h->round = rid - 1;
        begin_round(h);
        Buf tmp, tot;
        XL_TRY(dalloc(c, k::compact_temp_bytes(h->cap), &tmp, "compaction scratch"));
        XL_TRY(dalloc(c, 8, &tot, "count"));
        HIP_TRY(c, k::table16_stamped(h->table.as<Slot16>(), h->cap, h->round, h->didx.as<uint32_t>(), h->cap,
                                      tot.as<uint32_t>(), tmp.p, c->stream));
        uint32_t n2 = 0;
        XL_TRY(ctl_read(c, tot.p, 4, &n2));
        h->didx_n = (int64_t)n2;
      }
      for (RulePlan& p : s.variants) XL_TRY(eval_plan(p));
      ++pass;
      st->iterations++;
      int64_t d = 0;
      XL_TRY(finish_round(h, &d));
      record(d);
      st->new_tuples_total += d;
    }
    return XL_OK;
  }

  bool batched_gather(const Stratum& s) {
    return c->batched_rounds > 0 && heads.size() == 1 && heads[0]->gathered && heads[0]->gather_ready &&
           s.variants.size() == 1 && s.variants[0].driver_delta && head_of(s.variants[0].head) == heads[0].get();
  }

  bool batched_selfjoin() const { return heads.size() == 1 && heads[0]->sj_on; }

  // The rounds of a self-joined closure after the first `pass`, batched_rounds
  // per host read.  A round (and its merge) enqueued past the fixpoint sees
  // that the round before it added nothing and returns.
  xl_status run_selfjoin_batched(HeadRun* h, int64_t pass, int64_t max_iterations) {
    const int B = c->batched_rounds;
    Buf acc;
    XL_TRY(dalloc(c, (size_t)B * 8 * CNT_N, &acc, "round counters"));
    HIP_TRY(c, k::row_popcount(h->bits.as<uint32_t>(), h->range0, h->row_words, h->scnt.as<uint32_t>(), c->stream));
    HIP_TRY(c, k::row_popcount(h->dbits.as<uint32_t>(), h->range0, h->row_words, h->dcnt[0].as<uint32_t>(),
                               c->stream));
    int cur = 0;
    int64_t delta = 1;
    while (delta > 0) {
      if (pass >= max_iterations)
        return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                   " reached before the fixpoint");
      const int nb = (int)std::min<int64_t>(B, max_iterations - pass);
      HIP_TRY(c, hipMemsetAsync(acc.p, 0, (size_t)nb * 8 * CNT_N, c->stream));
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
      for (int r = 0; r < nb; ++r) {
        SelfJoinArgs a{};
        a.full = h->bits.as<uint32_t>();
        a.delta = (cur ? h->gbits : h->dbits).as<uint32_t>();
        a.next = (cur ? h->dbits : h->gbits).as<uint32_t>();
        a.full_cnt = h->scnt.as<uint32_t>();
        a.delta_cnt = h->dcnt[cur].as<uint32_t>();
        a.next_cnt = h->dcnt[cur ^ 1].as<uint32_t>();
        a.range0 = h->range0;
        a.zoff = (int64_t)h->kp.lo[1] - h->kp.lo[0];
        a.row_words = h->row_words;
        a.counters = acc.as<unsigned long long>() + (size_t)r * CNT_N;
        a.prev = r ? a.counters - CNT_N + CNT_APPENDED : nullptr;
        HIP_TRY(c, k::self_join_round(a, c->stream));
        HIP_TRY(c, k::self_join_merge(h->bits.as<uint32_t>(), a.next, h->range0 * (int64_t)h->row_words,
                                      h->scnt.as<uint32_t>(), a.next_cnt, a.prev, h->range0, c->stream));
        cur ^= 1;
      }
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
      std::vector<u64> cnt((size_t)nb * CNT_N);
      XL_TRY(ctl_read(c, acc.p, (size_t)nb * 8 * CNT_N, cnt.data()));
      if (c->profile) {
        float ms = 0;
        HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        st->emit_ms += ms;
      }
      for (int r = 0; r < nb && delta > 0; ++r) {
        const u64* cr = cnt.data() + (size_t)r * CNT_N;
        if (c->profile) {
          st->emit_launches++;
          st->emit_candidates += (int64_t)cr[CNT_CANDIDATES];
          st->emit_new += (int64_t)cr[CNT_APPENDED];
        }
        delta = (int64_t)cr[CNT_APPENDED];
        st->iterations++;
        record(delta);
        st->new_tuples_total += delta;
        cands += (int64_t)cr[CNT_CANDIDATES];
        h->keys += delta;
        ++pass;
        if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
          return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                                   std::to_string(h->rel->max_rows));
      }
    }
    return XL_OK;
  }

  xl_status run_gather_batched(const RulePlan& p, HeadRun* h, int64_t max_iterations) {
    const int B = c->batched_rounds;
    Buf acc;
    XL_TRY(dalloc(c, (size_t)B * 8 * CNT_N, &acc, "round counters"));
    std::vector<hipEvent_t> evs;
    if (c->profile) {
      evs.resize(2 * (size_t)B, nullptr);
      for (auto& e : evs) HIP_TRY(c, hipEventCreate(&e));
    }
    auto destroy_events = [&]() {
      for (auto& e : evs)
        if (e) (void)hipEventDestroy(e);
      evs.clear();
    };
    int64_t pass = 0, delta = 1;
    xl_status status = XL_OK;
    while (delta > 0 && status == XL_OK) {
      if (pass >= max_iterations) {
        status = c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                     " reached before the fixpoint");
        break;
      }
      const int nb = (int)std::min<int64_t>(B, max_iterations - pass);
      HIP_TRY(c, hipMemsetAsync(acc.p, 0, (size_t)nb * 8 * CNT_N, c->stream));
      for (int r = 0; r < nb; ++r) {
        GatherArgs a{};
        XL_TRY(gather_args(p, h, a));
        a.counters = acc.as<unsigned long long>() + (size_t)r * CNT_N;
        if (c->profile) HIP_TRY(c, hipEventRecord(evs[2 * r], c->stream));
        HIP_TRY(c, k::gather_round(a, c->stream));
        if (c->profile) HIP_TRY(c, hipEventRecord(evs[2 * r + 1], c->stream));
        if (!a.by_a)  // the by-row kernel empties each delta row it reads itself
          HIP_TRY(c, k::clear_flagged_rows((h->gcur ? h->gbits : h->dbits).as<uint32_t>(),
                                           h->gflag[h->gcur].as<uint32_t>(), h->range0, h->row_words, nullptr,
                                           nullptr, c->stream));
        h->gcur ^= 1;
      }
      std::vector<u64> cnt((size_t)nb * CNT_N);  // at most 64 blocks of 64 B: one control read
      XL_TRY(ctl_read(c, acc.p, (size_t)nb * 8 * CNT_N, cnt.data()));
      int done = nb;
      for (int r = 0; r < nb; ++r)
        if (cnt[(size_t)r * CNT_N + CNT_APPENDED] == 0) {
          done = r + 1;
          break;
        }
      for (int r = 0; r < done; ++r) {
        const u64* cr = cnt.data() + (size_t)r * CNT_N;
        st->iterations++;
        record((int64_t)cr[CNT_APPENDED]);
        st->new_tuples_total += (int64_t)cr[CNT_APPENDED];
        cands += (int64_t)cr[CNT_CANDIDATES];
        h->keys += (int64_t)cr[CNT_APPENDED];
        if (c->profile) {
          float ms = 0;
          HIP_TRY(c, hipEventElapsedTime(&ms, evs[2 * r], evs[2 * r + 1]));
          st->gather_ms += ms;
          st->gather_launches++;
          st->gather_candidates += (int64_t)cr[CNT_CANDIDATES];
          st->gather_new += (int64_t)cr[CNT_APPENDED];
        }
      }
      pass += done;
      delta = (int64_t)cnt[(size_t)(done - 1) * CNT_N + CNT_APPENDED];
    }
    destroy_events();
    if (status != XL_OK) return status;
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // Batched pull rounds: a sum/logsumexp stratum whose one carried-value rule
  // adds or subtracts a column of e (every key with an in-edge from a delta
  // key gets a value, so the marks need no join) enqueues `batched_rounds`
  // rounds per host read.  Each round marks, then pulls straight from the mark
  // words, writes no delta rows, and leaves its delta size in its counters;
  // rounds enqueued past the fixpoint find no marks and change nothing.
  bool batched_pull(const Stratum& s) {
    if (c->batched_rounds <= 0 || heads.size() != 1 || !heads[0]->ds || s.variants.size() != 1 ||
        !s.variants[0].driver_delta || head_of(s.variants[0].head) != heads[0].get())
      return false;
    int fcol = 0;
    return affine_value(s.variants[0], &fcol) != 0;
  }

  xl_status run_pull_batched(const RulePlan& p, HeadRun* h, int64_t max_iterations) {
    const StepPlan& sp = p.steps[0];
    int fcol = 0;
    const int fast = affine_value(p, &fcol);
    const int64_t nsd = h->nrank_d * h->range1;
    IndexProbe fwd{};
    XL_TRY(get_index(sp.rel, sp.key_col, &fwd, -1, nullptr, 0, true));
    const int B = c->batched_rounds;
    Buf acc, longs;
    XL_TRY(dalloc(c, (size_t)B * 8 * CNT_N, &acc, "round counters"));
    std::vector<hipEvent_t> evs;
    if (c->profile) {
      evs.resize(2 * (size_t)B, nullptr);
      for (auto& e : evs) HIP_TRY(c, hipEventCreate(&e));
    }
    auto destroy_events = [&]() {
      for (auto& e : evs)
        if (e) (void)hipEventDestroy(e);
      evs.clear();
    };
    int64_t pass = 0, delta = h->dn;
    u64 fatal = 0;
    xl_status status = XL_OK;
    while (delta > 0 && status == XL_OK) {
      if (pass >= max_iterations) {
        status = c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                     " reached before the fixpoint");
        break;
      }
      const int nb = (int)std::min<int64_t>(B, max_iterations - pass);
      HIP_TRY(c, hipMemsetAsync(acc.p, 0, (size_t)nb * 8 * CNT_N, c->stream));
      for (int r = 0; r < nb; ++r) {
        // the mark pass also clears the presence bits this round's pull
        // writes (the round before last's, no longer read)
        HIP_TRY(c, k::dense_mark_out(fwd, p.carried_ycol, h->kp.lo[1], (uint32_t)h->range1, (uint32_t)h->nrank_d,
                                     h->dcur_pres.as<uint32_t>(), h->dchg.as<uint32_t>(),
                                     h->dnext_pres.as<uint32_t>(), c->stream));
        DensePullArgs q{};
        XL_TRY(pull_args(p, h, fast, fcol, q));
        q.mark = h->dchg.as<uint32_t>();
        q.n = nsd;
        if (!longs.p) {  // once per run: the rounds pull over the same index
          XL_TRY(dalloc(c, 4, &longs, "rows in long lists"));
          HIP_TRY(c, k::long_rows(q.rev, longs.as<uint32_t>(), c->stream));
        }
        q.long_rows = longs.as<uint32_t>();
        q.long_min = (uint32_t)(sp.rel->nrows / 4);
        q.counters = acc.as<unsigned long long>() + (size_t)r * CNT_N;
        if (c->profile) HIP_TRY(c, hipEventRecord(evs[2 * r], c->stream));
        HIP_TRY(c, k::dense_pull_marks(q, c->stream));
        if (c->profile) HIP_TRY(c, hipEventRecord(evs[2 * r + 1], c->stream));
        std::swap(h->dcur.p, h->dnext.p);
        std::swap(h->dcur_pres.p, h->dnext_pres.p);
      }
      std::vector<u64> cnt((size_t)nb * CNT_N);
      XL_TRY(ctl_read(c, acc.p, (size_t)nb * 8 * CNT_N, cnt.data()));
      for (int r = 0; r < nb && delta > 0; ++r) {
        const u64* cr = cnt.data() + (size_t)r * CNT_N;
        delta = (int64_t)cr[CNT_APPENDED];
        fatal |= cr[CNT_FATAL];
        st->iterations++;
        record(delta);
        st->new_tuples_total += delta;
        cands += (int64_t)cr[CNT_CANDIDATES];
        h->keys += (int64_t)cr[CNT_INSERTED];
        if (c->profile) {
          float ms = 0;
          HIP_TRY(c, hipEventElapsedTime(&ms, evs[2 * r], evs[2 * r + 1]));
          st->pull_ms += ms;
          st->pull_launches++;
          st->pull_new += delta;
          st->pull_candidates += (int64_t)cr[CNT_CANDIDATES];
        }
        ++pass;
      }
    }
    destroy_events();
    // the next presence bits are clear between rounds everywhere else
    HIP_TRY(c, k::fill_bytes(h->dnext_pres.p, 0, (size_t)(nsd / 32) * 4, c->stream));
    if (fatal) return c->fail(XL_DEVICE_ERROR, "marked key without a contribution (internal)");
    h->dn = 0;
    if (status != XL_OK) return status;
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  xl_status eval_dense_pull(const RulePlan& p, HeadRun* h) {
    h->pulled = true;
    h->pull_n = 0;
    Source src = resolve_driver(p);
    if (src.n == 0) return XL_OK;
    const StepPlan& sp = p.steps[0];
    StageArgs a{};
    a.src.n = src.n;
    a.src.ncols = p.driver->arity;
    for (int j = 0; j < a.src.ncols; ++j) {
      a.src.col[j] = src.col[j];
      a.src.act[j] = p.driver_act[j];
    }
    a.has_index = 1;
    XL_TRY(get_index(sp.rel, sp.key_col, &a.idx));
    a.idx.key_slot = (int8_t)sp.key_slot;
    for (int j = 0; j < sp.rel->arity; ++j) a.idx.act[j] = sp.act[j];
    XL_TRY(fill_ops(a, p, 0));
    int fcol = 0;
    const int fast = affine_value(p, &fcol);
    const int64_t nsd = h->nrank_d * h->range1;
    if (fast) {
      // every key with an in-edge from a delta key receives a value, so the
      // marks are the delta presence rows pushed to the out-neighbours (the
      // mark bits are clear: the previous list pass cleared what it listed)
      IndexProbe fwd{};
      XL_TRY(get_index(sp.rel, sp.key_col, &fwd, -1, nullptr, 0, true));
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
      HIP_TRY(c, k::dense_mark_out(fwd, p.carried_ycol, h->kp.lo[1], (uint32_t)h->range1, (uint32_t)h->nrank_d,
                                   h->dcur_pres.as<uint32_t>(), h->dchg.as<uint32_t>(), nullptr, c->stream));
      if (c->profile) {
        HIP_TRY(c, hipEventRecord(ev[1], c->stream));
        HIP_TRY(c, hipEventSynchronize(ev[1]));
        float ms = 0;
        HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        st->emit_ms += ms;
        st->emit_launches++;
        st->emit_source_rows += src.n;
      }
    }
    a.emit.mode = EM_MARK;
    a.emit.key.nkey = 2;
    a.emit.key.slot[0] = (int8_t)p.key_slot[0];
    a.emit.key.slot[1] = (int8_t)p.key_slot[1];
    a.emit.key.lo[0] = h->kp.lo[0];
    a.emit.key.lo[1] = h->kp.lo[1];
    a.emit.val_slot = (int8_t)p.val_slot;
    a.emit.dmap = h->dmap.as<uint32_t>();
    a.emit.dmap_n = (uint32_t)h->dmap_n;
    a.emit.row_bits = (u64)h->range1;
    a.emit.nrank = (uint32_t)h->nrank_d;
    a.emit.dchg = h->dchg.as<uint32_t>();
    a.emit.counters = c->dcounters;
    u64 cnt[CNT_N];
    if (!fast) {
      HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
      HIP_TRY(c, k::stage_launch(a, c->stream, EMIT_GRID));
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
      XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
      if (cnt[CNT_FATAL]) return stage_fatal(cnt[CNT_FATAL], "key outside the dense domain (internal)");
      if (c->profile) {
        float ms = 0;
        HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        st->emit_ms += ms;
        st->emit_launches++;
        st->emit_source_rows += src.n;
        st->emit_candidates += (int64_t)cnt[CNT_CANDIDATES];
      }
      cands += (int64_t)cnt[CNT_CANDIDATES];
    }
    const int64_t ns = nsd;
    Buf tmp, tot, list;
    XL_TRY(dalloc(c, k::bits_list_temp_bytes(ns), &tmp, "compaction scratch"));
    XL_TRY(dalloc(c, 8, &tot, "count"));
    HIP_TRY(c, k::bits_list(h->dchg.as<uint32_t>(), ns, nullptr, tot.as<uint32_t>(), tmp.p, false, c->stream));
    uint32_t n = 0;
    XL_TRY(ctl_read(c, tot.p, 4, &n));
    if (n == 0) return XL_OK;
    XL_TRY(dalloc(c, (size_t)n * 4, &list, "marked keys"));
    HIP_TRY(c, k::bits_list(h->dchg.as<uint32_t>(), ns, list.as<uint32_t>(), tot.as<uint32_t>(), tmp.p, true,
                            c->stream));
    for (int j = 0; j < 3; ++j) XL_TRY(dalloc(c, (size_t)n * 4, &h->ndrow[j], "delta rows"));
    DensePullArgs q{};
    XL_TRY(pull_args(p, h, fast, fcol, q));
    q.list = list.as<uint32_t>();
    q.n = n;
    q.k0 = h->ndrow[0].as<uint32_t>();
    q.k1 = h->ndrow[1].as<uint32_t>();
    q.v = h->ndrow[2].as<uint32_t>();
    q.counters = c->dcounters;
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
    HIP_TRY(c, k::dense_pull(q, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
    XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
    if (cnt[CNT_FATAL]) return c->fail(XL_DEVICE_ERROR, "marked key without a contribution (internal)");
    if (c->profile) {
      float ms = 0;
      HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
      st->pull_ms += ms;
      st->pull_launches++;
      st->pull_candidates += (int64_t)cnt[CNT_CANDIDATES];
      st->pull_new += (int64_t)n;
    }
    if (fast) cands += (int64_t)cnt[CNT_CANDIDATES];  // no mark pass: count the in-edges the fold examined
    h->keys += (int64_t)cnt[CNT_INSERTED];
    h->pull_n = n;
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // Tile layout (as many slots as fit 128 KB of LDS, or fewer so that every
  // CU gets a workgroup; a multiple of 32 slots) and e's rows sorted by
  // (tile of Y, Z) with offsets per (tile, Z): a tile's workgroup reads only
  // the rows that land in it, and one tile's rows of consecutive Z are
  // consecutive.
  xl_status build_tile_index(const RulePlan& p, HeadRun* h) {
    const StepPlan& sp = p.steps[0];
    Relation* e = sp.rel;
    const uint32_t max_tile = 32768;
    uint32_t nt = (uint32_t)((h->range1 + max_tile - 1) / max_tile);
    if (c->dense_tiles > 0) nt = (uint32_t)c->dense_tiles;
    else nt = std::max<uint32_t>(nt, (uint32_t)((256 + h->n0 - 1) / std::max<int64_t>(h->n0, 1)));
    uint32_t tile = (uint32_t)(((h->range1 + nt - 1) / nt + 31) / 32 * 32);
    tile = std::min<uint32_t>(std::max<uint32_t>(tile, 32), max_tile);
    h->tile = tile;
    h->ntiles = (uint32_t)((h->range1 + tile - 1) / tile);
    const int64_t n = e->nrows;
    IndexProbe& q = h->tidx;
    q = IndexProbe{};
    q.ncols = e->arity;
    const int zc = sp.key_col;
    const int64_t zr = n ? (int64_t)e->hi[zc] - e->lo[zc] + 1 : 0;
    const int64_t nkeys = zr * (h->ntiles + 1);
    if (nkeys >= ((int64_t)1 << 31)) return c->fail(XL_UNSUPPORTED, "tiled index key range too large");
    q.key_lo = n ? e->lo[zc] : 0;
    q.key_range = (uint32_t)zr;
    XL_TRY(dalloc(c, (size_t)(nkeys + 1) * 4, &h->toff, "tiled index offsets"));
    if (n == 0) {
      HIP_TRY(c, hipMemsetAsync(h->toff.p, 0, 4, c->stream));
      return XL_OK;
    }
    if (n > ((int64_t)1 << 30)) return c->fail(XL_UNSUPPORTED, "relation " + e->name + " too large to tile");
    // A loaded relation with Z in its first column and Y in its second is in
    // (Z, Y) order, so a stable sort by the tile of Y alone puts it in
    // (tile, Z) order when every Y lies in the head's domain; otherwise the
    // rows are sorted by the whole (tile, Z) key.
    const bool presorted = !head_of(e) && e->sorted && zc == 0 && p.carried_ycol == 1 && e->types[1] == T_I32 &&
                           (int64_t)e->lo[1] >= h->kp.lo[1] && (int64_t)e->hi[1] - h->kp.lo[1] < h->range1;
    Buf keys, keys2, perm, perm2, tmp;
    XL_TRY(dalloc(c, (size_t)n * 4, &keys, "index keys"));
    XL_TRY(dalloc(c, (size_t)n * 4, &keys2, "index keys"));
    XL_TRY(dalloc(c, (size_t)n * 4, &perm, "index permutation"));
    XL_TRY(dalloc(c, (size_t)n * 4, &perm2, "index permutation"));
    XL_TRY(dalloc(c, k::radix_temp_bytes(n), &tmp, "sort scratch"));
    HIP_TRY(c, k::tile_keys(e->col[zc], e->col[p.carried_ycol], n, e->lo[zc], h->kp.lo[1], h->tile, h->ntiles,
                            (uint32_t)zr, presorted, keys.as<uint32_t>(), c->stream));
    HIP_TRY(c, k::iota_u32(perm.as<uint32_t>(), n, c->stream));
    int alt = 0;
    const int key_bits = presorted ? bitlen((uint64_t)h->ntiles) : bitlen((uint64_t)nkeys - 1);
    HIP_TRY(c, k::radix_sort_u32(keys.as<uint32_t>(), perm.as<uint32_t>(), keys2.as<uint32_t>(), perm2.as<uint32_t>(),
                                 n, std::max(1, key_bits), tmp.p, c->stream, &alt));
    uint32_t* sk = alt ? keys2.as<uint32_t>() : keys.as<uint32_t>();
    uint32_t* spm = alt ? perm2.as<uint32_t>() : perm.as<uint32_t>();
    int fcol = 0;
    if (affine_value(p, &fcol)) {
      h->tcols.push_back(std::make_unique<Buf>());
      XL_TRY(dalloc(c, (size_t)n * 8, h->tcols.back().get(), "tiled index pairs"));
      HIP_TRY(c, k::tile_pairs(spm, e->col[zc], e->col[p.carried_ycol], e->col[fcol], n, e->lo[zc], h->kp.lo[1],
                               h->tile, h->ntiles, (uint32_t)zr, h->tcols.back()->p, presorted ? sk : nullptr,
                               c->stream));
    } else {
      uint32_t* tc[MAXC] = {};
      for (int j = 0; j < e->arity; ++j) {
        h->tcols.push_back(std::make_unique<Buf>());
        XL_TRY(dalloc(c, (size_t)n * 4, h->tcols.back().get(), "tiled index column"));
        tc[j] = h->tcols.back()->as<uint32_t>();
        q.col[j] = tc[j];
      }
      HIP_TRY(c, k::gather_cols(e->col, tc, e->arity, spm, n, c->stream));
      if (presorted)  // the whole keys of the rows in their new order
        HIP_TRY(c, k::tile_keys(q.col[zc], q.col[p.carried_ycol], n, e->lo[zc], h->kp.lo[1], h->tile, h->ntiles,
                                (uint32_t)zr, false, sk, c->stream));
    }
    HIP_TRY(c, k::csr_offsets(sk, n, (uint32_t)nkeys, h->toff.as<uint32_t>(), c->stream));
    return XL_OK;
  }

  // One round of the carried-value variant over a dense min/max head: one
  // workgroup per (rank, tile of second-key slots) with the tile in LDS.
  xl_status eval_dense_tiles(const RulePlan& p, HeadRun* h) {
    if (h->dn == 0) return XL_OK;
    DenseTileArgs a{};
    XL_TRY(tile_args(p, h, a));
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
    HIP_TRY(c, k::dense_min_tiles(a, c->stream));
    if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
    u64 cnt[CNT_N];
    XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
    if (c->profile) {
      float ms = 0;
      HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
      st->emit_ms += ms;
      st->emit_launches++;
      st->emit_source_rows += h->dn;
      st->emit_candidates += (int64_t)cnt[CNT_CANDIDATES];
      st->emit_new += (int64_t)cnt[CNT_APPENDED];
    }
    cands += (int64_t)cnt[CNT_CANDIDATES];
    h->keys += (int64_t)cnt[CNT_INSERTED];
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // Delta rows of a tiled head from its delta bits, grouped by rank (count
  // and write passes; the write pass also fills roff); the row total goes to
  // *total on the device.  With tcnt (the round's per-tile counts) one
  // launch that sums the counts itself replaces both passes.
  xl_status tile_delta_rows(HeadRun* h, uint32_t* total, Buf* ltmp, const uint32_t* tcnt) {
    if (tcnt) {
      HIP_TRY(c, k::tile_delta_rows(h->dchg.as<uint32_t>(), tcnt, (uint32_t)h->n0, h->ntiles, h->tile,
                                    (uint32_t)h->range1, h->dvals.as<uint32_t>(), h->dict.as<uint32_t>(), h->kp.lo[1],
                                    h->rel->types[h->nkey], h->fold, h->drow[0].as<uint32_t>(),
                                    h->drow[1].as<uint32_t>(), h->drow[2].as<uint32_t>(), h->roff.as<uint32_t>(),
                                    total, c->stream));
      return XL_OK;
    }
    const int64_t ns = std::max<int64_t>(h->n0, 1) * h->range1;
    for (bool write : {false, true})
      HIP_TRY(c, k::dense_delta_from_bits(h->dchg.as<uint32_t>(), ns, (uint32_t)h->range1, h->dvals.as<uint32_t>(),
                                          h->dict.as<uint32_t>(), h->kp.lo[1], h->rel->types[h->nkey], h->fold,
                                          h->drow[0].as<uint32_t>(), h->drow[1].as<uint32_t>(),
                                          h->drow[2].as<uint32_t>(), h->n0 > 0 ? h->roff.as<uint32_t>() : nullptr,
                                          total, ltmp->p, write, c->stream));
    return XL_OK;
  }

  // Tiled min/max stratum, rounds enqueued in batches (option
  // "batched_rounds"): every kernel of a round takes its sizes from device
  // memory (the rank offsets of the delta rows, the delta bits), the delta
  // row buffers hold any delta (one row per slot), and each round's delta
  // size goes to a device array that the host reads once per batch.  Rounds
  // enqueued past the fixpoint find an empty delta and change nothing, so
  // the pass count and per-pass sizes are the round-by-round ones.
  bool batched_tiles(const Stratum& s) {
    if (c->batched_rounds <= 0 || heads.size() != 1 || !heads[0]->tiled || s.variants.size() != 1 ||
        !s.variants[0].driver_delta || head_of(s.variants[0].head) != heads[0].get())
      return false;
    HeadRun* h = heads[0].get();
    const int64_t ns = std::max<int64_t>(h->n0, 1) * h->range1;
    return (double)ns * 12 <= (double)c->arena.largest_free() / 2;  // delta rows for every slot
  }

  xl_status run_tiles_batched(const RulePlan& p, HeadRun* h, int64_t max_iterations) {
    const int64_t ns = std::max<int64_t>(h->n0, 1) * h->range1;
    if (h->dcap < ns) {  // room for a delta row per slot, keeping the seed's rows
      Buf nd[3];
      for (int j = 0; j < 3; ++j) {
        XL_TRY(dalloc(c, (size_t)ns * 4, &nd[j], "delta rows"));
        if (h->dn)
          HIP_TRY(c, hipMemcpyAsync(nd[j].p, h->drow[j].p, (size_t)h->dn * 4, hipMemcpyDeviceToDevice, c->stream));
      }
      for (int j = 0; j < 3; ++j) {
        std::swap(h->drow[j].p, nd[j].p);
        h->drow[j].c = c;
      }
      h->dcap = ns;
    }
    DenseTileArgs a{};
    XL_TRY(tile_args(p, h, a));
    const int B = c->batched_rounds;
    Buf acc, rounds, ltmp, tcnt;
    XL_TRY(dalloc(c, 8 * CNT_N, &acc, "round counters"));
    XL_TRY(dalloc(c, (size_t)B * 4, &rounds, "round delta sizes"));
    XL_TRY(dalloc(c, k::bits_list_temp_bytes(ns), &ltmp, "compaction scratch"));
    // one-launch delta rows from per-tile counts when the tiles are few
    // enough for each listing workgroup to sum the counts before its tile
    const uint64_t nwork = (uint64_t)h->n0 * h->ntiles;
    if (h->n0 > 0 && nwork <= k::TL_MAX_WORK && h->tile <= k::TL_MAX_TILE && h->range1 % 32 == 0) {
      XL_TRY(dalloc(c, (size_t)nwork * 4, &tcnt, "tile delta counts"));
      a.tcnt = tcnt.as<uint32_t>();
    }
    HIP_TRY(c, hipMemsetAsync(acc.p, 0, 8 * CNT_N, c->stream));
    a.counters = acc.as<unsigned long long>();
    std::vector<hipEvent_t> evs;
    if (c->profile) {
      evs.resize(2 * (size_t)B, nullptr);
      for (auto& e : evs) HIP_TRY(c, hipEventCreate(&e));
    }
    auto destroy_events = [&]() {
      for (auto& e : evs)
        if (e) (void)hipEventDestroy(e);
      evs.clear();
    };
    int64_t pass = 0, delta = h->dn;
    xl_status status = XL_OK;
    while (delta > 0 && status == XL_OK) {
      if (pass >= max_iterations) {
        status = c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                     " reached before the fixpoint");
        break;
      }
      const int nb = (int)std::min<int64_t>(B, max_iterations - pass);
      for (int r = 0; r < nb; ++r) {
        if (c->profile) HIP_TRY(c, hipEventRecord(evs[2 * r], c->stream));
        HIP_TRY(c, k::dense_min_tiles(a, c->stream));
        if (c->profile) HIP_TRY(c, hipEventRecord(evs[2 * r + 1], c->stream));
        XL_TRY(tile_delta_rows(h, rounds.as<uint32_t>() + r, &ltmp, a.tcnt));
      }
      std::vector<uint32_t> n(nb);
      XL_TRY(ctl_read(c, rounds.p, (size_t)nb * 4, n.data()));
      int done = nb;
      for (int r = 0; r < nb; ++r)
        if (n[r] == 0) {
          done = r + 1;
          break;
        }
      for (int r = 0; r < done; ++r) {
        st->iterations++;
        record(n[r]);
        st->new_tuples_total += n[r];
        if (c->profile) {
          float ms = 0;
          HIP_TRY(c, hipEventElapsedTime(&ms, evs[2 * r], evs[2 * r + 1]));
          st->emit_ms += ms;
          st->emit_launches++;
          st->emit_source_rows += r == 0 ? delta : n[r - 1];
        }
      }
      pass += done;
      delta = n[done - 1];
    }
    destroy_events();
    u64 tot[CNT_N];
    XL_TRY(ctl_read(c, acc.p, sizeof(tot), tot));
    cands += (int64_t)tot[CNT_CANDIDATES];
    if (c->profile) {
      st->emit_candidates += (int64_t)tot[CNT_CANDIDATES];
      st->emit_new += (int64_t)tot[CNT_APPENDED];
    }
    h->keys += (int64_t)tot[CNT_INSERTED];
    h->dn = 0;
    if (status != XL_OK) return status;
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                               std::to_string(h->rel->max_rows));
    return XL_OK;
  }

  // Arguments of the tiled min/max round kernel for the current delta rows.
  xl_status tile_args(const RulePlan& p, HeadRun* h, DenseTileArgs& a) {
    const StepPlan& sp = p.steps[0];
    a.dk1 = h->drow[1].as<uint32_t>();
    a.dval = h->drow[2].as<uint32_t>();
    a.roff = h->roff.as<uint32_t>();
    a.dict = h->dict.as<uint32_t>();
    a.n0 = (uint32_t)h->n0;
    a.range1 = (uint32_t)h->range1;
    a.lo1 = h->kp.lo[1];
    if (!h->toff.p) XL_TRY(build_tile_index(p, h));
    a.tile = h->tile;
    a.ntiles = h->ntiles;
    a.idx = h->tidx;
    a.toff = h->toff.as<uint32_t>();
    for (int j = 0; j < sp.rel->arity; ++j) a.idx.act[j] = sp.act[j];
    a.ycol = p.carried_ycol;
    a.slot_s = (int8_t)p.cv_slot_s;
    a.slot_z = (int8_t)p.cv_slot_z;
    a.slot_p = (int8_t)p.cv_slot_p;
    a.slot_y = (int8_t)p.key_slot[1];
    a.val_slot = (int8_t)p.val_slot;
    a.val_type = p.val_type;
    a.is_max = h->agg == Agg::MAX;
    int fcol = 0;
    a.fast = (int8_t)affine_value(p, &fcol);
    a.fcol = (int8_t)fcol;
    if (a.fast && !h->tcols.empty()) a.pairs = (const uint2*)h->tcols[0]->p;
    if (a.fast && h->tcols.empty()) a.pairs = (const uint2*)h->toff.p;  // no rows: never read
    a.nops = (int32_t)p.stage_ops[0].size();
    for (int i = 0; i < a.nops; ++i) a.ops[i] = p.stage_ops[0][i];
    for (size_t i = 0; i < p.stage_consts[0].size(); ++i) a.consts[i] = p.stage_consts[0][i];
    a.vals = h->dvals.as<uint32_t>();
    a.pres = h->dpres.as<uint32_t>();
    a.chg = h->dchg.as<uint32_t>();
    a.counters = c->dcounters;
    return XL_OK;
  }

  // Two index steps whose keys the driver row binds both (e.g. the children
  // of both members of a same-generation pair): one launch walks the product
  // of the two match lists, with both stages' micro-ops, instead of
  // materializing the first step's bindings.  Set heads only: a row whose
  // product is too long is refused by the kernel and the rule then runs
  // again with the two steps apart, which insert-if-absent makes harmless.
  bool product_plan(const RulePlan& p, const HeadRun* h, std::vector<MicroOp>* ops, std::vector<uint32_t>* consts) {
    if (p.steps.size() != 2 || !h->is_set || h->frontier) return false;
    const int k2 = p.steps[1].key_slot;
    bool by_driver = false;
    for (int j = 0; j < p.driver->arity; ++j)
      by_driver = by_driver || (p.driver_act[j].kind == CA_BIND && p.driver_act[j].slot == k2);
    if (!by_driver) return false;
    *ops = p.stage_ops[0];
    *consts = p.stage_consts[0];
    const int shift = (int)p.stage_consts[0].size();
    for (MicroOp op : p.stage_ops[1]) {
      if (op.a < 0) op.a = (int8_t)(op.a - shift);
      if (op.b < 0) op.b = (int8_t)(op.b - shift);
      ops->push_back(op);
    }
    for (uint32_t v : p.stage_consts[1]) consts->push_back(v);
    return ops->size() <= (size_t)MAXOPS && consts->size() <= (size_t)MAXK;
  }

  xl_status eval_plan(const RulePlan& p, bool allow_product = true) {
    HeadRun* h = head_of(p.head);
    if (h->frontier && p.driver_delta) return eval_frontier(p, h);
    if (h->gathered && p.driver_delta) return eval_gathered(p, h);
    if (h->ds && p.driver_delta) return eval_dense_pull(p, h);
    if (h->tiled && p.driver_delta) return eval_dense_tiles(p, h);
    const int nst = (int)p.steps.size();
    const int nkst = nst > 0 ? nst : 1;
    Source src = resolve_driver(p);
    HeadRun* hd = batch_j && p.driver_delta ? head_of(p.driver) : nullptr;
    if (hd) {  // batched rounds: the delta range is on the device
      if (hd->is_set) {
        for (int j = 0; j < hd->nkey; ++j) src.col[j] = hd->rows[j].as<uint32_t>();
        src.n = hd->rows_cap;  // bounds the grid only
      } else {
        for (int j = 0; j <= h->nkey; ++j) src.col[j] = batch_rows[j];
        src.n = batch_rows_cap;
      }
    }
    if (src.n == 0) return XL_OK;
    std::vector<MicroOp> pops;
    std::vector<uint32_t> pconsts;
    const bool product = allow_product && c->product_joins && product_plan(p, h, &pops, &pconsts);
    bool refused = false;
    // materialized bindings between stages
    std::vector<std::unique_ptr<Buf>> live_bufs;
    RowSource rs{};
    rs.n = src.n;
    rs.ncols = p.driver->arity;
    for (int j = 0; j < rs.ncols; ++j) {
      rs.col[j] = src.col[j];
      rs.act[j] = p.driver_act[j];
    }
    for (int ks = 0; ks < nkst; ++ks) {
      StageArgs a{};
      a.src = rs;
      a.has_index = nst > 0;
      if (nst > 0) {
        const StepPlan& sp = p.steps[ks];
        XL_TRY(get_index(sp.rel, sp.key_col, &a.idx));
        a.idx.key_slot = (int8_t)sp.key_slot;
        for (int j = 0; j < sp.rel->arity; ++j) a.idx.act[j] = sp.act[j];
      }
      XL_TRY(fill_ops(a, p, ks));
      if (product) {
        const StepPlan& s2 = p.steps[1];
        a.has_idx2 = 1;
        XL_TRY(get_index(s2.rel, s2.key_col, &a.idx2));
        a.idx2.key_slot = (int8_t)s2.key_slot;
        for (int j = 0; j < s2.rel->arity; ++j) a.idx2.act[j] = s2.act[j];
        a.nops = (int)pops.size();
        for (int i = 0; i < a.nops; ++i) a.ops[i] = pops[i];
        for (size_t i = 0; i < pconsts.size(); ++i) a.consts[i] = pconsts[i];
      }
      a.emit.counters = c->dcounters;
      if (!product && ks + 1 < nkst) {
        // intermediate: count -> scan -> materialize the live slots
        const std::vector<int>& live = p.live_after[ks];
        a.emit.mode = EM_MAT;
        a.emit.nout = (int)live.size();
        int64_t total = 0;
        Buf offs;
        XL_TRY(counted_pass(a, &total, &offs));
        RowSource next{};
        next.n = total;
        next.ncols = (int)live.size();
        for (size_t q = 0; q < live.size(); ++q) {
          live_bufs.push_back(std::make_unique<Buf>());
          XL_TRY(dalloc(c, (size_t)std::max<int64_t>(total, 1) * 4, live_bufs.back().get(), "join bindings"));
          a.emit.out_slot[q] = (int8_t)live[q];
          a.emit.out_col[q] = live_bufs.back()->as<uint32_t>();
          next.col[q] = a.emit.out_col[q];
          next.act[q].kind = CA_BIND;
          next.act[q].slot = (int8_t)live[q];
        }
        a.emit.chunk_off = offs.as<u64>();
        a.emit.mat_base = 0;
        if (total > 0) HIP_TRY(c, k::stage_launch(a, c->stream, 1 << 16));
        rs = next;
        if (total == 0) return XL_OK;
        continue;
      }
      // final stage: emit into the head
      a.emit.key.nkey = p.nkey;
      a.emit.key.slot[0] = (int8_t)p.key_slot[0];
      a.emit.key.slot[1] = (int8_t)(p.nkey == 2 ? p.key_slot[1] : p.key_slot[0]);
      a.emit.key.lo[0] = h->kp.lo[0];
      a.emit.key.lo[1] = h->kp.lo[1];
      a.emit.key.shift = h->kp.shift;
      a.emit.val_slot = (int8_t)p.val_slot;
      a.emit.val_type = p.val_type;
      if (hd) {
        // batched rounds: the driver's delta range, the target's append base,
        // load limit and counters belong to the batch; nothing is read back
        a.src_range = hd->b_bnd + (batch_j - 1);
        a.emit.counters = h->b_cnt;
        a.emit.limit = h->b_limit;
        a.emit.mask = (u64)h->cap - 1;
        if (h->is_set) {
          a.emit.mode = EM_SET;
          a.emit.table = h->table.as<u64>();
          a.emit.row_col[0] = h->rows[0].as<uint32_t>();
          a.emit.row_col[1] = h->nkey == 2 ? h->rows[1].as<uint32_t>() : h->rows[0].as<uint32_t>();
          a.emit.row_base = h->b_base;
          a.emit.row_cap = h->rows_cap;
        } else {
          a.emit.mode = h->is_minmax ? EM_MINMAX : EM_HAGG;
          a.emit.table16 = h->table.as<Slot16>();
          a.emit.is_max = h->agg == Agg::MAX;
          a.emit.round = batch_round;
          a.emit.delta_idx = batch_idx + h->b_base;
          a.emit.delta_lim = batch_delta_lim;
          a.emit.acc = batch_acc;
          a.emit.fold_kind = h->fold;
          a.emit.agg_identity = h->fold == k::FOLD_LSE ? 0xff800000u : 0u;  // -inf, or zero
        }
        HIP_TRY(c, k::stage_launch(a, c->stream, batch_grid));
        if (product) break;  // the one launch covered both steps
        continue;
      }
      if (h->dcount) {
        const DevIndex* dx = degree_index(p);
        if (dx) {  // the group's count is the index degree of its key
          HIP_TRY(c, k::index_degree_add(dx->probe.off, dx->probe.key_range, dx->probe.key_lo, h->kp.lo[0],
                                         (uint32_t)h->range0, h->counts.as<uint32_t>(), c->dcheck, c->stream));
          cands += src.n;
          return XL_OK;
        }
        a.emit.mode = EM_DCOUNT;
        a.emit.bits = h->counts.as<uint32_t>();
        a.emit.row_bits = (u64)h->range1;
        HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
        HIP_TRY(c, k::stage_launch(a, c->stream, 1 << 16));
        u64 cnt[CNT_N];
        XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
        if (cnt[CNT_FATAL]) return stage_fatal(cnt[CNT_FATAL], "count key outside the head domain (internal)");
        cands += (int64_t)cnt[CNT_CANDIDATES];
        return XL_OK;
      }
      if (h->is_sortagg || h->sorted_set) {
        const bool lead = keys_lead(p);
        a.emit.mode = EM_MAT;
        a.emit.mat_packed = 1;
        int64_t total = 0;
        Buf offs;
        XL_TRY(counted_pass(a, &total, &offs));
        cands += total;
        if (total == 0) return XL_OK;
        h->in_order = h->cn == 0 && lead;
        const size_t kb = key_bytes(h);
        if (h->cn + total > h->ccap) {
          const int64_t ncap = std::max<int64_t>(h->cn + total, h->ccap * 2);
          Buf nk, nv;
          XL_TRY(dalloc(c, (size_t)ncap * kb, &nk, "aggregate candidates"));
          if (!h->sorted_set) XL_TRY(dalloc(c, (size_t)ncap * 4, &nv, "aggregate candidates"));
          if (h->cn) {
            HIP_TRY(c, hipMemcpyAsync(nk.p, h->ckey.p, (size_t)h->cn * kb, hipMemcpyDeviceToDevice, c->stream));
            if (!h->sorted_set)
              HIP_TRY(c, hipMemcpyAsync(nv.p, h->cval.p, (size_t)h->cn * 4, hipMemcpyDeviceToDevice, c->stream));
          }
          std::swap(h->ckey.p, nk.p);
          std::swap(h->cval.p, nv.p);
          h->ckey.c = h->cval.c = c;
          h->ccap = ncap;
        }
        a.emit.out_key = h->ckey.as<u64>();
        a.emit.key32 = kb == 4;
        a.emit.out_val = h->cval.as<uint32_t>();
        a.emit.chunk_off = offs.as<u64>();
        a.emit.mat_base = h->cn;
        HIP_TRY(c, k::stage_launch(a, c->stream, 1 << 16));
        h->cn += total;
        return XL_OK;
      }
      // set / min / max: single pass with insert-or-improve, retried after growth
      for (int attempt = 0;; ++attempt) {
        if (attempt > 8) return c->fail(XL_DEVICE_ERROR, "hash table growth did not converge");
        if (nst == 0 || ks == 0) {  // the driver may live in this head's row list
          Source s2 = resolve_driver(p);
          for (int j = 0; j < a.src.ncols && ks == 0; ++j) a.src.col[j] = s2.col[j];
        }
        // Every wavefront may insert one more batch of 64 keys after the load
        // limit is crossed, so the limit leaves room for all of them: the
        // table can never fill and the row list never overflows.
        const int64_t waves = std::min<int64_t>((a.src.n + 63) / 64, (int64_t)EMIT_GRID * 4);
        if (h->dv) {  // every slot exists up front: nothing can overflow
          HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
          a.emit.limit = ~0ull;
          a.emit.mode = EM_DMIN;
          a.emit.bits = h->dvals.as<uint32_t>();
          a.emit.row_bits = (u64)h->range1;
          a.emit.dmap = h->dmap.as<uint32_t>();
          a.emit.dmap_n = (uint32_t)h->dmap_n;
          a.emit.dpres = h->dpres.as<uint32_t>();
          a.emit.dchg = h->dchg.as<uint32_t>();
          a.emit.is_max = h->agg == Agg::MAX;
          a.emit.delta_idx = h->lean ? nullptr : h->didx.as<uint32_t>() + h->didx_n;
        } else if (h->dense) {  // bitmap and delta bitmap cover the whole domain
          HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
          a.emit.limit = ~0ull;
          a.emit.mode = EM_BITSET;
          a.emit.bits = h->bits.as<uint32_t>();
          a.emit.row_bits = h->row_bits;
          a.emit.dchg = h->dbits.as<uint32_t>();
        } else {
        const int64_t max_keys = std::min<int64_t>(h->cap / 2, h->cap - WAVE_SLACK * waves - 1024);
        if (h->keys >= max_keys) {
          XL_TRY(grow(h, std::max<int64_t>(h->keys * 2, h->keys + WAVE_SLACK * waves + 1024)));
          continue;
        }
        HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
        a.emit.limit = (u64)(max_keys - h->keys);
        a.emit.mask = (u64)h->cap - 1;
        }
        if (h->dense || h->dv) {
          // EM_BITSET / EM_DMIN configured above
        } else if (h->is_set) {
          a.emit.mode = EM_SET;
          a.emit.table = h->table.as<u64>();
          a.emit.row_col[0] = h->rows[0].as<uint32_t>();
          a.emit.row_col[1] = h->nkey == 2 ? h->rows[1].as<uint32_t>() : h->rows[0].as<uint32_t>();
          a.emit.row_base = h->nrows;
          a.emit.row_cap = h->rows_cap;
        } else {
          a.emit.mode = EM_MINMAX;
          a.emit.table16 = h->table.as<Slot16>();
          a.emit.is_max = h->agg == Agg::MAX;
          a.emit.round = h->round;
          a.emit.delta_idx = h->didx.as<uint32_t>() + h->didx_n;
        }
        if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
        HIP_TRY(c, k::stage_launch(a, c->stream, EMIT_GRID));
        if (c->profile) HIP_TRY(c, hipEventRecord(ev[1], c->stream));
        if (before_count_read) {  // work that does not need this launch's counts, enqueued before waiting for them
          const auto f = std::move(before_count_read);
          before_count_read = nullptr;
          XL_TRY(f());
        }
        u64 cnt[CNT_N];
        XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
        if (c->profile) {
          float ms = 0;
          HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
          st->emit_ms += ms;
          st->emit_launches++;
          st->emit_source_rows += a.src.n;
          st->emit_candidates += (int64_t)cnt[CNT_CANDIDATES];
          st->emit_new += (int64_t)(h->is_set ? cnt[CNT_APPENDED] : cnt[CNT_INSERTED] + cnt[CNT_APPENDED]);
        }
        if (product && cnt[CNT_FATAL] == 16) {
          refused = true;  // some product rows were skipped: the rule runs again unfused below
        } else if (cnt[CNT_FATAL]) {
          return stage_fatal(cnt[CNT_FATAL], h->dv ? "key outside the dense domain (internal)"
                                                   : "hash table probe exhausted or row list overflow (internal)");
        }
        cands += (int64_t)cnt[CNT_CANDIDATES];
        if (h->dense) {
          h->keys += (int64_t)cnt[CNT_APPENDED];
          h->round_new += (int64_t)cnt[CNT_APPENDED];
        } else if (h->is_set) {
          h->nrows += (int64_t)cnt[CNT_APPENDED];
          h->keys += (int64_t)cnt[CNT_APPENDED];
        } else {
          h->keys += (int64_t)cnt[CNT_INSERTED];
          h->didx_n += (int64_t)cnt[CNT_APPENDED];
        }
        if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
          return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows " +
                                                   std::to_string(h->rel->max_rows));
        if (!cnt[CNT_OVERFLOW]) break;
        XL_TRY(grow(h, h->keys * 2 + 1));  // (lists this round's min/max slots again)
      }
      if (product) break;  // the one launch covered both steps
    }
    if (refused) return eval_plan(p, false);
    return XL_OK;
  }

  // Candidate keys of sorted aggregation are 32-bit when the packed key fits.
  size_t key_bytes(const HeadRun* h) const {
    const int kbits = h->nkey == 2 ? h->bits0 + h->kp.shift : h->bits0;
    return kbits <= 32 ? 4 : 8;
  }

  xl_status ensure_drow(HeadRun* h, int64_t n) {
    if (n <= h->dcap) return XL_OK;
    const int64_t ncap = std::max<int64_t>(n, h->dcap * 2);
    for (int j = 0; j <= h->nkey; ++j) XL_TRY(dalloc(c, (size_t)ncap * 4, &h->drow[j], "delta rows"));
    h->dcap = ncap;
    return XL_OK;
  }

  void begin_round(HeadRun* h) {
    h->round++;
    h->round_new = 0;
    h->round_begin = h->nrows;
    h->didx_n = 0;
    h->cn = 0;
    h->in_order = false;
  }

  xl_status finish_round(HeadRun* h, int64_t* delta) {
    if (h->frontier && h->frontier_ready) {  // a frontier round produced the new delta rows
      h->fcur ^= 1;
      *delta = h->fnew;
      return XL_OK;
    }
    if (h->gathered && h->gather_ready) {  // a gathered round wrote the next delta rows
      h->gcur ^= 1;
      *delta = h->fnew;
      return XL_OK;
    }
    if (h->sorted_set) {  // its rows are made at materialization
      *delta = 0;
      return XL_OK;
    }
    if (h->once && (h->dense || h->is_minmax)) {  // no round follows
      *delta = h->dense ? h->round_new : h->didx_n;
      return XL_OK;
    }
    if (h->dense) {
      *delta = h->round_new;
      // A listed pair reads a whole row (4 * row_words bytes), the generic
      // join one candidate per set bit of it, so rows wider than 128 words
      // wait until the average row has a bit per four words.  Chains of 100
      // nodes, evaluate and read: 4,000 nodes (125 words) 1.48 ms ORing from
      // the seed on, 2.13 by the generic join; 8,000 nodes (250 words, up to
      // a bit per five words) 2.76 against 2.42; 16,384 nodes 5.67 against
      // 3.41.
      if (h->selfjoin && (h->row_words <= 128 || 4.0 * (double)h->keys >= (double)h->range0 * h->row_words)) {
        h->sj_on = true;  // this round's new tuples in dbits are the delta as they are
        return XL_OK;
      }
      if (h->gathered) {  // seed round: its new tuples in dbits are the first delta rows
        h->gather_ready = true;
        h->gcur = 0;
        if (h->round_new) {
          uint32_t* lo = h->gbound[0].as<uint32_t>();
          HIP_TRY(c, k::row_bounds(h->dbits.as<uint32_t>(), h->range0, h->row_words, h->gflag[0].as<uint32_t>(), lo,
                                   lo + h->range0, c->stream));
        }
        return XL_OK;
      }
      if (h->resident) {  // the resident launch reads the seed's delta rows from dbits
        h->frontier_ready = true;
        h->fn = h->round_new ? h->range0 : 0;
        return XL_OK;
      }
      if (h->frontier) return frontier_from_bits(h);  // seed round -> first frontier
      // this round's new tuples, in key order, become the delta rows
      const int64_t nbits = (int64_t)(h->nkey == 2 ? (u64)h->range0 * h->row_bits : (u64)((h->range0 + 31) / 32) * 32);
      Buf tmp, tot;
      XL_TRY(dalloc(c, k::bits_list_temp_bytes(nbits), &tmp, "compaction scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      auto keys = [&](bool write) {
        return k::bits_keys(h->dbits.as<uint32_t>(), nbits, h->row_bits, h->kp.lo[0], h->kp.lo[1], h->nkey, true,
                            h->drow[0].as<uint32_t>(), h->nkey == 2 ? h->drow[1].as<uint32_t>() : nullptr,
                            tot.as<uint32_t>(), tmp.p, write, c->stream);
      };
      HIP_TRY(c, keys(false));
      uint32_t n = 0;
      XL_TRY(ctl_read(c, tot.p, 4, &n));
      if ((int64_t)n != h->round_new) return c->fail(XL_DEVICE_ERROR, "delta bitmap count mismatch (internal)");
      XL_TRY(ensure_drow(h, n));
      if (n) HIP_TRY(c, keys(true));
      h->dn = n;
      return XL_OK;
    }
    if (h->is_set) {
      h->dbeg = h->round_begin;
      h->dend = h->nrows;
      *delta = h->dend - h->dbeg;
      return XL_OK;
    }
    if (h->dcount) {
      *delta = 0;
      return XL_OK;  // counted in place; rows are produced at materialization
    }
    if (h->ds && h->pulled) {  // the pull wrote the next delta rows and values
      h->pulled = false;
      for (int j = 0; j < 3; ++j) {
        std::swap(h->drow[j].p, h->ndrow[j].p);
        h->drow[j].c = c;
        h->ndrow[j].reset();
      }
      h->dcap = h->pull_n;
      h->dn = h->pull_n;
      std::swap(h->dcur.p, h->dnext.p);
      std::swap(h->dcur_pres.p, h->dnext_pres.p);
      HIP_TRY(c, k::fill_bytes(h->dnext_pres.p, 0, (size_t)(h->nrank_d * h->range1 / 32) * 4, c->stream));
      *delta = h->dn;
      return XL_OK;
    }
    if (h->tiled) {  // delta rows from the delta bits, grouped by rank (the write pass fills roff)
      const int64_t ns = std::max<int64_t>(h->n0, 1) * h->range1;
      Buf ltmp, tot;
      XL_TRY(dalloc(c, k::bits_list_temp_bytes(ns), &ltmp, "compaction scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      auto rows = [&](bool write) {
        return k::dense_delta_from_bits(h->dchg.as<uint32_t>(), ns, (uint32_t)h->range1, h->dvals.as<uint32_t>(),
                                   h->dict.as<uint32_t>(), h->kp.lo[1], h->rel->types[h->nkey], h->fold,
                                   h->drow[0].as<uint32_t>(), h->drow[1].as<uint32_t>(), h->drow[2].as<uint32_t>(),
                                   h->n0 > 0 ? h->roff.as<uint32_t>() : nullptr, tot.as<uint32_t>(), ltmp.p, write,
                                   c->stream);
      };
      HIP_TRY(c, rows(false));
      uint32_t n = 0;
      XL_TRY(ctl_read(c, tot.p, 4, &n));
      XL_TRY(ensure_drow(h, n));
      if (n) HIP_TRY(c, rows(true));
      h->dn = n;
      *delta = n;
      return XL_OK;
    }
    if (h->dv && !h->ds) {
      XL_TRY(ensure_drow(h, h->didx_n));
      HIP_TRY(c, k::dense_delta_rows(h->didx.as<uint32_t>(), h->didx_n, h->dvals.as<uint32_t>(),
                                     h->dchg.as<uint32_t>(), h->dict.as<uint32_t>(), (uint32_t)h->range1,
                                     h->kp.lo[1], h->rel->types[h->nkey], h->fold, h->drow[0].as<uint32_t>(),
                                     h->nkey == 2 ? h->drow[1].as<uint32_t>() : nullptr,
                                     h->drow[h->nkey].as<uint32_t>(), c->stream));
      h->dn = h->didx_n;
      *delta = h->dn;
      return XL_OK;
    }
    if (h->is_minmax) {
      XL_TRY(ensure_drow(h, h->didx_n));
      HIP_TRY(c, k::table16_rows_from_idx(h->table.as<Slot16>(), h->didx.as<uint32_t>(), h->didx_n,
                                          h->kp, h->rel->types[h->nkey], h->fold, h->drow[0].as<uint32_t>(),
                                          h->nkey == 2 ? h->drow[1].as<uint32_t>() : nullptr,
                                          h->drow[h->nkey].as<uint32_t>(), c->stream));
      h->dn = h->didx_n;
      *delta = h->dn;
      return XL_OK;
    }
    // sorted aggregation of this round's candidates
    const int64_t n = h->cn;
    if (n == 0) {
      h->dn = 0;
      *delta = 0;
      return XL_OK;
    }
    const int kbits = h->nkey == 2 ? h->bits0 + h->kp.shift : h->bits0;
    const int kb = (int)key_bytes(h);
    Buf k2, v2, tmp, flag, pos, tot;
    int alt = 0;
    if (!h->in_order) {
      XL_TRY(dalloc(c, (size_t)n * kb, &k2, "sort keys"));
      XL_TRY(dalloc(c, (size_t)n * 4, &v2, "sort values"));
      XL_TRY(dalloc(c, k::radix_temp_bytes(n), &tmp, "sort scratch"));
      if (kb == 4)
        HIP_TRY(c, k::radix_sort_u32(h->ckey.as<uint32_t>(), h->cval.as<uint32_t>(), k2.as<uint32_t>(),
                                     v2.as<uint32_t>(), n, kbits, tmp.p, c->stream, &alt));
      else
        HIP_TRY(c, k::radix_sort_u64(h->ckey.as<u64>(), h->cval.as<uint32_t>(), k2.as<u64>(), v2.as<uint32_t>(),
                                     n, kbits, tmp.p, c->stream, &alt));
    }
    void* sk = alt ? k2.p : h->ckey.p;
    uint32_t* sv = alt ? v2.as<uint32_t>() : h->cval.as<uint32_t>();
    XL_TRY(dalloc(c, (size_t)n * 4, &flag, "segment flags"));
    XL_TRY(dalloc(c, (size_t)n * 4, &pos, "segment ids"));
    XL_TRY(dalloc(c, 8, &tot, "count"));
    tmp.reset();
    XL_TRY(dalloc(c, k::scan_temp_bytes(n), &tmp, "scan scratch"));
    HIP_TRY(c, k::seg_heads(sk, kb, n, flag.as<uint32_t>(), c->stream));
    HIP_TRY(c, k::scan_exclusive_u32(flag.as<uint32_t>(), pos.as<uint32_t>(), n, tot.as<uint32_t>(), tmp.p,
                                     c->stream));
    uint32_t nseg = 0;
    XL_TRY(ctl_read(c, tot.p, 4, &nseg));
    Buf starts;
    XL_TRY(dalloc(c, (size_t)nseg * 4, &starts, "segment starts"));
    HIP_TRY(c, k::seg_starts(flag.as<uint32_t>(), pos.as<uint32_t>(), n, starts.as<uint32_t>(), c->stream));
    XL_TRY(ensure_drow(h, nseg));
    HIP_TRY(c, k::seg_reduce(sk, kb, sv, starts.as<uint32_t>(), nseg, n, h->kp, h->rel->types[h->nkey], h->fold,
                             h->drow[0].as<uint32_t>(), h->nkey == 2 ? h->drow[1].as<uint32_t>() : nullptr,
                             h->drow[h->nkey].as<uint32_t>(), c->stream));
    if (h->ds) {  // seed round of a dense head: the folded rows become the first delta
      HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
      HIP_TRY(c, k::dense_apply_rows(h->drow[0].as<uint32_t>(), h->drow[1].as<uint32_t>(), h->drow[2].as<uint32_t>(),
                                     nseg, h->dmap.as<uint32_t>(), (uint32_t)h->dmap_n, (uint32_t)h->range1,
                                     (uint32_t)h->nrank_d, h->kp,
                                     h->fold, h->rel->types[h->nkey], h->dcur.as<uint32_t>(),
                                     h->dcur_pres.as<uint32_t>(), h->dvals.as<uint32_t>(), h->dpres.as<uint32_t>(),
                                     c->dcounters, c->stream));
      u64 cnt[CNT_N];
      XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
      if (cnt[CNT_FATAL]) return c->fail(XL_DEVICE_ERROR, "key outside the dense domain (internal)");
      h->keys += (int64_t)cnt[CNT_INSERTED];
      if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
        return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows");
      h->dn = nseg;
      h->cn = 0;
      *delta = nseg;
      return XL_OK;
    }
    if (h->once) {  // nothing to merge with: the folded rows are the relation
      h->keys = nseg;
      if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
        return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows");
      h->dn = nseg;
      h->cn = 0;
      *delta = nseg;
      return XL_OK;
    }
    if (h->keys + (int64_t)nseg > h->cap / 2) XL_TRY(grow(h, h->keys + nseg));
    HIP_TRY(c, hipMemsetAsync(c->dcounters, 0, 8 * CNT_N, c->stream));
    HIP_TRY(c, k::agg_merge(h->table.as<Slot16>(), (u64)h->cap - 1, h->drow[0].as<uint32_t>(),
                            h->nkey == 2 ? h->drow[1].as<uint32_t>() : nullptr, h->drow[h->nkey].as<uint32_t>(),
                            nseg, h->kp, h->rel->types[h->nkey], h->fold, c->dcounters, c->stream));
    u64 cnt[CNT_N];
    XL_TRY(ctl_read(c, c->dcounters, sizeof(cnt), cnt));
    if (cnt[CNT_FATAL]) return c->fail(XL_DEVICE_ERROR, "hash table probe exhausted (internal)");
    h->keys += (int64_t)cnt[CNT_INSERTED];
    if (h->rel->max_rows > 0 && h->keys > h->rel->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->rel->name + " exceeds its max_rows");
    h->dn = nseg;
    h->cn = 0;
    *delta = nseg;
    return XL_OK;
  }

  // Key-column bounds come from the planner's domains (a superset is enough
  // for packing and index ranges); i32 value columns are scanned.
  xl_status set_bounds(HeadRun* h) {
    Relation* r = h->rel;
    if (r->nrows == 0) return XL_OK;
    for (int j = 0; j < h->nkey; ++j) {
      r->lo[j] = (int32_t)h->dom_lo[j];
      r->hi[j] = (int32_t)h->dom_hi[j];
    }
    if (h->nkey < r->arity && r->types[h->nkey] == T_I32 && !h->vbounds) {
      uint32_t lo, hi;
      XL_TRY(image_bounds(c, &r->col[h->nkey], &r->types[h->nkey], 1, r->nrows, &lo, &hi));
      r->lo[h->nkey] = image_i32(lo);
      r->hi[h->nkey] = image_i32(hi);
    }
    return XL_OK;
  }

  xl_status materialize(HeadRun* h) {
    XL_TRY(materialize_rows(h));
    return set_bounds(h);
  }

  xl_status materialize_rows(HeadRun* h) {
    Relation* r = h->rel;
    if (h->dense && h->nkey == 1) {  // one bitmap row: the set bits in order
      const int64_t nbits = (h->range0 + 31) / 32 * 32;
      Buf tmp, tot, out;
      XL_TRY(dalloc(c, k::bits_list_temp_bytes(nbits), &tmp, "compaction scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      XL_TRY(dalloc(c, (size_t)std::max<int64_t>(h->keys, 1) * 4, &out, "relation column"));
      HIP_TRY(c, k::bits_keys(h->bits.as<uint32_t>(), nbits, 1, h->kp.lo[0], 0, 1, false, out.as<uint32_t>(), nullptr,
                              tot.as<uint32_t>(), tmp.p, false, c->stream));
      uint32_t n = 0;
      XL_TRY(ctl_read(c, tot.p, 4, &n));
      if ((int64_t)n != h->keys) return c->fail(XL_DEVICE_ERROR, "bitmap key count mismatch (internal)");
      HIP_TRY(c, k::bits_keys(h->bits.as<uint32_t>(), nbits, 1, h->kp.lo[0], 0, 1, false, out.as<uint32_t>(), nullptr,
                              tot.as<uint32_t>(), tmp.p, true, c->stream));
      h->rows[0].reset();
      relation_free_storage(r);
      r->col[0] = (uint32_t*)out.keep();
      r->nrows = n;
      r->sorted = true;
      return XL_OK;
    }
    if (h->dense) {  // every tuple is a set bit: rows in ascending (x, y)
      // off (range0 + 1 words) doubles as the CSR offsets of the finished
      // relation by its first column, kept as a ready index for later strata
      Buf cnt, off, tmp;
      XL_TRY(dalloc(c, (size_t)h->range0 * 4, &cnt, "row counts"));
      XL_TRY(dalloc(c, (size_t)(h->range0 + 1) * 4, &off, "row offsets"));
      XL_TRY(dalloc(c, k::scan_temp_bytes(h->range0), &tmp, "scan scratch"));
      HIP_TRY(c, k::row_popcount(h->bits.as<uint32_t>(), h->range0, h->row_words, cnt.as<uint32_t>(), c->stream));
      HIP_TRY(c, k::scan_exclusive_u32(cnt.as<uint32_t>(), off.as<uint32_t>(), h->range0,
                                       off.as<uint32_t>() + h->range0, tmp.p, c->stream));
      // the receipt's count is the row count; the bitmap's own total is
      // compared on the device (flag read at the end of the run), and the
      // rows are written only up to the allocated count
      const int64_t n = h->keys;
      HIP_TRY(c, k::check_eq(off.as<uint32_t>() + h->range0, (uint32_t)n, c->dcheck, CHECK_BITMAP_ROWS, c->stream));
      h->rows[0].reset();
      h->rows[1].reset();
      Buf out[2];
      for (int j = 0; j < 2; ++j) XL_TRY(dalloc(c, (size_t)std::max<int64_t>(n, 1) * 4, &out[j], "relation column"));
      HIP_TRY(c, k::bits_to_rows(h->bits.as<uint32_t>(), h->range0, h->row_words, off.as<uint32_t>(), h->kp.lo[0],
                                 h->kp.lo[1], out[0].as<uint32_t>(), out[1].as<uint32_t>(), n, c->stream));
      relation_free_storage(r);
      for (int j = 0; j < 2; ++j) r->col[j] = (uint32_t*)out[j].keep();
      r->nrows = n;
      r->sorted = true;
      auto ix = std::make_unique<DevIndex>();
      ix->rel = r;
      ix->col = 0;
      ix->probe.off = off.as<uint32_t>();
      ix->probe.ncols = 2;
      for (int j = 0; j < 2; ++j) ix->probe.col[j] = r->col[j];
      ix->probe.key_lo = h->kp.lo[0];
      ix->probe.key_range = (uint32_t)h->range0;
      ix->owned.push_back(std::make_unique<Buf>(c));
      ix->owned.back()->p = off.keep();
      kept.push_back(std::move(ix));
      return XL_OK;
    }
    if (h->dcount) {
      const int64_t n = h->range0 * h->range1;
      Buf tmp, tot;
      XL_TRY(dalloc(c, k::compact_temp_bytes(n), &tmp, "compaction scratch"));
      XL_TRY(dalloc(c, 16, &tot, "count"));
      if (n <= BOUNDS_ONE_MAX) {
        // few slots: the rows go to columns sized for every slot, and their
        // count and the value column's bounds come back in one read
        Buf out[3];
        for (int j = 0; j <= h->nkey; ++j) XL_TRY(dalloc(c, (size_t)std::max<int64_t>(n, 1) * 4, &out[j], "relation column"));
        HIP_TRY(c, k::dcount_rows(h->counts.as<uint32_t>(), n, h->range1, h->kp, out[0].as<uint32_t>(),
                                  h->nkey == 2 ? out[1].as<uint32_t>() : nullptr, out[h->nkey].as<uint32_t>(),
                                  std::max<int64_t>(n, 1), tot.as<uint32_t>(), tmp.p, c->stream));
        const bool i32 = r->types[h->nkey] == T_I32;
        if (i32)
          HIP_TRY(c, k::bounds_one(out[h->nkey].as<int32_t>(), tot.as<uint32_t>(), n, tot.as<int32_t>() + 1,
                                   c->stream));
        int32_t t[3] = {0, 0, 0};
        XL_TRY(ctl_read(c, tot.p, i32 ? 12 : 4, t));
        const uint32_t m = (uint32_t)t[0];
        relation_free_storage(r);
        for (int j = 0; j <= h->nkey; ++j) r->col[j] = (uint32_t*)out[j].keep();
        r->nrows = (int64_t)m;
        r->sorted = true;  // counters in key order
        h->keys = (int64_t)m;
        if (i32 && m > 0) {
          r->lo[h->nkey] = t[1];
          r->hi[h->nkey] = t[2];
          h->vbounds = true;
        }
        if (r->max_rows > 0 && r->nrows > r->max_rows)
          return c->fail(XL_CAPACITY_EXCEEDED, "relation " + r->name + " exceeds its max_rows");
        return XL_OK;
      }
      HIP_TRY(c, k::dcount_rows(h->counts.as<uint32_t>(), n, h->range1, h->kp, nullptr, nullptr, nullptr, 0,
                                tot.as<uint32_t>(), tmp.p, c->stream));
      uint32_t m = 0;
      XL_TRY(ctl_read(c, tot.p, 4, &m));
      Buf out[3];
      for (int j = 0; j <= h->nkey; ++j) XL_TRY(dalloc(c, (size_t)std::max<uint32_t>(m, 1) * 4, &out[j], "relation column"));
      HIP_TRY(c, k::dcount_rows(h->counts.as<uint32_t>(), n, h->range1, h->kp, out[0].as<uint32_t>(),
                                h->nkey == 2 ? out[1].as<uint32_t>() : nullptr, out[h->nkey].as<uint32_t>(),
                                (int64_t)m, tot.as<uint32_t>(), tmp.p, c->stream));
      relation_free_storage(r);
      for (int j = 0; j <= h->nkey; ++j) r->col[j] = (uint32_t*)out[j].keep();
      r->nrows = (int64_t)m;
      r->sorted = true;
      h->keys = (int64_t)m;
      if (r->max_rows > 0 && r->nrows > r->max_rows)
        return c->fail(XL_CAPACITY_EXCEEDED, "relation " + r->name + " exceeds its max_rows");
      return XL_OK;
    }
    if (h->dv) {
      const int64_t n = h->keys;
      const int64_t ns = full_slots(h);
      for (Buf* b : {&h->dcur, &h->dnext, &h->ndrow[0], &h->ndrow[1], &h->ndrow[2]}) b->reset();  // rounds are over
      Buf out[3], tmp, tot;
      for (int j = 0; j <= h->nkey; ++j) XL_TRY(dalloc(c, (size_t)std::max<int64_t>(n, 1) * 4, &out[j], "relation column"));
      XL_TRY(dalloc(c, h->ds ? k::target_rows_temp_bytes(h->range1, h->nrank_d) : k::compact_temp_bytes(ns), &tmp,
                    "compaction scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      if (h->ds)
        HIP_TRY(c, k::target_rows(h->dvals.as<uint32_t>(), h->dpres.as<uint32_t>(), h->dict.as<uint32_t>(), h->n0,
                                  h->range1, h->nrank_d, h->kp, r->types[h->nkey], h->fold, out[0].as<uint32_t>(),
                                  out[1].as<uint32_t>(), out[2].as<uint32_t>(), std::max<int64_t>(n, 1),
                                  tot.as<uint32_t>(), tmp.p, c->stream));
      else
        HIP_TRY(c, k::dense_rows(h->dvals.as<uint32_t>(), h->dpres.as<uint32_t>(), h->dict.as<uint32_t>(), ns,
                                 h->range1, h->kp, r->types[h->nkey], h->fold, out[0].as<uint32_t>(),
                                 h->nkey == 2 ? out[1].as<uint32_t>() : nullptr, out[h->nkey].as<uint32_t>(),
                                 std::max<int64_t>(n, 1), tot.as<uint32_t>(), tmp.p, c->stream));
      HIP_TRY(c, k::check_eq(tot.as<uint32_t>(), (uint32_t)n, c->dcheck, CHECK_VALUE_ROWS, c->stream));
      relation_free_storage(r);
      for (int j = 0; j <= h->nkey; ++j) r->col[j] = (uint32_t*)out[j].keep();
      r->nrows = n;
      r->sorted = true;  // rows rank by rank: ascending keys
    } else if (h->sorted_set) {
      return materialize_sorted_set(h);
    } else if (h->is_sortagg && h->once) {  // folded in key order
      Buf none[3];
      for (int j = 0; j <= h->nkey; ++j)
        if (!h->drow[j].p) XL_TRY(dalloc(c, 4, &none[j], "relation column"));
      relation_free_storage(r);
      for (int j = 0; j <= h->nkey; ++j) r->col[j] = (uint32_t*)(h->drow[j].p ? h->drow[j] : none[j]).keep();
      r->nrows = h->keys;
      r->sorted = true;
    } else if (h->is_set) {
      relation_free_storage(r);
      for (int j = 0; j < h->nkey; ++j) r->col[j] = (uint32_t*)h->rows[j].keep();
      r->nrows = h->nrows;
      r->key_cols = h->nkey;
    } else {
      Buf out[3];
      const int64_t n = h->keys;
      for (int j = 0; j <= h->nkey; ++j) XL_TRY(dalloc(c, (size_t)std::max<int64_t>(n, 1) * 4, &out[j], "relation column"));
      Buf tmp, tot;
      XL_TRY(dalloc(c, k::compact_temp_bytes(h->cap), &tmp, "compaction scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      HIP_TRY(c, k::table16_compact(h->table.as<Slot16>(), h->cap, h->kp, r->types[h->nkey], h->fold,
                                    out[0].as<uint32_t>(), h->nkey == 2 ? out[1].as<uint32_t>() : nullptr,
                                    out[h->nkey].as<uint32_t>(), std::max<int64_t>(n, 1), tot.as<uint32_t>(), tmp.p,
                                    c->stream));
      HIP_TRY(c, k::check_eq(tot.as<uint32_t>(), (uint32_t)n, c->dcheck, CHECK_VALUE_ROWS, c->stream));
      relation_free_storage(r);
      for (int j = 0; j <= h->nkey; ++j) r->col[j] = (uint32_t*)out[j].keep();
      r->nrows = n;
      r->key_cols = h->nkey;
    }
    return XL_OK;
  }

  // Rows of a sorted set head: its candidate keys sorted (unless they ascend
  // already), the distinct ones unpacked.
  xl_status materialize_sorted_set(HeadRun* h) {
    Relation* r = h->rel;
    const int64_t n = h->cn;
    Buf out[2];
    uint32_t m = 0;
    if (n == 0) {
      for (int j = 0; j < h->nkey; ++j) XL_TRY(dalloc(c, 4, &out[j], "relation column"));
    } else {
      const bool wide = key_bytes(h) == 8;
      const int kbits = h->nkey == 2 ? h->bits0 + h->kp.shift : h->bits0;
      Buf k2, tmp, cnt, off, tot;
      int alt = 0;
      if (!h->in_order) {
        XL_TRY(dalloc(c, (size_t)n * (wide ? 8 : 4), &k2, "sort keys"));
        XL_TRY(dalloc(c, k::radix_temp_bytes(n), &tmp, "sort scratch"));
        if (wide)
          HIP_TRY(c, k::radix_sort_u64(h->ckey.as<u64>(), nullptr, k2.as<u64>(), nullptr, n, kbits, tmp.p, c->stream,
                                       &alt));
        else
          HIP_TRY(c, k::radix_sort_u32(h->ckey.as<uint32_t>(), nullptr, k2.as<uint32_t>(), nullptr, n, kbits, tmp.p,
                                       c->stream, &alt));
      }
      const void* sk = alt ? k2.p : h->ckey.p;
      const int64_t nt = k::row_tiles(n);
      XL_TRY(dalloc(c, (size_t)nt * 4, &cnt, "row counts"));
      XL_TRY(dalloc(c, (size_t)nt * 4, &off, "row offsets"));
      XL_TRY(dalloc(c, k::scan_temp_bytes(nt), &tmp, "scan scratch"));
      XL_TRY(dalloc(c, 8, &tot, "count"));
      HIP_TRY(c, k::count_rows(sk, wide, nullptr, n, cnt.as<uint32_t>(), c->stream));
      HIP_TRY(c, k::scan_exclusive_u32(cnt.as<uint32_t>(), off.as<uint32_t>(), nt, tot.as<uint32_t>(), tmp.p,
                                       c->stream));
      XL_TRY(ctl_read(c, tot.p, 4, &m));
      if (r->max_rows > 0 && (int64_t)m > r->max_rows)
        return c->fail(XL_CAPACITY_EXCEEDED, "relation " + r->name + " exceeds its max_rows " +
                                                 std::to_string(r->max_rows));
      k::RowPack rp{};
      rp.by = h->nkey;
      for (int j = 0; j < h->nkey; ++j) {
        XL_TRY(dalloc(c, (size_t)m * 4, &out[j], "relation column"));
        const int bits = j == 0 ? h->bits0 : h->kp.shift;
        rp.type[j] = T_I32;
        rp.lo[j] = (uint32_t)h->kp.lo[j] ^ 0x80000000u;
        rp.mask[j] = bits >= 32 ? 0xffffffffu : (1u << bits) - 1u;
        rp.shift[j] = j == 0 && h->nkey == 2 ? h->kp.shift : 0;
        rp.ltype[j] = XL_I32;  // stored images stay as they are
        rp.dst[j] = out[j].p;
      }
      HIP_TRY(c, k::unpack_rows(rp, sk, wide, nullptr, n, off.as<uint32_t>(), c->stream));
    }
    relation_free_storage(r);
    for (int j = 0; j < h->nkey; ++j) r->col[j] = (uint32_t*)out[j].keep();
    r->nrows = h->keys = m;
    r->sorted = true;
    return XL_OK;
  }

  // Indexes over heads of the running stratum describe the relation as it
  // was when they were built; each pass rebuilds them from the current rows.
  // All of a pass's joins with a head of the stratum read the relation as it
  // was when the pass began (Alg. 1: every variant of round k sees S_k), so
  // those indexes are built up front, before any variant adds tuples.
  xl_status snapshot_head_indexes(const std::vector<RulePlan>& plans) {
    indexes.erase(std::remove_if(indexes.begin(), indexes.end(),
                                 [&](const std::unique_ptr<DevIndex>& ix) { return head_of(ix->rel) != nullptr; }),
                  indexes.end());
    for (const RulePlan& p : plans)
      for (const StepPlan& sp : p.steps)
        if (head_of(sp.rel)) {
          IndexProbe probe;
          XL_TRY(get_index(sp.rel, sp.key_col, &probe));
        }
    return XL_OK;
  }

  // ------------------------------------------------------------ strata
  // A triangle-join stratum (see RulePlan::wcoj): count -> scan ->
  // materialize straight into the head's columns, in ascending (X, Y, Z)
  // order; no hash table or bitmap is needed because every (driver row, Z)
  // pair is produced once.
  xl_status run_wcoj(const RulePlan& p) {
    Relation* h = p.head;
    relation_free_storage(h);
    WcojArgs a{};
    IndexProbe ia{};
    XL_TRY(get_index(p.driver, p.tri_a[0], &ia, p.tri_a[1], nullptr, 1));
    XL_TRY(get_index(p.tri_brel, p.tri_b[0], &a.ib, p.tri_b[1], nullptr, 1));
    XL_TRY(get_index(p.tri_crel, p.tri_c[0], &a.ic, p.tri_c[1], nullptr, 1));
    a.ax = ia.col[p.tri_a[0]];
    a.ay = ia.col[p.tri_a[1]];
    a.na = p.driver->nrows;
    a.bz = a.ib.col[p.tri_b[1]];
    a.cz = a.ic.col[p.tri_c[1]];
    a.probe_shorter = c->wcoj_shorter;
    auto finish = [&](int64_t n) -> xl_status {
      h->nrows = n;
      h->lo[0] = p.driver->lo[p.tri_a[0]];
      h->hi[0] = p.driver->hi[p.tri_a[0]];
      h->lo[1] = p.driver->lo[p.tri_a[1]];
      h->hi[1] = p.driver->hi[p.tri_a[1]];
      h->lo[2] = p.tri_brel->lo[p.tri_b[1]];
      h->hi[2] = p.tri_brel->hi[p.tri_b[1]];
      record(n);
      st->new_tuples_total += n;
      return XL_OK;
    };
    if (a.na == 0 || p.tri_brel->nrows == 0 || p.tri_crel->nrows == 0) return finish(0);
    Buf work, flags, flag_pos, crow, cw, cofs, tmp, tot;
    XL_TRY(dalloc(c, (size_t)a.na * 4, &work, "triangle work"));
    XL_TRY(dalloc(c, (size_t)a.na * 4, &flags, "triangle row flags"));
    XL_TRY(dalloc(c, (size_t)a.na * 4, &flag_pos, "triangle row positions"));
    XL_TRY(dalloc(c, std::max(k::scan_temp_bytes(a.na), k::scan_temp_bytes(a.na + 1)), &tmp, "scan scratch"));
    XL_TRY(dalloc(c, 16, &tot, "count"));
    a.work = work.as<uint32_t>();
    HIP_TRY(c, k::wcoj_work(a, c->stream));
    // flags and positions in separate arrays: the scan then takes its
    // one-launch form (it reads other tiles' flags)
    HIP_TRY(c, k::nonzero_flags(work.as<uint32_t>(), a.na, flags.as<uint32_t>(), c->stream));
    HIP_TRY(c, k::scan_exclusive_u32(flags.as<uint32_t>(), flag_pos.as<uint32_t>(), a.na, tot.as<uint32_t>(), tmp.p,
                                     c->stream));
    uint32_t nz = 0;
    XL_TRY(ctl_read(c, tot.p, 4, &nz));
    if (nz == 0) return finish(0);
    flags.reset();
    Buf seg;
    XL_TRY(dalloc(c, (size_t)nz * 4, &crow, "triangle rows"));
    XL_TRY(dalloc(c, (size_t)(nz + 1) * 8, &cw, "triangle row work"));
    XL_TRY(dalloc(c, (size_t)nz * 12, &seg, "triangle row lists"));
    a.seg = seg.as<uint32_t>();
    HIP_TRY(c, k::wcoj_compact(a, flag_pos.as<uint32_t>(), nz, crow.as<uint32_t>(), cw.as<unsigned long long>(),
                               c->stream));
    work.reset();
    flag_pos.reset();
    XL_TRY(dalloc(c, (size_t)(nz + 1) * 8, &cofs, "triangle row offsets"));
    XL_TRY(dalloc(c, k::scan_temp_bytes(nz), &tmp, "scan scratch"));
    HIP_TRY(c, k::scan_exclusive_u64(cw.as<u64>(), cofs.as<u64>(), nz, cofs.as<u64>() + nz, tmp.p, c->stream));
    u64 items = 0;
    XL_TRY(ctl_read(c, cofs.as<u64>() + nz, 8, &items));
    if (items >= ((u64)1 << 40)) return c->fail(XL_UNSUPPORTED, "triangle join with more than 2^40 probes");
    a.crow = crow.as<uint32_t>();
    a.cofs = cofs.as<unsigned long long>();
    a.nz = nz;
    a.items = items;
    const u64 nchunks = (items + k::WC_CHUNK - 1) / k::WC_CHUNK;
    Buf ccnt, coff, tmp2;
    XL_TRY(dalloc(c, (size_t)nchunks * 4, &ccnt, "chunk counts"));
    XL_TRY(dalloc(c, (size_t)nchunks * 4, &coff, "chunk offsets"));
    XL_TRY(dalloc(c, k::scan_temp_bytes((int64_t)nchunks), &tmp2, "scan scratch"));
    a.chunk_cnt = ccnt.as<uint32_t>();
    // one bit per probe, kept by the count pass for the write pass; without
    // room for it the write pass probes again
    Buf mask;
    if (dalloc(c, (size_t)nchunks * (k::WC_CHUNK / 8), &mask, "triangle hits") != XL_OK) mask.reset();
    a.mask = mask.as<u64>();
    float ms_total = 0;
    auto timed = [&](bool mat) -> xl_status {
      if (c->profile) HIP_TRY(c, hipEventRecord(ev[0], c->stream));
      HIP_TRY(c, k::wcoj_probe(a, mat, c->stream));
      if (c->profile) {
        HIP_TRY(c, hipEventRecord(ev[1], c->stream));
        HIP_TRY(c, hipEventSynchronize(ev[1]));
        float ms = 0;
        HIP_TRY(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        ms_total += ms;
      }
      return XL_OK;
    };
    XL_TRY(timed(false));
    HIP_TRY(c, k::scan_exclusive_u32(ccnt.as<uint32_t>(), coff.as<uint32_t>(), (int64_t)nchunks, tot.as<uint32_t>(),
                                     tmp2.p, c->stream));
    uint32_t n = 0;
    XL_TRY(ctl_read(c, tot.p, 4, &n));
    if (h->max_rows > 0 && (int64_t)n > h->max_rows)
      return c->fail(XL_CAPACITY_EXCEEDED, "relation " + h->name + " exceeds its max_rows " +
                                               std::to_string(h->max_rows));
    Buf out[3];
    for (int j = 0; j < 3; ++j) {
      xl_status got = dalloc(c, (size_t)std::max<uint32_t>(n, 1) * 4, &out[j], "relation column");
      if (got != XL_OK && mask.p) {
        mask.reset();
        a.mask = nullptr;
        got = dalloc(c, (size_t)std::max<uint32_t>(n, 1) * 4, &out[j], "relation column");
      }
      XL_TRY(got);
    }
    a.chunk_off = coff.as<uint32_t>();
    a.out0 = out[0].as<uint32_t>();
    a.out1 = out[1].as<uint32_t>();
    a.out2 = out[2].as<uint32_t>();
    if (n) XL_TRY(timed(true));
    cands += (int64_t)items;
    if (c->profile) {
      st->wcoj_ms += ms_total;
      st->wcoj_launches += n ? 2 : 1;
      st->wcoj_candidates += (int64_t)items;
      st->wcoj_new += n;
    }
    for (int j = 0; j < 3; ++j) h->col[j] = (uint32_t*)out[j].keep();
    h->sorted = true;
    return finish(n);
  }

  xl_status run_stratum(Stratum& s, int64_t max_iterations) {
    if (s.full.size() == 1 && s.full[0].wcoj) {
      heads.clear();
      return run_wcoj(s.full[0]);
    }
    heads.clear();
    // rows the heads keep from before the run (set, min and max heads resume;
    // count, sum and logsumexp heads are recomputed from empty)
    int64_t rows_before = 0;
    for (Relation* h : s.heads) {
      const Agg a = prog->head_agg(h);
      if (a == Agg::NONE || a == Agg::MIN || a == Agg::MAX) rows_before += h->nrows;
    }
    XL_TRY(setup_heads(s));
    for (auto& h : heads) begin_round(h.get());
    XL_TRY(snapshot_head_indexes(s.full));
    // A stratum that runs as one resident frontier launch builds that
    // launch's indexes (inputs only) while its seed round runs: the host's
    // launches then overlap the seed kernel instead of following its count
    // read.
    struct ClearHook {
      std::function<xl_status()>& f;
      ~ClearHook() { f = nullptr; }
    } clear_hook{before_count_read};
    if (s.recursive && heads.size() == 1 && heads[0]->resident && s.variants.size() == 1 &&
        s.variants[0].driver_delta && head_of(s.variants[0].head) == heads[0].get())
      before_count_read = [this, &s]() {
        FrontierArgs f{};
        return frontier_args(s.variants[0], heads[0].get(), f);
      };
    for (RulePlan& p : s.full) XL_TRY(eval_plan(p));
    before_count_read = nullptr;
    int64_t total = 0;
    for (auto& h : heads) {
      int64_t d = 0;
      XL_TRY(finish_round(h.get(), &d));
      total += d;
      st->new_tuples_total += d;
    }
    const int32_t seed_record = st->rounds_recorded;
    const int64_t seeded = total;
    record(total);
    if (s.recursive && total > 0 && batched_tiles(s)) {
      XL_TRY(run_tiles_batched(s.variants[0], heads[0].get(), max_iterations));
      total = 0;
    }
    if (s.recursive && total > 0 && batched_pull(s)) {
      XL_TRY(run_pull_batched(s.variants[0], heads[0].get(), max_iterations));
      total = 0;
    }
    if (s.recursive && total > 0 && batched_gather(s)) {
      XL_TRY(run_gather_batched(s.variants[0], heads[0].get(), max_iterations));
      total = 0;
    }
    if (s.recursive && total > 0 && batched_sets(s)) {
      XL_TRY(run_sets_batched(s, max_iterations));
      total = 0;
    }
    if (s.recursive && total > 0 && batched_values(s)) {
      XL_TRY(run_values_batched(s, heads[0].get(), max_iterations));
      total = 0;
    }
    if (s.recursive && total > 0 && resident_frontier(s)) {
      if (max_iterations == 0)
        return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap 0 reached before the fixpoint");
      XL_TRY(run_frontier_resident(s.variants[0], heads[0].get(), max_iterations));
      total = 0;
    }
    if (s.recursive) {
      int64_t pass = 0;
      while (total > 0) {
        if (batched_selfjoin()) {
          XL_TRY(run_selfjoin_batched(heads[0].get(), pass, max_iterations));
          break;
        }
        if (pass >= max_iterations)
          return c->fail(XL_CONVERGENCE_FAILURE, "iteration cap " + std::to_string(max_iterations) +
                                                     " reached before the fixpoint");
        ++pass;
        st->iterations++;
        for (auto& h : heads) begin_round(h.get());
        XL_TRY(snapshot_head_indexes(s.variants));
        for (RulePlan& p : s.variants) XL_TRY(eval_plan(p));
        total = 0;
        for (auto& h : heads) {
          int64_t d = 0;
          XL_TRY(finish_round(h.get(), &d));
          total += d;
          st->new_tuples_total += d;
        }
        record(total);
      }
    }
    // indexes over this stratum's heads saw unfinished relations; the rest
    // stay valid (a relation is final once its stratum ends)
    for (auto& h : heads)
      indexes.erase(std::remove_if(indexes.begin(), indexes.end(),
                                   [&](const std::unique_ptr<DevIndex>& ix) { return ix->rel == h->rel; }),
                    indexes.end());
    kept.clear();
    for (auto& h : heads) XL_TRY(materialize(h.get()));
    if (!s.recursive) {
      // a non-recursive stratum records the rows it produced; heads built from
      // sorted candidates, counters or index degrees only have them now
      int64_t produced = -rows_before;
      for (auto& h : heads) produced += h->rel->nrows;
      st->new_tuples_total += produced - seeded;
      if (seed_record < XL_STATS_ROUNDS) st->delta_rows[seed_record] = produced;
    }
    for (auto& ix : kept) indexes.push_back(std::move(ix));
    kept.clear();
    heads.clear();
    return XL_OK;
  }
};

}  // namespace

xl_status run_program(Program* p, int64_t max_iterations, xl_fixpoint_stats* st) {
  Context* c = p->ctx;
  memset(st, 0, sizeof(*st));
  if (c->device < 0) return c->fail(XL_INVALID_ARGUMENT, "planning-only context cannot run programs");
  if (max_iterations < 0) return c->fail(XL_INVALID_ARGUMENT, "negative iteration cap");
  c->arena.reset_peak();
  c->runs++;
  const int64_t ctl0 = c->control_bytes;
  {
    const xl_status s0 = resolve_wide_constants(p);
    if (s0 != XL_OK) {
      st->status = s0;
      return s0;
    }
  }
  hipEvent_t e0, e1;
  HIP_TRY(c, hipEventCreate(&e0));
  HIP_TRY(c, hipEventCreate(&e1));
  HIP_TRY(c, hipEventRecord(e0, c->stream));
  HIP_TRY(c, hipMemsetAsync(c->dcheck, 0, 8, c->stream));
  xl_status s = XL_OK;
  {
    Runner run{c, p, st};
    if (c->profile) {
      HIP_TRY(c, hipEventCreate(&run.ev[0]));
      HIP_TRY(c, hipEventCreate(&run.ev[1]));
    }
    for (Stratum& str : p->strata) {
      s = run.run_stratum(str, max_iterations);
      if (s != XL_OK) break;
    }
    st->candidates_total = run.cands;
  }
  // the consistency flags ride on the run's final synchronization: the copy
  // into the control block's last word is complete once e1 is
  unsigned long long* check_host = (unsigned long long*)((char*)c->pinned + CTL_CHECK_OFFSET);
  *check_host = 0;
  (void)hipMemcpyAsync(check_host, c->dcheck, 8, hipMemcpyDeviceToHost, c->stream);
  (void)hipEventRecord(e1, c->stream);
  (void)hipEventSynchronize(e1);
  if (s == XL_OK && *check_host) {
    const unsigned long long f = *check_host;
    s = c->fail(XL_DEVICE_ERROR, std::string("internal consistency check failed:") +
                                     (f & CHECK_BITMAP_ROWS ? " bitmap row count" : "") +
                                     (f & CHECK_VALUE_ROWS ? " value row count" : "") +
                                     (f & CHECK_COUNT_DOMAIN ? " count key outside the head domain" : ""));
  }
  float ms = 0;
  (void)hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  st->ms_total = ms;
  st->strata = (int32_t)p->strata.size();
  for (auto& h : p->heads) st->derived_tuples += h.rel->nrows;
  st->peak_workspace_bytes = (int64_t)c->arena.peak();
  st->control_bytes_read = c->control_bytes - ctl0;
  st->status = s;
  return s;
}

}  // namespace xlh
