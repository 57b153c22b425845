// Host half of libpkv: argument validation, the checkpoint layout, the work
// list and the RoPE correction tables.  Pure C++ (no HIP calls), so every
// validation path runs without a GPU.
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <limits>
#include <new>
#include <vector>

#include "pkv.h"
#include "pkv_internal.h"

namespace pkv {
namespace {

bool is_pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }

int ilog2(int64_t x) {
  int r = 0;
  while ((int64_t(1) << r) < x) ++r;
  return r;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

pkv_status_t check_model(const pkv_model_t* m) {
  if (!m) return PKV_ERR_INVALID_ARGUMENT;
  if (m->num_layers < 1 || m->num_kv_heads < 1) return PKV_ERR_INVALID_ARGUMENT;
  if (m->head_dim < 16 || m->head_dim > kMaxHeadDim || m->head_dim % 16 != 0) return PKV_ERR_INVALID_ARGUMENT;
  if (int64_t(m->num_kv_heads) * m->head_dim > kMaxRowElems) return PKV_ERR_INVALID_ARGUMENT;
  if (m->block_tokens < 1 || m->block_tokens > kMaxBlockTokens) return PKV_ERR_INVALID_ARGUMENT;
  if ((int64_t(m->block_tokens) * m->num_kv_heads * m->head_dim) % 32 != 0) return PKV_ERR_INVALID_ARGUMENT;
  if (!is_pow2(m->page_size) || m->page_size > (1 << 20)) return PKV_ERR_INVALID_ARGUMENT;
  // One page of one cache is at most 2 GiB: the kernels address inside a page with 32-bit offsets.
  if (int64_t(m->page_size) * m->num_kv_heads * m->head_dim * 2 > (int64_t(1) << 31)) return PKV_ERR_INVALID_ARGUMENT;
  if (m->pool_pages < 1) return PKV_ERR_INVALID_ARGUMENT;
  if (!(isfinite(m->rope_theta) && m->rope_theta > 0.0)) return PKV_ERR_INVALID_ARGUMENT;
  if (m->out_dtype != PKV_OUT_FP16 && m->out_dtype != PKV_OUT_BF16) return PKV_ERR_INVALID_ARGUMENT;
  if (m->rope_style != PKV_ROPE_HALF && m->rope_style != PKV_ROPE_INTERLEAVED) return PKV_ERR_INVALID_ARGUMENT;
  if (m->rotary_dim != 0 && (m->rotary_dim < 16 || m->rotary_dim > m->head_dim || m->rotary_dim % 16 != 0))
    return PKV_ERR_INVALID_ARGUMENT;
  if (m->kv_layout != PKV_KV_SEPARATE && m->kv_layout != PKV_KV_PAIRED) return PKV_ERR_INVALID_ARGUMENT;
  if (m->reserved != 0) return PKV_ERR_INVALID_ARGUMENT;
  if (m->inv_freq) {
    const int32_t R = m->rotary_dim ? m->rotary_dim : m->head_dim;
    for (int32_t i = 0; i < R / 2; ++i)
      if (!isfinite(m->inv_freq[i])) return PKV_ERR_INVALID_ARGUMENT;
  }
  // Cache elements per layer and in total must stay far from int64 overflow.
  const double elems = 2.0 * double(m->num_layers) * double(m->pool_pages) * m->page_size * m->num_kv_heads * m->head_dim;
  if (elems > 1e18) return PKV_ERR_INVALID_ARGUMENT;
  return PKV_OK;
}

// RoPE helpers: rotated channels per head, the frequency of pair i, and the
// pair that element e of key piece j rotates (k = 8j + e; -1 = none).
int32_t rotary_dim(const pkv_model_t& m) { return m.rotary_dim ? m.rotary_dim : m.head_dim; }

double rope_frequency(const pkv_model_t& m, int64_t i) {
  const int32_t R = rotary_dim(m);
  return m.inv_freq ? m.inv_freq[i] : pow(m.rope_theta, -2.0 * double(i) / double(R));
}

int64_t rope_table_pair(const pkv_model_t& m, int64_t k) {
  const int64_t D = m.head_dim, R = rotary_dim(m);
  const int64_t j = k / 8, e = k % 8;
  if (m.rope_style == PKV_ROPE_HALF) {
    // Piece j < R/16 holds channels [8j, 8j+8) and [R/2 + 8j, ...): pairs 8j + e.
    return 8 * j < R / 2 ? 8 * j + e : -1;
  }
  // Interleaved: piece j holds channels [8j, 8j+8) (elements 0..3 are its four
  // pairs) and [D/2 + 8j, ...) (elements 4..7); a pair rotates if inside [0, R).
  const int64_t first = e < 4 ? 8 * j : D / 2 + 8 * j;
  return first + 8 <= R ? first / 2 + e % 4 : -1;
}

pkv_status_t check_request_fields(const pkv_request_t& r) {
  if (r.reserved != 0) return PKV_ERR_INVALID_ARGUMENT;
  if (r.suffix_tokens < 0 || r.num_logical_pages < 0 || r.dst_row0 < 0) return PKV_ERR_INVALID_ARGUMENT;
  if (r.dst_row0 > (int64_t(1) << 50)) return PKV_ERR_INVALID_ARGUMENT;
  if (r.suffix_tokens > 0 && (!r.tags || !r.repair_mask)) return PKV_ERR_INVALID_ARGUMENT;
  if (r.num_logical_pages > 0 && !r.page_table) return PKV_ERR_INVALID_ARGUMENT;
  if (r.payload_offset % 16 != 0 || r.scale_offset % 4 != 0) return PKV_ERR_INVALID_ARGUMENT;
  if (r.payload_offset > (uint64_t(1) << 56) || r.scale_offset > (uint64_t(1) << 56)) return PKV_ERR_INVALID_ARGUMENT;
  return PKV_OK;
}

pkv_status_t check_tags(const pkv_request_t& r, int64_t nb) {
  for (int64_t b = 0; b < nb; ++b)
    if (r.tags[b] > PKV_TAG_K4V4) return PKV_ERR_BAD_TAG;
  return PKV_OK;
}

uint64_t tile_bytes(const pkv_model_t& m, int bits) {
  return uint64_t(m.block_tokens) * m.num_kv_heads * m.head_dim * bits / 8;
}

// Append a range, merging it with the previous one (if that one is at index
// >= first) when it starts at most `gap` bytes after that one ends.
void add_range(std::vector<CopyRange>& v, size_t first, uint64_t off, uint64_t len, uint64_t gap) {
  if (v.size() > first && v.back().off + v.back().len <= off && off - (v.back().off + v.back().len) <= gap)
    v.back().len = off + len - v.back().off;
  else
    v.push_back(CopyRange{off, len});
}

// Windows of the staged restore for one request: the most consecutive reused
// blocks (payload order, offsets from the layer's start) that span at most
// kStagePayloadBytes (one block, at most 16 MiB, always fits), each with its
// copies (blocks closer than kHostGapBytes merged).
void add_stage_windows(RequestCopies& rc, const std::vector<CopyRange>& blocks) {
  for (size_t i = 0; i < blocks.size();) {
    const uint64_t lo = blocks[i].off;
    size_t j = i + 1;
    while (j < blocks.size() && blocks[j].off + blocks[j].len - lo <= kStagePayloadBytes) ++j;
    StageWindow w;
    w.lo = lo;
    w.hi = blocks[j - 1].off + blocks[j - 1].len;
    w.copy0 = int64_t(rc.stage_copies.size());
    for (size_t a = i; a < j;) {
      size_t b = a + 1;
      while (b < j && blocks[b].off - (blocks[b - 1].off + blocks[b - 1].len) <= kHostGapBytes) ++b;
      const uint64_t c0 = blocks[a].off, c1 = blocks[b - 1].off + blocks[b - 1].len;
      rc.stage_copies.push_back(StageCopy{c0, c0 - lo, c1 - c0});
      a = b;
    }
    w.copy1 = int64_t(rc.stage_copies.size());
    rc.windows.push_back(w);
    i = j;
  }
}

// Marks physical pages as written; a page marked twice is written through two
// (request, logical page) pairs, since each pair is marked once.  One bit per
// page of the pool while the pool is not far larger than the pages touched, a
// sorted list of the pages otherwise.
class PageOwners {
 public:
  PageOwners(int64_t pool_pages, int64_t touched) {
    if (pool_pages / 1024 <= touched) bits_.assign(size_t(pool_pages + 63) / 64, 0);
  }
  void mark(int32_t page) {
    if (bits_.empty()) {
      pages_.push_back(page);
      return;
    }
    uint64_t& w = bits_[size_t(page) / 64];
    const uint64_t bit = uint64_t(1) << (page % 64);
    twice_ |= (w & bit) != 0;
    w |= bit;
  }
  bool twice() {
    if (!pages_.empty()) {
      std::sort(pages_.begin(), pages_.end());
      twice_ = std::adjacent_find(pages_.begin(), pages_.end()) != pages_.end();
    }
    return twice_;
  }

 private:
  std::vector<uint64_t> bits_;
  std::vector<int32_t> pages_;
  bool twice_ = false;
};

}  // namespace

int32_t page_shift(const pkv_model_t& m) { return ilog2(m.page_size) + (m.kv_layout == PKV_KV_PAIRED ? 1 : 0); }

int64_t layer_elems(const pkv_model_t& m) {
  return (m.kv_layout == PKV_KV_PAIRED ? 2 : 1) * m.pool_pages * int64_t(m.page_size) * m.num_kv_heads * m.head_dim;
}

uint64_t cache_bytes(const pkv_model_t& m) { return uint64_t(m.num_layers) * uint64_t(layer_elems(m)) * 2; }

bool cache_ranges(const pkv_model_t& m, const void* k_cache, const void* v_cache, uint64_t bytes, ByteRange (&ranges)[2],
                  int& count) {
  const uintptr_t k = reinterpret_cast<uintptr_t>(k_cache), v = reinterpret_cast<uintptr_t>(v_cache);
  if (k % 16 || v % 16) return false;
  if (m.kv_layout == PKV_KV_PAIRED) {
    if (v != k + uint64_t(m.page_size) * m.num_kv_heads * m.head_dim * 2) return false;
    ranges[0] = ByteRange{k_cache, bytes};
    count = 1;
    return true;
  }
  if (k < v + bytes && v < k + bytes) return false;
  ranges[0] = ByteRange{k_cache, bytes};
  ranges[1] = ByteRange{v_cache, bytes};
  count = 2;
  return true;
}

namespace {

// Whether the pieces that a store instruction writes next to each other make
// whole pieces of `bytes` bytes (of a cache that starts on one): they fill half
// a head's row, or half its rotary channels and half the others where
// rotate-half pairs stop short of the row.
bool stores_whole(const pkv_model_t& m, int32_t bytes) {
  return m.head_dim % bytes == 0 && (m.rope_style == PKV_ROPE_INTERLEAVED || m.rotary_dim % bytes == 0);
}

// Whether every work item is one row.
bool single_rows(const pkv_model_t& m) { return std::min(unit_tokens(m), m.page_size) == 1; }

}  // namespace

int restore_workgroups_per_cu(const HostPlan& hp) {
  // The memory system streams best with about 32K output elements of work in
  // flight per compute unit (two thirds of that for plans reading half a byte
  // or more per byte written, 1.14x for those reading under 0.3; three
  // quarters for units that do not rotate their keys, and again for separate K
  // and V caches; 0.72 of it, in either layout, for rows narrow enough to take
  // workgroups under 256 threads): so many units at a time, between 8 and 16
  // waves' worth (two to four 4-wave workgroups; from 6 waves for narrow rows).
  const pkv_plan_info_t& info = hp.info;
  const int waves = std::max(1, hp.workgroup / 64);
  const bool narrow = hp.workgroup < kWorkgroup;
  const int lo = std::max(1, (narrow ? 6 : 8) / waves), hi = std::max(1, 16 / waves);
  if (info.num_units == 0 || info.bytes_written == 0 || info.restored_rows == 0) return hi;
  const double ratio = double(info.bytes_read) / double(info.bytes_written);
  const double rotated = double(hp.rotated_rows) / double(info.restored_rows);
  const double target =
      32768.0 * (ratio >= 0.49 ? 2.0 / 3.0 : ratio >= 0.3 ? 1.0 : 1.14) * (0.75 + 0.25 * rotated) *
      (narrow ? 0.72 : hp.model.kv_layout == PKV_KV_SEPARATE ? 0.75 : 1.0);
  const double unit_elems =
      double(info.restored_rows) * hp.model.num_kv_heads * hp.model.head_dim / double(info.num_units);
  double n = std::floor(target / unit_elems + 0.5);
  // Narrow rows of whole 128-byte lines that rotate and read less than they
  // write hold fewer tokens per thread, and want more waves the smaller the
  // units, whatever the size of a workgroup: where units are 4096 elements, 10 of
  // them while the restore writes no more than the 256 MB cache holds (10.5 below
  // half a byte read per byte written), 8.5 above (as the target says below half).
  const bool cached = info.bytes_written <= uint64_t(256) << 20;
  if (narrow && stores_whole(hp.model, 128) && !single_rows(hp.model) && rotated >= 0.5 && ratio < 0.8 &&
      (ratio >= 0.49 || (ratio >= 0.3 && cached)))
    n = std::floor((ratio < 0.49 ? 10.5 : cached ? 10.0 : 8.5) * std::sqrt(4096.0 / unit_elems) / waves + 0.5);
  return n < lo ? lo : n > hi ? hi : int(n);
}

namespace {

// Rows stored at device scope.  The write stream bounds the kernel, and the
// 8B-shaped 32-layer restore takes 847 us that way against 886 (5.34 GB, 6.3
// against 6.0 TB/s), one layer of 690 units, launches back to back, 8.0 against 9.6
// (8.1 against 9.5 on paired pages).  It needs
//   whole 64-byte sectors, by the rows and by the caches' addresses: parts of
//     sectors are written through one by one (8 heads of 96, 16 layers: 1100 us
//     against 550), where the L2 puts them together;
//   units of 2 KB and more: single rows below that (one-token pages) are 1-9%
//     slower with it (2 heads of 128: mixed tags 1.02x, 4-bit 1.06x), larger ones
//     level or up to 16% faster (4 heads of 256, 48 MB: 0.84x; 8 heads of 128, 360
//     MB: mixed 1.01x, FP16 1.00x, 4-bit 1.07x);
//   and for pieces of half a 128-byte line (heads of 64): little read beside
//     the writes (below 0.42 bytes per byte written: 10-40% faster, 8 heads, K8V4
//     and 4-bit), keys that do not rotate, or a launch that writes up to 64 MB
//     (5-29% faster); above, mixed tags are 4-6% slower with it.
bool device_stores(const HostPlan& hp, int64_t units, uintptr_t k_cache, uintptr_t v_cache) {
  const pkv_model_t& m = hp.model;
  if (!stores_whole(m, 64) || (k_cache | v_cache) % 64 != 0) return false;
  if (single_rows(m) && m.num_kv_heads * m.head_dim < 1024) return false;
  if (stores_whole(m, 128)) return true;
  const pkv_plan_info_t& info = hp.info;
  return double(info.bytes_read) < 0.42 * double(info.bytes_written) || 2 * hp.rotated_rows < info.restored_rows ||
         double(info.bytes_written) * double(units) <= 64e6 * double(info.num_units);
}

// Launches of at most this many rounds of resident workgroups take the late
// start order of the restore kernel.  Separate caches run fewer
// workgroups at a time and gain from it longer: us late / early, 690
// workgroups a layer, separate (512 resident) and paired (768): 4 layers 30.0 /
// 30.8 and 29.6 / 30.0, 8 layers (10.8 and 7.2 rounds) 59.1 / 61.2 and 55.8 /
// 54.8, 16 layers 124.2 / 124.3 and 116.8 / 114.3, 32 layers 244.8 / 242.9 and
// 230.9 / 222.4.  Rows narrow enough for workgroups under kWorkgroup threads take
// it at any depth: on the 32-layer 8B-shaped workload's share of one KV head per
// GPU (one-wave workgroups of two tokens per thread) it measured 102-112 us
// against 127-135 us, and within 1% of the early order at two and four heads.
//
// Rows of partial sectors (heads of 80 and 96) gain nothing past kLateRounds: late
// / early at 8 to 11 rounds, separate caches, is 1.03-1.08 on average and up to
// 1.44 (35 layers of 8 heads of 80, K8V4: 109 us against 83), where whole sectors
// have 0.93-0.996.  Nor does one round at kOneRound workgroups suit them: 8 heads
// of 96, 530 to 755 workgroups, five mixes, 1.06 of the time at two to a compute
// unit, up to 1.22; whole sectors 0.96-0.98 (8, 16 and 32 heads of 128, 4 of 256).
constexpr int64_t kLateRoundsSeparate = 12;
constexpr int64_t kLateRounds = 6;

}  // namespace

RestoreLaunch restore_launch(const HostPlan& hp, int64_t units, uintptr_t k_cache, uintptr_t v_cache) {
  RestoreLaunch r;
  const bool sectors = stores_whole(hp.model, 64);
  const int64_t rounds = hp.model.kv_layout == PKV_KV_SEPARATE && sectors ? kLateRoundsSeparate : kLateRounds;
  r.late = hp.workgroup < kWorkgroup || units <= rounds * hp.cus * hp.per_cu;
  r.one_round =
      hp.workgroup == kWorkgroup && sectors && hp.per_cu < kOneRound && units <= kOneRound * int64_t(hp.cus);
  r.device = device_stores(hp, units, k_cache, v_cache);
  r.single = single_rows(hp.model);
  return r;
}

uint32_t link_groups(const HostPlan& hp, int64_t units) {
  const int64_t item = std::max<int64_t>(1, int64_t(hp.info.bytes_read) / hp.info.num_units);
  if (item < 1024 && units * hp.workgroup < (int64_t(1) << 32)) return 0;
  int64_t groups = std::min<int64_t>(16 * ceil_div(240000, 16 * item), 4096);
  if (item * units <= 8000000) groups = std::max<int64_t>(groups, 64);
  return uint32_t(std::min(groups, units));
}

// Threads of a restore workgroup: enough that each thread owns at most four
// tokens of the largest unit (units stop at page ends), in whole waves, at
// most kWorkgroup.  Rows of 8 heads x 128 keep 256; a one-head row of 128
// takes one wave, so shards with few heads per GPU do not leave most of each
// workgroup idle.
int32_t restore_workgroup(const pkv_model_t& m) {
  const int64_t cols = int64_t(m.num_kv_heads) * m.head_dim / 16;
  const int64_t tokens = std::min<int64_t>(unit_tokens(m), m.page_size);
  const int64_t threads = (cols * ceil_div(tokens, 4) + 63) / 64 * 64;
  return int32_t(std::max<int64_t>(64, std::min<int64_t>(kWorkgroup, threads)));
}

int32_t unit_tokens(const pkv_model_t& m) {
  const int64_t per = kUnitElems / (int64_t(m.num_kv_heads) * m.head_dim);
  return int32_t(std::max<int64_t>(1, std::min<int64_t>(per, m.block_tokens)));
}

uint64_t layer_payload_bytes(const pkv_model_t& m, const uint8_t* tags, int64_t nb) {
  uint64_t total = 0;
  for (int64_t b = 0; b < nb; ++b) total += tile_bytes(m, kKeyBits[tags[b]]) + tile_bytes(m, kValueBits[tags[b]]);
  return total;
}

namespace {

// The scale copies of layer l: each request's layer as one, neighbours merged.
void layer_scale_copies(const HostPlan& hp, int64_t l, std::vector<CopyRange>& scales) {
  for (const RequestCopies& rc : hp.copies)
    if (rc.scales_needed)
      add_range(scales, 0, (rc.scale_offset + uint64_t(l) * rc.layer_scales) * 2, rc.layer_scales * 2, 0);
}

}  // namespace

void layer_copies(const HostPlan& hp, int64_t l, std::vector<CopyRange>& payload, std::vector<CopyRange>& scales) {
  payload.clear();
  scales.clear();
  for (const RequestCopies& rc : hp.copies)
    for (const CopyRange& c : rc.ranges)
      payload.push_back(CopyRange{rc.payload_offset + uint64_t(l) * rc.layer_bytes + c.off, c.len});
  layer_scale_copies(hp, l, scales);
}

StageStep stage_step(const RequestCopies& rc, int64_t l, size_t window) {
  const StageWindow& w = rc.windows[window];
  StageStep st;
  st.payload_base = rc.payload_offset + uint64_t(l) * rc.layer_bytes;
  st.win_lo = st.payload_base + w.lo;
  st.win_hi = st.payload_base + w.hi;
  st.scale0 = rc.scales_needed ? rc.scale_offset + uint64_t(l) * rc.layer_scales : 0;
  st.scale_elems = rc.scales_needed && window == 0 ? rc.layer_scales : 0;
  return st;
}

// Whether the streamed restore pulls its copies with a kernel instead of
// enqueueing them on DMA streams.  A DMA copy takes about 16 us of its stream
// beyond its transfer, and a layer's events and launch some more, while two
// streams move 57 GB/s and the kernel 54, so the kernel is ahead while copies
// are small.  us by kernel / by DMA, 8 heads and 32 layers: 300 tokens 383 /
// 1354, 1024 tokens (1 MB a copy) 1157 / 1540, 3000 tokens (2.6 MB) 3330 / 3617,
// 8192 tokens (4.7 MB) 8336 / 8239; two heads (1.2 MB) 2258 / 2977.  The average
// counts payload and scale copies alike: over 190 streamed restores, 40 of them
// with one payload copy of 0.5-8 MB and one scale copy a layer, the choice is
// never behind DMA alone (at most 1.002 of its time).
bool pulls(const HostPlan& h) {
  const uint64_t copies = uint64_t(h.info.host_copies);
  return h.info.host_copy_bytes < copies * (4ull << 20) &&
         h.info.host_copy_bytes / kPullBytes < (uint64_t(1) << 28);
}
namespace {

// The pieces of one layer: the copies of layer_copies(), cut.
void cut_pieces(HostPlan& hp) {
  hp.pieces.clear();
  hp.pull_layer_bytes = 0;
  const auto cut = [&](uint64_t off, uint64_t stride, uint64_t len, uint32_t scales) {
    for (uint64_t o = 0; o < len; o += kPullBytes)
      hp.pieces.push_back(PullPiece{off + o, stride, uint32_t(std::min(len - o, kPullBytes)), scales});
    hp.pull_layer_bytes += len;
  };
  for (const RequestCopies& rc : hp.copies) {
    for (const CopyRange& c : rc.ranges) cut(rc.payload_offset + c.off, rc.layer_bytes, c.len, 0);
    if (rc.scales_needed) cut(rc.scale_offset * 2, rc.layer_scales * 2, rc.layer_scales * 2, 1);
  }
}

}  // namespace

pkv_status_t build_host_plan(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                             HostPlan* out) {
  pkv_status_t st = check_model(model);
  if (st != PKV_OK) return st;
  if (num_requests < 0 || (num_requests > 0 && !requests) || !out) return PKV_ERR_INVALID_ARGUMENT;
  const pkv_model_t& m = *model;
  const int64_t B = m.block_tokens, H = m.num_kv_heads, D = m.head_dim, P = m.page_size, L = m.num_layers;
  const int lp2 = ilog2(P);

  // Field, tag and page checks, request by request.
  for (int32_t r = 0; r < num_requests; ++r) {
    const pkv_request_t& q = requests[r];
    if ((st = check_request_fields(q)) != PKV_OK) return st;
    const int64_t nb = ceil_div(q.suffix_tokens, B);
    if ((st = check_tags(q, nb)) != PKV_OK) return st;
  }
  HostPlan& hp = *out;
  try {
    // Every page touched by a row of a reused block: in range, mapped, and
    // written through one (request, logical page) pair only.
    int64_t pages = 0;
    for (int32_t r = 0; r < num_requests; ++r) pages += (requests[r].suffix_tokens >> lp2) + 1;
    PageOwners owners(m.pool_pages, pages);
    for (int32_t r = 0; r < num_requests; ++r) {
      const pkv_request_t& q = requests[r];
      const int64_t nb = ceil_div(q.suffix_tokens, B);
      int64_t last_lp = -1;
      for (int64_t b = 0; b < nb; ++b) {
        if (q.repair_mask[b]) continue;
        const int64_t n_valid = std::min<int64_t>(B, q.suffix_tokens - b * B);
        const int64_t first_row = q.dst_row0 + b * B;
        const int64_t last_row = first_row + n_valid - 1;
        for (int64_t lp = std::max(first_row >> lp2, last_lp + 1); lp <= (last_row >> lp2); ++lp) {
          if (lp >= q.num_logical_pages) return PKV_ERR_PAGE_OUT_OF_RANGE;
          const int32_t pp = q.page_table[lp];
          if (pp == -1) return PKV_ERR_PAGE_UNMAPPED;
          if (pp < -1 || pp >= m.pool_pages) return PKV_ERR_PAGE_OUT_OF_RANGE;
          owners.mark(pp);
          last_lp = lp;
        }
      }
    }
    if (owners.twice()) return PKV_ERR_PAGE_ALIAS;
    if (int64_t(num_requests) * D > std::numeric_limits<int32_t>::max()) return PKV_ERR_INVALID_ARGUMENT;

    // Build: the work items of one layer, the cos/sin tables, what the
    // host-memory restores copy.
    hp.model = m;
    hp.log2_page = lp2;
    hp.units.clear();
    hp.rows.clear();
    hp.page_tables.clear();
    memset(&hp.info, 0, sizeof(hp.info));
    hp.info.num_requests = num_requests;
    hp.info.cache_bytes = cache_bytes(m);
    hp.req_payload_bytes.assign(size_t(num_requests), 0);
    hp.copies.assign(size_t(num_requests), RequestCopies());
    hp.tables.assign(size_t(num_requests) * size_t(D), 0.0);
    hp.workgroup = restore_workgroup(m);
    hp.rotated_rows = 0;
    hp.stage_ok = true;
    const int64_t per_unit = unit_tokens(m);
    std::vector<uint64_t> block_off;
    std::vector<CopyRange> reused;  // the reused blocks' K + V tiles, payload order
    int64_t pt_off = 0;
    for (int32_t r = 0; r < num_requests; ++r) {
      const pkv_request_t& q = requests[r];
      const int64_t nb = ceil_div(q.suffix_tokens, B);
      // cos / sin of Delta * f_i in double precision, laid out in the
      // kernel's element order: entry 8j + e is the pair that element e of
      // key piece j rotates (rope_table_pair); pass-through entries are (1, 0).
      for (int64_t k = 0; k < D / 2; ++k) {
        const int64_t i = rope_table_pair(m, k);
        const double ang = i >= 0 ? double(q.delta) * rope_frequency(m, i) : 0.0;
        hp.tables[size_t(r) * D + 2 * k] = q.delta && i >= 0 ? cos(ang) : 1.0;
        hp.tables[size_t(r) * D + 2 * k + 1] = q.delta && i >= 0 ? sin(ang) : 0.0;
      }
      RequestCopies& rc = hp.copies[size_t(r)];
      rc.unit0 = rc.unit1 = int64_t(hp.units.size());
      rc.payload_offset = q.payload_offset;
      rc.scale_offset = q.scale_offset;
      rc.layer_scales = uint64_t(nb) * H * 4;
      rc.layer_bytes = 0;
      rc.scales_needed = false;
      // Block offsets inside one layer (runs by tag, ascending blocks) and the
      // reused ones' ranges in that order, so that neighbours merge into one
      // copy; merging stays inside this request's layer, so copies never overlap.
      block_off.resize(size_t(nb));
      reused.clear();
      for (int tag = 0; tag < 4; ++tag) {
        const uint64_t len = tile_bytes(m, kKeyBits[tag]) + tile_bytes(m, kValueBits[tag]);
        for (int64_t b = 0; b < nb; ++b) {
          if (q.tags[b] != tag) continue;
          block_off[size_t(b)] = rc.layer_bytes;
          if (!q.repair_mask[b]) {
            reused.push_back(CopyRange{rc.layer_bytes, len});
            add_range(rc.ranges, 0, rc.layer_bytes, len, kHostGapBytes);
            rc.scales_needed |= tag != PKV_TAG_FP16;
          }
          rc.layer_bytes += len;
        }
      }
      if (rc.scales_needed && rc.layer_scales * 2 > kStageScaleBytes) hp.stage_ok = false;
      add_stage_windows(rc, reused);
      hp.req_payload_bytes[size_t(r)] = uint64_t(L) * rc.layer_bytes;
      if (nb > 0) {
        hp.info.payload_bytes =
            std::max<uint64_t>(hp.info.payload_bytes, q.payload_offset + uint64_t(L) * rc.layer_bytes);
        hp.info.scale_bytes =
            std::max<uint64_t>(hp.info.scale_bytes, (q.scale_offset + uint64_t(L) * rc.layer_scales) * 2);
      }
      for (int64_t b = 0; b < nb; ++b) {
        if (q.repair_mask[b]) continue;
        const int tag = q.tags[b];
        const int64_t n_valid = std::min<int64_t>(B, q.suffix_tokens - b * B);
        const uint64_t k_base = q.payload_offset + block_off[size_t(b)];
        const uint64_t v_base = k_base + tile_bytes(m, kKeyBits[tag]);
        // Split the block into units of at most `per_unit` tokens that
        // never cross a page boundary, so a unit writes slots of one page.
        // A page's run of rows is cut into equal parts (17 -> 9 + 8, not 16 + 1).
        for (int64_t t0 = 0, len = 0; t0 < n_valid; t0 += len) {
          const int64_t row = q.dst_row0 + b * B + t0, slot = row & (P - 1);
          const int64_t run = std::min<int64_t>(P - slot, n_valid - t0);
          len = ceil_div(run, ceil_div(run, per_unit));
          Unit u;
          u.k_off = k_base + uint64_t(t0) * H * D * kKeyBits[tag] / 8;
          u.v_off = v_base + uint64_t(t0) * H * D * kValueBits[tag] / 8;
          u.scale_off = q.scale_offset + uint64_t(b) * H * 4;
          u.payload_stride = rc.layer_bytes;
          u.meta = unit_meta(len, tag, q.delta != 0, uint64_t(nb) * H);
          u.ref = int64_t(r) * D;
          u.slot0 = int32_t(slot);
          u.page0 = q.page_table[row >> lp2];  // validated above; one page per unit
          u.page1 = u.page2 = 0;
          hp.units.push_back(u);
          if (hp.keep_rows) hp.rows.push_back(UnitRows{row, pt_off});
        }
        hp.info.restored_rows += n_valid;
        if (q.delta != 0) hp.rotated_rows += n_valid;
        hp.info.bytes_read += uint64_t(n_valid) * H * D * (kKeyBits[tag] + kValueBits[tag]) / 8;
        if (tag != PKV_TAG_FP16) hp.info.bytes_read += uint64_t(H) * 4 * 2;
      }
      rc.unit1 = int64_t(hp.units.size());
      pt_off += q.num_logical_pages;
    }
    // Every layer repeats the one built.
    hp.layer_units = int64_t(hp.units.size());
    hp.info.restored_rows *= L;
    hp.rotated_rows *= L;
    hp.info.bytes_read *= uint64_t(L);
    for (const RequestCopies& rc : hp.copies)
      for (const CopyRange& c : rc.ranges) {
        hp.info.host_copy_bytes += uint64_t(L) * c.len;
        hp.info.host_copies += L * int64_t((c.len + kHostChunkBytes - 1) / kHostChunkBytes);
      }
    std::vector<CopyRange> scales;
    for (int64_t l = 0; l < L; ++l) {
      scales.clear();
      layer_scale_copies(hp, l, scales);
      for (const CopyRange& c : scales) {
        hp.info.host_copy_bytes += c.len;
        hp.info.host_copies += int64_t((c.len + kHostChunkBytes - 1) / kHostChunkBytes);
      }
    }
    if (pulls(hp)) cut_pieces(hp);
  } catch (const std::bad_alloc&) {
    return PKV_ERR_OUT_OF_MEMORY;
  }
  if (hp.layer_units > std::numeric_limits<int32_t>::max() / L) return PKV_ERR_INVALID_ARGUMENT;
  hp.info.num_units = hp.layer_units * L;
  hp.info.bytes_written = uint64_t(hp.info.restored_rows) * H * D * 2 * 2;
  return PKV_OK;
}

int32_t gather_workgroup(const pkv_model_t& m) {
  return 64 * std::min<int32_t>(m.num_kv_heads, kGatherMaxWaves);
}

int32_t gather_loads(const pkv_model_t& m) {
  const int32_t rows = 64 / (m.head_dim / 8);  // per load
  return (m.block_tokens + rows - 1) / rows;
}

uint32_t gather_image(const pkv_model_t& m) {
  const uint64_t image = uint64_t(m.block_tokens) * m.num_kv_heads * m.head_dim;
  return gather_loads(m) <= 8 && m.num_kv_heads <= kGatherMaxWaves && image <= kTileImageMax ? uint32_t(image) : 0;
}

GatherLaunch gather_launch(const pkv_model_t& m, int64_t units) {
  GatherLaunch g;
  const int32_t nload = gather_loads(m);
  const int64_t tiles = units * 2 * m.num_kv_heads;
  g.loads = nload <= 2 ? 2 : nload <= 4 ? 4 : 8;
  g.split = g.group = 1;
  g.wide = m.block_tokens > 2 * m.page_size + 1 || layer_elems(m) * 2 >= (int64_t(1) << 32);
  g.grid = 0;
  const auto fits = [&](GatherLaunch::Kernel kernel, int64_t grid, int32_t threads) {
    if (grid * threads >= (int64_t(1) << 32)) return false;
    g.kernel = kernel;
    g.grid = uint32_t(grid);
    g.threads = threads;
    return true;
  };
  const int32_t wg = gather_workgroup(m);
  if (nload <= 8) {
    if (fits(GatherLaunch::kTile, ceil_div(tiles, wg / 64), wg)) return g;
  } else if (nload <= kSplitLoads * kGatherMaxWaves) {
    g.split = int32_t(ceil_div(nload, kSplitLoads));
    g.group = g.split < kSplitWaves ? kSplitWaves / g.split : 1;
    if (fits(GatherLaunch::kSplit, ceil_div(tiles, g.group), 64 * g.split * g.group)) return g;
  }
  if (!fits(GatherLaunch::kGeneral, 2 * units, wg)) g.kernel = GatherLaunch::kNone;
  return g;
}

int gather_workgroups_per_cu(const HostPlan& hp) {
  const pkv_plan_info_t& info = hp.info;
  const int waves = hp.workgroup / 64;
  if (gather_image(hp.model) == 0 || gather_loads(hp.model) != 8 || hp.model.head_dim % 128 != 0 || 16 % waves != 0 ||
      info.bytes_read == 0)
    return 0;
  // Rounds of the 24 waves a compute unit holds without a cap.
  if (2 * info.num_units * waves <= 8 * 24 * int64_t(hp.cus)) return 0;
  const double ratio = double(info.bytes_written) / double(info.bytes_read);
  return ratio >= 0.4 && ratio <= 0.85 ? 16 / waves : 0;
}

pkv_status_t build_checkpoint_plan(const pkv_model_t* model, const pkv_checkpoint_request_t* requests,
                                   int32_t num_requests, HostPlan* out) {
  pkv_status_t st = check_model(model);
  if (st != PKV_OK) return st;
  if (num_requests < 0 || (num_requests > 0 && !requests) || !out) return PKV_ERR_INVALID_ARGUMENT;
  const pkv_model_t& m = *model;
  const int64_t B = m.block_tokens, H = m.num_kv_heads, D = m.head_dim, P = m.page_size, L = m.num_layers;
  const int lp2 = ilog2(P);
  // Fields and tags.
  for (int32_t r = 0; r < num_requests; ++r) {
    const pkv_checkpoint_request_t& q = requests[r];
    if (q.reserved != 0 || q.reserved2 != 0) return PKV_ERR_INVALID_ARGUMENT;
    if (q.suffix_tokens < 0 || q.num_logical_pages < 0 || q.src_row0 < 0 || q.src_row0 > (int64_t(1) << 50))
      return PKV_ERR_INVALID_ARGUMENT;
    if (q.suffix_tokens > 0 && !q.tags) return PKV_ERR_INVALID_ARGUMENT;
    if (q.num_logical_pages > 0 && !q.page_table) return PKV_ERR_INVALID_ARGUMENT;
    if (q.payload_offset % 16 != 0 || q.scale_offset % 4 != 0) return PKV_ERR_INVALID_ARGUMENT;
    if (q.payload_offset > (uint64_t(1) << 56) || q.scale_offset > (uint64_t(1) << 56)) return PKV_ERR_INVALID_ARGUMENT;
    const int64_t nb = ceil_div(q.suffix_tokens, B);
    for (int64_t b = 0; b < nb; ++b)
      if (q.tags[b] > PKV_TAG_K4V4) return PKV_ERR_BAD_TAG;
  }
  // Every source row on a mapped, in-range page.
  for (int32_t r = 0; r < num_requests; ++r) {
    const pkv_checkpoint_request_t& q = requests[r];
    if (q.suffix_tokens == 0) continue;
    const int64_t first = q.src_row0 >> lp2, last = (q.src_row0 + q.suffix_tokens - 1) >> lp2;
    for (int64_t lp = first; lp <= last; ++lp) {
      if (lp >= q.num_logical_pages) return PKV_ERR_PAGE_OUT_OF_RANGE;
      const int32_t pp = q.page_table[lp];
      if (pp == -1) return PKV_ERR_PAGE_UNMAPPED;
      if (pp < -1 || pp >= m.pool_pages) return PKV_ERR_PAGE_OUT_OF_RANGE;
    }
  }
  // Output ranges of different requests must not overlap.
  std::vector<std::pair<uint64_t, uint64_t>> pr, sr;
  for (int32_t r = 0; r < num_requests; ++r) {
    const pkv_checkpoint_request_t& q = requests[r];
    const int64_t nb = ceil_div(q.suffix_tokens, B);
    if (nb == 0) continue;
    pr.emplace_back(q.payload_offset, q.payload_offset + uint64_t(L) * layer_payload_bytes(m, q.tags, nb));
    sr.emplace_back(q.scale_offset, q.scale_offset + uint64_t(L) * nb * H * 4);
  }
  for (auto* v : {&pr, &sr}) {
    std::sort(v->begin(), v->end());
    for (size_t i = 1; i < v->size(); ++i)
      if ((*v)[i].first < (*v)[i - 1].second) return PKV_ERR_INVALID_ARGUMENT;
  }

  HostPlan& hp = *out;
  hp.kind = 1;
  hp.workgroup = gather_workgroup(m);
  hp.model = m;
  hp.log2_page = lp2;
  hp.units.clear();
  hp.rows.clear();
  hp.tables.clear();
  hp.page_tables.clear();
  memset(&hp.info, 0, sizeof(hp.info));
  hp.info.num_requests = num_requests;
  hp.info.kind = 1;
  hp.info.cache_bytes = cache_bytes(m);
  try {
    hp.req_payload_bytes.assign(size_t(num_requests), 0);
    for (int32_t r = 0; r < num_requests; ++r) {
      const pkv_checkpoint_request_t& q = requests[r];
      const int64_t nb = ceil_div(q.suffix_tokens, B);
      const int64_t pt_off = int64_t(hp.page_tables.size());
      hp.page_tables.insert(hp.page_tables.end(), q.page_table, q.page_table + q.num_logical_pages);
      if (nb == 0) continue;
      std::vector<uint64_t> block_off(nb);
      uint64_t pos = 0;
      for (int tag = 0; tag < 4; ++tag)
        for (int64_t b = 0; b < nb; ++b)
          if (q.tags[b] == tag) {
            block_off[b] = pos;
            pos += tile_bytes(m, kKeyBits[tag]) + tile_bytes(m, kValueBits[tag]);
          }
      const uint64_t layer_bytes = pos;
      hp.req_payload_bytes[r] = uint64_t(L) * layer_bytes;
      hp.info.payload_bytes = std::max<uint64_t>(hp.info.payload_bytes, q.payload_offset + uint64_t(L) * layer_bytes);
      hp.info.scale_bytes = std::max<uint64_t>(hp.info.scale_bytes, (q.scale_offset + uint64_t(L) * nb * H * 4) * 2);
      for (int64_t b = 0; b < nb; ++b) {
        const int tag = q.tags[b];
        const int64_t row = q.src_row0 + b * B, n_valid = std::min<int64_t>(B, q.suffix_tokens - b * B);
        const int64_t first = row >> lp2, last = (row + n_valid - 1) >> lp2;
        Unit u;
        u.k_off = q.payload_offset + block_off[size_t(b)];
        u.v_off = u.k_off + tile_bytes(m, kKeyBits[tag]);
        u.scale_off = q.scale_offset + uint64_t(b) * H * 4;
        u.payload_stride = layer_bytes;
        u.meta = unit_meta(n_valid, tag, false, uint64_t(nb) * H);
        u.ref = pt_off + first;
        u.slot0 = int32_t(row & (P - 1));
        u.page0 = q.page_table[first];
        u.page1 = first + 1 <= last ? q.page_table[first + 1] : -1;
        u.page2 = first + 2 <= last ? q.page_table[first + 2] : -1;
        hp.units.push_back(u);
        if (hp.keep_rows) hp.rows.push_back(UnitRows{row, pt_off});
      }
      hp.info.bytes_written += uint64_t(L) * (layer_bytes + uint64_t(nb) * H * 4 * 2);
      hp.info.restored_rows += int64_t(L) * q.suffix_tokens;
    }
    hp.layer_units = int64_t(hp.units.size());
  } catch (const std::bad_alloc&) {
    return PKV_ERR_OUT_OF_MEMORY;
  }
  if (hp.layer_units > std::numeric_limits<int32_t>::max() / L) return PKV_ERR_INVALID_ARGUMENT;
  hp.info.num_units = hp.layer_units * L;
  hp.info.bytes_read = uint64_t(hp.info.restored_rows) * H * D * 2 * 2;
  return PKV_OK;
}

}  // namespace pkv

namespace {

// A work item of one layer in full, as the test hooks report it.
struct UnitView {
  uint64_t k_off, v_off, scale_off;
  int64_t row0, pt_off;
  int32_t table_off;  // checkpoint: the block's first page
  int32_t layer;
  int32_t tag;        // bits 0-7: pkv_tag_t; bit 8: rotate keys
  int32_t n_valid;
  int32_t page1, page2;  // restore: the unit's page and 0; checkpoint: the block's next two pages
};
static_assert(sizeof(UnitView) == 64, "UnitView layout");

// Every layer's work items, in launch order.
void unit_views(const pkv::HostPlan& hp, void* out) {
  UnitView* v = static_cast<UnitView*>(out);
  for (int32_t l = 0; l < hp.model.num_layers; ++l)
    for (size_t i = 0; i < hp.units.size(); ++i) {
      const pkv::Unit& u = hp.units[i];
      const bool write = hp.kind == 1;
      *v++ = UnitView{pkv::unit_k_off(u, uint32_t(l)), pkv::unit_v_off(u, uint32_t(l)),
                      pkv::unit_scale_off(u, uint32_t(l)), hp.rows[i].row0, hp.rows[i].pt_off,
                      write ? u.page0 : int32_t(u.ref), l, pkv::unit_tag(u) | (pkv::unit_rotates(u) ? 256 : 0),
                      pkv::unit_tokens_of(u), write ? u.page1 : u.page0, write ? u.page2 : 0};
    }
}

}  // namespace

extern "C" {

pkv_status_t pkv_payload_size(const pkv_model_t* model, const pkv_request_t* request, uint64_t* payload_bytes,
                              uint64_t* scale_elems) {
  pkv_status_t st = pkv::check_model(model);
  if (st != PKV_OK) return st;
  if (!request || !payload_bytes || !scale_elems) return PKV_ERR_INVALID_ARGUMENT;
  if (request->suffix_tokens < 0) return PKV_ERR_INVALID_ARGUMENT;
  const int64_t nb = pkv::ceil_div(request->suffix_tokens, model->block_tokens);
  if (nb > 0 && !request->tags) return PKV_ERR_INVALID_ARGUMENT;
  if ((st = pkv::check_tags(*request, nb)) != PKV_OK) return st;
  *payload_bytes = uint64_t(model->num_layers) * pkv::layer_payload_bytes(*model, request->tags, nb);
  *scale_elems = uint64_t(model->num_layers) * uint64_t(nb) * model->num_kv_heads * 4;
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): the host-built work list, so tests
// can check every address the kernel derives from it without a GPU.
pkv_status_t pkv_internal_host_units(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                                     void* units_out, int64_t capacity, int64_t* count) {
  if (!count) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  hp.keep_rows = true;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  *count = hp.info.num_units;
  if (units_out && capacity >= *count) unit_views(hp, units_out);
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): how launches of a plan run on a
// device of 256 compute units, as 5 int64: workgroups to a compute unit, late,
// one_round, device, single.  `layers` of the plan's layers at a time (0: all of them).
pkv_status_t pkv_internal_restore_launch(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                                         int64_t layers, uint64_t k_cache, uint64_t v_cache, int64_t* out) {
  if (!out) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  hp.cus = 256;
  hp.per_cu = pkv::restore_workgroups_per_cu(hp);
  const pkv::RestoreLaunch r = pkv::restore_launch(hp, layers ? layers * hp.layer_units : hp.info.num_units,
                                                   uintptr_t(k_cache), uintptr_t(v_cache));
  const int64_t v[5] = {hp.per_cu, r.late, r.one_round, r.device, r.single};
  memcpy(out, v, sizeof(v));
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): link_groups() for all layers, or for `units` work items if not 0.
pkv_status_t pkv_internal_link_groups(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                                      int64_t units, int64_t* groups) {
  if (!groups) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK || hp.info.num_units == 0) return PKV_ERR_INVALID_ARGUMENT;
  *groups = pkv::link_groups(hp, units ? units : hp.info.num_units);
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): threads per restore workgroup.
pkv_status_t pkv_internal_restore_workgroup(const pkv_model_t* model, int32_t* threads) {
  if (!model || !threads) return PKV_ERR_INVALID_ARGUMENT;
  *threads = pkv::restore_workgroup(*model);
  return PKV_OK;
}

pkv_status_t pkv_plan_repair(int32_t suffix_tokens, int32_t block_tokens, int64_t dirty_tokens,
                             const float* importance, double kappa, uint8_t* repair_mask, int64_t* nonlocal_tokens) {
  if (suffix_tokens < 0 || block_tokens < 1 || block_tokens > pkv::kMaxBlockTokens || dirty_tokens < 0)
    return PKV_ERR_INVALID_ARGUMENT;
  if (!(kappa >= 0.0 && kappa <= 1.0)) return PKV_ERR_INVALID_ARGUMENT;
  const int64_t N = suffix_tokens, B = block_tokens, nb = (N + B - 1) / B;
  if (N > 0 && (!importance || !repair_mask)) return PKV_ERR_INVALID_ARGUMENT;
  for (int64_t i = 0; i < N; ++i)
    if (!std::isfinite(importance[i])) return PKV_ERR_INVALID_ARGUMENT;
  const int64_t d = std::min<int64_t>(dirty_tokens, N);
  const int64_t candidates = N - d;
  int64_t k = int64_t(std::floor(kappa * double(candidates) + 0.5));
  k = std::min<int64_t>(std::max<int64_t>(k, 0), candidates);
  try {
    std::vector<uint8_t> mask(size_t(nb), 0);
    // Eq. 9: the dirty window D = [0, d) rounds to blocks [0, ceil(d / B)).
    for (int64_t b = 0; b < (d + B - 1) / B; ++b) mask[size_t(b)] = 1;
    // Eq. 11: the k best-scoring candidates (score descending, index ascending).
    if (k > 0) {
      std::vector<std::pair<float, int32_t>> cand(static_cast<size_t>(candidates));
      for (int64_t i = 0; i < candidates; ++i) cand[size_t(i)] = {importance[d + i], int32_t(d + i)};
      auto better = [](const std::pair<float, int32_t>& a, const std::pair<float, int32_t>& b) {
        return a.first > b.first || (a.first == b.first && a.second < b.second);
      };
      if (k < candidates) std::nth_element(cand.begin(), cand.begin() + (k - 1), cand.end(), better);
      for (int64_t j = 0; j < k; ++j) mask[size_t(cand[size_t(j)].second / B)] = 1;  // Eq. 12
    }
    std::copy(mask.begin(), mask.end(), repair_mask);
  } catch (const std::bad_alloc&) {
    return PKV_ERR_OUT_OF_MEMORY;
  }
  if (nonlocal_tokens) *nonlocal_tokens = k;
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): the (cos, sin) tables of a restore
// plan, [num_requests][D/2][2] in the kernel's element order.
pkv_status_t pkv_internal_host_tables(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                                      double* out, int64_t capacity, int64_t* count) {
  if (!count) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  *count = int64_t(hp.tables.size());
  if (out && capacity >= *count && *count > 0) memcpy(out, hp.tables.data(), hp.tables.size() * sizeof(double));
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): the gap below which the streamed
// restore merges two copies of one layer.
uint64_t pkv_internal_host_gap_bytes() { return pkv::kHostGapBytes; }

// Internal test hook (not part of pkv.h): the streamed restore's schedule.
// ranges_out receives (offset, length) byte pairs, payload ranges first,
// then scale ranges; layers_out receives [3][L + 1] starts: units, payload
// ranges, scale ranges.  Counts are returned even when the buffers are short.
pkv_status_t pkv_internal_stream_schedule(const pkv_model_t* model, const pkv_request_t* requests,
                                          int32_t num_requests, uint64_t* ranges_out, int64_t capacity,
                                          int64_t* n_payload, int64_t* n_scale, int64_t* layers_out) {
  if (!n_payload || !n_scale || !layers_out || !model) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  const int64_t L = model->num_layers;
  std::vector<pkv::CopyRange> payload, scales, all_payload, all_scales;
  for (int64_t l = 0; l <= L; ++l) {
    layers_out[l] = l * hp.layer_units;
    layers_out[L + 1 + l] = int64_t(all_payload.size());
    layers_out[2 * (L + 1) + l] = int64_t(all_scales.size());
    if (l == L) break;
    pkv::layer_copies(hp, l, payload, scales);
    all_payload.insert(all_payload.end(), payload.begin(), payload.end());
    all_scales.insert(all_scales.end(), scales.begin(), scales.end());
  }
  *n_payload = int64_t(all_payload.size());
  *n_scale = int64_t(all_scales.size());
  if (ranges_out && capacity >= *n_payload + *n_scale) {
    size_t k = 0;
    for (const auto* v : {&all_payload, &all_scales})
      for (const pkv::CopyRange& c : *v) {
        ranges_out[2 * k] = c.off;
        ranges_out[2 * k + 1] = c.len;
        ++k;
      }
  }
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): the pieces of one layer that the
// streamed restore's copy kernel takes, 4 uint64 each (byte offset, bytes from
// layer to layer, length, 1 for the scales); none where DMA copies are used.
pkv_status_t pkv_internal_pull_pieces(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                                      uint64_t* out, int64_t capacity, int64_t* count) {
  if (!count) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  *count = int64_t(hp.pieces.size());
  if (out && capacity >= *count)
    for (const pkv::PullPiece& p : hp.pieces) {
      const uint64_t v[4] = {p.off, p.stride, p.len, p.scales};
      memcpy(out, v, sizeof(v));
      out += 4;
    }
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): the schedule of the staged
// (allocation-free) restore.  steps_out receives 8 int64 per step (u0, u1,
// win_lo, win_hi, scale0, scale_elems, copy0, copy1), copies_out 3 uint64 per
// copy (src, dst, len); *stage_ok is 0 when the plan cannot be staged.
// Counts are returned even when the buffers are short.
pkv_status_t pkv_internal_stage_schedule(const pkv_model_t* model, const pkv_request_t* requests,
                                         int32_t num_requests, int64_t* steps_out, int64_t step_capacity,
                                         uint64_t* copies_out, int64_t copy_capacity, int64_t* n_steps,
                                         int64_t* n_copies, int32_t* stage_ok) {
  if (!n_steps || !n_copies || !stage_ok) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_host_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  *n_steps = *n_copies = 0;
  *stage_ok = hp.stage_ok ? 1 : 0;
  for (int64_t l = 0; hp.stage_ok && l < model->num_layers; ++l)
    for (const pkv::RequestCopies& rc : hp.copies)
      for (size_t w = 0; w < rc.windows.size(); ++w) {
        const pkv::StageStep s = pkv::stage_step(rc, l, w);
        const int64_t copy0 = *n_copies, u = l * hp.layer_units;
        for (int64_t c = rc.windows[w].copy0; c < rc.windows[w].copy1; ++c, ++*n_copies)
          if (copies_out && *n_copies < copy_capacity) {
            const pkv::StageCopy& cp = rc.stage_copies[size_t(c)];
            copies_out[3 * *n_copies] = s.payload_base + cp.src;
            copies_out[3 * *n_copies + 1] = cp.dst;
            copies_out[3 * *n_copies + 2] = cp.len;
          }
        if (steps_out && *n_steps < step_capacity) {
          const int64_t v[8] = {u + rc.unit0, u + rc.unit1, int64_t(s.win_lo), int64_t(s.win_hi), int64_t(s.scale0),
                                int64_t(s.scale_elems), copy0, *n_copies};
          memcpy(steps_out + 8 * *n_steps, v, sizeof(v));
        }
        ++*n_steps;
      }
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): gather_launch() as 7 int64: kernel,
// loads, split, group, threads, wide, grid.
pkv_status_t pkv_internal_gather_launch(const pkv_model_t* model, int64_t units, int64_t* out) {
  pkv_status_t st = pkv::check_model(model);
  if (st != PKV_OK || units < 1 || !out) return PKV_ERR_INVALID_ARGUMENT;
  const pkv::GatherLaunch g = pkv::gather_launch(*model, units);
  const int64_t v[7] = {g.kernel, g.loads, g.split, g.group, g.threads, g.wide, g.grid};
  memcpy(out, v, sizeof(v));
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): gather_workgroups_per_cu() on a device of 256 compute units.
pkv_status_t pkv_internal_gather_cap(const pkv_model_t* model, const pkv_checkpoint_request_t* requests,
                                     int32_t num_requests, int32_t* per_cu) {
  if (!per_cu) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  pkv_status_t st = pkv::build_checkpoint_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  hp.cus = 256;
  *per_cu = pkv::gather_workgroups_per_cu(hp);
  return PKV_OK;
}

// Internal test hook (not part of pkv.h): the work list of a checkpoint plan.
pkv_status_t pkv_internal_checkpoint_units(const pkv_model_t* model, const pkv_checkpoint_request_t* requests,
                                           int32_t num_requests, void* units_out, int64_t capacity, int64_t* count,
                                           int32_t* workgroup) {
  if (!count || !workgroup) return PKV_ERR_INVALID_ARGUMENT;
  pkv::HostPlan hp;
  hp.keep_rows = true;
  pkv_status_t st = pkv::build_checkpoint_plan(model, requests, num_requests, &hp);
  if (st != PKV_OK) return st;
  *count = hp.info.num_units;
  *workgroup = hp.workgroup;
  if (units_out && capacity >= *count) unit_views(hp, units_out);
  return PKV_OK;
}

const char* pkv_status_string(pkv_status_t s) {
  switch (s) {
    case PKV_OK: return "ok";
    case PKV_ERR_INVALID_ARGUMENT: return "invalid argument";
    case PKV_ERR_BAD_TAG: return "bad precision tag";
    case PKV_ERR_PAGE_OUT_OF_RANGE: return "page out of range";
    case PKV_ERR_PAGE_UNMAPPED: return "page unmapped";
    case PKV_ERR_PAGE_ALIAS: return "physical page written through two logical pages";
    case PKV_ERR_OUT_OF_MEMORY: return "out of memory";
    case PKV_ERR_DEVICE: return "device error";
  }
  return "unknown status";
}

}  // extern "C"
