// Internal structures shared by the host plan builder and the device kernel.
#ifndef PKV_INTERNAL_H
#define PKV_INTERNAL_H

#include <stdint.h>

#include <vector>

#include "pkv.h"

namespace pkv {

constexpr int kMaxHeadDim = 512;

// The hardware deals a launch's workgroups to the eight XCDs in turn
// (workgroup b runs on XCD b % 8), each XCD with its own L2.  Kernels take
// their work item from xcd_grouped(b, grid), which renumbers the workgroups
// so that kXcdGroup consecutive work items run on one XCD and share its L2
// (neighbouring payload tiles, scale lines, work items).  It is a permutation
// of [0, grid); the last, partial round of 8 * kXcdGroup keeps its order.
constexpr int64_t kXcdCount = 8;
constexpr int64_t kXcdGroup = 8;
constexpr int64_t xcd_grouped(int64_t b, int64_t grid) {
  const int64_t round = kXcdCount * kXcdGroup;
  if (b >= grid / round * round) return b;
  const int64_t slot = b / kXcdCount;
  return slot / kXcdGroup * round + (b % kXcdCount) * kXcdGroup + slot % kXcdGroup;
}
constexpr int kMaxRowElems = 4096;   // num_kv_heads * head_dim
constexpr int kMaxBlockTokens = 1024;
constexpr int kWorkgroup = 256;       // threads per workgroup
// Target output per unit: units of about 16K elements per cache (32 KiB of
// binary16/bfloat16) keep workgroups short, so the launch drains evenly.
constexpr int kUnitElems = 16384;

// Key / value bits per channel of each tag (Eq. 14 tiers plus uniform 4-bit).
constexpr int kKeyBits[4] = {16, 8, 8, 4};
constexpr int kValueBits[4] = {16, 8, 4, 4};

// Division of 32-bit numbers by a divisor known on the host, by a
// multiplication: with m = ceil(2^64 / d), floor(x / d) is the high word of
// x * m, exactly, for every x below 2^32 (the error x * (m * d - 2^64) stays
// below 2^64).  m = 0 stands for d = 1.
struct Divider {
  uint64_t m;
  uint32_t d;
};
constexpr Divider divider(uint32_t d) { return Divider{d == 1 ? 0 : ~uint64_t(0) / d + 1, d}; }
constexpr uint32_t divide(const Divider& v, uint32_t x) {
  return v.m == 0 ? x : uint32_t(((v.m >> 32) * x + ((v.m & 0xFFFFFFFFu) * x >> 32)) >> 32);
}

// The work items of a launch: `count` to a layer, from layer `first` on.  (A
// launch of one layer skips the division: it is on the way to the first load.)
struct LayerItems {
  Divider count;
  uint32_t first, layers;
};
constexpr LayerItems layer_items(int64_t first, int64_t layers, int64_t count) {
  return LayerItems{divider(uint32_t(count)), uint32_t(first), uint32_t(layers)};
}
constexpr uint32_t layer_of(const LayerItems& v, uint32_t item) { return v.layers == 1 ? 0 : divide(v.count, item); }

// One work item of one layer.  Restore: every head of up to n_valid consecutive
// tokens of one reused block of one request.  Checkpoint write: one whole block
// of one request.  The checkpoint and the caches repeat themselves layer by
// layer, so a plan holds the work items of layer 0 and the strides that lead to
// the other layers: work item w of a launch is item w % count of its layer
// w / count (LayerItems).  64 bytes.  (A list of every layer's items took 0.5-2 ms to build
// and upload for the 32- and 80-layer models, as long as the restore itself,
// and was read from HBM; one layer's takes 0.03-0.05 ms and stays in the L2s.)
struct Unit {
  uint64_t k_off;           // byte offset of the unit's first K row in the payload, layer 0
  uint64_t v_off;           // byte offset of its first V row, layer 0
  uint64_t scale_off;       // binary16-element offset of the block's (head 0, K, scale) entry, layer 0
  uint64_t payload_stride;  // payload bytes from one layer of the request to the next
  uint64_t meta;            // unit_meta(): tokens, tag, rotation, scale stride
  int64_t ref;              // restore: offset, in doubles, of the request's [D/2][2] (cos, sin) table;
                            //   checkpoint: index of the block's first page in the page tables
  int32_t slot0;            // slot of the unit's first row in its (first) page
  int32_t page0;            // physical page of the unit's rows, or of a checkpoint block's first rows
  int32_t page1, page2;     // checkpoint: the block's next two physical pages, -1 past its last page
};
static_assert(sizeof(Unit) == 64, "Unit layout");

// meta: bits 0-10 tokens of the unit, 11-12 pkv_tag_t, 13 rotate keys (Delta != 0),
// 16-63 the request's (block, head) pairs: the scale entries of one layer, four elements each.
constexpr uint64_t unit_meta(int64_t n_valid, int tag, bool rotate, uint64_t scale_entries) {
  return uint64_t(n_valid) | uint64_t(tag) << 11 | uint64_t(rotate) << 13 | scale_entries << 16;
}
constexpr int32_t unit_tokens_of(const Unit& u) { return int32_t(u.meta & 0x7FF); }
constexpr int32_t unit_tag(const Unit& u) { return int32_t(u.meta >> 11 & 3); }
constexpr bool unit_rotates(const Unit& u) { return (u.meta >> 13 & 1) != 0; }
constexpr uint64_t unit_k_off(const Unit& u, uint32_t layer) { return u.k_off + layer * u.payload_stride; }
constexpr uint64_t unit_v_off(const Unit& u, uint32_t layer) { return u.v_off + layer * u.payload_stride; }
constexpr uint64_t unit_scale_off(const Unit& u, uint32_t layer) { return u.scale_off + layer * (u.meta >> 16 << 2); }

#ifdef __HIPCC__
// sizeof(T) / 64 scalar loads of 64 bytes from `p`, all of them in registers
// before anything that uses them (the empty asm).  A workgroup's first load of
// data waits for its launch arguments and then for its work item.  Left alone
// the compiler loads both piece by piece, each where it is first used, seven
// scalar loads one behind the other; in one go each, units of several rows are
// restored up to 7% faster (one layer, 690 workgroups, launches back to back: 8.0
// us against 8.0-8.1).
typedef uint32_t ScalarLine __attribute__((ext_vector_type(16), aligned(4)));
template <typename T>
__device__ __forceinline__ T load_scalars(const __attribute__((address_space(4))) void* p) {
  static_assert(sizeof(T) == 64 || sizeof(T) == 128, "whole 64-byte loads");
  const auto* lines = static_cast<const __attribute__((address_space(4))) ScalarLine*>(p);
  if constexpr (sizeof(T) == 64) {
    ScalarLine a = lines[0];
    asm volatile("" : "+s"(a));
    return __builtin_bit_cast(T, a);
  } else {
    struct {
      ScalarLine a, b;
    } v{lines[0], lines[1]};
    asm volatile("" : "+s"(v.a), "+s"(v.b));
    return __builtin_bit_cast(T, v);
  }
}
// A kernel's arguments (its one parameter, of type T), and a work item.
template <typename T>
__device__ __forceinline__ T launch_args() {
  return load_scalars<T>((const __attribute__((address_space(4))) void*)__builtin_amdgcn_kernarg_segment_ptr());
}
__device__ __forceinline__ Unit load_unit(const Unit* u) {
  return load_scalars<Unit>((const __attribute__((address_space(4))) void*)(reinterpret_cast<uintptr_t>(u)));
}
#endif

// Where a unit sits in its request, kept only for the test hooks.
struct UnitRows {
  int64_t row0;    // logical row of the unit's first token (destination / old context)
  int64_t pt_off;  // index of the request's first page-table entry
};

struct CopyRange {
  uint64_t off, len;  // bytes
};
// Streamed restore: two copies of one layer whose ranges are at most this
// many bytes apart are merged into one (the repair blocks between them are
// copied too): one host -> device copy costs a fixed setup time that a gap
// of this size takes to transfer at link speed.
#ifndef PKV_HOST_GAP_BYTES
#define PKV_HOST_GAP_BYTES (512u << 10)
#endif
constexpr uint64_t kHostGapBytes = PKV_HOST_GAP_BYTES;
// Streamed restore: copy streams that copy chunks are dealt to.
#ifndef PKV_HOST_COPY_STREAMS
#define PKV_HOST_COPY_STREAMS 2
#endif
constexpr int kHostCopyStreams = PKV_HOST_COPY_STREAMS;
static_assert(kHostCopyStreams >= 1 && kHostCopyStreams <= 32, "copy streams are tracked in a 32-bit mask");
// Streamed restore: copies are cut into chunks of at most this many bytes,
// dealt to the copy streams by load.  One DMA stream alone moves ~40 GB/s;
// two busy together fill the host link (~57 GB/s).  Measured on the
// 8B-shaped 32-layer checkpoint: 16 MiB chunks on two streams 16.8 ms
// (uniform 4-bit) and 31.7 ms (mixed tags), against 33.2 / 33.0 ms with one
// stream and unchunked copies; 4 MiB chunks or four streams were no better.
#ifndef PKV_HOST_CHUNK_BYTES
#define PKV_HOST_CHUNK_BYTES (16ull << 20)
#endif
constexpr uint64_t kHostChunkBytes = PKV_HOST_CHUNK_BYTES;

// Streamed restore from host memory that the device can read in place: pieces
// of at most this many bytes, copied by a kernel (pull_kernel), each the same
// distance apart from layer to layer.
constexpr uint64_t kPullBytes = 64u << 10;
struct PullPiece {
  uint64_t off, stride;  // bytes into the payload or the scales: layer 0, and from layer to layer
  uint32_t len;
  uint32_t scales;       // 1: of the scales
};

// The allocation-free streamed restore stages a checkpoint that it cannot read in
// place through a static device buffer: payload windows in its first kStagePayloadBytes, one
// request-layer's scales in the kStageScaleBytes after them.
constexpr uint64_t kStagePayloadBytes = 64ull << 20;
constexpr uint64_t kStageScaleBytes = 4ull << 20;

// One window of that restore, of one request, relative to a layer's payload:
// the most consecutive reused blocks, in payload order, that span at most
// kStagePayloadBytes.  Payload byte o of the window sits at stage offset
// o - lo.  For each layer and request in turn, all on the caller's stream: the
// request-layer's scales and then each window's copies go from host memory into
// the stage, and the units whose K rows start in the window are restored.
struct StageWindow {
  uint64_t lo, hi;
  int64_t copy0, copy1;  // its payload copies in RequestCopies::stage_copies
};
struct StageCopy {
  uint64_t src;  // payload byte offset from the layer's start
  uint64_t dst;  // byte offset into the stage
  uint64_t len;
};

struct RequestCopies;
// One window of one layer, in absolute checkpoint offsets.
struct StageStep {
  uint64_t payload_base;    // payload byte the window's copies are relative to
  uint64_t win_lo, win_hi;  // payload bytes
  uint64_t scale0;          // binary16 element of the request-layer's scales
  uint64_t scale_elems;     // elements staged before this step (0: none; the stage already holds them)
};
StageStep stage_step(const RequestCopies& rc, int64_t l, size_t window);

// What the host-memory restores move for one request, the same in every layer.
struct RequestCopies {
  uint64_t payload_offset, layer_bytes;  // bytes
  uint64_t scale_offset, layer_scales;   // binary16 elements
  bool scales_needed;                    // some reused block is quantized
  int64_t unit0, unit1;                  // the request's units of a layer
  std::vector<CopyRange> ranges;         // merged payload copies, from the layer's start, ascending
  std::vector<StageWindow> windows;
  std::vector<StageCopy> stage_copies;
};

// Everything the plan needs on the device, built on the host.
struct HostPlan {
  int32_t kind = 0;  // 0 = restore, 1 = checkpoint write
  int32_t workgroup = kWorkgroup;
  pkv_model_t model;
  std::vector<Unit> units;         // of one layer, request by request
  std::vector<double> tables;      // per request [D/2][2]
  std::vector<int32_t> page_tables;  // checkpoint plans
  pkv_plan_info_t info;
  int32_t log2_page;
  int64_t layer_units = 0;                  // units.size(), kept when the list itself is dropped
  std::vector<RequestCopies> copies;        // restore plans, per request
  std::vector<PullPiece> pieces;            // restore plans that pull their copies (pulls()): those of one layer
  uint64_t pull_layer_bytes = 0;            // bytes of `pieces`
  int32_t cus = 0;     // compute units of the plan's device; 0 when it could not be queried
  int32_t per_cu = 0;  // restore plans: restore_workgroups_per_cu()
  int64_t rotated_rows = 0;  // restore plans: restored rows whose keys rotate (shift != 0)
  std::vector<uint64_t> req_payload_bytes;  // per request: bytes of its checkpoint payload, all layers
  // Restore plans: whether every request-layer's scales fit the staged restore's static buffer.
  bool stage_ok = false;
  bool keep_rows = false;  // test hooks: fill `rows`, one entry per unit
  std::vector<UnitRows> rows;
};

// Whether the streamed restore of a plan copies with a kernel (plan.cpp).
bool pulls(const HostPlan& hp);

// Copies of layer l of a streamed restore, in order: payload byte ranges and
// scale byte ranges (neighbouring requests' scales as one).
void layer_copies(const HostPlan& hp, int64_t l, std::vector<CopyRange>& payload, std::vector<CopyRange>& scales);

// Restore workgroups resident per compute unit, chosen per plan: 8 to 16
// waves (for 4-wave workgroups two to four, one wave per SIMD each; 16 waves
// is the register limit), 6 to 16 for narrow rows.  Measured on the 8B-shaped 32-layer restore,
// destination rows 7 slots into a page (units of 9, 16 and 7 tokens), us at
// 2 / 3 / 4 workgroups per CU, paired pages:
//   FP16 (read:write 1.00)  1200-1208 / 1233-1248 / 1240-1250
//   K8V8 (0.50)              889-892 /  915-916 /  956-958
//   mixed (0.47)             906-953 /  905-913 /  941-952
//   K8V4 (0.38)              861-867 /  836-837 /  884-885
//   K4V4 (0.25)              874-875 /      780 /  806-816
// separate caches:
//   FP16 1311-1325 / 1333-1347 / 1333-1349, K8V8 963 / 1041 / 1050-1053,
//   mixed 973-991 / 1015-1030 / 1039-1046, K8V4 907-908 / 954-957 / 979-980,
//   K4V4 895-896 / 851-856 / 896-899;
// and with page-aligned rows (16-token units), paired: mixed 891-898 /
// 952-961 / 965, K4V4 774-776 / 836-837 / 847: the best count falls as units
// grow.  Unshifted plans (no rotation, no table) run best with fewer.
// Rows narrow enough for workgroups under 256 threads, in either layout, want
// three quarters as much in flight, and more of it the less they read; us at
// 3 / 4 / 6 / 8 two-wave workgroups per CU (4 heads, units of 5.5K elements):
//   mixed 479 / 481 / 498 / 497,  FP16 620 / 640 / 652 / 649,  K4V4 444 / 406 / 425 / 429;
//   8 heads x 64, mixed 513 / 514 / 545 / 560;
// at 6 / 8 / 9 / 12 / 16 one-wave workgroups (units of 2.7K elements, one head of
// 128 on 32-token pages, 80 layers):
//   mixed 651 / 611 / 616 / 635 / 645,  FP16 812 / 836 / 847 / 856 / 847,
//   K4V4 656 / 551 / 531 / 523 / 537;
// two heads on 16-token pages: mixed 245 / 235 / 235 / 237 / 242.  Units of 1.4K
// elements and less (one head on 16-token pages, one-token pages) are fastest
// at the 16 waves the registers allow.  That count is too low for rotating rows
// of whole lines that read a half to 0.8 of a byte per byte written, and below
// that for launches that the 256 MB cache holds; mean of 19 to 54 drawn restores
// of 1, 2 and 4 heads of 128 and one of 256 over the fastest count of each, this
// rule / the one above:
//   0.49-0.8, writing up to 100 MB 1.02 / 1.10, to 300 MB 1.005 / 1.07, over 700 MB 1.01 / 1.04;
//   0.3-0.49, up to 100 MB 1.015 / 1.035, to 300 MB 1.01 / 1.03.
int restore_workgroups_per_cu(const HostPlan& hp);

// Launches that fit on the device at this many 256-thread workgroups to a
// compute unit are all resident at once, whatever cap the plan has for longer
// ones: one layer of the 8B-shaped restore (690 workgroups on 256 compute
// units, separate caches, launches back to back) takes 8.0 us at three and 8.9 at
// two, which leaves 178 for a second round.  At four to a compute unit 1012 workgroups were slower than at two
// (14.3 against 13.7 us).
constexpr int kOneRound = 3;

// How a launch of `units` restore work items into these caches runs.
struct RestoreLaunch {
  bool late;       // the late start order (Stage in restore.hip)
  bool one_round;  // kOneRound workgroups to a compute unit instead of HostPlan::per_cu
  bool device;     // stores at device scope
  bool single;     // work items of one row
};
RestoreLaunch restore_launch(const HostPlan& hp, int64_t units, uintptr_t k_cache, uintptr_t v_cache);

// Workgroups of a launch of `units` work items that reads the checkpoint over
// the host link and takes its items in a loop (restore_link_kernel); 0: an
// ordinary launch.  240 KB of reads in flight fill the link, so the workgroups are
// as many, in sixteens, as make that with one item each; at least 64 where the
// whole launch reads up to 8 MB, which it is over with soon.  8 layers of 4096
// tokens, 8 heads of 128, us with 16 / 32 / 64 / 128 / 256 workgroups, an ordinary
// launch, and copied into the stage in windows:
//   K8V4  817 / 858 / 803 / 802 / 811, 820, 1016    FP16  2182 / 2162 / 2132 / 2145 / 2389, 2439, 2359
// and two large layers (32768 tokens, 208 MB) of FP16 4364 / 4327 / 4265 / 4279 / 4756, 5079, 4475.
// Over 90 restores of all shapes these counts take 0.983 of the ordinary launch's
// time (4 over 1.05 of it; 350 to 500 KB in flight are 1.05-1.15), and products and
// additions of another stream beside one of them 245 us with 16 FP16 workgroups,
// 306 with 32, 483 / 731 / 763 with 64 / 128 / 256, 849 beside an ordinary launch and
// 172 alone.  Items under 1 KB (narrow rows on one-token pages) need thousands of
// workgroups, which an ordinary launch starts faster (8 layers, 64-byte items: 4.9
// times slower with 2048 in a loop); it takes them while it can hold them, fewer
// than 2^32 threads.
uint32_t link_groups(const HostPlan& hp, int64_t units);

// The same for the checkpoint write, 0 for no cap: staged tiles of 8 loads per
// lane (32-token blocks at head_dim 128) run best with 16 waves, 128 KB of
// loads, on a compute unit instead of the 24 that fit, while the checkpoint
// is between 0.4 and 0.85 of the cache rows it is read from.  Measured on the
// 8B-shaped 32-layer write, us with 24 / 16 waves (written / read in
// parentheses), 8 heads:
//   FP16 and K8V8 in halves (0.75)  1368 / 1293    K8V8 (0.50)             1097 / 1022
//   30% FP16, 70% K8V8 (0.65)       1277 / 1180    the mixed tags (0.47)   1094 / 1029
//   K8V4 (0.38)                     1019 / 1001    K8V4, K4V4 (0.31)        943 / 983
//   FP16 (1.00)                     1447 / 1454    K4V4 (0.25)              908 / 983
// four heads: mixed 551 / 525, K8V4 504 / 490, K4V4 452 / 474, FP16 707 / 743;
// heads of 256 gain the same.  Not so tiles whose lanes are not all busy (8 heads of 80
// and 96, 3 of 96, mixed tags: 1.03-1.12 of the uncapped time), heads of 64 (1.00-1.04),
// nor launches of up to about eight rounds of 24 waves (8 heads of 128: 1.01-1.07);
// one and two heads alike.  Tiles of 4 loads, and tiles split over several
// waves, measured level or slower with a cap, and so did workgroups whose waves
// do not make 16 (five heads: 647 at 24 waves, 755 at 15).
int gather_workgroups_per_cu(const HostPlan& hp);

// Validate and build the host side of a plan.  Makes no HIP call.
pkv_status_t build_host_plan(const pkv_model_t* model, const pkv_request_t* requests, int32_t num_requests,
                             HostPlan* out);

// Same for a checkpoint write (quantize-and-gather).
pkv_status_t build_checkpoint_plan(const pkv_model_t* model, const pkv_checkpoint_request_t* requests,
                                   int32_t num_requests, HostPlan* out);

// Checkpoint kernel: one wave per (head, K|V) tile of a block (larger tiles
// are dealt to several), at most kGatherMaxWaves waves per workgroup.
constexpr int kGatherMaxWaves = 16;
// A checkpoint unit carries the block's first three source pages, enough
// for every block when block_tokens <= 2 * page_size + 1; blocks on more
// pages are looked up in the page table.
constexpr int kUnitPages = 3;
int32_t gather_workgroup(const pkv_model_t& m);
// 16-byte loads per lane that cover a tile.
int32_t gather_loads(const pkv_model_t& m);
// Bytes of LDS in which a workgroup of the tile kernel assembles a tile of
// every head's codes before it writes them as one run; 0 where a workgroup is
// not one wave per head, a tile is more than 8 loads per lane or its 8-bit
// image more than kTileImageMax.  (Larger tiles staged whole in a workgroup
// per CU ran 18-20% slower on the 70B-shaped write: the barrier left the CU
// without loads in flight while it wrote.)
constexpr uint32_t kTileImageMax = 64u << 10;
uint32_t gather_image(const pkv_model_t& m);

// Which kernel a checkpoint write of `units` work items (all layers) takes, and its launch.
//   kTile   one wave per tile of at most 8 loads per lane, `loads` of them in registers (2, 4 or 8);
//   kSplit  tiles of 9 to 128 loads on `split` waves of kSplitLoads each, `group` tiles to a workgroup of about
//           kSplitWaves waves;
//   kGeneral  larger tiles, and writes whose tiles are more than one launch of the other two can hold (it takes
//           at most kGatherMaxWaves waves per block and cache, each looping over its heads, where those take one per
//           tile and more: with 256 heads of 16 they reach the limit 16 times sooner);
//   kNone   a launch is limited to 2^32 - 1 threads.
// `wide`: blocks on more than kUnitPages pages, and layer slices whose rows are out of a 32-bit offset's reach, look
// their pages up (load_tile).
constexpr int kSplitLoads = 8;
constexpr int kSplitWaves = 8;
struct GatherLaunch {
  enum Kernel : int32_t { kNone, kTile, kSplit, kGeneral } kernel;
  int32_t loads, split, group, threads;
  bool wide;
  uint32_t grid;
};
GatherLaunch gather_launch(const pkv_model_t& m, int64_t units);

// The plan object behind pkv_plan_t: host metadata and one piece of device memory (PlanMemory, or an allocation of its
// own where it is larger).
}  // namespace pkv
struct pkv_plan {
  pkv::HostPlan host;  // units, tables, page tables and pieces are dropped after upload
  void* device_mem = nullptr;
  pkv::Unit* d_units = nullptr;
  double* d_tables = nullptr;
  int32_t* d_page_tables = nullptr;
  int device = -1;
  // LDS bytes a workgroup claims so that at most restore_workgroups_per_cu() or
  // gather_workgroups_per_cu() of them are resident on a compute unit (0: no cap).
  uint32_t cap_lds = 0;
  // The same for restore launches in one round (RestoreLaunch::one_round).
  uint32_t one_round_lds = 0;
  // Streamed restore: copy streams and events (hipStream_t / hipEvent_t),
  // created on first use.  events[0] marks the caller's stream at entry;
  // events[1 + l * n + k] the end of layer l's chunks on copy stream k.
  std::vector<void*> copy_streams;
  std::vector<void*> events;
  // Pieces of one layer for pull_kernel (HostPlan::pieces), part of device_mem.
  pkv::PullPiece* d_pieces = nullptr;
  int64_t pull_pieces = 0;
};
namespace pkv {
// Copy a built host plan to device memory on the current device and wrap it.
pkv_status_t upload_plan(HostPlan&& hp, pkv_plan** out);

// Bytes of one layer of a request's checkpoint (tags already validated).
uint64_t layer_payload_bytes(const pkv_model_t& m, const uint8_t* tags, int64_t nb);

// Tokens per unit for a model: about kUnitElems output elements, at most one block.
int32_t unit_tokens(const pkv_model_t& m);
int32_t restore_workgroup(const pkv_model_t& m);

// Cache geometry by layout.  A page's slots start at page << page_shift slot
// rows from the layer's start (log2 P, plus one when a page holds its K and V
// slots back to back); a layer spans layer_elems elements of either cache.
int32_t page_shift(const pkv_model_t& m);
int64_t layer_elems(const pkv_model_t& m);
uint64_t cache_bytes(const pkv_model_t& m);  // of each separate cache, or of the paired one

// The cache pointers of a call against the model's layout: both 16-byte
// aligned; separate caches of cache_bytes each must not overlap; a paired
// cache has v_cache = k_cache + P*H*D elements.  `ranges` receives the byte
// ranges the caches occupy (two, or one for a paired cache) for overlap
// checks against other buffers; returns false on a bad placement.
struct ByteRange {
  const void* p;
  uint64_t n;
};
bool cache_ranges(const pkv_model_t& m, const void* k_cache, const void* v_cache, uint64_t bytes, ByteRange (&ranges)[2],
                  int& count);

// What kind of memory a kernel argument is (hipPointerGetAttributes), so that
// no launch ever gets a pointer the kernel would fault on.
//   kernel_accessible: device or managed memory of the plan's device as is,
//     or pinned host memory through its device mapping (*out receives the
//     address the kernel uses); pageable host memory or another device's
//     memory is PKV_ERR_INVALID_ARGUMENT.
//   device_resident: device or managed memory of the plan's device only.
pkv_status_t kernel_accessible(const pkv_plan* plan, const void* p, const void** out);
pkv_status_t device_resident(const pkv_plan* plan, const void* p);

}  // namespace pkv

#endif  // PKV_INTERNAL_H
