// Internal launch interface between the C ABI layer (api.cpp) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace crisp {

constexpr int kHeadDim = 128;

// Shape-derived sizes shared by host and kernels.
struct Dims {
  int hq, hkv, G, n, B, nb, b;  // b = min(B, n) proxy rows
  int64_t cap;                  // nb * (nb + 1) / 2
};

// Estimator work split: each workgroup owns `bps` whole key blocks.
struct EstSplit {
  int bps;
  int splits;
};
EstSplit est_split(const Dims& d);

// Workspace layout (byte offsets; every region 256-byte aligned).
struct WsLayout {
  size_t rowstat, rowfinal, parts, masks, qbar, kbar, atil, rhist, rstate, rowinfo, sched, total;
};
WsLayout ws_layout(const Dims& d);

// Partial-result slots of the sparse kernel's schedule area (split rows): a caller's
// workspace provides up to kWorkspaceSlots; the library's own static area, used by the
// entry point that allocates nothing, up to kStaticSlots within kStaticSchedBytes.
constexpr int kWorkspaceSlots = 1024;
constexpr int kStaticSlots = 64;
constexpr size_t kStaticSchedBytes = (size_t)16 << 20;

// Bytes of the longest-first work list used by the persistent sparse kernel, with at
// most max_slots partial-result slots.
size_t attn_schedule_bytes(const Dims& d, int max_slots = kWorkspaceSlots);

// Device address of the library's static schedule area on the current device (its
// kStaticSchedBytes are a file-scope device array; each device holds its own copy).
hipError_t static_schedule_area(void** p);

// sched == nullptr: static grid (dense, or sparse without a work list); otherwise sched
// holds attn_schedule_bytes(d, max_slots) bytes.
hipError_t launch_attn(const Dims& d, float scale, const uint16_t* q, const uint16_t* k, const uint16_t* v,
                       const int32_t* row_ptr, const int32_t* col_idx, int64_t col_cap, bool dense,
                       uint16_t* o, void* sched, hipStream_t stream, int max_slots = kWorkspaceSlots);

// What the estimator leaves to launch_select, which then takes it from the workspace: kScores
// nothing (C_struct, p_v and p_s are written); kCombine p_v and p_s (C_struct and the per-row
// normalisers are written; layers of at most kFoldBlocks blocks).  kCombinePool: as kCombine,
// and the block means of all Q heads and KV groups were made beside the pass; kPool: C_struct
// is left as well (layers of at most kSmallSelectBlocks blocks).
enum class EstTail { kScores, kCombine, kCombinePool, kPool };
hipError_t launch_estimate(const Dims& d, float scale, int w_sink, int w_local, const uint16_t* q,
                           const uint16_t* k, float* c_struct, float* p_v, float* p_s, char* ws,
                           hipStream_t stream, EstTail tail = EstTail::kScores);

// Layers of at most this many blocks take the one-launch-per-head selection.
constexpr int kSmallSelectBlocks = 64;
// Up to this many blocks one workgroup per head selects from the pooled logits on, and in
// prefill forms the head's p_v and p_s from the estimator's sums.
constexpr int kFoldBlocks = 256;
// Up to this many query rows (heads x tokens) the pooling runs beside the estimator's pass,
// for every head (the routes are not known yet), and up to kSmallSelectBlocks blocks the
// combine inside the selection.  That saves one or two launches for the pooling of the VS
// heads' Q, which passes under the pass while Q is small or in the caches.  Whole prefill, apart / beside, us,
// inputs in the caches; and after 1 GiB of other writes: 4k tokens, 2 heads 73.1 / 67.3; 88.2 / 77.5.
// 32 heads: 2k 75.2 / 70.0; 89.5 / 81.0, 4k 117.5 / 112.9; 131.0 / 125.8, 8k (the limit) 316.1 / 310.9; 329.2 /
// 329.4.  16k, 16 heads (the limit) 522.0 / 519.5; 533.1 / 538.1.  Above it the launches saved no longer
// outweigh the reads of Q from HBM: 10k, 32 heads 515.8 / 512.0; 529.4 / 535.7, 16k, 32 heads 1036.6 /
// 1037.2; 1053.0 / 1064.3, 32k, 16 heads 1168.1 / 1167.5; 1191.0 / 1202.2.  The first pass of a fresh layer with
// its new buffers, by the host's clock: 2k 116.1 / 111.5, 8k 300.6 / 299.9.
constexpr int64_t kPoolBesideRows = 262144;

// route_score is C_struct (tau = tau_proxy) or D_JS (tau = tau_jsd); vs_mode 0 is the
// noise floor (floor_mode 0: mean, 1: median), 1 gamma coverage; kbar_all: K_bar of
// every KV group is already in ws.  tail: what launch_estimate on the same
// ws left to this call (route_score, p_v or p_s are then not read).
hipError_t launch_select(const Dims& d, float scale, float alpha, float tau, float gamma, int k_min, int vs_mode,
                         int floor_mode, bool kbar_all, const uint16_t* q, const uint16_t* k, const float* route_score,
                         const float* p_v, const float* p_s, int8_t* route, int32_t* row_ptr, int32_t* col_idx,
                         int64_t col_cap, uint8_t* dir_mask, char* ws, hipStream_t stream, EstTail tail = EstTail::kScores);

// route = dense and full causal CSR lists (col_cap >= nb (nb + 1) / 2).
hipError_t launch_dense_lists(const Dims& d, int8_t* route, int32_t* row_ptr, int32_t* col_idx, int64_t col_cap,
                              hipStream_t stream);

// D_JS per query head into jsd[hq]; leaves K_bar of every KV group in ws.
hipError_t launch_jsd(const Dims& d, float scale, const uint16_t* q, const uint16_t* k, const float* p_v,
                      float* jsd, char* ws, hipStream_t stream);

// Debug build only (CRISP_DEBUG): these wait for the stream.  *found = 1 if any of
// the n bf16 values is infinite or NaN; *code = 0 if every row of the lists keeps the
// list invariants, else 1 (row_ptr out of range or decreasing), 2 (an entry outside
// [0, qb]) or 3 (entries not strictly increasing).
hipError_t debug_nonfinite(const uint16_t* p, size_t n, hipStream_t stream, int* found);
hipError_t debug_lists(const Dims& d, const int32_t* row_ptr, const int32_t* col_idx, int64_t cap,
                       hipStream_t stream, int* code);

}  // namespace crisp
