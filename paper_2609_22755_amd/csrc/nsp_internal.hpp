// Internal host/device interface of libnsp: per-item descriptors, work units
// and the kernel launchers.  Not part of the public ABI (include/nsp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nsp {

// One item of the work list in the attention layout.  Offsets are in
// elements of the respective tensor, 64-bit.
struct ItemDesc {
  int64_t q_off;    // Q / O / dO / dQ block: [L][hq][D]
  int64_t kv_off;   // K / V / dK / dV block: [L][hkv][D]
  int64_t lse_off;  // LSE / Delta block: [hq][L] (float32)
  int64_t q_row0;   // q_off / D: first D-row of the item in Q
  int32_t L;
  int32_t hq;
  int32_t hkv;
  int32_t active;   // 1 if the call computes this item (work-list item mask)
};

// Tile geometry shared by host scheduling and the kernels.
constexpr int kFwdWaves = 8;  // waves per forward / dQ workgroup (two per SIMD)
constexpr int kFwdBM = 32 * kFwdWaves;   // query rows per forward / dQ workgroup
constexpr int kFwdBN = 64;    // keys per inner iteration
constexpr int kBwdBN = 128;   // keys per dK/dV workgroup (4 waves x 32)
constexpr int kBwdBM = 64;    // query rows per dK/dV pipeline step (two 32-row sub-steps)
// Forward and dQ units of a call: 256 query rows by eight waves, 128 rows by four (two
// workgroups a compute unit), or 128 rows by eight in two groups that share the
// keys.
enum QKind { kQWhole = 0, kQHalf = 1, kQKeys = 2 };
// Consecutive LPT units placed on one XCD (about the workgroups an XCD runs at once).
constexpr int kXcdGroupFwd = 32;
// dK/dV unit tile field: 128-key tile index, and the flag of a unit that
// takes its query tiles from the item end down to the diagonal.
constexpr int kKvDescending = 1 << 30;
constexpr int kKvTileMask = kKvDescending - 1;
// Key-tile pairs per dK/dV gang (the workgroups one XCD runs at once).
constexpr int kKvGang = 32;

// Split dK/dV units (lists whose units would leave compute units idle, see
// kv_split in the schedule builder).  A piece is a run of a key tile's steps
// (ascending query tiles from the diagonal, the query heads of the group
// inner): all of them (slot < 0: the workgroup stores the gradients), or some,
// whose float32 sums go to a slot of the partial buffer.
struct KvPiece {
  int32_t item, tile, heads, g;   // as in a dK/dV unit, no direction flag
  int32_t first, count;           // steps
  int32_t slot, pad;
};
// A key tile in several pieces: its partial sums are slots slot .. slot+count-1.
struct KvReduce {
  int32_t item, tile, g, slot, count, pad[3];
};
// Floats of one slot: dK then dV of a 128-key tile.
constexpr int64_t kv_slot_floats(int D) { return 2 * (int64_t)kBwdBN * D; }
// Slots of the partial buffer: the cuts between 256 shares make at most 2 * 255
// pieces of cut tiles.  The buffer has this size for every list, so that a
// workspace of a larger list serves a smaller one.
constexpr int kKvSlots = 512;
constexpr size_t kv_part_bytes(int D) { return kKvSlots * (size_t)kv_slot_floats(D) * sizeof(float); }

// Work unit: int4 {item, tile, a, b}.
//   forward / dQ : a = local query head, b = local KV head
//   dK / dV      : a = first local query head | (end local query head << 16),
//                  b = local KV head
// The forward and dQ units of a schedule (device): per-XCD queues one after
// another, queue x is units[off[x] .. off[x+1]).
struct QPass {
  int4 *units = nullptr;
  int *off = nullptr;
  int n_units = 0;
  int longest = 0;         // entries of the longest queue
  int kind = kQWhole;      // QKind
  bool one_shot = false;   // one workgroup a unit, also with more units than fit at once
};

struct Schedule {
  ItemDesc *items = nullptr;   // device
  QPass fwd, dq;
  int4 *kv_units = nullptr;    // device, dK/dV units, per-XCD queues one after another
  int *kv_qoff = nullptr;      // device, 9 ints: queue x is kv_units[kv_qoff[x] .. kv_qoff[x+1])
  KvPiece *kv_pieces = nullptr;   // device, split dK/dV: the pieces, workgroup by workgroup
  int2 *kv_wgs = nullptr;         // device, workgroup b runs pieces kv_wgs[b].x .. kv_wgs[b].y - 1
  KvReduce *kv_reduce = nullptr;  // device, the key tiles in several pieces
  int n_kv_wgs = 0, n_kv_reduce = 0;
  bool small = false;             // dK/dV and dQ in one launch
  bool dq_first = false;          // dQ before dK/dV, with Delta, instead of a preprocess pass
  int n_items = 0;
  int n_kv_units = 0, kv_longest = 0;
  int64_t q_rows = 0;          // sum_j L_j * hq_j
  int64_t q_elems = 0, kv_elems = 0, lse_elems = 0;
};

struct AttnArgs {
  const void *q, *k, *v;
  const void *o;          // forward: output; backward: input
  void *o_out;
  float *lse;
  const float *lse_in;
  const void *dout;
  bool o_f32;             // backward: type of o (o is null for a dQ pass that reads delta and lse2)
  void *dq, *dk, *dv;
  float *delta;           // workspace: -Delta = -rowsum(dO * O)
  float *lse2;            // workspace: lse * log2(e)
  int *queue;             // workspace: unit queue heads, one per XCD and pass (zeroed before the pass)
  const ItemDesc *items;
  const int4 *units;
  const KvPiece *pieces;  // split dK/dV
  const int2 *wgs;
  const KvReduce *reduce;
  int n_reduce;
  bool small;             // with the split pass, dQ units (128-row ones) in the same launch
  float *part;            // split dK/dV: partial sums, kv_slot_floats a slot
  const int *qoff;        // start of each XCD's queue in `units`, and the end
  int q_longest;          // entries of the longest of them
  int q_kind;             // QKind of the units
  bool one_shot;          // one workgroup a unit, also with more units than compute units
  int n_items;
  float scale;            // softmax scale
  float scale_log2;       // softmax scale * log2(e)
};

// Re-layout copy task: move ntok runs of `cpt` 16-byte chunks.
// Byte offsets; replica r of the source lies at src + r * rep_stride.
struct CopyTask {
  int64_t dst, src;
  int64_t dst_ts, src_ts;   // bytes between consecutive tokens
  int64_t rep_stride;
  int32_t t0, ntok;
  int32_t cpt, nrep;
};

// Device scratch of the allocation-free backward: a schedule region, 256
// bytes of unit-queue heads, then -Delta and lse*log2(e) (float32, each part
// 256-byte aligned), then the partial sums of a split dK/dV pass.
constexpr size_t kScratchBytes = size_t(96) << 20;
constexpr size_t kScratchSchedBytes = size_t(8) << 20;
// The address of the current device's scratch (looked up once per device).
hipError_t noalloc_scratch(char **ptr);

// Record a thread-local error message (returned by nsp_last_error) and
// return `status`; also clears it when called with NSP_OK and no format.
int32_t set_error(int32_t status, const char *fmt, ...);

// Compute units of the current device (looked up once per device).
hipError_t compute_units(int *cus);

hipError_t launch_attn_fwd(int head_dim, bool o_f32, const AttnArgs &a, int n_units, hipStream_t s);
// One workgroup a dQ unit (a.units, of kind a.q_kind).
hipError_t launch_bwd_preprocess(int head_dim, bool o_f32, const AttnArgs &a, int n_units, hipStream_t s);
hipError_t launch_bwd_dq(int head_dim, bool g_f32, const AttnArgs &a, int n_units, hipStream_t s);
// With a.wgs the split pass (n_units workgroups over a.pieces, with a.small the
// dQ units of a.units too, then the sums of the a.n_reduce tiles of a.reduce),
// else the units of a.units.
hipError_t launch_bwd_dkdv(int head_dim, bool g_f32, const AttnArgs &a, int n_units, hipStream_t s);
hipError_t launch_relayout(const void *src, void *dst, const CopyTask *tasks, int n_tasks,
                           int sum_mode, hipStream_t s);

}  // namespace nsp
