// Device-side building blocks for gfx950 (CDNA4): bf16 MFMA, LDS transpose
// reads and tile staging.
//
// MFMA v_mfma_f32_32x32x16_bf16 lane layout (one 64-lane wave):
//   A (32 x 16, M x K): lane l supplies row l%32, k = 8*(l/32) + j, j = 0..7
//   B (16 x 32, K x N): lane l supplies column l%32, k = 8*(l/32) + j
//   C (32 x 32):        lane l holds column l%32, element i holds
//                       row 8*(i/4) + 4*(l/32) + i%4
// Any permutation of k applied to A and B alike leaves the product unchanged;
// the kernels use that to feed the accumulator of one product (C layout) as
// the operand of the next without moving data between lanes.
//
// ds_read_b64_tr_b16: within each group of 16 lanes, lane i receives element
// i%4 of the 8-byte reads of lanes i/4 + 4e (e = 0..3).  If local lane j reads
// row r0 + j/4, columns c0 + 4*(j%4) .. +3 of a row-major tile, lane i gets
// rows r0..r0+3 of column c0 + i: the "transposed" MFMA operand, read
// straight from the row-major tile.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nsp {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x16 mfma32x32x16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x4 lds_read_tr4(const bf16 *p) {
  i16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)p);
  return __builtin_bit_cast(bf16x4, r);
}

__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// LDS tiles hold rows of D bf16 without padding; the 16-byte chunks of row r
// are permuted by an XOR with swz(r) so that the two read patterns of the
// kernels are free of bank conflicts on the 64 x 4-byte banks of the LDS:
//   * row reads (ds_read_b128, 16 lanes per cycle): 16 lanes read the same
//     logical chunk of 16 consecutive rows -> swz must be a bijection on
//     r mod 16 (D=128: one row per 256-byte bank line), or on (r/2) mod 8 for
//     each row parity (D=64: two rows per bank line);
//   * transpose reads (ds_read_b64_tr_b16, 32 lanes per cycle): rows r..r+3
//     (r a multiple of 4) x the aligned group of 4 chunks {q..q+3} -> the 4
//     rows must land in distinct 64-byte bank groups: swz(r+i) / 4 distinct
//     for i = 0..3 (D=128), or distinct for the two rows of each parity
//     (D=64).
template <int D>
__device__ __forceinline__ int swz(int r) {
  if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  else return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}

// Element offset of (row r, element column col) in a swizzled [rows][D] tile.
template <int D>
__device__ __forceinline__ int tile_off(int r, int col) {
  return r * D + ((((col >> 3) ^ swz<D>(r))) << 3) + (col & 7);
}

// Transposed operand for a 32-wide block of columns [c_blk, c_blk+32) and the
// 16 rows r_base + {4h..4h+3, 8+4h..8+4h+3} of a swizzled row-major LDS tile
// (h = lane/32).  Lane l receives column c_blk + l%32.  The row order matches
// the k order of an accumulator element block 8a..8a+7 (see the C layout
// above), so the result pairs with it in an MFMA.
template <int D>
__device__ __forceinline__ bf16x8 lds_tr_operand(const bf16 *tile, int r_base, int c_blk, int lane) {
  const int h = lane >> 5;
  const int g = lane >> 4;
  const int j = lane & 15;
  const int col = c_blk + 16 * (g & 1) + 4 * (j & 3);
  const int row = r_base + 4 * h + (j >> 2);
  bf16x4 lo = lds_read_tr4(tile + tile_off<D>(row, col));
  bf16x4 hi = lds_read_tr4(tile + tile_off<D>(row + 8, col));
  return cat4(lo, hi);
}

// Row operand: 8 consecutive elements [col, col+8) of row r of a swizzled tile
// (col a multiple of 8).
template <int D>
__device__ __forceinline__ bf16x8 lds_row8(const bf16 *tile, int r, int col) {
  return *(const bf16x8 *)(tile + tile_off<D>(r, col));
}

// Combine a per-lane value with the one of lane l^32 (the other half of the
// 32-wide MFMA column): v_permlane32_swap hands each lane its partner's value.
__device__ __forceinline__ float wave_max_halves(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float wave_sum_halves(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Buffer resource for raw (unformatted, unswizzled) loads from `base`: every
// byte offset below 2^31 is in range (callers keep offsets within their
// tensors).  Word 3 is the gfx9-family default for raw dword access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void *base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, 0x7fffffff, 0x00020000);
}

// Direct load of `bytes` (4 or 16) per lane from rsrc + voff into LDS: lane l
// lands at lds + bytes*l.  A buffer (MUBUF) load, not a global (FLAT) one: the
// compiler then still counts LDS reads precisely while such loads are in
// flight (with a FLAT one pending it waits for every outstanding LDS read).
template <int BYTES>
__device__ __forceinline__ void load_lds(__amdgpu_buffer_rsrc_t rs, unsigned voff, void *lds) {
  static_assert(BYTES == 4 || BYTES == 16, "load size");
  auto *dst = (__attribute__((address_space(3))) void *)lds;
  if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, voff, 0, 0, 0);
  else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 4, voff, 0, 0, 0);
}

// Buffer resource for rows r0.. of a tensor whose last valid row is L-1 (row
// stride `stride` elements, D elements used per row): the range ends with the
// data of row L-1, and is empty when r0 >= L.  An out-of-range buffer load
// returns zeros; with an LDS destination it writes zeros into LDS (checked on
// gfx950), and touches no memory.  Callers read at most kRsrcRows rows from
// r0, so the range is capped there (which keeps it in 32 bits); the
// arithmetic is branch-free scalar code, since a branch near the loads makes
// the compiler wait for every load in flight before the next LDS read.
constexpr int kRsrcRows = 1024;
template <int D>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const bf16 *src, int64_t stride, int r0, int L) {
  const int row_bytes = (int)stride * 2;
  const int bytes = max(0, min(L - r0, kRsrcRows) * row_bytes - (row_bytes - 2 * D));
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16 *>(src + (int64_t)r0 * stride), 0, bytes, 0x00020000);
}

// The same load issued as inline assembly (M0 = LDS base of lane 0; M0 is
// written only here in the kernels that use it).  The compiler does not see
// it, so it never adds waits of its own for LDS reads that it cannot tell
// apart from the load's destination; the caller orders the load against the
// reads of its LDS buffer (s_waitcnt vmcnt + workgroup barrier before reading,
// barrier before refilling).  The "memory" clobber keeps the compiler from
// moving other memory accesses across it.
template <int BYTES>
__device__ __forceinline__ void load_lds_untracked(__amdgpu_buffer_rsrc_t rs, unsigned voff, void *lds) {
  static_assert(BYTES == 4 || BYTES == 16, "load size");
  const unsigned m0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(rs)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(rs)
                 : "memory");
}

// Asynchronous copy of ROWS rows of D bf16 into an unpadded LDS tile
// [ROWS][D], by the NW waves of a workgroup, with direct buffer->LDS loads of
// 16 bytes per lane: each instruction moves 64 lanes x 16 bytes, lane l
// landing at the instruction's LDS base + 16*l (so one instruction fills
// 64/(D/8) consecutive rows).  Rows are r0 .. r0+ROWS-1 of a tensor with row
// stride `stride` elements; rows at or past L arrive as zeros (out-of-range
// loads, see rows_rsrc), so a tile wholly past L costs no memory traffic and
// the loads need no per-tile address arithmetic: each lane's byte offsets
// within a tile are fixed at construction.  `wave` must be wave-uniform.
// Completion: s_waitcnt vmcnt, then a workgroup barrier.
template <int D, int ROWS, int NW = 4>
struct TileLoader {
  static constexpr int LPR = D / 8;             // lanes per row
  static constexpr int RPI = 64 / LPR;          // rows per instruction
  static constexpr int PER_WAVE = ROWS / RPI / NW;
  static_assert(ROWS % (RPI * NW) == 0, "tile rows must split evenly over the waves");
  const bf16 *src;             // tensor base (row 0 of the item/head)
  int64_t stride;              // elements between rows
  unsigned voff[PER_WAVE];     // this lane's byte offset within a tile, per instruction
  int lds_off;                 // this wave's first LDS element within the tile

  // Lane l of instruction k fills LDS slot s = l % LPR of tile row
  // r = (first row of the wave) + l / LPR + k*RPI, so it fetches logical chunk
  // s ^ swz(r) of that row.
  __device__ __forceinline__ TileLoader(const bf16 *src_, int64_t stride_, int wave, int lane)
      : src(src_), stride(stride_) {
    const int row_base = wave * PER_WAVE * RPI + lane / LPR;
    const int slot = lane % LPR;
#pragma unroll
    for (int k = 0; k < PER_WAVE; ++k) {
      const int r = row_base + k * RPI;
      voff[k] = (unsigned)((r * (int)stride + ((slot ^ swz<D>(r)) & (LPR - 1)) * 8) * 2);
    }
    lds_off = wave * PER_WAVE * RPI * D;
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int r0, int L) const {
    return rows_rsrc<D>(src, stride, r0, L);
  }
  __device__ __forceinline__ bf16 *dst(bf16 *lds, int k) const { return lds + lds_off + k * RPI * D; }
  __device__ __forceinline__ void load(bf16 *lds, int r0, int L) const {
    const __amdgpu_buffer_rsrc_t rs = rsrc(r0, L);
#pragma unroll
    for (int k = 0; k < PER_WAVE; ++k) load_lds<16>(rs, voff[k], dst(lds, k));
  }
  __device__ __forceinline__ void load_untracked(bf16 *lds, int r0, int L) const {
    const __amdgpu_buffer_rsrc_t rs = rsrc(r0, L);
#pragma unroll
    for (int k = 0; k < PER_WAVE; ++k) load_lds_untracked<16>(rs, voff[k], dst(lds, k));
  }
};

// Row block of a wave: 32 rows of D bf16 between memory and the registers that
// the matrix products want (one row a lane, D/16 operands of 8 elements).
// Straight from memory such an access touches 32 rows an instruction, 16 bytes
// of each, and the address unit takes a cycle or more for every row: the query
// rows of a forward unit took 2.2 us and its stores 3.2 us of the 16 us that a
// unit of 300 tokens takes.  So rows go through LDS (in memory order, 16 bytes a
// lane, whole rows a few lanes wide), in a region of 32 * D elements that is the
// wave's own.
//
// Start the loads of rows r0 .. r0+31 (zeros at and past L; src, r0 and L
// uniform); after a wait for them, read_rows gives the operands.  (The lane is
// hidden from the compiler in all three, which would otherwise keep their
// per-lane addresses in registers from unit to unit.)
__device__ __forceinline__ int hidden(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
template <int D>
__device__ __forceinline__ void start_rows(const bf16 *src, int64_t stride, int r0, int L, bf16 *region, int lane) {
  const TileLoader<D, 32, 1> ld(src, stride, 0, hidden(lane));
  const uint64_t at = (uint64_t)(src + (int64_t)r0 * stride);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
  const int row_bytes = (int)stride * 2;
  const int bytes = __builtin_amdgcn_readfirstlane(max(0, min(L - r0, 32) * row_bytes - (row_bytes - 2 * D)));
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc((void *)((uint64_t)hi << 32 | lo), 0, bytes, 0x00020000);
#pragma unroll
  for (int k = 0; k < TileLoader<D, 32, 1>::PER_WAVE; ++k) load_lds_untracked<16>(rs, ld.voff[k], ld.dst(region, k));
}
template <int D>
__device__ __forceinline__ void read_rows(const bf16 *region, int lane_, bf16x8 *op) {
  const int lane = hidden(lane_);
#pragma unroll
  for (int k = 0; k < D / 16; ++k) op[k] = lds_row8<D>(region, lane & 31, 16 * k + 8 * (lane >> 5));
}

// Store the transposed accumulators acc[0 .. NB-1] (row = column of the output,
// column = output row, C layout), times mul, as 32 rows of 32 * NB elements
// from `out` on; only the first `rows` of them.  `region`: 32 * 32 * NB
// elements of LDS of the wave's own, 16-byte chunks swizzled by row.
template <int NB, bool F32>
__device__ __forceinline__ void store_rows(const f32x16 *acc, float mul, void *region, char *out, int64_t row_bytes,
                                           int rows, int lane_) {
  const int lane = hidden(lane_);
  constexpr int CH = NB * (F32 ? 8 : 4);       // 16-byte chunks a row
  const int l32 = lane & 31, h = lane >> 5;
  char *lds = (char *)region;
#pragma unroll
  for (int mb = 0; mb < NB; ++mb)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const f32x4 v = {acc[mb][4 * gq] * mul, acc[mb][4 * gq + 1] * mul, acc[mb][4 * gq + 2] * mul,
                       acc[mb][4 * gq + 3] * mul};
      const int c = F32 ? 8 * mb + 2 * gq + h : 4 * mb + gq;
      char *p = lds + 16 * (l32 * CH + (c ^ (l32 & (CH - 1))));
      if constexpr (F32) *(f32x4 *)p = v;
      else *(bf16x4 *)(p + 8 * h) = bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
    }
#pragma unroll
  for (int j = 0; j < CH / 2; ++j) {
    const int row = (64 * j + lane) / CH, c = (64 * j + lane) % CH;
    const f32x4 v = *(const f32x4 *)(lds + 16 * (row * CH + (c ^ (row & (CH - 1)))));
    if (row < rows) *(f32x4 *)(out + row * row_bytes + 16 * c) = v;
  }
}

// s_waitcnt: at most n buffer->LDS loads of this wave still in flight, no LDS
// operation in flight.  (gfx9 encoding: vmcnt[3:0] and [15:14], expcnt[6:4],
// lgkmcnt[11:8].)
template <int N>
__device__ __forceinline__ void wait_loads_le() {
  static_assert(N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

// Workgroup barrier that leaves the loads of later stages in flight (unlike
// __syncthreads, whose fence waits for every outstanding memory operation).
// The empty asm statements keep the compiler from moving LDS accesses across.
__device__ __forceinline__ void stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The value, computed at this point of the instruction stream: an empty
// volatile asm that takes and returns it in a VGPR, which the compiler keeps
// in order with the scheduling fences around it.
__device__ __forceinline__ float pin(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The wave index as a scalar (wave-uniform) value.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Wait for this wave's LDS (and scalar) operations only.
__device__ __forceinline__ void wait_lds() { wait_loads_le<63>(); }

// Per-XCD unit queues of a pass: queue x holds the units off[x] .. off[x+1]-1
// of the unit list.  Without heads workgroup b runs entry b / 8 of queue b % 8:
// workgroups go to the XCDs in turn, so that a queue's units share one.  With
// heads (ints in device memory, zero before the pass; entries taken) a workgroup
// takes units until every queue is empty.  It drains the queue of its own XCD
// first -- keeping the gangs of the order, and their L2 reuse, on one XCD -- then
// takes what is left in the others: XCDs run at different speeds, and a fixed
// unit-to-XCD map would leave the fast ones idle at the end.
//
// The first unit too comes from the queue of the XCD that the workgroup runs on,
// not from queue b % 8: which XCD workgroup 0 goes to depends on the hardware
// queue of the stream (XCD 7 on one stream of a process that uses two), and the
// leading units of the gangs then ran on another XCD than the rest of them.  dK/dV
// of one sequence of 4 / 1 heads (D = 128) on such a stream, entry b / 8 / fetched:
// 513 key tiles 8648 / 7574 us, 594 11722 / 10098, 704 14658 / 13364; forward of
// 594 4856 / 4746.  Where workgroup 0 is on XCD 0, 594 tiles: 10129 / 10117 and
// 4737 / 4745 (the fetch).
//
// One wave fetches.  The atomics go to memory past the XCDs' L2, about 1 us
// each, so the eight heads are read together to see which queue has units
// left: adding to eight empty queues in turn took 15 to 20 us at the end of a
// pass (12 items of 512 tokens, forward: 69 us, one workgroup a unit 51 us).
// Asking for the next unit while one runs was no faster: a unit taken that
// early is not there for the compute unit that goes idle first (32 items of
// 2048 tokens, forward: 1343 us against 1248).  Heads only grow, and a queue
// found empty is not asked again, so every workgroup stops after at most
// n_units + 8 fetches.
constexpr int kXcdQueues = 8;
// s_getreg operand for HW_REG_XCC_ID (register 20, bits 0..15): the XCD a
// wave runs on
constexpr int kHwRegXccId = 20 | (0 << 6) | ((16 - 1) << 11);

struct UnitQueue {
  int *heads;
  const int *off;
  int *s_slot;         // in LDS
  unsigned empty;      // queues found empty

  __device__ __forceinline__ UnitQueue(int *heads_, const int *off_, int *s_slot_)
      : heads(heads_), off(off_), s_slot(s_slot_), empty(0) {}
  __device__ __forceinline__ int count(int x) const { return off[x + 1] - off[x]; }

  // The next unit of the own queue, or of the first one after it that is not
  // empty (-1: none).  By a whole wave: lane x looks at queue x.
  __device__ __forceinline__ int fetch() {
    const int lane = threadIdx.x & 63, own = (int)(__builtin_amdgcn_s_getreg(kHwRegXccId) % kXcdQueues);
    int y = own;
    for (;;) {
      if (!(empty >> y & 1)) {
        int k = 0;
        if (lane == 0) k = atomicAdd(heads + y, 1);
        k = __builtin_amdgcn_readfirstlane(k);
        if (k < count(y)) return off[y] + k;
        empty |= 1u << y;
      }
      const int x = lane & 7;
      const int h = __hip_atomic_load(heads + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned left = (unsigned)__ballot(h < count(x)) & 0xffu & ~empty;
      if (left == 0) return -1;
      y = (own + __builtin_ctz((left | left << kXcdQueues) >> own)) % kXcdQueues;
    }
  }
  // The workgroup's first unit (-1: none).
  __device__ __forceinline__ int first() {
    if (heads) return next();
    const int x = (int)blockIdx.x % kXcdQueues, i = (int)blockIdx.x / kXcdQueues;
    return i < count(x) ? off[x] + i : -1;
  }
  // Its next unit (-1: none).  Also the barrier between a unit's last LDS
  // accesses and the next unit's first; stores to memory stay in flight across
  // it.
  __device__ __forceinline__ int next() {
    if (!heads) return -1;
    if (wave_id() == 0) {
      const int s = fetch();
      if (threadIdx.x == 0) *s_slot = s;
    }
    wait_lds();
    stage_barrier();
    return __builtin_amdgcn_readfirstlane(*s_slot);
  }
};

// Wait for this wave's outstanding global (and LDS) operations.
__device__ __forceinline__ void wait_all_loads() { __builtin_amdgcn_s_waitcnt(0); }

}  // namespace nsp
