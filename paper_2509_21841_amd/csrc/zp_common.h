// Shared device-side types and small helpers for the gfx950 kernels of the attention engine.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

#define ZP_LDS __attribute__((address_space(3)))

// One unit of attention work: a block of query rows against one run of keys of the same sequence.
// Whole sequences and (Q chunk, KV chunk) pairs (Sec. 3.2) both reduce to this.
struct zp_tile {
  int32_t q_tok0;    // first packed query token of the block
  int32_t q_rows;    // query rows in the block
  int32_t q_pos0;    // position of the first query row inside its sequence
  int32_t k_tok0;    // first packed token of the key run
  int32_t k_len;     // keys in the run
  int32_t k_pos0;    // position of the first key inside the sequence
  int32_t out_row0;  // first output row (packed token, or partial-result row)
  int32_t part;      // dK/dV: which share of the block's iterations (zp_part_of); 0: all of them. A record is 32 bytes
};

// dK/dV of a block of keys whose iterations several workgroups share: share `part` of `n`, whose sums lie at `slot` + part among
// all shares of the launch.
#define ZP_PART_MAX 63
struct zp_part {
  int part, n, slot;
};
inline int32_t zp_part_code(int part, int n, int slot) { return part | n << 6 | slot << 12; }
__device__ __forceinline__ zp_part zp_part_of(int32_t code) { return {code & 63, code >> 6 & 63, code >> 12}; }

// n / d for a wave-uniform n (any 32-bit value) on the scalar unit; m = zp_div_magic(d). The estimate falls short by one at
// most. (The compiler's division runs on the vector unit: some 30 dependent instructions in front of the tile record.)
inline uint32_t zp_div_magic(uint32_t d) { return 0xffffffffu / d; }
__device__ __forceinline__ int zp_udiv(int n, int d, uint32_t m) {
  const uint32_t q = __umulhi((uint32_t)n, m);
  return (int)((uint32_t)n - q * (uint32_t)d >= (uint32_t)d ? q + 1 : q);
}

// The tile record of a workgroup in scalar registers (it is the same for all its lanes, which the compiler cannot know
// where the item was claimed at run time: the record would come through the vector memory path and the tile copies'
// address arithmetic run on the vector unit). Tables are written before the kernel starts.
template <class P>
__device__ __forceinline__ zp_tile zp_load_tile(P p) {
  zp_tile t;
#define ZP_U(f) t.f = __builtin_amdgcn_readfirstlane(p->f)
  ZP_U(q_tok0); ZP_U(q_rows); ZP_U(q_pos0); ZP_U(k_tok0); ZP_U(k_len); ZP_U(k_pos0); ZP_U(out_row0); ZP_U(part);
#undef ZP_U
  return t;
}
// `idx` of the table in device memory (read through the scalar cache), or of the launch arguments (from `first` on) if
// there is none
#define ZP_TILE(tiles, inl, first, idx)                                                                            \
  ((tiles) ? zp_load_tile((const __attribute__((address_space(4))) zp_tile *)(uintptr_t)(tiles) + (idx))           \
           : zp_load_tile((inl).t + (first) + (idx)))
// The same for a launch that may have its sequences in its arguments (n_seq of them): the tile of their idx-th block of query rows, the
// last block of a sequence first, or of keys, the first block first.
#define ZP_TILE_OF(tiles, inl, n_seq, first, keys, idx) ((n_seq) ? zp_seq_tile((inl).words, n_seq, idx, keys) : ZP_TILE(tiles, inl, first, idx))

// A launch's tile table where it is short: in the launch arguments themselves (4 KB at most in all), so that nothing is
// uploaded in front of the launch.
#define ZP_INLINE_TILES 112
struct zp_inline_tiles {
  union {
    zp_tile t[ZP_INLINE_TILES];
    // or the sequences themselves (zp_put_seq): three words of each, then, 16 bits each, the sequence of every block
    uint32_t words[ZP_INLINE_TILES * 8];
  };
};

// Whole sequences, longest first, in launch arguments: their blocks of 128 rows are numbered through, and a workgroup works out the record
// of its own from the sequence's first token, length and first block.
#define ZP_SEQ_BLOCK 128
inline bool zp_seqs_fit(int64_t n_seq, int64_t n_blocks) { return n_seq * 12 + (n_blocks + 1) / 2 * 4 <= (int64_t)sizeof(zp_inline_tiles); }
// Host side: the i-th of n_seq sequences; returns the number of the first block behind it.
inline int zp_put_seq(zp_inline_tiles &inl, int n_seq, int i, int first, int32_t tok0, int32_t len) {
  uint32_t *w = inl.words + 3 * i;
  w[0] = (uint32_t)tok0; w[1] = (uint32_t)len; w[2] = (uint32_t)first;
  const int end = first + (len + ZP_SEQ_BLOCK - 1) / ZP_SEQ_BLOCK;
  for (int b = first; b < end; b++) inl.words[3 * n_seq + b / 2] |= (uint32_t)i << 16 * (b & 1);
  return end;
}
__device__ __forceinline__ zp_tile zp_seq_tile(const uint32_t *words, int n_seq, int block, bool keys) {
  const uint32_t two = __builtin_amdgcn_readfirstlane(words[3 * n_seq + (block >> 1)]);
  const uint32_t *w = words + 3 * ((block & 1) ? two >> 16 : two & 0xffff);
  const int tok0 = __builtin_amdgcn_readfirstlane(w[0]), len = __builtin_amdgcn_readfirstlane(w[1]);
  const int nth = block - __builtin_amdgcn_readfirstlane(w[2]), last = (len - 1) / ZP_SEQ_BLOCK;
  const int r0 = (keys ? nth : last - nth) * ZP_SEQ_BLOCK, rows = min(ZP_SEQ_BLOCK, len - r0);
  zp_tile t;
  t.q_tok0 = tok0 + r0; t.q_rows = keys ? len - r0 : rows; t.q_pos0 = r0;
  t.k_tok0 = keys ? tok0 + r0 : tok0; t.k_len = keys ? rows : len; t.k_pos0 = keys ? r0 : 0;
  t.out_row0 = tok0 + r0; t.part = 0;
  return t;
}

// How a launch hands its work items to workgroups. The XCDs of a chip do not run equally fast (on the cards measured
// the same four finish an equal share 4-8 % later than the other four), and the hardware deals workgroups to them
// round-robin, so with one item per workgroup the fast ones idle at the end. Items 0 .. n_static-1 are therefore taken
// by number (workgroup b runs item b, on XCD b % 8, no cost), and the last ones -- the cheapest of the launch -- are
// claimed at run time from one counter per XCD by the workgroups behind them, of which the launch holds more than
// there are items left: a workgroup whose own XCD has none left takes one from a neighbour, surplus workgroups exit.
// A claim costs its workgroup an atomic round trip (about a microsecond), so launches of light items claim the last
// eighth and launches of heavy items (dyn_div = 2) the last half.
// counters: 8 ints, ZP_COUNTER_STRIDE apart, zero before the launch. n_items and n_static are multiples of 8.
#define ZP_COUNTER_STRIDE 32
#define ZP_COUNTER_BYTES (8 * ZP_COUNTER_STRIDE * 4)
struct zp_work_split {
  int32_t *counters;
  int32_t n_items, n_static;
  int32_t dyn_div;  // 1 / dyn_div of the items are claimed at run time (0: the default, 8)
};
#define ZP_CLAIM_MIN_ITEMS (8 * 128)  // smaller launches take every item by number
// Host side: the split and the grid of a launch of n_items (a multiple of 8) items.
inline int zp_plan_work_split(zp_work_split &ws, int32_t *counters, int n_items) {
  ws.counters = counters;
  ws.n_items = n_items;
  if (n_items < ZP_CLAIM_MIN_ITEMS || counters == nullptr) {
    ws.n_static = n_items;
    return n_items;
  }
  const int div = ws.dyn_div >= 2 ? ws.dyn_div : 8;
  ws.n_static = (n_items / 8 * (div - 1) / div) * 8;
  const int n_dyn = n_items - ws.n_static;
  return ws.n_static + ((n_dyn * 3 / 2 + 7) / 8) * 8;
}
// Device side: the item of this workgroup, or -1 if there is none left for it. `slot` is one int of LDS. All threads
// of the workgroup must call it (it holds a barrier for the workgroups that claim).
__device__ __forceinline__ int zp_item_of_block(const zp_work_split &ws, int *slot) {
  const int b = blockIdx.x;
  if (b < ws.n_static) return __builtin_amdgcn_readfirstlane(b);
  if (threadIdx.x == 0) {
    const int per = (ws.n_items - ws.n_static) >> 3, x = b & 7;
    int item = -1;
    for (int j = 0; j < 8 && item < 0; j++) {
      const int y = (x + j) & 7;
      const int k = atomicAdd(ws.counters + y * ZP_COUNTER_STRIDE, 1);
      if (k < per) item = ws.n_static + 8 * k + y;
    }
    *slot = item;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*slot);
}

// The kernels that put two waves on every 16 query rows work on 64 rows at a time. Their table is in the launch arguments, as
// tiles of 64 rows (ordered by cost, none empty) where that many fit, else as the tiles of 128, whose halves are two workgroups.
enum zp_pair_mode { ZP_PAIR_NONE = 0, ZP_PAIR_TILES = 1, ZP_PAIR_HALVES = 2 };
// The item of workgroup b (halves: both on one XCD, the later rows first) and, of its tile, the 64 rows.
__device__ __forceinline__ int zp_pair_item(int mode, int b, int &half) {
  const int y = b >> 3;
  half = mode == ZP_PAIR_HALVES ? 1 - (y & 1) : 0;
  return mode == ZP_PAIR_HALVES ? (y >> 1) * 8 + (b & 7) : b;
}
__device__ __forceinline__ bool zp_pair_rows(zp_tile &t, int half) {
  if (64 * half >= t.q_rows) return false;
  t.q_tok0 += 64 * half; t.q_pos0 += 64 * half; t.out_row0 += 64 * half;
  t.q_rows = min(64, t.q_rows - 64 * half);
  return true;
}

// Parameters shared by the attention kernels. Strides are token strides in elements.
struct zp_attn_params {
  const __bf16 *q, *k, *v;
  int64_t q_stride, k_stride, v_stride;
  const zp_tile *tiles;
  int32_t n_tiles, Hq, Hkv, grp;
  uint32_t m_hkv, m_grp;  // zp_div_magic of Hkv and grp (set by the launcher)
  float scale_log2;  // scale * log2(e)
  float scale;
  void *o;           // bf16 [.][Hq][d] (whole) or float [part_rows][Hq][d] (partial)
  int64_t o_stride;  // token stride of o in elements
  float *lse;        // [Hq][lse_stride]
  int64_t lse_stride;
  int32_t update;    // partial kernel only: merge the result into the running (o, lse) found at the output rows
  int32_t pair;      // by the kernel for launches that leave much of the chip idle: zp_pair_mode
  int32_t n_seq;     // sequences in `inl`; 0: tiles
  int32_t turns;     // head dimension 128: by the kernel of three workgroups per CU
  zp_work_split work;  // which workgroups take their item by number and which claim one (set by the launcher)
  zp_inline_tiles inl; // the tile table if `tiles` is null
};
static_assert(sizeof(zp_attn_params) <= 4096, "kernel arguments are limited to 4 KB");

// Parameters of the two backward kernels. Strides as above.
struct zp_bwd_params {
  const __bf16 *q, *k, *v, *o, *dout;
  int64_t q_stride, k_stride, v_stride, o_stride, do_stride;
  const float *lse;   // [Hq][T]
  float *dvec;        // [Hq][T] scratch: -D_i = -(dO_i . O_i)
  float *lse2;        // [Hq][T] scratch: -LSE_i / scale
  float *parts;       // scratch: sums of the shares of shared blocks, [slot][Hkv][dK, dV of 128 rows]
  int32_t *part_done; // [slot][Hkv], zero before the launch: shares of the block that are done (at its first slot)
  const zp_tile *dq_tiles;
  const zp_tile *kv_tiles;
  int32_t n_dq_tiles, n_kv_tiles, Hq, Hkv, grp, T;
  uint32_t m_hkv, m_grp;  // zp_div_magic of Hkv and grp (set by the launcher)
  float scale_log2, scale;
  __bf16 *dq, *dk, *dv;      // outputs (bf16, overwritten) ...
  int64_t dq_stride, dkv_stride;
  int32_t dq_pair;           // dQ by the kernel for launches that leave much of the chip idle: zp_pair_mode
  int32_t kv_pair;           // dK/dV at head dimension 128 by workgroups of two groups of four waves
  int32_t n_seq;             // sequences in `inl`; 0: tiles
  int32_t share_its;         // iterations of a share of a shared block (its last one takes what is left)
  int32_t kv_split;          // dK/dV by the kernel for launches that leave most of the chip idle
  int32_t both;              // that and dq_pair in one launch (there: the workgroups of dK/dV, which come first)
  int32_t accumulate;        // ... or, when set, float accumulators of the same shapes that the results are ADDED to
  zp_work_split work_dq, work_kv;  // work hand-out of the two launches (counters set by the C ABI, the rest by the launcher)
  zp_inline_tiles inl;  // the dQ tiles and, behind them, the dK/dV tiles if dq_tiles and kv_tiles are null
};
static_assert(sizeof(zp_bwd_params) <= 4096, "kernel arguments are limited to 4 KB");

// blockIdx -> (unit, head-in-group). Workgroups are dealt to the 8 XCDs round-robin by blockIdx, so
// units (tile, kv head) are dealt round-robin too -- the cost-sorted list stays balanced across XCDs --
// while the grp query heads of one unit get consecutive slots on the SAME XCD and share K/V in its L2.
__device__ __forceinline__ void zp_block_to_unit(int bid, int grp, uint32_t m_grp, int &unit, int &hh) {
  const int x = bid & 7, y = bid >> 3, yq = zp_udiv(y, grp, m_grp);
  hh = y - yq * grp;
  unit = yq * 8 + x;
}

__device__ __forceinline__ float zp_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max / sum across the two lanes l and l^32 that hold the two halves of one 32x32 MFMA column.
__device__ __forceinline__ float zp_pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float zp_pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// max / sum across the four lanes l%16, +16, +32, +48 that hold one column of a 16x16 MFMA accumulator.
__device__ __forceinline__ float zp_quad_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return zp_pair_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float zp_quad_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return zp_pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// The gfx950 transposing 8-byte LDS read (ds_read_b64_tr_b16): within each group of 16 lanes, lane i passes the address of
// 4 consecutive 16-bit elements of row i/4, columns 4*(i%4)..+3 of a 4x16 block, and receives column i of rows 0..3.
__device__ __forceinline__ bf16x8 zp_cat(bf16x4 a, bf16x4 b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// The swizzle of tiles read as operands of the 16x16x32 MFMA: what the 16-byte chunk index of row `row` (r3 r2 r1 r0 in
// binary) is XORed with. Both read patterns touch each of the 64 banks once per phase of the LDS pipe:
//  - row-wise ds_read_b128 (lane l: row l%16, chunk c + l/16): a phase serves lanes 0-3, 12-15 and 20-27 (or the other
//    half of 0-31), that is eight rows with r2 == r3 at chunk c and the other eight at chunk c ^ 1; the map has to be
//    one-to-one both as it is and with r2 ^ r3 added to its lowest bit. (Rows 0-7 on the chunk pairs in order and rows
//    8-15 with the chunks exchanged is one-to-one only as it is: twice the LDS cycles, by counter.)
//  - transposing ds_read_b64_tr_b16 (32 lanes: 8 consecutive rows x 2 chunks): eight different chunk pairs (D = 64: four
//    in each 128-byte half).
template <int D>
__device__ __forceinline__ int zp_swz16_mask(int row) {
  const int x = ((row >> 2) ^ (row >> 3)) & 1, r3 = (row >> 3) & 1;
  if (D == 128) return (x << 3) | ((row & 3) << 1) | r3;
  return (x << 2) | (row & 2) | r3;
}

// The same bank pattern with the highest bit of the XOR turned into padding at D = 128: the chunk index is XORed with
// r1 r0 r3 only, and groups 1 and 2 of every four groups of four rows lie 128 bytes further (asynchronous copies write
// 1 KB, four rows, at a time and can put each anywhere). Read addresses of k-steps two apart and of 16-column blocks
// four apart then differ by a constant instead of an XOR, so that two and four registers per lane (row_part, tr_part)
// and immediate offsets reach everything. At D = 64 that many k-steps and blocks is all there are: zp_swz16 as it is.
template <int D>
struct zp_pad16 {
  static constexpr int ROWB = 2 * D, R16 = D == 128 ? 4096 + 256 : 2048;  // bytes of a row and of 16 rows
  __device__ __forceinline__ static int mask(int row) {
    return D == 128 ? ((row & 3) << 1) | ((row >> 3) & 1) : zp_swz16_mask<64>(row);
  }
  // offset of the g-th KB of rows (D = 128: four, 64: eight)
  __device__ __forceinline__ static int group(int g) {
    return D == 128 ? (g >> 2) * R16 + (g & 3) * 1024 + (((g & 3) + 1) >> 1) * 128 : g * 1024;
  }
  __device__ __forceinline__ static int row(int r) { return D == 128 ? group(r >> 2) + (r & 3) * 256 : r * ROWB; }
  // row operand of k-steps of parity `par` (k-step k: + k / 2 * 128), rows of the first 16
  __device__ __forceinline__ static int row_part(int lane, int par) {
    const int r = lane & 15, q = lane >> 4;
    return row(r) + (((4 * par + q) ^ mask(r)) << 4);
  }
  // transposed operand of 16-column blocks db with db % 4 == dq (db: + db / 4 * 128), first 16 rows (see zp_lds16::tr_at)
  __device__ __forceinline__ static int tr_part(int lane, int dq) {
    const int i = lane & 15, r = 4 * (lane >> 4) + (i >> 2);
    return row(r) + (((2 * dq + ((i >> 1) & 1)) ^ mask(r)) << 4) + ((i & 1) << 3);
  }
};

// ---- asynchronous global -> LDS copies -------------------------------------------------------------
// The direct-to-LDS loads are issued from inline assembly so that they stay truly asynchronous: the
// compiler does not track them, inserts no waits for them, and its workgroup barriers do not drain them.
// Ordering is explicit: zp_wait_async*() before the barrier that publishes a staged tile. Each lane's bytes
// land at (wave-uniform LDS base in M0) + lane * size. The compiler checks no hardware hazard for inline assembly,
// so each block pads itself: s_mov m0 plus s_nop 3 put five wait states between any vector instruction that
// wrote the scalar base (a v_readlane restoring a spilled SGPR, a v_readfirstlane) and the load that reads it,
// and cover the one wait state M0 needs before a direct-to-LDS load.
__device__ __forceinline__ unsigned zp_lds_addr(const void *p) {
  return (unsigned)(unsigned long long)(ZP_LDS const char *)p;
}
__device__ __forceinline__ void zp_dma16(const void *g, unsigned lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, off\n" ::"v"(g), "s"(lds_base_uniform) : "memory");
}
__device__ __forceinline__ void zp_dma4(const void *g, unsigned lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 3\n\tglobal_load_lds_dword %0, off\n" ::"v"(g), "s"(lds_base_uniform) : "memory");
}

// Copy of 64 consecutive floats (one per lane), issued by every wave of the workgroup to the same
// destination so that all waves have the same number of loads in flight.
__device__ __forceinline__ void zp_stage_async_f32x64(float *lds_dst, const float *gsrc, int first, int last_valid,
                                                      int lane) {
  int i = first + lane;
  if (i > last_valid) i = last_valid;
  zp_dma4(gsrc + i, __builtin_amdgcn_readfirstlane(zp_lds_addr(lds_dst)));
}
// wait for every outstanding vector-memory operation of this wave (vmcnt = 0), nothing else
__device__ __forceinline__ void zp_wait_async() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// wait until at most N vector-memory operations of this wave are outstanding (N compile-time, <= 63)
template <int N>
__device__ __forceinline__ void zp_wait_async_upto() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// 16-byte direct-to-LDS load addressed as (wave-uniform 64-bit base) + (per-lane 32-bit byte offset)
__device__ __forceinline__ void zp_dma16_so(const void *sbase_uniform, unsigned voff, unsigned lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1\n" ::"v"(voff), "s"(sbase_uniform),
               "s"(lds_base_uniform)
               : "memory");
}
// the same with 4 bytes per lane
__device__ __forceinline__ void zp_dma4_so(const void *sbase_uniform, unsigned voff, unsigned lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dword %0, %1\n" ::"v"(voff), "s"(sbase_uniform),
               "s"(lds_base_uniform)
               : "memory");
}
__device__ __forceinline__ const void *zp_uniform_ptr(const void *p) {
  unsigned long long v = (unsigned long long)p;
  unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (const void *)(((unsigned long long)hi << 32) | lo);
}

// Per-thread state of the asynchronous [64][D] tile copy: the lane's byte offsets inside a tile are worked
// out once (they carry the LDS swizzle); issuing a tile is then scalar address arithmetic plus the loads.
// `init` takes the tensor base of the row run and the token stride (64 * stride * 2 bytes must fit 32 bits);
// `issue` copies rows row0 .. row0+63 (rows past rows_total clamp to the last valid row).
// PAD: LDS layout of the tile, zp_pad16 instead of zp_swz16.
template <int D, int NW = 4, bool PAD = false>
struct zp_stager {
  static constexpr int PER_WAVE = 64 * D * 2 / 1024 / NW;  // 1 KiB wave-loads per wave (NW = 4: the four waves share a 64-row tile; NW = 8: they cover its first 32 rows)
  static constexpr int LOADS = PER_WAVE;
  unsigned off[PER_WAVE];  // bytes from the tile's first row
  int64_t stride;
  const __bf16 *base;
  int w, lane;
  __device__ __forceinline__ static void row_chunk(int blk, int lane, int &r, int &c) {
    r = D == 128 ? blk * 4 + (lane >> 4) : blk * 8 + (lane >> 3);
    c = (lane & (D / 8 - 1)) ^ (PAD ? zp_pad16<D>::mask(r) : zp_swz16_mask<D>(r));
  }
  // where in the LDS tile this wave's n-th load goes
  __device__ __forceinline__ int dest(int n) const {
    return PAD ? zp_pad16<D>::group(w * PER_WAVE + n) : (w * PER_WAVE + n) * 1024;
  }
  __device__ __forceinline__ void init(const __bf16 *gbase, int64_t tok_stride, int tid) {
    lane = tid & 63;
    w = __builtin_amdgcn_readfirstlane(tid >> 6);
    stride = tok_stride;
    base = gbase;
#pragma unroll
    for (int n = 0; n < PER_WAVE; n++) {
      int r, c;
      row_chunk(w * PER_WAVE + n, lane, r, c);
      off[n] = (unsigned)(((int64_t)r * tok_stride + c * 8) * 2);
    }
  }
  // extra: a wave-uniform element offset added to every source address (e.g. head * D)
  __device__ __forceinline__ void issue(char *lds_tile, int row0, int rows_total, int64_t extra = 0) const {
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(zp_lds_addr(lds_tile));
    if (__builtin_expect(row0 + 64 <= rows_total, 1)) {  // (the rest behind the loop around it)
      const void *sb = zp_uniform_ptr(base + (int64_t)row0 * stride + extra);
#pragma unroll
      for (int n = 0; n < PER_WAVE; n++) zp_dma16_so(sb, off[n], lds0 + dest(n));
    } else {
      int ln = lane;
      asm volatile("" : "+v"(ln));  // keeps the rare path's addresses out of the registers of the loop around it
#pragma unroll
      for (int n = 0; n < PER_WAVE; n++) {
        int r, c;
        row_chunk(w * PER_WAVE + n, ln, r, c);
        int gr = row0 + r;
        if (gr > rows_total - 1) gr = rows_total - 1;
        zp_dma16(base + (int64_t)gr * stride + c * 8 + extra, lds0 + dest(n));
      }
    }
  }
};

// LDS read addresses of one lane for the two operand patterns of the 16x16x32 MFMA on a [64][D] zp_swz16 tile. Lane l
// holds row (or column) l % 16 and the k-slots 8 (l / 16) .. + 7.
// rows_at(kb, kk): 16 bytes of row 16*kb + l%16, head-dim elements 32*kk + 8*(l/16) ..+7  (row-major operand)
// tr_at(kp, db): the transposed operand of 32 rows and 16 columns: column 16*db + l%16; k-slots 0-3 of the lane are rows
//   32*kp + 4*(l/16) ..+3, k-slots 4-7 the rows 16 further -- the order in which two accumulators of 16 rows each hold
//   their rows, so that a product's accumulators are the next product's other operand without moving between lanes.
template <int D>
struct zp_lds16 {
  static constexpr int ROWB = D * 2;
  int row_off[D / 32];
  int tr_off[D / 16];
  __device__ __forceinline__ void init_abs(int lane, const char *base) {
    const int r16 = lane & 15, q = lane >> 4;
    const int b = (int)(unsigned)(unsigned long long)(const ZP_LDS char *)base;
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) {
      row_off[kk] = b + r16 * ROWB + (((4 * kk + q) ^ zp_swz16_mask<D>(r16)) << 4);
      // opaque from here on: the compiler would otherwise split the sum again and redo the add at every read
      asm volatile("" : "+v"(row_off[kk]));
    }
    const int tr = 4 * q + (r16 >> 2);
#pragma unroll
    for (int db = 0; db < D / 16; db++) {
      tr_off[db] = b + tr * ROWB + (((2 * db + ((r16 >> 1) & 1)) ^ zp_swz16_mask<D>(tr)) << 4) + ((r16 & 1) << 3);
      asm volatile("" : "+v"(tr_off[db]));
    }
  }
  // moves all addresses by `bytes` (wave-uniform)
  __device__ __forceinline__ void move(int bytes) {
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) row_off[kk] += bytes;
#pragma unroll
    for (int db = 0; db < D / 16; db++) tr_off[db] += bytes;
  }
  __device__ __forceinline__ bf16x8 rows_at(int tile_off, int kb, int kk) const {
    return *(const ZP_LDS bf16x8 *)(unsigned long long)(unsigned)(row_off[kk] + tile_off + kb * 16 * ROWB);
  }
  __device__ __forceinline__ bf16x8 tr_at(int tile_off, int kp, int db) const {
    const int o = tile_off + kp * 32 * ROWB;
    s16x4 u0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)(unsigned)(tr_off[db] + o));
    s16x4 u1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)(unsigned)(tr_off[db] + o + 16 * ROWB));
    return zp_cat(__builtin_bit_cast(bf16x4, u0), __builtin_bit_cast(bf16x4, u1));
  }
};

// A lane's read addresses in a tile of the zp_pad16 layout; everything but these six is an immediate offset.
template <int D>
struct zp_pad16_addr {
  typedef zp_pad16<D> L;
  unsigned row[2], tr[4];
  __device__ __forceinline__ void init(int lane, const char *tile) {
#pragma unroll
    for (int par = 0; par < 2; par++) {
      row[par] = zp_lds_addr(tile) + L::row_part(lane, par);
      asm volatile("" : "+v"(row[par]));  // opaque: see zp_lds16
    }
#pragma unroll
    for (int dq = 0; dq < 4; dq++) {
      tr[dq] = zp_lds_addr(tile) + L::tr_part(lane, dq);
      asm volatile("" : "+v"(tr[dq]));
    }
  }
  __device__ __forceinline__ void move_rows(int bytes) {
#pragma unroll
    for (int par = 0; par < 2; par++) row[par] += bytes;
  }
  __device__ __forceinline__ void move_cols(int bytes) {
#pragma unroll
    for (int dq = 0; dq < 4; dq++) tr[dq] += bytes;
  }
  // off: byte offset of the tile; rb: 16 rows; k: k-step; db: 16 columns (of 32 rows)
  __device__ __forceinline__ bf16x8 rows(int off, int rb, int k) const {
    return *(const ZP_LDS bf16x8 *)(unsigned long long)(row[k & 1] + off + rb * L::R16 + (k >> 1) * 128);
  }
  __device__ __forceinline__ bf16x8 cols(int off, int db) const {
    const unsigned o = tr[db & 3] + off + (db >> 2) * 128;
    s16x4 u0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)o);
    s16x4 u1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)(o + L::R16));
    return zp_cat(__builtin_bit_cast(bf16x4, u0), __builtin_bit_cast(bf16x4, u1));
  }
};

// Writes 16 rows of bf16 results held as 16x16x32 MFMA accumulators (lane l: row l%16, columns 16 db + 4 (l/16) ..+3),
// scaled by mul, to dst, dst + stride, ... (n_valid rows of them). They pass through ZP_ROWS_LDS bytes of LDS of this wave's
// own, so that a store instruction covers whole rows (16 bytes per lane) instead of 16 rows' pieces of 32 bytes each: a
// quarter of the cache line accesses. (The pieces kept a workgroup's end busy for about 3 us on short sequences.)
#define ZP_ROWS_LDS_OF(D) (16 * (2 * (D) + 32))
#define ZP_ROWS_LDS ZP_ROWS_LDS_OF(128)
template <int D>
__device__ __forceinline__ void zp_store_rows(char *lds, const f32x4 (&acc)[D / 16], float mul, __bf16 *dst, int64_t stride,
                                              int n_valid, int lane) {
  constexpr int ROWB = D * 2 + 32, CPR = D / 8, RPI = 64 / CPR;  // 16-byte chunks per row, rows per store instruction
  ZP_LDS char *w = (ZP_LDS char *)lds + (lane & 15) * ROWB + (lane >> 4) * 8;
#pragma unroll
  for (int db = 0; db < D / 16; db++)
    *(ZP_LDS bf16x4 *)(w + db * 32) = bf16x4{(__bf16)(acc[db][0] * mul), (__bf16)(acc[db][1] * mul), (__bf16)(acc[db][2] * mul),
                                             (__bf16)(acc[db][3] * mul)};
  const int r0 = lane / CPR, c = lane % CPR;
#pragma unroll
  for (int i = 0; i < 16 / RPI; i++) {
    const int r = r0 + i * RPI;
    const bf16x8 v = *(const ZP_LDS bf16x8 *)((const ZP_LDS char *)lds + r * ROWB + c * 16);
    if (r < n_valid) *(bf16x8 *)(dst + (int64_t)r * stride + c * 8) = v;
  }
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <class F, int... I>
__device__ __forceinline__ void zp_static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void zp_static_for(F &&f) {
  zp_static_for_impl(f, std::make_integer_sequence<int, N>{});
}
