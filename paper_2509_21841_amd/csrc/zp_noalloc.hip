// varlen_attn_fwd for callers that cannot allocate or upload: the ordered tile table of the forward kernel is
// built ON the device, from sequence boundaries passed by value in the launch arguments, into a file-scope device
// array. Nothing is allocated, no host buffer is read by the device, so the call can sit under HIP graph capture or in
// a serving loop that forbids hipMalloc. The attention kernel itself is the one varlen_attn_fwd launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "../../include/zeppelin_attn.h"
#include "zp_common.h"
#include "zp_pair.h"

extern "C" int zp_launch_attn_fwd(const zp_attn_params *p, int d, int partial, int block_rows, hipStream_t stream);
extern "C" int zp_attn_fwd_block_rows(int d);
extern "C" int zp_report_hip_error(int hip_error, const char *what);

// The forward kernel's work counters (ZP_COUNTER_BYTES) and its tile table: ZP_NOALLOC_MAX_TILES records of 32 bytes. One copy per GPU the library runs on, held until the
// process ends. In host code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[ZP_COUNTER_BYTES + (size_t)ZP_NOALLOC_MAX_TILES * sizeof(zp_tile)];

namespace {

constexpr int BM = 128;  // query rows per tile (the forward kernel's block)

// Launch arguments of the planning kernel: the batch description by value (under 4 KB of kernel arguments).
struct PlanArgs {
  int32_t S;
  int32_t n_tiles;
  int32_t cu[ZP_NOALLOC_MAX_SEQS + 1];
  uint32_t skip_bits[(ZP_NOALLOC_MAX_SEQS + 31) / 32];
};
static_assert(sizeof(PlanArgs) + sizeof(void *) <= 4096, "kernel arguments are limited to 4 KB");

// Query blocks of sequence s (none if it is flagged).
__device__ __forceinline__ void seq_blocks(const PlanArgs &a, int s, int &L, int &n_blk) {
  const bool skip = (a.skip_bits[s >> 5] >> (s & 31)) & 1u;
  L = a.cu[s + 1] - a.cu[s];
  n_blk = skip ? 0 : (L + BM - 1) / BM;
}

// One thread per tile, in the order the host planner of varlen_attn_fwd uses: sequence by sequence, longest first
// (equal lengths: lower index first), inside a sequence the last query block first. Tile (s, b) therefore sits behind
// all blocks of the sequences ordered before s and behind the later blocks of s -- a closed form, so no sort and no
// atomics, and the table is the same on every call.
static_assert(ZP_NOALLOC_MAX_SEQS % 4 == 0, "lengths are read four at a time");
constexpr int PLAN_NT = 256;
__global__ __launch_bounds__(PLAN_NT) void plan_fwd_tiles_kernel(PlanArgs a, int32_t *counters, zp_tile *tiles) {
  constexpr int PER = (ZP_NOALLOC_MAX_SEQS + PLAN_NT - 1) / PLAN_NT;
  __shared__ int __align__(16) length[ZP_NOALLOC_MAX_SEQS], first_tile[ZP_NOALLOC_MAX_SEQS + 1], wave_sum[PLAN_NT / 64];
  // the attention kernel's work counters start from zero on every call
  if (blockIdx.x == 0 && threadIdx.x < 8) counters[threadIdx.x * ZP_COUNTER_STRIDE] = 0;
  // A running sum over the sequences, PER of them per thread: over a wave's lanes, then over the waves. The lengths go to LDS, from where
  // every tile compares four with its own at a time. Bound: that loop's chain (read from the launch arguments one sequence after the other,
  // and with the sum by one thread, 768 sequences kept the attention kernel waiting for some 90 us: 57928 tokens, 32/8 heads, d = 128,
  // the whole call 427 us, now 376; with the table from the host 335).
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, s0 = threadIdx.x * PER;
  int blocks[PER], mine = 0;
#pragma unroll
  for (int j = 0; j < PER; j++) {
    int L = 0;
    blocks[j] = 0;
    if (s0 + j < a.S) seq_blocks(a, s0 + j, L, blocks[j]);
    if (s0 + j < ZP_NOALLOC_MAX_SEQS) length[s0 + j] = blocks[j] ? L : 0;
    mine += blocks[j];
  }
  int sum = mine;
#pragma unroll
  for (int by = 1; by < 64; by *= 2) {
    const int before = __shfl_up(sum, by);
    if (lane >= by) sum += before;
  }
  if (lane == 63) wave_sum[w] = sum;
  __syncthreads();
  sum -= mine;
  for (int i = 0; i < w; i++) sum += wave_sum[i];
  if (threadIdx.x == 0) first_tile[0] = 0;
#pragma unroll
  for (int j = 0; j < PER; j++) {
    sum += blocks[j];
    if (s0 + j < a.S) first_tile[s0 + j + 1] = sum;
  }
  __syncthreads();
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n_tiles || i >= first_tile[a.S]) return;
  // the sequence that owns tile i in (sequence, block) numbering: last s with first_tile[s] <= i
  int lo = 0, hi = a.S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first_tile[mid] <= i) lo = mid; else hi = mid - 1;
  }
  const int s = lo, b = i - first_tile[s];
  int L, nb;
  seq_blocks(a, s, L, nb);
  int slot = nb - 1 - b;
#pragma unroll 8  // (reads of several steps in flight)
  for (int s4 = 0; s4 < a.S; s4 += 4) {
    const int4 l4 = *(const int4 *)(length + s4);
    const int l[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
    for (int j = 0; j < 4; j++)
      if (l[j] > L || (l[j] == L && s4 + j < s)) slot += (l[j] + BM - 1) / BM;
  }
  zp_tile t;
  t.q_tok0 = a.cu[s] + b * BM;
  t.q_rows = L - b * BM < BM ? L - b * BM : BM;
  t.q_pos0 = b * BM;
  t.k_tok0 = a.cu[s];
  t.k_len = L;
  t.k_pos0 = 0;
  t.out_row0 = t.q_tok0;
  t.part = 0;
  tiles[slot] = t;
}

// The same order on the host, for a table of at most ZP_INLINE_TILES records.
void fill_inline(const PlanArgs &a, zp_inline_tiles &inl) {
  int order[ZP_INLINE_TILES], n = 0;  // sequences with blocks, longest first; equal lengths in ascending index
  auto len = [&](int s) { return a.cu[s + 1] - a.cu[s]; };
  for (int s = 0; s < a.S; s++) {
    if (((a.skip_bits[s >> 5] >> (s & 31)) & 1u) || len(s) == 0) continue;
    int i = n++;
    for (; i > 0 && len(order[i - 1]) < len(s); i--) order[i] = order[i - 1];
    order[i] = s;
  }
  int slot = 0;
  for (int i = 0; i < n; i++) {
    const int s = order[i], L = len(s);
    for (int r0 = (L - 1) / BM * BM; r0 >= 0; r0 -= BM)
      inl.t[slot++] = zp_tile{a.cu[s] + r0, L - r0 < BM ? L - r0 : BM, r0, a.cu[s], L, 0, a.cu[s] + r0, 0};
  }
}

// The sequences themselves in the same order (zp_seqs_fit has looked at their number).
void fill_seqs(const PlanArgs &a, int n_seq, zp_inline_tiles &inl) {
  int order[sizeof(zp_inline_tiles) / 12], n = 0;
  auto len = [&](int s) { return a.cu[s + 1] - a.cu[s]; };
  for (int s = 0; s < a.S; s++)
    if (!((a.skip_bits[s >> 5] >> (s & 31)) & 1u) && len(s) > 0) order[n++] = s;
  std::sort(order, order + n, [&](int x, int y) { return len(x) != len(y) ? len(x) > len(y) : x < y; });
  int block = 0;
  for (int i = 0; i < n; i++) block = zp_put_seq(inl, n_seq, i, block, a.cu[order[i]], len(order[i]));
}

std::mutex g_mu;
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES] = {};

// Device address of this GPU's copy of the array, looked up once per device with that device current.
int scratch_for_current_device(void **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return zp_report_hip_error((int)e, "hipGetDevice");
  if (dev < 0 || dev >= MAX_DEVICES) return ZP_EUNSUPPORTED;
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return zp_report_hip_error((int)e, "hipGetSymbolAddress");
    if (!ptr) return zp_report_hip_error((int)hipErrorInvalidSymbol, "hipGetSymbolAddress");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return ZP_OK;
}

}  // namespace

extern "C" int varlen_attn_fwd_noalloc(const void *q, const void *k, const void *v, int64_t q_stride, int64_t k_stride,
                                       int64_t v_stride, const int32_t *cu, const uint8_t *seq_skip, void *o,
                                       int64_t o_stride, float *lse, const zp_shape *sh, void *stream) {
  // the same argument checks as varlen_attn_fwd, all before anything touches the device
  if (!sh) return ZP_EINVAL;
  if (sh->T < 0 || sh->S < 0 || sh->Hq <= 0 || sh->Hkv <= 0) return ZP_EINVAL;
  if (!(sh->scale >= 0.f) || std::isinf(sh->scale)) return ZP_EINVAL;
  if (sh->d != 64 && sh->d != 128) return ZP_EUNSUPPORTED;
  if (sh->Hq % sh->Hkv) return ZP_EUNSUPPORTED;
  if (!cu || cu[0] != 0) return ZP_EINVAL;
  for (int s = 0; s < sh->S; s++)
    if (cu[s + 1] < cu[s]) return ZP_EINVAL;
  if (cu[sh->S] != sh->T) return ZP_EINVAL;
  if (sh->T == 0) return ZP_OK;
  if (!q || !k || !v || !o || !lse) return ZP_EINVAL;
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return ZP_EINVAL;
  auto bad_stride = [&](int64_t st, int H) { return st < (int64_t)H * sh->d || (st % 8) || st > (1 << 24); };
  if (bad_stride(q_stride, sh->Hq) || bad_stride(o_stride, sh->Hq) || bad_stride(k_stride, sh->Hkv) ||
      bad_stride(v_stride, sh->Hkv))
    return ZP_EINVAL;
  // the fixed limits of this entry point
  if (sh->S > ZP_NOALLOC_MAX_SEQS) return ZP_ETOOLARGE;
  if (zp_attn_fwd_block_rows(sh->d) != BM) return ZP_EUNSUPPORTED;
  PlanArgs a;
  a.S = sh->S;
  for (size_t i = 0; i < sizeof(a.skip_bits) / sizeof(a.skip_bits[0]); i++) a.skip_bits[i] = 0;
  int n_seq = 0;
  int64_t n_tiles = 0, sum = 0, longest = 0;  // query blocks; key tiles they see, the last block of the longest sequence
  for (int s = 0; s <= sh->S; s++) a.cu[s] = cu[s];
  for (int s = 0; s < sh->S; s++) {
    if (seq_skip && seq_skip[s]) { a.skip_bits[s >> 5] |= 1u << (s & 31); continue; }
    const int64_t nb = ((int64_t)cu[s + 1] - cu[s] + BM - 1) / BM, last = ((int64_t)cu[s + 1] - cu[s] + 63) / 64;
    n_tiles += nb;
    n_seq += nb > 0;
    sum += nb > 0 ? nb * (nb - 1) + last : 0;  // 2, 4, ... and the last block
    longest = std::max(longest, last);
  }
  if (n_tiles > ZP_NOALLOC_MAX_TILES) return ZP_ETOOLARGE;
  if (n_tiles == 0) return ZP_OK;
  a.n_tiles = (int32_t)n_tiles;

  zp_attn_params p{};
  p.n_tiles = a.n_tiles;
  const int64_t items = (n_tiles * sh->Hkv + 7) / 8 * 8 * (sh->Hq / sh->Hkv);
  if (n_tiles <= ZP_INLINE_TILES && items < ZP_CLAIM_MIN_ITEMS) {
    // a short table goes into the launch arguments (and the shared array is not touched)
    fill_inline(a, p.inl);
  } else if (zp_seqs_fit(n_seq, n_tiles) && zp_seqs_pay(sum, sh->Hq, sh->d, ZP_SEQS_NOALLOC)) {
    fill_seqs(a, n_seq, p.inl);
    p.n_seq = n_seq;
  } else {
    void *tiles = nullptr;
    const int rc = scratch_for_current_device(&tiles);
    if (rc) return rc;
    // Every slot the attention kernel reads is rewritten by the planning kernel of the same call, on the same stream,
    // and so are the work counters in front of the table: nothing of an earlier call survives into this one.
    hipLaunchKernelGGL(plan_fwd_tiles_kernel, dim3((unsigned)((n_tiles + PLAN_NT - 1) / PLAN_NT)), dim3(PLAN_NT), 0, (hipStream_t)stream, a,
                       (int32_t *)tiles, (zp_tile *)((char *)tiles + ZP_COUNTER_BYTES));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return zp_report_hip_error((int)e, "plan_fwd_tiles launch");
    p.tiles = (const zp_tile *)((char *)tiles + ZP_COUNTER_BYTES);
    p.work.counters = (int32_t *)tiles;
  }
  p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v;
  p.q_stride = q_stride; p.k_stride = k_stride; p.v_stride = v_stride;
  p.Hq = sh->Hq; p.Hkv = sh->Hkv; p.grp = sh->Hq / sh->Hkv;
  zp_plan_fwd_pair(p, sh->d);
  p.turns = zp_fwd_turns(sh->d, sum, n_tiles, longest, sh->Hq);
  p.scale = sh->scale > 0.f ? sh->scale : 1.0f / std::sqrt((float)sh->d);
  p.scale_log2 = p.scale * 1.4426950408889634f;
  p.o = o; p.o_stride = o_stride; p.lse = lse; p.lse_stride = sh->T;
  const hipError_t e = (hipError_t)zp_launch_attn_fwd(&p, sh->d, 0, BM, (hipStream_t)stream);
  if (e != hipSuccess) return zp_report_hip_error((int)e, "attn_fwd launch");
  return ZP_OK;
}
