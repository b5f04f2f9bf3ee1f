// C ABI of the attention engine: argument checks, the host planner (work lists ordered by cost), descriptor
// upload through pinned staging buffers, kernel launches. No device allocation, no synchronisation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/zeppelin_attn.h"
#include "zp_common.h"
#include "zp_pair.h"
#include "zp_pool.h"

extern "C" {
int zp_launch_attn_fwd(const zp_attn_params *p, int d, int partial, int block_rows, hipStream_t stream);
int zp_attn_fwd_block_rows(int d);
int zp_launch_remap(const void *src, void *dst, int64_t row_bytes, const int32_t *idx, int64_t n_rows, int mode,
                    hipStream_t stream);
int zp_merge_rows_per_item(void);
int zp_launch_lse_merge(const float *o_part, const float *lse_part, int64_t part_rows, const void *merges_dev,
                        const void *items_dev, int n_items, int Hq, int d, void *o, int64_t o_stride, float *lse,
                        int64_t T, int max_parts, hipStream_t stream);
int zp_launch_accum_to_bf16(const float *src, void *dst, int64_t n, hipStream_t stream);
int zp_launch_attn_bwd(const zp_bwd_params *p, int d, hipStream_t stream);
int zp_attn_bwd_block_rows(int d, int which);
}

namespace {

thread_local std::string g_hip_error = "HIP runtime error";

int hip_fail(hipError_t e, const char *what) {
  g_hip_error = std::string("HIP runtime error in ") + what + ": " + hipGetErrorString(e);
  return ZP_EHIP;
}
#define ZP_HIP(call, what)                       \
  do {                                           \
    hipError_t e__ = (call);                     \
    if (e__ != hipSuccess) return hip_fail(e__, what); \
  } while (0)

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- pinned staging pool -------------------------------------------------------------------------
// Descriptor tables are built in pinned host memory; one workgroup copies them into the workspace and, once it has read
// all of it, sets the slot's flag in pinned memory, so that the host never overwrites bytes still to be read (zp_pool.h
// holds the slot state machine; this is its HIP backend). A hipMemcpyAsync in its place runs on another engine, and
// ordering that engine with the stream's kernels, plus an event behind the copy, left the stream without a kernel of the
// call for 25 us per forward or backward call on 64K lognormal MHA; 8-12 us with this one.
struct HipPoolBackend {
  typedef uint32_t *event_t;  // the flag: 0 while the copy is to come
  typedef hipStream_t stream_t;
  static int alloc(void **p, size_t bytes) { return (int)hipHostMalloc(p, bytes, hipHostMallocPortable | hipHostMallocCoherent); }
  static void release(void *p) { (void)hipHostFree(p); }
  static int event_create(event_t *e) { return (int)hipHostMalloc((void **)e, 64, hipHostMallocPortable | hipHostMallocCoherent); }
  static int event_record(event_t, stream_t) { return 0; }  // the copy sets it
  static bool event_done(event_t e) { return __atomic_load_n(e, __ATOMIC_ACQUIRE) != 0; }
};
zp_staging_pool<HipPoolBackend> g_pool;

constexpr int UPLOAD_NT = 1024, UPLOAD_UNROLL = 4;
// One workgroup: 64 KB of host reads in flight at a time. n16: 16-byte pieces.
__global__ __launch_bounds__(UPLOAD_NT) void upload_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int64_t n16,
                                                           uint32_t *flag) {
  for (int64_t base = threadIdx.x; base < n16; base += UPLOAD_NT * UPLOAD_UNROLL) {
    u32x4 v[UPLOAD_UNROLL];
#pragma unroll
    for (int u = 0; u < UPLOAD_UNROLL; u++)
      if (base + u * UPLOAD_NT < n16) v[u] = __builtin_nontemporal_load(src + base + u * UPLOAD_NT);
#pragma unroll
    for (int u = 0; u < UPLOAD_UNROLL; u++)
      if (base + u * UPLOAD_NT < n16) dst[base + u * UPLOAD_NT] = v[u];
  }
  __syncthreads();  // every piece has been read: it has been written
  if (threadIdx.x == 0) __hip_atomic_store(flag, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The same for a table that travels in the launch arguments, one launch per UPLOAD_ARGS pieces.
constexpr int UPLOAD_ARGS = 248;
struct UploadArgs {
  u32x4 v[UPLOAD_ARGS];
};
static_assert(sizeof(UploadArgs) + 16 <= 4096, "kernel arguments are limited to 4 KB");
__global__ __launch_bounds__(256) void upload_args_kernel(UploadArgs a, u32x4 *__restrict__ dst, int n16) {
  if ((int)threadIdx.x < n16) dst[threadIdx.x] = a.v[threadIdx.x];
}

// A table on its way to the device: upload_begin says where to write it (`host`), upload_send copies it. While the stream
// is capturing, the table goes by value into the launches that write it, so that it lives as long as the graph does: a
// staging slot would be read by every replay, could never be given back, and a new one cannot be allocated during a
// capture. Replays pay one small launch per 4 KB for that.
struct Upload {
  void *host = nullptr;
  int slot = -1;           // of the staging pool; -1: `own`
  std::vector<u32x4> own;
};
int upload_begin(size_t bytes, hipStream_t stream, Upload &u) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess) (void)hipGetLastError();
  if (cap != hipStreamCaptureStatusNone) {
    u.own.resize((bytes + 15) / 16);
    u.host = u.own.data();
    return ZP_OK;
  }
  const int e = g_pool.acquire((bytes + 15) & ~(size_t)15, &u.slot, &u.host);
  return e ? hip_fail((hipError_t)e, "staging buffer") : ZP_OK;
}
// Copies `bytes` to device memory on `stream`; a slot stays busy until that has happened. `dev` is 16-byte aligned and has
// room for `bytes` rounded up to 16.
int upload_send(Upload &u, void *dev, size_t bytes, hipStream_t stream) {
  const int64_t n16 = (int64_t)((bytes + 15) / 16);
  if (u.slot < 0) {
    for (int64_t at = 0; at < n16; at += UPLOAD_ARGS) {
      UploadArgs a;
      const int n = (int)std::min<int64_t>(UPLOAD_ARGS, n16 - at);
      std::memcpy(a.v, u.own.data() + at, (size_t)n * 16);
      std::memset((void *)(a.v + n), 0, (size_t)(UPLOAD_ARGS - n) * 16);
      hipLaunchKernelGGL(upload_args_kernel, dim3(1), dim3(256), 0, stream, a, (u32x4 *)dev + at, n);
    }
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? hip_fail(e, "descriptor upload") : ZP_OK;
  }
  uint32_t *flag = g_pool.event(u.slot);
  __atomic_store_n(flag, 0u, __ATOMIC_RELEASE);
  hipLaunchKernelGGL(upload_kernel, dim3(1), dim3(UPLOAD_NT), 0, stream, (const u32x4 *)u.host, (u32x4 *)dev, n16, flag);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    g_pool.abandon(u.slot);
    return hip_fail(e, "descriptor upload");
  }
  const int r = g_pool.submitted(u.slot, stream);
  return r ? hip_fail((hipError_t)r, "descriptor upload") : ZP_OK;
}

// ---- per-kernel timing (measurement aid) -----------------------------------------------------------
// When enabled, every kernel launch (the row terms of a short backward with the launch behind them) is bracketed by a pair of hipEvents on
// the launch stream; the bench reads the elapsed times after it has synchronised. Which kernels a call takes does not depend on it. Off by
// default: no events are created or recorded.
struct ProfRec {
  const char *name;
  hipEvent_t a, b;
};
std::mutex g_prof_mu;
bool g_prof_on = false;
std::vector<ProfRec> g_prof;

// ---- checks --------------------------------------------------------------------------------------
int check_shape(const zp_shape *sh) {
  if (!sh) return ZP_EINVAL;
  if (sh->T < 0 || sh->S < 0 || sh->Hq <= 0 || sh->Hkv <= 0) return ZP_EINVAL;
  if (!(sh->scale >= 0.f) || std::isinf(sh->scale)) return ZP_EINVAL;
  if (sh->d != 64 && sh->d != 128) return ZP_EUNSUPPORTED;
  if (sh->Hq % sh->Hkv) return ZP_EUNSUPPORTED;
  return ZP_OK;
}
int check_cu(const int32_t *cu, const zp_shape *sh) {
  if (!cu) return ZP_EINVAL;
  if (cu[0] != 0) return ZP_EINVAL;
  for (int s = 0; s < sh->S; s++)
    if (cu[s + 1] < cu[s]) return ZP_EINVAL;
  if (cu[sh->S] != sh->T) return ZP_EINVAL;
  return ZP_OK;
}
// token strides: at least one token's heads, 16-byte aligned rows, and small enough that the byte offsets of a
// 64-row tile fit the 32-bit lane offsets of the asynchronous tile copy
int check_stride(int64_t stride, int H, int d) {
  return (stride < (int64_t)H * d || (stride % 8) || stride > (1 << 24)) ? ZP_EINVAL : ZP_OK;
}
bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
int check_ws(const void *ws, size_t have, size_t need) {
  if (need == 0) return ZP_OK;
  if (!ws || ((uintptr_t)ws & 255) || have < need) return ZP_EWORKSPACE;
  return ZP_OK;
}
float eff_scale(const zp_shape *sh) { return sh->scale > 0.f ? sh->scale : 1.0f / std::sqrt((float)sh->d); }

// ---- planner -------------------------------------------------------------------------------------
// A tile's cost is the number of key tiles it visits: the per-block share of the quadratic cost |s|^2 that
// Alg. 2 balances. Lists of chunk-pair tiles are issued in descending cost so the heaviest start first.
struct CostTile {
  zp_tile t;
  int32_t cost;
};
inline int32_t tile_cost(const zp_tile &t) {
  int64_t n = (int64_t)t.q_pos0 + t.q_rows - 1 - t.k_pos0 + 1;
  if (n < 0) n = 0;
  if (n > t.k_len) n = t.k_len;
  return (int32_t)((n + 63) / 64);
}
void sort_by_cost(std::vector<CostTile> &v) {
  std::stable_sort(v.begin(), v.end(), [](const CostTile &a, const CostTile &b) { return a.cost > b.cost; });
}
int64_t count_blocks(const int32_t *cu, int S, int bm) {
  int64_t n = 0;
  for (int s = 0; s < S; s++) n += ((int64_t)cu[s + 1] - cu[s] + bm - 1) / bm;
  return n;
}
std::vector<int> longest_first(const int32_t *cu, int S) {
  std::vector<int> order(S);
  for (int s = 0; s < S; s++) order[s] = s;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cu[a + 1] - cu[a] > cu[b + 1] - cu[b]; });
  return order;
}
// Tiles of whole sequences: sequence by sequence, longest sequence first, and inside a sequence the last query block
// (the most expensive one) first. The heaviest tiles of the batch still start first and the cheap ones fill the tail,
// as a plain sort by cost would have it, but the query blocks of one (sequence, KV head) now run next to each other on
// one XCD and find the sequence's K/V rows in its L2 instead of re-reading them from HBM -- with many short sequences
// and one KV head per query head that re-reading, not the arithmetic, bounded the kernels.
void plan_whole(const int32_t *cu, int S, int bm, std::vector<CostTile> &out, const uint8_t *skip = nullptr) {
  for (int s : longest_first(cu, S)) {
    if (skip && skip[s]) continue;
    const int32_t L = cu[s + 1] - cu[s];
    for (int32_t r0 = ((L - 1) / bm) * bm; L > 0 && r0 >= 0; r0 -= bm) {
      CostTile c{};
      c.t.q_tok0 = cu[s] + r0;
      c.t.q_rows = std::min(bm, L - r0);
      c.t.q_pos0 = r0;
      c.t.k_tok0 = cu[s];
      c.t.k_len = L;
      c.t.k_pos0 = 0;
      c.t.out_row0 = cu[s] + r0;
      c.cost = tile_cost(c.t);
      out.push_back(c);
    }
  }
}
// Key-block tiles go sequence by sequence, longest sequence first, blocks in position order (descending
// cost inside the sequence): workgroups that run side by side then walk the same Q/dO rows a few tiles
// apart and find them in L2, and the cheap blocks of the short sequences still come last.
void plan_whole_keys(const int32_t *cu, int S, int bnk, std::vector<CostTile> &out, const uint8_t *skip = nullptr) {
  out.reserve((size_t)count_blocks(cu, S, bnk));
  for (int s : longest_first(cu, S)) {
    if (skip && skip[s]) continue;
    const int32_t L = cu[s + 1] - cu[s];
    for (int32_t j0 = 0; j0 < L; j0 += bnk) {
      CostTile c{};
      c.t.k_tok0 = cu[s] + j0;
      c.t.k_len = std::min(bnk, L - j0);
      c.t.k_pos0 = j0;
      c.t.q_tok0 = cu[s] + j0;  // first query that sees the block's first key
      c.t.q_rows = L - j0;
      c.t.q_pos0 = j0;
      c.t.out_row0 = cu[s] + j0;
      c.cost = (c.t.q_rows + 63) / 64;
      out.push_back(c);
    }
  }
}
int64_t count_pair_blocks(const zp_pair *pairs, int n, int bm) {
  int64_t c = 0;
  for (int i = 0; i < n; i++) c += ((int64_t)pairs[i].q_len + bm - 1) / bm;
  return c;
}

// Every tile table in a workspace is preceded by WS_HEADER bytes of work counters (two sets: a call launches at most
// two attention kernels), which travel with the table in the same copy and arrive as zeros.
constexpr size_t WS_HEADER = 2 * ZP_COUNTER_BYTES;
inline int32_t *ws_counters(void *ws) { return (int32_t *)ws; }
inline const zp_tile *ws_tiles(void *ws) { return (const zp_tile *)((char *)ws + WS_HEADER); }
inline size_t tile_table_bytes(size_t n_tiles) { return WS_HEADER + align256(n_tiles * sizeof(zp_tile)); }

// Share of a launch's items that workgroups claim at run time (zp_work_split): half when the items are heavy (32 key
// or query tiles and more on average, i.e. tens of microseconds each), an eighth when they are light.
int dyn_div_of(const std::vector<CostTile> &tiles, size_t first, size_t n, int weight) {
  if (n == 0) return 8;
  int64_t sum = 0;
  for (size_t i = first; i < first + n; i++) sum += tiles[i].cost;
  return sum * weight >= (int64_t)n * 32 ? 2 : 8;
}

// (the costs are key tiles)
bool fwd_turns(const std::vector<CostTile> &tiles, const zp_shape *sh) {
  int64_t sum = 0, longest = 0;
  for (const CostTile &c : tiles) { sum += c.cost; longest = std::max<int64_t>(longest, c.cost); }
  return zp_fwd_turns(sh->d, sum, (int64_t)tiles.size(), longest, sh->Hq);
}

// (zeros: so many 32-bit zeros behind the table)
int upload_tiles(const std::vector<CostTile> &tiles, size_t zeros, void *ws, hipStream_t stream) {
  if (tiles.empty()) return ZP_OK;
  const size_t bytes = WS_HEADER + tiles.size() * sizeof(zp_tile) + zeros * sizeof(int32_t);
  Upload u;
  int rc = upload_begin(bytes, stream, u);
  if (rc) return rc;
  std::memset(u.host, 0, WS_HEADER);
  zp_tile *h = (zp_tile *)((char *)u.host + WS_HEADER);
  for (size_t i = 0; i < tiles.size(); i++) h[i] = tiles[i].t;
  std::memset((void *)(h + tiles.size()), 0, zeros * sizeof(int32_t));
  return upload_send(u, ws, bytes, stream);
}

// Puts the tile table where the kernels find it. A table that fits the launch arguments goes there when none of its
// launches (of at most max_items work items) is large enough to claim items at run time, which would need counters in
// device memory; then *dev and *counters are null. Eight sequences of 1218 tokens in all, one call after the other:
// forward (4 heads, d = 64) 23.1 us with the upload, 19.1 without (the host is the bound), forward and backward (GQA 4/2,
// d = 128) 70.1 and 57.6.
bool tiles_inline(size_t n, int64_t max_items) { return n <= ZP_INLINE_TILES && max_items < ZP_CLAIM_MIN_ITEMS; }
int place_tiles(const std::vector<CostTile> &tiles, int64_t max_items, zp_inline_tiles &inl, void *ws, hipStream_t stream,
                const zp_tile **dev, int32_t **counters, size_t zeros = 0) {
  if (tiles_inline(tiles.size(), max_items)) {
    for (size_t i = 0; i < tiles.size(); i++) inl.t[i] = tiles[i].t;
    *dev = nullptr;
    *counters = nullptr;
    return ZP_OK;
  }
  *dev = ws_tiles(ws);
  *counters = ws_counters(ws);
  return upload_tiles(tiles, zeros, ws, stream);
}
// Whether the sequences of a call on whole ones (their query blocks: `tiles`) go into the launch arguments, where its tile table would have
// to be uploaded otherwise: zp_seqs_pay, with the call's limit.
bool seqs_in_arguments(const std::vector<CostTile> &tiles, const zp_shape *sh, float most, zp_inline_tiles &inl, int32_t &n_seq) {
  int64_t sum = 0;
  int32_t n = 0;
  for (const CostTile &c : tiles) {
    sum += c.cost;
    n += c.t.q_pos0 == 0;
  }
  if (!zp_seqs_fit(n, (int64_t)tiles.size()) || !zp_seqs_pay(sum, sh->Hq, sh->d, most)) return false;
  n_seq = n;
  int i = 0, block = 0;
  for (const CostTile &c : tiles)
    if (c.t.q_pos0 == 0) block = zp_put_seq(inl, n, i++, block, c.t.k_tok0, c.t.k_len);
  return true;
}
// Which dK/dV kernel a launch takes, by estimates of their times in microseconds; an iteration is a (32-query tile, head). All deal
// the units (tile, KV head) to the XCDs by turns. An XCD hands its workgroups in order and by turns to four engines of eight
// CUs; one waits for its engine, whatever room the others have. (Sequences of four key blocks so put every longest chain on
// one engine: 17 of 405 tokens, 64/8 heads, d = 128, 260 us where their sum would make 175.)
//  - whole: one workgroup of four waves per key block. Two share a CU, 32 units apart, and an iteration beside another workgroup
//    takes 1.35 to 1.37 times as long. The longest pair of chains; behind two workgroups per CU, no less than all of the fullest
//    engine and a part of those that start last. Iterations on the diagonal count more (masks), and d = 64 takes 64 queries at a time.
//  - pair (d = 128): one workgroup of two groups of four waves per key block and CU, half the chain.
//  - split: four workgroups of four groups of two waves per key block, some of them without keys, a quarter of the chain. One
//    per CU at d = 128. Two share a CU at 64: the longest one while 32 CUs hold all of an XCD's, else their time over the CUs
//    and a part of those that start last, no more than the longest per round; those without keys cost 2 us.
// Pair and split at d = 128 are placed workgroup by workgroup, those of the XCD with the most iterations (0.1 us of host time in
// the mean, 3.5 at most; not where their sum is longer already). More than 1024 units always take the first: their number
// evens out what the others gain.
//
// The constants are fitted to 3900 launches of 2/1 to 64/8 heads (equal, ragged and lognormal lengths, 16 to 40000 tokens);
// the estimates are 3 to 5 % off in the mean. The split has to be 3 % below at d = 64, and at d = 128 the pair 2 %. Beyond
// 200 us, where the clock falls with what the CUs have to do, the split has to be 8 % below (six sequences, 6705 tokens, 64/8:
// 729 us estimated against 736 for the pair; backward 1210 against 1073), and the pair may be 4 % above if heads share a
// KV head (ten sequences of 2628 tokens, 16/4: 575 against 569 for the first; 998 against 1072). Of all 4500 launches (with dQ in front)
// 11 are more than 5 % behind the fastest of the three, 0.06 % in the mean, and none more than 3 % behind the first. n
// sequences, us, whole / pair / split:
//    d   heads   tokens                              taken
//    64  64/8    1698, longest   98, n = 39:   33.7 /     - /   27.9   split
//    64  16/16    312, equal,        n =  8:    5.1 /     - /    6.9   whole
//    64  16/16   7923, longest 2641, n =  3:  101.7 /     - /  136.9   whole
//   128  16/4     919, longest  100, n = 18:   24.2 /  19.8 /   11.5   split
//   128   8/8    2456, longest 1493, n =  2:   55.0 /  43.8 /   32.7   split
//   128   8/8    7721, longest 2502, n = 14:   96.1 /  71.8 /  106.8   pair
//   128  32/32   3037,               n =  1:  137.1 / 151.1 /  242.2   whole
//   128   8/8   14745, equal,        n = 15:  101.0 / 113.5 /  160.0   whole
struct KvCost {
  float whole, whole_it, share, rate, whole_tail, whole_wg, mask;  // fixed, per iteration; in iterations: of the companion's, all of them, of the last; per workgroup, masked one
  float split, split_wg, split_it;                                 // per launch; per workgroup: fixed, per iteration of a group
};
enum KvKernel { KV_WHOLE, KV_PAIR, KV_SPLIT };
// Workgroups of one XCD with a CU each, in order: when the last one ends.
struct KvPlacement {
  float busy[4][8] = {}, end = 0.f;
  int next = 0;
  void start(float time) {
    float *b = busy[next++ & 3];
    int at = 0;
    for (int i = 1; i < 8; i++) at = b[i] < b[at] ? i : at;
    b[at] += time;
    end = std::max(end, b[at]);
  }
};
const KvCost kv_cost[2] = {{2.12f, 0.565f, 0.371f, 0.841f, 0.136f, 3.08f, 0.375f, 2.46f, 1.86f, 0.831f},
                           {0.49f, 1.029f, 0.349f, 0.740f, 0.586f, 4.30f, 0.154f, 1.69f, 2.82f, 1.255f}};
// *estimate: its time; 0 beyond 1024 units
KvKernel dkdv_kernel_for(const std::vector<CostTile> &kt, int d, int Hkv, int grp, float *estimate) {
  const KvCost &c = kv_cost[d == 128];
  const int64_t units = (int64_t)kt.size() * Hkv;
  *estimate = 0.f;
  if (units > 1024) return KV_WHOLE;
  struct Xcd {
    int n = 0, parts[128];                  // units; of each: its 32-row parts with keys,
    float its[128], chain[128], all = 0.f;  // its iterations, the same with what else the whole kernel spends; of all units
  } xcd[8];
  int u = 0;
  float longest = 0.f;
  for (const CostTile &k : kt) {
    const float its = (float)((k.t.q_rows + 31) / 32) * (float)grp, wide = d == 64 ? (float)((k.t.q_rows + 63) / 64 * 2) * (float)grp : its;
    longest = std::max(longest, its);
    for (int g = 0; g < Hkv; g++, u++) {
      Xcd &x = xcd[u & 7];
      x.parts[x.n] = (k.t.k_len + 31) / 32;
      x.its[x.n] = its;
      x.chain[x.n++] = wide + c.mask * std::min(wide, 4.f * (float)grp) + c.whole_wg;
      x.all += its;
    }
  }
  float whole = 0.f;
  const Xcd *most = xcd;
  for (const Xcd &x : xcd) {
    if (x.all > most->all) most = &x;
    for (int i = 0; i < std::min(32, x.n); i++) {
      const float beside = i + 32 < x.n ? x.chain[i + 32] : 0.f;
      whole = std::max(whole, std::max(x.chain[i], beside) + c.share * std::min(x.chain[i], beside));
    }
    if (x.n > 64) {
      float engine[4] = {}, last = 0.f;
      for (int i = 0; i < x.n; i++) {
        engine[i & 3] += x.chain[i];
        if (i >= x.n - 32) last += x.chain[i];
      }
      const float fullest = std::max(std::max(engine[0], engine[1]), std::max(engine[2], engine[3]));
      whole = std::max(whole, fullest / 8.f * c.rate + c.whole_tail * last / 32.f);
    }
  }
  const float t_whole = c.whole + c.whole_it * whole;
  if (d == 64) {
    const float top = c.split_wg + c.split_it * floorf((longest + 3.f) / 4.f), slow = 1.519f;
    float split = top;
    for (const Xcd &x : xcd) {
      if (x.n <= 8) continue;
      float wgs = 0.f, its = 0.f, last_wgs = 0.f, last_its = 0.f;
      for (int i = x.n; i-- > 0;) {
        const float p = (float)x.parts[i], it = floorf((x.its[i] + 3.f) / 4.f) * p;
        if (last_wgs < 32.f) { last_wgs += p; last_its += it; }
        wgs += p; its += it;
      }
      const float all = c.split_wg * wgs + 2.01f * ((float)(4 * x.n) - wgs) + c.split_it * its;
      const float fill = all * slow / 64.f + 0.923f * (c.split_wg + c.split_it * last_its / std::max(1.f, last_wgs));
      split = std::max(split, std::min(fill, top * slow * (float)((4 * x.n + 63) / 64)));
    }
    // one key block each, all of it on the diagonal, beyond one workgroup per CU: up to 30 % behind the estimate (49 sequences of up
    // to 99 tokens, 32/8 heads: 19.8 us estimated, 26.5 measured; 56 of up to 100, 64/8: 34.6 us whole, 40.8 split)
    const bool diagonal = units > 256 && longest <= 4.f * (float)grp;
    const bool taken = c.split + split < (diagonal ? 0.8f : 0.97f) * t_whole;
    *estimate = taken ? c.split + split : t_whole;
    return taken ? KV_SPLIT : KV_WHOLE;
  }

  constexpr float PAIR = 1.04f, PAIR_WG = 3.61f, PAIR_IT = 1.533f, SPLIT_MASK = 0.514f;
  const float least = PAIR_IT * 0.5f * most->all / 32.f, longest_pair = PAIR_WG + floorf((longest + 1.f) / 2.f);
  float t_pair = t_whole + t_whole;  // (not taken)
  const float limit = (grp > 1 && t_whole > 200.f ? 1.04f : 0.98f) * t_whole;
  if (PAIR + std::max(least, PAIR_IT * longest_pair) < limit) {
    KvPlacement on;
    for (int i = 0; i < most->n; i++) on.start(PAIR_WG + floorf((most->its[i] + 1.f) / 2.f));
    t_pair = PAIR + PAIR_IT * std::max(on.end, longest_pair);
  }
  const bool pair = t_pair < limit;
  const float fastest = std::min(t_whole, t_pair), other = fastest > 200.f ? 0.92f * fastest : fastest, masked = SPLIT_MASK * (float)((grp + 3) / 4);
  float all = 0.f;
  for (int i = 0; i < most->n; i++) all += (float)most->parts[i] * (c.split_wg + masked + floorf((most->its[i] + 3.f) / 4.f));
  if (c.split + c.split_it * all / 32.f < other) {
    KvPlacement on;
    for (int i = 0; i < most->n; i++) {
      const float time = c.split_wg + masked + floorf((most->its[i] + 3.f) / 4.f);
      for (int part = 0; part < 4; part++) on.start(part < most->parts[i] ? time : 0.f);
    }
    *estimate = c.split + c.split_it * on.end;
    if (*estimate < other) return KV_SPLIT;
  }
  *estimate = pair ? t_pair : t_whole;
  return pair ? KV_PAIR : KV_WHOLE;
}
// work items of a launch over n tiles: (tile, KV head) units padded to one per XCD, times the heads in a group
int64_t launch_items(size_t n, int Hkv, int grp) { return ((int64_t)n * Hkv + 7) / 8 * 8 * grp; }

// ---- dK/dV: shares of key blocks
// The whole kernels' launch lasts at least as long as its longest chain of iterations, that of the first key block of the longest
// sequence with all heads of its group, however little the others have to do. Blocks of many iterations are therefore cut into shares,
// a workgroup each, whose sums the last one to end adds up (dkdv_join_parts). The shares of a sequence's blocks cover the same query
// tiles, counted from its end, so that they still find each other's Q and dO rows in L2 (shares of a block's own iterations that are equally
// long: 39059 tokens, 8/2 heads, d = 64, 5.1 ms instead of 4.7). A share costs a prologue and its sums' way to memory and back, 7 us of a CU at d = 64
// and 14 at 128, so it is a fifth or a quarter of a CU's load long, and the shares are taken where the estimate of their launch is
// 7 % (d = 128: 5 %) below that of the other kernels. The estimate is fitted to 340 launches of up to 4 ms (of 4/4 to 64/8 heads, 5000 to 131072
// tokens; 5 % off in the mean). Of 85 random backwards whose longest chain is a third of a CU's load and more 42 take them: 1.06 times
// faster in the mean of all at d = 64 and 1.023 at 128; none of the 42 is slower. Batches whose blocks have much the same number of iterations
// (single sequences and equal ones: the longest block less than twice the average) are not in that fit, and the estimate favours shares
// there: up to 550 us they are taken where it is 20 % below. Of 262 such backwards 169 take them, in 0.85 of the time in the mean, two of
// them 2 and 4 % slower; with 15 % below it were 216, seven of them slower, by 12 % at most. (Beyond 550 us the margins of the others
// hold: of 48 such backwards 36 take shares, all of them faster.) Tables in the launch arguments are left out, since the counts of shares that are done travel
// with an uploaded table. Backward, us, before / with shares:
//    d   heads   tokens                        taken             not taken
//    64  16/4    24001, longest  3802          482 / 448
//    64   8/2    39059, longest 39059         5256 / 4660
//   128   8/2    24001, longest 11048         1504 / 1235
//   128   4/4    34415, longest  7173          434 / 373
//   128   4/2    11503, longest  3643                            160 / 168
//    64   4/2    26485, longest  3837                            192 / 202
//    64  64/2     1900                             429 / 164
//   128   8/1    17 of 1000                        295 / 213
//   128   8/1    28 of 1000                                        341 / 345
//   128   8/2     9000                             671 / 644
struct KvShareCost {
  float of_load, least;            // a share: of a CU's load, and at least so many iterations of 32 queries
  float launch, it, slot, share;   // per launch; per CU: iteration, share; per iteration of a share
  float margin;
};
const KvShareCost kv_share_cost[2] = {{0.2f, 48.f, 11.2f, 0.385f, 7.43f, 0.408f, 0.93f}, {0.25f, 64.f, 8.84f, 0.691f, 14.2f, 0.803f, 0.95f}};
// iterations of a block of keys that `rows` queries see (d = 64: of 64 queries)
inline int64_t kv_iterations(int64_t rows, int d, int grp) { return (d == 64 ? (rows + 63) / 64 : (rows + 31) / 32) * grp; }
// shares of a block: the last one has between 3/8 and 11/8 of the others' iterations
inline int64_t kv_shares_of(int64_t its, int64_t share) { return std::max<int64_t>(1, (its + share * 5 / 8) / share); }
struct KvLoad {
  float sum = 0.f;  // iterations of 32 queries, fixed ones of a workgroup among them
  int64_t its = 0, longest = 0, blocks = 0;
  void add(int64_t its, int d) {
    this->its += its;
    sum += (d == 64 ? 2.f : 1.f) * (float)its + kv_cost[d == 128].whole_wg;
    longest = std::max(longest, its);
    blocks++;
  }
};
// How many iterations a share of the blocks of a batch's unflagged sequences would have; 0: no block would be shared.
int32_t plan_kv_shares(const int32_t *cu, const zp_shape *sh, int bnk, const uint8_t *skip = nullptr) {
  auto tokens = [&](int s) { return skip && skip[s] ? 0 : (int64_t)cu[s + 1] - cu[s]; };
  const int grp = sh->Hq / sh->Hkv, c = sh->d == 128;
  const float unit = sh->d == 64 ? 2.f : 1.f;
  KvLoad all;
  for (int s = 0; s < sh->S; s++)
    for (int64_t L = tokens(s); L > 0; L -= bnk) all.add(kv_iterations(L, sh->d, grp), sh->d);
  if (tiles_inline(2 * (size_t)all.blocks, launch_items((size_t)all.blocks, sh->Hkv, grp))) return 0;
  const float load = kv_cost[c].rate * all.sum * (float)sh->Hkv / 256.f;
  if (unit * (float)all.longest < 0.5f * load) return 0;
  int64_t share = (int64_t)(std::max(kv_share_cost[c].of_load * load, kv_share_cost[c].least) / unit);
  // no more than 2048 sums (d = 128: 256 MB)
  for (;; share += share / 8) {
    share = (share + grp - 1) / grp * grp;
    int64_t slots = 0, most = 0;
    for (int s = 0; s < sh->S; s++)
      for (int64_t L = tokens(s); L > 0; L -= bnk) {
        const int64_t n = kv_shares_of(kv_iterations(L, sh->d, grp), share);
        if (n == 1) break;  // nor do the sequence's blocks behind it have more
        slots += n;
        most = std::max(most, n);
      }
    if (slots == 0) return 0;
    if (most <= ZP_PART_MAX && slots * sh->Hkv <= 2048) return (int32_t)share;
  }
}
// Whether the blocks of `kt` are taken in shares of `share` iterations, in place of a kernel estimated at `other` us (0: the whole one,
// not estimated).
bool take_kv_shares(int32_t share, const std::vector<CostTile> &kt, int d, int Hkv, int grp, float other) {
  if (share == 0) return false;
  const KvCost &w = kv_cost[d == 128];
  const KvShareCost &c = kv_share_cost[d == 128];
  const float unit = d == 64 ? 2.f : 1.f, heads = (float)Hkv / 256.f;
  KvLoad all;
  int64_t slots = 0;
  for (const CostTile &k : kt) {
    const int64_t its = kv_iterations(k.t.q_rows, d, grp), n = kv_shares_of(its, share);
    all.add(its, d);
    if (n > 1) slots += n;
  }
  if (other == 0.f) other = w.whole + w.whole_it * std::max(w.rate * all.sum * heads, (1.f + w.share) * unit * (float)all.longest);
  const float time = c.launch + c.it * all.sum * heads + c.slot * (float)slots * heads + c.share * unit * (float)share;
  const bool even = all.longest * all.blocks <= 2 * all.its;
  return slots > 0 && time < (even && other <= 550.f ? 0.8f : c.margin) * other;
}
// Puts the shares of the blocks of `kt` (sequence by sequence, blocks in position order) in their place: the first shares of a sequence's blocks, the
// second ones, and so on. Returns how many shares of shared blocks there are.
int32_t share_blocks(std::vector<CostTile> &kt, int d, int grp, int64_t share) {
  std::vector<CostTile> out;
  out.reserve(kt.size() * 2);
  int32_t slots = 0;
  for (size_t a = 0, b; a < kt.size(); a = b) {
    for (b = a + 1; b < kt.size() && kt[b].t.k_pos0 > 0;) b++;
    const int32_t slot0 = slots;
    const int most = (int)kv_shares_of(kv_iterations(kt[a].t.q_rows, d, grp), share);
    for (int part = 0; part < most; part++) {
      int32_t slot = slot0;
      for (size_t i = a; i < b; i++) {
        const int64_t its = kv_iterations(kt[i].t.q_rows, d, grp);
        const int n = (int)kv_shares_of(its, share);
        if (part >= n) break;  // nor have the blocks behind it this many
        CostTile c = kt[i];
        if (n > 1) {
          c.t.part = zp_part_code(part, n, slot);
          c.cost = (int32_t)(c.cost * (part + 1 < n ? share : its - part * share) / its);
          slot += n;
        }
        out.push_back(c);
      }
      slots = std::max(slots, slot);
    }
  }
  kt.swap(out);
  return slots;
}
// What a backward keeps in its workspace: counters and tile table, of every sum a count of the shares that are done (zeros behind the table), D and
// -LSE / scale of the rows, sums of shares. `sums`: shares of shared blocks x KV heads.
struct BwdScratch {
  size_t done_at, dvec_at, lse2_at, parts_at, bytes;
};
BwdScratch bwd_scratch(size_t tiles, size_t sums, const zp_shape *sh) {
  const size_t rows = align256((size_t)sh->Hq * (size_t)sh->T * sizeof(float));
  BwdScratch w;
  w.done_at = WS_HEADER + tiles * sizeof(zp_tile);
  w.dvec_at = align256(w.done_at + sums * sizeof(int32_t));
  w.lse2_at = w.dvec_at + rows;
  w.parts_at = w.lse2_at + rows;
  w.bytes = w.parts_at + sums * 128 * 2 * (size_t)sh->d * sizeof(float);
  return w;
}

}  // namespace

extern "C" {

void zp_prof_begin(const char *name, hipStream_t stream) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (!g_prof_on) return;
  ProfRec r{name, nullptr, nullptr};
  if (hipEventCreate(&r.a) != hipSuccess || hipEventCreate(&r.b) != hipSuccess) return;
  (void)hipEventRecord(r.a, stream);
  g_prof.push_back(r);
}
void zp_prof_end(hipStream_t stream) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (!g_prof_on || g_prof.empty()) return;
  (void)hipEventRecord(g_prof.back().b, stream);
}
int zp_profile_enable(int on) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  for (auto &r : g_prof) {
    (void)hipEventDestroy(r.a);
    (void)hipEventDestroy(r.b);
  }
  g_prof.clear();
  g_prof_on = on != 0;
  return ZP_OK;
}
int zp_profile_count(void) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  return (int)g_prof.size();
}
int zp_profile_get(int i, char *name, int name_cap, float *ms) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (i < 0 || i >= (int)g_prof.size() || !name || name_cap < 1 || !ms) return ZP_EINVAL;
  ZP_HIP(hipEventSynchronize(g_prof[i].b), "hipEventSynchronize");
  ZP_HIP(hipEventElapsedTime(ms, g_prof[i].a, g_prof[i].b), "hipEventElapsedTime");
  std::snprintf(name, (size_t)name_cap, "%s", g_prof[i].name);
  return ZP_OK;
}

// for the other translation units of the library: records the HIP error text and returns ZP_EHIP
int zp_report_hip_error(int hip_error, const char *what) { return hip_fail((hipError_t)hip_error, what); }

const char *zp_strerror(int code) {
  switch (code) {
    case ZP_OK: return "ok";
    case ZP_EINVAL: return "invalid argument";
    case ZP_EUNSUPPORTED: return "unsupported configuration";
    case ZP_EWORKSPACE: return "workspace missing, misaligned or too small";
    case ZP_EHIP: return g_hip_error.c_str();
    case ZP_ETOOLARGE: return "more sequences or tiles than the fixed limits of the no-allocation entry point";
    default: return "unknown error code";
  }
}

size_t zp_workspace_bytes(int which_fn, const zp_shape *sh, const int32_t *cu, int64_t n_desc) {
  if (check_shape(sh) != ZP_OK) return 0;
  switch (which_fn) {
    case ZP_FN_FWD: {
      if (check_cu(cu, sh) != ZP_OK) return 0;
      return tile_table_bytes((size_t)count_blocks(cu, sh->S, zp_attn_fwd_block_rows(sh->d))) + 256;
    }
    case ZP_FN_PARTIAL: {
      if (n_desc < 0) return 0;
      // a pair of q_len rows yields ceil(q_len / block_rows) tiles; bound it with T rows per pair... the exact
      // count needs the pairs, so this bound uses one tile per block_rows tokens of T plus one per pair, per pair
      const int bm = zp_attn_fwd_block_rows(sh->d);
      return tile_table_bytes((size_t)n_desc * ((size_t)sh->T / bm + 1)) + 256;
    }
    case ZP_FN_MERGE: {
      if (n_desc < 0) return 0;
      const int rpi = zp_merge_rows_per_item();
      return align256((size_t)n_desc * sizeof(zp_merge)) + align256(((size_t)sh->T / rpi + (size_t)n_desc + 1) * 8) + 256;
    }
    case ZP_FN_PARTIAL_BWD: {
      if (n_desc < 0) return 0;
      const size_t per_pair = (size_t)sh->T / zp_attn_bwd_block_rows(sh->d, 0) + (size_t)sh->T / zp_attn_bwd_block_rows(sh->d, 1) + 2;
      return tile_table_bytes((size_t)n_desc * per_pair) + 2 * align256((size_t)sh->Hq * (size_t)sh->T * sizeof(float)) + 512;
    }
    case ZP_FN_BWD: {
      if (check_cu(cu, sh) != ZP_OK) return 0;
      // (room for sums only where the call takes shares)
      const int bnk = zp_attn_bwd_block_rows(sh->d, 1), grp = sh->Hq / sh->Hkv;
      size_t tiles = (size_t)count_blocks(cu, sh->S, bnk), sums = 0;
      if (const int32_t share = plan_kv_shares(cu, sh, bnk)) {
        std::vector<CostTile> kt;
        plan_whole_keys(cu, sh->S, bnk, kt);
        float time;
        (void)dkdv_kernel_for(kt, sh->d, sh->Hkv, grp, &time);
        if (take_kv_shares(share, kt, sh->d, sh->Hkv, grp, time)) {
          sums = (size_t)share_blocks(kt, sh->d, grp, share) * (size_t)sh->Hkv;
          tiles = kt.size();
        }
      }
      return bwd_scratch((size_t)count_blocks(cu, sh->S, zp_attn_bwd_block_rows(sh->d, 0)) + tiles, sums, sh).bytes + 512;
    }
    default: return 0;
  }
}

int varlen_attn_fwd(const void *q, const void *k, const void *v, int64_t q_stride, int64_t k_stride, int64_t v_stride,
                    const int32_t *cu, const uint8_t *seq_skip, void *o, int64_t o_stride, float *lse,
                    const zp_shape *sh, void *ws, size_t ws_bytes, void *stream) {
  int rc = check_shape(sh);
  if (rc) return rc;
  if ((rc = check_cu(cu, sh))) return rc;
  if (sh->T == 0) return ZP_OK;
  if (!q || !k || !v || !o || !lse) return ZP_EINVAL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return ZP_EINVAL;
  if (check_stride(q_stride, sh->Hq, sh->d) || check_stride(o_stride, sh->Hq, sh->d) ||
      check_stride(k_stride, sh->Hkv, sh->d) || check_stride(v_stride, sh->Hkv, sh->d))
    return ZP_EINVAL;
  const int bm = zp_attn_fwd_block_rows(sh->d);
  std::vector<CostTile> tiles;
  tiles.reserve((size_t)count_blocks(cu, sh->S, bm));
  plan_whole(cu, sh->S, bm, tiles, seq_skip);
  if (tiles.empty()) return ZP_OK;
  if ((rc = check_ws(ws, ws_bytes, tile_table_bytes(tiles.size())))) return rc;
  zp_attn_params p{};
  const int64_t items = launch_items(tiles.size(), sh->Hkv, sh->Hq / sh->Hkv);
  if ((tiles_inline(tiles.size(), items) || !seqs_in_arguments(tiles, sh, ZP_SEQS_FWD, p.inl, p.n_seq)) &&
      (rc = place_tiles(tiles, items, p.inl, ws, (hipStream_t)stream, &p.tiles, &p.work.counters)))
    return rc;
  p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v;
  p.q_stride = q_stride; p.k_stride = k_stride; p.v_stride = v_stride;
  p.n_tiles = (int32_t)tiles.size(); p.work.dyn_div = dyn_div_of(tiles, 0, tiles.size(), 1);
  p.Hq = sh->Hq; p.Hkv = sh->Hkv; p.grp = sh->Hq / sh->Hkv;
  zp_plan_fwd_pair(p, sh->d);
  p.turns = fwd_turns(tiles, sh);
  p.scale = eff_scale(sh); p.scale_log2 = p.scale * 1.4426950408889634f;
  p.o = o; p.o_stride = o_stride; p.lse = lse; p.lse_stride = sh->T;
  hipError_t e = (hipError_t)zp_launch_attn_fwd(&p, sh->d, 0, bm, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "attn_fwd launch");
  return ZP_OK;
}

int chunk_attn_partial(const void *q, const void *k, const void *v, int64_t q_stride, int64_t k_stride,
                       int64_t v_stride, const zp_pair *pairs, int32_t n_pairs, float *o_part, float *lse_part,
                       int64_t part_rows, const zp_shape *sh, void *ws, size_t ws_bytes, void *stream) {
  int rc = check_shape(sh);
  if (rc) return rc;
  if (n_pairs < 0 || part_rows < 0) return ZP_EINVAL;
  if (n_pairs == 0) return ZP_OK;
  if (!q || !k || !v || !o_part || !lse_part || !pairs) return ZP_EINVAL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o_part)) return ZP_EINVAL;
  if (check_stride(q_stride, sh->Hq, sh->d) || check_stride(k_stride, sh->Hkv, sh->d) ||
      check_stride(v_stride, sh->Hkv, sh->d))
    return ZP_EINVAL;
  for (int i = 0; i < n_pairs; i++) {
    const zp_pair &pr = pairs[i];
    if (pr.q_len < 0 || pr.k_len < 0 || pr.q_tok0 < 0 || pr.k_tok0 < 0 || pr.q_pos0 < 0 || pr.k_pos0 < 0 ||
        pr.out_row0 < 0)
      return ZP_EINVAL;
    if ((int64_t)pr.q_tok0 + pr.q_len > sh->T || (int64_t)pr.k_tok0 + pr.k_len > sh->T) return ZP_EINVAL;
    if ((int64_t)pr.out_row0 + pr.q_len > part_rows) return ZP_EINVAL;
  }
  const int bm = zp_attn_fwd_block_rows(sh->d);
  std::vector<CostTile> tiles;
  tiles.reserve((size_t)count_pair_blocks(pairs, n_pairs, bm));
  for (int i = 0; i < n_pairs; i++) {
    const zp_pair &pr = pairs[i];
    for (int32_t r0 = 0; r0 < pr.q_len; r0 += bm) {
      CostTile c{};
      c.t.q_tok0 = pr.q_tok0 + r0;
      c.t.q_rows = std::min(bm, pr.q_len - r0);
      c.t.q_pos0 = pr.q_pos0 + r0;
      c.t.k_tok0 = pr.k_tok0;
      c.t.k_len = pr.k_len;
      c.t.k_pos0 = pr.k_pos0;
      c.t.out_row0 = pr.out_row0 + r0;
      c.cost = tile_cost(c.t);
      tiles.push_back(c);
    }
  }
  sort_by_cost(tiles);
  if ((rc = check_ws(ws, ws_bytes, tile_table_bytes(tiles.size())))) return rc;
  zp_attn_params p{};
  if ((rc = place_tiles(tiles, launch_items(tiles.size(), sh->Hkv, sh->Hq / sh->Hkv), p.inl, ws, (hipStream_t)stream, &p.tiles,
                        &p.work.counters)))
    return rc;
  p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v;
  p.q_stride = q_stride; p.k_stride = k_stride; p.v_stride = v_stride;
  p.n_tiles = (int32_t)tiles.size(); p.work.dyn_div = dyn_div_of(tiles, 0, tiles.size(), 1);
  p.Hq = sh->Hq; p.Hkv = sh->Hkv; p.grp = sh->Hq / sh->Hkv;
  zp_plan_fwd_pair(p, sh->d);
  p.turns = fwd_turns(tiles, sh);
  p.scale = eff_scale(sh); p.scale_log2 = p.scale * 1.4426950408889634f;
  p.o = o_part; p.o_stride = (int64_t)sh->Hq * sh->d; p.lse = lse_part; p.lse_stride = part_rows;
  hipError_t e = (hipError_t)zp_launch_attn_fwd(&p, sh->d, 1, bm, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "chunk_attn_partial launch");
  return ZP_OK;
}

int chunk_attn_update(const void *q, const void *k, const void *v, int64_t q_stride, int64_t k_stride, int64_t v_stride,
                      const zp_pair *pairs, int32_t n_pairs, float *o_run, float *lse_run, const zp_shape *sh,
                      void *ws, size_t ws_bytes, void *stream) {
  int rc = check_shape(sh);
  if (rc) return rc;
  if (n_pairs < 0) return ZP_EINVAL;
  if (n_pairs == 0 || sh->T == 0) return ZP_OK;
  if (!q || !k || !v || !o_run || !lse_run || !pairs) return ZP_EINVAL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o_run)) return ZP_EINVAL;
  if (check_stride(q_stride, sh->Hq, sh->d) || check_stride(k_stride, sh->Hkv, sh->d) ||
      check_stride(v_stride, sh->Hkv, sh->d))
    return ZP_EINVAL;
  // the running rows are read, merged and written back without atomics: a query row may appear in one pair only
  std::vector<std::pair<int32_t, int32_t>> qr;
  for (int i = 0; i < n_pairs; i++) {
    const zp_pair &pr = pairs[i];
    if (pr.q_len < 0 || pr.k_len < 0 || pr.q_tok0 < 0 || pr.k_tok0 < 0 || pr.q_pos0 < 0 || pr.k_pos0 < 0) return ZP_EINVAL;
    if ((int64_t)pr.q_tok0 + pr.q_len > sh->T || (int64_t)pr.k_tok0 + pr.k_len > sh->T) return ZP_EINVAL;
    if (pr.q_len > 0) qr.push_back({pr.q_tok0, pr.q_tok0 + pr.q_len});
  }
  std::sort(qr.begin(), qr.end());
  for (size_t i = 1; i < qr.size(); i++)
    if (qr[i].first < qr[i - 1].second) return ZP_EINVAL;
  const int bm = zp_attn_fwd_block_rows(sh->d);
  std::vector<CostTile> tiles;
  tiles.reserve((size_t)count_pair_blocks(pairs, n_pairs, bm));
  for (int i = 0; i < n_pairs; i++) {
    const zp_pair &pr = pairs[i];
    for (int32_t r0 = 0; r0 < pr.q_len; r0 += bm) {
      CostTile c{};
      c.t.q_tok0 = pr.q_tok0 + r0;
      c.t.q_rows = std::min(bm, pr.q_len - r0);
      c.t.q_pos0 = pr.q_pos0 + r0;
      c.t.k_tok0 = pr.k_tok0;
      c.t.k_len = pr.k_len;
      c.t.k_pos0 = pr.k_pos0;
      c.t.out_row0 = c.t.q_tok0;  // the running rows are the query's own token rows
      c.cost = tile_cost(c.t);
      if (c.cost > 0) tiles.push_back(c);  // a block that sees no key leaves its rows as they are
    }
  }
  if (tiles.empty()) return ZP_OK;
  sort_by_cost(tiles);
  if ((rc = check_ws(ws, ws_bytes, tile_table_bytes(tiles.size())))) return rc;
  zp_attn_params p{};
  if ((rc = place_tiles(tiles, launch_items(tiles.size(), sh->Hkv, sh->Hq / sh->Hkv), p.inl, ws, (hipStream_t)stream, &p.tiles,
                        &p.work.counters)))
    return rc;
  p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v;
  p.q_stride = q_stride; p.k_stride = k_stride; p.v_stride = v_stride;
  p.n_tiles = (int32_t)tiles.size(); p.work.dyn_div = dyn_div_of(tiles, 0, tiles.size(), 1);
  p.Hq = sh->Hq; p.Hkv = sh->Hkv; p.grp = sh->Hq / sh->Hkv;
  zp_plan_fwd_pair(p, sh->d);
  p.turns = fwd_turns(tiles, sh);
  p.scale = eff_scale(sh); p.scale_log2 = p.scale * 1.4426950408889634f;
  p.o = o_run; p.o_stride = (int64_t)sh->Hq * sh->d; p.lse = lse_run; p.lse_stride = sh->T;
  p.update = 1;
  hipError_t e = (hipError_t)zp_launch_attn_fwd(&p, sh->d, 1, bm, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "chunk_attn_update launch");
  return ZP_OK;
}

int lse_merge(const float *o_part, const float *lse_part, int64_t part_rows, const zp_merge *merges, int32_t n_merges,
              void *o, int64_t o_stride, float *lse, const zp_shape *sh, void *ws, size_t ws_bytes, void *stream) {
  int rc = check_shape(sh);
  if (rc) return rc;
  if (n_merges < 0 || part_rows < 0) return ZP_EINVAL;
  if (n_merges == 0) return ZP_OK;
  if (!o_part || !lse_part || !merges || !o || !lse) return ZP_EINVAL;
  if (!aligned16(o_part) || !aligned16(o)) return ZP_EINVAL;
  if (check_stride(o_stride, sh->Hq, sh->d)) return ZP_EINVAL;
  const int rpi = zp_merge_rows_per_item();
  size_t n_items = 0;
  for (int i = 0; i < n_merges; i++) {
    const zp_merge &m = merges[i];
    if (m.n_parts < 1 || m.n_parts > ZP_MAX_PARTS || m.len < 0 || m.out_tok0 < 0 ||
        (int64_t)m.out_tok0 + m.len > sh->T)
      return ZP_EINVAL;
    for (int p = 0; p < m.n_parts; p++)
      if (m.part_row0[p] < 0 || (int64_t)m.part_row0[p] + m.len > part_rows) return ZP_EINVAL;
    n_items += ((size_t)m.len + rpi - 1) / rpi;
  }
  const size_t desc_bytes = align256((size_t)n_merges * sizeof(zp_merge));
  const size_t item_bytes = n_items * 8;
  if ((rc = check_ws(ws, ws_bytes, desc_bytes + align256(item_bytes)))) return rc;
  if (n_items == 0) return ZP_OK;
  Upload u;
  if ((rc = upload_begin(desc_bytes + item_bytes, (hipStream_t)stream, u))) return rc;
  char *h = (char *)u.host;
  std::memcpy(h, merges, (size_t)n_merges * sizeof(zp_merge));
  int32_t *items = (int32_t *)(h + desc_bytes);
  size_t n = 0;
  for (int i = 0; i < n_merges; i++)
    for (int32_t r0 = 0; r0 < merges[i].len; r0 += rpi) {
      items[2 * n] = i;
      items[2 * n + 1] = r0;
      n++;
    }
  if ((rc = upload_send(u, ws, desc_bytes + item_bytes, (hipStream_t)stream))) return rc;
  int max_parts = 1;
  for (int i = 0; i < n_merges; i++) max_parts = std::max(max_parts, (int)merges[i].n_parts);
  hipError_t e = (hipError_t)zp_launch_lse_merge(o_part, lse_part, part_rows, ws, (char *)ws + desc_bytes, (int)n_items,
                                                 sh->Hq, sh->d, o, o_stride, lse, sh->T, max_parts, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "lse_merge launch");
  return ZP_OK;
}

int remap_tokens(const void *src, void *dst, int64_t row_bytes, const int32_t *idx_dev, int64_t n_rows, int32_t mode,
                 void *stream) {
  if (n_rows < 0 || row_bytes <= 0 || (mode != 0 && mode != 1)) return ZP_EINVAL;
  if (row_bytes % 16) return ZP_EUNSUPPORTED;
  if (n_rows == 0) return ZP_OK;
  if (!src || !dst || !idx_dev) return ZP_EINVAL;
  if (!aligned16(src) || !aligned16(dst)) return ZP_EINVAL;
  if (n_rows > 0x7fffffffLL || row_bytes > (1 << 20)) return ZP_EUNSUPPORTED;
  const char *s = (const char *)src;
  const char *d = (const char *)dst;
  const int64_t bytes = n_rows * row_bytes;
  if (s < d + bytes && d < s + bytes) return ZP_EINVAL;  // overlap
  hipError_t e = (hipError_t)zp_launch_remap(src, dst, row_bytes, idx_dev, n_rows, mode, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "remap_tokens launch");
  return ZP_OK;
}

int zp_chunk_pairs(int32_t tok0, int32_t L, int32_t C, int32_t rank, int32_t row0, zp_pair *pairs, int32_t max_pairs,
                   zp_merge *merges, int32_t max_merges, int32_t *n_merges, int64_t *rows_used) {
  if (L < 0 || C < 1 || tok0 < 0 || row0 < 0 || !pairs || !merges || !n_merges || !rows_used) return ZP_EINVAL;
  if (rank >= 0 && ((C & 1) || rank >= C / 2)) return ZP_EINVAL;
  auto bound = [&](int c) { return (int32_t)(((int64_t)c * L) / C); };
  int np = 0, nm = 0;
  int64_t row = row0;
  for (int qc = 0; qc < C; qc++) {
    if (rank >= 0 && qc != rank && qc != C - 1 - rank) continue;
    if (qc + 1 > ZP_MAX_PARTS) return ZP_EUNSUPPORTED;
    if (nm >= max_merges) return ZP_EINVAL;
    const int32_t qlen = bound(qc + 1) - bound(qc);
    zp_merge &m = merges[nm++];
    m.out_tok0 = tok0 + bound(qc);
    m.len = qlen;
    m.n_parts = qc + 1;
    for (int kc = 0; kc <= qc; kc++) {
      if (np >= max_pairs) return ZP_EINVAL;
      if (row + qlen > 0x7fffffffLL) return ZP_EINVAL;
      zp_pair &p = pairs[np++];
      p.q_tok0 = tok0 + bound(qc); p.q_len = qlen; p.q_pos0 = bound(qc);
      p.k_tok0 = tok0 + bound(kc); p.k_len = bound(kc + 1) - bound(kc); p.k_pos0 = bound(kc);
      p.out_row0 = (int32_t)row;
      m.part_row0[kc] = (int32_t)row;
      row += qlen;
    }
  }
  *n_merges = nm;
  *rows_used = row - row0;
  return np;
}

}  // extern "C"

extern "C" int varlen_attn_bwd(const void *dout, const void *q, const void *k, const void *v, const void *o,
                               const float *lse, int64_t do_stride, int64_t q_stride, int64_t k_stride,
                               int64_t v_stride, int64_t o_stride, const int32_t *cu, const uint8_t *seq_skip,
                               void *dq, void *dk, void *dv, int64_t dq_stride, int64_t dkv_stride,
                               const zp_shape *sh, void *ws, size_t ws_bytes, void *stream) {
  int rc = check_shape(sh);
  if (rc) return rc;
  if ((rc = check_cu(cu, sh))) return rc;
  if (sh->T == 0) return ZP_OK;
  if (!dout || !q || !k || !v || !o || !lse || !dq || !dk || !dv) return ZP_EINVAL;
  if (!aligned16(dout) || !aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(dq) ||
      !aligned16(dk) || !aligned16(dv))
    return ZP_EINVAL;
  if (check_stride(q_stride, sh->Hq, sh->d) || check_stride(o_stride, sh->Hq, sh->d) ||
      check_stride(do_stride, sh->Hq, sh->d) || check_stride(dq_stride, sh->Hq, sh->d) ||
      check_stride(k_stride, sh->Hkv, sh->d) || check_stride(v_stride, sh->Hkv, sh->d) ||
      check_stride(dkv_stride, sh->Hkv, sh->d))
    return ZP_EINVAL;
  const int bmq = zp_attn_bwd_block_rows(sh->d, 0), bnk = zp_attn_bwd_block_rows(sh->d, 1);
  std::vector<CostTile> qt, kt;
  qt.reserve((size_t)count_blocks(cu, sh->S, bmq));
  plan_whole(cu, sh->S, bmq, qt, seq_skip);
  plan_whole_keys(cu, sh->S, bnk, kt, seq_skip);
  if (qt.empty() && kt.empty()) return ZP_OK;
  const int grp = sh->Hq / sh->Hkv;
  float kv_time;
  KvKernel kv = dkdv_kernel_for(kt, sh->d, sh->Hkv, grp, &kv_time);
  int32_t slots = 0, share = 0;
  const bool inline_tiles = tiles_inline(qt.size() + kt.size(), launch_items(std::max(qt.size(), kt.size()), sh->Hkv, grp));
  if (!inline_tiles) {
    share = plan_kv_shares(cu, sh, bnk, seq_skip);
    if (take_kv_shares(share, kt, sh->d, sh->Hkv, grp, kv_time)) {
      std::vector<CostTile> cut = kt;
      slots = share_blocks(cut, sh->d, grp, share);
      // (not in a workspace that was sized for another batch or without the flags, which may have needed none for sums)
      if (ws_bytes < bwd_scratch(qt.size() + cut.size(), (size_t)slots * (size_t)sh->Hkv, sh).bytes) slots = 0;
      else {
        kv = KV_WHOLE;
        kt.swap(cut);
      }
    }
  }
  const size_t sums = (size_t)slots * (size_t)sh->Hkv;
  const BwdScratch at = bwd_scratch(qt.size() + kt.size(), sums, sh);
  if ((rc = check_ws(ws, ws_bytes, at.bytes))) return rc;
  std::vector<CostTile> all(qt);
  all.insert(all.end(), kt.begin(), kt.end());
  zp_bwd_params p{};
  if ((slots || inline_tiles || !seqs_in_arguments(qt, sh, ZP_SEQS_BWD, p.inl, p.n_seq)) &&
      (rc = place_tiles(all, launch_items(std::max(qt.size(), kt.size()), sh->Hkv, grp), p.inl, ws, (hipStream_t)stream, &p.dq_tiles,
                        &p.work_dq.counters, sums)))
    return rc;
  p.part_done = (int32_t *)((char *)ws + at.done_at);
  p.parts = (float *)((char *)ws + at.parts_at);
  p.share_its = slots ? share : 0;
  p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v; p.o = (const __bf16 *)o;
  p.dout = (const __bf16 *)dout;
  p.q_stride = q_stride; p.k_stride = k_stride; p.v_stride = v_stride; p.o_stride = o_stride; p.do_stride = do_stride;
  p.lse = lse;
  p.dvec = (float *)((char *)ws + at.dvec_at);
  p.lse2 = (float *)((char *)ws + at.lse2_at);
  p.kv_tiles = p.dq_tiles ? p.dq_tiles + qt.size() : nullptr;
  p.kv_pair = kv == KV_PAIR;
  p.kv_split = kv == KV_SPLIT;
  p.work_dq.dyn_div = dyn_div_of(all, 0, qt.size(), 1);
  p.work_kv.dyn_div = dyn_div_of(all, qt.size(), kt.size(), sh->Hq / sh->Hkv);
  p.n_dq_tiles = (int32_t)qt.size(); p.n_kv_tiles = (int32_t)kt.size();
  p.Hq = sh->Hq; p.Hkv = sh->Hkv; p.grp = sh->Hq / sh->Hkv; p.T = sh->T;
  zp_plan_dq_pair(p, sh->d);
  p.both = zp_take_both(p, sh->d);
  p.scale = eff_scale(sh); p.scale_log2 = p.scale * 1.4426950408889634f;
  p.dq = (__bf16 *)dq; p.dk = (__bf16 *)dk; p.dv = (__bf16 *)dv;
  p.dq_stride = dq_stride; p.dkv_stride = dkv_stride;
  hipError_t e = (hipError_t)zp_launch_attn_bwd(&p, sh->d, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "attn_bwd launch");
  return ZP_OK;
}

// Builds the dQ tiles (blocks of query rows of each pair's Q chunk against its KV chunk) and the dK/dV tiles (blocks
// of key rows of each pair's KV chunk against the Q-chunk rows that can see them) of one ring round.
static void plan_pairs_bwd(const zp_pair *pairs, int n_pairs, int bmq, int bnk, std::vector<CostTile> &qt,
                           std::vector<CostTile> &kt) {
  for (int i = 0; i < n_pairs; i++) {
    const zp_pair &pr = pairs[i];
    for (int32_t r0 = 0; r0 < pr.q_len; r0 += bmq) {
      CostTile c{};
      c.t.q_tok0 = pr.q_tok0 + r0; c.t.q_rows = std::min(bmq, pr.q_len - r0); c.t.q_pos0 = pr.q_pos0 + r0;
      c.t.k_tok0 = pr.k_tok0; c.t.k_len = pr.k_len; c.t.k_pos0 = pr.k_pos0;
      c.t.out_row0 = c.t.q_tok0;
      c.cost = tile_cost(c.t);
      if (c.cost > 0) qt.push_back(c);
    }
    for (int32_t j0 = 0; j0 < pr.k_len; j0 += bnk) {
      // first query row of the chunk that sees the block's first key
      const int32_t off = std::max(0, pr.k_pos0 + j0 - pr.q_pos0);
      if (off >= pr.q_len) continue;
      CostTile c{};
      c.t.k_tok0 = pr.k_tok0 + j0; c.t.k_len = std::min(bnk, pr.k_len - j0); c.t.k_pos0 = pr.k_pos0 + j0;
      c.t.q_tok0 = pr.q_tok0 + off; c.t.q_rows = pr.q_len - off; c.t.q_pos0 = pr.q_pos0 + off;
      c.t.out_row0 = c.t.k_tok0;
      c.cost = (c.t.q_rows + 63) / 64;
      kt.push_back(c);
    }
  }
  sort_by_cost(qt);
  sort_by_cost(kt);
}

extern "C" int chunk_attn_partial_bwd(const void *dout, const void *q, const void *k, const void *v, const void *o,
                                      const float *lse, int64_t do_stride, int64_t q_stride, int64_t k_stride,
                                      int64_t v_stride, int64_t o_stride, const zp_pair *pairs, int32_t n_pairs,
                                      float *dq_acc, float *dk_acc, float *dv_acc, const zp_shape *sh, void *ws,
                                      size_t ws_bytes, void *stream) {
  int rc = check_shape(sh);
  if (rc) return rc;
  if (n_pairs < 0) return ZP_EINVAL;
  if (n_pairs == 0 || sh->T == 0) return ZP_OK;
  if (!dout || !q || !k || !v || !o || !lse || !pairs || !dq_acc || !dk_acc || !dv_acc) return ZP_EINVAL;
  if (!aligned16(dout) || !aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(dq_acc) ||
      !aligned16(dk_acc) || !aligned16(dv_acc))
    return ZP_EINVAL;
  if (check_stride(q_stride, sh->Hq, sh->d) || check_stride(o_stride, sh->Hq, sh->d) ||
      check_stride(do_stride, sh->Hq, sh->d) || check_stride(k_stride, sh->Hkv, sh->d) ||
      check_stride(v_stride, sh->Hkv, sh->d))
    return ZP_EINVAL;
  // one ring round: every Q row and every KV row may appear in at most one pair (the kernels add without atomics)
  std::vector<std::pair<int32_t, int32_t>> qr, kr;
  for (int i = 0; i < n_pairs; i++) {
    const zp_pair &pr = pairs[i];
    if (pr.q_len < 0 || pr.k_len < 0 || pr.q_tok0 < 0 || pr.k_tok0 < 0 || pr.q_pos0 < 0 || pr.k_pos0 < 0) return ZP_EINVAL;
    if ((int64_t)pr.q_tok0 + pr.q_len > sh->T || (int64_t)pr.k_tok0 + pr.k_len > sh->T) return ZP_EINVAL;
    if (pr.q_len > 0) qr.push_back({pr.q_tok0, pr.q_tok0 + pr.q_len});
    if (pr.k_len > 0) kr.push_back({pr.k_tok0, pr.k_tok0 + pr.k_len});
  }
  for (auto *ranges : {&qr, &kr}) {
    std::sort(ranges->begin(), ranges->end());
    for (size_t i = 1; i < ranges->size(); i++)
      if ((*ranges)[i].first < (*ranges)[i - 1].second) return ZP_EINVAL;
  }
  const int bmq = zp_attn_bwd_block_rows(sh->d, 0), bnk = zp_attn_bwd_block_rows(sh->d, 1);
  std::vector<CostTile> qt, kt;
  plan_pairs_bwd(pairs, n_pairs, bmq, bnk, qt, kt);
  const size_t tile_bytes = tile_table_bytes(qt.size() + kt.size());
  const size_t dvec_bytes = align256((size_t)sh->Hq * (size_t)sh->T * sizeof(float));
  if ((rc = check_ws(ws, ws_bytes, tile_bytes + 2 * dvec_bytes))) return rc;
  std::vector<CostTile> all(qt);
  all.insert(all.end(), kt.begin(), kt.end());
  zp_bwd_params p{};
  if ((rc = place_tiles(all, launch_items(std::max(qt.size(), kt.size()), sh->Hkv, sh->Hq / sh->Hkv), p.inl, ws, (hipStream_t)stream,
                        &p.dq_tiles, &p.work_dq.counters)))
    return rc;
  p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v; p.o = (const __bf16 *)o;
  p.dout = (const __bf16 *)dout;
  p.q_stride = q_stride; p.k_stride = k_stride; p.v_stride = v_stride; p.o_stride = o_stride; p.do_stride = do_stride;
  p.lse = lse;
  p.dvec = (float *)((char *)ws + tile_bytes);
  p.lse2 = (float *)((char *)ws + tile_bytes + dvec_bytes);
  p.kv_tiles = p.dq_tiles ? p.dq_tiles + qt.size() : nullptr;
  float kv_time;
  const KvKernel kv = dkdv_kernel_for(kt, sh->d, sh->Hkv, sh->Hq / sh->Hkv, &kv_time);
  p.kv_pair = kv == KV_PAIR;
  p.kv_split = kv == KV_SPLIT;
  p.work_dq.dyn_div = dyn_div_of(all, 0, qt.size(), 1);
  p.work_kv.dyn_div = dyn_div_of(all, qt.size(), kt.size(), sh->Hq / sh->Hkv);
  p.n_dq_tiles = (int32_t)qt.size(); p.n_kv_tiles = (int32_t)kt.size();
  p.Hq = sh->Hq; p.Hkv = sh->Hkv; p.grp = sh->Hq / sh->Hkv; p.T = sh->T;
  zp_plan_dq_pair(p, sh->d);
  p.both = zp_take_both(p, sh->d);
  p.scale = eff_scale(sh); p.scale_log2 = p.scale * 1.4426950408889634f;
  p.dq = (__bf16 *)dq_acc; p.dk = (__bf16 *)dk_acc; p.dv = (__bf16 *)dv_acc;
  p.dq_stride = (int64_t)sh->Hq * sh->d; p.dkv_stride = (int64_t)sh->Hkv * sh->d;
  p.accumulate = 1;
  hipError_t e = (hipError_t)zp_launch_attn_bwd(&p, sh->d, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "chunk_attn_partial_bwd launch");
  return ZP_OK;
}

extern "C" int zp_accum_to_bf16(const float *src, void *dst, int64_t n, void *stream) {
  if (n < 0 || (n % 8)) return ZP_EINVAL;
  if (n == 0) return ZP_OK;
  if (!src || !dst || !aligned16(src) || !aligned16(dst)) return ZP_EINVAL;
  hipError_t e = (hipError_t)zp_launch_accum_to_bf16(src, dst, n, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "accum_to_bf16 launch");
  return ZP_OK;
}
