// Causal attention forward over a work list of (query block, key run) tiles: bf16 MFMA for K Q^T and V^T P^T,
// K/V tiles staged through LDS, online softmax kept per lane.
//
// Orientation. Scores are computed transposed, S^T = K Q^T with the 16x16x32 MFMA: accumulator lane l then holds ONE
// query (column l%16) and 4 keys per 16-key block (rows 4(l/16) + c). A wave owns two 16-query sub-blocks, so every K
// operand read from LDS feeds two MFMAs. The bf16 probabilities are already laid out as the B operand of
// O^T += V^T P^T (k-slots 0-3 of a lane are its keys of one 16-key block, 4-7 those of the next), and V^T comes from
// the row-major V tile in LDS through the transposing LDS read with the matching key order (zp_pad16_addr).
#include <type_traits>
#include "zp_common.h"

namespace {

constexpr int BN = 64;  // keys per LDS tile

// The partial sum of a lane's probabilities of a tile above which the reference maximum of its rows has to move.
constexpr float P_SUM_MAX = 4096.0f;

// A row's reference is worked out anew where `far` has one of its four lanes; m: this lane's largest score of the tile.
// Returns what the row's sums are multiplied by; its probabilities of the tile are taken again with ref. A row that has seen no
// key yet keeps waiting (nm = +inf), and every one of them is zero.
__device__ __forceinline__ float fwd_move_reference(uint64_t far, float m, float c_log2, float &nm, float &ref) {
  m = zp_quad_max(m) * c_log2;
  uint32_t rows = (uint32_t)far | (uint32_t)(far >> 32);  // the four lanes of a row are 16 apart
  rows = ((rows | rows >> 16) & 0xffff) * 0x10001u;
  const bool moves = __builtin_amdgcn_inverse_ballot_w64((uint64_t)rows << 32 | rows);
  const float mc_old = -nm, mc = moves ? fmaxf(mc_old, m) : mc_old;
  const bool none = mc == -INFINITY;
  const float alpha = none ? 1.0f : zp_exp2(mc_old - mc);
  nm = -mc;
  ref = none ? 0.f : -mc;
  return alpha;
}

// Asynchronous copies of the [64][D] tiles of one run of keys, tile by tile (see zp_stager). Neighbouring loads of a wave that
// differ by whole rows share a lane offset, and the rows are added to the scalar base.
template <int D, bool TURNS>
struct fwd_stager {
  typedef zp_pad16<D> L;
  static constexpr int PW = 64 * D * 2 / 1024 / 4, SHARE = TURNS ? PW / 2 : 1, ROWS = D == 128 ? 4 : 8;  // loads per wave and tile; per offset; rows of a load
  unsigned off[PW / SHARE];
  unsigned row_bytes;
  const char *tile;  // the next one
  int w;
  __device__ __forceinline__ void init(const __bf16 *first, int64_t tok_stride, int lane, int wave) {
    w = __builtin_amdgcn_readfirstlane(wave);
    row_bytes = (unsigned)tok_stride * 2;
    tile = (const char *)first;
#pragma unroll
    for (int i = 0; i < PW / SHARE; i++) off[i] = lane_offset(i * SHARE, lane, 64);
  }
  // of load n, for a tile of n_rows valid rows; the rows behind repeat the last one
  __device__ __forceinline__ unsigned lane_offset(int n, int lane, int n_rows) const {
    const int r = (w * PW + n) * ROWS + lane / (D / 8);
    return (unsigned)min(r, n_rows - 1) * row_bytes + (((lane & (D / 8 - 1)) ^ L::mask(r)) << 4);
  }
  // load N of a tile of 64 valid rows
  template <int N>
  __device__ __forceinline__ void piece(unsigned lds_tile) const {
    zp_dma16_so(zp_uniform_ptr(tile + (uint64_t)(N % SHARE * ROWS) * row_bytes), off[N / SHARE], __builtin_amdgcn_readfirstlane(lds_tile + L::group(w * PW + N)));
  }
  // the tile after the next one is the next one
  __device__ __forceinline__ void move() { tile += (uint64_t)64 * row_bytes; }
  // all loads of a tile of n_rows (64 or more: 64) valid rows
  __device__ __forceinline__ void issue(unsigned lds_tile, int n_rows) const {
    if (__builtin_expect(n_rows >= 64, 1)) {
      zp_static_for<PW>([&](auto n) { piece<decltype(n)::value>(lds_tile); });
    } else {
#pragma unroll
      for (int n = 0; n < PW; n++) {
        int ln = threadIdx.x & 63;
        asm volatile("" : "+v"(ln));  // keeps the rare path's offsets out of the registers of the loop around it
        zp_dma16_so(zp_uniform_ptr(tile), lane_offset(n, ln, n_rows), __builtin_amdgcn_readfirstlane(lds_tile + L::group(w * PW + n)));
      }
    }
  }
};

// The scores of NKB blocks of 16 keys from block KB0 of a tile on (at byte offset Kb) for one wave of two 16-query sub-blocks, as
// fenced steps of one LDS operand and the MFMAs it feeds (sub-blocks QB0 to QB1 - 1), operands requested two steps ahead.
// `piece(integral_constant<int, n>)` is called after step n.
template <int D, bool MASK, int QB0, int QB1, int KB0, int NKB, class Piece>
__device__ __forceinline__ void fwd_scores(int Kb, const bf16x8 (&qreg)[2][D / 32], f32x4 (&s)[2][NKB], int j0, int q4,
                                           const int (&nvis_lane)[2], const zp_pad16_addr<D> &la, Piece &&piece) {
  constexpr int N = NKB * (D / 32);  // operand n: key block n % NKB, k-step n / NKB
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  bf16x8 a[N];
  a[0] = la.rows(Kb, KB0, 0);
  a[1] = la.rows(Kb, KB0 + 1, 0);
  zp_static_for<N>([&](auto nn) {
    constexpr int n = nn.value, kb = n % NKB, k = n / NKB;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qb = QB0; qb < QB1; qb++)
      s[qb][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[n], qreg[qb][k], k == 0 ? zero : s[qb][kb], 0, 0, 0);
    if constexpr (n + 2 < N) a[n + 2] = la.rows(Kb, KB0 + (n + 2) % NKB, (n + 2) / NKB);
    piece(nn);
  });
  __builtin_amdgcn_sched_barrier(0);
  if (MASK) {
#pragma unroll
    for (int qb = QB0; qb < QB1; qb++)
#pragma unroll
      for (int kb = 0; kb < NKB; kb++)
#pragma unroll
        for (int r = 0; r < 4; r++)
          if (j0 + 16 * (KB0 + kb) + q4 + r >= nvis_lane[qb]) s[qb][kb][r] = -INFINITY;
  }
}

// Probabilities of NKB blocks of 16 keys: the B operands pb of their part of the second product, and the lane's sums over the keys
// of even (ta) and odd (tb) blocks.
template <int NKB>
__device__ __forceinline__ void fwd_take(const f32x4 (&s)[NKB], float c_log2, float ref, bf16x8 *pb, float &ta, float &tb) {
#pragma unroll
  for (int kb = 0; kb < NKB; kb++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const float p = zp_exp2(__builtin_fmaf(s[kb][r], c_log2, ref));
      // the row sum is taken over the unrounded probabilities: LSE has to hold to 1e-3 also for rows with few keys
      if (kb & 1) tb += p; else ta += p;
      pb[kb >> 1][(kb & 1) * 4 + r] = (__bf16)p;
    }
}
template <int NKB>
__device__ __forceinline__ float fwd_max(const f32x4 (&s)[NKB], float m) {
#pragma unroll
  for (int kb = 0; kb < NKB; kb++)
#pragma unroll
    for (int r = 0; r < 4; r++) m = fmaxf(m, s[kb][r]);
  return m;
}

// Scores and probabilities of one 64-key tile (K at byte offset Kb from the base the lane addresses carry, compile-time at the call
// sites) for one wave of two 16-query sub-blocks. ONLY1: no query of sub-block 0 sees a key of this tile. WHOLE: all scores first,
// else 32 keys at a time, which needs 16 registers less. FIRST: the rows' first tile (o_acc holds nothing yet), which gives them
// their reference. `between` is called in front of the softmax arithmetic of WHOLE and FIRST.
//
// The probabilities are taken against the reference the rows already have, nm = -(reference) in scaled log2 units, and
// only their sum is looked at: a maximum per tile costs 20 of 136 vector operations and puts a cross-lane exchange in
// front of the first exp2, while all that it protects against is a reference so far below the scores that the
// probabilities grow out of range. When the 16 probabilities of one of a row's four lanes add up to more than P_SUM_MAX
// (or to NaN), the row's maximum is worked out and its probabilities of the tile taken again (32 keys at a time: from scores
// multiplied out again, those of the first half are gone). A row that has seen no key yet has nm = +inf, which ends there. The
// other rows of the wave keep their reference, so that no bit of a row depends on the tokens behind it. Probabilities, sums and O
// are floating point throughout, so the reference's distance from the row maximum costs no precision.
//
// Bound: the power limit and the vector issue port. The 16x16x32 MFMA accumulates twice as many products per accumulator access as
// the 32x32x16; a register-only loop on random operands holds 1885-1956 TFLOP/s with it (zp_mfma_probe) against 1520-1800, at the
// price of twice the issue slots. On four 16384-token sequences (GQA 32/8, d = 128) the 32x32x16 form took 7.66 ms and this one 7.11.
template <int D, bool WHOLE, bool FIRST, bool MASK, bool ONLY1, class Piece, class Between>
__device__ __forceinline__ void fwd_tile_scores(int Kb, const bf16x8 (&qreg)[2][D / 32], bf16x8 (&pb)[2][2], f32x4 (&o_acc)[2][D / 16],
                                                float (&nm)[2], float (&l_sum)[2], float c_log2, int j0, int q4, const int (&nvis_lane)[2],
                                                const zp_pad16_addr<D> &la, Piece &&piece, Between &&between) {
  constexpr int DB = D / 16, QB0 = ONLY1 ? 1 : 0, N = 2 * (D / 32);
  auto no_piece = [](auto) {};
  auto second = [&](auto nn) { piece(std::integral_constant<int, N + decltype(nn)::value>{}); };
  float ta[2] = {0.f, 0.f}, tb[2] = {0.f, 0.f};
  if constexpr (WHOLE || FIRST) {
    f32x4 s[2][4];
    fwd_scores<D, MASK, QB0, 2, 0, 4>(Kb, qreg, s, j0, q4, nvis_lane, la, piece);
    between();
    auto take = [&](int qb, float ref) {
      ta[qb] = tb[qb] = 0.f;
      fwd_take(s[qb], c_log2, ref, pb[qb], ta[qb], tb[qb]);
    };
    uint64_t far[2] = {~0ull, ~0ull};  // lanes of out-of-range sums
    if constexpr (!FIRST) {
#pragma unroll
      for (int qb = QB0; qb < 2; qb++) take(qb, nm[qb]);
#pragma unroll
      for (int qb = QB0; qb < 2; qb++) far[qb] = __builtin_amdgcn_ballot_w64(!(ta[qb] + tb[qb] <= P_SUM_MAX));
    }
    // (unlikely: behind the loop's own code, which a short sequence's few tiles have to fetch as well)
    if (FIRST || __builtin_expect((far[QB0] | far[1]) != 0, 0)) {
#pragma unroll
      for (int qb = QB0; qb < 2; qb++) {
        float ref;
        const float alpha = fwd_move_reference(far[qb], fwd_max(s[qb], -INFINITY), c_log2, nm[qb], ref);
        if constexpr (!FIRST) {
          l_sum[qb] *= alpha;
#pragma unroll
          for (int i = 0; i < DB; i++)
#pragma unroll
            for (int r = 0; r < 4; r++) o_acc[qb][i][r] *= alpha;
        }
        take(qb, ref);
      }
    }
  } else {
    f32x4 s[2][2];
    fwd_scores<D, MASK, QB0, 2, 0, 2>(Kb, qreg, s, j0, q4, nvis_lane, la, piece);
#pragma unroll
    for (int qb = QB0; qb < 2; qb++) fwd_take(s[qb], c_log2, nm[qb], pb[qb], ta[qb], tb[qb]);
    fwd_scores<D, MASK, QB0, 2, 2, 2>(Kb, qreg, s, j0, q4, nvis_lane, la, second);
#pragma unroll
    for (int qb = QB0; qb < 2; qb++) fwd_take(s[qb], c_log2, nm[qb], pb[qb] + 1, ta[qb], tb[qb]);
    uint64_t far[2];  // lanes of out-of-range sums
#pragma unroll
    for (int qb = QB0; qb < 2; qb++) far[qb] = __builtin_amdgcn_ballot_w64(!(ta[qb] + tb[qb] <= P_SUM_MAX));
    // (unlikely: behind the loop's own code, which a short sequence's few tiles have to fetch as well)
    if (__builtin_expect((far[QB0] | far[1]) != 0, 0)) {
      zp_static_for<2 - QB0>([&](auto q) {
        constexpr int qb = QB0 + decltype(q)::value;
        if (far[qb] == 0) return;
        float m = -INFINITY, ref;
        zp_static_for<2>([&](auto half) {
          fwd_scores<D, MASK, qb, qb + 1, 2 * decltype(half)::value, 2>(Kb, qreg, s, j0, q4, nvis_lane, la, no_piece);
          m = fwd_max(s[qb], m);
        });
        const float alpha = fwd_move_reference(far[qb], m, c_log2, nm[qb], ref);
        l_sum[qb] *= alpha;
        ta[qb] = tb[qb] = 0.f;
#pragma unroll
        for (int i = 0; i < DB; i++)
#pragma unroll
          for (int r = 0; r < 4; r++) o_acc[qb][i][r] *= alpha;
        zp_static_for<2>([&](auto half) {
          fwd_scores<D, MASK, qb, qb + 1, 2 * decltype(half)::value, 2>(Kb, qreg, s, j0, q4, nvis_lane, la, no_piece);
          fwd_take(s[qb], c_log2, ref, pb[qb] + decltype(half)::value, ta[qb], tb[qb]);
        });
      });
    }
  }
#pragma unroll
  for (int qb = QB0; qb < 2; qb++) l_sum[qb] += ta[qb] + tb[qb];  // (zero before the first tile)
}

// The second product of the tile, V at byte offset Vb, operands three steps ahead.
template <int D, bool FIRST, bool ONLY1, class Piece>
__device__ __forceinline__ void fwd_tile_values(int Vb, const bf16x8 (&pb)[2][2], f32x4 (&o_acc)[2][D / 16], const zp_pad16_addr<D> &la,
                                                const bf16x8 (&ahead)[3], Piece &&piece) {
  constexpr int DB = D / 16, QB0 = ONLY1 ? 1 : 0;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  bf16x8 va[2 * DB];  // operand n: 32 keys n / DB, 16 columns n % DB
#pragma unroll
  for (int n = 0; n < 3; n++) va[n] = ahead[n];
  zp_static_for<2 * DB>([&](auto nn) {
    constexpr int n = nn.value, kp = n / DB, db = n % DB;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qb = QB0; qb < 2; qb++)
      o_acc[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[n], pb[qb][kp], FIRST && kp == 0 ? zero : o_acc[qb][db], 0, 0, 0);
    if constexpr (n + 3 < 2 * DB) va[n + 3] = la.cols(Vb + 2 * ((n + 3) / DB) * zp_pad16<D>::R16, (n + 3) % DB);
    piece(nn);
  });
  if constexpr (FIRST && ONLY1)
    for (int i = 0; i < DB; i++) o_acc[0][i] = zero;
  __builtin_amdgcn_sched_barrier(0);
}

// Normalises and writes O and LSE of a wave's QB sub-blocks of 16 rows (rb: their first rows in the block). own: LDS of the
// wave's own for zp_store_rows.
template <int D, bool PARTIAL, int QB>
__device__ __forceinline__ void fwd_finish(const zp_attn_params &p, const zp_tile &t, int h, int lane, const int (&rb)[QB],
                                           const f32x4 (&o_acc)[QB][D / 16], const float (&nm)[QB], const float (&l_sum)[QB], char *own) {
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
#pragma unroll
  for (int qb = 0; qb < QB; qb++) {
    const int row = rb[qb] + c16;
    const float l_tot = zp_quad_sum(l_sum[qb]);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    float lse = -INFINITY;
    {
#pragma clang fp contract(off)  // one rounding more or less from kernel to kernel otherwise
      if (l_tot > 0.f) lse = __logf(l_tot) - nm[qb] * 0.6931471805599453f;
    }
    const int64_t orow = (int64_t)t.out_row0 + row;
    if (PARTIAL) {
      if (row >= t.q_rows) continue;
      // weights of the running row (w_old) and of this partial (w_new, its 1/l folded in); without update: 0 and 1/l
      float w_old = 0.f, w_new = inv, lse_out = lse;
      if (p.update) {
        const float lse_old = p.lse[(int64_t)h * p.lse_stride + orow];
        const float mx = fmaxf(lse_old, lse);
        if (mx == -INFINITY) {
          w_new = 0.f;
        } else {
          const float e_old = __expf(lse_old - mx), e_new = __expf(lse - mx);
          const float tot = e_old + e_new;
          lse_out = mx + __logf(tot);
          w_old = e_old / tot;
          w_new = e_new / tot * inv;
        }
      }
      if (q4 == 0) p.lse[(int64_t)h * p.lse_stride + orow] = lse_out;
      float *op = (float *)p.o + orow * p.o_stride + (int64_t)h * D + q4;
#pragma unroll
      for (int db = 0; db < D / 16; db++) {
        f32x4 v4 = {o_acc[qb][db][0] * w_new, o_acc[qb][db][1] * w_new, o_acc[qb][db][2] * w_new, o_acc[qb][db][3] * w_new};
        if (w_old > 0.f) {  // a row that has seen no key yet may hold anything
          const f32x4 old = *(const f32x4 *)(op + db * 16);
          v4[0] += w_old * old[0]; v4[1] += w_old * old[1]; v4[2] += w_old * old[2]; v4[3] += w_old * old[3];
        }
        *(f32x4 *)(op + db * 16) = v4;
      }
    } else {
      if (q4 == 0 && row < t.q_rows) p.lse[(int64_t)h * p.lse_stride + orow] = lse;
      zp_store_rows<D>(own, o_acc[qb], inv, (__bf16 *)p.o + ((int64_t)t.out_row0 + rb[qb]) * p.o_stride + (int64_t)h * D,
                       p.o_stride, t.q_rows - rb[qb], lane);
    }
  }
}

// One workgroup of four waves per 128 query rows. Two forms:
//  - K and V of a tile and of the next one in four buffers, the next tile's copies spread over the score product, one barrier per tile;
//    two workgroups per CU at d = 128 (68 KB of LDS, 206 registers), three at 64 (32 KB, 154; 8 sequences of 4096 tokens, GQA 32/8:
//    631 us with two, 568 with three).
//  - TURNS (d = 128): three buffers by turns (51 KB), scores 32 keys at a time (168 registers), three workgroups per CU. The next K
//    tile comes in during the scores, the next V tile goes, behind a second barrier, where K was. A third wave on the SIMD fills what
//    the other two leave of its issue slots, above all while one of them starts or ends an item; a wave alone takes 15 % longer. 64K
//    lognormal tokens MHA, by counter, two -> three: SQ_ACTIVE_INST_ANY per SQ_BUSY_CU_CYCLES 0.82 -> 0.96, matrix pipe busy 0.49 -> 0.54 of
//    the cycles, which are 10 % fewer, at 1.85 instead of 1.91 GHz.
// A row's first tile has a body of its own: no probabilities against a reference that is not there yet, no zeros to add to.
// Two workgroups -> TURNS, us: 64K lognormal tokens MHA 1329 -> 1284, 64 x 1K MHA 729 -> 686, four sequences of 16384 7120 -> 7090,
// 700 of up to 59 tokens, 64/8 heads: 502 (without the first tile's body) -> 445 -> 353; one of 14351 among 33137 tokens, 4 heads:
// 289 -> 344. See zp_fwd_turns for which is taken. The results are the same bits.
template <int D, bool TURNS>
constexpr size_t fwd_lds() { return (TURNS ? 3 : 4) * 4 * (size_t)zp_pad16<D>::R16 + 16; }
template <int D, bool TURNS, bool PARTIAL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TURNS || D == 64 ? 3 : 2, TURNS || D == 64 ? 3 : 2))) void attn_fwd_kernel(zp_attn_params p) {
  constexpr int TILEB = 4 * zp_pad16<D>::R16;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int item = __builtin_amdgcn_readfirstlane(zp_item_of_block(p.work, (int *)(smem + (TURNS ? 3 : 4) * TILEB)));
  if (item < 0) return;
  int unit, hh;
  zp_block_to_unit(item, p.grp, p.m_grp, unit, hh);
  if (unit >= p.n_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const int h = g * p.grp + hh;
  const zp_tile t = ZP_TILE_OF(p.tiles, p.inl, p.n_seq, 0, false, tile_idx);

  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  // A wave's two sub-blocks of 16 query rows are the w-th from the front and the w-th from the back of the block, so
  // that all four waves see about the same number of keys and meet the barriers together.
  const int rb[2] = {16 * w, 16 * (7 - w)};
  const int row[2] = {rb[0] + c16, rb[1] + c16};  // this lane's query rows inside the block

  // number of keys of the run visible to a query row r: clamp(q_pos0 + r - k_pos0 + 1, 0, k_len)
  auto nvis_of = [&](int r) {
    int n = t.q_pos0 + r - t.k_pos0 + 1;
    return n < 0 ? 0 : (n > t.k_len ? t.k_len : n);
  };
  // rows behind the block's last one repeat it (and are not stored)
  const int rowc[2] = {min(row[0], t.q_rows - 1), min(row[1], t.q_rows - 1)};
  const int nvis_lane[2] = {nvis_of(rowc[0]), nvis_of(rowc[1])};
  // fewest and most keys a sub-block's rows see (none if the block ends before it)
  const int nvis0_min = nvis_of(rb[0]), nvis1_min = nvis_of(rb[1]);
  const int nvis0_max = rb[0] < t.q_rows ? nvis_of(rb[0] + 15) : 0, nvis1_max = rb[1] < t.q_rows ? nvis_of(rb[1] + 15) : 0;
  const int n_kt = (nvis_of(t.q_rows - 1) + BN - 1) / BN;

  // Q^T operands: 8 consecutive head-dim elements of this lane's queries per 32-wide k-step
  bf16x8 qreg[2][D / 32];
#pragma unroll
  for (int qb = 0; qb < 2; qb++) {
    const __bf16 *qp = p.q + (int64_t)(t.q_tok0 + rowc[qb]) * p.q_stride + (int64_t)h * D + 2 * q4;
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) qreg[qb][kk] = *(const bf16x8 *)(qp + 32 * kk);
  }
  // No wait here: the first tile copy is issued right behind these loads so that the two memory latencies of the
  // prologue overlap; the explicit wait in front of the first barrier covers both (and tells the compiler that the
  // register operands have arrived: a wait of its own inside the key loop would drain the copies in flight).

  typedef fwd_stager<D, TURNS> stager;
  constexpr int PW = stager::PW;
  stager kst, vst;
  kst.init(p.k + (int64_t)t.k_tok0 * p.k_stride + (int64_t)g * D, p.k_stride, lane, w);
  vst.init(p.v + (int64_t)t.k_tok0 * p.v_stride + (int64_t)g * D, p.v_stride, lane, w);
  zp_pad16_addr<D> la;
  la.init(lane, smem);
  const unsigned lds0 = zp_lds_addr(smem);

  f32x4 o_acc[2][D / 16];
  float nm[2] = {INFINITY, INFINITY};  // minus the running reference maximum, in scaled log2 units
  float l_sum[2] = {0.f, 0.f};         // this lane's share of the row sums
  const float c_log2 = p.scale_log2;

  if (n_kt > 0) {
    kst.issue(lds0, t.k_len);
    vst.issue(lds0 + TILEB, t.k_len);
  }
  kst.move();
  vst.move();
  zp_wait_async();
  __syncthreads();

  auto no_output = [&] {
#pragma unroll
    for (int qb = 0; qb < 2; qb++)
#pragma unroll
      for (int i = 0; i < D / 16; i++) o_acc[qb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // one key tile, K in LDS buffer KB (a compile-time constant, so every LDS address is register + immediate), V in VB, the next K
  // and V to KN and VN
  auto key_tile = [&](int it, auto KB, auto VB, auto KN, auto VN, auto first) {
    constexpr int Kb = decltype(KB)::value * TILEB, Vb = decltype(VB)::value * TILEB;
    constexpr bool FIRST = decltype(first)::value;
    const unsigned k_next = lds0 + decltype(KN)::value * TILEB, v_next = lds0 + decltype(VN)::value * TILEB;
    const int j0 = it * BN;
    // which sub-blocks have a row that sees a key of this tile, and whether some row sees only a part of it
    const bool act0 = j0 < nvis0_max, act1 = j0 < nvis1_max;
    const bool masked = j0 + BN > (act0 ? nvis0_min : nvis1_min);
    // the next tiles are fetched inside the products when they have 64 valid keys and this wave computes an unmasked tile (the
    // common case), else in front of them
    const bool fetch = it + 1 < n_kt;
    const bool fused = fetch && act0 && !masked && j0 + 2 * BN <= t.k_len;
    if (__builtin_expect(fetch && !fused, 0)) {
      kst.issue(k_next, t.k_len - j0 - BN);
      if constexpr (!TURNS) vst.issue(v_next, t.k_len - j0 - BN);
    }
    constexpr int EVERY = 4 * (D / 32) / PW / (TURNS ? 1 : 2);
    auto k_piece = [&](auto n) {
      constexpr int N = decltype(n)::value / EVERY;
      if constexpr (decltype(n)::value % EVERY != 0) return;
      else if constexpr (TURNS) kst.template piece<N>(k_next);
      else if constexpr (N % 2 == 0) kst.template piece<N / 2>(k_next);
      else vst.template piece<N / 2>(v_next);
    };
    auto v_piece = [&](auto n) {
      if constexpr (TURNS && decltype(n)::value % EVERY == 0) vst.template piece<decltype(n)::value / EVERY>(v_next);
    };
    auto no_piece = [](auto) {};
    bf16x8 pb[2][2], va[3];
    auto v_first = [&] {
#pragma unroll
      for (int n = 0; n < 3; n++) va[n] = la.cols(Vb, n);
    };
    auto v_ahead = [&] {
      if constexpr (!TURNS) v_first();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto scores = [&](auto mask, auto only1, auto &&piece) {
      fwd_tile_scores<D, !TURNS, FIRST, decltype(mask)::value, decltype(only1)::value>(Kb, qreg, pb, o_acc, nm, l_sum, c_log2, j0, q4, nvis_lane, la, piece, v_ahead);
    };
    auto values = [&](auto only1, auto &&piece) { fwd_tile_values<D, FIRST, decltype(only1)::value>(Vb, pb, o_acc, la, va, piece); };
    const std::true_type yes;
    const std::false_type no;
    if constexpr (TURNS) {
      if (!act0) { if (act1) scores(yes, yes, no_piece); }
      else if (masked) scores(yes, no, no_piece);
      else if (fused) scores(no, no, k_piece);
      else scores(no, no, no_piece);
      kst.move();
      // V of this tile has landed (the next K may be in flight), and everybody is done with K
      if (fetch) zp_wait_async_upto<PW>();
      else zp_wait_async();
      __syncthreads();
      if (__builtin_expect(fetch && !fused, 0)) vst.issue(v_next, t.k_len - j0 - BN);
      v_first();
      if (!act0) { if (act1) values(yes, no_piece); else if (FIRST) no_output(); }
      else if (fused) values(no, v_piece);
      else values(no, no_piece);
    } else {
      if (!act0) {
        if (act1) { scores(yes, yes, no_piece); values(yes, no_piece); }
        else if (FIRST) no_output();
      } else if (masked) { scores(yes, no, no_piece); values(no, no_piece); }
      else if (fused) { scores(no, no, k_piece); values(no, no_piece); }
      else { scores(no, no, no_piece); values(no, no_piece); }
      kst.move();
    }
    vst.move();
    // the next K (and V, or it may be in flight) has landed, and everybody is done with V
    if (TURNS && fetch) zp_wait_async_upto<PW>();
    else zp_wait_async();
    if (!TURNS || fetch) __syncthreads();
  };
#define ZP_N(n) std::integral_constant<int, n>{}
  if (n_kt == 0) {
    no_output();
  } else if constexpr (TURNS) {
    key_tile(0, ZP_N(0), ZP_N(1), ZP_N(2), ZP_N(0), std::true_type{});
    for (int it = 1; it < n_kt; it += 3) {
      key_tile(it, ZP_N(2), ZP_N(0), ZP_N(1), ZP_N(2), std::false_type{});
      if (it + 1 < n_kt) key_tile(it + 1, ZP_N(1), ZP_N(2), ZP_N(0), ZP_N(1), std::false_type{});
      if (it + 2 < n_kt) key_tile(it + 2, ZP_N(0), ZP_N(1), ZP_N(2), ZP_N(0), std::false_type{});
    }
  } else {
    key_tile(0, ZP_N(0), ZP_N(1), ZP_N(2), ZP_N(3), std::true_type{});
    for (int it = 1; it < n_kt; it += 2) {
      key_tile(it, ZP_N(2), ZP_N(3), ZP_N(0), ZP_N(1), std::false_type{});
      if (it + 1 < n_kt) key_tile(it + 1, ZP_N(0), ZP_N(1), ZP_N(2), ZP_N(3), std::false_type{});
    }
  }
#undef ZP_N
  if (TURNS) __syncthreads();  // the rows go out through the tiles' LDS
  int ln = threadIdx.x & 63;
  asm volatile("" : "+v"(ln));  // worked out again: what depends on the lane would keep registers through the loop
  fwd_finish<D, PARTIAL, 2>(p, t, h, ln, rb, o_acc, nm, l_sum, smem + w * ZP_ROWS_LDS);
}

// ---- launches that leave much of the chip idle: two waves per 16 query rows ---------------------------------------
// The score wave of a pair: softmax arithmetic of a tile (SM, s -> pn; 2: masked) with the score product of the next one (SC:
// K at lk, into sn) spread over it. Returns the lanes whose rows' reference moved; their O is then to be multiplied by alpha.
// What a row computes, and in which order, is what attn_fwd_kernel computes: the results are the same bits.
// ahead: the first K operands, requested by the step before; on return those of the tile behind (lk moves there by `step`).
constexpr int PAIR_KA = 4;
template <int D, int SM, bool SC>
__device__ __forceinline__ uint64_t fwd_pair_scores(const bf16x8 (&qreg)[D / 32], bf16x8 (&pn)[2], f32x4 (&s)[4], f32x4 (&sn)[4], float &nm,
                                                    float &l_sum, float &alpha, float c_log2, int j0, int q4, int nvis_lane,
                                                    zp_pad16_addr<D> &lk, bf16x8 (&ahead)[PAIR_KA], int step) {
  constexpr int N = SC ? 4 * (D / 32) : 0, KA = PAIR_KA, EP = N ? N : 1;
  constexpr int LEAD = SC ? 0 : 18;  // steps of the softmax arithmetic in front of the first MFMA
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  bf16x8 a[N + KA];
  if constexpr (SC)
    for (int n = 0; n < KA; n++) a[n] = ahead[n];
  float ta = 0.f, tb = 0.f, x[16];
  // step e: element e's fma, e - 1's exp2, e - 2's sum and conversion
  auto stage = [&](auto ee, auto st) {
    constexpr int e = decltype(ee)::value, kb = e / 4, r = e % 4;
    if constexpr (SM == 0 || e < 0 || e >= 16) return;
    else if constexpr (decltype(st)::value == 0) {
      if (SM == 2 && j0 + 16 * kb + q4 + r >= nvis_lane) s[kb][r] = -INFINITY;
      x[e] = __builtin_fmaf(s[kb][r], c_log2, nm);
    } else if constexpr (decltype(st)::value == 1) {
      x[e] = zp_exp2(x[e]);
    } else {
      if (kb & 1) tb += x[e]; else ta += x[e];
      pn[kb >> 1][(kb & 1) * 4 + r] = (__bf16)x[e];
    }
  };
  auto arith = [&](auto from, auto to) {
    zp_static_for<decltype(to)::value - decltype(from)::value>([&](auto i) {
      constexpr int e = decltype(from)::value + decltype(i)::value;
      stage(std::integral_constant<int, e>{}, std::integral_constant<int, 0>{});
      stage(std::integral_constant<int, e - 1>{}, std::integral_constant<int, 1>{});
      stage(std::integral_constant<int, e - 2>{}, std::integral_constant<int, 2>{});
    });
  };
  __builtin_amdgcn_sched_barrier(0);
  arith(std::integral_constant<int, 0>{}, std::integral_constant<int, LEAD>{});
  zp_static_for<N>([&](auto nn) {
    constexpr int n = nn.value;
    __builtin_amdgcn_sched_barrier(0);
    sn[n % 4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[n], qreg[n / 4], n / 4 == 0 ? zero : sn[n % 4], 0, 0, 0);
    if constexpr (n + KA < N) a[n + KA] = lk.rows(0, (n + KA) % 4, (n + KA) / 4);
    else {
      if constexpr (n + KA == N) lk.move_rows(step);
      ahead[n + KA - N] = lk.rows(0, (n + KA - N) % 4, (n + KA - N) / 4);
    }
    arith(std::integral_constant<int, LEAD + n * (18 - LEAD) / EP>{}, std::integral_constant<int, LEAD + (n + 1) * (18 - LEAD) / EP>{});
  });
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (SM == 0) return 0;
  float t = ta + tb;
  const uint64_t far = __builtin_amdgcn_ballot_w64(!(t <= P_SUM_MAX));
  if (__builtin_expect(far != 0, 0)) {
    float m = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 4; kb++)
#pragma unroll
      for (int r = 0; r < 4; r++) m = fmaxf(m, s[kb][r]);
    float ref;
    alpha = fwd_move_reference(far, m, c_log2, nm, ref);
    l_sum *= alpha;
    ta = tb = 0.f;
#pragma unroll
    for (int kb = 0; kb < 4; kb++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const float p = zp_exp2(__builtin_fmaf(s[kb][r], c_log2, ref));
        if (kb & 1) tb += p; else ta += p;
        pn[kb >> 1][(kb & 1) * 4 + r] = (__bf16)p;
      }
    t = ta + tb;
  }
  l_sum += t;
  return far;
}

// The value wave: the second product of a tile (V at lv), the probabilities p of its rows, and whether (and by what) O is
// multiplied first. ahead, step: as above.
template <int D>
constexpr int PAIR_VA = D / 16;
template <int D>
__device__ __forceinline__ void fwd_pair_values(f32x4 (&o_acc)[D / 16], const bf16x8 (&p)[2], int moved, unsigned al, zp_pad16_addr<D> &lv,
                                                bf16x8 (&ahead)[PAIR_VA<D>], int step) {
  constexpr int DB = D / 16, N = 2 * DB, VA = PAIR_VA<D>;
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(moved) != 0, 0)) {
    const float alpha = *(const ZP_LDS float *)(unsigned long long)al;
#pragma unroll
    for (int i = 0; i < DB; i++)
#pragma unroll
      for (int r = 0; r < 4; r++) o_acc[i][r] *= alpha;
  }
  bf16x8 va[N];
  for (int n = 0; n < VA; n++) va[n] = ahead[n];
  zp_static_for<N>([&](auto nn) {
    constexpr int n = nn.value;
    __builtin_amdgcn_sched_barrier(0);
    o_acc[n % DB] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[n], p[n / DB], o_acc[n % DB], 0, 0, 0);
    constexpr int v = n + VA;
    if constexpr (v < N) va[v] = lv.cols(2 * (v / DB) * zp_pad16<D>::R16, v % DB);
    else {
      if constexpr (v == N) lv.move_cols(step);
      ahead[v - N] = lv.cols(2 * ((v - N) / DB) * zp_pad16<D>::R16, (v - N) % DB);
    }
  });
  __builtin_amdgcn_sched_barrier(0);
}

constexpr int PAIR_BUFS = 4;  // staged K and V tiles: 136 KB of the 156 KB of LDS at d = 128
template <int D>
constexpr size_t pair_lds() { return 2 * PAIR_BUFS * 4 * (size_t)zp_pad16<D>::R16 + 2 * 4 * 2048 + 4 * 4 * 256 + 2 * 4 * 16; }

// 64 query rows per workgroup of eight waves: waves 0-3 work out the scores and probabilities of 16 rows each, waves 4-7, on
// the same SIMDs, the second product of the same rows one tile behind them, and issue the copies. Probabilities pass through
// LDS, two tiles' worth; one barrier per tile.
//
// Bound: the serial chain of a workgroup's key tiles. A wave's MFMAs, LDS reads, copies and vector operations issue one after
// the other, so a wave alone on its SIMD takes their sum: 2450 cycles per tile with attn_fwd_kernel (32 rows per wave, d =
// 128), 1850 with 16 rows per wave and one wave per SIMD, also when its products and arithmetic are pipelined across
// tiles, and 1450 with two waves that share the work (1750, 1350 and 1120 at d = 64). Of these 1450 the score wave's own
// operations are about 1200: sixteen exp2 and what goes with them 450, MFMAs and K operands 450, the rest hand-over and
// barrier. One sequence of 4000 tokens, 4 heads: 71.4 -> 43.3 us at d = 128, 51.9 -> 33.5 at 64; 300 tokens: 10.1 -> 7.3
// and 8.0 -> 6.1. It works on half as many rows per CU as attn_fwd_kernel at twice the LDS reads per MFMA, so that launches
// that fill the chip are faster there: zp_plan_fwd_pair has the rule.
template <int D, bool PARTIAL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 4))) void attn_fwd_pair_kernel(zp_attn_params p) {
  constexpr int TILEB = 4 * zp_pad16<D>::R16, NB = PAIR_BUFS;
  typedef zp_stager<D, 4, true> stager;
  constexpr int PW = stager::PER_WAVE;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char *Ks = smem;                  // [NB][BN][D]: tile j in buffer j % NB
  char *Vs = smem + NB * TILEB;     // [NB][BN][D]
  char *Ps = smem + 2 * NB * TILEB; // [2][4][2][64 x 16 bytes]: a tile's probabilities, pair by pair
  char *As = Ps + 2 * 4 * 2048;     // [2][4][64]: what O is multiplied by; behind them the rows' sums and references
  char *Fs = As + 4 * 4 * 256;      // [2][4]: whether it is

  int unit, hh;
  int half;
  zp_block_to_unit(zp_pair_item(p.pair, blockIdx.x, half), p.grp, p.m_grp, unit, hh);
  if (unit >= p.n_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const int h = g * p.grp + hh;
  zp_tile t = ZP_TILE((const zp_tile *)nullptr, p.inl, 0, tile_idx);
  if (!zp_pair_rows(t, half)) return;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
  const bool values = __builtin_amdgcn_readfirstlane(tid >> 8) != 0;
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  const int rb = 16 * w;
  auto nvis_of = [&](int r) {
    int n = t.q_pos0 + r - t.k_pos0 + 1;
    return n < 0 ? 0 : (n > t.k_len ? t.k_len : n);
  };
  // rows behind the block's last one repeat it (and are not stored)
  const int nvis_lane = nvis_of(min(rb + c16, t.q_rows - 1)), nvis_min = nvis_of(rb);
  const int n_kt = (nvis_of(t.q_rows - 1) + BN - 1) / BN;              // tiles the workgroup stages
  const int n_w = rb < t.q_rows ? (nvis_of(min(rb + 15, t.q_rows - 1)) + BN - 1) / BN : 0;  // tiles this pair's rows see

  stager kst, vst;
  kst.init(p.k + (int64_t)t.k_tok0 * p.k_stride + (int64_t)g * D, p.k_stride, tid & 255);
  vst.init(p.v + (int64_t)t.k_tok0 * p.v_stride + (int64_t)g * D, p.v_stride, tid & 255);
  static_assert(NB == 4, "the counts of copies in flight below");
  const int n4 = min(n_kt, NB);
  const unsigned own_p = zp_lds_addr(Ps) + w * 2048 + lane * 16, own_a = zp_lds_addr(As) + w * 256 + lane * 4, own_f = zp_lds_addr(Fs) + w * 16;

  if (!values) {
    // the block's query rows (to the buffer of V that is filled last) and K of the first NB tiles
    {
      stager qst;
      qst.init(p.q + (int64_t)t.q_tok0 * p.q_stride + (int64_t)h * D, p.q_stride, tid);
      qst.issue(Vs + (NB - 1) * TILEB, 0, t.q_rows);
    }
#pragma unroll
    for (int j = 0; j < NB; j++)
      if (j < n_kt) kst.issue(Ks + j * TILEB, j * BN, t.k_len);
    zp_pad16_addr<D> lk;  // of the K tile in hand
    lk.init(lane, Ks);
    float nm = INFINITY, l_sum = 0.f, alpha = 1.f;
    const float c_log2 = p.scale_log2;
    f32x4 s[2][4];  // scores of tile j in s[j % 2]
    bf16x8 pb[2];
    // the query rows and K of tile 0; behind them K of the others
    if (n4 == 4) zp_wait_async_upto<3 * PW>();
    else if (n4 == 3) zp_wait_async_upto<2 * PW>();
    else if (n4 == 2) zp_wait_async_upto<PW>();
    else zp_wait_async();
    __syncthreads();
    bf16x8 qreg[D / 32], ahead[PAIR_KA];
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) {
      const unsigned at = lk.row[kk & 1] + (unsigned)((2 * NB - 1) * TILEB + w * zp_pad16<D>::R16 + (kk >> 1) * 128);
      qreg[kk] = *(const ZP_LDS bf16x8 *)(unsigned long long)at;
    }
#pragma unroll
    for (int n = 0; n < PAIR_KA; n++) ahead[n] = lk.rows(0, n % 4, n / 4);
    if (n_w > 0) {
      int no_step = 0;
      fwd_pair_scores<D, 0, true>(qreg, pb, s[0], s[0], nm, l_sum, alpha, c_log2, 0, q4, nvis_lane, lk, ahead, no_step);
    }
    lk.move_rows(TILEB);
    zp_wait_async();
    auto key_tile = [&](int it, auto PAR) {
      constexpr int par = decltype(PAR)::value;
      // K of tile it + 2 and what the value wave needs next have landed; the value wave is done with the probabilities two
      // tiles back
      __syncthreads();
      if (it == 0) {
#pragma unroll
        for (int n = 0; n < PAIR_KA; n++) ahead[n] = lk.rows(0, n % 4, n / 4);
      }
      if (it < n_w) {
        uint64_t far;
        const int j0 = it * BN, step = ((it + 1) & (NB - 1)) == NB - 1 ? -(NB - 1) * TILEB : TILEB;
        if (it + 1 >= n_w) far = fwd_pair_scores<D, 2, false>(qreg, pb, s[par], s[par ^ 1], nm, l_sum, alpha, c_log2, j0, q4, nvis_lane, lk, ahead, step);
        else if (j0 + BN > nvis_min) far = fwd_pair_scores<D, 2, true>(qreg, pb, s[par], s[par ^ 1], nm, l_sum, alpha, c_log2, j0, q4, nvis_lane, lk, ahead, step);
        else far = fwd_pair_scores<D, 1, true>(qreg, pb, s[par], s[par ^ 1], nm, l_sum, alpha, c_log2, j0, q4, nvis_lane, lk, ahead, step);
        *(ZP_LDS bf16x8 *)(unsigned long long)(own_p + par * 4 * 2048) = pb[0];
        *(ZP_LDS bf16x8 *)(unsigned long long)(own_p + par * 4 * 2048 + 1024) = pb[1];
        *(ZP_LDS int *)(unsigned long long)(own_f + par * 64) = far != 0;
        if (far != 0) *(ZP_LDS float *)(unsigned long long)(own_a + par * 1024) = alpha;
      }
    };
    for (int it = 0; it < n_kt; it += 2) {
      key_tile(it, std::integral_constant<int, 0>{});
      if (it + 1 < n_kt) key_tile(it + 1, std::integral_constant<int, 1>{});
    }
    *(ZP_LDS float *)(unsigned long long)(own_a + 2048) = l_sum;
    *(ZP_LDS float *)(unsigned long long)(own_a + 3072) = nm;
    __syncthreads();  // the last tile's probabilities, the rows' sums and references
  } else {
#pragma unroll
    for (int j = 0; j < NB - 1; j++)
      if (j < n_kt) vst.issue(Vs + j * TILEB, j * BN, t.k_len);
    zp_pad16_addr<D> lv;  // of the V tile in hand
    lv.init(lane, Vs);
    f32x4 o_acc[1][D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; i++) o_acc[0][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();  // (the score waves' first product)
    bf16x8 ahead[PAIR_VA<D>];
    for (int it = 0; it <= n_kt; it++) {
      // V of tile it and K of it + 2 have landed (behind them V of it + 1 and K of it + 3), the probabilities of tile it - 1
      // are there; everybody is done with K of tile it and V of it - 2
      if (it + 3 < n_kt) zp_wait_async_upto<2 * PW>();
      else if (it + 1 < n_kt) zp_wait_async_upto<PW>();
      else zp_wait_async();
      __syncthreads();
      const unsigned par = (it - 1) & 1;
      bf16x8 pr[2];
      int moved;
      if (it > 0) {
        moved = *(const ZP_LDS int *)(unsigned long long)(own_f + par * 64);
        pr[0] = *(const ZP_LDS bf16x8 *)(unsigned long long)(own_p + par * 4 * 2048);
        pr[1] = *(const ZP_LDS bf16x8 *)(unsigned long long)(own_p + par * 4 * 2048 + 1024);
      } else {
#pragma unroll
        for (int n = 0; n < PAIR_VA<D>; n++) ahead[n] = lv.cols(2 * (n / (D / 16)) * zp_pad16<D>::R16, n % (D / 16));
      }
      if (it + NB < n_kt) kst.issue(Ks + (it & (NB - 1)) * TILEB, (it + NB) * BN, t.k_len);
      if (it > 0 && it - 2 + NB < n_kt) vst.issue(Vs + ((it - 2) & (NB - 1)) * TILEB, (it - 2 + NB) * BN, t.k_len);
      if (it > 0 && it <= n_w)
        fwd_pair_values<D>(o_acc[0], pr, moved, own_a + par * 1024, lv, ahead, ((it - 1) & (NB - 1)) == NB - 1 ? -(NB - 1) * TILEB : TILEB);
    }
    const float l_sum[1] = {*(const ZP_LDS float *)(unsigned long long)(own_a + 2048)}, nm[1] = {*(const ZP_LDS float *)(unsigned long long)(own_a + 3072)};
    // K's buffers are free: the rows go out through them
    fwd_finish<D, PARTIAL, 1>(p, t, h, lane, {rb}, o_acc, nm, l_sum, Ks + w * ZP_ROWS_LDS_OF(D));
  }
}

}  // namespace

extern "C" void zp_prof_begin(const char *name, hipStream_t stream);
extern "C" void zp_prof_end(hipStream_t stream);

// Host-side launcher used by the C ABI. Returns a hipError_t as int.
extern "C" int zp_launch_attn_fwd(const zp_attn_params *p, int d, int partial, int block_rows, hipStream_t stream) {
  const int units = p->n_tiles * p->Hkv;
  if (units == 0) return 0;
  zp_attn_params q = *p;
  q.m_hkv = zp_div_magic(p->Hkv); q.m_grp = zp_div_magic(p->grp);
  const int grid = zp_plan_work_split(q.work, p->work.counters, ((units + 7) / 8) * 8 * p->grp);
  p = &q;
  (void)block_rows;
  if (q.pair) {
    const int pair_grid = ((units + 7) / 8) * 8 * p->grp * (q.pair == ZP_PAIR_HALVES ? 2 : 1);
    zp_prof_begin(partial ? "attn_fwd_partial_pair" : "attn_fwd_pair", stream);
#define ZP_FWD_PAIR(D, PART) hipLaunchKernelGGL((attn_fwd_pair_kernel<D, PART>), dim3(pair_grid), dim3(512), pair_lds<D>(), stream, q)
    if (d == 128) {
      if (partial) ZP_FWD_PAIR(128, true); else ZP_FWD_PAIR(128, false);
    } else {
      if (partial) ZP_FWD_PAIR(64, true); else ZP_FWD_PAIR(64, false);
    }
#undef ZP_FWD_PAIR
    zp_prof_end(stream);
    return (int)hipGetLastError();
  }
#define ZP_FWD_LAUNCH(D, TURNS, PART)                                                                   \
  do {                                                                                                  \
    zp_prof_begin(PART ? (TURNS ? "attn_fwd_partial_turns" : "attn_fwd_partial") : TURNS ? "attn_fwd_turns" : "attn_fwd", stream); \
    hipLaunchKernelGGL((attn_fwd_kernel<D, TURNS, PART>), dim3(grid), dim3(256), (fwd_lds<D, TURNS>()), stream, *p); \
    zp_prof_end(stream);                                                                                \
  } while (0)
  if (d == 128) {
    if (p->turns) {
      if (partial) ZP_FWD_LAUNCH(128, true, true); else ZP_FWD_LAUNCH(128, true, false);
    } else {
      if (partial) ZP_FWD_LAUNCH(128, false, true); else ZP_FWD_LAUNCH(128, false, false);
    }
  } else {
    if (partial) ZP_FWD_LAUNCH(64, false, true); else ZP_FWD_LAUNCH(64, false, false);
  }
#undef ZP_FWD_LAUNCH
  return (int)hipGetLastError();
}

extern "C" int zp_attn_fwd_block_rows(int d) { (void)d; return 128; }
