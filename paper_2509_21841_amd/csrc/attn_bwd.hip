// Backward of causal varlen attention, two kernels. Deterministic: no result is added to by atomics. (Shares of a block of keys count
// themselves done by an atomic, which decides who adds their sums up, not in which order: dkdv_join_parts.) Short launches do both
// kernels' work in one, behind a small one for the row terms (attn_bwd_both_kernel).
//   attn_bwd_dq   owns a block of query rows, walks the visible key tiles:  S^T = K Q^T, dP^T = V dO^T,
//                 dS^T = P^T o (dP^T - D), dQ^T += K^T dS^T.  Also computes D_i = dO_i . O_i and stores it.
//   attn_bwd_dkdv owns a block of key rows, walks the query tiles at or after it and the query heads of its
//                 KV group:  S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.
// Both recompute P from the forward's LSE. In each kernel the accumulator of the first two products already
// has the register layout the third/fourth product needs as its B operand; the transposed A operands
// (K^T, Q^T, dO^T) come from the row-major LDS tiles through the transposing LDS read.
#include <algorithm>
#include <type_traits>
#include "zp_common.h"

namespace {

constexpr int BWD_NT = 256;
constexpr float LOG2E = 1.4426950408889634f;

// adds the scaled accumulators of one row to float values: 4 consecutive columns of every 16
template <int D>
__device__ __forceinline__ void add_acc_rows(float *dst, const f32x4 (&acc)[D / 16], float mul) {
#pragma unroll
  for (int db = 0; db < D / 16; db++) {
    f32x4 cur = *(const f32x4 *)(dst + db * 16);
    cur[0] += acc[db][0] * mul; cur[1] += acc[db][1] * mul; cur[2] += acc[db][2] * mul; cur[3] += acc[db][3] * mul;
    *(f32x4 *)(dst + db * 16) = cur;
  }
}

// D = dO . O of a lane's row, whose four lanes hold 8 consecutive head-dim elements of every 32 each. The dot instruction rounds once
// per two products: 32 of N(0, 1) values are off by 1.90e-7 (rms, against 64 bits), 1.97e-7 as a chain of fused multiply-adds, for
// a sixth of the vector operations.
template <int D>
__device__ __forceinline__ float row_d(const bf16x8 (&doreg)[D / 32], const bf16x8 (&oreg)[D / 32]) {
  float sum = 0.f;
#pragma unroll
  for (int kk = 0; kk < D / 32; kk++)
#pragma unroll
    for (int e = 0; e < 8; e += 2)
      sum = __builtin_amdgcn_fdot2_f32_bf16((bf16x2){doreg[kk][e], doreg[kk][e + 1]}, (bf16x2){oreg[kk][e], oreg[kk][e + 1]}, sum, false);
  return zp_quad_sum(sum);
}

// ------------------------------------------------------------------------------------------- dQ
// 32 of a tile's 64 keys (half `half`) for one wave of two 16-query sub-blocks: S^T and dP^T, dS^T, dQ^T += K^T dS^T, all on the
// 16x16x32 MFMA (attn_fwd.hip has the orientation and the layouts; zp_lds16 the LDS side). Steps of one LDS operand
// and the two MFMAs it feeds are fenced, operands requested two (rows) and three (transposed) steps ahead, the first two
// transposed ones in front of the dS arithmetic. ONLY1: no query of sub-block 0 sees a key of this half.
// `piece(integral_constant<int, n>)` is called in every second step of the first two products when PIECES is set: the
// caller issues one asynchronous copy of the next tile there, far enough apart that none waits for the address unit
// behind the copies of the other waves. Kb, Vb: byte offsets of the K and V tile from the base the lane offsets carry.
template <int D, bool MASK, bool ONLY1, bool PIECES, class Piece>
__device__ __forceinline__ void dq_half(int Kb, int Vb, int half, const bf16x8 (&qreg)[2][D / 32],
                                        const bf16x8 (&doreg)[2][D / 32], f32x4 (&dq_acc)[2][D / 16], float c_log2,
                                        const float (&lse2)[2], const f32x4 (&negD)[2], int j0, int q4,
                                        const int (&nvis_lane)[2], const zp_lds16<D> &lo, Piece &&piece) {
  constexpr int KK = D / 32, DB = D / 16, N = 4 * KK, QB0 = ONLY1 ? 1 : 0;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  // the dP^T chains start from -D (a lane holds one query per sub-block): the accumulator then holds dP - D
  f32x4 s[2][2], dp[2][2];
  bf16x8 x[N];  // operand n: K and V alternating, key block n / 2 % 2 of the half, k-step n / 4
  auto load = [&](auto nn) {
    constexpr int n = decltype(nn)::value;
    if constexpr (n < N) x[n] = lo.rows_at(n % 2 ? Vb : Kb, 2 * half + n / 2 % 2, n / 4);
  };
  load(std::integral_constant<int, 0>{});
  load(std::integral_constant<int, 1>{});
  zp_static_for<N>([&](auto nn) {
    constexpr int n = nn.value, kb = n / 2 % 2, k = n / 4;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qb = QB0; qb < 2; qb++) {
      if constexpr (n % 2 == 0) s[qb][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], qreg[qb][k], k == 0 ? zero : s[qb][kb], 0, 0, 0);
      else dp[qb][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], doreg[qb][k], k == 0 ? negD[qb] : dp[qb][kb], 0, 0, 0);
    }
    load(std::integral_constant<int, n + 2>{});
    if constexpr (PIECES && n % 2 == 0) piece(std::integral_constant<int, n / 2>{});
  });
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 xt[DB];
  xt[0] = lo.tr_at(Kb, half, 0);
  xt[1] = lo.tr_at(Kb, half, 1);
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 dsb[2];
#pragma unroll
  for (int qb = QB0; qb < 2; qb++)
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        float pv = zp_exp2(__builtin_fmaf(s[qb][kb][r], c_log2, -lse2[qb]));
        if (MASK && j0 + 32 * half + 16 * kb + q4 + r >= nvis_lane[qb]) pv = 0.f;
        dsb[qb][4 * kb + r] = (__bf16)(pv * dp[qb][kb][r]);
      }
  xt[2] = lo.tr_at(Kb, half, 2);
  zp_static_for<DB>([&](auto nn) {
    constexpr int n = nn.value;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qb = QB0; qb < 2; qb++)
      dq_acc[qb][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[n], dsb[qb], dq_acc[qb][n], 0, 0, 0);
    if constexpr (n + 3 < DB) xt[n + 3] = lo.tr_at(Kb, half, n + 3);
  });
  __builtin_amdgcn_sched_barrier(0);
}

// Two waves per SIMD (two workgroups of four waves per CU, 64 KB of LDS each). An MFMA takes about 20 cycles of the
// issuing wave's vector issue time, and a wave issues its LDS, scalar and wait instructions one after the other as
// well; with a second wave on the SIMD all of that runs under the other wave's MFMAs. Working through a tile in two
// 32-key halves keeps the wave within the 256 registers this needs. Three at head dimension 64 (168 registers, 32 KB of
// LDS): 8 sequences of 4096 tokens, GQA 32/8, 761 us with two and 713 with three; 64 x 1K MHA 561 and 481.
template <int D>
__global__ __launch_bounds__(BWD_NT) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2, D == 64 ? 3 : 2))) void attn_bwd_dq_kernel(zp_bwd_params p) {
  constexpr int TILEB = 64 * D * 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char *Ks = smem;               // [2][64][D]
  char *Vs = smem + 2 * TILEB;   // [2][64][D]

  const int item = __builtin_amdgcn_readfirstlane(zp_item_of_block(p.work_dq, (int *)(smem + 4 * TILEB)));
  if (item < 0) return;
  int unit, hh;
  zp_block_to_unit(item, p.grp, p.m_grp, unit, hh);
  if (unit >= p.n_dq_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const int h = g * p.grp + hh;
  const zp_tile t = ZP_TILE_OF(p.dq_tiles, p.inl, p.n_seq, 0, false, tile_idx);

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  // the wave's two sub-blocks of 16 query rows, the w-th from the front and the w-th from the back of the block, so that
  // all four waves see about the same number of keys
  const int rb[2] = {16 * w, 16 * (7 - w)};
  const int row[2] = {rb[0] + c16, rb[1] + c16};

  auto nvis_of = [&](int r) {
    int n = t.q_pos0 + r - t.k_pos0 + 1;
    return n < 0 ? 0 : (n > t.k_len ? t.k_len : n);
  };
  // rows behind the block's last one repeat it (and are not stored)
  const int rowc[2] = {min(row[0], t.q_rows - 1), min(row[1], t.q_rows - 1)};
  const int nvis_lane[2] = {nvis_of(rowc[0]), nvis_of(rowc[1])};
  const int nvis0_min = nvis_of(rb[0]), nvis1_min = nvis_of(rb[1]);
  const int nvis0_max = rb[0] < t.q_rows ? nvis_of(rb[0] + 15) : 0, nvis1_max = rb[1] < t.q_rows ? nvis_of(rb[1] + 15) : 0;
  const int n_kt = (nvis_of(t.q_rows - 1) + 63) / 64;

  zp_stager<D> kst, vst;
  kst.init(p.k + (int64_t)t.k_tok0 * p.k_stride + (int64_t)g * D, p.k_stride, tid);
  vst.init(p.v + (int64_t)t.k_tok0 * p.v_stride + (int64_t)g * D, p.v_stride, tid);
  zp_lds16<D> lo;
  lo.init_abs(lane, smem);

  // Row operands first, the first tile copy right behind them (the two memory latencies overlap), their first use
  // after that. The explicit wait before the first barrier covers all of it and tells the compiler that the register
  // operands have arrived (a wait of its own inside the key loop would drain the copies in flight every iteration).
  bf16x8 qreg[2][D / 32], doreg[2][D / 32], oreg[2][D / 32];
  float lse_nat[2];
#pragma unroll
  for (int qb = 0; qb < 2; qb++) {
    const int64_t tok = (int64_t)t.q_tok0 + rowc[qb];
    const __bf16 *qp = p.q + tok * p.q_stride + (int64_t)h * D + 2 * q4;
    const __bf16 *dop = p.dout + tok * p.do_stride + (int64_t)h * D + 2 * q4;
    const __bf16 *op = p.o + tok * p.o_stride + (int64_t)h * D + 2 * q4;
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) {
      qreg[qb][kk] = *(const bf16x8 *)(qp + 32 * kk);
      doreg[qb][kk] = *(const bf16x8 *)(dop + 32 * kk);
      oreg[qb][kk] = *(const bf16x8 *)(op + 32 * kk);
    }
    lse_nat[qb] = p.lse[(int64_t)h * p.T + tok];
  }
  if (n_kt > 0) {
    kst.issue(Ks, 0, t.k_len);
    vst.issue(Vs, 0, t.k_len);
  }
  float lse2[2];
  f32x4 negD[2];
#pragma unroll
  for (int qb = 0; qb < 2; qb++) {
    const float Dq = row_d<D>(doreg[qb], oreg[qb]);
    lse2[qb] = lse_nat[qb] * LOG2E;
    negD[qb] = f32x4{-Dq, -Dq, -Dq, -Dq};
    if (row[qb] < t.q_rows && q4 == 0) {
      // negated and pre-divided so that the second kernel can seed its MFMA accumulators with them
      const int64_t at = (int64_t)h * p.T + t.q_tok0 + row[qb];
      p.dvec[at] = -Dq;
      p.lse2[at] = -lse_nat[qb] / p.scale;
    }
  }

  f32x4 dq_acc[2][D / 16];
#pragma unroll
  for (int qb = 0; qb < 2; qb++)
#pragma unroll
    for (int i = 0; i < D / 16; i++) dq_acc[qb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c_log2 = p.scale_log2;

  zp_wait_async();
  __syncthreads();

  constexpr int PW = zp_stager<D>::PER_WAVE;
  // one key tile out of LDS buffer BUF (compile-time, so that every LDS address is a register plus an immediate)
  auto key_tile = [&](int it, auto BUF) {
    constexpr int buf = decltype(BUF)::value;
    const int j0 = it * 64;
    const bool act0 = j0 < nvis0_max, act1 = j0 < nvis1_max;  // sub-blocks with a row that sees a key of this tile
    const bool compute = act0 || act1;
    const bool masked = j0 + 64 > (act0 ? nvis0_min : nvis1_min);
    // the next tile is fetched inside the first half of this tile's arithmetic when it has 64 valid keys and this
    // wave computes an unmasked tile (the common case), else in front of it
    const bool fetch = it + 1 < n_kt;
    const bool fused = fetch && act0 && !masked && j0 + 128 <= t.k_len;
    if (fetch && !fused) {
      kst.issue(Ks + (buf ^ 1) * TILEB, j0 + 64, t.k_len);
      vst.issue(Vs + (buf ^ 1) * TILEB, j0 + 64, t.k_len);
    }
    // the same copies one load at a time, K and V alternating (2 * PW loads = one per k-step)
    // (the sources are worked out unconditionally: a value defined under a branch would not stay in scalar registers)
    const void *pc_k = zp_uniform_ptr(kst.base + (int64_t)(j0 + 64) * kst.stride);
    const void *pc_v = zp_uniform_ptr(vst.base + (int64_t)(j0 + 64) * vst.stride);
    auto stage_piece = [&](auto n) {
      constexpr int N = decltype(n)::value, i = N / 2;
      static_assert(2 * PW == 2 * (D / 32), "one copy per two steps");
      if constexpr (N % 2 == 0)
        zp_dma16_so(pc_k, kst.off[i], __builtin_amdgcn_readfirstlane(zp_lds_addr(Ks + (buf ^ 1) * TILEB) + (kst.w * PW + i) * 1024));
      else
        zp_dma16_so(pc_v, vst.off[i], __builtin_amdgcn_readfirstlane(zp_lds_addr(Vs + (buf ^ 1) * TILEB) + (vst.w * PW + i) * 1024));
    };
    if (compute) {
      constexpr int Kb = buf * TILEB, Vb = (2 + buf) * TILEB;  // byte offsets of the tiles from smem
      if (masked || !act0) {
        // the halves of a tile on the diagonal one by one: a half that none of the wave's rows sees is left out
        if (act0) dq_half<D, true, false, false>(Kb, Vb, 0, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
        else dq_half<D, true, true, false>(Kb, Vb, 0, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
        if (j0 + 32 < nvis0_max) dq_half<D, true, false, false>(Kb, Vb, 1, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
        else if (j0 + 32 < nvis1_max) dq_half<D, true, true, false>(Kb, Vb, 1, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
      } else if (fused) {
        dq_half<D, false, false, true>(Kb, Vb, 0, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
        dq_half<D, false, false, false>(Kb, Vb, 1, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
      } else {
        dq_half<D, false, false, false>(Kb, Vb, 0, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
        dq_half<D, false, false, false>(Kb, Vb, 1, qreg, doreg, dq_acc, c_log2, lse2, negD, j0, q4, nvis_lane, lo, stage_piece);
      }
    }
    zp_wait_async();
    __syncthreads();
  };
  for (int it = 0; it < n_kt; it += 2) {
    key_tile(it, std::integral_constant<int, 0>{});
    if (it + 1 < n_kt) key_tile(it + 1, std::integral_constant<int, 1>{});
  }

#pragma unroll
  for (int qb = 0; qb < 2; qb++) {
    const int64_t at = ((int64_t)t.q_tok0 + rb[qb]) * p.dq_stride + (int64_t)h * D;
    if (!p.accumulate) zp_store_rows<D>(smem + w * ZP_ROWS_LDS, dq_acc[qb], p.scale, p.dq + at, p.dq_stride, t.q_rows - rb[qb], lane);
    else if (row[qb] < t.q_rows) add_acc_rows<D>((float *)p.dq + at + c16 * p.dq_stride + q4, dq_acc[qb], p.scale);
  }
}

// ---- dQ of launches that leave much of the chip idle: two waves per 16 query rows
// A wave's LDS read addresses: K and V rows of its 32 keys of the tile in hand, and the transposed K operands of its half of
// the columns of the tile before.
template <int D>
struct dq_pair_addr {
  typedef zp_pad16<D> L;
  static constexpr int NC = D / 32;  // 16-column blocks of a wave
  unsigned k[2], v[2], t[NC];
  __device__ __forceinline__ void init(int lane, int half, const char *ks, const char *vs) {
#pragma unroll
    for (int par = 0; par < 2; par++) {
      const int at = L::row_part(lane, par) + half * 2 * L::R16;
      k[par] = zp_lds_addr(ks) + at;
      v[par] = zp_lds_addr(vs) + at;
      asm volatile("" : "+v"(k[par]), "+v"(v[par]));  // opaque: see zp_lds16
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      t[c] = zp_lds_addr(ks) + (D == 128 ? L::tr_part(lane, c) + half * 128 : L::tr_part(lane, 2 * half + c));
      asm volatile("" : "+v"(t[c]));
    }
  }
  __device__ __forceinline__ bf16x8 rows(const unsigned (&a)[2], int rb, int kk) const {
    return *(const ZP_LDS bf16x8 *)(unsigned long long)(a[kk & 1] + rb * L::R16 + (kk >> 1) * 128);
  }
  __device__ __forceinline__ bf16x8 cols(int h, int c) const {
    const unsigned o = t[c] + h * 2 * L::R16;
    s16x4 u0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)o);
    s16x4 u1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)(o + L::R16));
    return zp_cat(__builtin_bit_cast(bf16x4, u0), __builtin_bit_cast(bf16x4, u1));
  }
};

// A step of one wave of a pair: S^T, dP^T and dS^T of its 32 keys of a tile (SP; dS to LDS address out), and dQ^T += K^T dS^T of
// the tile before for its columns (DQ: dS of that tile's two halves at in; the second one only if `both`).
template <int D, bool SP, bool MASK, bool DQ, class Copies>
__device__ __forceinline__ void dq_pair_step(const bf16x8 (&qreg)[D / 32], const bf16x8 (&doreg)[D / 32], f32x4 (&dq_acc)[D / 32], float c_log2,
                                             float lse2, const f32x4 &negD, int key0, int q4, int nvis_lane, const dq_pair_addr<D> &la,
                                             unsigned in, unsigned out, bool both, Copies &&copies) {
  constexpr int KK = D / 32, NC = D / 32, N1 = SP ? 4 * KK : 0, N2 = DQ ? 2 * NC : 0, XA = 6;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  bf16x8 x[N1 + 1], xt[N2 + 1], dsb[2];
  f32x4 s[2], dp[2];
  auto load = [&](auto nn) {  // operand n: K and V alternating, 16 keys n / 2 % 2, k-step n / 4
    constexpr int n = decltype(nn)::value;
    if constexpr (n < N1) x[n] = la.rows(n % 2 ? la.v : la.k, n / 2 % 2, n / 4);
  };
  zp_static_for<XA>(load);
  if constexpr (DQ) {
    dsb[0] = *(const ZP_LDS bf16x8 *)(unsigned long long)in;
    dsb[1] = *(const ZP_LDS bf16x8 *)(unsigned long long)(in + 1024);
  }
  __builtin_amdgcn_sched_barrier(0);
  copies();  // while the first operands arrive
  zp_static_for<N1>([&](auto nn) {
    constexpr int n = nn.value, kb = n / 2 % 2, k = n / 4;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (n % 2 == 0) s[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], qreg[k], k == 0 ? zero : s[kb], 0, 0, 0);
    else dp[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], doreg[k], k == 0 ? negD : dp[kb], 0, 0, 0);
    load(std::integral_constant<int, n + XA>{});
    if constexpr (N2 != 0 && n % 2 == 1) xt[n / 2] = la.cols(n / 2 / NC, n / 2 % NC);
  });
  __builtin_amdgcn_sched_barrier(0);
  // dS element e: its fma, exp2, product and conversion one step apart, over the MFMAs of the second product
  float e0[8];
  bf16x8 dsn;
  auto stage = [&](auto ee, auto st) {
    constexpr int e = decltype(ee)::value, kb = e / 4, r = e % 4;
    if constexpr (!SP || e < 0 || e >= 8) return;
    else if constexpr (decltype(st)::value == 0) e0[e] = __builtin_fmaf(s[kb][r], c_log2, -lse2);
    else if constexpr (decltype(st)::value == 1) {
      e0[e] = zp_exp2(e0[e]);
      if (MASK && key0 + 16 * kb + q4 + r >= nvis_lane) e0[e] = 0.f;
    } else dsn[e] = (__bf16)(e0[e] * dp[kb][r]);
  };
  auto arith = [&](auto ee) {
    constexpr int e = decltype(ee)::value;
    stage(std::integral_constant<int, e>{}, std::integral_constant<int, 0>{});
    stage(std::integral_constant<int, e - 1>{}, std::integral_constant<int, 1>{});
    stage(std::integral_constant<int, e - 2>{}, std::integral_constant<int, 2>{});
  };
  if constexpr (DQ) {
    if constexpr (!SP) zp_static_for<N2>([&](auto nn) { xt[nn.value] = la.cols(nn.value / NC, nn.value % NC); });
    zp_static_for<N2>([&](auto nn) {
      constexpr int n = nn.value, h = n / NC, c = n % NC;
      __builtin_amdgcn_sched_barrier(0);
      if (SP || h == 0 || both) dq_acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[n], dsb[h], dq_acc[c], 0, 0, 0);
      zp_static_for<10 / N2>([&](auto u) { arith(std::integral_constant<int, n * (10 / N2) + decltype(u)::value>{}); });
    });
    __builtin_amdgcn_sched_barrier(0);
    zp_static_for<10 - 10 / N2 * N2>([&](auto u) { arith(std::integral_constant<int, 10 / N2 * N2 + decltype(u)::value>{}); });
  } else {
    zp_static_for<10>([&](auto u) { arith(u); });
  }
  if constexpr (SP) *(ZP_LDS bf16x8 *)(unsigned long long)out = dsn;
}

constexpr int PAIR_BUFS = 4;
template <int D>
constexpr size_t dq_pair_lds() { return 2 * PAIR_BUFS * 4 * (size_t)zp_pad16<D>::R16 + 2 * 4 * 2048; }

// 64 query rows per workgroup of eight waves. Waves w and w + 4 share 16 rows: each works out dS for 32 of a tile's 64 keys,
// hands it over through LDS, and adds the tile before to dQ for half of the columns. One barrier per tile. What a row
// computes, and in which order, is what attn_bwd_dq_kernel computes.
//
// Bound: the serial chain of a workgroup's key tiles (see attn_fwd_pair_kernel). Per tile 2850 cycles with
// attn_bwd_dq_kernel alone on a CU and 2250 here at d = 128, 1930 and 1550 at d = 64; MFMAs alone take 1070 of the 2250, the
// arithmetic between them 800, operand reads and copies the rest. Forward and backward of 1218 tokens, GQA 4/2, d = 128:
// dQ 14.0 -> 11.6 us; zp_plan_dq_pair has more figures and the rule.
// block: of the kernel's own. PRE: D and -LSE / scale have been worked out (attn_bwd_rows_kernel).
template <int D, bool PRE>
__device__ __forceinline__ void dq_pair_rows(const zp_bwd_params &p, int block, char *smem) {
  constexpr int TILEB = 4 * zp_pad16<D>::R16, NB = PAIR_BUFS;
  typedef zp_stager<D, 8, true> stager;
  constexpr int PW = stager::PER_WAVE;
  char *Ks = smem;                   // [NB][64][D]: tile j in buffer j % NB
  char *Vs = smem + NB * TILEB;      // [NB][64][D]
  char *Ss = smem + 2 * NB * TILEB;  // [2][4][2][64 x 16 bytes]: a tile's dS, pair by pair, half by half

  int unit, hh;
  int part;
  zp_block_to_unit(zp_pair_item(p.dq_pair, block, part), p.grp, p.m_grp, unit, hh);
  if (unit >= p.n_dq_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const int h = g * p.grp + hh;
  zp_tile t = ZP_TILE((const zp_tile *)nullptr, p.inl, 0, tile_idx);
  if (!zp_pair_rows(t, part)) return;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
  const int half = __builtin_amdgcn_readfirstlane(tid >> 8);
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  const int rb = 16 * w, row = rb + c16;
  auto nvis_of = [&](int r) {
    int n = t.q_pos0 + r - t.k_pos0 + 1;
    return n < 0 ? 0 : (n > t.k_len ? t.k_len : n);
  };
  const int rowc = min(row, t.q_rows - 1);  // rows behind the block's last one repeat it (and are not stored)
  const int nvis_lane = nvis_of(rowc), nvis_min = nvis_of(rb), nvis_max = rb < t.q_rows ? nvis_of(rb + 15) : 0;
  const int n_kt = (nvis_of(t.q_rows - 1) + 63) / 64;

  stager kst, vst;
  kst.init(p.k + (int64_t)t.k_tok0 * p.k_stride + (int64_t)g * D, p.k_stride, tid);
  vst.init(p.v + (int64_t)t.k_tok0 * p.v_stride + (int64_t)g * D, p.v_stride, tid);
  // row operands first, the first two tiles' copies right behind them (see attn_bwd_dq_kernel)
  bf16x8 qreg[D / 32], doreg[D / 32], oreg[D / 32];  // (PRE: not O)
  const int64_t tok = (int64_t)t.q_tok0 + rowc;
#pragma unroll
  for (int kk = 0; kk < D / 32; kk++) {
    qreg[kk] = *(const bf16x8 *)(p.q + tok * p.q_stride + (int64_t)h * D + 2 * q4 + 32 * kk);
    doreg[kk] = *(const bf16x8 *)(p.dout + tok * p.do_stride + (int64_t)h * D + 2 * q4 + 32 * kk);
    if (!PRE) oreg[kk] = *(const bf16x8 *)(p.o + tok * p.o_stride + (int64_t)h * D + 2 * q4 + 32 * kk);
  }
  const float lse_nat = p.lse[(int64_t)h * p.T + tok];
  const float minus_d = PRE ? p.dvec[(int64_t)h * p.T + tok] : 0.f;
#pragma unroll
  for (int j = 0; j < 2; j++)
    if (j < n_kt) {
      kst.issue(Ks + j * TILEB, 64 * j, t.k_len);
      vst.issue(Vs + j * TILEB, 64 * j, t.k_len);
    }
  dq_pair_addr<D> la;
  la.init(lane, half, Ks, Vs);
  const unsigned own = zp_lds_addr(Ss) + w * 2048 + lane * 16;
  const float Dq = PRE ? -minus_d : row_d<D>(doreg, oreg), lse2 = lse_nat * LOG2E;
  const f32x4 negD = {-Dq, -Dq, -Dq, -Dq};
  f32x4 dq_acc[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) dq_acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c_log2 = p.scale_log2;
  zp_wait_async();

  for (int it = 0; it <= n_kt; it++) {
    // tile `it` has landed (the one behind it may be in flight), dS of the tile before is there; everybody is done with V of
    // tile it - 1, K of it - 2 and dS of it - 2
    if (it > 1) {
      if (it + 1 < n_kt) zp_wait_async_upto<2 * PW>();
      else zp_wait_async();
    }
    __syncthreads();
    auto copies = [&] {
      if (it + 2 < n_kt) {
        kst.issue(Ks + ((it + 2) & (NB - 1)) * TILEB, (it + 2) * 64, t.k_len);
        vst.issue(Vs + ((it + 2) & (NB - 1)) * TILEB, (it + 2) * 64, t.k_len);
      }
    };
    const int key0 = 64 * it + 32 * half;
    const unsigned out = own + (it & 1) * 4 * 2048 + half * 1024, in = own + ((it - 1) & 1) * 4 * 2048;
    if (it < n_kt && key0 < nvis_max) {
      if (it == 0) dq_pair_step<D, true, true, false>(qreg, doreg, dq_acc, c_log2, lse2, negD, key0, q4, nvis_lane, la, in, out, true, copies);
      else if (key0 + 32 > nvis_min) dq_pair_step<D, true, true, true>(qreg, doreg, dq_acc, c_log2, lse2, negD, key0, q4, nvis_lane, la, in, out, true, copies);
      else dq_pair_step<D, true, false, true>(qreg, doreg, dq_acc, c_log2, lse2, negD, key0, q4, nvis_lane, la, in, out, true, copies);
    } else if (it > 0 && 64 * (it - 1) < nvis_max) {
      dq_pair_step<D, false, false, true>(qreg, doreg, dq_acc, c_log2, lse2, negD, key0, q4, nvis_lane, la, in, out, 64 * (it - 1) + 32 < nvis_max, copies);
    } else {
      copies();
    }
    const int step = (it & (NB - 1)) == NB - 1 ? -(NB - 1) * TILEB : TILEB, step_t = it == 0 ? 0 : ((it - 1) & (NB - 1)) == NB - 1 ? -(NB - 1) * TILEB : TILEB;
#pragma unroll
    for (int i = 0; i < 2; i++) { la.k[i] += step; la.v[i] += step; }
#pragma unroll
    for (int i = 0; i < D / 32; i++) la.t[i] += step_t;
  }

  if (!PRE && half == 0 && row < t.q_rows && q4 == 0) {
    const int64_t r = (int64_t)h * p.T + t.q_tok0 + row;
    p.dvec[r] = -Dq;
    p.lse2[r] = -lse_nat / p.scale;
  }
  // V's buffers are free: everybody has passed the barrier behind the last product that reads them
  const int64_t at = ((int64_t)t.q_tok0 + rb) * p.dq_stride + (int64_t)h * D + half * (D / 2);
  if (!p.accumulate) zp_store_rows<D / 2>(Vs + (half * 4 + w) * ZP_ROWS_LDS_OF(D / 2), dq_acc, p.scale, p.dq + at, p.dq_stride, t.q_rows - rb, lane);
  else if (row < t.q_rows) add_acc_rows<D / 2>((float *)p.dq + at + c16 * p.dq_stride + q4, dq_acc, p.scale);
}

template <int D>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bwd_dq_pair_kernel(zp_bwd_params p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dq_pair_rows<D, false>(p, blockIdx.x, smem);
}

// -D and -LSE / scale of the rows of the dQ kernel's tiles, bit for bit what it would leave: 64 rows of a head per workgroup.
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_rows_kernel(zp_bwd_params p) {
  int unit, hh, part;
  zp_block_to_unit(zp_pair_item(p.dq_pair, blockIdx.x, part), p.grp, p.m_grp, unit, hh);
  if (unit >= p.n_dq_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), h = (unit - tile_idx * p.Hkv) * p.grp + hh;
  zp_tile t = ZP_TILE((const zp_tile *)nullptr, p.inl, 0, tile_idx);
  if (!zp_pair_rows(t, part)) return;
  const int lane = threadIdx.x & 63, c16 = lane & 15, q4 = 4 * (lane >> 4), row = 16 * (threadIdx.x >> 6) + c16;
  const int64_t tok = (int64_t)t.q_tok0 + min(row, t.q_rows - 1);
  const __bf16 *dop = p.dout + tok * p.do_stride + (int64_t)h * D + 2 * q4, *op = p.o + tok * p.o_stride + (int64_t)h * D + 2 * q4;
  bf16x8 doreg[D / 32], oreg[D / 32];
#pragma unroll
  for (int kk = 0; kk < D / 32; kk++) {
    doreg[kk] = *(const bf16x8 *)(dop + 32 * kk);
    oreg[kk] = *(const bf16x8 *)(op + 32 * kk);
  }
  const float lse_nat = p.lse[(int64_t)h * p.T + tok], Dq = row_d<D>(doreg, oreg);
  if (row < t.q_rows && q4 == 0) {
    p.dvec[(int64_t)h * p.T + tok] = -Dq;
    p.lse2[(int64_t)h * p.T + tok] = -lse_nat / p.scale;
  }
}

// ------------------------------------------------------------------------------------------- dK, dV
// Tile fields: k_tok0/k_len/k_pos0 = this block of key rows; q_tok0/q_rows/q_pos0 = the query rows of the
// same sequence from the first one that can see the block's first key to the end of the sequence.
//
// Head dimension 64: K and V operands in registers, 64-query tiles whose two 32-query blocks are software pipelined
// (dkdv_tile). Head dimension 128: the kernel further below.

// Two neighbouring elements (registers r, r + 1 of an accumulator; the queries at positions qpos and qpos + 1) of P and
// dS, packed as bf16. The accumulators were seeded with -LSE/scale and -D, so P = exp2(S c) and dS = P dP.
template <bool MASK>
__device__ __forceinline__ void dkdv_pair(const f32x4 &s, const f32x4 &dp, int r, int qpos, int kpos, int qpos_end,
                                          float c_log2, unsigned &p_pk, unsigned &ds_pk) {
  float p0 = zp_exp2(s[r] * c_log2), p1 = zp_exp2(s[r + 1] * c_log2);
  if (MASK) {
    if (qpos < kpos || qpos >= qpos_end) p0 = 0.f;
    if (qpos + 1 < kpos || qpos + 1 >= qpos_end) p1 = 0.f;
  }
  const bf16x2 pp = {(__bf16)p0, (__bf16)p1};
  const bf16x2 dd = {(__bf16)(p0 * dp[r]), (__bf16)(p1 * dp[r + 1])};
  p_pk = __builtin_bit_cast(unsigned, pp);
  ds_pk = __builtin_bit_cast(unsigned, dd);
  asm volatile("" : "+v"(p_pk), "+v"(ds_pk));  // keeps the arithmetic in the step it is written in
}

__device__ __forceinline__ bf16x8 dkdv_operand(const unsigned (&v)[4]) {
  return __builtin_bit_cast(bf16x8, (u32x4){v[0], v[1], v[2], v[3]});
}

// One 64-query tile = two 32-query blocks in four phases of D / 16 steps, two LDS operands and the four MFMAs (one per
// 16-key sub-block) they feed in a step:
//   A: S,dP(0) | B: S,dP(1) || P,dS(0) | C: dV,dK(0) || P,dS(1) | D: dV,dK(1) || the caller's copies
// A wave issues in order, so the overlap is written into the program order: every step is fenced and its LDS operands
// are requested two steps ahead. ONLY0: no query of the tile sees a key of sub-block 1.
// `piece(integral_constant<int, n>)` is called after each half of a step of phase D (n = 0 .. 2 * D / 16 - 1): the
// caller's asynchronous copies of a later tile are issued there, one load at a time.
// `lo` carries the addresses of the tile's Q rows; its dO rows are ZP_TILEB behind; seed: LDS address of the tile's
// -LSE/scale plus the lane's 4 (l / 16) floats, -D is D_OFF bytes behind.
template <int D, int D_OFF, bool MASK, bool ONLY0, class Piece>
__device__ __forceinline__ void dkdv_tile(unsigned seed, const bf16x8 (&kreg)[2][D / 32], const bf16x8 (&vreg)[2][D / 32],
                                          f32x4 (&dk_acc)[2][D / 16], f32x4 (&dv_acc)[2][D / 16], int qpos0,
                                          const int (&kpos)[2], int qpos_end, float c_log2, const zp_lds16<D> &lo,
                                          Piece &&piece) {
  constexpr int QN = D / 16, PPS = 8 / QN, CB = ONLY0 ? 1 : 2;  // steps per phase; pairs of P/dS elements per step
  constexpr int TILEB = 64 * D * 2;
  f32x4 ls[2][2], ds[2][2];  // seeds: [32-query block][16 rows], the 4 query rows this lane holds
  f32x4 s[2][2][2], dp[2][2][2];
  auto load_seed = [&](int blk) {
#pragma unroll
    for (int rb = 0; rb < 2; rb++) {
      ls[blk][rb] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + (blk * 32 + rb * 16) * 4);
      ds[blk][rb] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + D_OFF + (blk * 32 + rb * 16) * 4);
    }
  };
  // operand pair of global step t (phase t / QN): rows of Q,dO for A and B (16 rows i % 2, k-step i / 2), transposed
  // pieces of dO,Q for C and D (16 columns i)
  bf16x8 x[4 * QN + 2], y[4 * QN + 2];
  // (y before x: the wait for x then covers both)
  auto load_ops = [&](auto tt, auto yy) {
    constexpr int t = decltype(tt)::value, ph = t / QN, i = t % QN;
    constexpr bool is_y = decltype(yy)::value;
    if constexpr (ph < 2) (is_y ? y[t] : x[t]) = lo.rows_at(is_y ? TILEB : 0, 2 * ph + i % 2, i / 2);
    else if constexpr (ph < 4) (is_y ? y[t] : x[t]) = lo.tr_at(is_y ? 0 : TILEB, ph - 2, i);
  };
  unsigned ppk[2][2][4], dpk[2][2][4];  // [block][sub-block][elements 2j, 2j + 1]
  // element pair e of a block: 16 rows e / 4, sub-block e / 2 % 2, registers 2 (e % 2) and + 1; worked out in four stages,
  // one behind each MFMA of a step
  float e0[PPS], e1[PPS], d0[PPS], d1[PPS];
  auto pair_stage = [&](int blk, int e, int u, int stage) {
    const int rb = e / 4, cb = e / 2 % 2, r = 2 * (e % 2);
    if (cb >= CB) return;
    if (stage == 0) {
      e0[u] = s[blk][rb][cb][r] * c_log2;
      e1[u] = s[blk][rb][cb][r + 1] * c_log2;
    } else if (stage == 1) {
      e0[u] = zp_exp2(e0[u]);
      e1[u] = zp_exp2(e1[u]);
    } else if (stage == 2) {
      if (MASK) {
        const int qpos = qpos0 + blk * 32 + rb * 16 + r;
        if (qpos < kpos[cb] || qpos >= qpos_end) e0[u] = 0.f;
        if (qpos + 1 < kpos[cb] || qpos + 1 >= qpos_end) e1[u] = 0.f;
      }
      d0[u] = e0[u] * dp[blk][rb][cb][r];
      d1[u] = e1[u] * dp[blk][rb][cb][r + 1];
    } else {
      unsigned pp = __builtin_bit_cast(unsigned, (bf16x2){(__bf16)e0[u], (__bf16)e1[u]});
      unsigned dd = __builtin_bit_cast(unsigned, (bf16x2){(__bf16)d0[u], (__bf16)d1[u]});
      asm volatile("" : "+v"(pp), "+v"(dd));
      ppk[blk][cb][2 * rb + e % 2] = pp;
      dpk[blk][cb][2 * rb + e % 2] = dd;
      return;
    }
    asm volatile("" : "+v"(e0[u]), "+v"(e1[u]));
    if (stage == 2) asm volatile("" : "+v"(d0[u]), "+v"(d1[u]));
  };
  load_seed(0);
  load_ops(std::integral_constant<int, 0>{}, std::true_type{});
  load_ops(std::integral_constant<int, 0>{}, std::false_type{});
  load_ops(std::integral_constant<int, 1>{}, std::true_type{});
  load_ops(std::integral_constant<int, 1>{}, std::false_type{});
  zp_static_for<4 * QN>([&](auto tt) {
    constexpr int t = tt.value, ph = t / QN, i = t % QN;
    // the MFMAs of a step: the x operand with each sub-block, then the y operand; what else belongs to the step goes
    // between them a little at a time
    zp_static_for<4>([&](auto mm) {
      constexpr int m = mm.value, cb = m % 2;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (cb < CB) {
        if constexpr (ph < 2) {
          constexpr int rb = i % 2, k = i / 2;
          if constexpr (m < 2) s[ph][rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[t], kreg[cb][k], k == 0 ? ls[ph][rb] : s[ph][rb][cb], 0, 0, 0);
          else dp[ph][rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[t], vreg[cb][k], k == 0 ? ds[ph][rb] : dp[ph][rb][cb], 0, 0, 0);
        } else {
          if constexpr (m < 2) dv_acc[cb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[t], dkdv_operand(ppk[ph - 2][cb]), dv_acc[cb][i], 0, 0, 0);
          else dk_acc[cb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[t], dkdv_operand(dpk[ph - 2][cb]), dk_acc[cb][i], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (m % 2 == 0) load_ops(std::integral_constant<int, t + 2>{}, std::integral_constant<bool, m == 0>{});
      if constexpr (ph == 1 || ph == 2) {
#pragma unroll
        for (int u = 0; u < PPS; u++) pair_stage(ph - 1, i * PPS + u, u, m);
      }
      if constexpr (t == QN / 2 && m == 1) load_seed(1);
      if constexpr (ph == 3 && m % 2 == 1) piece(std::integral_constant<int, 2 * i + m / 2>{});
    });
  });
  __builtin_amdgcn_sched_barrier(0);
}

// The end of a workgroup that has gone through one share of its block's iterations: its sums go to scratch memory, and the share that
// is done last adds all of them up, in their order whichever it is (no workgroup waits for another). Returns whether this is the one
// (dk_acc, dv_acc then hold the block's sums). slot: an int of LDS that nobody needs any more. Bound: memory, 128 KB per share written and read
// at d = 128, 64 KB at 64 -- 256 shares at a time take some 14 and 7 us, 4.8 TB/s.
template <int D>
__device__ __forceinline__ bool dkdv_join_parts(const zp_bwd_params &p, const zp_part &part, int g, int tid, int *slot, f32x4 (&dk_acc)[2][D / 16],
                                                f32x4 (&dv_acc)[2][D / 16]) {
  constexpr int64_t SLOT = 128 * D * 2;  // floats
  constexpr int ONE = 2 * (D / 16) * 64 * 4;  // of a wave and sum
  const int at = (tid >> 6) * 2 * ONE + (tid & 63) * 4;
  auto of = [&](int i) { return p.parts + ((int64_t)(part.slot + i) * p.Hkv + g) * SLOT + at; };
  {
    float *own = of(part.part);
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
      for (int i = 0; i < D / 16; i++) {
        *(f32x4 *)(own + (cb * (D / 16) + i) * 256) = dk_acc[cb][i];
        *(f32x4 *)(own + ONE + (cb * (D / 16) + i) * 256) = dv_acc[cb][i];
      }
  }
  zp_wait_async();  // this wave's have been written
  __syncthreads();  // everybody's
  if (tid == 0) *slot = __hip_atomic_fetch_add(p.part_done + (int64_t)part.slot * p.Hkv + g, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*slot) != part.n - 1) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  for (int n = 0; n < part.n; n++) {
    const float *in = of(n);
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
      for (int i = 0; i < D / 16; i++) {
        const f32x4 a = *(const f32x4 *)(in + (cb * (D / 16) + i) * 256), b = *(const f32x4 *)(in + ONE + (cb * (D / 16) + i) * 256);
        if (n == 0) {
          dk_acc[cb][i] = a;
          dv_acc[cb][i] = b;
        } else {
          dk_acc[cb][i] += a;
          dv_acc[cb][i] += b;
        }
      }
  }
  return true;
}

__global__ __launch_bounds__(BWD_NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bwd_dkdv64_kernel(zp_bwd_params p) {
  constexpr int D = 64;
  constexpr int TILEB = 64 * D * 2;
  constexpr int NBUF = 4;                       // tiles are fetched three iterations ahead
  constexpr int LOADS = 2 * (TILEB / 4096) + 2; // async loads one wave issues per staged tile
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char *Qs = smem;                              // [NBUF][2][64][D]: a tile's Q rows and, behind them, its dO rows
  float *Ls = (float *)(smem + 2 * NBUF * TILEB);  // [NBUF][64] -LSE / scale
  float *Ds = Ls + NBUF * 64;                   // [NBUF][64] -D

  const int unit = __builtin_amdgcn_readfirstlane(zp_item_of_block(p.work_kv, (int *)(Ds + NBUF * 64)));
  if (unit < 0 || unit >= p.n_kv_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const zp_tile t = ZP_TILE_OF(p.kv_tiles, p.inl, p.n_seq, p.n_dq_tiles, true, tile_idx);

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  // the wave's two sub-blocks of 16 key rows, the w-th from the front and the w-th from the back of the block, so that
  // all four waves are seen by about the same number of queries
  const int kb[2] = {16 * w, 16 * (7 - w)};
  const int krow[2] = {kb[0] + c16, kb[1] + c16};
  const int kpos[2] = {t.k_pos0 + krow[0] - q4, t.k_pos0 + krow[1] - q4};  // less the lane's first query row: see dkdv_pair

  bf16x8 kreg[2][D / 32], vreg[2][D / 32];
#pragma unroll
  for (int cb = 0; cb < 2; cb++) {
    // rows behind the block's last key repeat it: a key column never mixes with another, and those are not stored
    const int64_t ktok = (int64_t)t.k_tok0 + min(krow[cb], t.k_len - 1);
    const __bf16 *kp = p.k + ktok * p.k_stride + (int64_t)g * D + 2 * q4;
    const __bf16 *vp = p.v + ktok * p.v_stride + (int64_t)g * D + 2 * q4;
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) {
      kreg[cb][kk] = *(const bf16x8 *)(kp + 32 * kk);
      vreg[cb][kk] = *(const bf16x8 *)(vp + 32 * kk);
    }
  }

  f32x4 dk_acc[2][D / 16], dv_acc[2][D / 16];
#pragma unroll
  for (int cb = 0; cb < 2; cb++)
#pragma unroll
    for (int i = 0; i < D / 16; i++) dk_acc[cb][i] = dv_acc[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c_log2 = p.scale_log2;

  const int n_qt = (t.q_rows + 63) / 64;
  // iterations: query tiles outermost (last tile first), heads of the group innermost; of the block, and of this workgroup's share
  const zp_part part = zp_part_of(t.part);
  const int n_all = n_qt * p.grp, it0 = part.part * p.share_its, n_it = part.part + 1 < part.n ? p.share_its : n_all - it0;

  zp_stager<D> qst, ost;
  qst.init(p.q + (int64_t)t.q_tok0 * p.q_stride + (int64_t)g * p.grp * D, p.q_stride, tid);
  ost.init(p.dout + (int64_t)t.q_tok0 * p.do_stride + (int64_t)g * p.grp * D, p.do_stride, tid);
  zp_lds16<D> lo;  // of the tile in hand: moved on by a buffer after every tile
  lo.init_abs(lane, smem);
  unsigned seed = zp_lds_addr(Ls) + q4 * 4;
  // Iteration order: query tiles from the END of the sequence backwards, the heads of the group innermost.
  // Workgroups of one sequence that start together then read the same (tile, head) at the same time and
  // share it in L2; the diagonal (masked) tiles come last.
  const int qt0 = zp_udiv(it0, p.grp, p.m_grp);
  int st_hh = it0 - qt0 * p.grp, st_qt = n_qt - 1 - qt0;  // head and query tile of the next tile to request
  int buf = 0, cur_qt = st_qt, cur_hh = st_hh;
  auto staged = [&] { if (++st_hh == p.grp) { st_hh = 0; st_qt--; } };
  auto stage = [&](int buf) {
    const int hh = st_hh, i0 = st_qt * 64;
    const int h = g * p.grp + hh;
    qst.issue(Qs + 2 * buf * TILEB, i0, t.q_rows, (int64_t)hh * D);
    ost.issue(Qs + (2 * buf + 1) * TILEB, i0, t.q_rows, (int64_t)hh * D);
    const int64_t base = (int64_t)h * p.T + t.q_tok0;
    zp_stage_async_f32x64(Ls + buf * 64, p.lse2 + base, i0, t.q_rows - 1, lane);
    zp_stage_async_f32x64(Ds + buf * 64, p.dvec + base, i0, t.q_rows - 1, lane);
  };
  // The same copies for a tile of 64 valid rows, cut into pieces that dkdv_tile issues between the MFMAs of its
  // last phase: every piece but the first one load (same order as `stage`).
  constexpr int PW = zp_stager<D>::PER_WAVE;
  const void *pc_q, *pc_o, *pc_l, *pc_d;
  unsigned pc_buf = 0;
  auto stage_piece = [&](auto n) {
    constexpr int N = decltype(n)::value;
    if constexpr (N == 0) {
      return;
    } else if constexpr (N <= PW) {
      zp_dma16_so(pc_q, qst.off[N - 1], __builtin_amdgcn_readfirstlane(zp_lds_addr(Qs) + 2 * pc_buf * TILEB + (qst.w * PW + N - 1) * 1024));
    } else if constexpr (N <= 2 * PW) {
      zp_dma16_so(pc_o, ost.off[N - PW - 1], __builtin_amdgcn_readfirstlane(zp_lds_addr(Qs) + (2 * pc_buf + 1) * TILEB + (ost.w * PW + N - PW - 1) * 1024));
    } else if constexpr (N == 2 * PW + 1) {
      zp_dma4_so(pc_l, lane * 4, __builtin_amdgcn_readfirstlane(zp_lds_addr(Ls) + pc_buf * 256));
    } else if constexpr (N == 2 * PW + 2) {
      zp_dma4_so(pc_d, lane * 4, __builtin_amdgcn_readfirstlane(zp_lds_addr(Ds) + pc_buf * 256));
    }
  };
  auto no_piece = [](auto) {};

  // prologue: tile 0 is requested right behind the K/V register operands (the two memory latencies overlap) and
  // one explicit wait covers both -- it also tells the compiler that the register operands have arrived (a wait of
  // its own inside the loop would drain the copies in flight every iteration); tiles 1 and 2 follow and stay in flight
  if (n_it > 0) stage(0);
  staged();
  zp_wait_async();
  if (n_it > 1) stage(1);
  staged();
  if (n_it > 2) stage(2);
  staged();
  __syncthreads();

  const int k0_min = t.k_pos0 + kb[0], k1_min = t.k_pos0 + kb[1];  // first positions of the sub-blocks
  const int qpos_end = t.q_pos0 + t.q_rows;
  const int qpos_end_l = qpos_end - q4;
  constexpr int D_OFF = NBUF * 256;

  for (int it = 0; it < n_it; it++) {
    const int i0 = cur_qt * 64;
    if (++cur_hh == p.grp) { cur_hh = 0; cur_qt--; }
    const int ahead = n_it - 1 - it;  // tiles after this one
    const int qpos0 = t.q_pos0 + i0;  // position of the tile's first query
    // sub-blocks with a key that some query of the tile sees
    const bool act0 = qpos0 + 63 >= k0_min, act1 = qpos0 + 63 >= k1_min && kb[1] < t.k_len;
    const bool masked = qpos0 < (act1 ? k1_min : k0_min) + 15 || qpos0 + 64 > qpos_end;
    // the tile three iterations ahead is fetched inside this tile's arithmetic when it is a full tile and this
    // wave computes an unmasked one (the common case), else in front of it
    const bool fetch = ahead >= NBUF - 1;
    const bool fused = fetch && act1 && !masked && st_qt * 64 + 64 <= t.q_rows;
    pc_buf = (buf + NBUF - 1) & (NBUF - 1);
    // the sources of that tile are worked out unconditionally (and, past the end, in vain): values defined under a
    // wave's branch would not stay in scalar registers
    {
      const int i0n = st_qt * 64;
      pc_q = zp_uniform_ptr(qst.base + (int64_t)i0n * qst.stride + (int64_t)st_hh * D);
      pc_o = zp_uniform_ptr(ost.base + (int64_t)i0n * ost.stride + (int64_t)st_hh * D);
      const int64_t base = (int64_t)(g * p.grp + st_hh) * p.T + t.q_tok0 + i0n;
      pc_l = zp_uniform_ptr(p.lse2 + base);
      pc_d = zp_uniform_ptr(p.dvec + base);
    }
    if (fetch && !fused) stage(pc_buf);

    if (act1) {
      if (masked) dkdv_tile<D, D_OFF, true, false>(seed, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, lo, no_piece);
      else if (fused) dkdv_tile<D, D_OFF, false, false>(seed, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, lo, stage_piece);
      else dkdv_tile<D, D_OFF, false, false>(seed, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, lo, no_piece);
    } else if (act0) {
      dkdv_tile<D, D_OFF, true, true>(seed, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, lo, no_piece);
    }
    // the next tile must have landed; the ones behind it may stay in flight
    if (ahead >= NBUF - 1) zp_wait_async_upto<(NBUF - 2) * LOADS>();
    else if (ahead == 2) zp_wait_async_upto<LOADS>();
    else zp_wait_async();
    __syncthreads();
    staged();
    buf = (buf + 1) & (NBUF - 1);
    lo.move(buf ? 2 * TILEB : -2 * (NBUF - 1) * TILEB);
    seed += buf ? 256 : -(NBUF - 1) * 256;
  }
  if (part.n && !dkdv_join_parts<D>(p, part, g, tid, (int *)(Ds + NBUF * 64), dk_acc, dv_acc)) return;

#pragma unroll
  for (int cb = 0; cb < 2; cb++) {
    const int64_t at = ((int64_t)t.k_tok0 + kb[cb]) * p.dkv_stride + (int64_t)g * D;
    if (!p.accumulate) {
      char *own = smem + w * ZP_ROWS_LDS;
      zp_store_rows<D>(own, dk_acc[cb], p.scale, p.dk + at, p.dkv_stride, t.k_len - kb[cb], lane);
      zp_store_rows<D>(own, dv_acc[cb], 1.0f, p.dv + at, p.dkv_stride, t.k_len - kb[cb], lane);
    } else if (krow[cb] < t.k_len) {
      add_acc_rows<D>((float *)p.dk + at + c16 * p.dkv_stride + q4, dk_acc[cb], p.scale);
      add_acc_rows<D>((float *)p.dv + at + c16 * p.dkv_stride + q4, dv_acc[cb], 1.0f);
    }
  }
}

// ---------------------------------------------------------------------------- dK, dV at head dimension 128
// A lane's LDS read addresses in the zp_pad16 layout: of the Q and dO tiles (relative to the first buffer; everything
// else is an immediate offset) and of the wave's V rows.
template <int D>
struct dkdv_lds_addr {
  typedef zp_pad16<D> L;
  unsigned row[2], tr[4], v[2][2];
  __device__ __forceinline__ void init(int lane, const char *tiles, const char *v0, const char *v1) {
#pragma unroll
    for (int par = 0; par < 2; par++) {
      const int r = L::row_part(lane, par);
      row[par] = zp_lds_addr(tiles) + r;
      v[0][par] = zp_lds_addr(v0) + r;
      v[1][par] = zp_lds_addr(v1) + r;
      asm volatile("" : "+v"(row[par]), "+v"(v[0][par]), "+v"(v[1][par]));  // opaque: see zp_lds16
    }
#pragma unroll
    for (int dq = 0; dq < 4; dq++) {
      tr[dq] = zp_lds_addr(tiles) + L::tr_part(lane, dq);
      asm volatile("" : "+v"(tr[dq]));
    }
  }
  // off: byte offset of the tile from the first buffer; rb: 16 rows; k: k-step; db: 16 columns
  __device__ __forceinline__ bf16x8 rows(int off, int rb, int k) const {
    return *(const ZP_LDS bf16x8 *)(unsigned long long)(row[k & 1] + off + rb * L::R16 + (k >> 1) * 128);
  }
  __device__ __forceinline__ bf16x8 vrows(int cb, int k) const {
    return *(const ZP_LDS bf16x8 *)(unsigned long long)(v[cb][k & 1] + (k >> 1) * 128);
  }
  __device__ __forceinline__ bf16x8 cols(int off, int db) const {
    const unsigned o = tr[db & 3] + off + (db >> 2) * 128;
    s16x4 u0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)o);
    s16x4 u1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ZP_LDS s16x4 *)(unsigned long long)(o + L::R16));
    return zp_cat(__builtin_bit_cast(bf16x4, u0), __builtin_bit_cast(bf16x4, u1));
  }
};

// One 32-query tile. Four runs of D / 16 steps of one LDS operand (the dP run: one of dO, and both of V every second step)
// and two MFMAs -- S, dP, dV^T, dK^T -- each a fenced pipeline with its operands two steps ahead; the last two steps of
// a run request the first operands of the next one. One run at a time keeps the operands in flight within 28 registers
// (all four streams two steps ahead would not fit beside the accumulators). Q_OFF, O_OFF: byte offsets of the tile's Q and
// dO rows; seed: LDS address of its -LSE/scale plus the lane's floats, -D is D_OFF bytes behind. ONLY0: no query of the
// tile sees a key of sub-block 1.
template <int D, int Q_OFF, int O_OFF, int D_OFF, bool MASK, bool ONLY0, bool PIECES, class Piece>
__device__ __forceinline__ void dkdv_block(unsigned seed, const bf16x8 (&kreg)[2][D / 32], f32x4 (&dk_acc)[2][D / 16],
                                           f32x4 (&dv_acc)[2][D / 16], int qpos0, const int (&kpos)[2], int qpos_end,
                                           float c_log2, const dkdv_lds_addr<D> &la, Piece &&piece) {
  constexpr int N = D / 16, KK = D / 32, CB = ONLY0 ? 1 : 2;
  f32x4 s[2][2], dp[2][2], ls[2], ds[2];
#pragma unroll
  for (int rb = 0; rb < 2; rb++) {  // -LSE/scale and -D of the 4 query rows this lane holds of each 16
    ls[rb] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + rb * 64);
    ds[rb] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + D_OFF + rb * 64);
  }
  bf16x8 x[N], y[N], v[KK][2], xo[N], yo[N];  // step i: 16 rows i % 2, k-step i / 2 (S, dP); 16 columns i (dV^T, dK^T)
  auto load_v = [&](int k) {
#pragma unroll
    for (int cb = 0; cb < CB; cb++) v[k][cb] = la.vrows(cb, k);
  };
  x[0] = la.rows(Q_OFF, 0, 0); x[1] = la.rows(Q_OFF, 1, 0);
  zp_static_for<N>([&](auto ii) {
    constexpr int i = ii.value, rb = i % 2, k = i / 2;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cb = 0; cb < CB; cb++) s[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i], kreg[cb][k], k == 0 ? ls[rb] : s[rb][cb], 0, 0, 0);
    if constexpr (i + 2 < N) x[i + 2] = la.rows(Q_OFF, i % 2, k + 1);
    else y[i + 2 - N] = la.rows(O_OFF, i % 2, 0);
    if constexpr (i == N - 2) load_v(0);
    if constexpr (PIECES) piece(ii);
  });
  zp_static_for<N>([&](auto ii) {
    constexpr int i = ii.value, rb = i % 2, k = i / 2;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cb = 0; cb < CB; cb++) dp[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[i], v[k][cb], k == 0 ? ds[rb] : dp[rb][cb], 0, 0, 0);
    if constexpr (i + 2 < N) y[i + 2] = la.rows(O_OFF, i % 2, k + 1);
    else xo[i + 2 - N] = la.cols(O_OFF, i + 2 - N);
    if constexpr (rb == 0 && k + 1 < KK) load_v(k + 1);
  });
  __builtin_amdgcn_sched_barrier(0);
  unsigned ppk[2][4], dpk[2][4];
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int e = 0; e < 4; e++)
      dkdv_pair<MASK>(s[e / 2][cb], dp[e / 2][cb], 2 * (e % 2), qpos0 + 16 * (e / 2) + 2 * (e % 2), kpos[cb], qpos_end, c_log2, ppk[cb][e], dpk[cb][e]);
  zp_static_for<N>([&](auto ii) {
    constexpr int i = ii.value;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cb = 0; cb < CB; cb++) dv_acc[cb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xo[i], dkdv_operand(ppk[cb]), dv_acc[cb][i], 0, 0, 0);
    if constexpr (i + 2 < N) xo[i + 2] = la.cols(O_OFF, i + 2);
    else yo[i + 2 - N] = la.cols(Q_OFF, i + 2 - N);
  });
  zp_static_for<N>([&](auto ii) {
    constexpr int i = ii.value;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cb = 0; cb < CB; cb++) dk_acc[cb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yo[i], dkdv_operand(dpk[cb]), dk_acc[cb][i], 0, 0, 0);
    if constexpr (i + 2 < N) yo[i + 2] = la.cols(Q_OFF, i + 2);
  });
  __builtin_amdgcn_sched_barrier(0);
}

// The end of a dK/dV workgroup of two groups of four waves, which have gone through the iterations by turns: the first group
// adds up and writes dK, the second one dV, each with what the other hands over through LDS (D KB).
template <int D>
__device__ __forceinline__ void dkdv_add_groups(const zp_bwd_params &p, const zp_tile &t, int g, int group, int w, int lane, const int (&kb)[2],
                                                f32x4 (&dk_acc)[2][D / 16], f32x4 (&dv_acc)[2][D / 16], char *smem) {
  constexpr int ACCB = (D / 16) * 1024;  // bytes of one accumulator of one wave
  __syncthreads();  // (the tiles have been read)
  ZP_LDS char *give = (ZP_LDS char *)smem + ((group * 4 + w) * 2) * ACCB + lane * 16;
  const ZP_LDS char *take = (const ZP_LDS char *)smem + (((group ^ 1) * 4 + w) * 2) * ACCB + lane * 16;
  auto hand_over = [&](const f32x4 (&acc)[2][D / 16]) {
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
      for (int i = 0; i < D / 16; i++) *(ZP_LDS f32x4 *)(give + cb * ACCB + i * 1024) = acc[cb][i];
  };
  auto finish = [&](f32x4 (&acc)[2][D / 16], __bf16 *out, float mul) {
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
      for (int i = 0; i < D / 16; i++) {
        const f32x4 v = *(const ZP_LDS f32x4 *)(take + cb * ACCB + i * 1024);
        acc[cb][i][0] += v[0]; acc[cb][i][1] += v[1]; acc[cb][i][2] += v[2]; acc[cb][i][3] += v[3];
      }
    __syncthreads();  // the rows pass through LDS on their way out
#pragma unroll
    for (int cb = 0; cb < 2; cb++) {
      const int64_t at = ((int64_t)t.k_tok0 + kb[cb]) * p.dkv_stride + (int64_t)g * D;
      if (!p.accumulate) zp_store_rows<D>(smem + (group * 4 + w) * ZP_ROWS_LDS, acc[cb], mul, out + at, p.dkv_stride, t.k_len - kb[cb], lane);
      else if (kb[cb] + (lane & 15) < t.k_len) add_acc_rows<D>((float *)out + at + (lane & 15) * p.dkv_stride + 4 * (lane >> 4), acc[cb], mul);
    }
  };
  if (group == 0) hand_over(dv_acc);
  else hand_over(dk_acc);
  __syncthreads();
  if (group == 0) finish(dk_acc, p.dk, p.scale);
  else finish(dv_acc, p.dv, 1.0f);
}

// Two waves per SIMD for head dimension 128 as well: two independent workgroups of four waves per CU (69 KB of LDS
// each), a wave holding its K operands (32 registers) and its dK^T/dV^T accumulators (128) and working on 32-query
// tiles, one product at a time; the V operands do not fit beside them in 256 registers and are read from LDS, where the
// workgroup's 128 V rows are staged once. The wave's LDS, vector, scalar and wait instructions issue in line with its
// MFMAs; a second wave on the SIMD, from a workgroup that meets its own barriers, runs under all of that.
//
// Bound: the power limit and vector issue. On one card, this kernel against the two it replaces (32x32x16 MFMA; one wave per
// SIMD with K and V in registers for long sequences, this split with an XOR per LDS read for short ones): 128K
// long-tail GQA batch 25.17 -> 22.97 ms, four 16384-token sequences 15.49 -> 14.22, 64K lognormal MHA 2.70 -> 2.39,
// 64 x 1K MHA 1.45 -> 1.29. The one-wave form on the 16x16x32 MFMA took 24.9 ms on the long-tail batch; with an XOR for
// every LDS read (32 to the 64 vector operations a tile needs) this one took 24.7.
//
// G = 2: both of a CU's workgroups become groups of one, which go through the iterations of ONE key block by turns and add up
// their accumulators at the end. The same work per CU and half the chain, at the price of a prologue and an end that
// nothing else runs beside (9.3 us per workgroup) and of meeting at one barrier: for launches of a few waves of workgroups, in which the
// longest chains and the last wave decide. (Its scalar registers are five short: three are read back from lanes of a vector
// register per two tiles.) 8000 ragged tokens, 32/8 heads: 500 -> 360 us, 10709 tokens, 8/8: 121 -> 88; 64K lognormal MHA
// 2315 -> 2818.
template <int G>
__global__ __launch_bounds__(G * BWD_NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bwd_dkdv128_kernel(zp_bwd_params p) {
  constexpr int D = 128, QT = 32;
  constexpr int TILEB = 2 * zp_pad16<128>::R16;         // a staged tile: 32 query rows
  typedef zp_stager<D, 8, true> stager;               // 4 waves x 2 wave-loads = the first 32 rows of its 64-row pattern
  constexpr int PW = stager::PER_WAVE;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int group = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  char *Qs = smem + group * 4 * TILEB;             // [2][2][32][D] of the group: two buffers (three would not fit two workgroups
                                                   // per CU) of a tile's Q rows and, behind them, its dO rows
  char *Vs = smem + G * 4 * TILEB;                 // [128][D]: the workgroup's V rows, staged once
  // [2][2][64]: a tile's 32 values of -LSE / scale and, behind them, of -D (the copies write 64 floats, the upper half
  // of no use: no lane mask to set up)
  float *Ls = (float *)(Vs + 8 * zp_pad16<128>::R16) + group * 4 * 64;

  const int unit = __builtin_amdgcn_readfirstlane(zp_item_of_block(p.work_kv, (int *)(Vs + 8 * zp_pad16<128>::R16 + G * 4 * 64 * 4)));
  if (unit < 0 || unit >= p.n_kv_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const zp_tile t = ZP_TILE_OF(p.kv_tiles, p.inl, p.n_seq, p.n_dq_tiles, true, tile_idx);

  const int tid = G == 1 ? threadIdx.x : threadIdx.x & 255, lane = tid & 63, w = tid >> 6;
  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  // the wave's two sub-blocks of 16 key rows: see attn_bwd_dkdv64_kernel
  const int kb[2] = {16 * w, 16 * (7 - w)};
  const int krow[2] = {kb[0] + c16, kb[1] + c16};
  const int kpos[2] = {t.k_pos0 + krow[0] - q4, t.k_pos0 + krow[1] - q4};

  // K operands in registers; V operands from LDS (rows past the block's last key repeat it: a key column never
  // mixes with another, and those columns are not stored)
  bf16x8 kreg[2][D / 32];
#pragma unroll
  for (int cb = 0; cb < 2; cb++) {
    const __bf16 *kp = p.k + ((int64_t)t.k_tok0 + min(krow[cb], t.k_len - 1)) * p.k_stride + (int64_t)g * D + 2 * q4;
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) kreg[cb][kk] = *(const bf16x8 *)(kp + 32 * kk);
  }

  f32x4 dk_acc[2][D / 16], dv_acc[2][D / 16];
#pragma unroll
  for (int cb = 0; cb < 2; cb++)
#pragma unroll
    for (int i = 0; i < D / 16; i++) dk_acc[cb][i] = dv_acc[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c_log2 = p.scale_log2;

  const int n_qt = (t.q_rows + QT - 1) / QT;
  // iterations: query tiles outermost (last tile first), heads of the group innermost; of the block, and (G = 1) of this workgroup's share
  const zp_part part = zp_part_of(G == 1 ? t.part : 0);
  const int n_all = n_qt * p.grp, it0 = part.part * p.share_its, n_it = part.part + 1 < part.n ? p.share_its : n_all - it0;

  stager qst, ost;
  qst.init(p.q + (int64_t)t.q_tok0 * p.q_stride + (int64_t)g * p.grp * D, p.q_stride, tid);
  ost.init(p.dout + (int64_t)t.q_tok0 * p.do_stride + (int64_t)g * p.grp * D, p.do_stride, tid);
  dkdv_lds_addr<D> la;
  la.init(lane, Qs, Vs + kb[0] / 16 * zp_pad16<128>::R16, Vs + kb[1] / 16 * zp_pad16<128>::R16);
  {
    zp_stager<D, 4, true> vst;
    vst.init(p.v + (int64_t)t.k_tok0 * p.v_stride + (int64_t)g * D, p.v_stride, tid);
    for (int half = G == 1 ? 0 : group; half < (G == 1 ? 2 : group + 1); half++) vst.issue(Vs + half * 4 * zp_pad16<128>::R16, 64 * half, t.k_len);
  }
  const unsigned seed = zp_lds_addr(Ls) + q4 * 4;
  // a group's iterations are group, group + G, ...
  auto on = [&](int &hh, int &qt, int by) {
    for (int i = 0; i < by; i++)
      if (++hh == p.grp) { hh = 0; qt--; }
  };
  const int qt0 = G == 1 ? zp_udiv(it0, p.grp, p.m_grp) : 0;
  int st_hh = it0 - qt0 * p.grp, st_qt = n_qt - 1 - qt0;  // head and query tile of the next tile to request
  on(st_hh, st_qt, group);
  int cur_qt = st_qt, cur_hh = st_hh;
  auto staged = [&] { on(st_hh, st_qt, G); };
  auto stage = [&](int buf) {
    const int hh = st_hh, i0 = st_qt * QT;
    const int h = g * p.grp + hh;
    qst.issue(Qs + 2 * buf * TILEB, i0, t.q_rows, (int64_t)hh * D);
    ost.issue(Qs + (2 * buf + 1) * TILEB, i0, t.q_rows, (int64_t)hh * D);
    // waves 0 and 2 fetch the one row vector, 1 and 3 the other
    int r = i0 + (lane & 31);
    if (r > t.q_rows - 1) r = t.q_rows - 1;
    zp_dma4((qst.w & 1 ? p.dvec : p.lse2) + (int64_t)h * p.T + t.q_tok0 + r,
            __builtin_amdgcn_readfirstlane(zp_lds_addr(Ls) + buf * 512 + (qst.w & 1) * 256));
  };
  // the same copies for a tile of 32 valid rows, one per step of the S run but the first
  const void *pc_q, *pc_o, *pc_s;
  unsigned pc_buf = 0;
  auto stage_piece = [&](auto n) {
    constexpr int N = decltype(n)::value;
    static_assert(2 * PW + 2 <= D / 16, "the copies of a tile fit the steps of one chain");
    if constexpr (N == 0) {
      return;
    } else if constexpr (N <= PW) {
      zp_dma16_so(pc_q, qst.off[N - 1], __builtin_amdgcn_readfirstlane(zp_lds_addr(Qs) + 2 * pc_buf * TILEB + qst.dest(N - 1)));
    } else if constexpr (N <= 2 * PW) {
      zp_dma16_so(pc_o, ost.off[N - PW - 1], __builtin_amdgcn_readfirstlane(zp_lds_addr(Qs) + (2 * pc_buf + 1) * TILEB + ost.dest(N - PW - 1)));
    } else if constexpr (N == 2 * PW + 1) {
      zp_dma4_so(pc_s, (lane & 31) * 4, __builtin_amdgcn_readfirstlane(zp_lds_addr(Ls) + pc_buf * 512 + (qst.w & 1) * 256));
    }
  };
  auto no_piece = [](auto) {};

  if (group < n_it) stage(0);
  staged();
  zp_wait_async();
  __syncthreads();

  const int k0_min = t.k_pos0 + kb[0], k1_min = t.k_pos0 + kb[1];  // first positions of the sub-blocks
  const int qpos_end = t.q_pos0 + t.q_rows, qpos_end_l = qpos_end - q4;
  constexpr int D_OFF = 256;

  // one tile out of buffer BUF (compile-time, so that every LDS address is a register plus an immediate)
  auto query_tile = [&](int it, auto BUF) {
    constexpr int buf = decltype(BUF)::value;
    const int i0 = cur_qt * QT;
    on(cur_hh, cur_qt, G);
    const int qpos0 = t.q_pos0 + i0;        // position of the tile's first query
    // sub-blocks with a key that some query of the tile sees
    const bool here = G == 1 || it < n_it;
    const bool act0 = here && qpos0 + QT - 1 >= k0_min, act1 = here && qpos0 + QT - 1 >= k1_min && kb[1] < t.k_len;
    const bool masked = qpos0 < (act1 ? k1_min : k0_min) + 15 || qpos0 + QT > qpos_end;
    // the next tile is fetched inside this tile's S run when it is a full tile and this wave computes an unmasked one
    // (the common case), else in front; its sources are worked out unconditionally (and, past the end, in vain): values
    // defined under a wave's branch would not stay in scalar registers
    const bool fetch = it + G < n_it;
    const bool fused = fetch && act1 && !masked && st_qt * QT + QT <= t.q_rows;
    pc_buf = buf ^ 1;
    {
      const int i0n = st_qt * QT;
      pc_q = zp_uniform_ptr(qst.base + (int64_t)i0n * qst.stride + (int64_t)st_hh * D);
      pc_o = zp_uniform_ptr(ost.base + (int64_t)i0n * ost.stride + (int64_t)st_hh * D);
      const int64_t base = (int64_t)(g * p.grp + st_hh) * p.T + t.q_tok0 + i0n;
      pc_s = zp_uniform_ptr((qst.w & 1 ? p.dvec : p.lse2) + base);
    }
    if (fetch && !fused) stage(buf ^ 1);
    if (act1) {
      if (masked) dkdv_block<D, 2 * buf * TILEB, (2 * buf + 1) * TILEB, D_OFF, true, false, false>(seed + buf * 512, kreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, no_piece);
      else if (fused) dkdv_block<D, 2 * buf * TILEB, (2 * buf + 1) * TILEB, D_OFF, false, false, true>(seed + buf * 512, kreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, stage_piece);
      else dkdv_block<D, 2 * buf * TILEB, (2 * buf + 1) * TILEB, D_OFF, false, false, false>(seed + buf * 512, kreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, no_piece);
    } else if (act0) {
      dkdv_block<D, 2 * buf * TILEB, (2 * buf + 1) * TILEB, D_OFF, true, true, false>(seed + buf * 512, kreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, no_piece);
    }
    staged();
    zp_wait_async();
    __syncthreads();
  };
  for (int it = 0; it < n_it; it += 2 * G) {
    query_tile(it + group, std::integral_constant<int, 0>{});
    if (it + G < n_it) query_tile(it + G + group, std::integral_constant<int, 1>{});
  }
  if constexpr (G == 2) {
    dkdv_add_groups<D>(p, t, g, group, w, lane, kb, dk_acc, dv_acc, smem);
    return;
  }
  if (part.n && !dkdv_join_parts<D>(p, part, g, tid, (int *)Ls, dk_acc, dv_acc)) return;

#pragma unroll
  for (int cb = 0; cb < 2; cb++) {
    const int64_t at = ((int64_t)t.k_tok0 + kb[cb]) * p.dkv_stride + (int64_t)g * D;
    if (!p.accumulate) {
      char *own = smem + w * ZP_ROWS_LDS;
      zp_store_rows<D>(own, dk_acc[cb], p.scale, p.dk + at, p.dkv_stride, t.k_len - kb[cb], lane);
      zp_store_rows<D>(own, dv_acc[cb], 1.0f, p.dv + at, p.dkv_stride, t.k_len - kb[cb], lane);
    } else if (krow[cb] < t.k_len) {
      add_acc_rows<D>((float *)p.dk + at + c16 * p.dkv_stride + q4, dk_acc[cb], p.scale);
      add_acc_rows<D>((float *)p.dv + at + c16 * p.dkv_stride + q4, dv_acc[cb], 1.0f);
    }
  }
}

// A 32-query tile for one wave of 16 key rows: the four products S, dP, dV^T, dK^T as one pipeline of 4 D / 16 steps of one LDS
// operand and its MFMA, operands requested AHEAD steps ahead. exp2 runs under the dP product, dS = P dP under the dV product.
// Q_OFF, O_OFF, seed, D_OFF: as for dkdv_block. V fits the registers here. `piece(integral_constant<int, n>)`, n = 0 .. D / 16, is
// called every third step: the caller's copies of a later tile go there one by one.
template <int D, int AHEAD, int Q_OFF, int O_OFF, int D_OFF, bool MASK, class Piece>
__device__ __forceinline__ void dkdv_half_block(unsigned seed, const bf16x8 (&kreg)[D / 32], const bf16x8 (&vreg)[D / 32], f32x4 (&dk_acc)[D / 16],
                                                f32x4 (&dv_acc)[D / 16], int qpos0, int kpos, int qpos_end, float c_log2,
                                                const zp_pad16_addr<D> &la, Piece &&piece) {
  constexpr int N = D / 16, EPS = 8 / N;  // steps of a product; elements of P or dS per step
  f32x4 s[2], dp[2], ls[2], ds[2];
#pragma unroll
  for (int rb = 0; rb < 2; rb++) {  // -LSE/scale and -D of the 4 query rows this lane holds of each 16
    ls[rb] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + rb * 64);
    if (D == 128) ds[rb] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + D_OFF + rb * 64);
  }
  bf16x8 x[4 * N];  // step i of a product: 16 rows i % 2, k-step i / 2 (S, dP); 16 columns i (dV^T, dK^T)
  auto load = [&](auto nn) {
    constexpr int n = decltype(nn)::value, ph = n / N, i = n % N;
    if constexpr (ph < 2) x[n] = la.rows(ph ? O_OFF : Q_OFF, i % 2, i / 2);
    else if constexpr (ph < 4) x[n] = la.cols(ph == 2 ? O_OFF : Q_OFF, i);
  };
  zp_static_for<AHEAD>(load);
  float pe[8], de[8];
  unsigned ppk[4], dpk[4];  // elements 2j, 2j + 1: 16 rows j / 2, registers 2 (j % 2) and + 1
  zp_static_for<4 * N>([&](auto nn) {
    constexpr int n = nn.value, ph = n / N, i = n % N, rb = i % 2, k = i / 2;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (ph == 0) s[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], kreg[k], k == 0 ? ls[rb] : s[rb], 0, 0, 0);
    else if constexpr (ph == 1) dp[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], vreg[k], k == 0 ? ds[rb] : dp[rb], 0, 0, 0);
    else if constexpr (ph == 2) dv_acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], dkdv_operand(ppk), dv_acc[i], 0, 0, 0);
    else dk_acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[n], dkdv_operand(dpk), dk_acc[i], 0, 0, 0);
    load(std::integral_constant<int, n + AHEAD>{});
    if constexpr (D == 64 && (n == 0 || n == 1)) ds[n] = *(const ZP_LDS f32x4 *)(unsigned long long)(seed + D_OFF + n * 64);
    if constexpr (n % 3 == 1 && n / 3 <= N) piece(std::integral_constant<int, n / 3>{});
    if constexpr (ph == 1 || ph == 2) {
#pragma unroll
      for (int e = i * EPS; e < i * EPS + EPS; e++) {
        const int er = e / 4, r = e % 4, qpos = qpos0 + 16 * er + r;
        if (ph == 1) {
          pe[e] = zp_exp2(s[er][r] * c_log2);
          if (MASK && (qpos < kpos || qpos >= qpos_end)) pe[e] = 0.f;
          if (e % 2) ppk[e / 2] = __builtin_bit_cast(unsigned, (bf16x2){(__bf16)pe[e - 1], (__bf16)pe[e]});
        } else {
          de[e] = pe[e] * dp[er][r];
          if (e % 2) dpk[e / 2] = __builtin_bit_cast(unsigned, (bf16x2){(__bf16)de[e - 1], (__bf16)de[e]});
        }
      }
    }
  });
  __builtin_amdgcn_sched_barrier(0);
}

// A group's LDS in the kernel below: two buffers of 32 Q and dO rows, two of row vectors.
template <int D>
constexpr int split_own() { return 8 * zp_pad16<D>::R16 + 1024; }

// dK, dV of launches that whole key blocks do not spread over the chip: a workgroup owns 32 key rows instead of 128. Its eight
// waves are four groups of two; the groups go through the (query tile, head) iterations by turns, each with staging buffers of
// its own (140 KB of LDS in all at D = 128), and the two waves of a group, on one SIMD, share the tile and do 16 key rows
// each. The groups' accumulators are added up at the end, through LDS, in their order.
//
// One workgroup per CU at d = 128, two at 64 (70 KB of LDS, all of 128 registers: what a second one adds is worth a third).
// Bound: a group's chain of iterations: 1.21 us each at d = 128, 0.81 at 64 (2850 and 1900 cycles, of which the MFMAs of a SIMD's
// two waves are 1024 and 512, their arithmetic under MFMAs about as much, hand-over and addresses 600); with one wave per
// group and 32 key rows per wave, whose operations issue one after the other, 1.50 and 0.86. 1000 tokens, 4/2 heads, d = 128:
// one wave per group 31.7 us, two 27.1; 4000 tokens 105.6 and 85.5 (61.8 and 58.6 at d = 64). See dkdv_kernel_for for when it is used.
// block: of the kernel's own
template <int D>
__device__ __forceinline__ void dkdv_split_rows(const zp_bwd_params &p, int block, char *smem) {
  constexpr int QT = 32, AHEAD = D == 64 ? 3 : 6;
  typedef zp_pad16<D> L;
  constexpr int TILEB = 2 * L::R16;                // a staged tile: 32 query rows
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave & 3, half = wave >> 2;
  char *own = smem + group * split_own<D>();
  float *Ls = (float *)(own + 4 * TILEB);          // [2][2][64]: see attn_bwd_dkdv128_kernel

  // the four workgroups of a key block on one XCD
  const int x = block & 7, y = block >> 3, part = y & 3, unit = (y >> 2) * 8 + x;
  if (unit >= p.n_kv_tiles * p.Hkv) return;
  const int tile_idx = zp_udiv(unit, p.Hkv, p.m_hkv), g = unit - tile_idx * p.Hkv;
  const zp_tile t = ZP_TILE_OF(p.kv_tiles, p.inl, p.n_seq, p.n_dq_tiles, true, tile_idx);
  if (32 * part >= t.k_len) return;

  const int c16 = lane & 15, q4 = 4 * (lane >> 4);
  const int kb = 32 * part + 16 * half, krow = kb + c16;  // the wave's key rows, the lane's
  const int kpos = t.k_pos0 + krow - q4;                  // less the lane's first query row, as qpos_end below

  // K and V operands in registers (rows behind the last key repeat it: a key column never mixes with another, and those are
  // not stored)
  bf16x8 kreg[D / 32], vreg[D / 32];
  const int64_t ktok = (int64_t)t.k_tok0 + min(krow, t.k_len - 1);
  const __bf16 *kp = p.k + ktok * p.k_stride + (int64_t)g * D + 2 * q4, *vp = p.v + ktok * p.v_stride + (int64_t)g * D + 2 * q4;
#pragma unroll
  for (int kk = 0; kk < D / 32; kk++) {
    kreg[kk] = *(const bf16x8 *)(kp + 32 * kk);
    vreg[kk] = *(const bf16x8 *)(vp + 32 * kk);
  }
  f32x4 dk_acc[D / 16], dv_acc[D / 16];
#pragma unroll
  for (int i = 0; i < D / 16; i++) dk_acc[i] = dv_acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // iterations: query tiles outermost (last tile first), heads of the group innermost; this group's are group, group + 4, ...
  const int n_qt = (t.q_rows + QT - 1) / QT, n_it = n_qt * p.grp;
  // of a tile the first wave copies the Q rows and -LSE / scale, the second one the dO rows and -D (a wave copies 32 rows by
  // itself: the first of the two waves of a 64-row pattern)
  zp_stager<D, 2, true> st;
  st.init((half ? p.dout : p.q) + (int64_t)t.q_tok0 * (half ? p.do_stride : p.q_stride) + (int64_t)g * p.grp * D, half ? p.do_stride : p.q_stride, lane);
  const float *rowvec = (half ? p.dvec : p.lse2) + (int64_t)g * p.grp * p.T + t.q_tok0;
  zp_pad16_addr<D> la;
  la.init(lane, own);
  // the query tile and head of an iteration four behind
  const int dq = zp_udiv(4, p.grp, p.m_grp), dh = 4 - dq * p.grp;
  auto on = [&](int &i0, int &hh) {
    const bool wrap = hh + dh >= p.grp;
    i0 -= QT * (wrap ? dq + 1 : dq);
    hh += wrap ? dh - p.grp : dh;
  };
  auto stage = [&](int i0, int hh, int buf) {
    st.issue(own + (2 * buf + half) * TILEB, i0, t.q_rows, (int64_t)hh * D);
    int r = i0 + (lane & 31);
    if (r > t.q_rows - 1) r = t.q_rows - 1;
    zp_dma4(rowvec + (int64_t)hh * p.T + r, __builtin_amdgcn_readfirstlane(zp_lds_addr(Ls) + buf * 512 + half * 256));
  };
  const unsigned seed = zp_lds_addr(Ls) + q4 * 4;
  const int k_min = t.k_pos0 + kb;
  const int qpos_end = t.q_pos0 + t.q_rows, qpos_end_l = qpos_end - q4;
  const float c_log2 = p.scale_log2;

  const int q0 = zp_udiv(group, p.grp, p.m_grp);
  int i0 = (n_qt - 1 - q0) * QT, next_i0 = i0, next_hh = group - q0 * p.grp;  // this iteration's first query row; the next one's
  if (group < n_it) stage(next_i0, next_hh, 0);
  on(next_i0, next_hh);
  auto query_tile = [&](int it, auto BUF) {
    constexpr int buf = decltype(BUF)::value;
    // the tile has landed; both waves of the group are done with the one before (and, the barrier being the workgroup's, so are
    // the other groups', which need not be)
    zp_wait_async();
    __syncthreads();
    const int qpos0 = t.q_pos0 + i0;
    const bool compute = it < n_it && qpos0 + QT - 1 >= k_min && kb < t.k_len, masked = qpos0 < k_min + 15 || qpos0 + QT > qpos_end;
    // at D = 128 the next tile is fetched inside this one's products when it is a full one (the common case): eight waves'
    // copies issued at once wait up to 140 cycles each for the address unit (4000 tokens, 4/2 heads: 91 us in front, 86 inside;
    // at D = 64, where the products have half as many steps for them, 58 and 65)
    const bool fused = D == 128 && compute && !masked && it + 4 < n_it && next_i0 + QT <= t.q_rows;
    if (it + 4 < n_it && !fused) stage(next_i0, next_hh, buf ^ 1);
    const void *pc_t = zp_uniform_ptr(st.base + (int64_t)next_i0 * st.stride + (int64_t)next_hh * D), *pc_r = zp_uniform_ptr(rowvec + (int64_t)next_hh * p.T + next_i0);
    auto stage_piece = [&](auto nn) {
      constexpr int n = decltype(nn)::value;
      if constexpr (n < decltype(st)::PER_WAVE)
        zp_dma16_so(pc_t, st.off[n], __builtin_amdgcn_readfirstlane(zp_lds_addr(own) + (2 * (buf ^ 1) + half) * TILEB + st.dest(n)));
      else
        zp_dma4_so(pc_r, (lane & 31) * 4, __builtin_amdgcn_readfirstlane(zp_lds_addr(Ls) + (buf ^ 1) * 512 + half * 256));
    };
    auto no_piece = [](auto) {};
    if (compute) {
      if (masked)
        dkdv_half_block<D, AHEAD, 2 * buf * TILEB, (2 * buf + 1) * TILEB, 256, true>(seed + buf * 512, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, no_piece);
      else if (D == 128 && fused)
        dkdv_half_block<D, AHEAD, 2 * buf * TILEB, (2 * buf + 1) * TILEB, 256, false>(seed + buf * 512, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, stage_piece);
      else
        dkdv_half_block<D, AHEAD, 2 * buf * TILEB, (2 * buf + 1) * TILEB, 256, false>(seed + buf * 512, kreg, vreg, dk_acc, dv_acc, qpos0, kpos, qpos_end_l, c_log2, la, no_piece);
    }
    i0 = next_i0;
    on(next_i0, next_hh);
  };
  for (int it = group; it - group < n_it; it += 8) {
    query_tile(it, std::integral_constant<int, 0>{});
    if (it - group + 4 < n_it) query_tile(it + 4, std::integral_constant<int, 1>{});
  }

  // add up the four groups' accumulators: of the four results (dK and dV of the two sub-blocks) a wave does half of the
  // columns of one
  constexpr int ACCB = (D / 16) * 64 * 16;  // bytes of one accumulator of one wave
  __syncthreads();
#pragma unroll
  for (int i = 0; i < D / 16; i++) {
    *(ZP_LDS f32x4 *)((ZP_LDS char *)smem + ((group * 2 + half) * 2) * ACCB + (i * 64 + lane) * 16) = dk_acc[i];
    *(ZP_LDS f32x4 *)((ZP_LDS char *)smem + ((group * 2 + half) * 2 + 1) * ACCB + (i * 64 + lane) * 16) = dv_acc[i];
  }
  __syncthreads();
  const int which = group & 1, ch = group >> 1;
  f32x4 sum[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) {
    const ZP_LDS char *at = (const ZP_LDS char *)smem + (half * 2 + which) * ACCB + ((ch * (D / 32) + i) * 64 + lane) * 16;
    sum[i] = *(const ZP_LDS f32x4 *)at;
#pragma unroll
    for (int o = 1; o < 4; o++) {
      const f32x4 v = *(const ZP_LDS f32x4 *)(at + o * 4 * ACCB);
      sum[i][0] += v[0]; sum[i][1] += v[1]; sum[i][2] += v[2]; sum[i][3] += v[3];
    }
  }
  __syncthreads();  // the rows pass through LDS on their way out
  const float mul = which ? 1.0f : p.scale;
  __bf16 *out = which ? p.dv : p.dk;
  const int64_t at = ((int64_t)t.k_tok0 + kb) * p.dkv_stride + (int64_t)g * D + ch * (D / 2);
  if (!p.accumulate) zp_store_rows<D / 2>(smem + wave * ZP_ROWS_LDS_OF(D / 2), sum, mul, out + at, p.dkv_stride, t.k_len - kb, lane);
  else {
    int first = kb;
    asm volatile("" : "+s"(first));  // krow worked out again: a register of its own through the loop was one too many at D = 64
    if (first + c16 < t.k_len) add_acc_rows<D / 2>((float *)out + at + c16 * p.dkv_stride + q4, sum, mul);
  }
}

template <int D>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2, D == 64 ? 4 : 2))) void attn_bwd_dkdv_split_kernel(zp_bwd_params p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dkdv_split_rows<D>(p, blockIdx.x, smem);
}

// dQ and dK/dV in one launch, where both would take the kernels for launches that leave part of the chip idle: the first p.both
// workgroups do what attn_bwd_dkdv_split_kernel does, the others what attn_bwd_dq_pair_kernel does. Neither then needs anything of the
// other's: attn_bwd_rows_kernel works out -D and -LSE / scale in front. (Worked out in the dK/dV workgroups instead, tile by tile, they
// took more of a CU's 64 bytes per cycle from L2 than Q and dO leave: an iteration 2.6 us instead of 1.2.) Bound: the longer of the two
// longest chains, and 4 us for the rows. Backward of 1218 tokens in eight sequences, GQA 4/2, d = 128: 23.8 -> 16.6 us, passes one
// after the other; zp_take_both has more figures and the rule.
template <int D>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bwd_both_kernel(zp_bwd_params p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int block = blockIdx.x;
  if (block < p.both) dkdv_split_rows<D>(p, block, smem);
  else dq_pair_rows<D, true>(p, block - p.both, smem);
}
template <int D>
constexpr size_t split_lds() {
  constexpr size_t loop = 4 * (size_t)split_own<D>(), end = 16 * (D / 16) * 64 * 16;
  return loop > end ? loop : end;
}

}  // namespace

extern "C" void zp_prof_begin(const char *name, hipStream_t stream);
extern "C" void zp_prof_end(hipStream_t stream);

extern "C" int zp_attn_bwd_block_rows(int d, int which) { (void)d; (void)which; return 128; }

extern "C" int zp_launch_attn_bwd(const zp_bwd_params *p_in, int d, hipStream_t stream) {
  zp_bwd_params params = *p_in;
  zp_bwd_params *p = &params;
  p->m_hkv = zp_div_magic(p->Hkv);
  p->m_grp = zp_div_magic(p->grp);
  const int dq_units = p->n_dq_tiles * p->Hkv;
  const int kv_units = p->n_kv_tiles * p->Hkv;
  // item numbering padded to a multiple of 8 (one residue per XCD); the kernels drop the padding
  int32_t *c = p->work_dq.counters;
  const int dq_grid = zp_plan_work_split(p->work_dq, c, ((dq_units + 7) / 8) * 8 * p->grp);
  const int kv_grid = zp_plan_work_split(p->work_kv, c ? c + ZP_COUNTER_BYTES / 4 : nullptr, ((kv_units + 7) / 8) * 8);
  const dim3 pair_grid(((dq_units + 7) / 8) * 8 * p->grp * (p->dq_pair == ZP_PAIR_HALVES ? 2 : 1)), split_grid(((kv_units + 7) / 8) * 8 * 4);
  if (p->both && dq_units > 0 && kv_units > 0) {
    const dim3 grid(split_grid.x + pair_grid.x);
    p->both = (int)split_grid.x;
    zp_prof_begin("attn_bwd_both", stream);
    if (d == 128) {
      hipLaunchKernelGGL(attn_bwd_rows_kernel<128>, pair_grid, dim3(256), 0, stream, *p);
      hipLaunchKernelGGL(attn_bwd_both_kernel<128>, grid, dim3(512), std::max(dq_pair_lds<128>(), split_lds<128>()), stream, *p);
    } else {
      hipLaunchKernelGGL(attn_bwd_rows_kernel<64>, pair_grid, dim3(256), 0, stream, *p);
      hipLaunchKernelGGL(attn_bwd_both_kernel<64>, grid, dim3(512), std::max(dq_pair_lds<64>(), split_lds<64>()), stream, *p);
    }
    zp_prof_end(stream);
    return (int)hipGetLastError();
  }
  if (dq_units > 0) {
    zp_prof_begin(p->dq_pair ? "attn_bwd_dq_pair" : "attn_bwd_dq", stream);
    if (p->dq_pair) {
      if (d == 128) hipLaunchKernelGGL(attn_bwd_dq_pair_kernel<128>, pair_grid, dim3(512), dq_pair_lds<128>(), stream, *p);
      else hipLaunchKernelGGL(attn_bwd_dq_pair_kernel<64>, pair_grid, dim3(512), dq_pair_lds<64>(), stream, *p);
    } else if (d == 128) hipLaunchKernelGGL((attn_bwd_dq_kernel<128>), dim3(dq_grid), dim3(BWD_NT), 4 * 64 * 128 * 2 + 16, stream, *p);
    else hipLaunchKernelGGL((attn_bwd_dq_kernel<64>), dim3(dq_grid), dim3(BWD_NT), 4 * 64 * 64 * 2 + 16, stream, *p);
    zp_prof_end(stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  if (kv_units > 0) {
    zp_prof_begin(p->kv_split ? "attn_bwd_dkdv_split" : p->kv_pair && d == 128 ? "attn_bwd_dkdv_pair" : p->share_its ? "attn_bwd_dkdv_shares" : "attn_bwd_dkdv", stream);
    if (p->kv_split) {
      if (d == 128) hipLaunchKernelGGL(attn_bwd_dkdv_split_kernel<128>, split_grid, dim3(512), split_lds<128>(), stream, *p);
      else hipLaunchKernelGGL(attn_bwd_dkdv_split_kernel<64>, split_grid, dim3(512), split_lds<64>(), stream, *p);
    } else if (d == 128) {
      constexpr size_t R16 = zp_pad16<128>::R16;
      if (p->kv_pair) hipLaunchKernelGGL(attn_bwd_dkdv128_kernel<2>, dim3(kv_grid), dim3(2 * BWD_NT), std::max(24 * R16 + 2 * 1024 + 16, (size_t)131072), stream, *p);
      else hipLaunchKernelGGL(attn_bwd_dkdv128_kernel<1>, dim3(kv_grid), dim3(BWD_NT), 16 * R16 + 1024 + 16, stream, *p);
    } else {
      hipLaunchKernelGGL(attn_bwd_dkdv64_kernel, dim3(kv_grid), dim3(BWD_NT), 8 * 64 * 64 * 2 + 2048 + 16, stream, *p);
    }
    zp_prof_end(stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}
