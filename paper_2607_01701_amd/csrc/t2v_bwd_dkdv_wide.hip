// Backward dK/dV kernel for long query loops: a workgroup of four waves owns 256 keys of one
// (clip, head), 64 per wave, and loops over the clip's queries in 32-query steps.
//
// What bounds it: the matrix cores, through power. The 32-keys-per-wave kernel
// (t2v_bwd_dkdv.hip) spends 56 LDS reads on 32 MFMAs and leaves the softmax arithmetic of its
// only wave per SIMD exposed (MFMAs busy 55% of cycles). Here every Q and dO operand feeds two
// key blocks, so at D = 128 a step of 64 MFMAs takes 72 LDS reads (1.1 per MFMA instead of
// 1.75) and half the LDS copies per MFMA, and the step is one hand-scheduled stream in which the
// softmax arithmetic runs under the MFMAs (64% busy, at a clock that the card lowers from 1.96
// to 1.82 GHz as it reaches its power limit). Measured on the heterogeneous mix (24 x 128):
// 34.9 -> 30.6 ms, 1,110 -> 1,267 TFLOP/s; results are bitwise those of the other kernel.
//
// Registers (D = 128): the dK and dV sums of 64 keys fill all 256 AGPRs; V operands take 64
// VGPRs; K operands, which would take 64 more, are read from an LDS tile instead (16 reads of
// the 72). LDS: 64 KB of K and five 16 KB stages of Q and dO. head_dim 64 keeps the other kernel:
// there a step's arithmetic is as long as its MFMAs, and two waves per SIMD, which can issue
// both at once, do better than one (1,131 against 1,085 TFLOP/s at 16,384 tokens).
#include "t2v_kernel_common.hpp"

namespace t2v {

using namespace kern;

namespace {

constexpr int kWideKeys = 256;  // keys per workgroup
constexpr int kBM = 32;         // queries per LDS stage and per step

constexpr int D = 128;          // head dim
constexpr int KK = D / 16;      // k-steps of the head-dim contraction
constexpr int DB = D / 32;      // 32-wide head-dim blocks
constexpr int kStages = 5;      // LDS stages
constexpr int kAhead = 4;       // operands read ahead of their MFMA
constexpr int kWideThreads = 256;
constexpr int kOps = 2 * (kBM * D / 512) / 4 + 1;  // DMA instructions per wave and stage
// Arithmetic per slot of a step: one P element from slot kPFirst on (when S of block 0 is
// ready), then two dS elements.
constexpr int kPRate = 1, kPFirst = KK + 1;
constexpr int kSRate = 2, kSFirst = kPFirst + 32 / kPRate;

constexpr int clamp32(int x) { return x < 0 ? 0 : x > 32 ? 32 : x; }

// Copy of 64 consecutive floats into LDS, one per lane: lane i takes row i0 + i, clamped to
// L - 1 (i0 < L).
T2V_DEV void rows_dma(float* lds, const float* g, int i0, int L, int lane) {
  const uint32_t r = static_cast<uint32_t>(min(lane, L - 1 - i0));
  const uint32_t dst = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)lds));
#if T2V_CHECKED
  if (!check_row(i0 + static_cast<int>(r), L)) {  // copy the segment's first row instead
    dma_lds4_s(g, 0u, dst);
    return;
  }
#endif
  dma_lds4_s(g + i0, r * 4, dst);
}

// LDS addresses of one step's operands: this lane's base in the Q and dO tiles (16-byte and
// transposing reads), in the next stage's Q tile, and in this wave's K rows.
struct StepAddr {
  uint32_t q, g, qr0, qr1, gr0, gr1, qnext, k;
  const float *lse2, *ndelta;
};

// One 32-query step. Slots: S of key block 0 (KK MFMAs), S of block 1 (KK), dP of both (2 KK),
// dV of both (4 DB), dK of both (4 DB); 64 MFMAs at D = 128. Block 0's scores come first so that
// its softmax runs under block 1's; P of a 16-query half is due at its dV products, dS at its dK
// products. `sync` sits between dP and dV: it waits for the next stage, whose first operands
// the dK slots read, and frees the previous stage's buffer for a new copy.
// aq holds this step's Q operands on entry and the next one's on return; kb likewise the first K
// operands. RAGGED: only the first nvalid queries count.
template <bool RAGGED, typename Sync>
T2V_DEV void dkdv_wide_step(const StepAddr& a, int nvalid, float c, bf16x8 (&aq)[KK], bf16x8 (&kb)[kAhead],
                            const bf16x8 (&vop)[2][KK], f32x16 (&dka)[2][DB], f32x16 (&dva)[2][DB], int lane,
                            Sync&& sync) {
  constexpr int AH = kAhead;
  const int G = lane >> 5;
  f32x16 s[2], dp[2], nd;
  s[0] = zero16();
  s[1] = zero16();
  f32x4 lv[4];
  bf16x8 ag[KK], pb[2][2], sb[2][2], bg[2][DB], bq[2][DB];
  auto read_k = [&](int i) { kb[i % AH] = read_opnd<D>(a.k, (i / KK) * 32, i % KK); };
  // Arithmetic unit u of 32: element u % 8 of 16-query half u / 16 of key block (u / 8) % 2, i.e.
  // in the order in which the dV (dK) products need the halves; the eighth converts the half.
  auto p_unit = [&](int u) {
    const int b = (u >> 3) & 1, h = u >> 4, r = 8 * h + (u & 7);
    float p = __builtin_amdgcn_exp2f(fmaf(s[b][r], c, -lv[r >> 2][r & 3]));
    if constexpr (RAGGED) {
      const int qi = (r >> 2) * 8 + G * 4 + (r & 3);
      p = qi < nvalid ? p : 0.0f;
    }
    pin(p);
    s[b][r] = p;
    if ((u & 7) == 7) {
      pb[b][h] = to_bf16x8(s[b], 8 * h);
      pin(pb[b][h]);
    }
  };
  auto s_unit = [&](int u) {
    const int b = (u >> 3) & 1, h = u >> 4, r = 8 * h + (u & 7);
    float x = s[b][r] * dp[b][r];
    pin(x);
    dp[b][r] = x;
    if ((u & 7) == 7) {
      sb[b][h] = to_bf16x8(dp[b], 8 * h);
      pin(sb[b][h]);
    }
  };
  auto arithmetic = [&](int slot) {
#pragma unroll
    for (int u = clamp32((slot - kPFirst) * kPRate); u < clamp32((slot + 1 - kPFirst) * kPRate); ++u)
      p_unit(u);
#pragma unroll
    for (int u = clamp32((slot - kSFirst) * kSRate); u < clamp32((slot + 1 - kSFirst) * kSRate); ++u)
      s_unit(u);
  };
  fence();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {  // S of block 0; the row statistics arrive
    s[0] = mfma(aq[kk], kb[kk % AH], s[0]);
    fence();
    read_k(kk + AH);
    const f32x4 x = *reinterpret_cast<const f32x4*>((kk < 4 ? a.lse2 : a.ndelta) + (kk & 3) * 8 + G * 4);
    if (kk < 4) {
      lv[kk & 3] = x;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) nd[(kk & 3) * 4 + e] = x[e];
    }
    fence();
  }
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {  // S of block 1
    s[1] = mfma(aq[kk], kb[(KK + kk) % AH], s[1]);
    fence();
    if (kk + KK + AH < 2 * KK) read_k(kk + KK + AH);
    if (kk >= KK - AH) ag[kk - (KK - AH)] = read_opnd<D>(a.g, 0, kk - (KK - AH));
    arithmetic(KK + kk);
    fence();
  }
#pragma unroll
  for (int i = 0; i < 2 * KK; ++i) {  // dP - Delta of both blocks (the accumulators start at -Delta)
    const int kk = i >> 1, b = i & 1;
    dp[b] = mfma(ag[kk], vop[b][kk], kk == 0 ? nd : dp[b]);
    fence();
    if (b == 0) {
      if (kk + AH < KK) ag[kk + AH] = read_opnd<D>(a.g, 0, kk + AH);
      if (kk >= KK - DB) bg[0][kk - (KK - DB)] = read_rows_opnd<D>(a.gr0, a.gr1, 0, kk - (KK - DB));
    }
    arithmetic(2 * KK + i);
    fence();
  }
  sync();
  fence();
#pragma unroll
  for (int i = 0; i < 4 * DB; ++i) {  // dV += P^T dO
    const int h = i / (2 * DB), b = (i / DB) & 1, db = i % DB;
    mfma_acc(dva[b][db], pb[b][h], bg[h][db]);
    fence();
    if (i < DB) bg[1][i] = read_rows_opnd<D>(a.gr0, a.gr1, 16, i);
    if (i >= 2 * DB && i < 3 * DB) bq[0][i - 2 * DB] = read_rows_opnd<D>(a.qr0, a.qr1, 0, i - 2 * DB);
    arithmetic(4 * KK + i);
    fence();
  }
#pragma unroll
  for (int i = 0; i < 4 * DB; ++i) {  // dK += dS^T Q; the next step's first operands arrive
    const int h = i / (2 * DB), b = (i / DB) & 1, db = i % DB;
    mfma_acc(dka[b][db], sb[b][h], bq[h][db]);
    fence();
    if (i < DB) bq[1][i] = read_rows_opnd<D>(a.qr0, a.qr1, 16, i);
    if (i >= 4 * DB - KK) aq[i - (4 * DB - KK)] = read_opnd<D>(a.qnext, 0, i - (4 * DB - KK));
    if (i >= 4 * DB - AH) read_k(i - (4 * DB - AH));
    arithmetic(4 * KK + 4 * DB + i);
    fence();
  }
}

__global__ __launch_bounds__(kWideThreads, 1) void attn_bwd_dkdv_wide_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v,
    const bf16* __restrict__ dout, const float* __restrict__ lse2, const float* __restrict__ ndelta,
    const Item* __restrict__ items, int H, int64_t T, float c, float scale, bf16* __restrict__ dk,
    bf16* __restrict__ dv, unsigned long long* __restrict__ trace) {
  constexpr int NS = kStages, BM = kBM;
  constexpr uint32_t kTile = BM * D * 2;  // bytes of one stage of Q or dO
  __shared__ __attribute__((aligned(1024))) bf16 sK[kWideKeys * D];
  __shared__ __attribute__((aligned(1024))) bf16 sQ[NS][BM * D];
  __shared__ __attribute__((aligned(1024))) bf16 sG[NS][BM * D];  // dO
  // Row statistics of a stage; each copy fills 64 floats, of which the first BM are used.
  __shared__ __attribute__((aligned(16))) float sL[NS][64];  // lse * log2(e)
  __shared__ __attribute__((aligned(16))) float sD[NS][64];  // -Delta

  const unsigned long long trace_t0 = trace != nullptr ? trace_clock() : 0ull;
  const Item it = items[blockIdx.x];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lk = it.len;   // keys of the sequence (this tile's rows)
  const int L = it.llen;   // queries of the sequence (the loop)
  const int64_t rs = static_cast<int64_t>(H) * D;
  const int64_t base = static_cast<int64_t>(it.row0) * rs + static_cast<int64_t>(it.head) * D;
  const int64_t qbase = static_cast<int64_t>(it.lrow0) * rs + static_cast<int64_t>(it.head) * D;
  const int64_t lbase = static_cast<int64_t>(it.head) * T + it.lrow0;
  const bf16* qh = q + qbase;
  const bf16* gh = dout + qbase;
  // Two waves copy lse2, two -Delta (the same rows twice, so every wave issues kOps copies a stage).
  const float* vec_src = (wave < 2 ? lse2 : ndelta) + lbase;
  const int key_wave0 = it.tile0 + wave * 64;

  const TileDma<D, BM, kWideThreads> dma(tid, rs);
  auto stage = [&](int t) {
    const int b = t % NS, i0 = t * BM;
    dma.copy(sQ[b], qh, rs, i0, L);
    dma.copy(sG[b], gh, rs, i0, L);
    rows_dma(wave < 2 ? sL[b] : sD[b], vec_src, i0, L, lane);
  };
  const int ntiles = (L + BM - 1) / BM;
  stage(0);
  const TileDma<D, kWideKeys, kWideThreads> kd(tid, rs);
  kd.copy(sK, k + base, rs, it.tile0, Lk);
  // V of this wave's 64 keys, as B operands (lane = key, elements along head dim).
  bf16x8 vop[2][KK];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int kj = key_wave0 + b * 32 + (lane & 31);
    const bool ok = kj < Lk;
    const int64_t off = base + kj * rs + (lane >> 5) * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) vop[b][kk] = load8(v + off + kk * 16, ok);
  }
  f32x16 dka[2][DB], dva[2][DB];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      dka[b][db] = zero16();
      dva[b][db] = zero16();
    }
  // Stage 0, the K tile and the operand loads complete here (see t2v_bwd_dkdv.hip).
  wait_vmcnt0();
#pragma unroll
  for (int t = 1; t < NS - 1; ++t)
    if (t < ntiles) stage(t);
  __syncthreads();

  const uint32_t oo = opnd_lane_off<D>(lane);
  const uint32_t ro0 = rows_lane_off<D>(lane, 0), ro1 = rows_lane_off<D>(lane, 1);
  const uint32_t kbase = lds_addr(sK) + oo + wave * 64 * 2 * D;
  const uint32_t lq = lds_addr(sQ), lg = lds_addr(sG);
  auto address = [&](int b, int nb) {
    const uint32_t tq = lq + b * kTile, tg = lg + b * kTile;
    return StepAddr{tq + oo, tg + oo, tq + ro0, tq + ro1, tg + ro0, tg + ro1, lq + nb * kTile + oo, kbase, sL[b], sD[b]};
  };
  auto publish = [] {  // a barrier without the waits that __syncthreads adds for reads in flight
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  bf16x8 aq[KK], kb[kAhead];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) aq[kk] = read_opnd<D>(lq + oo, 0, kk);
#pragma unroll
  for (int kk = 0; kk < kAhead; ++kk) kb[kk] = read_opnd<D>(kbase, 0, kk);
  int tt = 0, b = 0;
#if !T2V_CHECKED
  // Steps whose copy (stage tt + NS - 1) is a full tile: no branches inside a step. After the
  // wait, stages tt + 2 .. tt + NS - 2 may still be in flight.
  const char* qn = reinterpret_cast<const char*>(qh + static_cast<int64_t>(NS - 1) * BM * rs);
  const char* gn = reinterpret_cast<const char*>(gh + static_cast<int64_t>(NS - 1) * BM * rs);
  const uint32_t lv = wave < 2 ? lds_addr(sL) : lds_addr(sD);
  constexpr int kRowsPerCopy = 2048 / D;  // rows the four waves copy with one instruction each
  const int64_t jstep = static_cast<int64_t>(kRowsPerCopy) * rs * 2;
  for (const int nsteady = L / BM - (NS - 1); tt < nsteady; ++tt) {
    const int nb = b + 1 == NS ? 0 : b + 1;
    const uint32_t free_slot = b == 0 ? NS - 1 : b - 1;  // the buffer of step tt - 1
    dkdv_wide_step<false>(address(b, nb), BM, c, aq, kb, vop, dka, dva, lane, [&] {
      wait_vmcnt<(NS - 3) * kOps>();
      publish();
      const uint32_t dq_ = lq + free_slot * kTile + wave * 1024, dg_ = lg + free_slot * kTile + wave * 1024;
#pragma unroll
      for (int j = 0; j < BM / kRowsPerCopy; ++j) dma_lds16_s(qn + j * jstep, dma.off0, dq_ + j * 4096);
#pragma unroll
      for (int j = 0; j < BM / kRowsPerCopy; ++j) dma_lds16_s(gn + j * jstep, dma.off0, dg_ + j * 4096);
      const int i0 = (tt + NS - 1) * BM;
      dma_lds4_s(vec_src + i0, static_cast<uint32_t>(min(lane, L - 1 - i0)) * 4, lv + free_slot * 256);
      qn += static_cast<int64_t>(BM) * rs * 2;
      gn += static_cast<int64_t>(BM) * rs * 2;
    });
    b = nb;
  }
#endif
  for (; tt < ntiles; ++tt) {  // the last steps (in checked builds, all): general copies and masks
    const int nb = b + 1 == NS ? 0 : b + 1;
    dkdv_wide_step<true>(address(b, nb), L - tt * BM, c, aq, kb, vop, dka, dva, lane, [&] {
      wait_vmcnt0();
      publish();
      if (tt + NS - 1 < ntiles) stage(tt + NS - 1);
    });
    b = nb;
  }

  // Accumulators: lane = head-dim column db*32 + l32, register r = key 8 (r/4) + 4 G + r % 4. They
  // leave through this wave's own 16 KB of the K tile, written column by column ([head dim][key],
  // four keys a lane) and read back transposed, so a lane stores 16 bytes of one key row: 32
  // stores a wave in place of 256 two-byte ones.
  acc_settle();
  const int el = lane_again();
  const int eg = el >> 5, ej = el & 15, gr = el >> 4;
  bf16* tile = sK + wave * 64 * D;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const f32x16(&acc)[2][DB] = which == 0 ? dka : dva;
    const float m = which == 0 ? scale : 1.0f;
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          bf16x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = static_cast<bf16>(acc_read(acc[b2][db][4 * i + e]) * m);
          *reinterpret_cast<bf16x4*>(tile + swz_off<64>(db * 32 + (el & 31), b2 * 32 + 8 * i + 4 * eg)) = w;
        }
    bf16* const g = (which == 0 ? dk : dv) + base;
#pragma unroll
    for (int k16 = 0; k16 < 4; ++k16) {
      const int kj = key_wave0 + 16 * k16 + ej;
#pragma unroll
      for (int d32 = 0; d32 < DB; ++d32) {
        const int d0 = 32 * d32 + 8 * gr, r = d0 + (ej >> 2), col = 16 * k16 + 4 * (ej & 3);
        const bf16x4 lo = lds_read_tr4(tile + swz_off<64>(r, col));
        const bf16x4 hi = lds_read_tr4(tile + swz_off<64>(r + 4, col));
        bf16x8 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w[e] = lo[e];
          w[4 + e] = hi[e];
        }
        if (kj < Lk) *reinterpret_cast<bf16x8*>(g + kj * rs + d0) = w;
      }
    }
  }
  if (trace != nullptr) trace_end(trace, trace_t0, 2, blockIdx.x, wave == 0 && el == 0);
}

}  // namespace

int dkdv_wide_rows() { return kWideKeys; }

hipError_t launch_bwd_dkdv_wide(const AttnArgs& a, const Item* items, int n_items, hipStream_t stream) {
  if (a.head_dim != D) return hipErrorInvalidValue;
  const float c = a.scale * kLog2e;
  const float* lse2 = a.delta + a.total_tokens * a.heads;
  const dim3 grid(n_items), block(kWideThreads);
  hipLaunchKernelGGL(attn_bwd_dkdv_wide_kernel, grid, block, 0, stream, static_cast<const bf16*>(a.q),
                     static_cast<const bf16*>(a.k), static_cast<const bf16*>(a.v), static_cast<const bf16*>(a.dout),
                     lse2, a.delta, items, a.heads, a.total_tokens, c, a.scale, static_cast<bf16*>(a.dk),
                     static_cast<bf16*>(a.dv), a.trace);
  return hipGetLastError();
}
#if T2V_CHECKED
hipError_t dkdv_wide_check_take(unsigned int* rec, unsigned int canary) { return kern::check_take_here(rec, canary); }
#endif
}  // namespace t2v
