// Backward for short key segments (at most 256 keys each) at head_dim 128: one pass over the
// queries computes dQ, dK and dV together.
//
// What bounds it: HBM. With so few keys a query row is worth about as many flops as its bytes
// allow (180 flop per byte on the caption workload), and three separate passes (Delta, dK/dV, dQ)
// read q and dout two or three times and recompute the scores. When a workgroup holds all keys of
// a sequence, dQ needs no sum over workgroups, so here a workgroup takes one (sequence, head) and
// a piece of its queries, keeps K in LDS (V as operands in registers) and streams Q, dO and O
// through LDS once: Delta from the O and dO tiles, S, dP, then dV and dK into registers and dQ
// out, 5 matrix products instead of 7 and q, dout and out read once.
// Measured on 116,904 queries against 32-256 keys at 12 heads: 818 us for the three passes, 538 us
// here, 507 of them in this kernel and the rest in the reduce. In a profile of 55 launches (561 us in the
// mean) it moves 2.9 TB/s with the MFMAs busy 32%: four waves a CU with two barriers a step.
// dK and dV of a piece go to a partial slot and are summed by the reduce kernel in piece order,
// as for split loops (no atomics; results are reproducible bit for bit).
#include <type_traits>

#include "t2v_kernel_common.hpp"

namespace t2v {

using namespace kern;

namespace {

constexpr int D = 128;
constexpr int KK = D / 16;
constexpr int DB = D / 32;
constexpr int NT = 256;           // four waves
constexpr int kKeys = 256;        // keys a workgroup can hold
constexpr int BM = 32;            // queries per step and LDS stage
constexpr int NS = 3;             // LDS stages
constexpr int kOps = 3 * 2 + 1;   // DMA instructions per wave and stage: Q, dO, O and lse
constexpr int kSStride = 36;      // row stride (elements) of the dS tile: 72 bytes spread its rows over the banks

struct ShortArgs {
  const bf16 *q, *k, *v, *out, *dout;
  const float* lse;
  int H;
  int64_t T;
  float c, scale;
  bf16 *dq, *dk, *dv;
  float *ndelta, *lse2, *partial;
  unsigned long long* trace;
};

struct Lds {
  bf16 k[kKeys * D];
  bf16 q[NS][BM * D], g[NS][BM * D], o[NS][BM * D];
  bf16 s[kKeys * kSStride];  // dS of the current step, row = key, column = query
  float raw[NS][64];         // lse of a stage (the first BM are used)
  float l2[2][BM], nd[2][BM];  // lse * log2(e) and -Delta of this step and the next
};

// The element `off` bytes after a wave-uniform pointer.
template <typename V>
T2V_DEV V& at_offset(const void* base, uint32_t off) {
  return *reinterpret_cast<V*>(reinterpret_cast<char*>(const_cast<void*>(uniform_ptr(base))) + off);
}

// Sum over eight neighbouring lanes, in every lane.
T2V_DEV float sum8(float x) {
  auto add = [&](auto ctrl) {
    const int y = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true);
    x += __builtin_bit_cast(float, y);
  };
  add(std::integral_constant<int, 0xB1>{});   // quad_perm 1 0 3 2
  add(std::integral_constant<int, 0x4E>{});   // quad_perm 2 3 0 1
  add(std::integral_constant<int, 0x141>{});  // row_half_mirror: the other quad
  return x;
}

// One work item with KB 32-key blocks per wave: 1 for at most 128 keys, else 2.
template <int KB>
T2V_DEV void short_item(const ShortArgs& a, const Item& it, Lds& lds) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = lane >> 5, l32 = lane & 31;
  const int Lk = it.len, L = it.llen;
  const int64_t rs = static_cast<int64_t>(a.H) * D;
  const int64_t base = static_cast<int64_t>(it.row0) * rs + static_cast<int64_t>(it.head) * D;
  const int64_t qbase = static_cast<int64_t>(it.lrow0) * rs + static_cast<int64_t>(it.head) * D;
  const int64_t lbase = static_cast<int64_t>(it.head) * a.T + it.lrow0;
  const int ntiles = (L + BM - 1) / BM;

  const TileDma<D, BM, NT> dma(tid, rs);
  auto stage = [&](int t) {
    const int b = t % NS, i0 = t * BM;
    dma.copy(lds.q[b], a.q + qbase, rs, i0, L);
    dma.copy(lds.g[b], a.dout + qbase, rs, i0, L);
    dma.copy(lds.o[b], a.out + qbase, rs, i0, L);
    // Every wave copies the same row statistics, so each issues kOps copies a stage.
    const uint32_t r = static_cast<uint32_t>(min(lane, L - 1 - i0));
    const uint32_t dst = lds_addr(lds.raw[b]);
#if T2V_CHECKED
    if (!check_row(i0 + static_cast<int>(r), L)) {
      dma_lds4_s(a.lse + lbase, 0u, dst);
      return;
    }
#endif
    dma_lds4_s(a.lse + lbase + i0, r * 4, dst);
  };
  stage(0);
  const TileDma<D, 128 * KB, NT> kd(tid, rs);
  kd.copy(lds.k, a.k + base, rs, 0, Lk);
  bf16x8 vop[KB][KK];
  f32x16 dka[KB][DB], dva[KB][DB];
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    const int k0 = (wave * KB + b) * 32;
    const bf16* v0 = a.v + base + k0 * rs;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      vop[b][kk] = load8(&at_offset<bf16>(v0, l32 * static_cast<uint32_t>(rs * 2) + G * 16 + kk * 32), k0 + l32 < Lk);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      dka[b][db] = zero16();
      dva[b][db] = zero16();
    }
  }
  wait_vmcnt0();
  if (1 < ntiles) stage(1);
  __syncthreads();

  const uint32_t oo = opnd_lane_off<D>(lane);
  const uint32_t ro0 = rows_lane_off<D>(lane, 0), ro1 = rows_lane_off<D>(lane, 1);
  const uint32_t kbase = lds_addr(lds.k), kwave = kbase + oo + wave * KB * 32 * 2 * D;
  // -Delta and lse * log2(e) of step t: eight queries per wave, eight lanes each.
  auto row_stats = [&](int t, int b3) {
    const int ln = lane_again();
    const int dr = wave * 8 + (ln >> 3), sub = ln & 7;
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 x = swz_read8<D>(lds.o[b3], dr, 2 * sub + j), y = swz_read8<D>(lds.g[b3], dr, 2 * sub + j);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(static_cast<float>(x[e]), static_cast<float>(y[e]), acc);
    }
    acc = sum8(acc);
    const int i = t * BM + dr;
    if (sub == 0) {
      const float l2 = lds.raw[b3][dr] * kLog2e;
      lds.l2[t & 1][dr] = i < L ? l2 : kInf;  // P = 0 for the copies of the last row past the piece
      lds.nd[t & 1][dr] = -acc;
      if (i < L) {  // uniform bases and 32-bit lane offsets, here and in dq_store: fewer registers
        const int64_t at = lbase + t * BM;
        at_offset<float>(a.ndelta + at, dr * 4) = -acc;
        at_offset<float>(a.lse2 + at, dr * 4) = l2;
      }
    }
  };
  row_stats(0, 0);
  __syncthreads();

  // dQ^T of this wave's 32 head-dim columns, K^T dS^T over all keys (dS rows past the segment are
  // zero): k-step ks of the contraction.
  f32x16 dqa;
  auto dq_opnd = [&](int ks, bf16x8& kt, bf16x8& st) {
    kt = read_rows_opnd<D>(kbase + ro0, kbase + ro1, ks * 16, wave);
    st = lds_read_rows_operand(lds.s, kSStride, ks * 16, 0, lane);
  };
  auto dq_store = [&](int t) {
    const int ln = lane_again();
    if (t * BM + (ln & 31) < L) {
      bf16* rows = a.dq + qbase + static_cast<int64_t>(t) * BM * rs + wave * 32;
      const uint32_t off = static_cast<uint32_t>(ln & 31) * static_cast<uint32_t>(rs * 2) + (ln >> 5) * 8;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = static_cast<bf16>(dqa[i * 4 + e] * a.scale);
        at_offset<bf16x4>(rows, off + i * 16) = w;
      }
    }
  };
  constexpr int AH = 4;                // score operands read ahead of their MFMA
  constexpr int QH = KB == 2 ? 2 : 4;  // dQ operand pairs read ahead
  for (int t = 0, b3 = 0; t < ntiles; ++t) {
    const int n3 = b3 + 1 == NS ? 0 : b3 + 1;
    const uint32_t tq = lds_addr(lds.q[b3]), tg = lds_addr(lds.g[b3]);
    if (t + 2 < ntiles) stage(t + 2);  // into the buffers of step t - 1
    // First half: S and dP (32 queries x 32 keys per block: lane = key, register r = query
    // 8 (r/4) + 4 G + r % 4; dP starts at -Delta) interleaved with dQ of the previous step (of
    // step 0: nothing, not stored), P under the dP products.
    f32x16 s[KB], dp[KB];
    f32x4 l2[4];
    bf16x8 aq[KK], kb[KB][KK], ag[KK], kt[QH + 1], st[QH + 1], pb[KB][2], bg[2][DB];
    auto p_unit = [&](int u) {
      const int b = u >> 4, r = u & 15;
      float p = __builtin_amdgcn_exp2f(fmaf(s[b][r], a.c, -l2[r >> 2][r & 3]));
      pin(p);
      s[b][r] = p;
      if ((r & 7) == 7) {
        pb[b][r >> 3] = to_bf16x8(s[b], r & 8);
        pin(pb[b][r >> 3]);
      }
    };
    auto read_dq = [&](int ks) {
      if (ks < 8 * KB) dq_opnd(ks, kt[ks % (QH + 1)], st[ks % (QH + 1)]);
    };
    auto read_s = [&](int kk) {
      aq[kk] = read_opnd<D>(tq + oo, 0, kk);
#pragma unroll
      for (int b = 0; b < KB; ++b) kb[b][kk] = read_opnd<D>(kwave, b * 32, kk);
    };
#pragma unroll
    for (int ks = 0; ks < QH; ++ks) read_dq(ks);
#pragma unroll
    for (int kk = 0; kk < AH; ++kk) read_s(kk);
    dqa = zero16();
#pragma unroll
    for (int b = 0; b < KB; ++b) s[b] = zero16();
    fence();
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int b = 0; b < KB; ++b) s[b] = mfma(aq[kk], kb[b][kk], s[b]);
      dqa = mfma(kt[kk % (QH + 1)], st[kk % (QH + 1)], dqa);
      fence();
      read_dq(kk + QH);
      if (kk + AH < KK) read_s(kk + AH);
      if (kk < 4) {
        l2[kk] = *reinterpret_cast<const f32x4*>(lds.l2[t & 1] + kk * 8 + G * 4);
        const f32x4 nd = *reinterpret_cast<const f32x4*>(lds.nd[t & 1] + kk * 8 + G * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int b = 0; b < KB; ++b) dp[b][kk * 4 + e] = nd[e];
      }
      if (kk >= KK - AH) ag[kk - (KK - AH)] = read_opnd<D>(tg + oo, 0, kk - (KK - AH));
      fence();
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int b = 0; b < KB; ++b) dp[b] = mfma(ag[kk], vop[b][kk], dp[b]);
      if (KB == 2) dqa = mfma(kt[(KK + kk) % (QH + 1)], st[(KK + kk) % (QH + 1)], dqa);
      fence();
      read_dq(KK + kk + QH);
      if (kk + AH < KK) ag[kk + AH] = read_opnd<D>(tg + oo, 0, kk + AH);
      if (kk >= KK - DB) bg[0][kk - (KK - DB)] = read_rows_opnd<D>(tg + ro0, tg + ro1, 0, kk - (KK - DB));
#pragma unroll
      for (int u = 2 * KB * kk; u < 2 * KB * (kk + 1); ++u) p_unit(u);
      fence();
    }
    if (t > 0) dq_store(t - 1);
    // Stage t + 1 complete; what was issued after it may still be in flight: the copy of stage
    // t + 2 and the four dQ stores above (issued by every wave: step t - 1 is full).
    if (t + 2 >= ntiles)
      wait_vmcnt0();
    else if (t > 0)
      wait_vmcnt<kOps + 4>();
    else
      wait_vmcnt<kOps>();
    __syncthreads();  // the previous dS tile is read; stage t + 1 is visible
    // Second half: dV, with dS under it and out to the dS tile, the next step's row statistics, dK.
    bf16x8 sb[KB][2], bq[2][DB];
    auto s_unit = [&](int u) {
      const int b = u >> 4, r = u & 15;
      // Keys past the segment (copies of its last row) must not reach dQ.
      float x = (wave * KB + b) * 32 + l32 < Lk ? s[b][r] * dp[b][r] : 0.0f;
      pin(x);
      dp[b][r] = x;
      if ((r & 7) == 7) {
        const int h = r >> 3;
        sb[b][h] = to_bf16x8(dp[b], 8 * h);
        pin(sb[b][h]);
        bf16* row = lds.s + ((wave * KB + b) * 32 + l32) * kSStride + 16 * h + 4 * G;
        const bf16x8 y = sb[b][h];
        *reinterpret_cast<bf16x4*>(row) = bf16x4{y[0], y[1], y[2], y[3]};
        *reinterpret_cast<bf16x4*>(row + 8) = bf16x4{y[4], y[5], y[6], y[7]};
      }
    };
    fence();
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) {
      const int h = i / DB, db = i % DB;
#pragma unroll
      for (int b = 0; b < KB; ++b) mfma_acc(dva[b][db], pb[b][h], bg[h][db]);
      fence();
      if (h == 0) bg[1][db] = read_rows_opnd<D>(tg + ro0, tg + ro1, 16, db);
      if (h == 1) bq[0][db] = read_rows_opnd<D>(tq + ro0, tq + ro1, 0, db);
#pragma unroll
      for (int u = 2 * KB * i; u < 2 * KB * (i + 1); ++u) s_unit(u);
      fence();
    }
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) {
      const int h = i / DB, db = i % DB;
#pragma unroll
      for (int b = 0; b < KB; ++b) mfma_acc(dka[b][db], sb[b][h], bq[h][db]);
      fence();
      if (h == 0) bq[1][db] = read_rows_opnd<D>(tq + ro0, tq + ro1, 16, db);
      if (i == 1) row_stats(t + 1, n3);
      fence();
    }
    __syncthreads();  // dS and the next row statistics are visible; this step's tiles are read
    b3 = n3;
  }
  dqa = zero16();
#pragma unroll 2
  for (int ks = 0; ks < 8 * KB; ++ks) {
    bf16x8 kt, st;
    dq_opnd(ks, kt, st);
    dqa = mfma(kt, st, dqa);
  }
  dq_store(ntiles - 1);

  acc_settle();
  __syncthreads();  // every wave has read its last dS and K rows: the LDS is free
  // Accumulators: lane = head-dim column db*32 + l32, register r = key 8 (r/4) + 4 G + r % 4. They
  // leave through this wave's part of the LDS, as rows of fp32.
  const int el = lane_again();
  float* rows = reinterpret_cast<float*>(&lds) + wave * (KB * 32 * D);
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const f32x16(&acc)[KB][DB] = which == 0 ? dka : dva;
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          rows[(b * 32 + (r >> 2) * 8 + (el >> 5) * 4 + (r & 3)) * D + db * 32 + (el & 31)] = acc_read(acc[b][db][r]);
    const int c4 = (el & 31) * 4;
    const float m = which == 0 ? a.scale : 1.0f;
    float* slot = a.partial + static_cast<int64_t>(max(it.slot, 0)) * (2 * kKeys * D) + which * kKeys * D;
    bf16* grad = (which == 0 ? a.dk : a.dv) + base;
#pragma unroll 4
    for (int j = 0; j < KB * 16; ++j) {
      const int kr = 2 * j + (el >> 5), kj = wave * KB * 32 + kr;
      const f32x4 x = *reinterpret_cast<const f32x4*>(rows + kr * D + c4);
      if (kj >= Lk) continue;
      if (it.slot >= 0) {  // unscaled sums of this piece
        *reinterpret_cast<f32x4*>(slot + kj * D + c4) = x;
      } else {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = static_cast<bf16>(x[e] * m);
        *reinterpret_cast<bf16x4*>(grad + kj * rs + c4) = w;
      }
    }
  }
}

__global__ __launch_bounds__(NT, 1) void attn_bwd_short_kernel(ShortArgs a, const Item* __restrict__ items) {
  __shared__ __attribute__((aligned(1024))) Lds lds;
  const unsigned long long trace_t0 = a.trace != nullptr ? trace_clock() : 0ull;
  const Item it = items[blockIdx.x];
  if (it.len <= 128)
    short_item<1>(a, it, lds);
  else
    short_item<2>(a, it, lds);
  if (a.trace != nullptr) trace_end(a.trace, trace_t0, 2, blockIdx.x);
}

// Sum of one segment's partial slots in piece order, scaled (dK) and rounded. A workgroup takes
// 16 keys, both gradients; each thread four consecutive head-dim columns of one key at a time.
constexpr int kRedKeys = 16;
__global__ __launch_bounds__(NT) void short_reduce_kernel(const float* __restrict__ partial,
                                                         const Item* __restrict__ segs, int H, float scale,
                                                         bf16* __restrict__ dk, bf16* __restrict__ dv) {
  constexpr int C4 = D / 4;
  const Item it = segs[blockIdx.x / (kKeys / kRedKeys)];
  const int k0 = (blockIdx.x % (kKeys / kRedKeys)) * kRedKeys;
  const int64_t rs = static_cast<int64_t>(H) * D;
  constexpr int64_t kSlot = 2 * kKeys * D;
  for (int e = threadIdx.x; e < 2 * kRedKeys * C4; e += NT) {
    const int which = e / (kRedKeys * C4), key = k0 + (e / C4) % kRedKeys, c4 = e % C4;
    if (key >= it.len) continue;
    const float* src = partial + it.slot * kSlot + which * kKeys * D + key * D + c4 * 4;
    f32x4 acc = *reinterpret_cast<const f32x4*>(src);
    for (int p = 1; p < it.pieces; ++p) acc += *reinterpret_cast<const f32x4*>(src + p * kSlot);
    const float m = which == 0 ? scale : 1.0f;
    bf16x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = static_cast<bf16>(acc[i] * m);
    *reinterpret_cast<bf16x4*>((which == 0 ? dk : dv) + static_cast<int64_t>(it.row0 + key) * rs +
                               static_cast<int64_t>(it.head) * D + c4 * 4) = w;
  }
}

}  // namespace

int short_keys() { return kKeys; }

int64_t short_partial_slot_bytes() { return 2LL * kKeys * D * 4; }

hipError_t launch_bwd_short(const AttnArgs& a, const Item* items, int n_items, const Item* segs, int n_segs,
                            hipStream_t stream) {
  if (a.head_dim != D) return hipErrorInvalidValue;
  ShortArgs s{};
  s.q = static_cast<const bf16*>(a.q);
  s.k = static_cast<const bf16*>(a.k);
  s.v = static_cast<const bf16*>(a.v);
  s.out = static_cast<const bf16*>(a.out);
  s.dout = static_cast<const bf16*>(a.dout);
  s.lse = a.lse;
  s.H = a.heads;
  s.T = a.total_tokens;
  s.c = a.scale * kLog2e;
  s.scale = a.scale;
  s.dq = static_cast<bf16*>(a.dq);
  s.dk = static_cast<bf16*>(a.dk);
  s.dv = static_cast<bf16*>(a.dv);
  s.ndelta = a.delta;
  s.lse2 = a.delta + a.total_tokens * a.heads;
  s.partial = a.partial;
  s.trace = a.trace;
  hipLaunchKernelGGL(attn_bwd_short_kernel, dim3(n_items), dim3(NT), 0, stream, s, items);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && n_segs > 0) {
    hipLaunchKernelGGL(short_reduce_kernel, dim3(n_segs * (kKeys / kRedKeys)), dim3(NT), 0, stream, a.partial, segs,
                       a.heads, a.scale, s.dk, s.dv);
    e = hipGetLastError();
  }
  return e;
}
#if T2V_CHECKED
hipError_t short_check_take(unsigned int* rec, unsigned int canary) { return kern::check_take_here(rec, canary); }
#endif
}  // namespace t2v
