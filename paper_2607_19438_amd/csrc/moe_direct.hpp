// Grouped MoE GEMM for experts with few routed rows (decode batches, short prompts): weights go
// from HBM to matrix-core operands without an LDS stage.
//
// With a few dozen rows per expert the call is bound by streaming every active expert's packed
// weights once, so what matters is bytes in flight. The staged tiles (moe_kernel) dequantise a
// weight tile into LDS per 64-wide K step and close every step with a barrier that also waits for
// the activation DMA; their workgroups spent most of a step waiting (1.9 TB/s of weights).
// Here a wave owns 32 weight rows outright: it loads its own packed weights into registers, a stage
// of KS 64-wide K sub-steps ahead, dequantises them straight into the A operand of
// v_mfma_f32_32x32x16_bf16, and multiplies with the group's activation rows, which the workgroup's
// waves share through LDS (DMA, double-buffered, one barrier per stage).
//
// What bounds it (MI355X): no single unit. Counters of the gate/up launches (E=128 2048/768 Q4, E=64 2048/1056
// Q8): T=128 Q4 VALU busy 40%, MFMA 13%, LDS 7%, 139 MB fetched at 3.4 TB/s (a large copy reaches 5.2), waves
// 39% of their time in waits; T=4 Q4 24%, 8%, 4%, 2.5 TB/s, 52% (at most 1.5 four-wave workgroups per CU); T=777
// Q8 26%, 19%, 10%, 3.6 TB/s, 45% (two waves per SIMD). A K sub-step of a wave is ~84 VALU instructions (68 of
// them the dequantisation of 32 weights per lane) and 4 MFMAs per 32 rows, and a stage ends in a barrier, so the
// weight stream and the arithmetic overlap only as far as the few waves of a SIMD are at different places.
// Loading a stage's weights at once instead of refilling each register as it is used: T=16 gate/up 47.6 ->
// 44.2 us, T=128 75 -> 67 us (the four loads of a 128-byte line reach the vector L1 together).
//
// The MFMAs add the same products in the same K order as the staged tiles, so a row's result is
// bitwise the same whichever kernel computes it.
#pragma once

#include "qgemm_kernels.hpp"

namespace qg {

// A workgroup's item: a group of an expert's rows (the range of perm) and a column tile.
struct DirItem {
  int rows;        // rows of the group (0: nothing to do)
  int pbeg;
  int nt;
  const uint8_t* wq;
  const uint16_t* sc;
};

__device__ __forceinline__ int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

__device__ __forceinline__ const void* lane_pointer(const void* p, int lane) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
}

// The workgroup's item among (groups of BM rows, experts in order) x (nt_n column tiles), in order of
// the workgroups: each group's tiles spread over the XCDs, so heavy and light groups do too (its few
// activation rows are then read into every L2; dealing whole groups or contiguous ranges to an XCD left
// some CUs with a workgroup more, and contiguous ranges put the heavy experts of skewed routing on one
// XCD: gate/up T=500 skewed 129 us against 106). Every wave finds the item by
// itself: lane l holds experts 2l and 2l + 1 (their offsets and pointers all load at once, one memory
// round trip), a wave prefix sum of their group counts, and a ballot. No barrier.
template <int BM>
__device__ __forceinline__ DirItem dir_item(const TileArgs& a, const ExpertPtrs& ep, int nt_n) {
  const int lane = threadIdx.x & 63;
  const int ne = a.n_experts;
  const int32_t* off = a.offsets + a.e_begin;
  const int o0 = off[min(2 * lane, ne)];
  const int o1 = off[min(2 * lane + 1, ne)];
  const int o2 = off[min(2 * lane + 2, ne)];
  const void* w0 = ep.wq[2 * lane];
  const void* w1 = ep.wq[2 * lane + 1];
  const void* s0 = ep.sc[2 * lane];
  const void* s1 = ep.sc[2 * lane + 1];
  // an inconsistent table entry gives its expert no work (as in moe_kernel)
  const int c0 = (o0 < 0 || o1 > a.M || o1 < o0) ? 0 : o1 - o0;
  const int c1 = (o1 < 0 || o2 > a.M || o2 < o1) ? 0 : o2 - o1;
  const int t0 = (c0 + BM - 1) / BM;
  const int t1 = (c1 + BM - 1) / BM;
  int incl = t0 + t1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(incl, d, 64);
    if (lane >= d) incl += v;
  }
  DirItem it{0, 0, 0, nullptr, nullptr};
  const int item = (int)blockIdx.x;
  if (item >= lane_value(incl, 63) * nt_n) return it;
  const int g = item / nt_n;
  it.nt = item - g * nt_n;
  const int L = __builtin_ctzll(__ballot(incl > g));
  const int first = lane_value(incl - t0 - t1, L);
  const int n0 = lane_value(t0, L);
  const int in = g - first;
  const bool odd = in >= n0;
  const int beg = odd ? lane_value(o1, L) : lane_value(o0, L);
  const int end = odd ? lane_value(o2, L) : lane_value(o1, L);
  it.pbeg = beg + (odd ? in - n0 : in) * BM;
  it.rows = min(BM, end - it.pbeg);
  it.wq = static_cast<const uint8_t*>(odd ? lane_pointer(w1, L) : lane_pointer(w0, L));
  it.sc = static_cast<const uint16_t*>(odd ? lane_pointer(s1, L) : lane_pointer(s0, L));
  return it;
}

// NB 32-row activation blocks (the group's rows), KS 64-wide K sub-steps per stage, WV waves. n0: the
// wave's first weight row (SWI: its first column of h).
template <int FMT, int RB, int NB, int KS, int WV, bool SWI, bool FAST>
__device__ __forceinline__ void dir_body(const TileArgs& a, const DirItem& it, int n0, bool store, lds_char* x0,
                                         lds_char* x1) {
  constexpr int WL = (FMT == kQ8) ? 2 : 1;           // 16-byte weight loads per K sub-step
  constexpr int NW = KS * WL;
  constexpr int SD = KS / 2;                         // scale dwords per lane per stage
  constexpr int kSubBytes = RB * 32 * kRowBytes;     // one K sub-step of the activation stage
  constexpr int kStepBytes = (FMT == kQ8) ? kBK : kBK / 2;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31;
  const int lh = lane >> 5;
  const int K = a.K;
  const int nk = (K + kBK - 1) / kBK;
  const int nst = (nk + KS - 1) / KS;
  const uint32_t kblocks = (uint32_t)K >> 5;
  const uint32_t wrow_bytes = (FMT == kQ8) ? (uint32_t)K : (uint32_t)K >> 1;

  // --- weight rows ---
  // MFMA row i of the A operand is lane i's weight row; the accumulator of lane (token, half h),
  // register 4q + p, is row 8q + 4h + p. Plain: row i is weight row n0 + i. SWI: registers 0..7 are
  // the gate rows of h columns n0 + 8h + 0..7 and registers 8..15 their up rows, so each lane ends
  // with both halves of 8 consecutive columns. Rows past the matrix repeat its last row; their
  // sums are not stored.
  int row;
  if constexpr (SWI) {
    const int q = lr >> 3, half = (lr >> 2) & 1, p = lr & 3;
    const int hc = min(n0 + 8 * half + 4 * (q & 1) + p, a.swi_inter - 1);
    row = q < 2 ? hc : a.swi_inter + hc;
  } else {
    row = min(n0 + lr, a.N - 1) - n0;
  }
  const uint32_t wrows = SWI ? (uint32_t)a.N : (uint32_t)min(32, a.N - n0);
  const uint8_t* wqb = SWI ? it.wq : it.wq + (size_t)n0 * wrow_bytes;
  const uint16_t* scb = SWI ? it.sc : it.sc + (size_t)n0 * kblocks;
  const uint32_t woff = (uint32_t)row * wrow_bytes + 16u * lh;
  const uint32_t soff = ((uint32_t)row * kblocks + (uint32_t)(KS * lh)) * 2u;
  // lane half h holds the scales of blocks KS h .. KS h + KS - 1 of a stage: one load where K is whole
  // stages and every such run is naturally aligned (FAST), else one 2-byte load per block
  constexpr int SL = FAST ? SD : KS;
  // two register sets: a stage's weights are loaded all at once, one stage ahead, so the loads that
  // share a row's 128-byte lines follow each other
  uint4 w[2][NW];
  uint32_t s[2][SL];
  // The loads of a stage. Where K is not whole stages, loads past K (a ragged last sub-step, sub-steps
  // past it) carry an out-of-range offset and return zeros; no branch, so the loads in flight can be
  // counted.
  const int klim = (FMT == kQ8) ? K : K - 32 * lh;
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(wqb, wrows * wrow_bytes);
  const __amdgpu_buffer_rsrc_t sr = make_rsrc(scb, wrows * kblocks * 2u);
  auto issue = [&](int st, uint4 (&wv)[NW], uint32_t (&sv)[SL]) {
    if constexpr (FAST && KS == 4) {
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(sr, soff, st * 4 * KS, 0));
      sv[0] = v[0];
      sv[1] = v[1];
    } else if constexpr (FAST) {
      static_assert(KS == 2 || KS == 4, "two or four K sub-steps per stage");
      sv[0] = __builtin_amdgcn_raw_buffer_load_b32(sr, soff, st * 4 * KS, 0);
    } else {
      const int blk = st * 2 * KS + KS * lh;             // first block of this lane
#pragma unroll
      for (int j = 0; j < KS; ++j)
        sv[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(
            sr, blk + j < (int)kblocks ? soff + (uint32_t)(st * 4 * KS) + 2u * j : kOOB, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int ks = st * KS + i / WL, j = i % WL;
      if constexpr (FAST) {
        wv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wr, woff, ks * kStepBytes + 32 * j, 0));
      } else {
        const bool live = ks * kBK + ((FMT == kQ8) ? 32 * j : 0) < klim;
        wv[i] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(wr, live ? woff + (uint32_t)(ks * kStepBytes + 32 * j) : kOOB, 0, 0));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // --- activation rows: DMA of 8-row groups (1 KiB per K sub-step), group j by wave j % WV ---
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, (uint32_t)a.T * (uint32_t)K * 2u);
  constexpr int XG = (NB * 4 + WV - 1) / WV;
  uint32_t xoff[XG];
  int dma_c[XG];
#pragma unroll
  for (int i = 0; i < XG; ++i) {
    const int r = (wave + WV * i) * 8 + (lane >> 3);
    dma_c[i] = (lane & 7) ^ row_swizzle(r);
    int asg = r < it.rows ? a.perm[it.pbeg + r] : -1;
    if (asg >= a.M) asg = -1;
    // a missing row's offset stays past the buffer whatever K offset is added to it
    xoff[i] = asg >= 0 ? (uint32_t)(asg / a.topk) * (uint32_t)K * 2u + 16u * (uint32_t)dma_c[i]
                       : kOOB - 2u * (uint32_t)K - 2u * (uint32_t)kRowBytes;
  }
  auto issue_x = [&](int st, lds_char* dst) {
#pragma unroll
    for (int i = 0; i < XG; ++i) {
      const int g = wave + WV * i;
      if (g * 8 >= it.rows) break;
#pragma unroll
      for (int kt = 0; kt < KS; ++kt) {
        const int ks = st * KS + kt;
        lds_char* d = dst + kt * kSubBytes + g * 1024;
        if constexpr (FAST) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (__attribute__((address_space(3))) void*)d, 16, xoff[i],
                                                   ks * kRowBytes, 0, 0);
        } else {
          if (ks >= nk) break;
          const uint32_t o = ks * kBK + dma_c[i] * 8 < K ? xoff[i] + (uint32_t)(ks * kRowBytes) : kOOB;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (__attribute__((address_space(3))) void*)d, 16, o, 0, 0, 0);
        }
      }
    }
  };

  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = f32x16{};
  const int rsw = row_swizzle(lr);
  auto swap2 = [](uint32_t& u, uint32_t& v) {
    const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
    u = r[0];
    v = r[1];
  };

  // one stage over the activations in xs; MORE: not the last one, so K fills it
  auto step = [&](auto more, int st, const lds_char* xs, const uint4 (&wv)[NW], const uint32_t (&sv)[SL]) {
    constexpr bool MORE = decltype(more)::value;
    // every lane gets all 2 KS block scales of its row
    uint32_t sp[2][SD];
#pragma unroll
    for (int j = 0; j < SD; ++j) {
      const uint32_t v = FAST ? sv[j] : (sv[2 * j] & 0xFFFFu) | (sv[2 * j + 1] << 16);
      sp[0][j] = v;
      sp[1][j] = v;
      swap2(sp[0][j], sp[1][j]);
    }
#pragma unroll
    for (int kt = 0; kt < KS; ++kt) {
      if (!FAST && !MORE && st * KS + kt >= nk) break;
      const lds_char* xt = xs + kt * kSubBytes + lr * kRowBytes;
      bf16x8 xv[4][NB];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          xv[kk][b] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(
              xt + b * (32 * kRowBytes) + (((kk * 2 + lh) ^ rsw) << 4));
      // the two lane halves hold neighbouring 16-byte pieces of a row; K sub-step kk of the MFMA
      // needs elements 16 kk + 8 h .. + 7 in half h
      uint32_t d[4][WL];
      if constexpr (FMT == kQ8) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint4 v = wv[kt * 2 + j];
          d[2 * j][0] = v.x;
          d[2 * j + 1][0] = v.z;
          d[2 * j][1] = v.y;
          d[2 * j + 1][1] = v.w;
          swap2(d[2 * j][0], d[2 * j + 1][0]);
          swap2(d[2 * j][1], d[2 * j + 1][1]);
        }
      } else {
        const uint4 v = wv[kt];
        d[0][0] = v.x;
        d[2][0] = v.y;
        d[1][0] = v.z;
        d[3][0] = v.w;
        swap2(d[0][0], d[2][0]);
        swap2(d[1][0], d[3][0]);
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const int blk = 2 * kt + (kk >> 1);
        const uint32_t pair = sp[blk / KS][(blk % KS) >> 1];
        const float sf = fp16_to_f32((uint16_t)((blk % KS) & 1 ? pair >> 16 : pair));
        u32x4 u;
        if constexpr (FMT == kQ8) {
          u = dequant_q8_unit(d[kk][0], d[kk][1], sf);
        } else {
          float s24, s20, off;
          q4_factors(sf, s24, s20, off);
          u = dequant_q4_unit(d[kk][0], s24, s20, off);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u), xv[kk][b], acc[b], 0, 0, 0);
      }
    }
  };

  // weights first: the activation rows wait for perm
  issue(0, w[0], s[0]);
  issue_x(0, x0);
  wait_vmcnt_lgkm0<0>();
  // Each stage is entered through a barrier once its activation DMA has landed; only the NW + 1
  // (or more) weight and scale loads issued after that DMA may still be in flight. The general form's last
  // stage uses its weights behind run-time breaks, where their loads could be sunk to, so that fewer
  // follow the DMA than the count allows for: it is entered with nothing in flight.
  int st = 0;
  auto pair = [&](auto last) {       // stages st (of x0) and st + 1 (of x1)
    __builtin_amdgcn_s_barrier();
    issue_x(st + 1, x1);
    __builtin_amdgcn_sched_barrier(0);
    issue(st + 1, w[1], s[1]);
    step(std::true_type{}, st, x0, w[0], s[0]);
    wait_vmcnt_lgkm0<!FAST && decltype(last)::value ? 0 : NW + 1>();
    __builtin_amdgcn_s_barrier();
    if constexpr (decltype(last)::value) {
      step(std::false_type{}, st + 1, x1, w[1], s[1]);
    } else {
      issue_x(st + 2, x0);
      __builtin_amdgcn_sched_barrier(0);
      issue(st + 2, w[0], s[0]);
      step(std::true_type{}, st + 1, x1, w[1], s[1]);
      wait_vmcnt_lgkm0<NW + 1>();
    }
  };
  for (; st + 2 < nst; st += 2) pair(std::false_type{});
  if (st + 2 == nst) {
    pair(std::true_type{});
  } else {
    if constexpr (!FAST) wait_vmcnt_lgkm0<0>();
    __builtin_amdgcn_s_barrier();
    step(std::false_type{}, st, x0, w[0], s[0]);
  }

  // --- epilogue: lane (token lr of block b, half h) ---
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int r = 32 * b + lr;
    const int dst = r < it.rows ? a.perm[it.pbeg + r] : -1;
    if (!store || dst < 0 || dst >= a.M) continue;
    if constexpr (SWI) {
      const int hc = n0 + 8 * lh;
      uint16_t* hrow = a.h + (size_t)dst * a.swi_inter + hc;
      uint32_t o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = pack_bf16x2(swiglu_f32(acc[b][2 * i], acc[b][8 + 2 * i]),
                           swiglu_f32(acc[b][2 * i + 1], acc[b][9 + 2 * i]));
      if ((a.swi_inter & 7) == 0) {
        if (hc < a.swi_inter) *reinterpret_cast<uint4*>(hrow) = make_uint4(o[0], o[1], o[2], o[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (hc + i < a.swi_inter) hrow[i] = (uint16_t)(o[i >> 1] >> (16 * (i & 1)));
      }
    } else {
      float* yrow = a.y + (size_t)dst * a.N;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + 8 * q + 4 * lh;
        if ((a.N & 3) == 0) {
          if (n < a.N)
            *reinterpret_cast<f32x4*>(yrow + n) =
                f32x4{acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]};
        } else {
#pragma unroll
          for (int p = 0; p < 4; ++p)
            if (n + p < a.N) yrow[n + p] = acc[b][4 * q + p];
        }
      }
    }
  }
}

template <int FMT, int RB, int KS, int WV, bool SWI, int WPE>
__global__ __launch_bounds__(WV * 64, WPE) void moe_direct_kernel(TileArgs a, ExpertPtrs ep) {
  __shared__ __attribute__((aligned(1024))) char lx0[KS * RB * 32 * kRowBytes];
  __shared__ __attribute__((aligned(1024))) char lx1[KS * RB * 32 * kRowBytes];
  const int cols = SWI ? a.swi_inter : a.N;                 // output columns
  constexpr int CW = SWI ? 16 : 32;                          // per wave
  const int nt_n = (cols + CW * WV - 1) / (CW * WV);
  const DirItem it = dir_item<RB * 32>(a, ep, nt_n);
  if (it.rows <= 0) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a wave past the last column repeats the last wave's work (it takes part in the DMA and the
  // barriers) and stores nothing
  const int col = (it.nt * WV + wave) * CW;
  const bool store = col < cols;
  const int n0 = store ? col : (cols - 1) / CW * CW;
  const int nb = (it.rows + 31) >> 5;
  lds_char* x0 = (lds_char*)lx0;
  lds_char* x1 = (lds_char*)lx1;
  // whole stages, and scale runs of KS blocks naturally aligned in every row
  const bool fast = a.K % (KS * kBK) == 0 && (reinterpret_cast<uintptr_t>(it.sc) & (2 * KS - 1)) == 0;
  auto run_nb = [&](auto w) {
    constexpr bool W = decltype(w)::value;
    if constexpr (RB >= 4) {
      if (nb == 4) return dir_body<FMT, RB, 4, KS, WV, SWI, W>(a, it, n0, store, x0, x1);
      if (nb == 3) return dir_body<FMT, RB, 3, KS, WV, SWI, W>(a, it, n0, store, x0, x1);
    }
    if constexpr (RB >= 2) {
      if (nb == 2) return dir_body<FMT, RB, 2, KS, WV, SWI, W>(a, it, n0, store, x0, x1);
    }
    dir_body<FMT, RB, 1, KS, WV, SWI, W>(a, it, n0, store, x0, x1);
  };
  if (fast) run_nb(std::true_type{}); else run_nb(std::false_type{});
}

}  // namespace qg
