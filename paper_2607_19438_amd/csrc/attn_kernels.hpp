// Prefill flash attention for gfx950 (Section 3.1, prefill attention item): the score product
// and the output product run on the matrix cores, with an exact online softmax (running row
// maximum, rescaling of the running output) between them.
//
// A workgroup (4 waves) owns 128 query rows of one (batch, query head); wave w owns rows
// 32w..32w+31. Keys and values stream through LDS in blocks of 64 (double-buffered, the next
// block's global loads in flight during the current block's math). Per block and wave:
//   S^T = K Q^T   (v_mfma_f32_32x32x16_bf16: keys as the A rows from LDS, the wave's queries as
//                  the B columns, held in registers for the whole loop) -- so each lane owns one
//                  query and 32 of the block's keys, and a row maximum needs one lane exchange;
//   online softmax on the scores in registers (exp2 with the scale folded into log2 e);
//   O^T += V^T P^T (the same MFMA: V^T read from the row-major value block with gfx950's
//                  transposing LDS read, P^T straight from the score registers rounded to bf16
//                  -- the score layout is the B-operand layout once the MFMA's 16-element K order
//                  is chosen to match it).
// Keys and values both go from HBM to LDS by DMA, with no register staging.
// Rows are normalised by the running sum at the end and stored as bf16. Causal blocks above the
// diagonal are skipped; blocks on it are masked key by key.
//
// SPLIT (few workgroups): the workgroup owns 64 query rows, and wave w takes rows 32 (w % 2) .. + 31
// against the (w / 2)-th 32 keys of every block, so a query's keys are shared by two waves, each with its
// own maximum, sum and output, merged through LDS at the end. With few workgroups the call lasts as long
// as the chain of key blocks of its last query rows, walked by one wave per SIMD (0.69 blocks/us alone,
// 0.95 for two waves together); the split halves the chain and doubles the workgroups, at more DMA, LDS
// and barrier work per MFMA. Measured (unsplit -> split, us): causal 512 x 32/8 heads D=128 14.6 -> 11.1,
// 4 x 300 x 8/8 10.4 -> 8.5, 3 x 700 x 32/8 D=64 18.3 -> 15.3, 2048 x 32/4 D=128 48.1 -> 46.8, 4096 x 32/4
// 142 -> 155; not causal 2 x 1000 x 16/4 D=64 15.8 -> 14.8, 2048 x 32/4 D=128 66.8 -> 77.0.
#pragma once

#include "qgemm_kernels.hpp"

namespace qg {

constexpr int kAttnThreads = 256;   // four waves
constexpr int kAttnBK = 64;         // keys per block
template <bool SPLIT>
constexpr int kAttnBQ = SPLIT ? 64 : 128;   // query rows per workgroup

struct AttnArgs {
  const uint16_t* q;   // bf16 [B][S][H][D]
  const uint16_t* k;   // bf16 [B][S][Hkv][D]
  const uint16_t* v;   // bf16 [B][S][Hkv][D]
  uint16_t* o;         // bf16 [B][S][H][D]
  int B;
  int S;
  int H;
  int Hkv;
  float sl2;           // softmax scale * log2(e)
};

// The kernel body lives in a device function (the kernel below only forwards to it): its
// scheduling builtins exist for the GPU target only, and a kernel template's host-side stub is
// not emitted when its own body uses them.
// The value of lane l ^ 32 (the other MFMA lane half of the same query), with one VALU lane swap.
__device__ __forceinline__ float other_half(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // {x[l % 32], x[32 + l % 32]}
  const int lane = (int)(threadIdx.x & 63);
  return __builtin_bit_cast(float, (unsigned)(lane < 32 ? r[1] : r[0]));
}

template <int D, bool CAUSAL, bool SPLIT>
__device__ __forceinline__ void attn_body(const AttnArgs& a) {
  static_assert(D == 64 || D == 128, "head dimension 64 or 128");
  constexpr int BQ = kAttnBQ<SPLIT>;
  constexpr int NT = SPLIT ? 1 : 2;           // 32-key tiles of a block per wave
  constexpr int KCH = D / 8;                  // 16-byte chunks per key row
  constexpr int KSTEPS = D / 16;              // K16 steps of the score product
  constexpr int DT = D / 32;                  // 32-row tiles of O^T
  constexpr int KROWS_DMA = 1024 / (2 * D);   // key rows per 1 KiB DMA instruction
  constexpr int KDMA = kAttnBK / KROWS_DMA / 4;                 // key DMA instructions per wave
  // one __shared__ array per buffer, so the compiler can tell the key DMA into one buffer from
  // the LDS reads of the other and leaves the DMA in flight across them
  __shared__ __attribute__((aligned(16))) uint16_t ks0[kAttnBK * D];
  __shared__ __attribute__((aligned(16))) uint16_t ks1[kAttnBK * D];
  __shared__ __attribute__((aligned(16))) uint16_t vt0[kAttnBK * D];
  __shared__ __attribute__((aligned(16))) uint16_t vt1[kAttnBK * D];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31;     // this lane's query within the wave (MFMA column)
  const int hh = lane >> 5;      // MFMA lane half
  const int S = a.S, H = a.H;
  const int nqb = (S + BQ - 1) / BQ;
  int bh, qb;
  if (CAUSAL && SPLIT) {
    // the heaviest query blocks of all heads first, so that light ones fill in. Workgroups reach the 8
    // XCDs round-robin: with a multiple of 8 heads each XCD takes consecutive ones, which share keys and
    // values in its L2
    const int nbh = a.B * H;
    const int L = (int)blockIdx.x;
    qb = nqb - 1 - L / nbh;
    const int i = L - (nqb - 1 - qb) * nbh;
    bh = (nbh & 7) == 0 ? (i & 7) * (nbh >> 3) + (i >> 3) : i;
  } else if (CAUSAL) {
    // heavy members (query blocks nqb-1 .. nqb-ceil(nqb/2)) of all heads first, then the light
    // members in the same order: workgroups L and L + (heavy count) are complementary
    const int hi = (nqb + 1) >> 1;
    const int lo = nqb >> 1;
    const int nh = a.B * H * hi;
    const int L = (int)blockIdx.x;
    if (L < nh) {
      bh = L / hi;
      qb = nqb - 1 - (L - bh * hi);
    } else {
      const int J = L - nh;
      bh = J / lo;
      qb = J - bh * lo;
    }
  } else {
    const int item = xcd_tile((int)blockIdx.x, a.B * H * nqb);
    bh = item / nqb;
    qb = item - bh * nqb;
  }
  const int b = bh / H;
  const int h = bh - b * H;
  const int g = h / (H / a.Hkv);
  const int q0 = qb * BQ;
  const int kh = SPLIT ? wave >> 1 : 0;       // first 32-key tile of a block
  const int qs = q0 + (SPLIT ? wave & 1 : wave) * 32;   // the wave's first query position
  const int qrow = qs + col;                  // this lane's query position

  const size_t qstride = (size_t)H * D;       // elements between consecutive tokens of q / o
  const size_t kstride = (size_t)a.Hkv * D;
  const __amdgpu_buffer_rsrc_t qr = make_rsrc(a.q + (size_t)b * S * qstride + (size_t)h * D,
                                              (uint32_t)(((size_t)(S - 1) * qstride + D) * 2));
  const __amdgpu_buffer_rsrc_t kr = make_rsrc(a.k + (size_t)b * S * kstride + (size_t)g * D,
                                              (uint32_t)(((size_t)(S - 1) * kstride + D) * 2));
  const __amdgpu_buffer_rsrc_t vr = make_rsrc(a.v + (size_t)b * S * kstride + (size_t)g * D,
                                              (uint32_t)(((size_t)(S - 1) * kstride + D) * 2));

  // query fragments (B operand of K Q^T): step t needs q[qrow][16t + 8hh .. +8]
  bf16x8 qf[KSTEPS];
#pragma unroll
  for (int t = 0; t < KSTEPS; ++t) {
    const uint32_t off = qrow < S ? ((uint32_t)qrow * (uint32_t)qstride + 16u * t + 8u * hh) * 2u : kOOB;
    qf[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(qr, off, 0, 0));
  }

  // 16-byte chunk swizzle of a key row in LDS: any 16 consecutive keys read at one logical chunk
  // hit 16 distinct bank groups, and any 8 hit 8 distinct 16-byte groups of a 128-byte bank
  // window (rows are 256 bytes at D = 128; at D = 64 the rows are 128 bytes, the layout of the
  // GEMM tiles, and take their row swizzle)
  auto kswz = [](int key) { return (D == 128) ? (key & 15) : row_swizzle(key); };
  // keys: DMA straight into LDS; lane L of a 1 KiB instruction fills physical chunk L % KCH of
  // key row L / KCH, so it fetches the logical chunk that the swizzle puts there
  const int dkey = lane / KCH;
  // per-lane byte offsets within a block (key row krow + dkey of the block; rows at or past S lie
  // beyond the end of the buffer range and read as zeros, so no per-block test is needed)
  uint32_t kdma_off[KDMA];
#pragma unroll
  for (int i = 0; i < KDMA; ++i) {
    const int krow = (wave * KDMA + i) * KROWS_DMA;
    kdma_off[i] = ((uint32_t)(krow + dkey) * (uint32_t)kstride + 8u * (uint32_t)((lane % KCH) ^ kswz(krow + dkey))) * 2u;
  }
  const uint32_t kblock_bytes = (uint32_t)kAttnBK * (uint32_t)kstride * 2u;   // one key block
  auto dma_keys = [&](uint16_t* ks, int jb) {
    const uint32_t base = (uint32_t)jb * kblock_bytes;
#pragma unroll
    for (int i = 0; i < KDMA; ++i) {
      const int krow = (wave * KDMA + i) * KROWS_DMA;          // first key row of this instruction
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (__attribute__((address_space(3))) void*)(ks + krow * D), 16,
                                               kdma_off[i] + base, 0, 0, 0);
    }
  };
  // values: DMA straight into LDS too, row-major (key rows), 16-byte chunks XOR-swizzled by
  // vswz(key); the output product reads them with the transposing LDS read, which hands each
  // lane 4 keys of one dimension. The swizzle puts the 4 consecutive keys x 64 bytes that the
  // 32 lanes of one half-wave read on 256 distinct bytes of the bank space.
  auto vswz = [](int key) { return (D == 128) ? 4 * (key & 3) : 4 * ((key >> 1) & 1); };
  uint32_t vdma_off[KDMA];
#pragma unroll
  for (int i = 0; i < KDMA; ++i) {
    const int krow = (wave * KDMA + i) * KROWS_DMA;
    vdma_off[i] = ((uint32_t)(krow + dkey) * (uint32_t)kstride + 8u * (uint32_t)((lane % KCH) ^ vswz(krow + dkey))) * 2u;
  }
  auto dma_values = [&](uint16_t* vs, int jb) {
    const uint32_t base = (uint32_t)jb * kblock_bytes;
#pragma unroll
    for (int i = 0; i < KDMA; ++i) {
      const int krow = (wave * KDMA + i) * KROWS_DMA;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (__attribute__((address_space(3))) void*)(vs + krow * D), 16,
                                               vdma_off[i] + base, 0, 0, 0);
    }
  };

  int nkb = (S + kAttnBK - 1) / kAttnBK;
  if (CAUSAL) nkb = min(nkb, (q0 + BQ - 1) / kAttnBK + 1);

  f32x16 acc_o[DT];
#pragma unroll
  for (int i = 0; i < DT; ++i) acc_o[i] = f32x16{};
  float m_run = -__builtin_inff();   // running maximum of the raw scores q.k
  float l_run = 0.0f;
  const float sl2 = a.sl2;

  dma_keys(ks0, 0);
  dma_values(vt0, 0);
  wait_vmcnt_lgkm0<0>();
  __syncthreads();

  // LDS fragment reads: key rows (A operand of K Q^T) and transposed values (A operand of V^T P^T)
  auto rd_k = [&](const uint16_t* ksc, int t, int kt) {
    const int key = kt * 32 + col;
    const int c = 2 * t + hh;
    return *reinterpret_cast<const bf16x8*>(&ksc[key * D + ((c ^ kswz(key)) << 3)]);
  };
  // V^T fragment of MFMA step u, tile dt: lane (d = col, hh) needs the keys 16u + 4hh + {0..3}
  // and 16u + 8 + 4hh + {0..3} of dimension 32dt + col. In a transposing read each 16-lane group
  // returns, to lane i, element i % 4 of the 8-byte pieces that lanes 4r + i/4 (r = 0..3) point
  // at; so lane s of the group points at key (run start + s/4), dimensions 4(s%4)..+3 of the
  // group's 16, and lane i gets the run's 4 keys of dimension (group's first) + i.
  const int trk = (lane & 15) >> 2;                   // key within the run of 4
  const int trd = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);   // first of the 4 dims this lane points at
  auto rd_v = [&](const uint16_t* vtc, int u, int dt) {
    uint32_t w[4];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int key = 16 * u + 8 * half + 4 * hh + trk;
      const int dim = 32 * dt + trd;
      const int e = key * D + (((dim >> 3) ^ vswz(key)) << 3) + (dim & 7);
      typedef short v4i16 __attribute__((ext_vector_type(4)));
      const v4i16 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) v4i16*)(const_cast<uint16_t*>(vtc) + e));
      const uint2 rr = __builtin_bit_cast(uint2, r);
      w[2 * half] = rr.x;
      w[2 * half + 1] = rr.y;
    }
    return __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
  };

  // one key block: math on buffer (ksc, vtc) while the next block's keys stream into (ksn, vtn)
  auto step = [&](int jb, const uint16_t* ksc, const uint16_t* vtc, uint16_t* ksn, uint16_t* vtn) {
    const int j0 = jb * kAttnBK;
    const bool more = jb + 1 < nkb;
    if (more) {
      dma_keys(ksn, jb + 1);
      dma_values(vtn, jb + 1);
    }
    const int t0 = j0 + 32 * kh;            // the wave's first key of the block
    // (tiles and waves' queries both start at multiples of 32, so every query of a wave sees at least the
    // first key of a block that is not skipped)
    if ((!SPLIT || t0 < S) && (!CAUSAL || t0 <= qs + 31)) {
      // scores S^T[key][query] for the wave's keys of the block: two accumulators, one per 32-key tile
      // (SPLIT: even and odd K16 steps), so that no MFMA waits for the one before; the key fragments of
      // step t+2 are read from LDS while the MFMAs of step t run
      f32x16 sc[2] = {f32x16{}, f32x16{}};
      bf16x8 kf[3][NT];
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        kf[0][c] = rd_k(ksc, 0, kh + c);
        kf[1][c] = rd_k(ksc, 1, kh + c);
      }
      // raised wave priority while a wave issues its MFMAs: the SIMD's other wave fills the
      // issue slots between them with its softmax VALU work
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int t = 0; t < KSTEPS; ++t) {
#pragma unroll
        for (int c = 0; c < NT; ++c)
          if (t + 2 < KSTEPS) kf[(t + 2) % 3][c] = rd_k(ksc, t + 2, kh + c);
#pragma unroll
        for (int c = 0; c < NT; ++c) {
          f32x16& d = sc[SPLIT ? t & 1 : c];
          d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t % 3][c], qf[t], d, 0, 0, 0);
        }
        if (t + 2 < KSTEPS) QG_SG(kSchedDSRead, NT);
        QG_SG(kSchedMFMA, NT);
      }
      __builtin_amdgcn_s_setprio(0);
      if (SPLIT) sc[0] += sc[1];
      // key of register r in tile kt: t0 + kt*32 + (r/4)*8 + 4hh + r%4
      const bool need_mask = (CAUSAL && t0 + 32 * NT - 1 > qs) || t0 + 32 * NT > S;
      if (need_mask) {
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int kp = t0 + kt * 32 + (r >> 2) * 8 + 4 * hh + (r & 3);
            if (kp >= S || (CAUSAL && kp > qrow)) sc[kt][r] = -__builtin_inff();
          }
      }
      float mloc = -__builtin_inff();
#pragma unroll
      for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, sc[kt][r]);
      mloc = fmaxf(mloc, other_half(mloc));
      const float m_new = fmaxf(m_run, mloc);
      // The reference maximum m_run moves (and the running output and sum are rescaled, before
      // any of this block's output-product MFMAs) only when the block's maximum exceeds it by
      // more than 8 in exp2 units. Softmax does not depend on the reference as long as the
      // weights and their sum use the same one, and the threshold keeps every weight <= 2^8,
      // far inside fp32 and bf16 range; most blocks skip the rescale. (The first block always
      // moves it from -inf, with alpha = 0 on the empty sum.)
      if ((m_new - m_run) * sl2 > 8.0f) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sl2);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < DT; ++i) acc_o[i] *= alpha;
        m_run = m_new;
      }
      // p = exp2((s - m) * scale * log2 e), one fused multiply-add per score; P^T as packed bf16,
      // per key tile: registers (2i, 2i+1). The second half's exponentials (SPLIT: of the tile's
      // registers, else tile 1's) are written between the first output-product MFMAs so the two overlap.
      // SPLIT: a half whose keys so far all score -inf (keys with infinities) keeps maximum -inf, weights 0
      const float ms = (SPLIT && m_run == -__builtin_inff()) ? 0.0f : m_run * sl2;
      float lsum = 0.0f;
      uint32_t pf[NT][8];
      auto exp_half = [&](int second) {
#pragma unroll
        for (int i = 0; i < 8 * NT; i += 2) {
          const int kt = SPLIT ? 0 : second;
          const int r = SPLIT ? 8 * second + i : i;
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kt][r], sl2, -ms));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kt][r + 1], sl2, -ms));
          lsum += p0 + p1;
          pf[kt][r >> 1] = pack_bf16x2(p0, p1);
        }
      };
      exp_half(0);
      // O^T += V^T P^T: K16 step u covers the wave's keys 16u..16u+15; lane half hh supplies the keys
      // 16u + 4hh + {0..3} and 16u + 8 + 4hh + {0..3} (its score registers 8(u%2)..8(u%2)+7).
      // The value fragments of step u+1 are read from LDS while the MFMAs of step u run.
      bf16x8 vf[2][DT];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vf[0][dt] = rd_v(vtc, 2 * kh, dt);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int u = 0; u < 2 * NT; ++u) {
        if (u + 1 < 2 * NT) {
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) vf[(u + 1) & 1][dt] = rd_v(vtc, 2 * kh + u + 1, dt);
        }
        const int kt = u >> 1;
        const int r0 = (u & 1) * 4;
        const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pf[kt][r0], pf[kt][r0 + 1], pf[kt][r0 + 2], pf[kt][r0 + 3]});
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          acc_o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u & 1][dt], pb, acc_o[dt], 0, 0, 0);
        if (u == 0) exp_half(1);
      }
      __builtin_amdgcn_s_setprio(0);
      l_run += lsum;
    }

    wait_vmcnt_lgkm0<0>();   // the key and value DMA of the next block are in LDS
    __syncthreads();
  };

  for (int jb = 0; jb < nkb; jb += 2) {
    step(jb, ks0, vt0, ks1, vt1);
    if (jb + 1 < nkb) step(jb + 1, ks1, vt1, ks0, vt0);
  }

  if constexpr (SPLIT) {
    // Merge the two waves of the same queries: the second half's output, maximum and sum go through the
    // key and value buffers (the loop ends with a barrier), lane by lane. A wave that skipped every
    // tile has maximum -inf and takes weight 0; the first half always holds key 0.
    typedef __attribute__((address_space(3))) float lds_float;
    lds_float* mo = (lds_float*)((wave & 1) ? (lds_char*)ks1 : (lds_char*)ks0);
    lds_float* ml = (lds_float*)((wave & 1) ? (lds_char*)vt1 : (lds_char*)vt0);
    if (kh == 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4)
          *(__attribute__((address_space(3))) f32x4*)(mo + ((dt * 4 + a4) * 64 + lane) * 4) =
              f32x4{acc_o[dt][4 * a4], acc_o[dt][4 * a4 + 1], acc_o[dt][4 * a4 + 2], acc_o[dt][4 * a4 + 3]};
      ml[lane] = m_run;
      ml[64 + lane] = l_run;
    }
    __syncthreads();
    if (kh == 1) return;
    const float m1 = ml[lane];
    const float mm = fmaxf(m_run, m1);
    const float w0 = __builtin_amdgcn_exp2f((m_run - mm) * sl2);
    const float w1 = __builtin_amdgcn_exp2f((m1 - mm) * sl2);
    l_run = l_run * w0 + ml[64 + lane] * w1;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int a4 = 0; a4 < 4; ++a4) {
        const f32x4 o1 = *(const __attribute__((address_space(3))) f32x4*)(mo + ((dt * 4 + a4) * 64 + lane) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc_o[dt][4 * a4 + r] = acc_o[dt][4 * a4 + r] * w0 + o1[r] * w1;
      }
  }

  // normalise and store: lane (col, hh) holds o[qrow][dt*32 + 8a + 4hh + {0..3}] in acc_o[dt][4a..4a+3]
  const float l_tot = l_run + other_half(l_run);
  const float inv = 1.0f / l_tot;
  if (qrow < S) {
    uint16_t* orow = a.o + ((size_t)b * S + qrow) * qstride + (size_t)h * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int a4 = 0; a4 < 4; ++a4) {
        const uint32_t lo = pack_bf16x2(acc_o[dt][4 * a4] * inv, acc_o[dt][4 * a4 + 1] * inv);
        const uint32_t hi = pack_bf16x2(acc_o[dt][4 * a4 + 2] * inv, acc_o[dt][4 * a4 + 3] * inv);
        *reinterpret_cast<uint2*>(orow + dt * 32 + 8 * a4 + 4 * hh) = make_uint2(lo, hi);
      }
    }
  }
}

template <int D, bool CAUSAL, bool SPLIT>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_fwd_kernel(AttnArgs a) {
  attn_body<D, CAUSAL, SPLIT>(a);
}

}  // namespace qg
