// Fused reconstruct-then-attend decode kernel for an fp32 cache (gfx950).
//
// Same plan as the bf16 kernel (256 tokens x 256 predicted columns per
// workgroup, K pass with W as the row operand, V pass with X as the row
// operand), but four waves of 128 x 128, and the predictor product (Eq. 3) runs on
// v_mfma_f32_32x32x2f32: true fp32 products and fp32 accumulation, as the 1e-5
// tolerance of the fp32 configuration needs.  Its accumulators are blocks of 32 x 32 where the bf16
// kernel's are 16 x 16, so the attention epilogues are its own.  An fp32 MFMA operand is ONE value per lane (row or
// column = lane % 32, k = lane / 32), so both tiles are read from LDS in their
// natural layouts with scalar reads and W needs no transposition.  The main
// loop is single-buffered and synchronous: it serves the fp32 problems that are too large
// for fused_decode_small.h.
#pragma once
#include "common.h"
#include "fused_decode.h"

namespace echokv {
namespace fused32 {

using fused::BM; using fused::BN;
constexpr int NTHREADS = 256, WM = 128, WN = 128;      // 2 x 2 waves of 128 x 128
constexpr int BK = 16;            // input dims per tile
constexpr int XP = BK + 1;        // padded row pitch of the X tile (floats): conflict-free column reads

// The epilogues take accumulators of NTB blocks of 32 tokens x 4 blocks of 32 columns (whole heads).
//
// Keeps the 256 accumulators in the accumulation registers for the duration of an epilogue loop
// body: without it the compiler copies all of them to ordinary registers ahead of the loop over
// query heads and spills whatever else is live.
template <int I, int J>
__device__ __forceinline__ void pin_acc(floatx16_t (&acc)[I][J]) {
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// Softmax numerators of one (head, query head) pair from the lane-partial scores s
// (token tb * 32 + lane % 32 of the wave; the two lane halves hold the two halves of the head dims).
template <int NTB>
__device__ __forceinline__ void score_tail(float (&s)[NTB], float* pp, float* ml, int lane, int jw0, const fused::KExtra& x) {
  const int lr = lane & 31, lh = lane >> 5;
  float mx = -INFINITY;
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) {
    s[tb] += __shfl_xor(s[tb], 32, 64);
    const int tok = jw0 + tb * 32 + lr;
    if (tok < x.lo || tok >= x.hi) s[tb] = -INFINITY;
    mx = fmaxf(mx, s[tb]);
  }
  mx = wave_max(mx, 32);
  float sum = 0.f;
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) {
    const float p = (s[tb] == -INFINITY) ? 0.f : __expf(s[tb] - mx);
    sum += p;
    if (lh == 0) pp[tb * 32 + lr] = p;
  }
  sum = wave_sum(sum, 32);
  if (lane == 0) { ml[0] = mx; ml[1] = sum; }
}

// After the K pass: acc[cb][tb] holds K_hat^T (rows = head dims of the wave's 128 columns, lanes =
// tokens).  `tail(s, hw, g)` receives the lane-partial scores (Eq. 7) of head hw of the wave's tile and
// query head g of its group (token tb * 32 + lane % 32; add the other lane half for the total).
// qw: the queries of the wave's first head; jw0: its first token.
template <int HD, bool ROPE, int NTB, class Tail>
__device__ __forceinline__ void k_scores(floatx16_t (&acc)[4][NTB], const float* qw, int G,
                                         int lane, int jw0, int L, const fused::KExtra& x, Tail tail) {
  constexpr int HPW = 128 / HD, CBH = HD / 32;
  const int lr = lane & 31, lh = lane >> 5;
  if constexpr (!ROPE) {
#pragma unroll
    for (int hw = 0; hw < HPW; ++hw) {
      for (int g = 0; g < G; ++g) {
        pin_acc(acc);
        const float* qs = qw + (hw * G + g) * HD;
        float s[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) s[tb] = 0.f;
#pragma unroll
        for (int cb = 0; cb < CBH; ++cb) {
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const float4 qv = *reinterpret_cast<const float4*>(qs + cb * 32 + r4 * 8 + lh * 4);
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) {
              const floatx16_t& c = acc[hw * CBH + cb][tb];
              s[tb] = fmaf(qv.x, c[r4 * 4 + 0], s[tb]);
              s[tb] = fmaf(qv.y, c[r4 * 4 + 1], s[tb]);
              s[tb] = fmaf(qv.z, c[r4 * 4 + 2], s[tb]);
              s[tb] = fmaf(qv.w, c[r4 * 4 + 3], s[tb]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        tail(s, hw, g);
      }
    }
  } else {
    // Rotary embedding of the rebuilt key at its token's position, folded into the dot
    // product: feature c pairs with c + HD/2, which this lane holds HD/64 column blocks
    // further on.  With a = k_c, b = k_{c+HD/2}:
    //   q_c (a cos - b sin) + q_{c+HD/2} (b cos + a sin)
    //     = cos (a q_c + b q_{c+HD/2}) + sin (a q_{c+HD/2} - b q_c)
    // The accumulators are only read.  Masked tokens borrow the last valid table row.  The
    // table values and the accumulator reads of a (token block, column block) are shared by
    // the query heads of the group: the loop over them is innermost, unrolled to the
    // largest group size with a uniform skip.
    constexpr int HB = CBH / 2;
#pragma unroll
    for (int hw = 0; hw < HPW; ++hw) {
      float s[fused::MAXPAIR][NTB];
#pragma unroll
      for (int g = 0; g < fused::MAXPAIR; ++g)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) s[g][tb] = 0.f;
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        const int pos = min(jw0 + tb * 32 + lr, L - 1);
        const float* cr = x.cos + (int64_t)pos * (HD / 2) + lh * 4;
        const float* sr = x.sin + (int64_t)pos * (HD / 2) + lh * 4;
#pragma unroll
        for (int cb = 0; cb < HB; ++cb) {
          pin_acc(acc);
          float cc[16], ss[16], ka[16], kb[16];
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const float4 c4 = *reinterpret_cast<const float4*>(cr + cb * 32 + r4 * 8);
            const float4 s4 = *reinterpret_cast<const float4*>(sr + cb * 32 + r4 * 8);
            cc[r4 * 4] = c4.x; cc[r4 * 4 + 1] = c4.y; cc[r4 * 4 + 2] = c4.z; cc[r4 * 4 + 3] = c4.w;
            ss[r4 * 4] = s4.x; ss[r4 * 4 + 1] = s4.y; ss[r4 * 4 + 2] = s4.z; ss[r4 * 4 + 3] = s4.w;
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            ka[r] = acc[hw * CBH + cb][tb][r];
            kb[r] = acc[hw * CBH + cb + HB][tb][r];
          }
#pragma unroll
          for (int g = 0; g < fused::MAXPAIR; ++g) {
            if (g < G) {
              const float* qs = qw + (hw * G + g) * HD;
#pragma unroll
              for (int r4 = 0; r4 < 4; ++r4) {
                const float4 qa = *reinterpret_cast<const float4*>(qs + cb * 32 + r4 * 8 + lh * 4);
                const float4 qb = *reinterpret_cast<const float4*>(qs + (cb + HB) * 32 + r4 * 8 + lh * 4);
                const float q0[4] = {qa.x, qa.y, qa.z, qa.w}, q1[4] = {qb.x, qb.y, qb.z, qb.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const float a = ka[r4 * 4 + i], b = kb[r4 * 4 + i];
                  const float t1 = fmaf(a, q0[i], b * q1[i]);
                  const float t2 = fmaf(a, q1[i], -b * q0[i]);
                  s[g][tb] = fmaf(cc[r4 * 4 + i], t1, fmaf(ss[r4 * 4 + i], t2, s[g][tb]));
                }
              }
            }
          }
          asm volatile("" ::: "memory");       // keep the table loads of later rounds from piling up
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int g = 0; g < fused::MAXPAIR; ++g)
        if (g < G) tail(s[g], hw, g);
    }
  }
}

// After the V pass: acc[tb][cb] holds V_hat (rows = tokens, lanes = head dims).  sum_j p_j v_hat_j of one
// (head, query head) pair over the wave's tokens: dim cb * 32 + lane % 32 in o[cb], both lane halves.
template <int HD, int NTB>
__device__ __forceinline__ void value_sum(floatx16_t (&acc)[NTB][4], const float* pp, int hw, int lane, float (&o)[HD / 32]) {
  constexpr int CBH = HD / 32;
  const int lh = lane >> 5;
#pragma unroll
  for (int cb = 0; cb < CBH; ++cb) o[cb] = 0.f;
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) {
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 pv = *reinterpret_cast<const float4*>(pp + tb * 32 + r4 * 8 + lh * 4);
#pragma unroll
      for (int cb = 0; cb < CBH; ++cb) {
        const floatx16_t& c = acc[tb][hw * CBH + cb];
        o[cb] = fmaf(pv.x, c[r4 * 4 + 0], o[cb]);
        o[cb] = fmaf(pv.y, c[r4 * 4 + 1], o[cb]);
        o[cb] = fmaf(pv.z, c[r4 * 4 + 2], o[cb]);
        o[cb] = fmaf(pv.w, c[r4 * 4 + 3], o[cb]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int cb = 0; cb < CBH; ++cb) o[cb] += __shfl_xor(o[cb], 32, 64);
}

struct Args {
  const float* xa[2]; const float* xr[2]; const float* w[2];
  const float* q;
  float* part_o; float* part_ml;
  int32_t D, m, d_out, H_q, G, n_ret_heads;
  float scale;
  int32_t n_col_tiles, n_tiles;
  const float* rope_cos; const float* rope_sin;     // rotary tables, or null
  int32_t n_sink, n_recent;                         // uncompressed window (0, 0: none)
};

// Queries of the tile's heads -> LDS as fp32, pre-scaled by the softmax scale.
template <int HD, int NT, typename T>
__device__ __forceinline__ void load_queries(float* eq, const T* q, int b, int H_q, int G, int kvh0, float scale, int tid) {
  const int H_kv = H_q / G;
  for (int idx = tid; idx < (BN / HD) * G * HD; idx += NT) {
    const int c = idx % HD, pg = idx / HD;       // pg = head_in_tile * G + g
    const int kvh = kvh0 + pg / G;
    float v = 0.f;
    if (kvh < H_kv) v = Elem<T>::to_f32(q[((int64_t)b * H_q + kvh * G + pg % G) * HD + c]) * scale;
    eq[pg * HD + c] = v;
  }
}

struct EpiSmem {
  float q[fused::BN * fused::MAXPAIR];               // [(head in tile * G + g)][d], pre-scaled
  float p[4][fused::MAXPAIR][WM];                    // per wave and pair: softmax numerators of its tokens
  float ml[4][fused::MAXPAIR][2];                    // per wave and pair: max and sum
};
struct Smem {
  float x[BM * XP];
  float w[BK * BN];
  EpiSmem e;
};

template <bool SWAP>
__device__ __forceinline__ void gemm_pass(floatx16_t (&acc)[4][4], Smem& sm, const Args& a,
                                          const float* xa_tile, const float* xr_tile,
                                          const float* w_tile, int last, int n0, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  const int wt = wave >> 1, wc = wave & 1, lr = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int nk = (a.D + a.m) / BK, nka = a.D / BK;
  for (int kt = 0; kt < nk; ++kt) {
    const bool anchor = kt < nka;
    const float* xb = anchor ? xa_tile + kt * BK : xr_tile + (kt - nka) * BK;
    const int64_t ld = anchor ? a.D : a.m;
    float4 xs[4], ws[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = i * NTHREADS + tid, row = min(idx >> 2, last), c4 = idx & 3;
      xs[i] = *reinterpret_cast<const float4*>(xb + row * ld + c4 * 4);
      const int k = idx >> 6, n4 = idx & 63;
      const int n = min(n0 + n4 * 4, a.d_out - 4) - n0;      // clamp onto the last valid 4 columns
      ws[i] = *reinterpret_cast<const float4*>(w_tile + (int64_t)(kt * BK + k) * a.d_out + n);
    }
    __syncthreads();                      // previous tile fully consumed
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = i * NTHREADS + tid, row = idx >> 2, c4 = idx & 3;
      float* xd = &sm.x[row * XP + c4 * 4];
      xd[0] = xs[i].x; xd[1] = xs[i].y; xd[2] = xs[i].z; xd[3] = xs[i].w;
      const int k = idx >> 6, n4 = idx & 63;
      *reinterpret_cast<float4*>(&sm.w[k * BN + n4 * 4]) = ws[i];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < BK / 2; ++ks) {
      float xf[4], wf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        xf[i] = sm.x[(wt * WM + i * 32 + lr) * XP + ks * 2 + lh];
        wf[i] = sm.w[(ks * 2 + lh) * BN + wc * WN + i * 32 + lr];
      }
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (SWAP) acc[p][r] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[p], xf[r], acc[p][r], 0, 0, 0);
          else acc[p][r] = __builtin_amdgcn_mfma_f32_32x32x2f32(xf[p], wf[r], acc[p][r], 0, 0, 0);
        }
    }
  }
  __syncthreads();
}

template <int HD, bool ROPE>
__global__ __launch_bounds__(NTHREADS) void fused_decode_f32_kernel(Args a, SeqMeta meta) {
  __shared__ Smem sm;
  const int logical = blockIdx.x;
  const int ttile = logical / a.n_col_tiles, ctile = logical % a.n_col_tiles;
  const int b = find_seq(meta.tbase, meta.n, ttile);
  const int L = meta.len[b];
  const int j0 = (ttile - meta.tbase[b]) * BM;
  const int n0 = ctile * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wt = wave >> 1, wc = wave & 1;
  const int last = min(BM, L - j0) - 1;
  const int64_t row0 = meta.start[b] + j0;
  load_queries<HD, NTHREADS>(sm.e.q, a.q, b, a.H_q, a.G, a.n_ret_heads + n0 / HD, a.scale, tid);
  floatx16_t acc[4][4];
  gemm_pass<true>(acc, sm, a, a.xa[0] + row0 * a.D, a.xr[0] + row0 * a.m, a.w[0] + n0, last, n0, tid);
  const int jw0 = j0 + wt * WM;
  constexpr int HPW = WN / HD, CBH = HD / 32;
  const fused::KExtra x = fused::make_kextra(a.rope_cos, a.rope_sin, a.n_sink, a.n_recent, L);
  k_scores<HD, ROPE, 4>(acc, &sm.e.q[wc * HPW * a.G * HD], a.G, lane, jw0, L, x, [&](float (&s)[4], int hw, int g) {
    score_tail<4>(s, sm.e.p[wave][hw * a.G + g], sm.e.ml[wave][hw * a.G + g], lane, jw0, x);
  });
  gemm_pass<false>(acc, sm, a, a.xa[1] + row0 * a.D, a.xr[1] + row0 * a.m, a.w[1] + n0, last, n0, tid);
  if (jw0 >= L) return;
  const int H_kv = a.H_q / a.G, kvh0 = a.n_ret_heads + (n0 + wc * WN) / HD;
#pragma unroll
  for (int hw = 0; hw < HPW; ++hw) {
    if (kvh0 + hw >= H_kv) continue;
    for (int g = 0; g < a.G; ++g) {
      pin_acc(acc);
      const int pair = hw * a.G + g;
      const int64_t ph = ((int64_t)meta.sbase[b] + jw0 / kSlotTokens) * a.H_q + (kvh0 + hw) * a.G + g;
      float o[CBH];
      value_sum<HD, 4>(acc, sm.e.p[wave][pair], hw, lane, o);
#pragma unroll
      for (int cb = 0; cb < CBH; ++cb)
        if (lane < 32) a.part_o[ph * HD + cb * 32 + lane] = o[cb];
      if (lane == 0) { a.part_ml[ph * 2] = sm.e.ml[wave][pair][0]; a.part_ml[ph * 2 + 1] = sm.e.ml[wave][pair][1]; }
    }
  }
}

}  // namespace fused32

inline int launch_fused_decode_f32(int H_q, int H_kv, int d, int m, int d_out, int n_ret_heads,
                                   float scale, const float* ka,
                                   const float* va, const float* kr, const float* vr,
                                   const float* wk, const float* wv, const float* q,
                                   float* part_o, float* part_ml, SeqMeta& mt, int* fused_step,
                                   hipStream_t st, const KvExtras& ex = KvExtras()) {
  fused32::Args a;
  a.rope_cos = ex.rope_cos; a.rope_sin = ex.rope_sin; a.n_sink = ex.n_sink; a.n_recent = ex.n_recent;
  a.xa[0] = ka; a.xa[1] = va; a.xr[0] = kr; a.xr[1] = vr; a.w[0] = wk; a.w[1] = wv;
  a.q = q; a.part_o = part_o; a.part_ml = part_ml;
  a.D = H_kv * d; a.m = m; a.d_out = d_out; a.H_q = H_q; a.G = H_q / H_kv;
  a.n_ret_heads = n_ret_heads; a.scale = scale;
  a.n_col_tiles = (a.d_out + fused::BN - 1) / fused::BN;
  a.n_tiles = fused_fill_tiles(mt) * a.n_col_tiles;
  const dim3 g(a.n_tiles), blk(fused32::NTHREADS);
  const bool rope = ex.rope_cos != nullptr;
  if (d == 128 && rope) hipLaunchKernelGGL((fused32::fused_decode_f32_kernel<128, true>), g, blk, 0, st, a, mt);
  else if (d == 128) hipLaunchKernelGGL((fused32::fused_decode_f32_kernel<128, false>), g, blk, 0, st, a, mt);
  else if (rope) hipLaunchKernelGGL((fused32::fused_decode_f32_kernel<64, true>), g, blk, 0, st, a, mt);
  else hipLaunchKernelGGL((fused32::fused_decode_f32_kernel<64, false>), g, blk, 0, st, a, mt);
  if (hipGetLastError() != hipSuccess) return 7;
  *fused_step = 1;
  return 0;
}

}  // namespace echokv
