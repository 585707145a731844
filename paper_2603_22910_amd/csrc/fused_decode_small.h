// Fused reconstruct-then-attend decode for small problems (gfx950, bf16 and fp32 caches).
//
// The 256 x 256 tile of fused_decode.h needs a few thousand (token, column) tiles' worth of work to
// fill 256 compute units: one sequence of 1000 tokens of a 4-predicted-head layer is 8 workgroups.
// Here one workgroup of eight waves owns 16 * TB tokens x one 128-column slice of the predicted
// dims (one head of 128, or two of 64; fp32: one head) and everything about the slice is
// arranged for latency:
//  - waves 0-3 build K_hat, waves 4-7 build V_hat at the same time; the four waves of a side take every
//    fourth step of the input dims.  No operand is shared between waves, so both go straight from
//    global memory to registers: no LDS stage, no barrier in the main loop, two or three steps in flight.
//  - scores and the weighted value sum are linear in K_hat / V_hat, so the waves never add their
//    partial products up: each works out its share of q . k_hat_j and of sum_j p_j v_hat_j, and
//    only those (a few floats per token / per head dim) meet in LDS.
//  - the retained heads' streaming attention and the uncompressed window's attention run in further
//    workgroups of the same launch instead of launches of their own.
// MFMA form (16 x 16 x 32 bf16, 16 x 16 x 4 fp32): lane % 16 = row / column, lane / 16 = group of
// consecutive input dims.  A 16-byte load of row-major W holds VW output columns of one input dim; MFMA i
// takes element i of every lane, so it owns the columns VW * (lane % 16) + i.  bf16 needs 8 input dims
// per lane: eight such loads, transposed 8 x 8 in registers.
//
// What bounds it: bf16, a chain: about 3 us of every launch are the first round trip, 3-4 us the epilogues, and in between every workgroup reads
// its whole W slice (2 * d_in * 128 elements) for 16 * TB tokens through one unit's port to L2: 0.8 us per step of eight waves and 32 tokens, 10 KB
// each = 100 GB/s per unit, 43 bytes per clock at 2.4 GHz; with 64 tokens 1.25 us for 12 KB each.  With the W loads of all steps but the
// first left out, 1 x 1000 tokens (12 steps, 786 KB of W per workgroup) take 15.3 instead of 20.6 us with rotary tables and window, 14.7 instead of
// 18.6 without: a quarter of the call is W.  fp32, the matrix pipes of the units that have a workgroup.
// Measured against the 256 x 256 kernel with its separate launches (whole call, us, before -> after):
//   H_q/H_kv = 32/8, m = 512:  1 x 1000 tokens 84 -> 22 (with rotary tables and window 110 -> 26), 1 x 6000 86 -> 54
//   H_q/H_kv = 32/32, m = 2048: 1 x 500 tokens 225 -> 59, 1 x 1000 225 -> 76
//   fp32, 8 heads of 64, m = 256: 1 x 512 tokens 464 -> 17, 1 x 8000 509 -> 71
// With scores and value sums of three and more query heads per KV head on the matrix pipe, wave reductions on the vector unit and the
// merge without barriers, H_q/H_kv = 32/8, m = 512, rotary tables and window: 1 x 300 tokens 22.7 -> 20.8, 1 x 1000 23.0 -> 21.1, 1 x 3000 32.7 -> 30.1;
// without: 1 x 1000 22.3 -> 20.9; m = 384, packed W, 4 x 500-1500 58.4 -> 55.5
#pragma once
#include "common.h"
#include "fused_decode.h"
#include "attn_split.h"

namespace echokv {
namespace fsmall {

using fused::KExtra; using fused::MAXPAIR; using fused::u32x4_t; using fused::rsrc_t;
typedef float f32x4_t __attribute__((ext_vector_type(4)));
constexpr int NWAVES = 8, NTHREADS = 64 * NWAVES, KSPLIT = 4;

template <typename T>
struct Args {
  const T* xa[2]; const T* xr[2];             // anchor / retained cache K, V
  const T* w[2];                              // [d_in, d_out] row-major, or [d_out, d_in] (PACKED)
  const T* q; float* part_o; float* part_ml;
  int32_t D, m, d_out, H_q, G, n_ret_heads;
  float scale;
  int32_t n_ttiles, n_col_tiles;
  const float* rope_cos; const float* rope_sin;
  int32_t n_sink, n_recent;
  Streams<T> streams;                         // retained heads and window rows, behind the product's workgroups
  int32_t n_fused;                            // workgroups of the product
};

template <typename T, int HD> struct Cfg {
  static constexpr int VW = 16 / (int)sizeof(T);          // columns per 16-byte load: 8 / 4
  static constexpr int BN = sizeof(T) == 2 ? 128 : HD;    // columns of a workgroup
  static constexpr int NCG = BN / (16 * VW);              // column groups: 1, or HD / 64 (fp32)
  static constexpr int HPT = BN / HD;                     // heads of a workgroup
  static constexpr int KS = sizeof(T) == 2 ? 32 : 16;     // input dims per step
  static constexpr int NW = sizeof(T) == 2 ? 8 : 4 * NCG; // W loads per step
  // (128 / d) * G <= MAXPAIR, so HPT * G (head, query head) pairs fit the LDS arrays
};

// Accumulators of a wave's share of the tile.
template <typename T, int HD, int TB> struct Acc { f32x4_t v[Cfg<T, HD>::NCG * Cfg<T, HD>::VW][TB]; };

template <int TB>
struct Smem {
  float q[MAXPAIR * 128];                     // [pair][HD], pre-scaled
  float s[KSPLIT][MAXPAIR][16 * TB];          // score shares of the K waves
  float p[MAXPAIR][16 * TB];                  // softmax numerators
  float ml[MAXPAIR][2];
  float o[KSPLIT][MAXPAIR * 128];             // value shares of the V waves
};

template <typename T, int HD, int TB> struct Stage {
  u32x4_t x[TB];
  u32x4_t w[Cfg<T, HD>::NW];
};

// Per-wave operand addressing: raw buffers (uniform base, 32-bit byte offsets).
struct Io {
  rsrc_t xa, xr, w;
  int D, m, d_in, d_out, nka;                 // nka: steps inside the anchor row
  uint32_t last;                              // last valid token of the tile
  uint32_t wl;                                // lane part of the W offset
};

template <typename T, int HD, int TB, bool PACKED>
__device__ __forceinline__ void fetch(Stage<T, HD, TB>& s, const Io& io, int ks, int lane, int n0) {
  using C = Cfg<T, HD>;
  const int row = lane >> 2, ch = (lane & 3) * 16;      // see exchange
  const bool anchor = ks < io.nka;
  const uint32_t ld = (uint32_t)(anchor ? io.D : io.m) * sizeof(T);
  const int xoff = (anchor ? ks : ks - io.nka) * C::KS * (int)sizeof(T);
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const uint32_t voff = min((uint32_t)(tb * 16 + row), io.last) * ld + ch;
    s.x[tb] = anchor ? __builtin_amdgcn_raw_buffer_load_b128(io.xa, voff, xoff, 0)
                     : __builtin_amdgcn_raw_buffer_load_b128(io.xr, voff, xoff, 0);
  }
  if constexpr (PACKED) {              // bf16: 16 rows (output columns 8 row + i) x 32 input dims, as X
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t n = (uint32_t)min(8 * row + i, io.d_out - 1 - n0);
      s.w[i] = __builtin_amdgcn_raw_buffer_load_b128(io.w, n * (uint32_t)io.d_in * 2 + ch, ks * 64, 0);
    }
  } else if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int e = 0; e < 8; ++e)        // input dim 32 ks + 8 o + e
      s.w[e] = __builtin_amdgcn_raw_buffer_load_b128(io.w, io.wl, (ks * 32 + e) * io.d_out * 2, 0);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)        // input dim 16 ks + 4 o + j
#pragma unroll
      for (int cg = 0; cg < C::NCG; ++cg)
        s.w[j * C::NCG + cg] = __builtin_amdgcn_raw_buffer_load_b128(io.w, io.wl, ((ks * 16 + j) * io.d_out + cg * 64) * 4, 0);
  }
}

// The MFMA operand wants lane = 16 * (16-byte chunk) + row.  Loaded like that, four neighbouring lanes touch
// four rows, and the address unit takes a row per clock: four times as long per byte as for neighbouring
// lanes inside one row (measured: the 2 X loads of a step cost as much as its 8 W loads).  So rows are
// loaded as lane = 4 * row + chunk and change lanes through 1 KB of LDS that belongs to the wave (LDS
// operations of a wave stay in order: no barrier).  Chunk c of row r sits at chunk c ^ (r / 4 % 4):
// no bank conflicts in either direction.
__device__ __forceinline__ void lanes_out(const u32x4_t& v, char* buf, int lane) {
  const int row = lane >> 2, ch = lane & 3;
  *reinterpret_cast<u32x4_t*>(buf + row * 64 + ((ch ^ (row >> 2)) << 4)) = v;
}
__device__ __forceinline__ u32x4_t lanes_in(const char* buf, int lane) {
  const int row = lane & 15, ch = lane >> 4;
  return *reinterpret_cast<const u32x4_t*>(buf + row * 64 + ((ch ^ (row >> 2)) << 4));
}
template <typename T, int HD, int TB, bool PACKED>
__device__ __forceinline__ void exchange(Stage<T, HD, TB>& f, const Stage<T, HD, TB>& s, char* buf, int lane) {
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) lanes_out(s.x[tb], buf + tb * 1024, lane);
  if constexpr (PACKED) {
#pragma unroll
    for (int i = 0; i < 8; ++i) lanes_out(s.w[i], buf + (TB + i) * 1024, lane);
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) f.x[tb] = lanes_in(buf + tb * 1024, lane);
  if constexpr (PACKED) {
#pragma unroll
    for (int i = 0; i < 8; ++i) f.w[i] = lanes_in(buf + (TB + i) * 1024, lane);
  } else {
#pragma unroll
    for (int i = 0; i < Cfg<T, HD>::NW; ++i) f.w[i] = s.w[i];
  }
  asm volatile("" ::: "memory");
}
// LDS of a wave for it
template <int TB, bool PACKED> constexpr int exchange_bytes() { return (TB + (PACKED ? 8 : 0)) * 1024; }

// acc.v[cg * VW + i][tb]: KSIDE: rows = columns VW * (4 (lane / 16) + r) + i of group cg, lane % 16 = token;
// otherwise rows = tokens 4 (lane / 16) + r of block tb, lane % 16 = column slot.
template <typename T, int HD, int TB, bool PACKED, bool KSIDE>
__device__ __forceinline__ void mma(Acc<T, HD, TB>& acc, const Stage<T, HD, TB>& s) {
  using C = Cfg<T, HD>;
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      u32x4_t wt;
      if constexpr (PACKED) wt = s.w[i];
      else {
#pragma unroll
        for (int p = 0; p < 4; ++p)
          wt[p] = __builtin_amdgcn_perm(s.w[2 * p + 1][i >> 1], s.w[2 * p][i >> 1], (i & 1) ? 0x07060302u : 0x05040100u);
      }
      const bf16x8_t wf = __builtin_bit_cast(bf16x8_t, wt);
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        const bf16x8_t xf = __builtin_bit_cast(bf16x8_t, s.x[tb]);
        acc.v[i][tb] = KSIDE ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, acc.v[i][tb], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, wf, acc.v[i][tb], 0, 0, 0);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int cg = 0; cg < C::NCG; ++cg)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) {
            const float wf = __uint_as_float(s.w[j * C::NCG + cg][i]), xf = __uint_as_float(s.x[tb][j]);
            f32x4_t& d = acc.v[cg * 4 + i][tb];
            d = KSIDE ? __builtin_amdgcn_mfma_f32_16x16x4f32(wf, xf, d, 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_16x16x4f32(xf, wf, d, 0, 0, 0);
          }
  }
}

// This wave's share of the product: steps kq, kq + 4, ... of the input dims.  `between` runs once the
// first loads are on their way.  (Two register stages: a third one measured no faster.)
template <typename T, int HD, int TB, bool PACKED, bool KSIDE, class Between>
__device__ __forceinline__ void product(Acc<T, HD, TB>& acc, const Io& io, int kq, int lane, int n0, char* buf,
                                        Between between) {
  using C = Cfg<T, HD>;
  constexpr int NST = 2;
  const int n = (io.d_in / C::KS - kq + KSPLIT - 1) / KSPLIT;      // at least 1: the caller sees to KSPLIT steps and more
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < C::NCG * C::VW; ++i)
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc.v[i][tb][r] = 0.f;
  };
  Stage<T, HD, TB> st[NST];
  if constexpr (TB >= 4) {                     // (no registers left to overlap the two)
    between();
    clear();
    if (n <= 0) return;                        // (never; without the exit the registers do not suffice)
  }
#pragma unroll
  for (int u = 0; u < NST; ++u) fetch<T, HD, TB, PACKED>(st[u], io, kq + KSPLIT * min(u, n - 1), lane, n0);
  if constexpr (TB < 4) {
    between();
    clear();
  }
  for (int it = 0; it < n; it += NST) {
#pragma unroll
    for (int u = 0; u < NST; ++u) {
      Stage<T, HD, TB> f;
      exchange<T, HD, TB, PACKED>(f, st[u], buf, lane);
      if (it + u < n) mma<T, HD, TB, PACKED, KSIDE>(acc, f);
      fetch<T, HD, TB, PACKED>(st[u], io, kq + KSPLIT * min(it + u + NST, n - 1), lane, n0);
    }
  }
}

// Rotary table rows of the tile's tokens in LDS: [token][HD / 2] cos, then sin; 16-byte chunk ch of
// token row r sits at chunk ch ^ (r % chunks): the 16 token rows a wave reads hit different banks.
template <int HD, int TB> struct RopeTile {
  static constexpr int CH = HD / 8, TOK = 16 * TB, N = (TOK * CH + NTHREADS - 1) / NTHREADS;
  static constexpr int kBytes = 2 * TOK * HD / 2 * 4;
  f32x4_t c[N], s[N];
  __device__ __forceinline__ void load(const KExtra& x, int j0, int L, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = min(i * NTHREADS + tid, TOK * CH - 1);
      const int64_t at = (int64_t)min(j0 + idx / CH, L - 1) * (HD / 2) + idx % CH * 4;
      c[i] = *reinterpret_cast<const f32x4_t*>(x.cos + at);
      s[i] = *reinterpret_cast<const f32x4_t*>(x.sin + at);
    }
  }
  __device__ static __forceinline__ int at(int row, int ch) { return row * CH + (ch ^ (row & (CH - 1))); }
  __device__ __forceinline__ void store(f32x4_t* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = min(i * NTHREADS + tid, TOK * CH - 1);       // (spare threads repeat the last chunk)
      lds[at(idx / CH, idx % CH)] = c[i];
      lds[TOK * CH + at(idx / CH, idx % CH)] = s[i];
    }
  }
};

// Sum over the 16-lane rows of a wave: rows (0, 1) and (2, 3); then rows (0, 2) and (1, 3).
__device__ __forceinline__ float add_row_pair(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Shares of the scaled scores (Eq. 7) of the wave's K_hat share -> sm.s[kq].  A lane holds, per token
// block and column group, 4 * VW consecutive columns of one head.  Rotary embedding (fp32; bf16: rope_score_shares): the rotation of
// the key is moved onto the query, q'_c = q_c cos + q_{c + d/2} sin (c < d/2), q_c cos - q_{c - d/2} sin.
// The loop over the query heads stays a loop: every workgroup runs this code once, and unrolled its
// instructions alone take longer to fetch than to execute.
template <typename T, int HD, int TB, bool ROPE>
__device__ __forceinline__ void score_shares(Acc<T, HD, TB>& acc, Smem<TB>& sm, int G,
                                             int kq, int lane, const f32x4_t* tables) {
  static_assert(!ROPE || sizeof(T) == 4, "bf16 with rotary tables: rope_score_shares");
  using C = Cfg<T, HD>;
  using R = RopeTile<HD, TB>;
  constexpr int RUN = 4 * C::VW;               // columns of a lane and group
  constexpr int TP = ROPE ? 1 : TB;            // token blocks per round (their table rows are kept in registers)
  const int c = lane & 15, o = lane >> 4;
  const int hw = C::HPT == 2 ? o >> 1 : 0;
#pragma unroll
  for (int t0 = 0; t0 < TB; t0 += TP) {
#pragma unroll
    for (int cg = 0; cg < C::NCG; ++cg) {
      const int h0 = (cg * 16 * C::VW + RUN * o) % HD;      // first column inside the head
      const int hp = h0 < HD / 2 ? h0 + HD / 2 : h0 - HD / 2;
      f32x4_t cs[ROPE ? TP : 1][RUN / 4], sn[ROPE ? TP : 1][RUN / 4];
      if constexpr (ROPE) {
        const float sgn = h0 < HD / 2 ? 1.f : -1.f;
#pragma unroll
        for (int t = 0; t < TP; ++t) {
          const int row = (t0 + t) * 16 + c;
#pragma unroll
          for (int j = 0; j < RUN / 4; ++j) {
            cs[t][j] = tables[R::at(row, h0 % (HD / 2) / 4 + j)];
            sn[t][j] = tables[R::TOK * R::CH + R::at(row, h0 % (HD / 2) / 4 + j)];
            sn[t][j] *= sgn;
          }
        }
      }
#pragma nounroll
      for (int g = 0; g < G; ++g) {
        const float* qs = &sm.q[(hw * G + g) * HD];
        float s[TP];
#pragma unroll
        for (int t = 0; t < TP; ++t) s[t] = 0.f;
#pragma unroll
        for (int j = 0; j < RUN; j += 4) {
          const float4 qa = *reinterpret_cast<const float4*>(qs + h0 + j);
          float4 qp;
          if constexpr (ROPE) qp = *reinterpret_cast<const float4*>(qs + hp + j);
#pragma unroll
          for (int t = 0; t < TP; ++t) {
            float4 qv = qa;
            if constexpr (ROPE) {
              const f32x4_t cc = cs[t][j / 4], ss = sn[t][j / 4];
              qv.x = fmaf(qa.x, cc.x, qp.x * ss.x); qv.y = fmaf(qa.y, cc.y, qp.y * ss.y);
              qv.z = fmaf(qa.z, cc.z, qp.z * ss.z); qv.w = fmaf(qa.w, cc.w, qp.w * ss.w);
            }
            const float qq[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              s[t] = fmaf(qq[e], acc.v[cg * C::VW + (j + e) % C::VW][t0 + t][(j + e) / C::VW], s[t]);
          }
        }
#pragma unroll
        for (int t = 0; t < TP; ++t) {
          float v = add_row_pair(s[t]);
          if constexpr (C::HPT == 1) v = add_halves(v);
          float* dst = &sm.s[kq][hw * G + g][(t0 + t) * 16 + c];
          if ((C::HPT == 2 ? o & 1 : o) == 0) *dst = cg == 0 ? v : *dst + v;      // (one writer per word)
        }
      }
    }
  }
}

// The same for bf16 with rotary tables.  A dim's rotation partner is held by the lane 32 (heads of 64: 16) further on; two token blocks are
// exchanged against each other so that a lane holds both partners of 32 pairs for the tokens of one block, and the key
// is rotated once for all query heads (4 + 2 G operations per pair instead of 6 G with the rotation on the query, half the LDS reads).
// Whole calls with rotary tables and window, us: 32 heads over 8 of 128, m = 512: 300 tokens 24.0 -> 22.7, 1000 24.2 -> 22.9, 2000 33.5 -> 30.8, 8 x 400
// 40.6 -> 38.6, m = 384, 4 x 1500 70.3 -> 64.8; one query head per KV head 21.1 -> 20.9, heads of 64 16.2 -> 15.9.
template <int HD, int TB>
__device__ __forceinline__ void rope_score_shares(Acc<bf16_t, HD, TB>& acc, Smem<TB>& sm, int G, int kq, int lane, const f32x4_t* tables) {
  using R = RopeTile<HD, TB>;
  const int c = lane & 15, o = lane >> 4;
  const int hw = HD == 64 ? o >> 1 : 0, h0 = HD == 64 ? 0 : 32 * (o & 1);      // head, first dim of the lower partners
#pragma unroll
  for (int t0 = 0; t0 < TB; t0 += 2) {
    const int row = (t0 + (HD == 64 ? o & 1 : o >> 1)) * 16 + c;                 // this lane's token
    float lo[32], hi[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      const uint32_t a = __float_as_uint(acc.v[j & 7][t0][j >> 3]), b = __float_as_uint(acc.v[j & 7][t0 + 1][j >> 3]);
      if constexpr (HD == 64) {
        const auto x = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        lo[j] = __uint_as_float(x[0]); hi[j] = __uint_as_float(x[1]);
      } else {
        const auto x = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        lo[j] = __uint_as_float(x[0]); hi[j] = __uint_as_float(x[1]);
      }
    }
#pragma unroll
    for (int j = 0; j < 32; j += 4) {
      const f32x4_t cs = tables[R::at(row, (h0 + j) / 4)], sn = tables[R::TOK * R::CH + R::at(row, (h0 + j) / 4)];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = lo[j + e], y = hi[j + e];
        lo[j + e] = fmaf(x, cs[e], -y * sn[e]);
        hi[j + e] = fmaf(y, cs[e], x * sn[e]);
      }
    }
    if (G > fused::kVectorHeads) {       // four query heads at a time on the matrix pipe (see fma_heads)
#pragma nounroll
      for (int g0 = 0; g0 < G; g0 += 4) {
        const float* qs = &sm.q[(hw * G + min(g0 + (lane & 3), G - 1)) * HD + h0];
        floatx4_t s4[2] = {floatx4_t{0.f, 0.f, 0.f, 0.f}, floatx4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int j = 0; j < 32; j += 4) {
          const float4 a4 = *reinterpret_cast<const float4*>(qs + j), b4 = *reinterpret_cast<const float4*>(qs + HD / 2 + j);
          const float qa[4] = {a4.x, a4.y, a4.z, a4.w}, qb[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s4[0] = fma_heads(qa[e], lo[j + e], s4[0]);
            s4[1] = fma_heads(qb[e], hi[j + e], s4[1]);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float s = s4[0][i] + s4[1][i];
          if constexpr (HD == 128) s = add_row_pair(s);
          if (g0 + i < G && (HD == 64 || (o & 1) == 0)) sm.s[kq][hw * G + g0 + i][row] = s;
        }
      }
      continue;
    }
#pragma nounroll
    for (int g = 0; g < G; ++g) {
      const float* qs = &sm.q[(hw * G + g) * HD + h0];
      float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
      for (int j = 0; j < 32; j += 4) {
        const float4 qa = *reinterpret_cast<const float4*>(qs + j), qb = *reinterpret_cast<const float4*>(qs + HD / 2 + j);
        s0 = fmaf(qa.x, lo[j], fmaf(qb.x, hi[j], s0)); s1 = fmaf(qa.y, lo[j + 1], fmaf(qb.y, hi[j + 1], s1));
        s2 = fmaf(qa.z, lo[j + 2], fmaf(qb.z, hi[j + 2], s2)); s3 = fmaf(qa.w, lo[j + 3], fmaf(qb.w, hi[j + 3], s3));
      }
      float s = (s0 + s1) + (s2 + s3);
      if constexpr (HD == 128) s = add_row_pair(s);
      if (HD == 64 || (o & 1) == 0) sm.s[kq][hw * G + g][row] = s;
    }
  }
}

// Shares of sum_j p_j v_hat_j of the wave's V_hat share -> sm.o[kq].
template <typename T, int HD, int TB>
__device__ __forceinline__ void value_shares(Acc<T, HD, TB>& acc, Smem<TB>& sm, int G,
                                             int kq, int lane) {
  using C = Cfg<T, HD>;
  const int c = lane & 15, o = lane >> 4;
  const int hw = C::HPT == 2 ? c >> 3 : 0;
  if constexpr (sizeof(T) == 2) {
    if (G > fused::kVectorHeads) {       // four query heads at a time on the matrix pipe (see fma_heads)
#pragma nounroll
      for (int g0 = 0; g0 < G; g0 += 4) {
        const float* ps = sm.p[hw * G + min(g0 + (lane & 3), G - 1)] + 4 * o;
        floatx4_t v[C::VW];
#pragma unroll
        for (int i = 0; i < C::VW; ++i) v[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          const float4 p4 = *reinterpret_cast<const float4*>(ps + tb * 16);
          const float p[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < C::VW; ++i) v[i] = fma_heads(p[r], acc.v[i][tb][r], v[i]);
        }
        float x[C::VW];
#pragma unroll
        for (int i = 0; i < C::VW; ++i) x[i] = sum_rows(v[i][0], v[i][1], v[i][2], v[i][3]);      // row o: query head g0 + o
        if (g0 + o < G) {
          float* dst = &sm.o[kq][(hw * G + g0 + o) * HD + C::VW * c % HD];
          *reinterpret_cast<float4*>(dst) = make_float4(x[0], x[1], x[2], x[3]);
          *reinterpret_cast<float4*>(dst + 4) = make_float4(x[4], x[5], x[6], x[7]);
        }
      }
      return;
    }
  }
#pragma nounroll
  for (int g = 0; g < G; ++g) {
    const int pair = hw * G + g;
    float v[C::NCG * C::VW];
#pragma unroll
    for (int i = 0; i < C::NCG * C::VW; ++i) v[i] = 0.f;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const float4 p = *reinterpret_cast<const float4*>(&sm.p[pair][tb * 16 + 4 * o]);
#pragma unroll
      for (int i = 0; i < C::NCG * C::VW; ++i) {
        v[i] = fmaf(p.x, acc.v[i][tb][0], v[i]); v[i] = fmaf(p.y, acc.v[i][tb][1], v[i]);
        v[i] = fmaf(p.z, acc.v[i][tb][2], v[i]); v[i] = fmaf(p.w, acc.v[i][tb][3], v[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < C::NCG * C::VW; ++i) v[i] = add_halves(add_row_pair(v[i]));
    if (o == 0) {
#pragma unroll
      for (int i = 0; i < C::NCG * C::VW; ++i)
        sm.o[kq][pair * HD + ((i / C::VW) * 16 * C::VW + C::VW * c + i % C::VW) % HD] = v[i];
    }
  }
}

template <typename T, int HD, int TB, bool PACKED, bool ROPE>
__device__ __forceinline__ void fused_tile(const Args<T>& a, const StreamMeta& meta, Smem<TB>& sm, int wg) {
  using C = Cfg<T, HD>;
  constexpr int TOK = 16 * TB;
  const int ttile = wg % a.n_ttiles, ctile = wg / a.n_ttiles;
  const int b = find_seq(meta.s.tbase, meta.s.n, ttile);
  const int L = meta.s.len[b];
  const int j0 = (ttile - meta.s.tbase[b]) * TOK;
  const int n0 = ctile * C::BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int side = wave >> 2, kq = wave & 3;
  const int64_t row0 = meta.s.start[b] + j0;
  const int H_kv = a.H_q / a.G, kvh0 = a.n_ret_heads + n0 / HD;

  Io io;
  io.xa = fused::make_rsrc(a.xa[side] + row0 * a.D); io.xr = fused::make_rsrc(a.xr[side] + row0 * a.m);
  io.w = fused::make_rsrc(a.w[side] + (PACKED ? (int64_t)n0 * (a.D + a.m) : n0));
  io.D = a.D; io.m = a.m; io.d_in = a.D + a.m; io.d_out = a.d_out; io.nka = a.D / C::KS;
  io.last = (uint32_t)(min(TOK, L - j0) - 1);        // rows past the end repeat the last token (finite, masked)
  // columns past d_out (a lone last head of 64) repeat the last valid ones; their head is not written
  const int wcol = min(C::VW * (lane & 15), a.d_out - C::VW - n0);
  io.wl = (uint32_t)(((lane >> 4) * (C::KS / 4)) * a.d_out + wcol) * (uint32_t)sizeof(T);

  // queries and table rows are requested first, then the product's first steps; they go to LDS while those travel
  constexpr int NQ = (MAXPAIR * 128 + NTHREADS - 1) / NTHREADS;
  float qv[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int idx = min(i * NTHREADS + tid, C::HPT * a.G * HD - 1);
    const int pr = idx / HD, kvh = min(kvh0 + pr / a.G, H_kv - 1);      // (a head past the last one is not written)
    qv[i] = Elem<T>::to_f32(a.q[((int64_t)b * a.H_q + kvh * a.G + pr % a.G) * HD + idx % HD]) * a.scale;
  }
  const KExtra x = fused::make_kextra(a.rope_cos, a.rope_sin, a.n_sink, a.n_recent, L);
  RopeTile<HD, TB> rope;
  if constexpr (ROPE) rope.load(x, j0, L, tid);
  char* ext = reinterpret_cast<char*>(&sm) + sizeof(Smem<TB>);
  f32x4_t* tables = reinterpret_cast<f32x4_t*>(ext + NWAVES * exchange_bytes<TB, PACKED>());
  auto to_lds = [&]() {
    if constexpr (TB < 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (i * NTHREADS + tid < C::HPT * a.G * HD) sm.q[i * NTHREADS + tid] = qv[i];
    if constexpr (ROPE) rope.store(tables, tid);
  };
  Acc<T, HD, TB> acc;
  char* buf = ext + wave * exchange_bytes<TB, PACKED>();
  if (side == 0) product<T, HD, TB, PACKED, true>(acc, io, kq, lane, n0, buf, to_lds);
  else product<T, HD, TB, PACKED, false>(acc, io, kq, lane, n0, buf, to_lds);
  __syncthreads();                                   // queries are in LDS
  if (side == 0) {
    if constexpr (ROPE && sizeof(T) == 2) rope_score_shares<HD, TB>(acc, sm, a.G, kq, lane, tables);
    else score_shares<T, HD, TB, ROPE>(acc, sm, a.G, kq, lane, tables);
  }
  __syncthreads();
  // softmax numerators: one wave per (head, query head) pair
  const int npair = C::HPT * a.G;
  for (int pr = wave; pr < npair; pr += NWAVES) {
    float s = -INFINITY;
    if (lane < TOK) {
      s = (sm.s[0][pr][lane] + sm.s[1][pr][lane]) + (sm.s[2][pr][lane] + sm.s[3][pr][lane]);
      const int tok = j0 + lane;
      if (tok < x.lo || tok >= x.hi) s = -INFINITY;
    }
    const float mx = wave_max64(s);
    const float p = s == -INFINITY ? 0.f : __expf(s - mx);
    const float sum = wave_sum64(p);
    if (lane < TOK) sm.p[pr][lane] = p;
    if (lane == 0) { sm.ml[pr][0] = mx; sm.ml[pr][1] = sum; }
  }
  __syncthreads();
  if (side == 1) value_shares<T, HD, TB>(acc, sm, a.G, kq, lane);
  __syncthreads();
  const int64_t slot = meta.s.sbase[b] + j0 / TOK;
  for (int idx = tid; idx < npair * HD; idx += NTHREADS) {
    const int pr = idx / HD, c = idx % HD, kvh = kvh0 + pr / a.G;
    if (kvh >= H_kv) continue;
    const int64_t ph = slot * a.H_q + kvh * a.G + pr % a.G;
    a.part_o[ph * HD + c] = (sm.o[0][idx] + sm.o[1][idx]) + (sm.o[2][idx] + sm.o[3][idx]);
    if (c == 0) { a.part_ml[ph * 2] = sm.ml[pr][0]; a.part_ml[ph * 2 + 1] = sm.ml[pr][1]; }
  }
}

template <typename T, int HD, int TB, bool PACKED, bool ROPE>
__global__ __launch_bounds__(NTHREADS) void fused_decode_small_kernel(Args<T> a, StreamMeta meta) {
  constexpr int kStream = stream_smem_bytes<T, HD, NWAVES>();
  constexpr int kTile = (int)sizeof(Smem<TB>) + NWAVES * exchange_bytes<TB, PACKED>() + (ROPE ? RopeTile<HD, TB>::kBytes : 0);
  constexpr int kBytes = kTile > kStream ? kTile : kStream;
  __shared__ __attribute__((aligned(16))) char smem[kBytes];
  int wg = blockIdx.x;
  if (wg < a.n_fused) {
    // workgroups are dealt round robin to the 8 XCDs: each XCD takes a contiguous run of the
    // column-major order, so it reads few W slices and keeps them in its L2
    const int per = (a.n_fused + 7) >> 3;             // (n_fused is padded to a multiple of 8)
    const int logical = (wg & 7) * per + (wg >> 3);
    if (logical >= a.n_ttiles * a.n_col_tiles) return;
    fused_tile<T, HD, TB, PACKED, ROPE>(a, meta, *reinterpret_cast<Smem<TB>*>(smem), logical);
    return;
  }
  stream_workgroup<T, HD, NWAVES, 4>(a.streams, meta, wg - a.n_fused, smem);
}

}  // namespace fsmall

// tb: token blocks of 16 per workgroup: 2 or 4 (bf16), 1 or 2 (fp32).
template <typename T>
int launch_fused_decode_small(const fsmall::Args<T>& a, const StreamMeta& mt, int tb, bool packed, hipStream_t st);

}  // namespace echokv
