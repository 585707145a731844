// Fused reconstruct-then-attend decode kernel for gfx950 (bf16 MFMA), its key half on its own, and the
// stand-alone predictor product; the main loop they share is in fused_gemm.h.
//
// One workgroup owns a tile of 256 cached tokens x 256 predicted columns
// (two heads of 128, or four of 64).  For that tile it
//   1. runs the predictor product for K (Eq. 3) with W as the row operand so that each
//      lane ends up holding dims of K_hat^T for ONE token in each of four blocks: the score
//      q . k_hat_j (Eq. 7) is then a sum over the lane's own accumulators, over the four lanes
//      of a token, and with rotary tables, where a wave has half of every head's dims, over two waves;
//   2. takes the softmax numerators over each group of 64 tokens (max, sum of
//      exponentials), leaving p_j in LDS;
//   3. runs the predictor product for V with X as the row operand, so each
//      lane holds rows (tokens) of V_hat for one column per block and sum_j p_j v_hat_j
//      is a sum over the lane's own accumulators and four lanes as well;
//   4. joins the two groups of 64 tokens of a 128-token slot through LDS and writes one split-K partial
//      (max, sum, unnormalised o) per slot and head.
// K_hat and V_hat live only in accumulator registers: they never reach LDS or HBM.
// The retained heads' streaming attention and the window's run in further workgroups of the same launch.
//
// The predictor input row [anchor ; retained] (Eq. 3) is never materialised
// either: the k-loop walks the anchor cache for the first D input dims and
// the target's retained cache for the last m.
#pragma once
#include "common.h"
#include "fused_gemm.h"
#include "attn_split.h"

namespace echokv {

namespace fused {

constexpr int MAXPAIR = 8;   // query heads per 128 columns: (128 / head dim) * G at most
// Up to so many query heads per KV head the epilogues use the vector unit, beyond it fma_heads, whose instruction costs the same for one
// head and for four.  On the vector unit / the matrix pipe: one head, 8 x 4096 tokens 1222 / 1228 us, 20 x 1000 - 5000 1949 / 1966; two
// heads, 8 x 3000 79.7 / 80.6; three, 8 x 6000 175.0 / 174.4, heads of 64 69.2 / 68.3, 4 x 1000-9000 with rope 54.2 / 53.3; four heads (3140 - 24000
// tokens, rope, window) 319 / 308.  With rotary tables: the score kernel, one head, 40000 tokens 887 / 891, heads of 64, 8 x 4096
// 240.5 / 242.7, two heads of 64 98.1 / 99.2; in the fused kernel, where the two waves of 64 tokens share the dims, one head, 8 x 4096 1249 / 1253 (runs
// 9 apart), two, 8 x 6000 168.3 / 167.8, 17 calls of one and two heads of 64 and 128 within 1 % of each other: the matrix pipe alone there.
constexpr int kVectorHeads = 2;

struct Args {
  const bf16_t* xa[2];   // anchor cache K, V      [pool, D]
  const bf16_t* xr[2];   // retained cache K, V    [pool, m]
  const bf16_t* w[2];    // W_K, W_V               [D + m, d_out]
  const bf16_t* q;       // [nseq, H_q, d]
  float* part_o;         // [slots, H_q, d]
  float* part_ml;        // [slots, H_q, 2]
  bf16_t* out[2];        // store kernel only: K_hat / V_hat destination
  int64_t ldo;           // store kernel: row stride (elements)
  int32_t col0;          // store kernel: first column
  int32_t D, m, d_out, H_q, G, n_ret_heads;
  float scale;
  int32_t n_col_tiles, n_tiles;   // column tiles; token tiles * column tiles
  // paper-faithful extras (null / zero: off): rotary tables [positions, d/2] applied to the rebuilt
  // keys by token position; tokens held by the uncompressed window are masked out here
  const float* rope_cos; const float* rope_sin;
  int32_t n_sink, n_recent;
  float* s_out;          // score kernel only: S^T [H_q, s_ld], column = slot * 128 + token
  int64_t s_ld;
};

// LDS state of the attention epilogues; a pair: (head of the tile, query head of its group).
struct EpiSmem {
  float q[BN * MAXPAIR];               // [pair][d], pre-scaled
  float p[4][2 * MAXPAIR][WM];         // per 64 tokens and pair: score shares of one wave, then softmax numerators
  float ml[4][2 * MAXPAIR][2];         // max and sum
};
struct Smem {
  char st[2 * kStage];
  EpiSmem e;
};

// Workgroup id -> (token tile, column tile).  Consecutive workgroup ids go to
// different XCDs, so each XCD is given one contiguous range of logical tiles:
// the column tiles of a token tile then hit the same L2 copy of X.
__device__ __forceinline__ bool tile_of_block(const Args& a, int& ttile, int& ctile) {
  const int per_xcd = (a.n_tiles + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= a.n_tiles) return false;
  ttile = logical / a.n_col_tiles;
  ctile = logical % a.n_col_tiles;
  return true;
}

// Queries of the tile's nh heads -> LDS as fp32, pre-scaled by the softmax scale: [pair][HD], as they lie in memory.  Requested ahead of the
// first copies (behind them their wait would be for those as well) and stored once these are on their way.
struct Queries {
  static constexpr int N = BN * MAXPAIR / NTHREADS;
  bf16_t v[N];
  int n;
  __device__ __forceinline__ void load(const bf16_t* q, int n_, int tid) {
    n = n_;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = q[min(i * NTHREADS + tid, n - 1)];
  }
  __device__ __forceinline__ void store(float* eq, float scale, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (i * NTHREADS + tid < n) eq[i * NTHREADS + tid] = bf16_to_f32(v[i]) * scale;
  }
};

// Extras of the score epilogue: rotary tables (null: none) and the token range [lo, hi) of the
// sequence that counts (tokens outside are masked: past the end, or held by the window).
struct KExtra {
  const float* cos; const float* sin;
  int lo, hi;
};
__device__ __forceinline__ KExtra make_kextra(const float* cos, const float* sin, int n_sink,
                                              int n_recent, int L) {
  KExtra x;
  x.cos = cos; x.sin = sin;
  const bool win = n_sink + n_recent > 0;
  x.lo = win ? min(n_sink, L) : 0;
  x.hi = win ? max(x.lo, L - n_recent) : L;
  return x;
}

// A wave's share of the tile's heads (see column_of): N heads, of each CBH blocks of 16 columns; blocks b and b + HB are rotation partners.
template <int HD, bool SPLIT> struct Part {
  static constexpr int N = (SPLIT ? BN : WN) / HD, CBH = 8 / N, HB = CBH / 2;
  __device__ static __forceinline__ int head(int wc, int hw) { return SPLIT ? hw : wc * N + hw; }      // of the tile
  __device__ static __forceinline__ int dim(int b, int wc) { return SPLIT ? b / HB * (HD / 2) + wc * (HD / 4) + b % HB * 16 : 16 * b; }
  __device__ static constexpr __forceinline__ int block(int hw, int b) { return SPLIT ? b / HB * 4 + hw * HB + b % HB : hw * CBH + b; }      // of the accumulators
};

// After the K pass: acc[cb][tb] holds K_hat^T.  A lane owns rows 4 (lane / 16) + r of the wave's column blocks for
// the tokens 16 tb + lane % 16.  Hands out the scores (Eq. 7) of the tile's nh heads as tail(v, pair), v: that of the wave's token `lane`.
// SPLIT: the two waves of 64 tokens exchange half of their shares through share[pair][token], and wave column wc hands
// out the pairs with (hw + g) % 2 = wc; all waves of the workgroup come here.
// q: [pair][HD]; table(tb, hb, cs, sn): rotary table entries of the lane's token of block tb for the dims of block hb.
template <int HD, bool ROPE, bool SPLIT, class Table, class Tail>
__device__ __forceinline__ void k_scores(const Acc& acc, const float* q, float (*share)[WM], int nh, int G, int wc, int lane, Table table, Tail tail) {
  using P = Part<HD, SPLIT>;
  constexpr int CBH = P::CBH, HB = P::HB, MG = MAXPAIR * HD / 128;      // MG: query heads per KV head at most
  const int o = lane >> 4;
  uint32_t mine[P::N][MG / 2];               // SPLIT: shares of the pairs that this wave hands out
#pragma unroll
  for (int hw = 0; hw < P::N; ++hw)
#pragma unroll
    for (int i = 0; i < MG / 2; ++i) mine[hw][i] = 0;
  auto out = [&](float v, int hw, int g) __attribute__((always_inline)) {
    if constexpr (SPLIT) {
      // (as if / else of two stores the compiler selects between their addresses, and the array would lie in scratch memory)
      const uint32_t own = 0u - (uint32_t)(((hw + g) & 1) == wc);
      mine[hw][g / 2] = (own & __float_as_uint(v)) | (~own & mine[hw][g / 2]);
      if (!own) share[hw * G + g][lane] = v;
    } else {
      tail(v, P::head(wc, hw) * G + g);
    }
  };
  const float* qw = q + P::head(wc, 0) * G * HD + P::dim(0, wc) + 4 * o;
#pragma unroll
  for (int hw = 0; hw < P::N; ++hw) {
    if (P::head(wc, hw) >= nh) continue;
    if constexpr (ROPE) {
      // Rotary embedding of the rebuilt key at its token's position on its way into the dot product: feature c pairs with
      // c + HD/2.  With a = k_c, b = k_{c+HD/2}:
      //   q_c (a cos - b sin) + q_{c+HD/2} (b cos + a sin)
      // The rotated values are temporaries (written back they would cost hundreds of spilled registers), used by all query heads of
      // the group, in the fused kernel (SPLIT) by fma_heads for any number of them (see kVectorHeads).  Masked tokens borrow the last valid table row.
      constexpr int NG = MG / 4;             // groups of four query heads at most
      floatx4_t s[NG][4];
#pragma unroll
      for (int n = 0; n < NG; ++n)
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) s[n][tb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) {
        float ra[4][4], rb[4][4];
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
          float4 cs, sn;
          table(tb, hb, cs, sn);
          const floatx4_t& ka = acc.v[P::block(hw, hb)][tb];
          const floatx4_t& kb = acc.v[P::block(hw, hb + HB)][tb];
          const float cc[4] = {cs.x, cs.y, cs.z, cs.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ra[tb][i] = fmaf(ka[i], cc[i], -kb[i] * ss[i]);
            rb[tb][i] = fmaf(kb[i], cc[i], ka[i] * ss[i]);
          }
        }
        if (!SPLIT && G <= kVectorHeads) {
#pragma unroll
          for (int g = 0; g < kVectorHeads; ++g) {
            if (g >= G) continue;
            const float* qs = qw + (hw * G + g) * HD + hb * 16;
            const float4 qa = *reinterpret_cast<const float4*>(qs), qb = *reinterpret_cast<const float4*>(qs + HD / 2);
            const float q0[4] = {qa.x, qa.y, qa.z, qa.w}, q1[4] = {qb.x, qb.y, qb.z, qb.w};
#pragma unroll
            for (int tb = 0; tb < 4; ++tb)
#pragma unroll
              for (int i = 0; i < 4; ++i) s[0][tb][g] = fmaf(ra[tb][i], q0[i], fmaf(rb[tb][i], q1[i], s[0][tb][g]));
          }
        } else {
#pragma unroll
          for (int n = 0; n < NG; ++n) {
            if (4 * n < G) {
              const float* qs = qw + (hw * G + min(4 * n + (lane & 3), G - 1)) * HD + hb * 16;
              const float4 qa = *reinterpret_cast<const float4*>(qs), qb = *reinterpret_cast<const float4*>(qs + HD / 2);
              const float q0[4] = {qa.x, qa.y, qa.z, qa.w}, q1[4] = {qb.x, qb.y, qb.z, qb.w};
#pragma unroll
              for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int tb = 0; tb < 4; ++tb) s[n][tb] = fma_heads(q0[i], ra[tb][i], s[n][tb]);
#pragma unroll
                for (int tb = 0; tb < 4; ++tb) s[n][tb] = fma_heads(q1[i], rb[tb][i], s[n][tb]);
              }
            }
          }
        }
        if constexpr (!SPLIT) {
          asm volatile("" ::: "memory");       // keep the table reads of later rounds from piling up
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int n = 0; n < NG; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * n + i < G) out(sum_rows(s[n][0][i], s[n][1][i], s[n][2][i], s[n][3][i]), hw, 4 * n + i);
    } else if (G <= kVectorHeads) {
#pragma nounroll
      for (int g = 0; g < G; ++g) {
        const float* qs = qw + (hw * G + g) * HD;
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < CBH; ++b) {
          const float4 qv = *reinterpret_cast<const float4*>(qs + P::dim(b, 0));
#pragma unroll
          for (int tb = 0; tb < 4; ++tb) {
            const floatx4_t& k = acc.v[P::block(hw, b)][tb];
            s[tb] = fmaf(qv.x, k[0], s[tb]); s[tb] = fmaf(qv.y, k[1], s[tb]);
            s[tb] = fmaf(qv.z, k[2], s[tb]); s[tb] = fmaf(qv.w, k[3], s[tb]);
          }
        }
        out(sum_rows(s[0], s[1], s[2], s[3]), hw, g);
      }
    } else {
#pragma nounroll
      for (int g0 = 0; g0 < G; g0 += 4) {
        const float* qs = qw + (hw * G + min(g0 + (lane & 3), G - 1)) * HD;      // (heads past the last repeat it)
        floatx4_t s[4];
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) s[tb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < CBH; ++b) {
          const float4 q4 = *reinterpret_cast<const float4*>(qs + P::dim(b, 0));
          const float qv[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) s[tb] = fma_heads(qv[r], acc.v[P::block(hw, b)][tb][r], s[tb]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (g0 + i < G) out(sum_rows(s[0][i], s[1][i], s[2][i], s[3][i]), hw, g0 + i);
      }
    }
  }
  if constexpr (SPLIT) {
    static_assert(ROPE, "the loops over the query heads have to be unrolled");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the copies in flight stay in flight)
    barrier();
#pragma unroll
    for (int hw = 0; hw < P::N; ++hw) {
      if (hw >= nh) continue;
#pragma unroll
      for (int g = 0; g < MG; ++g)
        if (g < G && ((hw + g) & 1) == wc) tail(__uint_as_float(mine[hw][g / 2]) + share[hw * G + g][lane], hw * G + g);
    }
  }
}

// Table entries of a lane from memory (SPLIT): all it needs of its four tokens, requested at once.
template <int HD> struct TableRegs {
  static constexpr int HB = Part<HD, true>::HB;
  float4 cs[HB][4], sn[HB][4];
  __device__ __forceinline__ void load(const KExtra& x, int jw0, int L, int wc, int lane) {
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
      for (int tb = 0; tb < 4; ++tb) {
        const int64_t at = (int64_t)min(jw0 + tb * 16 + (lane & 15), L - 1) * (HD / 2) + wc * (HD / 4) + hb * 16 + 4 * (lane >> 4);
        cs[hb][tb] = *reinterpret_cast<const float4*>(x.cos + at);
        sn[hb][tb] = *reinterpret_cast<const float4*>(x.sin + at);
      }
  }
};
// ... and through LDS, where there is room for the tables of the tile's 256 tokens (the score kernel's stages, once its only pass is
// done): loaded from memory a lane's 16 bytes lie in another row than its neighbour's but three, and the address unit takes
// a row per clock.  Whole calls, value-absorbed, four query heads per KV head, from memory / so, us: 131072 tokens 347 / 343, 60000 with
// twice the predicted dims 223 / 219.  Per 64 tokens cos rows, then sin rows, of HD / 8 16-byte chunks; chunk ch of row r
// sits at ch ^ (r % (HD / 8)): no bank conflicts.  The two waves of a token group copy one table each.
template <int HD>
__device__ __forceinline__ void tables_to_lds(char* smem, const KExtra& x, int jw0, int L, int wt, int wc, int lane) {
  constexpr int CH = HD / 8, RPC = 64 / CH;               // chunks of a row, rows of a copy
  const int jb = min(jw0, L - 1), last = L - 1 - jb;
  const rsrc_t src = make_rsrc((wc ? x.sin : x.cos) + (int64_t)jb * (HD / 2));
#pragma unroll
  for (int i = 0; i < WM / RPC; ++i) {
    const int r = i * RPC + lane / CH;
    copy_to_lds(src, smem + (2 * wt + wc) * (WM * CH * 16) + i * 1024, (uint32_t)(min(r, last) * (HD * 2) + ((lane % CH) ^ (r % CH)) * 16), 0);
  }
}
template <int HD>
__device__ __forceinline__ void table_from_lds(const char* smem, int wt, int lane, int tb, int hb, float4& cs, float4& sn) {
  constexpr int CH = HD / 8;
  const int r = tb * 16 + (lane & 15);
  const char* at = smem + 2 * wt * (WM * CH * 16) + r * (CH * 16) + (((hb * 4 + (lane >> 4)) ^ (r % CH)) << 4);
  cs = *reinterpret_cast<const float4*>(at);
  sn = *reinterpret_cast<const float4*>(at + WM * CH * 16);
}

// Softmax numerators of one (head, query head) pair over the wave's 64 tokens -> pp, (max, sum) -> ml.  v: score of token `lane`.
__device__ __forceinline__ void score_tail(float v, float* pp, float* ml, int lane, int jw0, const KExtra& x) {
  const int tok = jw0 + lane;
  if (tok < x.lo || tok >= x.hi) v = -INFINITY;
  const float mx = wave_max64(v);
  const float p = v == -INFINITY ? 0.f : __expf(v - mx);
  pp[lane] = p;
  const float sum = wave_sum64(p);
  if (lane == 0) { ml[0] = mx; ml[1] = sum; }
}

// After the V pass: acc[cb][tb] holds V_hat; a lane owns tokens 16 tb + 4 (lane / 16) + r of column lane % 16 of the wave's blocks.  Hands out
// sum_j p_j v_hat_j over the wave's 64 tokens for its dims of the tile's nh heads as put(pair, dim, value), every (pair, dim) in one
// lane.  p: the numerators [pair][WM].
template <int HD, bool SPLIT, class Put>
__device__ __forceinline__ void value_sums(const Acc& acc, const float (*p)[WM], int nh, int G, int wc, int lane, Put put) {
  using P = Part<HD, SPLIT>;
  constexpr int CBH = P::CBH, NH = CBH < 4 ? 4 / CBH : 1;        // heads of four blocks
  const int c = lane & 15, o = lane >> 4;
#pragma unroll
  for (int n0 = 0; n0 < 8; n0 += 4) {          // blocks n0 ... n0 + 3, heads after heads
    const int hw0 = n0 / CBH;
    if (P::head(wc, hw0) >= nh) continue;
    if (G <= kVectorHeads) {
#pragma nounroll
      for (int g = 0; g < G; ++g) {
        float out[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tb = 0; tb < 4; ++tb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int hw = (n0 + i) / CBH;
            const float4 pv = *reinterpret_cast<const float4*>(&p[P::head(wc, hw) * G + g][tb * 16 + 4 * o]);
            const floatx4_t& v = acc.v[P::block(hw, (n0 + i) % CBH)][tb];
            out[i] = fmaf(pv.x, v[0], out[i]); out[i] = fmaf(pv.y, v[1], out[i]);
            out[i] = fmaf(pv.z, v[2], out[i]); out[i] = fmaf(pv.w, v[3], out[i]);
          }
        const int head = P::head(wc, (n0 + o) / CBH);        // (row o of 16 lanes has block n0 + o)
        const float v = sum_rows(out[0], out[1], out[2], out[3]);
        if (head < nh) put(head * G + g, P::dim((n0 + o) % CBH, wc) + c, v);
      }
    } else {
#pragma nounroll
      for (int g0 = 0; g0 < G; g0 += 4) {
        const int gl = min(g0 + (lane & 3), G - 1);
        floatx4_t out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
          float pv[NH][4];
#pragma unroll
          for (int j = 0; j < NH; ++j) {
            const float4 p4 = *reinterpret_cast<const float4*>(&p[P::head(wc, hw0 + j) * G + gl][tb * 16 + 4 * o]);
            pv[j][0] = p4.x; pv[j][1] = p4.y; pv[j][2] = p4.z; pv[j][3] = p4.w;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int hw = (n0 + i) / CBH;
              out[i] = fma_heads(pv[hw - hw0][r], acc.v[P::block(hw, (n0 + i) % CBH)][tb][r], out[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int head = P::head(wc, (n0 + i) / CBH);
          const float v = sum_rows(out[i][0], out[i][1], out[i][2], out[i][3]);
          if (head < nh && g0 + o < G) put(head * G + g0 + o, P::dim((n0 + i) % CBH, wc) + c, v);
        }
      }
    }
  }
}

// What a workgroup is about: its tile and the operands of its product.
struct Tile {
  int b, L, j0, n0, wave, lane, wt, wc;
  bool ok;
};
template <bool PACKED, bool SPLIT>
__device__ __forceinline__ Tile make_tile(const Args& a, const SeqMeta& meta, Pipe<PACKED, SPLIT>& pipe, char* smem, int passes, int which, int head_dim) {
  Tile t;
  int ttile, ctile;
  t.ok = tile_of_block(a, ttile, ctile);
  if (!t.ok) return t;
  t.b = find_seq(meta.tbase, meta.n, ttile);
  t.L = meta.len[t.b];
  t.j0 = (ttile - meta.tbase[t.b]) * BM;
  t.n0 = ctile * BN;
  t.lane = threadIdx.x & 63;
  t.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  t.wt = t.wave & 3; t.wc = t.wave >> 2;
  const int64_t row0 = meta.start[t.b] + t.j0;
  const int64_t woff = PACKED ? (int64_t)t.n0 * (a.D + a.m) : t.n0;
  Operands& op = pipe.op;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int s = passes == 2 ? p : which;
    op.xa[p] = a.xa[s] + row0 * a.D; op.xr[p] = a.xr[s] + row0 * a.m; op.w[p] = a.w[s] + woff;
  }
  op.D = a.D; op.m = a.m; op.d_out = a.d_out; op.run = head_dim / 4;
  // rows past the end of the sequence are clamped onto its last valid token, columns past d_out onto
  // the last valid ones, so that what is masked or skipped later is finite
  op.last = min(BM, t.L - t.j0) - 1;
  op.ncol = a.d_out - t.n0;
  op.nk = (a.D + a.m) / BK; op.nka = a.D / BK; op.total = passes * op.nk;
  op.rot = (t.j0 / BM * 3) % op.nk;
  pipe.smem = smem; pipe.wave = t.wave; pipe.lane = t.lane;
  pipe.half = op.ncol <= (SPLIT ? WN : t.wc * WN);
  return t;
}

template <int HD, bool PACKED, bool ROPE>
__global__ __launch_bounds__(NTHREADS) void fused_decode_kernel(Args a, Streams<bf16_t> streams, StreamMeta smeta) {
  __shared__ __attribute__((aligned(1024))) Smem sm;
  const int n_fused = (a.n_tiles + 7) / 8 * 8;
  if ((int)blockIdx.x >= n_fused) {
    stream_workgroup<bf16_t, HD, NWAVES, 8>(streams, smeta, blockIdx.x - n_fused, sm.st);
    return;
  }
  const SeqMeta& meta = smeta.s;
  constexpr bool SPLIT = ROPE;
  Pipe<PACKED, SPLIT> pipe;
  const Tile t = make_tile(a, meta, pipe, sm.st, 2, 0, HD);
  if (!t.ok) return;
  const int kvh0 = a.n_ret_heads + t.n0 / HD, nh = min(BN / HD, (a.d_out - t.n0) / HD);      // first KV head, heads of the tile
  Queries queries;
  queries.load(a.q + ((int64_t)t.b * a.H_q + kvh0 * a.G) * HD, nh * a.G * HD, threadIdx.x);
  pipe.begin();
  queries.store(sm.e.q, a.scale, threadIdx.x);
  pipe.first_landed();                             // (publishes the queries as well)
  const int jw0 = t.j0 + t.wt * WM;                // first token of this wave
  Acc acc;
  // ---- K_hat^T = W_K^T X^T; the last two tiles of the pass request the first two of the V pass
  pipe.template pass<true>(acc, 0);
  const KExtra x = make_kextra(a.rope_cos, a.rope_sin, a.n_sink, a.n_recent, t.L);
  TableRegs<HD> tables;
  if constexpr (ROPE) tables.load(x, jw0, t.L, t.wc, t.lane);
  k_scores<HD, ROPE, SPLIT>(acc, sm.e.q, sm.e.p[t.wt], nh, a.G, t.wc, t.lane,
                            [&](int tb, int hb, float4& cs, float4& sn) __attribute__((always_inline)) { cs = tables.cs[hb][tb]; sn = tables.sn[hb][tb]; },
                            [&](float s, int pair) __attribute__((always_inline)) {
                              score_tail(s, sm.e.p[t.wt][pair], sm.e.ml[t.wt][pair], t.lane, jw0, x);
                            });
  // ---- V_hat = X W_V
  pipe.template pass<false>(acc, pipe.op.nk);
  pipe.drain();
  // ---- the token groups 2 s and 2 s + 1 are the halves of a 128-token slot: all waves put their sums, relative to the larger of
  //      the two maxima, into LDS, and all threads add the halves up on the way out.  (The odd group's handed over first and
  //      the even one's added to them, half of the SIMDs had nothing to do in either half.)
  float (*xo)[2 * MAXPAIR * 128] = reinterpret_cast<float (*)[2 * MAXPAIR * 128]>(sm.st);
  auto rescale = [&](int wt, int pair, float& m) __attribute__((always_inline)) {      // of a group's sums, and the larger maximum
    const float own = sm.e.ml[wt][pair][0];
    m = fmaxf(own, sm.e.ml[wt ^ 1][pair][0]);
    return own == -INFINITY ? 0.f : __expf(own - m);
  };
  if (t.j0 + (t.wt & ~1) * WM < t.L)               // (the slot has a token)
    value_sums<HD, SPLIT>(acc, sm.e.p[t.wt], nh, a.G, t.wc, t.lane, [&](int pair, int dim, float v) __attribute__((always_inline)) {
      float m;
      xo[t.wt][pair * HD + dim] = v * rescale(t.wt, pair, m);
    });
  __syncthreads();
  const int npair = nh * a.G;
  for (int i = t.wave; i < 2 * npair; i += NWAVES) {
    const int s = i >= npair, pair = i - s * npair, w0 = 2 * s, jw = t.j0 + w0 * WM;
    if (jw >= t.L) continue;
    const int64_t ph = (int64_t)(meta.sbase[t.b] + jw / kSlotTokens) * a.H_q + kvh0 * a.G + pair;
#pragma unroll
    for (int dim = 0; dim < HD; dim += 64)
      a.part_o[ph * HD + dim + t.lane] = xo[w0][pair * HD + dim + t.lane] + xo[w0 + 1][pair * HD + dim + t.lane];
    if (t.lane == 0) {
      float m;
      const float l0 = sm.e.ml[w0][pair][1] * rescale(w0, pair, m);
      a.part_ml[ph * 2] = m;
      a.part_ml[ph * 2 + 1] = l0 + sm.e.ml[w0 + 1][pair][1] * rescale(w0 + 1, pair, m);
    }
  }
}

// Key half of the fused kernel on its own: K_hat^T of the tile, then the scaled scores of
// every (head, query head) of the tile written to S^T (base-2 logits: the caller folds log2 e
// into the scale).  Used when the value side is evaluated in the other association order
// (sum_j p_j x^V_j first, W_V afterwards), which stays valid under a rotary embedding.
template <int HD, bool ROPE>
__global__ __launch_bounds__(NTHREADS) void fused_kscores_kernel(Args a, Streams<bf16_t> streams, StreamMeta smeta) {
  __shared__ __attribute__((aligned(1024))) Smem sm;
  const int n_fused = (a.n_tiles + 7) / 8 * 8;
  if ((int)blockIdx.x >= n_fused) {
    score_stream_workgroup<HD, NWAVES>(streams, smeta, blockIdx.x - n_fused, a.s_out, a.s_ld, sm.st);
    return;
  }
  const SeqMeta& meta = smeta.s;
  Pipe<false, false> pipe;
  const Tile t = make_tile(a, meta, pipe, sm.st, 1, 0, HD);
  if (!t.ok) return;
  const int kvh0 = a.n_ret_heads + t.n0 / HD, nh = min(BN / HD, (a.d_out - t.n0) / HD);      // first KV head, heads of the tile
  Queries queries;
  queries.load(a.q + ((int64_t)t.b * a.H_q + kvh0 * a.G) * HD, nh * a.G * HD, threadIdx.x);
  pipe.begin();
  queries.store(sm.e.q, a.scale, threadIdx.x);
  pipe.first_landed();
  Acc acc;
  pipe.template pass<true>(acc, 0);
  const int jw0 = t.j0 + t.wt * WM;
  const KExtra x = make_kextra(a.rope_cos, a.rope_sin, 0, 0, t.L);
  if constexpr (ROPE) {
    pipe.drain();                          // the stages are free
    tables_to_lds<HD>(sm.st, x, jw0, t.L, t.wt, t.wc, t.lane);
    pipe.drain();
  } else {
    wait_copies<0>();                      // the copies past the end land before the workgroup's LDS is released
  }
  float* srow = a.s_out + (int64_t)kvh0 * a.G * a.s_ld + (int64_t)meta.sbase[t.b] * kSlotTokens + jw0 + t.lane;
  if (jw0 >= t.L) return;
  k_scores<HD, ROPE, false>(acc, sm.e.q, nullptr, nh, a.G, t.wc, t.lane, [&](int tb, int hb, float4& cs, float4& sn) __attribute__((always_inline)) {
    table_from_lds<HD>(sm.st, t.wt, t.lane, tb, hb, cs, sn);
  }, [&](float v, int pair) __attribute__((always_inline)) {
    if (jw0 + t.lane < t.L) srow[(int64_t)pair * a.s_ld] = v;
  });
}

// The same streaming workgroups with no product in front of them (every head is retained): four waves and no tiles, so that
// a unit holds several.  Whole calls, as workgroups of the product's kernel / so: 2 x 9496-56976 tokens, two heads of 64, 48.8 / 45.1 us, 29 x
// 53-318 tokens, eight heads of 128 50.5 / 47.4, with rope and window 84 / 76; one sequence of 40000, rope and window 94 / 101 (117 as two launches).
template <int HD>
__global__ __launch_bounds__(64 * kStreamWaves) void score_stream_kernel(Streams<bf16_t> streams, StreamMeta smeta, float* s_out, int64_t s_ld) {
  __shared__ __attribute__((aligned(16))) char smem[stream_smem_bytes<bf16_t, HD, kStreamWaves>()];
  score_stream_workgroup<HD, kStreamWaves>(streams, smeta, blockIdx.x, s_out, s_ld, smem);
}

// K_hat of the tile rotated to its tokens' positions, as store(tile row, column block, four values).  A lane holds dims of a head together
// with their partners, and the table entries serve every head of the tile; those of the next block of 16 tokens are requested ahead
// of this one's rotation.
template <int HD, class Store>
__device__ __forceinline__ void rotate_tile(const Args& a, const Tile& t, const Acc& acc, Store store) {
  using P = Part<HD, true>;
  constexpr int HB = P::HB;
  const int c = t.lane & 15, o = t.lane >> 4, j0 = t.wt * WM;
  float4 cs[2][HB], sn[2][HB];
  auto load = [&](int tb) __attribute__((always_inline)) {
    const int64_t at = (int64_t)min(t.j0 + j0 + tb * 16 + c, t.L - 1) * (HD / 2) + t.wc * (HD / 4) + 4 * o;
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      cs[tb & 1][hb] = *reinterpret_cast<const float4*>(a.rope_cos + at + hb * 16);
      sn[tb & 1][hb] = *reinterpret_cast<const float4*>(a.rope_sin + at + hb * 16);
    }
  };
  load(0);
#pragma unroll
  for (int tb = 0; tb < 4; ++tb) {
    if (t.j0 + j0 + tb * 16 >= t.L) break;               // (uniform: rows past the end are not stored)
    if (tb < 3) load(tb + 1);
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      const float4 cq = cs[tb & 1][hb], sq = sn[tb & 1][hb];
#pragma unroll
      for (int hw = 0; hw < P::N; ++hw) {
        const floatx4_t x = acc.v[P::block(hw, hb)][tb], y = acc.v[P::block(hw, hb + HB)][tb];
        store(j0 + tb * 16 + c, P::block(hw, hb), x[0] * cq.x - y[0] * sq.x, x[1] * cq.y - y[1] * sq.y, x[2] * cq.z - y[2] * sq.z, x[3] * cq.w - y[3] * sq.w);
        store(j0 + tb * 16 + c, P::block(hw, hb + HB), y[0] * cq.x + x[0] * sq.x, y[1] * cq.y + x[1] * sq.y, y[2] * cq.z + x[2] * sq.z, y[3] * cq.w + x[3] * sq.w);
      }
    }
  }
}

// Stand-alone predictor product (Eq. 3) with the same main loop: K_hat or V_hat
// (blockIdx.y) of the tile is rounded to bf16 and stored at
// out[row, col0 + column].  Output row = sbase[b]*kSlotTokens + j.  With an
// activation it is the first layer of the one-hidden-layer predictor
// (Appendix "Prediction Network Architecture").
// The accumulators go through LDS so that rows leave in 16-byte pieces, 512 contiguous bytes per wave and row.
// With rotary tables (a.rope_cos, heads of a.H_q dims) K_hat is rotated to its tokens' positions on that way; further workgroups
// rotate the retained keys (`rope`).
template <int ACT, bool OUT32 = false>   // activation before rounding: 0 none, 1 ReLU, 2 SiLU; OUT32: fp32 output
__global__ __launch_bounds__(NTHREADS) void recon_mfma_kernel(Args a, SeqMeta meta, RopeRows rope) {
  __shared__ __attribute__((aligned(1024))) char st[2 * kStage];
  const int which = blockIdx.y, n_fused = (a.n_tiles + 7) / 8 * 8;
  if ((int)blockIdx.x >= n_fused) {
    if (which == 0) rope_workgroup<NTHREADS>(rope, blockIdx.x - n_fused);
    return;
  }
  Pipe<false, true> pipe;
  const int head_dim = a.H_q == 64 ? 64 : 128;      // (which columns go to which wave matters to the rotation only)
  const Tile t = make_tile(a, meta, pipe, st, 1, which, head_dim);
  if (!t.ok) return;
  pipe.begin();
  pipe.first_landed();
  Acc acc;                                 // rows = columns, lanes = tokens: a lane holds 4 consecutive columns of a token
  pipe.template pass<true>(acc, 0);
  pipe.drain();
  const int lc = t.lane & 15, lo = t.lane >> 4;
  auto column = [&](int cb) __attribute__((always_inline)) { return column_of<true>(head_dim / 4, t.wc, cb >> 2, (cb & 3) * 16); };
  auto act = [](float v) {
    if constexpr (ACT == 1) return fmaxf(v, 0.f);
    else if constexpr (ACT == 2) return v / (1.f + __expf(-v));
    else return v;
  };
  bf16_t* out = which ? a.out[1] : a.out[0];
  const int64_t orow0 = (int64_t)meta.sbase[t.b] * kSlotTokens + t.j0;
  if constexpr (OUT32) {
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
      const int j = t.wt * WM + tb * 16 + lc;
      if (t.j0 + j >= t.L) continue;
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) {
        const int n = t.n0 + column(cb) + lo * 4;
        const floatx4_t v = acc.v[cb][tb];
        if (n < a.d_out)
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + (orow0 + j) * a.ldo + a.col0 + n) =
              make_float4(act(v[0]), act(v[1]), act(v[2]), act(v[3]));
      }
    }
    return;
  }
  // token row: 32 chunks of 16 bytes, chunk ch at ch ^ (token % 32)
  auto store = [&](int j, int cb, float x0, float x1, float x2, float x3) __attribute__((always_inline)) {
    const int ch = column(cb) / 8 + (lo >> 1);
    const u32x2_t w = {pack_bf16(x0, x1), pack_bf16(x2, x3)};
    *reinterpret_cast<u32x2_t*>(st + j * 512 + ((ch ^ (j & 31)) << 4) + (lo & 1) * 8) = w;
  };
  if (which == 0 && a.rope_cos) {
    if (a.H_q == 128) rotate_tile<128>(a, t, acc, store);
    else rotate_tile<64>(a, t, acc, store);
  } else {
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
      if (t.j0 + t.wt * WM + tb * 16 >= t.L) break;      // (uniform: rows past the end are not stored)
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) {
        const floatx4_t v = acc.v[cb][tb];
        store(t.wt * WM + tb * 16 + lc, cb, act(v[0]), act(v[1]), act(v[2]), act(v[3]));
      }
    }
  }
  __syncthreads();
  const int c = threadIdx.x & 31, n = t.n0 + c * 8;
  if (n >= a.d_out) return;
  for (int j = threadIdx.x >> 5; j < BM && t.j0 + j < t.L; j += NTHREADS / 32)
    *reinterpret_cast<u32x4_t*>(out + (orow0 + j) * a.ldo + a.col0 + n) =
        *reinterpret_cast<const u32x4_t*>(st + j * 512 + ((c ^ (j & 31)) << 4));
}

}  // namespace fused

// ---- host-side launchers ------------------------------------------------------------
// Paper-faithful extras of a decode call as the launchers take them (all zero: off).
struct KvExtras {
  const float* rope_cos = nullptr; const float* rope_sin = nullptr;
  int n_sink = 0, n_recent = 0;
};

template <typename T> inline bool fused_decode_supported(int d, int G) {
  return (d == 64 || d == 128) && (128 / d) * G <= fused::MAXPAIR;
}
template <typename T> inline bool recon_mfma_supported() { return sizeof(T) == 2; }

inline int fused_fill_tiles(SeqMeta& mt) {
  int acc = 0;
  for (int b = 0; b < mt.n; ++b) { mt.tbase[b] = acc; acc += (mt.len[b] + fused::BM - 1) / fused::BM; }
  mt.tbase[mt.n] = acc;
  return acc;
}

template <typename T>
inline int launch_fused_decode(int H_q, int H_kv, int d, int m, int d_out, int n_ret_heads,
                               float scale, const T* ka,
                               const T* va, const T* kr, const T* vr, const T* wk, const T* wv,
                               const T* q, float* part_o, float* part_ml, StreamMeta& smt,
                               int* fused_step, hipStream_t st, const Streams<T>& streams, bool packed = false,
                               const KvExtras& ex = KvExtras(), int x_width = 0) {
  if constexpr (sizeof(T) != 2) {
    return 6;
  } else {
    SeqMeta& mt = smt.s;
    fused::Args a;
    a.rope_cos = ex.rope_cos; a.rope_sin = ex.rope_sin; a.n_sink = ex.n_sink; a.n_recent = ex.n_recent;
    a.s_out = nullptr; a.s_ld = 0;
    a.xa[0] = ka; a.xa[1] = va; a.xr[0] = kr; a.xr[1] = vr; a.w[0] = wk; a.w[1] = wv;
    a.q = q; a.part_o = part_o; a.part_ml = part_ml;
    a.out[0] = a.out[1] = nullptr; a.ldo = 0; a.col0 = 0;
    a.D = H_kv * d; a.m = m; a.d_out = d_out; a.H_q = H_q; a.G = H_q / H_kv;
    if (x_width > 0) { a.D = x_width; a.m = 0; }     // predictor input = one matrix of that width (ka / va)
    a.n_ret_heads = n_ret_heads; a.scale = scale;
    a.n_col_tiles = (a.d_out + fused::BN - 1) / fused::BN;
    a.n_tiles = fused_fill_tiles(mt) * a.n_col_tiles;
    const int grid = ((a.n_tiles + 7) / 8) * 8 + streams.n_ret + streams.n_win;
    const dim3 g(grid), blk(fused::NTHREADS);
    const bool rope = ex.rope_cos != nullptr;
#define ECHOKV_FUSED_CASE(HD_, PK_) \
    do { if (rope) hipLaunchKernelGGL((fused::fused_decode_kernel<HD_, PK_, true>), g, blk, 0, st, a, streams, smt); \
         else hipLaunchKernelGGL((fused::fused_decode_kernel<HD_, PK_, false>), g, blk, 0, st, a, streams, smt); } while (0)
    if (d == 128 && packed) ECHOKV_FUSED_CASE(128, true);
    else if (d == 128) ECHOKV_FUSED_CASE(128, false);
    else if (packed) ECHOKV_FUSED_CASE(64, true);
    else ECHOKV_FUSED_CASE(64, false);
#undef ECHOKV_FUSED_CASE
    if (hipGetLastError() != hipSuccess) return 7;
    *fused_step = 1;
    return 0;
  }
}

// Scores of the predicted heads -> s_out (see fused_kscores_kernel).  `scale` must already
// include log2(e).
template <typename T>
inline int launch_fused_kscores(int H_q, int H_kv, int d, int m, int d_out, int n_ret_heads,
                                float scale, const T* ka, const T* kr, const T* wk, const T* q,
                                float* s_out, int64_t s_ld, StreamMeta& smt, hipStream_t st,
                                const Streams<T>& streams, const KvExtras& ex) {
  if constexpr (sizeof(T) != 2) {
    return 6;
  } else {
    SeqMeta& mt = smt.s;
    fused::Args a;
    a.xa[0] = a.xa[1] = ka; a.xr[0] = a.xr[1] = kr; a.w[0] = a.w[1] = wk;
    a.q = q; a.part_o = nullptr; a.part_ml = nullptr;
    a.out[0] = a.out[1] = nullptr; a.ldo = 0; a.col0 = 0;
    a.D = H_kv * d; a.m = m; a.d_out = d_out; a.H_q = H_q; a.G = H_q / H_kv;
    a.n_ret_heads = n_ret_heads; a.scale = scale;
    a.rope_cos = ex.rope_cos; a.rope_sin = ex.rope_sin; a.n_sink = 0; a.n_recent = 0;
    a.s_out = s_out; a.s_ld = s_ld;
    a.n_col_tiles = (a.d_out + fused::BN - 1) / fused::BN;
    a.n_tiles = fused_fill_tiles(mt) * a.n_col_tiles;
    if (a.n_tiles == 0) {                    // every head is retained
      const dim3 sg(streams.n_ret + streams.n_win), sb(64 * kStreamWaves);
      if (d == 128) hipLaunchKernelGGL((fused::score_stream_kernel<128>), sg, sb, 0, st, streams, smt, s_out, s_ld);
      else hipLaunchKernelGGL((fused::score_stream_kernel<64>), sg, sb, 0, st, streams, smt, s_out, s_ld);
      return hipGetLastError() != hipSuccess ? 7 : 0;
    }
    const dim3 g((a.n_tiles + 7) / 8 * 8 + streams.n_ret + streams.n_win), blk(fused::NTHREADS);
    const bool rope = ex.rope_cos != nullptr;
    if (d == 128 && rope) hipLaunchKernelGGL((fused::fused_kscores_kernel<128, true>), g, blk, 0, st, a, streams, smt);
    else if (d == 128) hipLaunchKernelGGL((fused::fused_kscores_kernel<128, false>), g, blk, 0, st, a, streams, smt);
    else if (rope) hipLaunchKernelGGL((fused::fused_kscores_kernel<64, true>), g, blk, 0, st, a, streams, smt);
    else hipLaunchKernelGGL((fused::fused_kscores_kernel<64, false>), g, blk, 0, st, a, streams, smt);
    if (hipGetLastError() != hipSuccess) return 7;
    return 0;
  }
}

// K_hat and V_hat of the sequences in `mt` -> out_k / out_v [rows, ldo] at
// column col0, output row = sbase[b]*kSlotTokens + j.  d_out = width of W (0: only the rows of `rope`).  With
// rope.cos K_hat is rotated by token position on its way out, heads of rope.d dims, and rope's own rows (the retained keys) are as well, by
// workgroups of the product's launch.  (A launch behind the product for K_hat won for fewer than 120 of its workgroups while the rotation was done on
// rounded rows from LDS.  Behind the product / on its way out of the accumulators, whole prefill calls of 32 heads over 8 of 128, us, and the product's
// workgroups: m = 512, 16 queries behind 500 tokens (12) 52.8 / 52.4, 100 behind 3000 (52) 65.5 / 64.9, 2000 alone (32) 103.8 / 102.8; m = 64,
// 100 behind 3000 (104) 60.3 / 58.7; 32 over 32, m = 2048, 300 behind 600 (64) 139.5 / 138.1.)
template <typename T>
inline int launch_recon_mfma(int D, int m, int d_out, const T* ka, const T* va, const T* kr, const T* vr,
                             const T* wk, const T* wv, T* out_k, T* out_v, int64_t ldo, int col0,
                             SeqMeta& mt, hipStream_t st, int act = 0, bool out_f32 = false,
                             const RopeRows& rope = RopeRows()) {
  if constexpr (sizeof(T) != 2) {
    return 6;
  } else {
    fused::Args a;
    a.xa[0] = ka; a.xa[1] = va; a.xr[0] = kr; a.xr[1] = vr; a.w[0] = wk; a.w[1] = wv;
    a.q = nullptr; a.part_o = nullptr; a.part_ml = nullptr;
    a.rope_cos = rope.cos; a.rope_sin = rope.sin; a.n_sink = a.n_recent = 0; a.s_out = nullptr; a.s_ld = 0;
    a.out[0] = out_k; a.out[1] = out_v; a.ldo = ldo; a.col0 = col0;
    a.D = D; a.m = m; a.d_out = d_out; a.H_q = rope.d; a.G = 1; a.n_ret_heads = 0; a.scale = 0.f;
    a.n_col_tiles = (a.d_out + fused::BN - 1) / fused::BN;
    a.n_tiles = fused_fill_tiles(mt) * a.n_col_tiles;
    const dim3 g((unsigned)((a.n_tiles + 7) / 8 * 8 + rope_workgroups(rope, fused::NTHREADS)), 2), blk(fused::NTHREADS);
    if (out_f32) hipLaunchKernelGGL((fused::recon_mfma_kernel<0, true>), g, blk, 0, st, a, mt, rope);
    else if (act == 1) hipLaunchKernelGGL(fused::recon_mfma_kernel<1>, g, blk, 0, st, a, mt, rope);
    else if (act == 2) hipLaunchKernelGGL(fused::recon_mfma_kernel<2>, g, blk, 0, st, a, mt, rope);
    else hipLaunchKernelGGL(fused::recon_mfma_kernel<0>, g, blk, 0, st, a, mt, rope);
    if (hipGetLastError() != hipSuccess) return 7;
    return 0;
  }
}

}  // namespace echokv
