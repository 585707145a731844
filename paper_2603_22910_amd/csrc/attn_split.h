// Split-K streaming decode attention over heads that are stored as rows: the target layer's
// retained heads, materialised predicted heads, or the uncompressed window.
#pragma once
#include "common.h"

namespace echokv {

// ---------------------------------------------------------------------------
// Uncompressed window of the target layer (the first n_sink positions and a
// ring of the n_recent latest, Sec. "Experimental Setting", paragraph "Implement details"): position p lives in
// row p (p < n_sink) or n_sink + (p - n_sink) % n_recent.
// ---------------------------------------------------------------------------
struct Window {
  int32_t n_sink, n_recent;      // n_sink + n_recent == 0: no window
  __host__ __device__ int rows() const { return n_sink + n_recent; }
  __host__ __device__ bool on() const { return n_sink + n_recent > 0; }
  // compressed-cache tokens [lo, hi) of a length-L sequence are NOT in the window
  __host__ __device__ int lo(int L) const { return on() ? (n_sink < L ? n_sink : L) : 0; }
  __host__ __device__ int hi(int L) const {
    if (!on()) return L;
    const int h = L - n_recent, l = lo(L);
    return h > l ? h : l;
  }
  __host__ __device__ int row_of(int p) const { return p < n_sink ? p : n_sink + (p - n_sink) % n_recent; }
  // position held by window row w of a length-L sequence, or -1 if the row is empty / stale
  __host__ __device__ int pos_of(int w, int L) const {
    if (w < n_sink) return w < L ? w : -1;
    if (n_recent == 0) return -1;
    const int t = L - 1 - n_sink, r = w - n_sink;      // ring coordinates of the last token, of the row
    if (t < 0) return -1;
    int back = (t - r) % n_recent;
    if (back < 0) back += n_recent;
    return t - back >= 0 ? n_sink + t - back : -1;
  }
};

// ---------------------------------------------------------------------------
// Split-K streaming attention over heads that are stored somewhere as rows
// (the target layer's retained heads, or materialised predicted heads):
// scores, online softmax and P.V for GT query heads of one KV head over one
// chunk of `split_tokens` tokens (Eq. 7).  Writes one partial
// (max, sum-exp, unnormalised o) per (chunk, query head).
//   LPR = lanes that share one row = d * sizeof(T) / 16.
// grid.x = chunks (tbase), grid.y = kv heads handled * (G / GT).
// ---------------------------------------------------------------------------
template <typename T>
struct AttnArgs {
  const T* k; const T* v;   // row r, head g at k + r*ld + col0 + g_local*d
  int64_t ld;
  int32_t col0;             // column of the first head handled
  int32_t head0;            // its KV head index (for the query / output head)
  int32_t row_mode;         // 0: row = start[b] + j ; 1: sbase[b]*kSlotTokens + j ; 2: j ;
                            // 3: window rows, row = (seq0 + b) * win.rows() + j, one chunk per sequence
  const T* q;               // [nseq, H_q, d]
  int32_t H_q, G, d;
  float scale;
  int32_t split_tokens;     // multiple of kSlotTokens
  float* part_o;            // [slots, H_q, d]
  float* part_ml;           // [slots, H_q, 2]
  int32_t slot_tokens = kSlotTokens;   // tokens per slot of SeqMeta::sbase (split_tokens is a multiple)
  // paper-faithful extras: rotary tables [positions, d/2] (null: none) applied to the key rows by
  // token position; window: modes 0-2 skip the tokens the window holds, mode 3 attends them
  const float* rope_cos = nullptr; const float* rope_sin = nullptr;
  Window win = {0, 0};
  int32_t seq0 = 0;         // mode 3: index of the launch's first sequence in the window buffers
  int32_t win_slot0 = 0;    // mode 3: partial of sequence b goes to slot win_slot0 + b
};

// LDS of one attn_split_body: per wave and query head the max, the sum and the o row.
template <typename T, int LPR, int GT, int NWAVES>
constexpr int attn_split_smem_bytes() { return NWAVES * GT * (2 + LPR * Elem<T>::kVec) * 4; }

// Tokens and rows of one workgroup's chunk.
struct ChunkRows {
  int64_t row0;             // pool row of token 0
  int beg, end;             // the compressed rows outside the window, or all window rows
  bool window;
  template <typename T>
  __device__ __forceinline__ ChunkRows(const AttnArgs<T>& a, const SeqMeta& meta, int b, int chunk, int L) {
    window = a.row_mode == 3;
    row0 = a.row_mode == 0 ? meta.start[b]
         : a.row_mode == 1 ? (int64_t)meta.sbase[b] * kSlotTokens
         : window ? (int64_t)(a.seq0 + b) * a.win.rows() : 0;
    beg = window ? 0 : max(chunk * a.split_tokens, a.win.lo(L));
    end = window ? a.win.rows() : min(a.win.hi(L), chunk * a.split_tokens + a.split_tokens);
  }
};
// The waves' sums of GT query heads, in LDS relative to their maxima, added up and written as one partial.
template <int GT, int NWAVES, int ROW, typename T>
__device__ __forceinline__ void write_chunk_partial(const AttnArgs<T>& a, const SeqMeta& meta, int b, int chunk, int qh0,
                                                    const float (*s_m)[GT], const float (*s_l)[GT], const float (*s_o)[GT][ROW]) {
  __syncthreads();
  const int slot = a.row_mode == 3 ? a.win_slot0 + b : meta.sbase[b] + chunk * (a.split_tokens / a.slot_tokens);
  for (int idx = threadIdx.x; idx < GT * a.d; idx += 64 * NWAVES) {
    const int g = idx / a.d, c = idx % a.d;
    float M = s_m[0][g];
#pragma unroll
    for (int w = 1; w < NWAVES; ++w) M = fmaxf(M, s_m[w][g]);
    float l = 0.f, acc = 0.f;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
      const float e = (s_m[w][g] == -INFINITY) ? 0.f : __expf(s_m[w][g] - M);
      l += s_l[w][g] * e; acc += s_o[w][g][c] * e;
    }
    const int64_t ph = (int64_t)slot * a.H_q + qh0 + g;
    a.part_o[ph * a.d + c] = acc;
    if (c == 0) { a.part_ml[ph * 2] = M; a.part_ml[ph * 2 + 1] = l; }
  }
}

// Sums over the four lanes of a quad of four values: lane i of it ends up with the sum of the i-th.
__device__ __forceinline__ float sum_quad4(float t0, float t1, float t2, float t3, int lane) {
  const bool odd = lane & 1, high = lane & 2;
  const float a0 = (odd ? t1 : t0) + dpp_move<0xB1>(odd ? t0 : t1), a1 = (odd ? t3 : t2) + dpp_move<0xB1>(odd ? t2 : t3);
  return (high ? a1 : a0) + dpp_move<0x4E>(high ? a0 : a1);
}

// One workgroup (see attn_split_body) for four query heads of a KV head and bf16 rows of 128 dims.  What bounds it: with rotary tables, the vector unit: a row is 16
// lanes of 8 dims, and scores, softmax and value sums of four heads in each of them were 200 instructions per row.  Here lane % 4
// stands for the query head wherever a value is the same for all lanes of a row: the scores' sums end there (11 instructions instead of 16), the
// softmax is worked out once per quad instead of four times, the values are multiplied four heads at a time by v_mfma_f32_4x4x1
// (fma_heads), rotation partners, eight lanes away, come by row rotation instead of through LDS.
// Whole calls, 32 heads over 8, before / so, us: 8 x 2048-36864 tokens, 3 heads retained, rope and window 292 / 285, 2 x 40000, 4 retained, the same
// 283 / 274, without rope 260 / 248, 8 x 6000, 7 retained, rope 135 / 120; 64 heads over 8, 4 x 5000, 4 retained, rope 93.9 / 83.6.  Rows of
// 64 dims, whose quads are two to a row, lose what they win (4 x 5000 tokens 23.8 / 24.6): attn_split_body_any.
template <int NWAVES, int UN>
__device__ __forceinline__ void attn_split_body4(const AttnArgs<bf16_t>& a, const SeqMeta& meta, int b, int chunk, int y, char* smem) {
  constexpr int GT = 4, LPR = 16, RPW = 64 / LPR, NRG = NWAVES * RPW;
  const int L = meta.len[b];
  const int gchunks = a.G / GT, hl = y / gchunks;
  const int qh0 = (a.head0 + hl) * a.G + (y % gchunks) * GT;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rl = lane / LPR, li = lane % LPR;
  const ChunkRows rows(a, meta, b, chunk, L);
  const int col = a.col0 + hl * a.d + li * 8;
  const bool rope = a.rope_cos != nullptr;
  const int hc = (li % (LPR / 2)) * 8;            // this lane's first column in the d/2-wide tables
  const float sgn = (li < LPR / 2) ? -1.f : 1.f;
  float qv[GT][8];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    load16<bf16_t>(a.q + ((int64_t)b * a.H_q + qh0 + g) * a.d + li * 8, qv[g]);
#pragma unroll
    for (int i = 0; i < 8; ++i) qv[g][i] *= a.scale;
  }
  float mx = -INFINITY, sm = 0.f;                 // of query head lane % 4, this lane's row group
  floatx4_t o[8];                                 // [dim][query head]
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // (uniform: MFMAs take all lanes, so row groups past the end go on with rows that count for nothing)
  for (int jb = rows.beg + wave * RPW; jb < rows.end; jb += NRG * UN) {
    uint4 kr[UN], vr[UN];
    int pos[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int j = jb + rl + u * NRG, jj = min(j, rows.end - 1);
      kr[u] = *reinterpret_cast<const uint4*>(a.k + (rows.row0 + jj) * a.ld + col);
      vr[u] = *reinterpret_cast<const uint4*>(a.v + (rows.row0 + jj) * a.ld + col);
      pos[u] = rows.window ? a.win.pos_of(jj, L) : jj;
      if (j >= rows.end) pos[u] = -1;
    }
    float sc[UN], mn = mx;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      float k[8];
      unpack_bf16x8(kr[u], k);
      if (rope) {        // feature i pairs with i + d/2, held by the lane LPR / 2 away
        const int64_t at = (int64_t)max(pos[u], 0) * (a.d / 2) + hc;
        float cs[8], sn[8];
#pragma unroll
        for (int i = 0; i < 8; i += 4) {
          const float4 c4 = *reinterpret_cast<const float4*>(a.rope_cos + at + i), s4 = *reinterpret_cast<const float4*>(a.rope_sin + at + i);
          cs[i] = c4.x; cs[i + 1] = c4.y; cs[i + 2] = c4.z; cs[i + 3] = c4.w;
          sn[i] = s4.x; sn[i + 1] = s4.y; sn[i + 2] = s4.z; sn[i + 3] = s4.w;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float other = dpp_move<0x128>(k[i]);      // rotate the row by 8
          k[i] = fmaf(k[i], cs[i], sgn * other * sn[i]);
        }
      }
      float t[GT];
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        t[g] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) t[g] = fmaf(qv[g][i], k[i], t[g]);
      }
      float s = sum_quad4(t[0], t[1], t[2], t[3], lane);
      s += dpp_move<0x124>(s);                    // rotate the row by 4, by 8
      s += dpp_move<0x128>(s);
      sc[u] = pos[u] >= 0 ? s : -INFINITY;
      mn = fmaxf(mn, sc[u]);
    }
    const float ref = mn == -INFINITY ? 0.f : mn;
    const float corr = __expf(mx - ref);          // mx = -inf at the start: 0, and o, sm are 0
    float p[UN], ps = 0.f;
#pragma unroll
    for (int u = 0; u < UN; ++u) { p[u] = __expf(sc[u] - ref); ps += p[u]; }     // a dead row: exp(-inf) = 0
    sm = sm * corr + ps;
    mx = mn;
    const float c0 = dpp_move<0x00>(corr), c1 = dpp_move<0x55>(corr), c2 = dpp_move<0xAA>(corr), c3 = dpp_move<0xFF>(corr);
#pragma unroll
    for (int i = 0; i < 8; ++i) { o[i][0] *= c0; o[i][1] *= c1; o[i][2] *= c2; o[i][3] *= c3; }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      float v[8];
      const uint32_t m = pos[u] >= 0 ? ~0u : 0u;  // (0 times what a dead row holds may not be 0)
      unpack_bf16x8(make_uint4(vr[u].x & m, vr[u].y & m, vr[u].z & m, vr[u].w & m), v);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = fma_heads(p[u], v[i], o[i]);
    }
  }
  // merge the row groups: first inside the wave, then across waves in LDS
  float (*s_m)[GT] = reinterpret_cast<float (*)[GT]>(smem);
  float (*s_l)[GT] = s_m + NWAVES;
  float (*s_o)[GT][LPR * 8] = reinterpret_cast<float (*)[GT][LPR * 8]>(s_l + NWAVES);
  float M = mx;
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
  const float w = mx == -INFINITY ? 0.f : __expf(mx - M);
  float l = sm * w;
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1) l += __shfl_xor(l, off, 64);
  if (lane < GT) { s_m[wave][lane] = M; s_l[wave][lane] = l; }
  const float w0 = dpp_move<0x00>(w), w1 = dpp_move<0x55>(w), w2 = dpp_move<0xAA>(w), w3 = dpp_move<0xFF>(w);
  float r[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    r[i] = sum_rows(o[i][0] * w0, o[i][1] * w1, o[i][2] * w2, o[i][3] * w3);      // row g of 16 lanes: query head g
  }
  float* dst = &s_o[wave][lane >> 4][li * 8];
  *reinterpret_cast<float4*>(dst) = make_float4(r[0], r[1], r[2], r[3]);
  *reinterpret_cast<float4*>(dst + 4) = make_float4(r[4], r[5], r[6], r[7]);
  write_chunk_partial<GT, NWAVES, LPR * 8>(a, meta, b, chunk, qh0, s_m, s_l, s_o);
}

// The same for any number of query heads, rows and type.
template <typename T, int LPR, int GT, int NWAVES, int UN>
__device__ __forceinline__ void attn_split_body_any(const AttnArgs<T>& a, const SeqMeta& meta, int b, int chunk,
                                                    int y, char* smem) {
  constexpr int VEC = Elem<T>::kVec;
  constexpr int RPW = 64 / LPR;        // row groups per wave
  constexpr int NRG = NWAVES * RPW;    // row groups per block
  const int L = meta.len[b];
  const int gchunks = a.G / GT;
  const int hl = y / gchunks;                    // local kv head
  const int qh0 = (a.head0 + hl) * a.G + (y % gchunks) * GT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rg = wave * RPW + lane / LPR;        // row group in block
  const int li = lane % LPR;                     // lane within row
  const ChunkRows rows(a, meta, b, chunk, L);
  const bool wmode = rows.window;
  const int64_t row0 = rows.row0;
  const int col = a.col0 + hl * a.d + li * VEC;
  const int jbeg = rows.beg, jend = rows.end;
  const bool rope = a.rope_cos != nullptr;
  const int hc = (li % (LPR / 2)) * VEC;          // this lane's first column in the d/2-wide tables

  float qv[GT][VEC];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    load16<T>(a.q + ((int64_t)b * a.H_q + qh0 + g) * a.d + li * VEC, qv[g]);
#pragma unroll
    for (int i = 0; i < VEC; ++i) qv[g][i] *= a.scale;
  }
  float mx[GT], sm[GT], o[GT][VEC];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    mx[g] = -INFINITY; sm[g] = 0.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i) o[g][i] = 0.f;
  }
  for (int j = jbeg + rg; j < jend; j += NRG * UN) {
    float kv[UN][VEC], vv[UN][VEC];
    int pos[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int jj = min(j + u * NRG, jend - 1);
      load16<T>(a.k + (row0 + jj) * a.ld + col, kv[u]);
      uint4 vr = *reinterpret_cast<const uint4*>(a.v + (row0 + jj) * a.ld + col);
      pos[u] = wmode ? a.win.pos_of(jj, L) : jj;
      if (j + u * NRG >= jend) pos[u] = -1;
      const uint32_t m = pos[u] >= 0 ? ~0u : 0u;      // (0 times what a dead row holds may not be 0)
      vr.x &= m; vr.y &= m; vr.z &= m; vr.w &= m;
      unpack16<T>(vr, vv[u]);
      if (rope) {        // feature i pairs with i + d/2, held by the lane LPR / 2 away
        const int pr = max(pos[u], 0);
        float cs[VEC], sn[VEC];
#pragma unroll
        for (int i = 0; i < VEC; i += 4) {
          const float4 c4 = *reinterpret_cast<const float4*>(a.rope_cos + (int64_t)pr * (a.d / 2) + hc + i);
          const float4 s4 = *reinterpret_cast<const float4*>(a.rope_sin + (int64_t)pr * (a.d / 2) + hc + i);
          cs[i] = c4.x; cs[i + 1] = c4.y; cs[i + 2] = c4.z; cs[i + 3] = c4.w;
          sn[i] = s4.x; sn[i + 1] = s4.y; sn[i + 2] = s4.z; sn[i + 3] = s4.w;
        }
        const float sgn = (li < LPR / 2) ? -1.f : 1.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          const float other = __shfl_xor(kv[u][i], LPR / 2, 64);
          kv[u][i] = fmaf(kv[u][i], cs[i], sgn * other * sn[i]);
        }
      }
    }
    // scores of the round's UN rows, then ONE change of the softmax reference per query head and
    // round (one correction factor instead of one per row)
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      float sc[UN];
      float mn = mx[g];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) t = fmaf(qv[g][i], kv[u][i], t);
        t = row_sum<LPR>(t);
        sc[u] = pos[u] >= 0 ? t : -INFINITY;
        mn = fmaxf(mn, sc[u]);
      }
      if (mn != -INFINITY) {                       // (uniform over the lanes of a row)
        const float corr = __expf(mx[g] - mn);     // mx = -inf at the start: 0, and o, sm are 0
        float p[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) p[u] = __expf(sc[u] - mn);     // a dead row: exp(-inf) = 0
        float ps = (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
        for (int u = 4; u < UN; u += 4) ps += (p[u] + p[u + 1]) + (p[u + 2] + p[u + 3]);
        sm[g] = sm[g] * corr + ps;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          float t = o[g][i] * corr;
#pragma unroll
          for (int u = 0; u < UN; ++u) t = fmaf(p[u], vv[u][i], t);
          o[g][i] = t;
        }
        mx[g] = mn;
      }
    }
  }
  // merge the NRG row groups: first inside the wave, then across waves in LDS
  float (*s_m)[GT] = reinterpret_cast<float (*)[GT]>(smem);
  float (*s_l)[GT] = s_m + NWAVES;
  float (*s_o)[GT][LPR * VEC] = reinterpret_cast<float (*)[GT][LPR * VEC]>(s_l + NWAVES);
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    float M = mx[g];
    for (int off = LPR; off < 64; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    const float w = (mx[g] == -INFINITY) ? 0.f : __expf(mx[g] - M);
    float l = sm[g] * w;
    for (int off = LPR; off < 64; off <<= 1) l += __shfl_xor(l, off, 64);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      float x = o[g][i] * w;
      for (int off = LPR; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
      o[g][i] = x;
    }
    if (lane < LPR) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) s_o[wave][g][li * VEC + i] = o[g][i];
    }
    if (lane == 0) { s_m[wave][g] = M; s_l[wave][g] = l; }
  }
  write_chunk_partial<GT, NWAVES, LPR * VEC>(a, meta, b, chunk, qh0, s_m, s_l, s_o);
}
// One workgroup of NWAVES waves: chunk `chunk` of sequence b, y = KV head * (G / GT) + group of query heads.
// UN: rows of a row group in flight (4; 8 where few waves share a compute unit).
template <typename T, int LPR, int GT, int NWAVES, int UN = 4>
__device__ __forceinline__ void attn_split_body(const AttnArgs<T>& a, const SeqMeta& meta, int b, int chunk, int y, char* smem) {
  if constexpr (GT == 4 && LPR == 16 && sizeof(T) == 2) attn_split_body4<NWAVES, UN>(a, meta, b, chunk, y, smem);
  else attn_split_body_any<T, LPR, GT, NWAVES, UN>(a, meta, b, chunk, y, smem);
}
// Waves of a SIMD that the kernels of streaming workgroups alone are compiled for: nothing but other waves hides the wait for their rows.  Left to
// itself the compiler takes 204 registers for attn_split_body4 (copies of its accumulators; 144 so), which leaves two.  Two / three, 8 KV heads, whole
// calls, us: all 8 retained, 8 x 8000 tokens 67.8 / 62.0, with rope and window 113 / 97.3; 64 query heads, 16 x 3000 with rope 116 / 94.4.
constexpr int kStreamOccupancy = 3;
template <typename T, int LPR, int GT>
__global__ __launch_bounds__(256, kStreamOccupancy) void attn_split_kernel(AttnArgs<T> a, SeqMeta meta) {
  __shared__ __attribute__((aligned(16))) char smem[attn_split_smem_bytes<T, LPR, GT, 4>()];
  const int b = find_seq(meta.tbase, meta.n, blockIdx.x);
  attn_split_body<T, LPR, GT, 4>(a, meta, b, blockIdx.x - meta.tbase[b], blockIdx.y, smem);
}


// The streaming part of a decode call as further workgroups of another kernel's launch: the retained heads
// (one workgroup per chunk of split_tokens, KV head and group of query heads), then the window's rows.
struct StreamMeta {
  SeqMeta s;
  int32_t cbase[kMaxSeqPerLaunch + 1];        // prefix sum of the retained heads' chunks per sequence
};
template <typename T> struct Streams {
  AttnArgs<T> ret, win;
  int32_t n_ret_chunks = 1, n_ret = 0, n_win = 0;     // chunks of all sequences; workgroups
};
template <typename T, int HD, int NWAVES, int GT = 4>
constexpr int stream_smem_bytes() { return attn_split_smem_bytes<T, HD * (int)sizeof(T) / 16, GT, NWAVES>(); }
// Chunk x and head group y of workgroup wg, n chunks x ny groups: the groups of a chunk follow each other 8
// workgroups apart, on one XCD and at one time, so that its L2 has the chunk's rows (whose heads lie side by side) and rotary
// tables already.  One head after the other, 131072 tokens with four retained heads read their tables, half
// the bytes of the rows, four times from memory (the whole call 368 us, like this 351).
__device__ __forceinline__ void stream_item(int wg, int n, int ny, int& x, int& y) {
  const int full = n & ~7;
  if (wg < full * ny) {
    const int r = wg % (8 * ny);
    x = wg / (8 * ny) * 8 + (r & 7); y = r >> 3;
  } else {
    wg -= full * ny;
    x = full + wg % (n - full); y = wg / (n - full);
  }
}
// Query heads of a KV head that share a workgroup's pass over its rows.
__host__ __device__ inline int stream_heads(int G) { return G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1; }
// GT: query heads that share a pass over the rows, 0: by the number of them per KV head.
template <typename T, int HD, int NWAVES, int UN, int GT = 0>
__device__ __forceinline__ void stream_workgroup(const Streams<T>& st, const StreamMeta& meta, int wg, char* smem) {
  const bool ret = wg < st.n_ret;
  if (!ret) wg -= st.n_ret;
  const AttnArgs<T> a = ret ? st.ret : st.win;
  const int n = ret ? st.n_ret_chunks : meta.s.n;
  int x, y;
  stream_item(wg, n, (ret ? st.n_ret : st.n_win) / n, x, y);
  const int b = ret ? find_seq(meta.cbase, meta.s.n, x) : x;
  const int chunk = ret ? x - meta.cbase[b] : 0;
  constexpr int LPR = HD * (int)sizeof(T) / 16;
  const int gt = GT ? GT : stream_heads(a.G);
  if (gt == 4) attn_split_body<T, LPR, 4, NWAVES, UN>(a, meta.s, b, chunk, y, smem);
  else if (gt == 2) attn_split_body<T, LPR, 2, NWAVES, UN>(a, meta.s, b, chunk, y, smem);
  else attn_split_body<T, LPR, 1, NWAVES, UN>(a, meta.s, b, chunk, y, smem);
}

// The same workgroups in a launch of their own: four waves each, so that a unit holds several.  A kernel for each GT, as one for all has the
// registers of the largest: one query head takes 111, two 124 (four waves, either), four 145.  A kernel for all with 205 / so, us: 32 heads, 31 of them retained, 8 x
// 8000 tokens, rope and window 655 / 578; 24 heads over 8, 7 retained, 8 x 8000 219 / 169, with rope and window 282 / 213; 56 over 8, 6 retained, 8 x 2000-12000
// the same 287 / 223.
constexpr int kStreamWaves = 4;
template <typename T, int HD, int GT>
__global__ __launch_bounds__(64 * kStreamWaves, kStreamOccupancy) void stream_kernel(Streams<T> st, StreamMeta meta) {
  __shared__ __attribute__((aligned(16))) char smem[stream_smem_bytes<T, HD, kStreamWaves, GT>()];
  stream_workgroup<T, HD, kStreamWaves, 4, GT>(st, meta, blockIdx.x, smem);
}
template <typename T>
inline int launch_streams(const Streams<T>& s, const StreamMeta& meta, hipStream_t st) {
  const dim3 grid(s.n_ret + s.n_win), blk(64 * kStreamWaves);
  const int gt = stream_heads(s.ret.G);
  auto launch = [&](auto* kernel) { hipLaunchKernelGGL(kernel, grid, blk, 0, st, s, meta); };
  if (s.ret.d == 128) launch(gt == 4 ? stream_kernel<T, 128, 4> : gt == 2 ? stream_kernel<T, 128, 2> : stream_kernel<T, 128, 1>);
  else launch(gt == 4 ? stream_kernel<T, 64, 4> : gt == 2 ? stream_kernel<T, 64, 2> : stream_kernel<T, 64, 1>);
  return hipGetLastError() != hipSuccess ? 7 : 0;
}

// ---------------------------------------------------------------------------
// Scores only, over heads stored as rows (the target layer's retained heads), one workgroup per chunk and y as in
// attn_split_body: S^T[h, slot * 128 + j] = scale * q_h . rot_j(k_j) for GT query heads of one KV
// head; base-2 logits if the caller folds log2(e) into the scale.
// What bounds it: with the rotary tables, their 64 bytes per lane and row beside the row's own.  A lane therefore holds
// the 8 dims at 8 li and their rotation partners at d / 2 + 8 li (d / 16 lanes per row): with 8 dims per lane both
// halves of a row loaded the same table entries, and exchanged the partners by shuffle.
// A wave's UN x (64 / LPR) rows are consecutive tokens, and each lane of a row stores the sums of its own share of the
// (row, query head) pairs: two stores instead of 16 of 16 bytes each.  As a kernel of its own, 131072 tokens with four retained heads
// and rope: 61 us, and 18 for the window's; here the call went from 376 to 351 us, short ones (4 x 2000-9000 tokens) from 113 to 88.
// ---------------------------------------------------------------------------
template <int HD, int GT, int NWAVES>
__device__ __forceinline__ void row_scores_body(const AttnArgs<bf16_t>& a, float* s_out, int64_t s_ld, const SeqMeta& meta,
                                                int b, int chunk, int y) {
  constexpr int LPR = HD / 16, RPW = 64 / LPR, UN = 4, ROWS = UN * RPW;      // rows of a wave and turn
  constexpr int NS = (UN * GT + LPR - 1) / LPR;
  const int L = meta.len[b];
  const int gchunks = a.G / GT, hl = y / gchunks;
  const int qh0 = (a.head0 + hl) * a.G + (y % gchunks) * GT;
  const int lane = threadIdx.x & 63, li = lane % LPR, rl = lane / LPR;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jend = min(L, chunk * a.split_tokens + a.split_tokens);
  const bool rope = a.rope_cos != nullptr;
  float q0[GT][8], q1[GT][8];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    const bf16_t* q = a.q + ((int64_t)b * a.H_q + qh0 + g) * HD + 8 * li;
    load16<bf16_t>(q, q0[g]);
    load16<bf16_t>(q + HD / 2, q1[g]);
#pragma unroll
    for (int i = 0; i < 8; ++i) { q0[g][i] *= a.scale; q1[g][i] *= a.scale; }
  }
  const bf16_t* k = a.k + meta.start[b] * a.ld + a.col0 + hl * HD + 8 * li;
  const float* ct = a.rope_cos + 8 * li;
  const float* st = a.rope_sin + 8 * li;
  float* dst = s_out + (int64_t)qh0 * s_ld + (int64_t)meta.sbase[b] * kSlotTokens;
  for (int jb = chunk * a.split_tokens + wave * ROWS; jb < jend; jb += NWAVES * ROWS) {
    float v[NS];
#pragma unroll
    for (int n = 0; n < NS; ++n) v[n] = 0.f;
    uint4 r0[UN], r1[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const bf16_t* row = k + (int64_t)min(jb + u * RPW + rl, jend - 1) * a.ld;
      r0[u] = *reinterpret_cast<const uint4*>(row);
      r1[u] = *reinterpret_cast<const uint4*>(row + HD / 2);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      float k0[8], k1[8];
      unpack_bf16x8(r0[u], k0);
      unpack_bf16x8(r1[u], k1);
      if (rope) {
        const int64_t t = (int64_t)min(jb + u * RPW + rl, jend - 1) * (HD / 2);
#pragma unroll
        for (int i = 0; i < 8; i += 4) {
          const float4 c4 = *reinterpret_cast<const float4*>(ct + t + i), s4 = *reinterpret_cast<const float4*>(st + t + i);
          const float c[4] = {c4.x, c4.y, c4.z, c4.w}, s[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x0 = k0[i + e], x1 = k1[i + e];
            k0[i + e] = fmaf(x0, c[e], -x1 * s[e]);
            k1[i + e] = fmaf(x1, c[e], x0 * s[e]);
          }
        }
      }
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float sc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) sc = fmaf(q0[g][i], k0[i], fmaf(q1[g][i], k1[i], sc));
        sc = row_sum<LPR>(sc);
        const int n = u * GT + g;                // lane n % LPR of the row stores pair n
        v[n / LPR] = li == n % LPR ? sc : v[n / LPR];
      }
    }
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      const int pair = n * LPR + li, j = jb + (pair / GT) * RPW + rl;
      if (pair < UN * GT && j < jend) dst[(int64_t)(pair % GT) * s_ld + j] = v[n];
    }
  }
}
// Workgroup wg of the retained heads' scores (Streams::ret), then of the window.
template <int HD, int NWAVES>
__device__ __forceinline__ void score_stream_workgroup(const Streams<bf16_t>& st, const StreamMeta& meta, int wg, float* s_out,
                                                       int64_t s_ld, char* smem) {
  if (wg >= st.n_ret) {
    stream_workgroup<bf16_t, HD, NWAVES, 4>(st, meta, wg, smem);
    return;
  }
  int x, y;
  stream_item(wg, st.n_ret_chunks, st.n_ret / st.n_ret_chunks, x, y);
  const int b = find_seq(meta.cbase, meta.s.n, x), chunk = x - meta.cbase[b];
  if (st.ret.G % 4 == 0) row_scores_body<HD, 4, NWAVES>(st.ret, s_out, s_ld, meta.s, b, chunk, y);
  else if (st.ret.G % 2 == 0) row_scores_body<HD, 2, NWAVES>(st.ret, s_out, s_ld, meta.s, b, chunk, y);
  else row_scores_body<HD, 1, NWAVES>(st.ret, s_out, s_ld, meta.s, b, chunk, y);
}

// ---------------------------------------------------------------------------
// Rotary embedding of key rows ahead of the prefill attention kernels (Sec. "Network
// Architecture": caches hold pre-rotation keys): row j of src [rows, n_heads * d] (pitch
// ld_src) is rotated to position j, feature i of a head pairing with i + d/2, and written
// to dst (pitch ld_dst; dst may be src).  One thread per 8 + 8 paired features and turn, the loads of all turns ahead.
// ---------------------------------------------------------------------------
struct RopeRows {
  const bf16_t* src = nullptr; bf16_t* dst = nullptr;
  int64_t ld_src = 0, ld_dst = 0;
  int32_t n_heads = 0, d = 0, rows = 0;
  const float* cos = nullptr; const float* sin = nullptr;      // [>= rows, d / 2]
};
// The first (HI = false) or second half's 8 features from both halves' and 8 table entries of their angle.
template <bool HI>
__device__ __forceinline__ uint4 rope8(uint4 lo, uint4 hi, const float4 (&cos)[2], const float4 (&sin)[2]) {
  float a[8], b[8], r[8];
  unpack_bf16x8(lo, a);
  unpack_bf16x8(hi, b);
#pragma unroll
  for (int i = 0; i < 8; i += 4) {
    const float4 c4 = cos[i / 4], s4 = sin[i / 4];
    const float c[4] = {c4.x, c4.y, c4.z, c4.w}, s[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) r[i + e] = HI ? b[i + e] * c[e] + a[i + e] * s[e] : a[i + e] * c[e] - b[i + e] * s[e];
  }
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = pack_bf16(r[2 * i], r[2 * i + 1]);
  return make_uint4(w[0], w[1], w[2], w[3]);
}
constexpr int kRopeTurns = 4;
__host__ __device__ inline int64_t rope_workgroups(const RopeRows& a, int threads) {
  const int64_t per = (int64_t)threads * kRopeTurns;
  return ((int64_t)a.rows * a.n_heads * (a.d / 16) + per - 1) / per;
}
template <int NT>
__device__ __forceinline__ void rope_workgroup(const RopeRows& a, int wg) {
  const int cpr = a.d / 16, half = a.d / 2, per_row = a.n_heads * cpr;
  const int64_t n = (int64_t)per_row * a.rows;
  uint4 lo[kRopeTurns], hi[kRopeTurns];
  float4 cs[kRopeTurns][2], sn[kRopeTurns][2];
  bf16_t* dp[kRopeTurns];
  const int64_t idx0 = (int64_t)wg * kRopeTurns * NT + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kRopeTurns; ++u) {
    const int64_t idx = min(idx0 + u * NT, n - 1);
    const int row = (int)(idx / per_row), rem = (int)(idx % per_row), head = rem / cpr, c = rem % cpr;
    const bf16_t* sp = a.src + (int64_t)row * a.ld_src + head * a.d + c * 8;
    lo[u] = *reinterpret_cast<const uint4*>(sp);
    hi[u] = *reinterpret_cast<const uint4*>(sp + half);
    const int64_t e = (int64_t)row * half + c * 8;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      cs[u][i] = *reinterpret_cast<const float4*>(a.cos + e + 4 * i);
      sn[u][i] = *reinterpret_cast<const float4*>(a.sin + e + 4 * i);
    }
    dp[u] = a.dst + (int64_t)row * a.ld_dst + head * a.d + c * 8;
  }
#pragma unroll
  for (int u = 0; u < kRopeTurns; ++u) {
    if (idx0 + u * NT >= n) return;
    *reinterpret_cast<uint4*>(dp[u]) = rope8<false>(lo[u], hi[u], cs[u], sn[u]);
    *reinterpret_cast<uint4*>(dp[u] + half) = rope8<true>(lo[u], hi[u], cs[u], sn[u]);
  }
}

}  // namespace echokv
