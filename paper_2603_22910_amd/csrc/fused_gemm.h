// Main loop of the predictor product (Eq. 3) on v_mfma_f32_16x16x32_bf16, shared by the fused decode
// kernel, its score-only half and the stand-alone product.
//
// One workgroup of eight waves owns 256 tokens x 256 predicted columns; wave w (wt = w % 4, wc = w / 4)
// holds 64 tokens x 128 columns (whole heads, or SPLIT: half the dims of every head of the tile) in 128 accumulators, so two waves
// share a SIMD and cover each other's barriers, LDS round trips and issue slots.  With one wave of 128 x 128 per SIMD the matrix
// pipe was busy 69 % of the time whatever the operands' way into LDS; an MFMA and six other
// instructions of one wave take 40 cycles, of two waves 32.
// The chip is power-limited under this loop, and of the two MFMA shapes the smaller one costs less: a loop of
// nothing but MFMAs on random operands settles at 2.03 PFLOP/s with 16 x 16 x 32 and at 1.76 with 32 x 32 x 16
// (which reads and writes twice the accumulator words per product).
//
// Both operands travel L2 -> LDS with `buffer_load ... lds` (no staging registers, no ds_write) in
// tiles of 64 input dims, two stages of 64 KB.  A stage is four 16 KB parts, X0 X1 (token halves of every
// wave) and W0 W1 (column halves of every wave), and a tile is four phases of sixteen MFMAs, one per
// (W half, X half): a part is free for the tile after next as soon as its last phase has begun, so the
// copies are a tile and a half ahead with two stages only.
//   phase 1  MFMA W0 Xa | read Xb, 1/4 W1    | copy W1 of tile t+1 -> wait for Xa W0 of t+1, barrier: Xa, W0 are free
//   phase 2  MFMA W0 Xb | read 3/4 W1         | copy Xa of tile t+2
//   phase 3  MFMA W1 Xb | read 3/4 W0 of t+1  | copy W0 of tile t+2 -> wait for Xb W1 of t+1, barrier: Xb, W1 are free
//   phase 4  MFMA W1 Xa | read 1/4 W0, Xa of t+1 | copy Xb of tile t+2
// Reads (6 KB per wave and phase), copies (2 per wave and phase) and the scalar work for them are spread over the phases and,
// by fences and scheduling groups, between the MFMAs of a phase: two MFMAs, the reads' first third, two MFMAs ..., then
// at most five scalar or vector instructions per MFMA.  The two waves of a SIMD run in step, so what stands in one place of
// the loop stops the matrix pipe for both.  All reads of a phase ahead of its MFMAs and ~20 scalar instructions
// around each copy cost 10 % (4000 tokens, d_in 6144, 2048 predicted dims, one round of workgroups: 256 -> 233 us, packed W 236 -> 211;
// 8 x 4096 tokens 1297 -> 1221); reads and copies spread over twelve MFMAs +0 / +5 %, reads behind each other MFMA +1-3 %; all
// reads of a tile in two of its phases and all copies in a burst behind a barrier cost 350 cycles per barrier.
// (a, b) = (0, 1) for the even tiles of a pass and (1, 0) for the odd ones: the half read ahead in phase 4 goes to the
// registers that phase 3 has left, so nothing is copied and 80 registers hold all fragments.
//
// Row-major W ([d_in, d_out]) lies in LDS as it lies in memory, [64 k][128 columns], and its fragments
// come from the LDS transpose read (16 lanes read 4 k x 16 columns, each ends up with one column's 4 k);
// packed W ([d_out, d_in]) is read like X.
//
// What bounds it: power.  The matrix pipe is busy 70 % of the cycles at the clock that leaves (1.85 GHz); the rest is
// waits around the two barriers of a tile and the epilogues.  Whole calls, four waves of 128 x 128 with 32 x 32 x 16 -> this:
// 8 x 4096 tokens, d_in 6144, 2048 predicted dims 1336 -> 1221 us, packed W 1382 -> 1196; 4000 tokens 243 -> 233,
// packed 227 -> 211; 3 x 6000 tokens, d_in 1024, 1024 predicted dims 128 -> 114.  Tried: s_setprio around the MFMAs
// 3 % slower.
//
// The LDS reads of the loop are instructions with waits of their own: in builtin form the compiler puts
// them behind every outstanding copy (s_waitcnt vmcnt(0)), which would drain the pipeline in every phase.
// The copies are counted (vmcnt), so the kernels must not spill, and nothing may touch a fragment's registers between its
// request and its wait: the build checks both.
#pragma once
#include "common.h"

namespace echokv {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
#ifndef ECHOKV_LDS
#define ECHOKV_LDS __attribute__((address_space(3)))
#endif

namespace fused {

constexpr int BM = 256;      // tokens per workgroup tile
constexpr int BN = 256;      // predicted columns per workgroup tile
constexpr int BK = 64;       // input dims per k-tile
constexpr int NWAVES = 8, NTHREADS = 64 * NWAVES;
constexpr int WM = 64, WN = 128;          // per-wave tile
constexpr int kPart = 16384, kStage = 4 * kPart;      // X0, X1, W0, W1

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// Global loads go through raw buffer instructions: a 128-bit resource (uniform base) + a 32-bit
// per-thread byte offset + a uniform byte offset, so no 64-bit address arithmetic is spent per load.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base) {
  // raw buffer, no stride, byte-granular range check far beyond any offset used here
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ void copy_to_lds(rsrc_t r, char* lds, uint32_t voff, int soff) {
#ifdef __HIP_DEVICE_COMPILE__      // (the host pass does not know the builtin)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (ECHOKV_LDS void*)lds, 16, voff, soff, 0, 0);
#endif
}
__device__ __forceinline__ uint32_t lds_offset(const void* p) { return (uint32_t)(uintptr_t)(ECHOKV_LDS const char*)p; }

// What the product of a workgroup reads: one or two passes (keys, then values) of the same shape over
// the same tokens and columns.  All uniform.
struct Operands {
  const bf16_t* xa[2];       // first row of the token tile in the anchor cache, pitch D
  const bf16_t* xr[2];       // ... in the retained cache, pitch m
  const bf16_t* w[2];        // first column of the tile: row-major W + n0, or packed W + n0 * d_in
  int D, m, d_out;           // d_out: pitch of row-major W
  int run;                   // head dim / 4 (SPLIT)
  int last;                  // last valid token of the tile: rows past it repeat it
  int ncol;                  // valid columns from the tile's first one on (>= 8): those past them repeat the last ones
  int nk, nka, total;        // k-tiles per pass, of them in the anchor row; passes * nk
  int rot;                   // k-tile visited first, three further on for each token tile of a sequence: rows are a power of two bytes apart, and
                             // workgroups that all walked the dims in step would pull from one memory channel at a time.  It goes by the tile's
                             // place in its sequence alone, so that the sums do not depend on what else is in the launch.  An eighth of the dims
                             // further on for each XCD (fewer L2 misses of W) is up to 2.4 % faster (prefill of 8192, 32 heads: 935 / 920 us, 4000 behind
                             // 4000 880 / 860, 8 x 4096 tokens 1306 / 1304), but a sequence's sums then follow the number of tiles of the launch
};

// Per-thread part of the copies.  Copy i (0, 1) of a wave fills 1 KB of a part: for rows of 64 dims (X,
// packed W) rows 8 (2 w + i) + lane / 8, for row-major W dims 4 (2 w + i) + lane / 16.  16-byte chunk c of
// row r sits at chunk c ^ swizzle(r) (rows of 64 dims: r / 2 % 8; row-major W: w_swizzle), so that neither the fragment
// reads nor the transpose reads collide on LDS banks, in whichever groups of lanes they are served; the swizzle is applied on the global side (the LDS side of a copy is linear).
struct Copies {
  uint32_t xrow;             // tile row of part 0, copy 0: + 32 h + 8 i for the others, before the clamp
  uint32_t ch;               // byte offset of the source chunk for i = 0; i = 1: ^ 64
  uint32_t w[2][2];          // [part][i]: byte offset in W (row-major: i = 0 only)
};

// Row-major W, dim k: bits 2 and 3 of the chunk from k % 4, bit 1 from k / 8 % 2.
__device__ __forceinline__ int w_swizzle(int k) { return ((k & 3) << 2) | (((k >> 3) & 1) << 1); }

// Column of the tile that is column x (0 ... 63) of wave column wc in W part h.  Plain: the wave column has the columns 128 wc ..., part h
// 64 of them, and a wave whose columns do not exist only copies.  SPLIT (run = head dim / 4): part 0 holds the first halves of the heads' dims, part 1
// the second ones, and of either half the wave columns take a run each: a dim and its rotation partner stay in one lane, and a wave reads
// half a token's rotary table entries for all heads of the tile instead of all of them for one.  Where the tile
// has no columns past 128 both parts' columns x < 32 then fit into one (half): both waves of a SIMD work on them, and there is no second part.
// The two waves of 64 tokens have to add their scores up, which costs as much as it brings where there are no tables to load: fused
// decode, plain / SPLIT, us: 8 x 2048-36864 tokens, 32 heads over 8, m = 384, rope 294 / 288, 2 x 40000, m = 512, rope 286 / 279, but 4 x 2000-12000, m =
// 384, no rope 131 / 137, and with the tables through LDS (the score kernel) 325 / 327.
// (Whole heads as parts would do the same without a second mapping for half, but rows of row-major W are mostly a multiple of 4 KB apart:
// with 256 bytes of each in a part instead of two times 128 a multi-head decode took 1.3 % longer.)
template <bool SPLIT>
__device__ __forceinline__ int column_of(int run, int wc, int h, int x) {
  return SPLIT ? x / run * (4 * run) + h * (2 * run) + wc * run + x % run : wc * 128 + h * 64 + x;
}

template <bool PACKED, bool SPLIT>
__device__ __forceinline__ void make_copies(Copies& c, const Operands& op, bool half, int wave, int lane) {
  auto column = [&](int wc, int h, int x) { return SPLIT && half ? column_of<SPLIT>(op.run, wc, x >> 5, x & 31) : column_of<SPLIT>(op.run, wc, h, x); };
  // part row r <-> token 64 (r / 32) + 32 h + r % 32: wave wt reads rows 32 wt .. of either part
  const int r0 = 16 * wave + (lane >> 3);
  c.xrow = (uint32_t)((r0 >> 5) * 64 + (r0 & 31));
  c.ch = (uint32_t)(((lane & 7) ^ (lane >> 4)) * 16);      // (row r0: r0 / 2 % 8 = lane / 16; 8 rows on: ^ 4)
  if constexpr (PACKED) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = r0 + 8 * i, n = min(column(r >> 6, h, r & 63), op.ncol - 1);
        c.w[h][i] = (uint32_t)n * (uint32_t)((op.D + op.m) * 2) + (c.ch ^ (i * 64));
      }
  } else {
    const int k = 2 * wave * 4 + (lane >> 4);            // (copy 1: k + 4, the same swizzle)
    const int ch = (lane & 15) ^ w_swizzle(k);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = min(column(ch >> 3, h, (ch & 7) * 8), op.ncol - 8);
      c.w[h][0] = (uint32_t)k * (uint32_t)(op.d_out * 2) + (uint32_t)n * 2;
      c.w[h][1] = 0;
    }
  }
}

// c ? a : b of two fields of a structure, without the branch that the ternary is at first: with it the
// compiler loads through a selected address, the structure then has to lie in scratch memory, and
// what was uniform is not known to be.
template <typename P> __device__ __forceinline__ P pick(bool c, P a, P b) {
  const uint64_t m = c ? ~0ull : 0ull;
  return (P)(((uint64_t)a & m) | ((uint64_t)b & ~m));
}
// Where the copies of one k-tile come from: worked out once per tile, uniform.
struct Src {
  const bf16_t* x; uint32_t ld2; int xoff;      // token tile in the anchor or retained cache, pitch and dim in bytes
  const bf16_t* w; int woff;                    // packed: dim in bytes, row-major: first row's offset in bytes
};
template <bool PACKED>
__device__ __forceinline__ Src source_of(const Operands& op, int t) {
  Src s;
  int i = min(t, op.total - 1);              // past the end: the last tile again (lands, is never multiplied)
  const bool second = i >= op.nk;
  i -= second ? op.nk : 0;
  i += op.rot;
  const int kt = i >= op.nk ? i - op.nk : i;
  const bool anchor = kt < op.nka;           // anchor dims first, then retained dims (Eq. 3): uniform selects
  s.x = pick(second, pick(anchor, op.xa[1], op.xr[1]), pick(anchor, op.xa[0], op.xr[0]));
  s.ld2 = pick(anchor, (uint32_t)op.D, (uint32_t)op.m) * 2;
  s.xoff = (anchor ? kt : kt - op.nka) * (BK * 2);
  s.w = pick(second, op.w[1], op.w[0]);
  s.woff = PACKED ? kt * (BK * 2) : kt * BK * op.d_out * 2;
  return s;
}
// Copy i (0, 1) of this wave's share of X part h / W part h of a tile (stage = its number % 2).
__device__ __forceinline__ void copy_x(char* smem, const Operands& op, const Copies& c, const Src& s, int stage, int h, int i, int wave) {
  char* dst = smem + stage * kStage + h * kPart + (2 * wave + i) * 1024;
  copy_to_lds(make_rsrc(s.x), dst, __umul24(min(c.xrow + 32 * h + 8 * i, (uint32_t)op.last), s.ld2) + (c.ch ^ (i * 64)), s.xoff);      // (row < 256, pitch < 2^24)
}
template <bool PACKED>
__device__ __forceinline__ void copy_w(char* smem, const Operands& op, const Copies& c, const Src& s, int stage, int h, int i, int wave) {
  char* dst = smem + stage * kStage + (2 + h) * kPart + (2 * wave + i) * 1024;
  if constexpr (PACKED) copy_to_lds(make_rsrc(s.w), dst, c.w[h][i], s.woff);
  else copy_to_lds(make_rsrc(s.w), dst, c.w[h][0], s.woff + i * 8 * op.d_out);
}

// Fragments: X half: 2 k-steps of 32 x 2 blocks of 16 tokens; W half: 2 k-steps x 4 blocks of 16 columns.  A lane
// holds 8 consecutive dims (k-step's octet lane / 16) of row / column lane % 16.
struct XFrag { u32x4_t v[2][2]; };
template <bool PACKED> struct WFrag;
template <> struct WFrag<true> { u32x4_t v[2][4]; };
template <> struct WFrag<false> { u32x2_t lo[2][4], hi[2][4]; };

// LDS byte addresses of a lane's first fragments for the stage in use (toggled by kStage per tile).
// Rows of 64 dims: k-step 1 is ^ 64; block b of 16 rows is + 2048 b.
template <bool PACKED> struct Lanes {
  uint32_t x;                // row 32 wt + lane % 16, chunk lane / 16
  uint32_t w;                // packed: row 64 wc + lane % 16; row-major: see below
  __device__ __forceinline__ void init(const char* smem, int wt, int wc, int lane) {
    const uint32_t base = lds_offset(smem);
    const int c = lane & 15, o = lane >> 4, rx = 32 * wt + c, rw = 64 * wc + c;
    x = base + (uint32_t)(rx * 128 + ((o ^ ((rx >> 1) & 7)) << 4));
    if constexpr (PACKED) {
      w = base + 2 * kPart + (uint32_t)(rw * 128 + ((o ^ ((rw >> 1) & 7)) << 4));
    } else {
      // transpose read: lane 4 j + a of a group of 16 supplies columns 4 a .. 4 a + 3 of dim j, the group o dims
      // 8 o + (0 .. 3), 4 rows on the other four.  Column block b: ^ 32 b, two bits that only the swizzle touches
      const int j = c >> 2, ch = (8 * wc + ((c & 3) >> 1)) ^ w_swizzle(8 * o + j);
      w = base + 2 * kPart + (uint32_t)((8 * o + j) * 256 + ch * 16 + (c & 1) * 8);
    }
  }
  __device__ __forceinline__ void next_stage() { x ^= kStage; w ^= kStage; }
};

// The reads are issued here and waited for in wait_*: the operands of the wait tie it to the registers.
// (Addresses are worked out from an opaque copy per read: shared between reads they would all stay in registers.)
__device__ __forceinline__ uint32_t opaque(uint32_t a) { asm volatile("" : "+v"(a)); return a; }
template <int PART>
__device__ __forceinline__ void read_x(XFrag& f, uint32_t base) {
  const uint32_t a = opaque(base);
  asm volatile("ds_read_b128 %0, %4 offset:%6\n\tds_read_b128 %1, %4 offset:%7\n\t"
               "ds_read_b128 %2, %5 offset:%6\n\tds_read_b128 %3, %5 offset:%7"
               : "=&v"(f.v[0][0]), "=&v"(f.v[0][1]), "=&v"(f.v[1][0]), "=&v"(f.v[1][1])
               : "v"(a), "v"(a ^ 64u), "n"(PART * kPart), "n"(PART * kPart + 2048));
}
__device__ __forceinline__ void wait_x(XFrag& f) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.v[0][0]), "+v"(f.v[0][1]), "+v"(f.v[1][0]), "+v"(f.v[1][1]));
}
// Quarter Q of a W part: k-step Q / 2, column blocks 2 (Q % 2) and the next.
template <int PART, int Q>
__device__ __forceinline__ void read_w(WFrag<true>& f, const Lanes<true>& l) {
  constexpr int K = Q >> 1, B = 2 * (Q & 1), O = PART * kPart + B * 2048;
  const uint32_t a = opaque(l.w);
  asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4"
               : "=&v"(f.v[K][B]), "=&v"(f.v[K][B + 1]) : "v"(a ^ (uint32_t)(K << 6)), "n"(O), "n"(O + 2048));
}
template <int PART, int Q>
__device__ __forceinline__ void read_w(WFrag<false>& f, const Lanes<false>& l) {
  constexpr int K = Q >> 1, B = 2 * (Q & 1), O = PART * kPart + K * 8192;      // 32 rows of 256 bytes; the hi dims: 4 rows on
  const uint32_t a = opaque(l.w);
  asm volatile("ds_read_b64_tr_b16 %0, %4 offset:%6\n\tds_read_b64_tr_b16 %1, %4 offset:%7\n\t"
               "ds_read_b64_tr_b16 %2, %5 offset:%6\n\tds_read_b64_tr_b16 %3, %5 offset:%7"
               : "=&v"(f.lo[K][B]), "=&v"(f.hi[K][B]), "=&v"(f.lo[K][B + 1]), "=&v"(f.hi[K][B + 1])
               : "v"(a ^ (uint32_t)(B << 5)), "v"(a ^ (uint32_t)((B + 1) << 5)), "n"(O), "n"(O + 1024));
}
__device__ __forceinline__ void wait_w(WFrag<true>& f) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.v[0][0]), "+v"(f.v[0][1]), "+v"(f.v[0][2]), "+v"(f.v[0][3]),
                                        "+v"(f.v[1][0]), "+v"(f.v[1][1]), "+v"(f.v[1][2]), "+v"(f.v[1][3]));
}
__device__ __forceinline__ void wait_w(WFrag<false>& f) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(f.lo[0][0]), "+v"(f.lo[0][1]), "+v"(f.lo[0][2]), "+v"(f.lo[0][3]),
                 "+v"(f.hi[0][0]), "+v"(f.hi[0][1]), "+v"(f.hi[0][2]), "+v"(f.hi[0][3]));
  asm volatile("" : "+v"(f.lo[1][0]), "+v"(f.lo[1][1]), "+v"(f.lo[1][2]), "+v"(f.lo[1][3]),
                    "+v"(f.hi[1][0]), "+v"(f.hi[1][1]), "+v"(f.hi[1][2]), "+v"(f.hi[1][3]));
}
__device__ __forceinline__ bf16x8_t frag(const WFrag<true>& f, int kk, int b) { return __builtin_bit_cast(bf16x8_t, f.v[kk][b]); }
__device__ __forceinline__ bf16x8_t frag(const WFrag<false>& f, int kk, int b) {
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.lo[kk][b], f.hi[kk][b], 0, 1, 2, 3));
}

// Accumulators of a wave, blocks of 16 columns x 16 tokens.  SWAP: W^T X^T, rows (4 (lane / 16) + r) = columns, lane % 16 =
// token; otherwise X W, rows = tokens, lane % 16 = column.
struct Acc { floatx4_t v[8][4]; };           // [column block][token block]
// Reads are issued ahead of a phase's MFMAs and waited for behind them: nothing crosses.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }
// Sixteen MFMAs of one (W half, X half), with the phase's LDS reads in up to three parts (read(0 .. 2)) and
// its two copies (copy(0 .. 1)) with whatever scalar work there is dealt out between them: the two waves of a SIMD run in
// step, so a burst of other instructions leaves the matrix pipe idle, while a few behind every MFMA are free.
// HALF: the columns of both parts in one.
template <bool SWAP, bool PACKED, bool HALF = false, class Read, class Copy>
__device__ __forceinline__ void mma16(Acc& acc, const WFrag<PACKED>& w, const XFrag& x, int wh, int xh, Read read, Copy copy) {
  auto block = [&](int b) __attribute__((always_inline)) { return HALF ? 4 * (b >> 1) + (b & 1) : 4 * wh + b; };
  auto mma = [&](int i) __attribute__((always_inline)) {
    const int kk = i >> 3, t = (i >> 2) & 1, b = i & 3;
    const bf16x8_t wf = frag(w, kk, b), xf = __builtin_bit_cast(bf16x8_t, x.v[kk][t]);
    floatx4_t& d = acc.v[block(b)][2 * xh + t];
    d = SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, d, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, wf, d, 0, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < 6; i += 2) {
    keep_order();
    mma(i);
    mma(i + 1);
    asm volatile("" : "+v"(acc.v[block(i & 3)][2 * xh + ((i >> 2) & 1)]), "+v"(acc.v[block((i & 3) + 1)][2 * xh + ((i >> 2) & 1)]));
    keep_order();
    read(i >> 1);
  }
  keep_order();
  copy(0);
  copy(1);
#pragma unroll
  for (int i = 6; i < 16; ++i) mma(i);
#pragma unroll
  for (int i = 6; i < 16; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);       // one MFMA
    __builtin_amdgcn_sched_group_barrier(0x4, 4, 0);       // up to four scalar instructions
    __builtin_amdgcn_sched_group_barrier(0x2, 1, 0);       // one vector instruction
    if (i == 8 || i == 12) __builtin_amdgcn_sched_group_barrier(0x10, 1, 0);      // a copy
  }
  keep_order();
#pragma unroll
  for (int b = 0; b < 4; ++b) asm volatile("" : "+v"(acc.v[block(b)][2 * xh]), "+v"(acc.v[block(b)][2 * xh + 1]));
}

__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
template <int N> __device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// State of a workgroup's product that outlives a pass.
template <bool PACKED, bool SPLIT> struct Pipe {
  Operands op;
  Copies cp;
  Lanes<PACKED> ln;
  char* smem;
  int wave, lane;
  bool half;                 // no columns past 128.  SPLIT: of the tile, W1 is neither copied nor multiplied; plain: this wave's do not exist

  // Requests k-tile 0 and all of k-tile 1 but its W1 (phase 1 of tile 0 does).  op, smem, wave, lane, half are set.
  __device__ __forceinline__ void begin() {
    make_copies<PACKED, SPLIT>(cp, op, half, wave, lane);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const Src s = source_of<PACKED>(op, t);
#pragma unroll
      for (int part = 0; part < 4 - t; ++part)       // Xa, W0, Xb, W1: the order in which they are waited for
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (SPLIT && part == 3 && half) continue;
          if (part & 1) copy_w<PACKED>(smem, op, cp, s, t, part >> 1, i, wave);
          else copy_x(smem, op, cp, s, t, (SPLIT && half ? 0 : t) ^ (part >> 1), i, wave);
        }
    }
  }

  // Phases 1-4 of tile t, PAR = its number in the pass % 2 (see the top of the file).  IDLE: the wave's
  // columns do not exist, it only copies and meets the others.
  template <bool SWAP, int PAR, bool IDLE>
  __device__ __forceinline__ void tile(Acc& acc, XFrag (&x)[2], WFrag<PACKED>& w0, WFrag<PACKED>& w1, int t, Src& src) {
    constexpr int A = PAR, B = PAR ^ 1;
    const int st = t & 1;
    Src s2;                                  // of tile t + 2; src: of tile t + 1
    auto w1_next = [&](int i) __attribute__((always_inline)) {
      copy_w<PACKED>(smem, op, cp, src, st ^ 1, 1, i, wave);
      if (i == 1) {
        int t2 = t + 2;
        asm volatile("" : "+s"(t2));         // (worked out here, between MFMAs, and nowhere else)
        s2 = source_of<PACKED>(op, t2);
      }
    };
    auto xa_next = [&](int i) __attribute__((always_inline)) { copy_x(smem, op, cp, s2, st, A, i, wave); };
    auto w0_next = [&](int i) __attribute__((always_inline)) { copy_w<PACKED>(smem, op, cp, s2, st, 0, i, wave); };
    auto xb_next = [&](int i) __attribute__((always_inline)) { copy_x(smem, op, cp, s2, st, B, i, wave); };
    if constexpr (IDLE) {
      w1_next(0); w1_next(1);
      wait_copies<4>();
      barrier();
      xa_next(0); xa_next(1); w0_next(0); w0_next(1);
      wait_copies<4>();
      barrier();
      xb_next(0); xb_next(1);
    } else {
      mma16<SWAP, PACKED>(acc, w0, x[A], 0, A, [&](int i) __attribute__((always_inline)) {
        if (i == 0) read_x<B>(x[B], ln.x);
        if (i == 1) read_w<1, 0>(w1, ln);
      }, w1_next);
      wait_x(x[B]);
      wait_copies<4>();                      // Xa, W0 of tile t + 1 (this wave's copies; the barrier: everyone's)
      barrier();
      mma16<SWAP, PACKED>(acc, w0, x[B], 0, B, [&](int i) __attribute__((always_inline)) {
        if (i == 0) read_w<1, 1>(w1, ln);
        if (i == 1) read_w<1, 2>(w1, ln);
        if (i == 2) read_w<1, 3>(w1, ln);
      }, xa_next);
      wait_w(w1);
      ln.next_stage();
      mma16<SWAP, PACKED>(acc, w1, x[B], 1, B, [&](int i) __attribute__((always_inline)) {
        if (i == 0) read_w<0, 0>(w0, ln);
        if (i == 1) read_w<0, 1>(w0, ln);
        if (i == 2) read_w<0, 2>(w0, ln);
      }, w0_next);
      wait_copies<4>();                      // Xb, W1 of tile t + 1
      barrier();
      mma16<SWAP, PACKED>(acc, w1, x[A], 1, A, [&](int i) __attribute__((always_inline)) {
        if (i == 0) read_w<0, 3>(w0, ln);
        if (i == 1) read_x<B>(x[B], ln.x);   // (the next tile's Xa is the part that is Xb here)
      }, xb_next);
      wait_w(w0);
      wait_x(x[B]);
    }
    src = s2;
  }
  // SPLIT, a tile with no columns past 128: two phases, X0 and X1, the copies a tile and a half ahead as well.  W0's fragments of the
  // next tile are read beside the second phase into the registers that W1's would take.  1.1 us per tile where 256 columns take
  // 1.6 (with 128 columns to each of four waves and the others only copying 1.17; with the parts in a ring of eight, two tiles
  // ahead, 1.27: twice the scalar instructions).
  //   phase 1  MFMA W0 X0 | read X1            | copy X0, W0 of tile t+2 -> wait for X0 W0 of t+1, barrier
  //   phase 2  MFMA W0 X1 | read W0, X0 of t+1 | copy X1 of tile t+2     -> wait for X1 of t+1, barrier
  template <bool SWAP>
  __device__ __forceinline__ void half_tile(Acc& acc, XFrag (&x)[2], WFrag<PACKED>& w, WFrag<PACKED>& next, int t, Src& s2) {
    const int st = t & 1;
    Src s3;                                  // of tile t + 3; s2: of tile t + 2
    mma16<SWAP, PACKED, true>(acc, w, x[0], 0, 0, [&](int i) __attribute__((always_inline)) {
      if (i == 0) read_x<1>(x[1], ln.x);
    }, [&](int i) __attribute__((always_inline)) {
      copy_x(smem, op, cp, s2, st, 0, i, wave);
      copy_w<PACKED>(smem, op, cp, s2, st, 0, i, wave);
    });
    wait_x(x[1]);
    wait_copies<6>();
    barrier();
    ln.next_stage();
    mma16<SWAP, PACKED, true>(acc, w, x[1], 0, 1, [&](int i) __attribute__((always_inline)) {
      if (i == 0) { read_w<0, 0>(next, ln); read_w<0, 1>(next, ln); }
      if (i == 1) { read_w<0, 2>(next, ln); read_w<0, 3>(next, ln); }
      if (i == 2) read_x<0>(x[0], ln.x);
    }, [&](int i) __attribute__((always_inline)) {
      copy_x(smem, op, cp, s2, st, 1, i, wave);
      if (i == 1) {
        int t3 = t + 3;
        asm volatile("" : "+s"(t3));
        s3 = source_of<PACKED>(op, t3);
      }
    });
    wait_w(next);
    wait_x(x[0]);
    wait_copies<6>();
    barrier();
    s2 = s3;
  }
  template <bool SWAP>
  __device__ __forceinline__ void half_tiles(Acc& acc, int t0) {
    XFrag x[2];
    WFrag<PACKED> w0, w1;
    read_x<0>(x[0], ln.x);
    read_w<0, 0>(w0, ln); read_w<0, 1>(w0, ln); read_w<0, 2>(w0, ln); read_w<0, 3>(w0, ln);
    wait_w(w0);
    wait_x(x[0]);
    barrier();                               // X0, W0 of the first tile are free
    const int t1 = t0 + op.nk;
    int t = t0;
    Src s2 = source_of<PACKED>(op, t0 + 2);
    for (; t + 1 < t1; t += 2) {
      half_tile<SWAP>(acc, x, w0, w1, t, s2);
      half_tile<SWAP>(acc, x, w1, w0, t + 1, s2);
    }
    if (t < t1) half_tile<SWAP>(acc, x, w0, w1, t, s2);
  }
  template <bool SWAP, bool IDLE>
  __device__ __forceinline__ void tiles(Acc& acc, int t0) {
    XFrag x[2];
    WFrag<PACKED> w0, w1;
    if constexpr (!IDLE) {
      read_x<0>(x[0], ln.x);
      read_w<0, 0>(w0, ln); read_w<0, 1>(w0, ln); read_w<0, 2>(w0, ln); read_w<0, 3>(w0, ln);
      wait_w(w0);
      wait_x(x[0]);
    }
    const int t1 = t0 + op.nk;
    int t = t0;
    Src src = source_of<PACKED>(op, t0 + 1);
    for (; t + 1 < t1; t += 2) {
      tile<SWAP, 0, IDLE>(acc, x, w0, w1, t, src);
      tile<SWAP, 1, IDLE>(acc, x, w0, w1, t + 1, src);
    }
    if (t < t1) tile<SWAP, 0, IDLE>(acc, x, w0, w1, t, src);
  }

  // One pass: k-tiles [t0, t0 + nk).  Every wave's copies of tile t0 have landed and a barrier has passed
  // (begin + first_landed, or the pass before).
  template <bool SWAP>
  __device__ __forceinline__ void pass(Acc& acc, int t0) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc.v[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    // worked out afresh from an opaque copy of the lane id: values that stayed live across the epilogue
    // between two passes would be spilled
    int l = lane;
    asm volatile("" : "+v"(l));
    make_copies<PACKED, SPLIT>(cp, op, half, wave, l);
    ln.init(smem + (t0 & 1) * kStage, wave & 3, wave >> 2, l);
    if constexpr (SPLIT) {
      if (half) half_tiles<SWAP>(acc, t0);
      else tiles<SWAP, false>(acc, t0);
    } else {
      if (half) tiles<SWAP, true>(acc, t0);
      else tiles<SWAP, false>(acc, t0);
    }
  }
  // (own LDS writes done, this wave's copies of tile 0 landed, everyone's after the barrier)
  __device__ __forceinline__ void first_landed() {
    asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
    barrier();
  }
  // After the last pass: the copies past the end have landed, the stages may be used for something else.
  __device__ __forceinline__ void drain() {
    wait_copies<0>();
    barrier();
  }
};

}  // namespace fused
}  // namespace echokv
