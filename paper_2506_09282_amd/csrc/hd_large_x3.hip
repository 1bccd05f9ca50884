// fp32 Stage I on the bf16 matrix instruction, for large batches: inference
// (Alg. 4) and single-pass training (Sec. II-C), with B packed or as given.
//
// Every fp32 value is the exact sum of three bf16 values: it rounded to bf16,
// what is left rounded to bf16, and the rest. A product of two values is taken as
// six of the nine products of parts, each exact, accumulated in fp32 by
// v_mfma_f32_32x32x16_bf16. The middle part is at most 2^-8 and the trailing one
// 2^-17 of a value in [1, 2), so the three products left out are together at most
// 2^-24 of the product, one rounding of the fp32 instruction, of either sign (parts
// by truncation: up to 2^-21, always towards zero). Six such instructions cost 192
// cycles for 16 features against 512 of the fp32 instruction.
// Against 64 bits, signs of X B that differ in 1e9 (normal X; the fp32 instruction
// 32x32x2 in brackets): F = 2 1.5 (2.2), 4 0.8 (3.7), 16 2.2 (15), 32 2.6 (15), 100
// 10 (26), 300 14 (49), 561 25 (70; the streaming kernel's 16x16x4 40), 784 22 (84),
// 1500 35 (113), 3072 55 (174).
//
// Measured (fp32 instruction in brackets; us): inference D = 10240 N = 4096,
// F = 784, K = 10 packed 334 (601), raw N = 500, F = 617, D = 10000, K = 26 65
// (151); N = 20000, F = 784 1590 (3546); training N = 4096, F = 784 358 (916),
// raw 397 (1638, fp32 vector units), raw N = 2048 195 (804). About 1.25 PFLOP/s of
// bf16 products, at the 1.9 GHz that this leaves of the clock.
//
// Range. A value with bits below 2^-133 (some values below 2^-110) is not the sum
// of its parts, inf has no parts, the largest values round to it, and near 2^128
// the order of a sum decides. So the bits of trailing parts are gathered in the
// split (one instruction for two values), and the largest sum where its sign is
// taken. A workgroup that saw such a value, or a sum that is not finite and not
// explained by NaN alone, does its passes again and takes the sums concerned from
// the fp32 instruction (CAREFUL, below). Both instructions take and give subnormal
// numbers. N = 4096, F = 784, us (all on the fp32 instruction in brackets): inference
// one row with inf 1300 (604), 1% of the rows with NaN 395 (602), all of X subnormal 1310
// (602); training 907 (917), 405 (919), 1560 (916).
//
// Work split. A workgroup holds a tile of 32 NTILES samples; each wave takes one
// unit of 64 dimensions per pass. B comes from L2 straight into registers (each
// fragment is used for NTILES tiles), X through LDS in chunks of 64 features,
// double-buffered, split into its parts on the way. Inference walks the
// slice's units and takes HardSign and Stage II after each pass; training walks
// its share of the sample tiles with one fixed unit per wave and adds each
// tile's signs to the class sums on the int8 matrix instruction
// (hd_train_breg.hip), which stay in registers to the end.
#include <algorithm>
#include <type_traits>

#include "hd_large.hpp"

namespace hd {

using namespace lg;

namespace {

// Groups of 16 features per X chunk: one X item (a row's group) per thread.
constexpr int chunk_groups(int ntiles) { return kThreads / (32 * ntiles); }
// A pass of two tiles against one of four, the split of B being the same (N = 10000,
// F = 784: 1000 us with two, 866 with four).
constexpr double kTwoTilePass = 0.6;
constexpr float kCHi = 0x1p50f;  // largest |C| in Stage II's three parts
constexpr float kHi = 0x1p50f;   // |X|, |B| up to which no sum of 2^20 products overflows

// Two floats rounded to bf16 (v_cvt_pk_bf16_f32), and the floats they stand for.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t round_pair(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float low_of(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float high_of(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two values into a word of each part (b in the upper half), in two halves. rest:
// the trailing parts' bits so far; a value that is not the sum of its parts leaves
// one in the lower half.
__device__ __forceinline__ void split2_lead(float a, float b, uint32_t& w0, float (&r)[2]) {
  w0 = round_pair(a, b);
  r[0] = a - low_of(w0);
  r[1] = b - high_of(w0);
}
__device__ __forceinline__ void split2_rest(const float (&r)[2], uint32_t& w1, uint32_t& w2,
                                            uint32_t& rest) {
  w1 = round_pair(r[0], r[1]);
  const float sa = r[0] - low_of(w1), sb = r[1] - high_of(w1);
  rest |= __float_as_uint(sa) | __float_as_uint(sb);
  w2 = round_pair(sa, sb);
}
__device__ __forceinline__ void split2(float a, float b, uint32_t& w0, uint32_t& w1, uint32_t& w2,
                                       uint32_t& rest) {
  float r[2];
  split2_lead(a, b, w0, r);
  split2_rest(r, w1, w2, rest);
}

// Eight values (slot order) into their three parts.
__device__ __forceinline__ void split8(const float (&x)[8], uint4 (&p)[3], uint32_t& rest) {
  uint32_t w[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) split2(x[2 * i], x[2 * i + 1], w[0][i], w[1][i], w[2][i], rest);
#pragma unroll
  for (int q = 0; q < 3; ++q) p[q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
}

__device__ __forceinline__ void split8(const float4& a, const float4& b, uint4 (&p)[3], uint32_t& rest) {
  const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  split8(x, p, rest);
}

// Order of the six products, parts of B and of X: lh, mh, mm, hh, hm, hl.
constexpr int kPartB[6] = {2, 1, 1, 0, 0, 0}, kPartX[6] = {0, 0, 1, 0, 1, 2};

// Largest magnitude but NaN among the 16-byte words at byte offsets offset_of(0),
// offset_of(1), ... of p, over a workgroup's threads; to the first offset past the end.
template <class Fn>
__device__ __forceinline__ float largest(const float* p, int64_t bytes, int tid, Fn&& offset_of) {
  constexpr int kBatch = 16;  // loads in flight
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p), 0, (int)bytes, 0x00020000);
  float m = 0.0f;
  for (uint32_t i = tid; offset_of(i - tid) < bytes; i += kBatch * kThreads) {
    float4 v[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      v[j] = __builtin_bit_cast(
          float4, __builtin_amdgcn_raw_buffer_load_b128(rs, offset_of(i + j * kThreads), 0, 0));
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      m = fmaxf(m, fmaxf(fmaxf(fabsf(v[j].x), fabsf(v[j].y)), fmaxf(fabsf(v[j].z), fabsf(v[j].w))));
  }
  return m;
}

struct X3Args {
  const float* X;
  const void* B;  // packed fragments, or row-major [F][D]
  const void* C;  // packed fragments, or row-major [K][D] (inference)
  const int32_t* y;
  int32_t *labels, *counts;
  float* scores;
  int N, F, D, K;
  int DS;        // inference: slices of D; training: groups of sample tiles
  void* workspace;
};

// RAW: B (and C) row-major. TRAIN: class sums, else inference. Returns true, with
// nothing written, where the sums are to be taken with CAREFUL (below).
template <int NTILES, int KB, bool RAW, bool TRAIN, bool CAREFUL>
__device__ __forceinline__ bool x3_body(const X3Args& a, int tid) {
  constexpr int NT = 32 * NTILES;
  constexpr int kGC = chunk_groups(NTILES);
  constexpr int IPT = NT * kGC / kThreads;  // X items (one row's 16 features) per thread
  constexpr int kSw = 8 / kGC;              // bank spread of a row's groups
  // S of four tiles lies in LDS between the passes, which frees its registers
  constexpr bool kPark = !TRAIN && NTILES == 4;
  constexpr int kBuf = kGC * NTILES * 3 * 1024;  // bytes of one X buffer
  static_assert(NTILES % 2 == 0 && IPT == 1 && (!kPark || KB == 1), "tiles in pairs");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ unsigned char s_row[NT];  // rows that hold a value that is not the sum of its parts
  const int lane = tid & 63, half = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N, F = a.F, D = a.D, K = a.K;
  const int G = (F + 15) / 16, nch = (G + kGC - 1) / kGC;
  const int nfs8 = (F + 7) / 8;
  const int units = (D + 63) / 64;
  const int ntiles = (int)cdiv(N, NT);
  // inference: tile, units [u_begin, u_end); training: one unit group, tiles [t_begin, t_end)
  int t_begin, t_end, u_begin, u_end;
  int slice = 0;
  if constexpr (TRAIN) {
    const int ncg = (units + kWaves - 1) / kWaves;
    const int cg = blockIdx.x % ncg, g = blockIdx.x / ncg;
    u_begin = cg * kWaves;
    u_end = min(units, u_begin + kWaves);
    t_begin = (int)((int64_t)ntiles * g / a.DS);
    t_end = (int)((int64_t)ntiles * (g + 1) / a.DS);
  } else {
    slice = blockIdx.x % a.DS;
    t_begin = blockIdx.x / a.DS;
    t_end = t_begin + 1;
    u_begin = (int)((int64_t)units * slice / a.DS);
    u_end = (int)((int64_t)units * (slice + 1) / a.DS);
  }

  // ---- X: chunk ch of tile t, item i of this thread -------------------------
  // Consecutive threads take the groups of a row's chunk.
  const int xg = tid % kGC;
  auto x_load = [&](int t, int ch, float4 (&v)[IPT][4]) __attribute__((always_inline)) {
    const int64_t n0 = (int64_t)t * NT;
    const int rows = (int)min((int64_t)NT, (int64_t)N - n0);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(a.X + n0 * F), 0, rows * F * 4, 0x00020000);
    const int f0 = (ch * kGC + xg) * 16;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int row = i * (kThreads / kGC) + tid / kGC;
      const int off = row < rows && f0 < F ? (row * F + f0) * 4 : 0x7ffffff0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        v[i][q] = __builtin_bit_cast(
            float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * q, 0, 0));
    }
  };
  // features past F (of the next row) to zero
  auto x_mask = [&](int ch, float4 (&v)[IPT][4]) __attribute__((always_inline)) {
    const int left = F - (ch * kGC + xg) * 16;
    if ((ch + 1) * kGC * 16 > F) {
#pragma unroll
      for (int i = 0; i < IPT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (4 * q + 0 >= left) v[i][q].x = 0.0f;
          if (4 * q + 1 >= left) v[i][q].y = 0.0f;
          if (4 * q + 2 >= left) v[i][q].z = 0.0f;
          if (4 * q + 3 >= left) v[i][q].w = 0.0f;
        }
    }
  };
  // Fragment of group g, tile t, part p: 1 KiB at ((g NTILES + t) 3 + p) of the
  // buffer; lane (n, h) at position (32 h + n) ^ kSw g (the groups of a row are
  // written together: distinct banks). Slot e of half h is feature
  // 8 (e / 4) + 2 (e % 4) + h of the group, as in the packed fp32 fragments of B.
  auto x_put = [&](int buf, const float4 (&v)[IPT][4], int i, uint32_t& rest)
                   __attribute__((always_inline)) {
    const int row = i * (kThreads / kGC) + tid / kGC;
    unsigned char* dst = lds + buf * kBuf + (xg * NTILES + row / 32) * 3 * 1024;
    const float ev[8] = {v[i][0].x, v[i][0].z, v[i][1].x, v[i][1].z,
                         v[i][2].x, v[i][2].z, v[i][3].x, v[i][3].z};
    const float od[8] = {v[i][0].y, v[i][0].w, v[i][1].y, v[i][1].w,
                         v[i][2].y, v[i][2].w, v[i][3].y, v[i][3].w};
    uint4 p[3];
    split8(ev, p, rest);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      *reinterpret_cast<uint4*>(dst + q * 1024 + ((row % 32) ^ (kSw * xg)) * 16) = p[q];
    split8(od, p, rest);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      *reinterpret_cast<uint4*>(dst + q * 1024 + ((32 + row % 32) ^ (kSw * xg)) * 16) = p[q];
  };
  auto x_get1 = [&](int buf, int g, int t, int q, uint4& x) __attribute__((always_inline)) {
    x = *reinterpret_cast<const uint4*>(lds + buf * kBuf + (g * NTILES + t) * 3 * 1024 +
                                        (lane ^ (kSw * g)) * 16 + q * 1024);
  };
  auto x_get = [&](int buf, int g, int t, uint4 (&x)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 3; ++q) x_get1(buf, g, t, q, x[q]);
  };

  // ---- B: the 16 features of group g, two blocks of 32 dimensions ------------
  const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.B), 0, RAW ? F * D * 4 : 2 * units * nfs8 * 1024, 0x00020000);
  auto b_load1 = [&](int u, int g, int b, int q, float4& v) __attribute__((always_inline)) {
    if constexpr (RAW) {
      // past F the offset is past the matrix (zero); past column D the next row's
      // values meet zero rows of C, or are not added
      const uint32_t off = (uint32_t)((16 * g + 8 * q + half) * D + 64 * u + 32 * b + col) * 4u;
      float t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        t[j] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(brs, off + (uint32_t)(8 * j * D), 0, 0));
      v = make_float4(t[0], t[1], t[2], t[3]);
    } else {
      const int fs = 2 * g + q;
      const int off = fs < nfs8 ? ((2 * u + b) * nfs8 + fs) * 1024 + lane * 16 : 0x7ffffff0;
      v = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(brs, off, 0, 0));
    }
  };
  auto b_load = [&](int u, int g, float4 (&v)[2][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 2; ++q) b_load1(u, g, b, q, v[b][q]);
  };

  // The leading parts' products and the others' are summed apart: the others
  // are 2^-8 of them, so only one rounding in 16 features counts (the fp32
  // instruction: eight). acc holds the whole sum after a pass.
  f32x16 acc[NTILES][2], low[NTILES][2];
  auto mma = [&](const uint4& bp, const uint4& xp, f32x16& c) __attribute__((always_inline)) {
    if constexpr (TRAIN)  // samples in rows
      TrBF16::stage1(c, xp, bp);
    else  // dimensions in rows
      TrBF16::stage1(c, bp, xp);
  };

  // One group: NTILES/2 phases of two tiles, 24 matrix instructions each, on B
  // parts bp and X parts x (phase 0's at entry, the next group's phase 0 at
  // exit). Meanwhile the next group's B parts are split from `raw`, which then
  // takes group gload's fragments. In a chunk's last group this thread's X
  // items of the next chunk are split into buffer nb; after the barrier in its
  // last phase, for which X is in registers by then, every wave has read what
  // it needs of this chunk and the next one is complete.
  auto group = [&](uint4 (&bp)[2][3], uint4 (&x)[2][3], float4 (&raw)[2][2], int u, int gload,
                   int buf, int gl, uint32_t (&restb)[2], auto last, float4 (&xv)[IPT][4], int nb,
                   uint32_t (&restx)[IPT]) __attribute__((always_inline)) {
    constexpr bool kLast = decltype(last)::value;
    constexpr int kPh = NTILES / 2;
    // Behind each matrix instruction (32 cycles, of which it takes 4 to issue) goes
    // half a pair's split, five or seven instructions of 4 cycles, and a load or two:
    // left to itself the compiler gathers the splits in blocks that the matrix unit
    // waits for.
    constexpr int kSlots = 24 * kPh;
    constexpr int kBar = kSlots - 12;                   // the barrier's slot
    constexpr int kXSlots = kPh == 1 ? 12 : 24;         // X's 16 halves: the first slots
    constexpr int kB0 = kPh == 1 ? 12 : 24, kBSlots = kPh == 1 ? 12 : 16;  // B's halves
    uint32_t bw[2][3][4], xw[3][4];
    uint4 xn[2][3];
    float br[2], xr[2];
    // half h of B's 16: pair h / 2 is (k, k + 1) of block b; a fragment's registers
    // take the next one once both of its pairs are read
    auto b_half = [&](int h) __attribute__((always_inline)) {
      const int b = h >> 3, k = (h >> 1) & 3;
      if (h % 2 == 0) {
        const float4 v = raw[b][k >> 1];
        split2_lead(k & 1 ? v.z : v.x, k & 1 ? v.w : v.y, bw[b][0][k], br);
        // (computed here, not where it is next used)
        asm volatile("" : "+v"(bw[b][0][k]), "+v"(br[0]), "+v"(br[1]));
        if (k & 1) b_load1(u, gload, b, k >> 1, raw[b][k >> 1]);
      } else {
        split2_rest(br, bw[b][1][k], bw[b][2][k], restb[b]);
        asm volatile("" : "+v"(bw[b][1][k]), "+v"(bw[b][2][k]));
      }
    };
    auto x_half = [&](int h) __attribute__((always_inline)) {  // half h of X's 16
      const int odd = h >> 3, k = (h >> 1) & 3;
      if (h % 2 == 0) {
        const float4 v = xv[0][k];
        split2_lead(odd ? v.y : v.x, odd ? v.w : v.z, xw[0][k], xr);
        asm volatile("" : "+v"(xw[0][k]), "+v"(xr[0]), "+v"(xr[1]));
      } else {
        split2_rest(xr, xw[1][k], xw[2][k], restx[0]);
        asm volatile("" : "+v"(xw[1][k]), "+v"(xw[2][k]));
        if (k == 3) {
          const int row = tid / kGC;
          unsigned char* dst = lds + nb * kBuf + (xg * NTILES + row / 32) * 3 * 1024 +
                               ((32 * odd + row % 32) ^ (kSw * xg)) * 16;
#pragma unroll
          for (int q = 0; q < 3; ++q)
            *reinterpret_cast<uint4*>(dst + q * 1024) =
                make_uint4(xw[q][0], xw[q][1], xw[q][2], xw[q][3]);
        }
      }
    };
    // B's trailing and middle parts are done with by the barrier's slot, where the
    // next group's take over their registers.
#pragma unroll
    for (int sl = 0; sl < kSlots; ++sl) {
      const int ph = sl / 24, m = sl % 24, c = m >> 2, t = (m >> 1) & 1, b = m & 1;
      mma(bp[b][kPartB[c]], x[t][kPartX[c]], c == 3 ? acc[2 * ph + t][b] : low[2 * ph + t][b]);
      if (kLast && sl == kBar) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      // X of the next phase, a fragment behind each of six
      const int rd = ph + 1 < kPh || !kLast ? m : sl - kBar;
      if (rd >= 0 && rd < 6) {
        if (ph + 1 < kPh)
          x_get1(buf, gl, 2 * ph + 2 + (rd & 1), rd >> 1, xn[rd & 1][rd >> 1]);
        else
          x_get1(kLast ? nb : buf, kLast ? 0 : gl + 1, rd & 1, rd >> 1, xn[rd & 1][rd >> 1]);
      }
      if constexpr (kLast) {
#pragma unroll
        for (int h = sl * 16 / kXSlots; h < (sl + 1) * 16 / kXSlots && h < 16; ++h) x_half(h);
      }
      if (sl >= kB0) {
#pragma unroll
        for (int h = (sl - kB0) * 16 / kBSlots; h < (sl - kB0 + 1) * 16 / kBSlots && h < 16; ++h)
          b_half(h);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (m == 23) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int q = 0; q < 3; ++q) x[t2][q] = xn[t2][q];
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        bp[b][q] = make_uint4(bw[b][q][0], bw[b][q][1], bw[b][q][2], bw[b][q][3]);
  };

  // ---- scores or class sums ---------------------------------------------------
  f32x4* park = reinterpret_cast<f32x4*>(lds + 2 * kBuf) + wave * (NTILES * 4 * 64) + lane;
  f32x16 sacc[TRAIN ? 1 : NTILES][KB];  // S^T of this wave's units
  i32x16 cacc[TRAIN ? 2 : 1][KB];       // class sums of this wave's unit
  float most = 0.0f;                    // largest |V| of all passes, or NaN
  // The C values of class block kb against the unit's dimensions.
  const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.C), 0, RAW && !TRAIN ? K * D * 4 : 0, 0x00020000);
  auto c_load = [&](int u, int kb, float4 (&cv)[2][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (RAW) {
          // past K the offset is past the matrix (zero); past column D the next
          // row's values, cleared
          const int d = 64 * u + 32 * b + 8 * q + 4 * half;
          const float4 v = __builtin_bit_cast(
              float4, __builtin_amdgcn_raw_buffer_load_b128(
                          crs, (uint32_t)((32 * kb + col) * D + d) * 4u, 0, 0));
          cv[b][q] = make_float4(d < D ? v.x : 0.0f, d + 1 < D ? v.y : 0.0f,
                                 d + 2 < D ? v.z : 0.0f, d + 3 < D ? v.w : 0.0f);
        } else {
          cv[b][q] = static_cast<const float4*>(
              a.C)[(((int64_t)(2 * u + b) * KB + kb) * 4 + q) * 64 + lane];
        }
      }
  };
  auto unpark = [&](int i) __attribute__((always_inline)) {
    if constexpr (kPark) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = park[(i * 4 + q) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) sacc[i][0][4 * q + r] = v[r];
      }
    }
  };
  auto put_park = [&](int i) __attribute__((always_inline)) {
    if constexpr (kPark) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        park[(i * 4 + q) * 64] = f32x4{sacc[i][0][4 * q], sacc[i][0][4 * q + 1],
                                       sacc[i][0][4 * q + 2], sacc[i][0][4 * q + 3]};
    }
  };
  auto clear_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
#pragma unroll
        for (int i = 0; i < (TRAIN ? 1 : NTILES); ++i) sacc[i][kb][r] = 0.0f;
#pragma unroll
        for (int i = 0; i < (TRAIN ? 2 : 1); ++i) cacc[i][kb][r] = 0;
      }
    if constexpr (kPark) {
#pragma unroll
      for (int i = 0; i < NTILES; ++i) put_park(i);
    }
  };
  clear_sums();
  auto note_most = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; r += 2)
        most = __builtin_elementwise_maximum(
            most, __builtin_elementwise_maximum(fabsf(acc[i][b][r]), fabsf(acc[i][b][r + 1])));
  };
  // Stage II of a finished unit: C in three parts against HardSign(V), or on
  // the fp32 instruction where a value of C is larger than 2^50 or has no three
  // parts (which are exact against +-1 at any size). c0: class block 0.
  auto stage2 = [&](int u, const float4 (&c0)[2][4]) __attribute__((always_inline)) {
    if constexpr (!TRAIN) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        float4 cv[2][4];
        if (kb > 0) {
          c_load(u, kb, cv);
        } else {
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) cv[b][q] = c0[b][q];
        }
        uint4 cp[2][2][3];  // [b][h][part]
        uint32_t rest = 0;
        float mx = 0.0f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            mx = fmaxf(fmaxf(fmaxf(mx, fabsf(cv[b][q].x)), fabsf(cv[b][q].y)),
                       fmaxf(fabsf(cv[b][q].z), fabsf(cv[b][q].w)));
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int h = 0; h < 2; ++h) split8(cv[b][2 * h], cv[b][2 * h + 1], cp[b][h], rest);
        const bool native_c = __builtin_amdgcn_ballot_w64(mx > kCHi || (rest & 0xffffu)) != 0;
#pragma unroll
        for (int i = 0; i < NTILES; ++i) {
          unpark(i);
          if (kb == 0) note_most(i);
          if (!native_c) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const f32x16& v = acc[i][b];
                uint4 hb;
                hb.x = sign_pair(v[8 * h + 0], v[8 * h + 1]);
                hb.y = sign_pair(v[8 * h + 2], v[8 * h + 3]);
                hb.z = sign_pair(v[8 * h + 4], v[8 * h + 5]);
                hb.w = sign_pair(v[8 * h + 6], v[8 * h + 7]);
#pragma unroll
                for (int p = 0; p < 3; ++p) TrBF16::stage1(sacc[i][kb], cp[b][h][p], hb);
              }
          } else {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const float c4[4] = {cv[b][q].x, cv[b][q].y, cv[b][q].z, cv[b][q].w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                  sacc[i][kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                      c4[j], hardsign(acc[i][b][4 * q + j]), sacc[i][kb], 0, 0, 0);
              }
          }
          put_park(i);
        }
      }
    }
  };
  auto class_sums = [&](int t) __attribute__((always_inline)) {
    if constexpr (TRAIN) {
      const int64_t n0 = (int64_t)t * NT;
      const int rows = (int)min((int64_t)NT, (int64_t)N - n0);
      const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<int32_t*>(a.y + n0), 0, rows * 4, 0x00020000);
#pragma unroll
      for (int i = 0; i < NTILES; ++i) {
        int yl[16];  // samples 8 q + 4 half + j of the tile
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const i32x4 v = __builtin_bit_cast(
              i32x4, __builtin_amdgcn_raw_buffer_load_b128(
                         yrs, (32 * i + 8 * q + 4 * half) * 4, 0, 0));
#pragma unroll
          for (int j = 0; j < 4; ++j) yl[4 * q + j] = v[j];
        }
        if (32 * i + 32 > rows) {  // rows past the last one have no label
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (32 * i + 8 * q + 4 * half + j >= rows) yl[4 * q + j] = -1;
        }
        note_most(i);
        i32x4 h[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x16& v = acc[i][b];
            h[b][q] = (int)(((v[4 * q] >= 0.0f ? 0x01u : 0xffu) |
                             (v[4 * q + 1] >= 0.0f ? 0x0100u : 0xff00u)) |
                            ((v[4 * q + 2] >= 0.0f ? 0x010000u : 0xff0000u) |
                             (v[4 * q + 3] >= 0.0f ? 0x01000000u : 0xff000000u)));
          }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const int k = 32 * kb + col;
          i32x4 oh;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            oh[q] = (int)(((yl[4 * q] == k ? 0x01u : 0u) | (yl[4 * q + 1] == k ? 0x0100u : 0u)) |
                          ((yl[4 * q + 2] == k ? 0x010000u : 0u) |
                           (yl[4 * q + 3] == k ? 0x01000000u : 0u)));
#pragma unroll
          for (int b = 0; b < 2; ++b)
            cacc[b][kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(oh, h[b], cacc[b][kb], 0, 0, 0);
        }
      }
    }
  };

  // ---- passes -------------------------------------------------------------------
  if (t_begin >= t_end || u_begin >= u_end) return false;
  const int npass = TRAIN ? t_end - t_begin : (u_end - u_begin + kWaves - 1) / kWaves;
  // this wave's unit in pass ps (a valid unit when it has none: computed, discarded)
  auto unit_of = [&](int ps) {
    const int u = TRAIN ? u_begin + wave : u_begin + ps * kWaves + wave;
    return u < u_end ? u : u_begin;
  };
  if constexpr (CAREFUL) {
    // All passes again: the same products in the same order, nothing overlapped, and
    // then on the fp32 matrix instruction, from which a sum is taken if its row or
    // its column holds a value that is not the sum of its parts, or if it is not
    // finite. So a sample's result does not depend on its neighbours. (Of the other
    // sums the sign is kept meanwhile.)
    constexpr int kPitch = kGC * 16 + 4;  // floats per row
    float* xf = reinterpret_cast<float*>(lds);
    for (int ps = 0; ps < npass; ++ps) {
      const int t = TRAIN ? t_begin + ps : t_begin;
      const int u = unit_of(ps);
      auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NTILES; ++i)
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][b][r] = low[i][b][r] = 0.0f;
      };
      clear();
      uint32_t restb[2] = {}, restx[IPT] = {};
      float4 v[IPT][4], bv[2][2];
      for (int ch = 0; ch < nch; ++ch) {
        x_load(t, ch, v);
        x_mask(ch, v);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IPT; ++i) x_put(0, v, i, restx[i]);
        __syncthreads();
        const int ng = min(kGC, G - ch * kGC);
        for (int gl = 0; gl < ng; ++gl) {
          uint4 bp[2][3], x[3];
          b_load(u, ch * kGC + gl, bv);
#pragma unroll
          for (int b = 0; b < 2; ++b) split8(bv[b][0], bv[b][1], bp[b], restb[b]);
#pragma unroll
          for (int i = 0; i < NTILES; ++i) {
            x_get(0, gl, i, x);
#pragma unroll
            for (int c = 0; c < 6; ++c)
#pragma unroll
              for (int b = 0; b < 2; ++b)
                mma(bp[b][kPartB[c]], x[kPartX[c]], c == 3 ? acc[i][b] : low[i][b]);
          }
        }
      }
      // Which sums are taken from the fp32 instruction, and the others' signs: bit
      // 16 b + r of tile i's word for sum r of block b.
      if (tid < NT) s_row[tid] = 0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < IPT; ++i)
        if (restx[i] & 0xffffu) s_row[i * (kThreads / kGC) + tid / kGC] = 1;
      __syncthreads();
      uint32_t pos[NTILES], again[NTILES], cols[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const uint64_t m = __builtin_amdgcn_ballot_w64((restb[b] & 0xffffu) != 0);
        cols[b] = (uint32_t)m | (uint32_t)(m >> 32);
      }
      bool any = false;
#pragma unroll
      for (int i = 0; i < NTILES; ++i) {
        const uint32_t rows = (uint32_t)__builtin_amdgcn_ballot_w64(s_row[32 * i + col] != 0);
        pos[i] = again[i] = 0;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          // this lane's bit of what lies in lanes, the register's of what lies in rows
          const uint32_t mine = (TRAIN ? cols[b] : rows) >> col & 1u;
          const uint32_t regs = (TRAIN ? rows : cols[b]) >> (4 * half);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float a = acc[i][b][r] + low[i][b][r];
            const bool from = mine | (regs >> (8 * (r >> 2) + (r & 3)) & 1u) |
                              !(fabsf(a) < __builtin_huge_valf());
            pos[i] |= a >= 0.0f ? 1u << (16 * b + r) : 0u;
            again[i] |= from ? 1u << (16 * b + r) : 0u;
          }
        }
        any |= again[i] != 0;
      }
      clear();
      if (__syncthreads_or(any)) {
        for (int ch = 0; ch < nch; ++ch) {
          x_load(t, ch, v);
          x_mask(ch, v);
          __syncthreads();
#pragma unroll
          for (int i = 0; i < IPT; ++i) {
            float4* dst = reinterpret_cast<float4*>(
                xf + (i * (kThreads / kGC) + tid / kGC) * kPitch + xg * 16);
            dst[0] = make_float4(v[i][0].x, v[i][0].z, v[i][1].x, v[i][1].z);
            dst[1] = make_float4(v[i][0].y, v[i][0].w, v[i][1].y, v[i][1].w);
            dst[2] = make_float4(v[i][2].x, v[i][2].z, v[i][3].x, v[i][3].z);
            dst[3] = make_float4(v[i][2].y, v[i][2].w, v[i][3].y, v[i][3].w);
          }
          __syncthreads();
          const int ng = min(kGC, G - ch * kGC);
          for (int gl = 0; gl < ng; ++gl) {
            b_load(u, ch * kGC + gl, bv);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
              for (int i = 0; i < NTILES; ++i) {
                const uint4 x = *reinterpret_cast<const uint4*>(
                    xf + (32 * i + col) * kPitch + gl * 16 + 8 * q + 4 * half);
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                  if constexpr (TRAIN)
                    TrF32::stage1(acc[i][b], x, bitcast<uint4>(bv[b][q]));
                  else
                    TrF32::stage1(acc[i][b], bitcast<uint4>(bv[b][q]), x);
                }
              }
          }
        }
      }
#pragma unroll
      for (int i = 0; i < NTILES; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float was = pos[i] >> (16 * b + r) & 1u ? 1.0f : -1.0f;
            acc[i][b][r] = again[i] >> (16 * b + r) & 1u ? acc[i][b][r] : was;
          }
      if constexpr (TRAIN) {
        class_sums(t);
      } else if (u_begin + ps * kWaves + wave < u_end) {
        float4 c0[2][4];
        c_load(u, 0, c0);
        stage2(u, c0);
      }
    }
  } else {
    float4 xv[IPT][4];
    float4 raw[2][2], r0[2][2];
    uint4 bp[2][3], xc[2][3];
    uint32_t restb[2] = {}, restx[IPT] = {};  // trailing parts' bits of all passes
    int buf = 0;
    auto b_start = [&](int u) __attribute__((always_inline)) {
      b_load(u, 0, r0);
      b_load(u, 1, raw);
    };
    b_start(unit_of(0));
    x_load(t_begin, 0, xv);
    x_mask(0, xv);
#pragma unroll
    for (int i = 0; i < IPT; ++i) x_put(0, xv, i, restx[i]);
    __syncthreads();
    x_get(0, 0, 0, xc[0]);
    x_get(0, 0, 1, xc[1]);

    for (int ps = 0; ps < npass; ++ps) {
      const int t = TRAIN ? t_begin + ps : t_begin;
      const int u = unit_of(ps);
      const int tn = TRAIN ? min(t + 1, t_end - 1) : t;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        split8(r0[b][0], r0[b][1], bp[b], restb[b]);
      }
#pragma unroll
      for (int i = 0; i < NTILES; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][b][r] = low[i][b][r] = 0.0f;
      for (int ch = 0; ch < nch; ++ch) {
        const bool lastc = ch + 1 == nch;
        const int nb = buf ^ 1, ng = min(kGC, G - ch * kGC), g0 = ch * kGC;
        // next chunk of X: of this tile, or the first of the next pass's tile
        x_load(lastc ? tn : t, lastc ? 0 : ch + 1, xv);
        for (int gl = 0; gl + 1 < ng; ++gl)
          group(bp, xc, raw, u, g0 + gl + 2, buf, gl, restb, std::false_type{}, xv, nb, restx);
        x_mask(lastc ? 0 : ch + 1, xv);
        group(bp, xc, raw, u, g0 + ng + 1, buf, ng - 1, restb, std::true_type{}, xv, nb, restx);
        buf = nb;
      }
#pragma unroll
      for (int i = 0; i < NTILES; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[i][b] += low[i][b];
      float4 c0[2][4];
      if constexpr (!TRAIN) c_load(u, 0, c0);
      if (ps + 1 < npass) b_start(unit_of(ps + 1));
      if constexpr (TRAIN)
        class_sums(t);
      else if (u_begin + ps * kWaves + wave < u_end)
        stage2(u, c0);
    }

    // outside the range of the split
    uint32_t rest = restb[0] | restb[1];
#pragma unroll
    for (int i = 0; i < IPT; ++i) rest |= restx[i];
    if (__syncthreads_or(rest & 0xffffu)) return true;
    if (__builtin_expect(__syncthreads_or(!(most < __builtin_huge_valf())), 0)) {
      // NaN in X or B makes its sums NaN on either instruction. Without inf or values
      // that could overflow there is nothing else.
      int first = tid;  // (a thread index of this part's own: see x3_kernel)
      asm volatile("" : "+v"(first));
      float big = 0.0f;  // largest magnitude but NaN
      for (int t = t_begin; t < t_end; ++t) {
        const int64_t n0 = (int64_t)t * NT;
        const int64_t count = min((int64_t)NT, (int64_t)N - n0) * F;
        big = fmaxf(big, largest(a.X + n0 * F, count * 4, first, [](uint32_t i) { return 16u * i; }));
      }
      const float* B = static_cast<const float*>(a.B);
      if constexpr (RAW) {
        // rows of the slice's columns, four at a time
        const uint32_t words = 16u * (u_end - u_begin);
        big = fmaxf(big, largest(B + 64 * u_begin, ((int64_t)F * D - 64 * u_begin) * 4, first,
                                 [&](uint32_t i) {
                                   const uint32_t f = i / words;
                                   return f < (uint32_t)F
                                              ? (f * (uint32_t)D + 4u * (i - f * words)) * 4u
                                              : 0xfffffff0u;
                                 }));
      } else {
        const int64_t per = (int64_t)2 * nfs8 * 256;  // floats per unit
        big = fmaxf(big, largest(B + u_begin * per, (u_end - u_begin) * per * 4, first,
                                 [](uint32_t i) { return 16u * i; }));
      }
      if (__syncthreads_or(big > kHi)) return true;
    }
  }

  if constexpr (TRAIN) {
    if (u_begin + wave >= u_end) return false;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int d = 64 * (u_begin + wave) + 32 * b + col;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int k = 32 * kb + 8 * (r >> 2) + 4 * half + (r & 3);
          if (k < K && d < D && cacc[b][kb][r] != 0)
            atomicAdd(&a.counts[(int64_t)k * D + d], cacc[b][kb][r]);
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NTILES; ++i) unpark(i);
    __syncthreads();
    finish_tile<NTILES, KB>(sacc, lds, a.labels, a.scores, N, K, a.DS, slice, t_begin * NT,
                            a.workspace);
  }
  return false;
}

// The careful form starts from a thread index of its own, which the compiler does
// not know to be the same: it would keep what both compute from it in registers.
template <int NTILES, int KB, bool RAW, bool TRAIN>
__device__ __forceinline__ void x3_kernel(const X3Args& a) {
  if (__builtin_expect(x3_body<NTILES, KB, RAW, TRAIN, false>(a, threadIdx.x), 0)) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    x3_body<NTILES, KB, RAW, TRAIN, true>(a, tid);
  }
}

template <int NTILES, int KB, bool RAW>
__global__ __launch_bounds__(kThreads, 1) void large_fused_kernel_x3(X3Args a) {
  x3_kernel<NTILES, KB, RAW, false>(a);
}

template <int NTILES, int KB, bool RAW>
__global__ __launch_bounds__(kThreads, 1) void bundle_mfma_kernel_x3(X3Args a) {
  x3_kernel<NTILES, KB, RAW, true>(a);
}

constexpr size_t x3_lds(int ntiles, int kb, bool train) {
  size_t bufs = (size_t)2 * chunk_groups(ntiles) * ntiles * 3 * 1024;
  if (!train && ntiles == 4) bufs += (size_t)kWaves * 4 * 4096;  // S between the passes
  const size_t red = train ? 0 : (size_t)kWaves * 32 * ntiles * 32 * kb * 4;
  return bufs > red ? bufs : red;
}

template <auto Kernel>
hipError_t launch_x3_kernel(const X3Args& a, int grid, size_t lds, hipStream_t stream) {
  static PerDeviceOnce once;
  const hipError_t attr = once_per_device(once, [&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(Kernel, dim3((unsigned)grid), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

// Sample tiles per workgroup in training: two; four with long rows and enough tiles
// to fill the chip (the class sums at the end of a pass, with the registers full,
// then weigh less than half the loads of B): packed N = 4096, F = 784 357 against 383
// us, raw N = 2048 201 against 222 us, but F = 100, N = 10000 196 against 178 us and
// N = 300, F = 617 49 against 30 us.
int train_tiles(int64_t N, int64_t F, int64_t D, int kb) {
  return kb <= 2 && F >= 512 && cdiv(N, 128) * cdiv(D, 256) >= num_cus() ? 4 : 2;
}

template <int KB, int NT>
hipError_t launch_infer(const X3Args& a, bool raw, int grid, hipStream_t stream) {
  constexpr size_t lds = x3_lds(NT, KB, false);
  static_assert(lds <= kLdsBytes, "LDS");
  return raw ? launch_x3_kernel<&large_fused_kernel_x3<NT, KB, true>>(a, grid, lds, stream)
             : launch_x3_kernel<&large_fused_kernel_x3<NT, KB, false>>(a, grid, lds, stream);
}

template <int NT, int KB, bool RAW>
hipError_t launch_train(const X3Args& a, int grid, hipStream_t stream) {
  return launch_x3_kernel<&bundle_mfma_kernel_x3<NT, KB, RAW>>(a, grid, x3_lds(NT, KB, true),
                                                               stream);
}

// Offsets into B, and into C as given, are 32-bit; row-major B is read up to 64
// rows past F, C up to 62 past K.
bool x3_sizes_ok(int64_t F, int64_t D, int64_t K, bool raw) {
  if (cdiv(K, 32) > 4 || F > (1 << 20)) return false;
  if (raw)
    return D <= (1 << 22) && F * D * 4 < ((int64_t)1 << 31) && K * D * 4 < ((int64_t)1 << 31);
  return cdiv(D, 64) * 2 * cdiv(F, 8) * 1024 < ((int64_t)1 << 31);
}

}  // namespace

X3Plan x3_plan(int64_t N, int64_t F, int64_t D, int64_t K, int act, bool raw, size_t ws_cap) {
  X3Plan p{};
  if (act != 0 || !x3_sizes_ok(F, D, K, raw)) return p;
  p.kb = kb_of(K);
  const int64_t cus = num_cus(), units = cdiv(D, 64), passes = cdiv(units, kWaves);
  // Sample tiles per workgroup: four, or two, where more class blocks' scores take
  // the registers or where the passes of four are too few for the chip (N = 500,
  // F = 1000, D = 4096, 64 workgroups of one pass: 77 us, with two tiles 49; on the
  // fp32 instruction 60).
  double best = -1.0;
  for (int nt : {4, 2}) {
    if (nt == 4 && p.kb > 1) continue;
    const double pass = nt == 4 ? 1.0 : kTwoTilePass;
    const int64_t tiles = cdiv(N, 32 * nt);
    // Whole rounds of one tile per compute unit unsplit, the tiles left over split
    // over D: the fewest rounds, each a slice's passes and about half a pass (at
    // F = 784) of starting and handing over. A slice has whole passes.
    const int64_t head = std::min(N, tiles / cus * cus * 32 * nt);
    const int64_t rest = N - head, rt = cdiv(rest, 32 * nt);
    int ds = 1;
    const double over = 400.0 / (double)F;
    double cost = (double)cdiv(rt, cus) * (pass * (double)passes + over);
    for (int d = 2; rest > 0 && d <= 64 && d <= passes; ++d) {
      if (sizeof(float) * (size_t)d * rest * K > ws_cap) break;
      const double c =
          (double)cdiv(rt * d, cus) * (pass * (double)cdiv(cdiv(units, d), kWaves) + over);
      if (c < 0.98 * cost) {
        cost = c;
        ds = d;
      }
    }
    cost += (double)(tiles / cus) * (pass * (double)passes + over);
    if (best >= 0.0 && cost >= 0.95 * best) continue;
    best = cost;
    p.nt = nt;
    p.head = head;
    p.ds = ds;
    p.ws = rest > 0 && ds > 1 ? sizeof(float) * (size_t)ds * rest * K : 0;
    const double rounds =
        pass * ((double)(tiles / cus) * (double)passes +
                (double)cdiv(rt * ds, cus) * (double)cdiv(cdiv(units, ds), kWaves));
    p.us = 14.0 + rounds * (1.05 * (double)cdiv(F, 16) + 5.0);
  }
  p.ok = true;
  return p;
}

hipError_t launch_x3(const X3Plan& p, const void* X, const void* B, const void* C, bool raw,
                     int32_t* labels, float* scores, int64_t N, int64_t F, int64_t D, int64_t K,
                     void* ws, Clear* clear, hipStream_t stream) {
  auto go = [&](int64_t n0, int64_t n, int ds) {
    const X3Args a{(const float*)X + n0 * F, B, C, nullptr, labels + n0, nullptr,
                   scores ? scores + n0 * K : nullptr, (int)n, (int)F, (int)D, (int)K, ds, ws};
    const int grid = (int)(cdiv(n, 32 * p.nt) * ds);
    return p.nt == 4   ? launch_infer<1, 4>(a, raw, grid, stream)
           : p.kb == 1 ? launch_infer<1, 2>(a, raw, grid, stream)
           : p.kb == 2 ? launch_infer<2, 2>(a, raw, grid, stream)
                       : launch_infer<4, 2>(a, raw, grid, stream);
  };
  if (p.head > 0) {
    const hipError_t e = go(0, p.head, 1);
    if (e != hipSuccess || p.head == N) return e;
  }
  const hipError_t e = go(p.head, N - p.head, p.ds);
  if (e != hipSuccess || p.ds == 1) return e;
  return launch_reduce_slices(ws, labels + p.head, scores ? scores + p.head * K : nullptr,
                              N - p.head, K, p.ds, clear, stream);
}

// Not by N: a training set fed in chunks gets the signs, and so the counts, of one
// call. Against the kernels for fp32 instructions the packed form is faster at all
// sizes measured (N = 1 F = 4 D = 64 6.9 against 9.8 us, N = 60 F = 561 D = 2048 27
// against 70, N = 1024 F = 561 D = 10240 89 against 243), the raw form above one
// group of features (D = 2048: F = 16 N = 32 7.0 against 5.1 us, N = 65536 106 against
// 105; F = 24 7.5 against 6.9 and 118 against 169; F = 100 N = 32 10.5 against 17.4).
bool bundle_x3_ok(int64_t N, int64_t F, int64_t D, int64_t K, bool raw) {
  return N >= 1 && N <= (1 << 30) && x3_sizes_ok(F, D, K, raw) && (!raw || F > 16);
}

hipError_t launch_bundle_x3(const void* X, const void* B, bool raw, const int32_t* y,
                            int32_t* counts, int64_t N, int64_t F, int64_t D, int64_t K,
                            hipStream_t stream) {
  const int kb = kb_of(K), nt = train_tiles(N, F, D, kb);
  const int64_t cus = num_cus(), ncg = cdiv(cdiv(D, 64), kWaves);
  const int64_t tiles = cdiv(N, 32 * nt);
  // groups of sample tiles: the fewest rounds, each a group's tiles and about
  // half a tile (at F = 784) of starting and adding the sums into counts
  const double over = 400.0 / (double)F;
  int64_t best = 1;
  double cost = -1.0;
  for (int64_t g = 1; g <= tiles; ++g) {
    const double c = (double)cdiv(ncg * g, cus) * ((double)cdiv(tiles, g) + over);
    if (cost < 0 || c < 0.98 * cost) {
      cost = c;
      best = g;
    }
    if (ncg * g > 8 * cus) break;
  }
  const X3Args a{(const float*)X, B, nullptr, y, nullptr, counts, nullptr, (int)N, (int)F, (int)D,
                 (int)K, (int)best, nullptr};
  const int grid = (int)(ncg * best);
  if (nt == 4)
    return kb == 1 ? (raw ? launch_train<4, 1, true>(a, grid, stream)
                          : launch_train<4, 1, false>(a, grid, stream))
                   : (raw ? launch_train<4, 2, true>(a, grid, stream)
                          : launch_train<4, 2, false>(a, grid, stream));
  if (raw)
    return kb == 1   ? launch_train<2, 1, true>(a, grid, stream)
           : kb == 2 ? launch_train<2, 2, true>(a, grid, stream)
                     : launch_train<2, 4, true>(a, grid, stream);
  return kb == 1   ? launch_train<2, 1, false>(a, grid, stream)
         : kb == 2 ? launch_train<2, 2, false>(a, grid, stream)
                   : launch_train<2, 4, false>(a, grid, stream);
}

}  // namespace hd
