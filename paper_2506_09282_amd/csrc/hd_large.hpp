// Shared between the large-batch kernels (hd_large*.hip): element-type
// traits, the tiled model image, Stage II on a finished 32x32 tile and the
// split-D workspace.
#pragma once

#include "hd_common.hpp"
#include "hd_internal.hpp"

namespace hd {
namespace lg {

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kLdsBytes = 160 * 1024 - 256;  // leave room for static LDS

template <typename U, typename V>
__device__ __forceinline__ U bitcast(const V& v) {
  static_assert(sizeof(U) == sizeof(V), "size");
  U u;
  __builtin_memcpy(&u, &v, sizeof(U));
  return u;
}

// ---------------------------------------------------------------------------
// Element-type traits. One "f-step" consumes one 16-byte fragment per lane of
// both operands: 16 features for bf16 (one 32x32x16 MFMA), 8 features for
// fp32 (four 32x32x2 MFMAs).
// ---------------------------------------------------------------------------
struct TrBF16 {
  typedef bf16raw elem;
  static constexpr int kFStep = 16;
  static constexpr int kVec = 8;  // elements per 16-byte group
  static constexpr int kEsz = 2;
  // element e of a 16-byte group held as four dwords: set, read, clear
  __device__ static void put(uint32_t (&t)[4], int e, elem x) {
    t[e >> 1] |= (uint32_t)x << (16 * (e & 1));
  }
  __device__ static elem get(const uint32_t (&t)[4], int e) {
    return (uint16_t)(t[e >> 1] >> (16 * (e & 1)));
  }
  __device__ static void clear(uint32_t (&t)[4], int e) { t[e >> 1] &= ~(0xffffu << (16 * (e & 1))); }
  // Stage I accumulator value v is >= 0 (the HardSign test, Eq. 1)
  __device__ static bool nonneg(float v) { return v >= 0.0f; }
  static constexpr int kStage1Mfma = 1;  // matrix instructions per stage1 call
  static constexpr int kCFrags = 2;  // 1 KiB C fragments per (d-block, class block)
  // LDS position of feature column c inside a sample row.
  __device__ static int lds_pos(int c) { return c; }
  __device__ static void stage1(f32x16& acc, const uint4& a, const uint4& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bitcast<bf16x8>(a), bitcast<bf16x8>(b), acc,
                                                  0, 0, 0);
  }
  // first step of a sum: the instruction's accumulator input is the constant 0
  __device__ static void stage1_init(f32x16& acc, const uint4& a, const uint4& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bitcast<bf16x8>(a), bitcast<bf16x8>(b),
                                                  f32x16{}, 0, 0, 0);
  }
};

struct TrF32 {
  typedef float elem;
  static constexpr int kFStep = 8;
  static constexpr int kVec = 4;
  static constexpr int kEsz = 4;
  __device__ static void put(uint32_t (&t)[4], int e, elem x) { t[e] = __float_as_uint(x); }
  __device__ static elem get(const uint32_t (&t)[4], int e) { return __uint_as_float(t[e]); }
  __device__ static void clear(uint32_t (&t)[4], int e) { t[e] = 0u; }
  __device__ static bool nonneg(float v) { return v >= 0.0f; }
  static constexpr int kStage1Mfma = 4;
  static constexpr int kCFrags = 4;
  // Within each group of 8 features the even ones are stored first, so a
  // lane of MFMA k-half g reads its four features (g, g+2, g+4, g+6) as one
  // 16-byte word.
  __device__ static int lds_pos(int c) {
    const int r = c & 7;
    return (c & ~7) + 4 * (r & 1) + (r >> 1);
  }
  __device__ static void stage1(f32x16& acc, const uint4& a, const uint4& b) {
    const float4 af = bitcast<float4>(a), bf = bitcast<float4>(b);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.x, bf.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.y, bf.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.z, bf.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.w, bf.w, acc, 0, 0, 0);
  }
  __device__ static void stage1_init(f32x16& acc, const uint4& a, const uint4& b) {
    const float4 af = bitcast<float4>(a), bf = bitcast<float4>(b);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.x, bf.x, f32x16{}, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.y, bf.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.z, bf.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af.w, bf.w, acc, 0, 0, 0);
  }
};

// int8 model variant: X and B int8, Stage I on the int8 matrix instruction
// with exact int32 accumulation (the accumulator registers hold the int32
// bits), HardSign on the exact integer; Stage II takes C widened to bf16
// (exact for |c| <= 128) through the bf16 path. One f-step is 32 features.
struct TrI8 {
  typedef int8_t elem;
  static constexpr int kFStep = 32;
  static constexpr int kVec = 16;
  static constexpr int kEsz = 1;
  static constexpr int kStage1Mfma = 1;
  static constexpr int kCFrags = 2;  // C tiles are the bf16 ones
  __device__ static void put(uint32_t (&t)[4], int e, elem x) {
    t[e >> 2] |= (uint32_t)(uint8_t)x << (8 * (e & 3));
  }
  __device__ static elem get(const uint32_t (&t)[4], int e) {
    return (int8_t)(uint8_t)(t[e >> 2] >> (8 * (e & 3)));
  }
  __device__ static void clear(uint32_t (&t)[4], int e) { t[e >> 2] &= ~(0xffu << (8 * (e & 3))); }
  __device__ static bool nonneg(float v) { return __float_as_int(v) >= 0; }
  __device__ static int lds_pos(int c) { return c; }
  __device__ static void stage1(f32x16& acc, const uint4& a, const uint4& b) {
    acc = bitcast<f32x16>(__builtin_amdgcn_mfma_i32_32x32x32_i8(
        bitcast<i32x4>(a), bitcast<i32x4>(b), bitcast<i32x16>(acc), 0, 0, 0));
  }
  __device__ static void stage1_init(f32x16& acc, const uint4& a, const uint4& b) {
    acc = bitcast<f32x16>(
        __builtin_amdgcn_mfma_i32_32x32x32_i8(bitcast<i32x4>(a), bitcast<i32x4>(b), i32x16{}, 0, 0, 0));
  }
};

// Largest sizes of the int8 variant for which every sum is exact: |V| <=
// 128 * 128 * F < 2^31 in int32, and |S| <= 128 * D <= 2^24 in fp32.
constexpr int64_t kI8MaxF = (int64_t(1) << 17) - 1;
constexpr int64_t kI8MaxD = int64_t(1) << 17;

// LDS row padding of an X tile: one 16-byte group (keeps the 32 rows read by
// one fragment load on distinct LDS banks).
template <class Tr>
constexpr int pad_of() {
  return 16 / Tr::kEsz;
}

// Number of f-steps and padded row pitch (elements) of the LDS X tile.
template <class Tr>
__host__ __device__ inline int nfs_of(int F) {
  return (F + Tr::kFStep - 1) / Tr::kFStep;
}
template <class Tr>
__host__ __device__ inline int pitch_of(int F) {
  // Padding by half a 16-byte group (bf16) / one group (fp32) keeps the
  // 32 rows read by one fragment load on distinct LDS banks.
  return nfs_of<Tr>(F) * Tr::kFStep + pad_of<Tr>();
}

// ---------------------------------------------------------------------------
// Tiled model image.
//   B tile (db, fs): 64 lanes x 16 bytes; lane l holds
//     bf16: B[16fs + 8(l/32) + e][32db + l%32], e = 0..7
//     fp32: B[8fs + 2j + l/32][32db + l%32],   j = 0..3
//   C tile, bf16 (db, h, kb): lane l holds C[32kb + l%32][32db + 16h + 4(l/32) + e]
//     for e = 0..3 and C[..][32db + 16h + 8 + 4(l/32) + e - 4] for e = 4..7
//   C tile, fp32 (db, kb, q): lane l holds C[32kb + l%32][32db + 8q + 4(l/32) + j]
// Out-of-range entries are zero. NDB is rounded up to even (64-dim units).
// ---------------------------------------------------------------------------
struct PackGeom {
  int ndb, nfs, kb;
  size_t b_bytes, c_bytes;
};

// Class blocks of 32 handled per launch: 1, 2 or 4.
inline int kb_of(int64_t K) {
  const int kb = (int)cdiv(K, 32);
  return kb == 3 ? 4 : kb;
}

// Sample tiles per workgroup of the F-chunked kernel: 4 when the accumulators
// fit in registers, fewer as class blocks grow.
template <class Tr>
constexpr int chunk_ntiles(int kb) {
  return kb > 2 ? (Tr::kEsz <= 2 ? 2 : 1) : kb == 2 ? 2 : 4;
}

template <class Tr>
PackGeom pack_geom(int64_t F, int64_t D, int64_t K) {
  PackGeom g;
  g.ndb = (int)(cdiv(D, 64) * 2);
  g.nfs = nfs_of<Tr>((int)F);
  g.kb = kb_of(K);
  g.b_bytes = (size_t)g.ndb * g.nfs * 1024;
  g.c_bytes = (size_t)g.ndb * g.kb * Tr::kCFrags * 1024;
  return g;
}

// ---------------------------------------------------------------------------
// Stage II on one finished 32x32 V^T tile (rows d of block db, columns n of
// one sample tile): activation, then accumulate S^T for every class block.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) {
  // round-to-nearest-even fp32 -> bf16 for finite values
  uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  ua = (ua + 0x7fffu + ((ua >> 16) & 1u)) >> 16;
  ub = (ub + 0x7fffu + ((ub >> 16) & 1u)) >> 16;
  return ua | (ub << 16);
}

__device__ __forceinline__ uint32_t sign_pair(float a, float b) {
  const uint32_t lo = a >= 0.0f ? 0x3F80u : 0xBF80u;
  const uint32_t hi = b >= 0.0f ? 0x3F80u : 0xBF80u;
  return lo | (hi << 16);
}

template <int KB, int ACT>
__device__ __forceinline__ void stage2_bf16(const f32x16& v, const uint4 (&cfr)[2][KB],
                                            f32x16 (&s)[KB]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if constexpr (ACT == 0) {
      uint4 hb;
      hb.x = sign_pair(v[8 * h + 0], v[8 * h + 1]);
      hb.y = sign_pair(v[8 * h + 2], v[8 * h + 3]);
      hb.z = sign_pair(v[8 * h + 4], v[8 * h + 5]);
      hb.w = sign_pair(v[8 * h + 6], v[8 * h + 7]);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bitcast<bf16x8>(cfr[h][kb]),
                                                        bitcast<bf16x8>(hb), s[kb], 0, 0, 0);
    } else {
      // Identity test mode: split v into three bf16 terms (about 24 bits).
      float r[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = v[8 * h + e];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        uint4 hb;
        hb.x = pack2_bf16(r[0], r[1]);
        hb.y = pack2_bf16(r[2], r[3]);
        hb.z = pack2_bf16(r[4], r[5]);
        hb.w = pack2_bf16(r[6], r[7]);
        const uint32_t w[4] = {hb.x, hb.y, hb.z, hb.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t bits = (w[e >> 1] >> (16 * (e & 1))) & 0xffffu;
          r[e] -= __uint_as_float(bits << 16);
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bitcast<bf16x8>(cfr[h][kb]),
                                                          bitcast<bf16x8>(hb), s[kb], 0, 0, 0);
      }
    }
  }
}

template <int KB, int ACT>
__device__ __forceinline__ void stage2_f32(const f32x16& v, const uint4 (&cfr)[KB][4],
                                           f32x16 (&s)[KB]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float h = ACT ? v[4 * q + j] : hardsign(v[4 * q + j]);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const float c = __uint_as_float(j == 0 ? cfr[kb][q].x
                                         : j == 1 ? cfr[kb][q].y
                                         : j == 2 ? cfr[kb][q].z
                                                  : cfr[kb][q].w);
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(c, h, s[kb], 0, 0, 0);
      }
    }
  }
}

// C fragments of one 64-dim unit (two d-blocks).
template <class Tr, int KB>
struct CFrags;
template <int KB>
struct CFrags<TrBF16, KB> {
  uint4 f[2][2][KB];  // [db2][h][kb]
  __device__ void load(const uint4* __restrict__ Cp, int db0, int lane) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          f[b][h][kb] = Cp[((int64_t)((db0 + b) * 2 + h) * KB + kb) * 64 + lane];
  }
  template <int ACT>
  __device__ void apply(const f32x16& v, int b, f32x16 (&s)[KB]) const {
    stage2_bf16<KB, ACT>(v, f[b], s);
  }
};
template <int KB>
struct CFrags<TrF32, KB> {
  uint4 f[2][KB][4];  // [db2][kb][q]
  __device__ void load(const uint4* __restrict__ Cp, int db0, int lane) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          f[b][kb][q] = Cp[(((int64_t)(db0 + b) * KB + kb) * 4 + q) * 64 + lane];
  }
  template <int ACT>
  __device__ void apply(const f32x16& v, int b, f32x16 (&s)[KB]) const {
    stage2_f32<KB, ACT>(v, f[b], s);
  }
};

template <int KB>
struct CFrags<TrI8, KB> : CFrags<TrBF16, KB> {
  template <int ACT>
  __device__ void apply(const f32x16& v, int b, f32x16 (&s)[KB]) const {
    f32x16 vf;  // the exact int32 sums as floats (sign and zero preserved)
#pragma unroll
    for (int r = 0; r < 16; ++r) vf[r] = (float)__float_as_int(v[r]);
    stage2_bf16<KB, ACT>(vf, this->f[b], s);
  }
};

// The value of the lane 32 away.
__device__ __forceinline__ uint32_t swap_halves(uint32_t v) {
  return (uint32_t)__shfl_xor((int)v, 32, kWave);
}

// LDS byte address of a pointer into the dynamic LDS array.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

typedef int rsrc_t __attribute__((ext_vector_type(4)));

// What v was read from is done with: the compiler waits for the read here, before
// any later assembly (a barrier after which other waves write there).
__device__ __forceinline__ void have(const uint4& v) {
  asm volatile("" ::"v"(bitcast<i32x4>(v)));
}

// 1 KiB from global memory straight into LDS: lane l's 16 bytes at byte offset
// `off` of the buffer land at lds + 16 l; offsets past the buffer's end
// deliver zeros. Issued as assembly so that the compiler does not take every
// later LDS read for one that may overlap it (it would wait for all loads
// before each read); it writes no register, and the waits are explicit.
__device__ __forceinline__ void dma_1k(rsrc_t rsrc, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds), "v"(off), "s"(rsrc)
               : "memory");
}

// The same with 4 bytes per lane.
__device__ __forceinline__ void dma_256(rsrc_t rsrc, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :
               : "s"(lds), "v"(off), "s"(rsrc)
               : "memory");
}

__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)p;
  rsrc_t r;
  r.x = (int)(uint32_t)a;
  r.y = (int)(uint32_t)(a >> 32);
  r.z = (int)bytes;
  r.w = 0x00020000;
  return r;
}

// Split of D: slice s writes its partial scores to part[s][N][K] at the start
// of the workspace with plain stores; a second launch (hd_large.hip) sums the
// slices in a fixed order, takes the argmax and clears what it read.
__device__ __forceinline__ float* slice_part(void* ws, int slice, int N, int K) {
  return reinterpret_cast<float*>(ws) + (int64_t)slice * N * K;
}
hipError_t launch_reduce_slices(void* ws, int32_t* labels, float* scores, int64_t N, int64_t K,
                                int ds, Clear* clear, hipStream_t stream);

// Combine the waves' partial scores through LDS, then argmax (Eq. 9) and
// write; with a split of D, leave this slice's partial scores for
// reduce_slices_kernel.
template <int NTILES, int KB>
__device__ void finish_tile(f32x16 (&sacc)[NTILES][KB], unsigned char* lds,
                            int32_t* __restrict__ labels, float* __restrict__ scores, int N, int K,
                            int DS, int slice, int n0, void* __restrict__ workspace) {
  constexpr int NT = 32 * NTILES;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __syncthreads();  // X tile no longer needed
  float* sred = reinterpret_cast<float*>(lds);  // [kWaves][NT][32*KB]
  constexpr int KP = 32 * KB;
#pragma unroll
  for (int t = 0; t < NTILES; ++t)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int k = 32 * kb + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int n = 32 * t + (lane & 31);
        sred[((int64_t)wave * NT + n) * KP + k] = sacc[t][kb][r];
      }
  __syncthreads();
  const int rows = min(NT, N - n0);
  if (DS == 1) {
    for (int n = tid; n < rows; n += kThreads) {
      float best = 0.0f;
      int best_k = 0;
      for (int k = 0; k < K; ++k) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += sred[((int64_t)w * NT + n) * KP + k];
        if (scores) scores[(int64_t)(n0 + n) * K + k] = s;
        if (k == 0 || s > best) {
          best = s;
          best_k = k;
        }
      }
      labels[n0 + n] = best_k;
    }
    return;
  }
  float* mypart = slice_part(workspace, slice, N, K) + (int64_t)n0 * K;
  for (int i = tid; i < rows * K; i += kThreads) {
    const int n = i / K, k = i - n * K;
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += sred[((int64_t)w * NT + n) * KP + k];
    mypart[i] = s;
  }
}

// Register budget shared by the kernels that keep one operand in registers
// (8 registers per f-step), two units' sums (64) and 32 result registers per
// class block: depth of the register ring between LDS and the matrix
// instructions (two per fragment, 64 cycles), a divisor of the unit's steps so
// that the ring's position is the same in every unit. Up to eight deep, less
// where the registers are full (a spilled register's reload would wait for
// every buffer-to-LDS load issued before it).
constexpr int ring_depth(int nfs, int kb) {
  if (nfs == 49) return 7;  // (nine steps of which are not in registers)
  const int regs = 8 * nfs + 64 + 32 * kb;
  for (int d : {8, 7, 6, 5, 4})
    if (nfs % d == 0 && (d == 4 || regs + 4 * d < 440)) return d;
  return 4;
}
// Most f-steps for each count of class blocks.
constexpr int max_steps(int kb) { return kb == 1 ? 40 : kb == 2 ? 32 : 20; }

}  // namespace lg

// Kernel with X in registers (hd_large_xreg.hip). head: samples of the first,
// unsplit launch; the others run with D in ds slices on `ws` bytes of
// workspace.
struct XregPlan {
  int kb, ds;
  int64_t head;
  size_t ws;
  bool ok;
};
struct XregArgs {
  const void* X;
  const uint4 *Bp, *Cp;
  int32_t* labels;
  float* scores;
  int F, K, ndb;
  void* workspace;
  Clear* clear;
  hipStream_t stream;
};
// The plan within ws_cap bytes of workspace; x4: X is 4-byte aligned.
XregPlan xreg_plan(int64_t N, int64_t F, int64_t D, int64_t K, int dt, int act, bool x4,
                   size_t ws_cap);
hipError_t launch_xreg(const XregPlan& p, XregArgs a, int64_t N, int dt);

// fp32 Stage I on the bf16 matrix instruction (hd_large_x3.hip); B and C packed
// fragments, or as given (raw). head, ds, ws as above.
struct X3Plan {
  int kb, ds, nt;  // nt: sample tiles per workgroup
  int64_t head;
  size_t ws;
  double us;  // about how long the call takes
  bool ok;
};
X3Plan x3_plan(int64_t N, int64_t F, int64_t D, int64_t K, int act, bool raw, size_t ws_cap);
hipError_t launch_x3(const X3Plan& p, const void* X, const void* B, const void* C, bool raw,
                     int32_t* labels, float* scores, int64_t N, int64_t F, int64_t D, int64_t K,
                     void* ws, Clear* clear, hipStream_t stream);

}  // namespace hd
