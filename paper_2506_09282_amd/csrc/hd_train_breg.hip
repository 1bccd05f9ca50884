// Single-pass training with B held in registers (bf16 and int8 models, rows of
// up to 40 f-steps): class sums of HardSign(X B), Sec. II-C.
//
// A wave keeps the Stage I operands of 64 columns of B in registers while
// units of 32 samples stream through LDS slots, filled by buffer-to-LDS loads
// and read by all four waves (256 columns per workgroup). HardSign turns a
// finished 32x32 tile of V = X B into +-1 bytes, which are an operand of the
// int8 matrix instruction as they lie, with the samples as the summation
// index: one instruction against the one-hot matrix of the unit's labels adds
// the tile to the sums of 32 classes, which stay in int32 accumulators until
// the workgroup's last unit. HardSign and the class sums of a unit run under
// the next unit's matrix instructions.
//
// Rows that are not 4-byte aligned (odd F): rows n with the same n mod Q
// (Q = 2 for bf16, up to 4 for int8) start at the same byte offset from a
// dword, so a unit takes 32 rows of one such class and reads them from the dword
// before. For int8, whose sums are exact in any order, B is loaded shifted by as
// many rows and no element is moved. For bf16 (SHIFT) each fragment is shifted on
// its way from LDS to the matrix instruction, with the word after it, so that a
// sample's sums are rounded alike wherever its row starts: in a chunk of a training
// set its index, and X itself, can be odd (N = 65536, F = 617, K = 26:
// 803 us, 791 with B shifted).
//
// Matrix-core bound, at the clock that dense matrix work leaves (about 1.8 GHz).
// Against X staged through registers between barriers (bundle_mfma_kernel),
// N = 65536, F = 617, D = 10240, K = 26: bf16 3715 -> 800 us (1.04 PFLOP/s),
// int8 3876 -> 444 us; against the double-buffered bundle_dma_kernel,
// N = 16384, F = 616, K = 10: bf16 389 -> 192 us.
#include "hd_large.hpp"

namespace hd {

using namespace lg;

namespace {

constexpr int kCols = 64 * kWaves;  // columns per workgroup
constexpr int kRows = 32;           // samples per unit

// LDS slot: a unit's fragments, then its labels (256 bytes, 32 used).
constexpr int slot_bytes(int nfs) { return nfs * 1024 + 256; }
constexpr int slots(int nfs) {
  const int r = kLdsBytes / slot_bytes(nfs);
  return r > 8 ? 8 : r;
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct BregArgs {
  const void* X;
  const uint4* Bp;
  const int32_t* y;
  int32_t* counts;
  int N, F, D, K, ndb, ngroups;
};

template <class Tr, int NFS, int KB, bool SHIFT>
__device__ __forceinline__ void bundle_breg(const BregArgs& a) {
  constexpr int DP = ring_depth(NFS, KB);
  constexpr int P = NFS / kWaves + 1;  // loads per wave and unit (fragments, labels)
  constexpr int R = slots(NFS);
  constexpr int MID = NFS / 2;
  constexpr int kOut = P * (R - 3);  // see large_fused_kernel_xreg
  constexpr int kSlot = slot_bytes(NFS);
  static_assert(NFS % 2 == 0 && (!SHIFT || Tr::kEsz == 2), "shift");
  static_assert(NFS % DP == 0 && P <= NFS - MID && R >= 3 && kOut <= 63, "schedule");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nfs = nfs_of<Tr>(a.F);
  const int cg = blockIdx.x / a.ngroups, g = blockIdx.x % a.ngroups;
  const uint32_t row_bytes = (uint32_t)a.F * Tr::kEsz;
  const int Q = row_bytes % 4 == 0 ? 1 : row_bytes % 2 == 0 ? 2 : 4;
  // the workgroup's class c of rows n = Q i + c, and its share of their units
  const int c = g % Q, gpc = a.ngroups / Q;
  const int rows_c = (a.N - c + Q - 1) / Q;
  const int units_c = (rows_c + kRows - 1) / kRows;
  const int u0 = (int)((int64_t)units_c * (g / Q) / gpc);
  const int u1 = (int)((int64_t)units_c * (g / Q + 1) / gpc);
  if (u0 >= u1) return;

  // this wave's two blocks of 32 columns (a valid block when it has none:
  // computed and not added)
  const int db0 = cg * (kCols / 32) + 2 * wave;
  const bool valid = db0 < a.ndb;
  const int db = valid ? db0 : cg * (kCols / 32);
  const uint32_t lbase = lds_addr(lds);
  const char* Xb = reinterpret_cast<const char*>(a.X);

  i32x16 cacc[2][KB];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) cacc[b][kb][r] = 0;

  // bytes before the row in its first dword
  const uint32_t sh = ((uint32_t)(uintptr_t)a.X + (uint32_t)c * row_bytes) & 3u;
  const int nfx = (int)((row_bytes + sh + 31u) / 32u);  // f-steps of a shifted row

  // B of this wave's columns as Stage I operands (int8: shifted by sh bytes)
  uint4 bs[NFS][2];
  {
    const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint4*>(a.Bp), 0, a.ndb * nfs * 1024, 0x00020000);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int s = 0; s < NFS; ++s)
        bs[s][b] = s < nfs ? __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                 brs, ((db + b) * nfs + s) * 1024 + lane * 16, 0, 0))
                           : make_uint4(0u, 0u, 0u, 0u);
    if (Tr::kEsz == 1 && sh != 0) {
      // the word before a lane's rows is the last one of the other half of
      // the wave: of this f-step (upper half) or of the one before
      const uint32_t k = 4u - sh;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        uint32_t o = swap_halves(bs[NFS - 1][b].w);
#pragma unroll
        for (int s = NFS - 1; s >= 0; --s) {
          const uint32_t op = s > 0 ? swap_halves(bs[s > 0 ? s - 1 : 0][b].w) : 0u;
          const uint4 v = bs[s][b];
          bs[s][b] = make_uint4(__builtin_amdgcn_alignbyte(v.x, half ? o : op, k),
                                __builtin_amdgcn_alignbyte(v.y, v.x, k),
                                __builtin_amdgcn_alignbyte(v.z, v.y, k),
                                __builtin_amdgcn_alignbyte(v.w, v.z, k));
          o = op;
        }
      }
    }
  }
  // Half of B in accumulation registers, which are matrix operands as they
  // are (left to itself the compiler copies each fragment to a vector register
  // before every use): as many f-steps as the sums leave room for.
  constexpr int kAcc = (256 - 64 - 32 * KB - 8) / 8 < NFS / 2 ? (256 - 64 - 32 * KB - 8) / 8 : NFS / 2;
#pragma unroll
  for (int s = 0; s < kAcc; ++s)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      u32x4 t = __builtin_bit_cast(u32x4, bs[s][b]);
      asm volatile("" : "+a"(t));
      bs[s][b] = __builtin_bit_cast(uint4, t);
    }
  // bf16: what the last f-step holds past the row is cleared (it meets zero rows of
  // B, but may be infinite or NaN)
  uint32_t mlast[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = (int)row_bytes - (nfs - 1) * 32 - half * 16 - 4 * q;
    mlast[q] = k >= 4 ? 0xffffffffu : k <= 0 ? 0u : 0xffffffffu >> (8 * (4 - k));
  }

  // load p of this wave for unit u into slot: fragment 4p + wave, or the labels
  auto issue = [&](int u, int slot, int p) {
    u = min(u, u1 - 1);
    const int64_t row0 = (int64_t)Q * kRows * u + c;
    const uint32_t dst = lbase + (uint32_t)(slot * kSlot);
    if (p < NFS / kWaves) {
      const int j = 4 * p + wave;
      const int64_t b0 = row0 * row_bytes - sh;
      const int64_t left = ((int64_t)a.N * row_bytes - b0 + 3) & ~(int64_t)3;
      const rsrc_t xrs = make_rsrc(Xb + b0, (uint32_t)(left < 0x7fff0000 ? left : 0x7fff0000));
      const uint32_t off = j < nfx ? (uint32_t)(lane & 31) * (uint32_t)Q * row_bytes +
                                         (uint32_t)half * 16u + (uint32_t)j * 32u
                                   : 0x7fff0000u;
      dma_1k(xrs, off, dst + (uint32_t)j * 1024u);
    } else {
      const int64_t left = ((int64_t)a.N - row0) * 4;
      const rsrc_t yrs = make_rsrc(a.y + row0, (uint32_t)(left < 0x7fff0000 ? left : 0x7fff0000));
      dma_256(yrs, lane < 32 ? (uint32_t)(lane * Q) * 4u : 0x7fff0000u, dst + NFS * 1024u);
    }
  };
#pragma unroll
  for (int i = 0; i < R - 1; ++i)
#pragma unroll
    for (int p = 0; p < P; ++p) issue(u0 + i, i, p);

  const unsigned char* frag = lds + lane * 16;
  uint4 ring[DP];
  // SHIFT: the word after a lane's 16 bytes is 512 bytes on in LDS in either half of
  // the wave (the other half's of this f-step, or of the next one), read two steps
  // ahead. Past the last f-step it is not the row's, as are the f-steps past nfs.
  uint32_t after[2];
  auto word_after = [&](const unsigned char* f) {
    return *reinterpret_cast<const uint32_t*>(f + 512);
  };
  auto clean = [&](uint4 v, int s) -> uint4 {
    if constexpr (SHIFT)
      v = make_uint4(__builtin_amdgcn_alignbyte(v.y, v.x, sh),
                     __builtin_amdgcn_alignbyte(v.z, v.y, sh),
                     __builtin_amdgcn_alignbyte(v.w, v.z, sh),
                     __builtin_amdgcn_alignbyte(after[s % 2], v.w, sh));
    if constexpr (Tr::kEsz == 2) {
      if (s >= (NFS > 8 ? NFS - 4 : 0)) {
        if (s == nfs - 1) {
          v.x &= mlast[0];
          v.y &= mlast[1];
          v.z &= mlast[2];
          v.w &= mlast[3];
        } else if (SHIFT && s >= nfs) {
          v.w = 0u;
        }
      }
    }
    return v;
  };
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int i = 0; i < DP; ++i) ring[i] = *reinterpret_cast<const uint4*>(frag + i * 1024);
  if constexpr (SHIFT) {
    after[0] = word_after(frag);
    after[1] = word_after(frag + 1024);
  }

  // HardSign of sums 4 q .. 4 q + 3 of a tile as +-1 bytes, a word of the B
  // operand of the class sums
  auto sign_word = [&](const f32x16& v, int q) -> int {
    const uint32_t b0 = Tr::nonneg(v[4 * q + 0]) ? 0x01u : 0xffu;
    const uint32_t b1 = Tr::nonneg(v[4 * q + 1]) ? 0x0100u : 0xff00u;
    const uint32_t b2 = Tr::nonneg(v[4 * q + 2]) ? 0x010000u : 0xff0000u;
    const uint32_t b3 = Tr::nonneg(v[4 * q + 3]) ? 0x01000000u : 0xff000000u;
    return (int)((b0 | b1) | (b2 | b3));
  };
  // one-hot bytes: class 32 kb + lane % 32 against samples 8 q + 4 half + 0..3
  auto hot_word = [&](const int4& y, int kb) -> int {
    const int k = 32 * kb + (lane & 31);
    return (int)(((y.x == k ? 0x01u : 0u) | (y.y == k ? 0x0100u : 0u)) |
                 ((y.z == k ? 0x010000u : 0u) | (y.w == k ? 0x01000000u : 0u)));
  };
  auto labels_of = [&](int u, int slot, int4 (&yl)[4]) {
    const int4* yp = reinterpret_cast<const int4*>(lds + slot * kSlot + NFS * 1024) + half;
#pragma unroll
    for (int q = 0; q < 4; ++q) yl[q] = yp[2 * q];
    const int left = rows_c - kRows * u;  // rows past the last one have no label
    if (left < kRows) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = 8 * q + 4 * half;
        if (n + 0 >= left) yl[q].x = -1;
        if (n + 1 >= left) yl[q].y = -1;
        if (n + 2 >= left) yl[q].z = -1;
        if (n + 3 >= left) yl[q].w = -1;
      }
    }
  };
  // Unit u from slot sl: Stage I into v, with the class sums of the previous
  // unit (sums pv, slot slp) spread over its first steps; the barrier in
  // the middle as in large_fused_kernel_xreg.
  auto unit = [&](f32x16 (&v)[2], const f32x16 (&pv)[2], int u, int sl, int sln, int slp,
                  auto first_unit) __attribute__((always_inline)) {
    constexpr bool kFirst = decltype(first_unit)::value;
    const unsigned char* fr = frag + sl * kSlot;
    const unsigned char* fn = frag + sln * kSlot;
    // the previous unit's work, a word of four values at a time: the one-hot
    // words, then each tile's sign words and its matrix instructions
    constexpr int kTasks = 4 * KB + 8, kPer = (kTasks + NFS - 3) / (NFS - 2);
    int4 yl[4];
    if constexpr (!kFirst) labels_of(u - 1, slp, yl);
    i32x4 oh[KB], h;
    auto task = [&](int t) __attribute__((always_inline)) {
      if (t < 4 * KB) {
        oh[t / 4][t % 4] = hot_word(yl[t % 4], t / 4);
      } else {
        const int b = (t - 4 * KB) / 4, q = t % 4;
        h[q] = sign_word(pv[b], q);
        if (q == 3) {
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
            cacc[b][kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(oh[kb], h, cacc[b][kb], 0, 0, 0);
        }
      }
    };
#pragma unroll
    for (int s = 0; s < NFS; ++s) {
      if (s == MID)
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kOut) : "memory");
      if (s >= MID && s - MID < P) issue(u + R - 1, slp, s - MID);
      const uint4 x = clean(ring[s % DP], s);
      if constexpr (SHIFT)
        after[s % 2] = word_after(s + 2 < NFS ? fr + (s + 2) * 1024 : fn + (s + 2 - NFS) * 1024);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        if (s == 0)
          Tr::stage1_init(v[b], x, bs[s][b]);
        else
          Tr::stage1(v[b], x, bs[s][b]);
      }
      ring[s % DP] = *reinterpret_cast<const uint4*>(s + DP < NFS ? fr + (s + DP) * 1024
                                                                  : fn + (s + DP - NFS) * 1024);
      if constexpr (!kFirst) {
        static_assert(2 < MID, "slot slp is read before the barrier that frees it");
        if (s == 2) {
#pragma unroll
          for (int q = 0; q < 4; ++q) have(bitcast<uint4>(yl[q]));
        }
#pragma unroll
        for (int t = (s - 1) * kPer; t < s * kPer; ++t)
          if (t >= 0 && t < kTasks) task(t);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, SHIFT ? 2 : 1, 0);
    }
  };
  auto tail = [&](const f32x16 (&pv)[2], int u, int slp) __attribute__((always_inline)) {
    int4 yl[4];
    labels_of(u, slp, yl);
    i32x4 oh[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int q = 0; q < 4; ++q) oh[kb][q] = hot_word(yl[q], kb);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      i32x4 h;
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = sign_word(pv[b], q);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        cacc[b][kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(oh[kb], h, cacc[b][kb], 0, 0, 0);
    }
  };
  f32x16 va[2], vb[2];
  auto nxt = [](int s) { return s == R - 1 ? 0 : s + 1; };
  auto prv = [](int s) { return s == 0 ? R - 1 : s - 1; };
  unit(va, va, u0, 0, 1, R - 1, std::true_type{});
  int u = u0 + 1, sl = 1;
  for (; u + 1 < u1; u += 2) {
    unit(vb, va, u, sl, nxt(sl), prv(sl), std::false_type{});
    sl = nxt(sl);
    unit(va, vb, u + 1, sl, nxt(sl), prv(sl), std::false_type{});
    sl = nxt(sl);
  }
  if (u < u1) {
    unit(vb, va, u, sl, nxt(sl), prv(sl), std::false_type{});
    tail(vb, u, sl);
  } else {
    tail(va, u - 1, prv(sl));
  }
  // no load into LDS is in flight when the workgroup ends
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (!valid) return;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int d = 32 * (db + b) + (lane & 31);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int k = 32 * kb + 8 * (r >> 2) + 4 * half + (r & 3);
        if (k < a.K && d < a.D && cacc[b][kb][r] != 0)
          atomicAdd(&a.counts[(int64_t)k * a.D + d], cacc[b][kb][r]);
      }
  }
}

template <class Tr, int NFS, int KB, bool SHIFT>
__global__ __launch_bounds__(kThreads, 1) void bundle_mfma_kernel_breg(BregArgs a) {
  bundle_breg<Tr, NFS, KB, SHIFT>(a);
}

template <class Tr, int NFS, int KB, bool SHIFT>
hipError_t launch_breg_t(const BregArgs& a, int grid, hipStream_t stream) {
  // (SHIFT reads up to 256 bytes past the last slot's labels)
  constexpr size_t lds = (size_t)slots(NFS) * slot_bytes(NFS) + (SHIFT ? 256 : 0);
  static_assert(lds <= 160 * 1024, "LDS");
  auto* k = &bundle_mfma_kernel_breg<Tr, NFS, KB, SHIFT>;
  static PerDeviceOnce once;
  const hipError_t attr = once_per_device(once, [&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

template <class Tr, int KB, bool SHIFT, int NFS = 8>
hipError_t launch_breg_steps(int steps, const BregArgs& a, int grid, hipStream_t stream) {
  if constexpr (NFS <= max_steps(KB)) {
    if (steps <= NFS) return launch_breg_t<Tr, NFS, KB, SHIFT>(a, grid, stream);
    return launch_breg_steps<Tr, KB, SHIFT, NFS + 4>(steps, a, grid, stream);
  }
  return hipErrorInvalidValue;
}

template <class Tr, bool SHIFT>
hipError_t launch_breg_tr(int steps, int kb, const BregArgs& a, int grid, hipStream_t stream) {
  if (kb == 1) return launch_breg_steps<Tr, 1, SHIFT>(steps, a, grid, stream);
  if (kb == 2) return launch_breg_steps<Tr, 2, SHIFT>(steps, a, grid, stream);
  return launch_breg_steps<Tr, 4, SHIFT>(steps, a, grid, stream);
}

}  // namespace

// X 4-byte aligned, or bf16 rows of odd length: those start at either offset anyway,
// and a chunk from an odd row on must not take another kernel than the whole.
bool bundle_breg_ok(const void* X, int64_t N, int64_t F, int64_t D, int64_t K, int dt) {
  if (dt == 0 || cdiv(K, 32) > 4) return false;
  if ((uintptr_t)X % 4 != 0 && !(dt == 1 && F % 2 != 0)) return false;
  const int64_t esz = dt == 1 ? 2 : 1, rb = F * esz;
  const int64_t maxsh = rb % 4 == 0 ? 0 : rb % 2 == 0 ? 2 : 3;
  return cdiv(rb + maxsh, 32) <= max_steps(kb_of(K)) && N <= (1 << 30) && D <= (1 << 29);
}

hipError_t launch_bundle_breg(const void* X, const void* packed, const int32_t* y,
                              int32_t* counts, int64_t N, int64_t F, int64_t D, int64_t K, int dt,
                              hipStream_t stream) {
  const int64_t esz = dt == 1 ? 2 : 1, rb = F * esz;
  const int64_t maxsh = rb % 4 == 0 ? 0 : rb % 2 == 0 ? 2 : 3;
  const int steps = (int)cdiv(rb + maxsh, 32);
  // Workgroups per class of rows: the fewest rounds over the chip, each round
  // a workgroup's units and about 250 f-steps' time of loading B and adding
  // the sums into counts.
  const int64_t Q = rb % 4 == 0 ? 1 : rb % 2 == 0 ? 2 : 4;
  const int64_t ncg = cdiv(D, kCols), units = cdiv(cdiv(N, Q), kRows), cus = num_cus();
  int64_t gpc = 1, cost = -1;
  for (int64_t n = 1; n <= units && n <= 4 * cus; ++n) {
    const int64_t c = cdiv(ncg * Q * n, cus) * (cdiv(units, n) * (steps + 4) + 250);
    if (cost < 0 || c < cost) {
      cost = c;
      gpc = n;
    }
    if (ncg * Q * n > 8 * cus) break;
  }
  const int64_t ngroups = Q * gpc;
  BregArgs a{X, (const uint4*)packed, y, counts, (int)N, (int)F, (int)D, (int)K,
             (int)(cdiv(D, 64) * 2), (int)ngroups};
  const int grid = (int)(ncg * ngroups);
  if (dt == 2) return launch_breg_tr<TrI8, false>(steps, kb_of(K), a, grid, stream);
  return Q == 1 ? launch_breg_tr<TrBF16, false>(steps, kb_of(K), a, grid, stream)
                : launch_breg_tr<TrBF16, true>(steps, kb_of(K), a, grid, stream);
}

}  // namespace hd
