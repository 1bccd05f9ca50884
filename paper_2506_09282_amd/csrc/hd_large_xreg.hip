// Large-batch fused inference with X held in registers (bf16 and int8 rows of
// up to 49 f-steps): Alg. 4's split of the batch, Stage I and II fused.
//
// Bound by the matrix cores: dense bf16 work lowers the clock to about
// 1.8 GHz, so what counts is matrix instructions per cycle and little data
// movement. A wave holds the Stage I operands of its 64 samples in registers
// for the whole call; B streams once per workgroup (256 samples) through a
// ring of LDS slots, one slot per 32 dimensions, filled by buffer-to-LDS loads
// and read by all four waves. Each B fragment is read from LDS once per wave
// for two matrix instructions (64 B per cycle and CU, half of what LDS
// delivers). HardSign and Stage II of a unit are spread over the steps of the
// next one, under its matrix instructions. Against the kernels that keep X in
// LDS and load B per wave (hd_large.hip): N = 65536, F = 617, D = 10240,
// K = 26, bf16 762 -> 649 us (1.33 PFLOP/s; the matrix units were waiting on
// the per-wave B ring), int8 440 -> 358 us; N = 4096 89 -> 70 us, 64 -> 44 us.
// Rows of 41 to 49 f-steps, a part of X in LDS: F = 784, K = 10, bf16, N = 300
// 55 -> 29 us, N = 4096 84 -> 74 us, N = 20000 506 -> 298 us.
#include "hd_large.hpp"

namespace hd {

using namespace lg;

static size_t xreg_ws_bytes(int ds, int64_t N, int64_t K);

namespace {

template <class Tr>
__device__ __forceinline__ uint32_t h_pair(float a, float b) {
  return (Tr::nonneg(a) ? 0x3F80u : 0xBF80u) | (Tr::nonneg(b) ? 0x3F800000u : 0xBF800000u);
}

constexpr int kNX = 2;                       // sample tiles of 32 per wave
constexpr int kXTile = 32 * kNX * kWaves;    // samples per workgroup

// Fragments per LDS slot: a unit's B steps, its C, whole loads per wave.
constexpr int unit_frags(int nfs, int kb) { return (nfs + 2 * kb + 3) / 4 * 4; }
// LDS slots: one being read, one complete, the others in flight.
constexpr int ring_slots(int nfs, int kb) {
  const int r = (kLdsBytes >> 10) / unit_frags(nfs, kb);
  return r > 8 ? 8 : r;
}

// Rows of 41 to 49 f-steps leave no registers for every step's X: every fifth
// step's X (nine of them) then lies in LDS, read two steps ahead, and what LDS
// is left holds three slots of half a unit each.
constexpr int kLdsSteps = 9;
constexpr bool x_in_lds(int nfs, int s) { return nfs > 40 && s % 5 == 4 && s / 5 < kLdsSteps; }
constexpr int half_frags(int nfs, int kb) { return ((nfs + 2 * kb + 1) / 2 + 3) / 4 * 4; }
constexpr size_t xreg_lds(int nfs, int kb) {
  return nfs > 40 ? (size_t)(3 * half_frags(nfs, kb) + kLdsSteps * kNX * kWaves) * 1024
                  : (size_t)ring_slots(nfs, kb) * unit_frags(nfs, kb) * 1024;
}

template <class Tr, int NFS, int KB>
__global__ __launch_bounds__(kThreads, 1) void large_fused_kernel_xreg(
    const typename Tr::elem* __restrict__ X, const uint4* __restrict__ Bp,
    const uint4* __restrict__ Cp, int32_t* __restrict__ labels, float* __restrict__ scores, int N,
    int F, int K, int ndb, int DS, void* __restrict__ workspace) {
  constexpr int DP = ring_depth(NFS, KB);
  constexpr bool HALF = NFS > 40;  // slots of half a unit, nine steps' X in LDS
  constexpr int UF = HALF ? half_frags(NFS, KB) : unit_frags(NFS, KB);  // fragments per LDS slot
  constexpr int P = UF / kWaves;  // loads per wave and slot
  constexpr int R = HALF ? 3 : ring_slots(NFS, KB);
  constexpr int MID = HALF ? UF / 2 : NFS / 2;
  constexpr int MID2 = HALF ? UF + (NFS - UF) / 2 : NFS;
  // loads of later units that may be outstanding when the next one must be complete
  constexpr int kOut = P * (R - 3);
  static_assert(NFS % DP == 0 && P <= NFS - MID && R >= 3 && kOut <= 63, "schedule");
  // halves: the second is complete before its first fragment is read, the
  // first is read when the second barrier frees its slot, and the next unit's
  // first is complete before its first fragment is read
  static_assert(!HALF || (MID <= UF - DP && MID2 >= UF && MID2 <= NFS - DP &&
                          MID2 + (P + 1) / 2 <= NFS), "schedule");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nfs = nfs_of<Tr>(F);
  const int slice = blockIdx.x % DS, tile = blockIdx.x / DS;
  const int n0 = tile * kXTile;
  const int rows = min(kXTile, N - n0);
  const int db0 = (int)((int64_t)ndb * slice / DS), db1 = (int)((int64_t)ndb * (slice + 1) / DS);
  const int U = db1 - db0;

  const uint32_t b_bytes = (uint32_t)ndb * nfs * 1024u;
  const rsrc_t brs = make_rsrc(Bp, b_bytes);
  const rsrc_t crs = make_rsrc(Cp, (uint32_t)ndb * 2 * KB * 1024u);
  const uint32_t lbase = lds_addr(lds);
  // load p of this wave for unit u into slot: fragment 4p + wave of the unit (of
  // its half hf)
  auto issue = [&](int u, int slot, int p, int hf) __attribute__((always_inline)) {
    const int i = 4 * p + wave, j = i + hf * UF;
    const int db = min(db0 + u, db1 - 1);
    const uint32_t dst = lbase + (uint32_t)(slot * UF + i) * 1024u;
    if (hf * UF + 4 * p + 3 < NFS || j < NFS) {
      const uint32_t off = j < nfs ? (uint32_t)(db * nfs + j) * 1024u : b_bytes;
      dma_1k(brs, off + (uint32_t)lane * 16u, dst);
    } else {
      const int c = min(j - NFS, 2 * KB - 1);
      dma_1k(crs, (uint32_t)(db * 2 * KB + c) * 1024u + (uint32_t)lane * 16u, dst);
    }
  };
#pragma unroll
  for (int i = 0; i < R - 1; ++i)
#pragma unroll
    for (int p = 0; p < P; ++p) issue(HALF ? 0 : i, i, p, HALF ? i : 0);

  // this wave's rows of X as Stage I operands
  uint4 xf[NFS][kNX];
  {
    // X is 4-byte aligned and read in whole dwords: rows past N are past the
    // resource's end and read as zero, except for what shares X's last dword.
    const char* xb = reinterpret_cast<const char*>(X) + (int64_t)n0 * F * Tr::kEsz;
    const uint32_t row_bytes = (uint32_t)F * Tr::kEsz;
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(xb), 0, (int)(((uint32_t)rows * row_bytes + 3u) & ~3u), 0x00020000);
    uint32_t after[kNX], sh[kNX];  // the first word past a row's f-steps; bytes to shift
#pragma unroll
    for (int t = 0; t < kNX; ++t) {
      const uint32_t b0 = (uint32_t)(32 * (kNX * wave + t) + (lane & 31)) * row_bytes;
      sh[t] = b0 & 3u;
      const uint32_t a0 = (b0 & ~3u) + (uint32_t)(lane >> 5) * 16u;
#pragma unroll
      for (int s = 0; s < NFS; ++s)
        xf[s][t] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(xrs, a0 + 32u * s, 0, 0));
      after[t] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xrs, a0 + 32u * NFS, 0, 0);
    }
    if (row_bytes % 4 != 0) {
      // rows that start inside a dword: the word after a lane's features is
      // the first one of the other half of the wave, of this f-step (lower
      // half) or of the next one
#pragma unroll
      for (int t = 0; t < kNX; ++t) {
        uint32_t o = swap_halves(xf[0][t].x);
#pragma unroll
        for (int s = 0; s < NFS; ++s) {
          const uint32_t on = swap_halves(s + 1 < NFS ? xf[s + 1 < NFS ? s + 1 : s][t].x : after[t]);
          const uint4 v = xf[s][t];
          xf[s][t] = make_uint4(__builtin_amdgcn_alignbyte(v.y, v.x, sh[t]),
                                __builtin_amdgcn_alignbyte(v.z, v.y, sh[t]),
                                __builtin_amdgcn_alignbyte(v.w, v.z, sh[t]),
                                __builtin_amdgcn_alignbyte((lane >> 5) ? on : o, v.w, sh[t]));
          o = on;
        }
      }
    }
    // features past F belong to the next row (or past the end): zero them
    const int rem = F - (nfs - 1) * Tr::kFStep;  // features of the last f-step
#pragma unroll
    for (int s = 0; s < NFS; ++s) {
      if (s >= nfs) {
#pragma unroll
        for (int t = 0; t < kNX; ++t) xf[s][t] = make_uint4(0u, 0u, 0u, 0u);
      } else if (s == nfs - 1) {
        const int keep = (rem - (lane >> 5) * Tr::kVec) * Tr::kEsz;  // bytes to keep
#pragma unroll
        for (int t = 0; t < kNX; ++t) {
          uint32_t w[4] = {xf[s][t].x, xf[s][t].y, xf[s][t].z, xf[s][t].w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int k = keep - 4 * q;
            w[q] = k >= 4 ? w[q] : k <= 0 ? 0u : w[q] & (0xffffffffu >> (8 * (4 - k)));
          }
          xf[s][t] = make_uint4(w[0], w[1], w[2], w[3]);
        }
      }
    }
  }

  f32x16 sacc[kNX][KB];
#pragma unroll
  for (int t = 0; t < kNX; ++t)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[t][kb][r] = 0.0f;

  const uint4* frag = reinterpret_cast<const uint4*>(lds) + lane;
  // X of the steps that lie in LDS (each wave its own)
  uint4* xlds = reinterpret_cast<uint4*>(lds) + (3 * UF + wave * kLdsSteps * kNX) * 64 + lane;
#pragma unroll
  for (int s = 0; s < NFS; ++s)
    if (x_in_lds(NFS, s)) {
#pragma unroll
      for (int t = 0; t < kNX; ++t) xlds[(s / 5 * kNX + t) * 64] = xf[s][t];
    }
  uint4 ring[DP];

  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int i = 0; i < DP; ++i) ring[i] = frag[i * 64];

  // Unit u from slot sl: Stage I into v, with Stage II of the previous unit
  // (sums pv, slot slp) spread over its first steps. In the middle, the wave
  // waits for its own loads of unit u + 1 and for the other waves; then every
  // wave has read what it needs of slot slp, which takes unit u + R - 1, and
  // unit u + 1 is complete before its first fragments are read.
  auto unit = [&](f32x16 (&v)[kNX], const f32x16 (&pv)[kNX], int u, int sl, int sln, int slp,
                  auto first) __attribute__((always_inline)) {
    constexpr bool kFirst = decltype(first)::value;
    // whole units: slots sl, sln (next), slp (previous); halves: sl and sln hold
    // this unit, slp the previous one's second half, then the next one's first
    const uint4* fr = frag + sl * (UF * 64);
    const uint4* fn = frag + sln * (UF * 64);
    const uint4* fp = frag + slp * (UF * 64);
    uint4 cf[2][KB];
    uint4 xl[kNX];
#pragma unroll
    for (int s = 0; s < NFS; ++s) {
      if (s == MID || s == MID2)
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kOut) : "memory");
      if constexpr (HALF) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
          if (s == MID + p / 2) issue(u + 1, slp, p, 0);
          if (s == MID2 + p / 2) issue(u + 1, sl, p, 1);
        }
      } else {
        if (s >= MID && s - MID < P) issue(u + R - 1, slp, s - MID, 0);
      }
      const uint4 a = ring[s % DP];
#pragma unroll
      for (int t = 0; t < kNX; ++t) {
        const uint4 x = x_in_lds(NFS, s) ? xl[t] : xf[s][t];
        if (s == 0)
          Tr::stage1_init(v[t], a, x);
        else
          Tr::stage1(v[t], a, x);
      }
      if (x_in_lds(NFS, s + 2)) {
#pragma unroll
        for (int t = 0; t < kNX; ++t) xl[t] = xlds[((s + 2) / 5 * kNX + t) * 64];
      }
      if constexpr (HALF)
        ring[s % DP] = s + DP < UF    ? fr[(s + DP) * 64]
                       : s + DP < NFS ? fn[(s + DP - UF) * 64]
                                      : fp[(s + DP - NFS) * 64];
      else
        ring[s % DP] = s + DP < NFS ? fr[(s + DP) * 64] : fn[(s + DP - NFS) * 64];
      if constexpr (!kFirst) {
        if (s < 2) {
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) cf[s][kb] = fp[(NFS - (HALF ? UF : 0) + s * KB + kb) * 64];
        }
        constexpr int kStep = NFS >= 20 ? (NFS / 2 - 6) / 4 : 1;  // steps between the four pieces
        constexpr int kS0 = NFS >= 12 ? 4 : 2;
        static_assert(kS0 + kStep < MID, "slot slp is read before the barrier that frees it");
        if (s == kS0 + kStep) {
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            have(cf[0][kb]);
            have(cf[1][kb]);
          }
        }
        if (s >= kS0 && s < kS0 + 4 * kStep && (s - kS0) % kStep == 0) {
          const int p = (s - kS0) / kStep, t = p >> 1, h = p & 1;
          uint4 hb;
          hb.x = h_pair<Tr>(pv[t][8 * h + 0], pv[t][8 * h + 1]);
          hb.y = h_pair<Tr>(pv[t][8 * h + 2], pv[t][8 * h + 3]);
          hb.z = h_pair<Tr>(pv[t][8 * h + 4], pv[t][8 * h + 5]);
          hb.w = h_pair<Tr>(pv[t][8 * h + 6], pv[t][8 * h + 7]);
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
            sacc[t][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                bitcast<bf16x8>(cf[h][kb]), bitcast<bf16x8>(hb), sacc[t][kb], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };
  auto tail = [&](const f32x16 (&pv)[kNX], int slp) __attribute__((always_inline)) {
    const uint4* fp = frag + slp * (UF * 64);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint4 cf[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) cf[kb] = fp[(NFS - (HALF ? UF : 0) + h * KB + kb) * 64];
#pragma unroll
      for (int t = 0; t < kNX; ++t) {
        uint4 hb;
        hb.x = h_pair<Tr>(pv[t][8 * h + 0], pv[t][8 * h + 1]);
        hb.y = h_pair<Tr>(pv[t][8 * h + 2], pv[t][8 * h + 3]);
        hb.z = h_pair<Tr>(pv[t][8 * h + 4], pv[t][8 * h + 5]);
        hb.w = h_pair<Tr>(pv[t][8 * h + 6], pv[t][8 * h + 7]);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          sacc[t][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              bitcast<bf16x8>(cf[kb]), bitcast<bf16x8>(hb), sacc[t][kb], 0, 0, 0);
      }
    }
  };
  f32x16 va[kNX], vb[kNX];
  int sl = 0;
  auto nxt = [](int s) { return s == R - 1 ? 0 : s + 1; };
  auto prv = [](int s) { return s == 0 ? R - 1 : s - 1; };
  // A unit's first slot, from the one before: the next slot, or (halves) the one
  // after its second half's
  auto adv = [&](int s) { return HALF ? prv(s) : nxt(s); };
  unit(va, va, 0, 0, 1, R - 1, std::true_type{});
  int u = 1;
  sl = adv(0);
  for (; u + 1 < U; u += 2) {
    unit(vb, va, u, sl, nxt(sl), prv(sl), std::false_type{});
    sl = adv(sl);
    unit(va, vb, u + 1, sl, nxt(sl), prv(sl), std::false_type{});
    sl = adv(sl);
  }
  if (u < U) {
    unit(vb, va, u, sl, nxt(sl), prv(sl), std::false_type{});
    tail(vb, HALF ? nxt(sl) : sl);
  } else {
    tail(va, prv(sl));
  }

  // ---- scores, argmax (Eq. 9) ------------------------------------------------
  const int half = lane >> 5;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (DS == 1) {
#pragma unroll
    for (int t = 0; t < kNX; ++t) {
      const int n = 32 * (kNX * wave + t) + (lane & 31);
      float best = -__builtin_huge_valf();
      int best_k = 0x7fffffff;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int k = 32 * kb + 8 * (r >> 2) + 4 * half + (r & 3);
          const float s = sacc[t][kb][r];
          if (k < K) {
            if (scores && n < rows) scores[(int64_t)(n0 + n) * K + k] = s;
            if (k == 0 || s > best) {
              best = s;
              best_k = k;
            }
          }
        }
      const float ob = __shfl_xor(best, 32, kWave);
      const int ok = __shfl_xor(best_k, 32, kWave);
      if (ob > best || (ob == best && ok < best_k)) best_k = ok;
      if (half == 0 && n < rows) labels[n0 + n] = best_k;
    }
    return;
  }
  float* mypart = slice_part(workspace, slice, N, K) + (int64_t)n0 * K;
#pragma unroll
  for (int t = 0; t < kNX; ++t) {
    const int n = 32 * (kNX * wave + t) + (lane & 31);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int k = 32 * kb + 8 * (r >> 2) + 4 * half + (r & 3);
        if (k < K && n < rows) mypart[(int64_t)n * K + k] = sacc[t][kb][r];
      }
  }
}

template <class Tr, int NFS, int KB>
hipError_t launch_xreg_t(const XregArgs& a, int64_t N, int ds) {
  constexpr size_t lds = xreg_lds(NFS, KB);
  static_assert(lds <= 160 * 1024, "LDS");
  auto* k = &large_fused_kernel_xreg<Tr, NFS, KB>;
  static PerDeviceOnce once;
  const hipError_t attr = once_per_device(once, [&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(k, dim3((unsigned)(cdiv(N, kXTile) * ds)), dim3(kThreads), lds, a.stream,
                     (const typename Tr::elem*)a.X, a.Bp, a.Cp, a.labels, a.scores, (int)N, a.F,
                     a.K, a.ndb, ds, a.workspace);
  return hipGetLastError();
}

// Instances: unit steps in fours up to max_steps, and 49 for one class block.
constexpr int most_steps(int kb) { return kb == 1 ? 49 : max_steps(kb); }

template <class Tr, int KB, int NFS = 8>
hipError_t launch_xreg_steps(int steps, const XregArgs& a, int64_t N, int ds) {
  if (KB == 1 && steps > 40 && steps <= 49) return launch_xreg_t<Tr, 49, 1>(a, N, ds);
  if constexpr (NFS <= max_steps(KB)) {
    if (steps <= NFS) return launch_xreg_t<Tr, NFS, KB>(a, N, ds);
    return launch_xreg_steps<Tr, KB, NFS + 4>(steps, a, N, ds);
  }
  return hipErrorInvalidValue;
}

template <class Tr>
hipError_t launch_xreg_tr(const XregPlan& p, const XregArgs& a, int64_t N, int ds) {
  const int steps = nfs_of<Tr>(a.F);
  if (p.kb == 1) return launch_xreg_steps<Tr, 1>(steps, a, N, ds);
  if (p.kb == 2) return launch_xreg_steps<Tr, 2>(steps, a, N, ds);
  return launch_xreg_steps<Tr, 4>(steps, a, N, ds);
}

// Split of D for `tiles` sample tiles: the fewest rounds of workgroups over the
// chip, each round a slice's units and about seven units' time of filling the
// registers with X and handing the scores over.
int xreg_slices(int64_t tiles, int ndb, int64_t N, int K, size_t ws_cap) {
  const int64_t cus = num_cus();
  int best = 1;
  int64_t cost = cdiv(tiles, cus) * (ndb + 7);
  for (int ds = 2; ds <= 64 && ds <= ndb; ++ds) {
    if (xreg_ws_bytes(ds, N, K) > ws_cap) break;
    const int64_t c = cdiv(tiles * ds, cus) * (cdiv(ndb, ds) + 9);
    if (c < cost) {
      cost = c;
      best = ds;
    }
  }
  return best;
}

}  // namespace

static size_t xreg_ws_bytes(int ds, int64_t N, int64_t K) {
  if (ds <= 1) return 0;
  return sizeof(float) * (size_t)ds * N * K;
}

XregPlan xreg_plan(int64_t N, int64_t F, int64_t D, int64_t K, int dt, int act, bool x4,
                   size_t ws_cap) {
  XregPlan p{};
  if (dt == 0 || act != 0 || !x4 || cdiv(K, 32) > 4) return p;
  p.kb = kb_of(K);
  // A few samples of one class block: four waves of which one has samples take
  // longer to start than the 32-sample tile in LDS (int8 N = 5, F = 1377 34.8
  // against 31.5 us, bf16 N = 9, F = 690 25.2 against 24.1, as given N = 11,
  // F = 78 26.8 against 24.4); N = 30, F = 1377 33.5 against 41.5.
  if (N <= 16 && p.kb == 1) return p;
  const int64_t steps = dt == 1 ? cdiv(F, TrBF16::kFStep) : cdiv(F, TrI8::kFStep);
  if (steps > most_steps(p.kb)) return p;
  const int64_t ndb = cdiv(D, 64) * 2;
  if (ndb * steps * 1024 >= ((int64_t)1 << 31) || ndb * 2 * p.kb * 1024 >= ((int64_t)1 << 31))
    return p;
  // Whole rounds of one tile per compute unit run unsplit; the tiles left over
  // are split over D in a second launch.
  const int64_t cus = num_cus(), tiles = cdiv(N, kXTile);
  p.head = tiles / cus * cus * kXTile;
  if (p.head > N) p.head = N;
  const int64_t rest = N - p.head;
  p.ds = rest > 0 ? xreg_slices(cdiv(rest, kXTile), (int)ndb, rest, (int)K, ws_cap) : 1;
  p.ws = rest > 0 ? xreg_ws_bytes(p.ds, rest, K) : 0;
  p.ok = true;
  return p;
}

hipError_t launch_xreg(const XregPlan& p, XregArgs a, int64_t N, int dt) {
  auto go = [&](int64_t n, int ds) {
    return dt == 1 ? launch_xreg_tr<TrBF16>(p, a, n, ds) : launch_xreg_tr<TrI8>(p, a, n, ds);
  };
  if (p.head > 0) {
    const hipError_t e = go(p.head, 1);
    if (e != hipSuccess || p.head == N) return e;
  }
  a.X = static_cast<const char*>(a.X) + p.head * a.F * (dt == 1 ? 2 : 1);
  a.labels += p.head;
  if (a.scores) a.scores += p.head * a.K;
  const hipError_t e = go(N - p.head, p.ds);
  if (e != hipSuccess || p.ds == 1) return e;
  return launch_reduce_slices(a.workspace, a.labels, a.scores, N - p.head, a.K, p.ds, a.clear,
                              a.stream);
}

}  // namespace hd
