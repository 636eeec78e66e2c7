// Dense projections of fp32 models: Y[M, N] = X[M, K] · W[N, K]^T on
// v_mfma_f32_16x16x4_f32 with the epilogue of the call fused.
//
// Block tile BM x BN x 32: k-tiles of 128-byte rows arrive by direct
// global->LDS DMA, NS stages in flight (16-byte chunks swizzled as in the bf16
// kernels), and a lane's 16-byte fragment feeds four MFMAs, MFMA e taking
// k = 16 kk + 4 (lane / 16) + e.  Every tile shape adds an element's products in
// that order, so a row's results do not depend on its batch.
//
// Weight rows are placed so that the two columns an epilogue combines sit in one
// lane: a wave's columns come in groups of 32, of which the first 16 hold a
// head's first rotary half (q/k/v) or the gate (gate/up) and the second 16 their
// partners.  The product therefore never goes through memory before its epilogue.
//
// Bound: fp32 MFMA rate (154 TFLOP/s in a large library product on this card) at
// hundreds of rows, the serial chain of k-tiles at a few rows, where a k-tile of a
// 32x64 tile takes 0.36 us (0.52 with its fragments read after the barrier instead
// of a k-tile ahead).  The kernel this one replaced (64x64 tiles of vector FMAs,
// one LDS buffer, the product stored and read back by an elementwise kernel) took,
// 960 rows at d 1024, f 2816: q/k/v 163 us, gate/up 257, down 166 plus 10 per
// epilogue; this one 59, 100 and 57 (110 TFLOP/s, the epilogue included).  At 60
// rows of d 128, f 512 (one user's tree) 10-64 us fell to 4-8.
#include <algorithm>
#include "common.h"
#include "kernels.h"

namespace atspeed {

namespace {

enum { FB_PLAIN = 0, FB_QKV = 1, FB_GU = 2 };

struct F32Args {
  const float* A;
  int lda;
  const int* Mdev;
  int Mt, N, K;
  const float* w0;
  const float* w1;
  const float* w2;
  int split;           // QKV: d_model; GU: d_ffn
  float* out;          // STORE, RESID [M, ldo]; GU [M, d_ffn]
  int ldo;
  int add;             // RESID: add the product to out
  float* q;            // QKV
  float* kdst;
  float* vdst;
  const float* cosT;
  const float* sinT;
  Rows rows;
  int kv_mode, Pmax, d, dh, H;
};

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ int swz32(int r) { return (r >> 1) & 7; }

__device__ __forceinline__ const void* uniform_base(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const void*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// One wave instruction: 8 tile rows of 128 bytes to LDS (lane i lands at byte
// 16 i).  Untracked by the compiler, which would otherwise drain every load at
// each use; the pipeline waits with explicit vmcnt counts.  No compiler code of
// this kernel uses M0.
__device__ __forceinline__ void dma_rows(unsigned char* dst, const void* base, uint32_t off) {
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)dst);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}

// A lane's 16 bytes of such an instruction by an ordinary load, for matrices that start
// at any element: an element's alignment is all it assumes.
typedef float f32x4_any_t __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4_any_t load_any(const void* base, uint32_t off) {
  typedef const __attribute__((address_space(1))) unsigned char global_byte_t;
  typedef const __attribute__((address_space(1))) f32x4_any_t global_f32x4_t;
  return *(global_f32x4_t*)((global_byte_t*)base + off);
}

// At most N vector loads outstanding, and no LDS read or write.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N < 64, "vmcnt holds 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (((N >> 4) & 3) << 14) | (0x7 << 4));
}

template <int WM, int WN, int TM, int TP, int NS, int BMAP, bool DMA>
__global__ void __launch_bounds__(64 * WM * WN) gemm_f32_kernel(F32Args a) {
  constexpr int NW = WM * WN, BM = WM * TM * 16, BN = WN * TP * 32;
  constexpr int NA = BM / (8 * NW), NB = BN / (8 * NW);   // DMA instructions per wave and stage
  static_assert(NA * 8 * NW == BM && NB * 8 * NW == BN, "whole DMA instructions per wave");
  constexpr int STAGE = (BM + BN) * 128;
  __shared__ __align__(1024) unsigned char lds[NS * STAGE];
  const int M = *a.Mdev;
  // Workgroup L runs on XCD L % 8; each XCD takes a contiguous run of tiles, the
  // M-tiles of one N-tile next to each other so that they share its weight rows
  // in that XCD's L2.
  const int Nt = (a.N + BN - 1) / BN, ntiles = a.Mt * Nt, per = (ntiles + 7) >> 3;
  const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (t >= ntiles) return;
  const int tile_n = t / a.Mt, m0 = (t - tile_n * a.Mt) * BM;
  if (m0 >= M) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave / WN, wave_n = wave % WN;
  const int lrow = lane >> 3;

  // DMA instruction j of a wave fills tile rows r0 .. r0+7, all of one matrix: a
  // wave-uniform base and a 32-bit byte offset per lane from it (the matrices
  // themselves may exceed 4 GB)
  const void* abase = uniform_base(a.A + (size_t)m0 * a.lda);
  uint32_t aoff[NA], boff[NB];
  const void* bbase[NB];
  int chi = 0;                          // lanes whose chunk lies in a k-tile's second 16 columns, per instruction
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int r = (wave * NA + j) * 8 + lrow, ch = (lane & 7) ^ swz32(r);
    const int gr = m0 + r < M ? r : M - 1 - m0;
    aoff[j] = (uint32_t)gr * (uint32_t)a.lda * 4u + ch * 16;
    chi |= (ch >> 2) << j;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int r0 = (wave * NB + j) * 8, r = r0 + lrow, ch = (lane & 7) ^ swz32(r);
    const float* w = a.w0;
    int base, row;                      // first row of the instruction's base, and this lane's row
    if (BMAP == FB_GU) {
      const int c0 = tile_n * (BN / 2) + (r0 >> 5) * 16 + (r0 & 15);
      w = (r0 & 16) ? a.w1 : a.w0;
      base = min(c0, a.split - 1);
      row = min(c0 + lrow, a.split - 1);
    } else if (BMAP == FB_QKV) {
      const int p0 = min(tile_n * BN + r0, a.N - 8);   // N = 3 d_model, a multiple of 32
      const int which = p0 / a.split, hc = p0 - which * a.split, pp = hc & (a.dh - 1);
      w = which == 0 ? a.w0 : (which == 1 ? a.w1 : a.w2);
      // within a head, group g of 32 columns holds rotary indices 16 g .. 16 g + 15 of both halves
      base = hc - pp + ((pp >> 5) << 4) + (pp & 15) + ((pp & 16) ? a.dh >> 1 : 0);
      row = base + lrow;
    } else {
      base = min(tile_n * BN + r0, a.N - 1);
      row = min(tile_n * BN + r, a.N - 1);
    }
    bbase[j] = uniform_base(w + (size_t)base * a.K);
    boff[j] = (uint32_t)(row - base) * (uint32_t)a.K * 4u + ch * 16;
    chi |= (ch >> 2) << (NA + j);
  }
  const int nst = (a.K + 31) >> 5;
  const bool half_tail = (a.K & 16) != 0;   // the last k-tile holds 16 columns: its other chunks repeat them, unused
  auto load = [&](int kt) {
    unsigned char* st = lds + (kt % NS) * STAGE;
    const uint32_t kb = (uint32_t)kt * 128u;
    const bool tail = half_tail && kt == nst - 1;
    if constexpr (DMA) {
#pragma unroll
      for (int j = 0; j < NA; ++j)
        dma_rows(st + (wave * NA + j) * 1024, abase, aoff[j] + kb - (tail && ((chi >> j) & 1) ? 64u : 0u));
#pragma unroll
      for (int j = 0; j < NB; ++j)
        dma_rows(st + BM * 128 + (wave * NB + j) * 1024, bbase[j],
                 boff[j] + kb - (tail && ((chi >> (NA + j)) & 1) ? 64u : 0u));
    } else {
      f32x4_any_t va[NA], vb[NB];
#pragma unroll
      for (int j = 0; j < NA; ++j) va[j] = load_any(abase, aoff[j] + kb - (tail && ((chi >> j) & 1) ? 64u : 0u));
#pragma unroll
      for (int j = 0; j < NB; ++j)
        vb[j] = load_any(bbase[j], boff[j] + kb - (tail && ((chi >> (NA + j)) & 1) ? 64u : 0u));
#pragma unroll
      for (int j = 0; j < NA; ++j) *reinterpret_cast<f32x4_any_t*>(st + (wave * NA + j) * 1024 + lane * 16) = va[j];
#pragma unroll
      for (int j = 0; j < NB; ++j)
        *reinterpret_cast<f32x4_any_t*>(st + BM * 128 + (wave * NB + j) * 1024 + lane * 16) = vb[j];
    }
  };

  f32x4_t acc[TM][2 * TP];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < 2 * TP; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, kg = lane >> 4;
  // Fragments of the next k-tile are read while this one's MFMAs issue, so a step
  // costs its MFMA chain and one barrier.  Stage kt % NS is free once every wave
  // holds k-tile kt's fragments, which the barrier of step kt tells.
  const int ra = wave_m * TM * 16 + fr, rb = wave_n * 2 * TP * 16 + fr;   // rows 16 apart share their swizzle
  int ao[2], bo[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    ao[kk] = ra * 128 + (((kk * 4 + kg) ^ swz32(ra)) << 4);
    bo[kk] = BM * 128 + rb * 128 + (((kk * 4 + kg) ^ swz32(rb)) << 4);
  }
  f32x4_t af[2][2][TM], bf[2][2][2 * TP];
  auto read = [&](int kt, auto Set) {
    constexpr int set = decltype(Set)::value;
    const unsigned char* st = lds + (kt % NS) * STAGE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[set][kk][i] = *reinterpret_cast<const f32x4_t*>(st + ao[kk] + i * 2048);
#pragma unroll
      for (int j = 0; j < 2 * TP; ++j) bf[set][kk][j] = *reinterpret_cast<const f32x4_t*>(st + bo[kk] + j * 2048);
    }
  };
  auto mma = [&](int kk, auto Set) {
    constexpr int set = decltype(Set)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 2 * TP; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[set][kk][i][e], bf[set][kk][j][e], acc[i][j], 0, 0, 0);
  };
  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  typedef std::integral_constant<int, 0> I0;
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nst) load(s);
  asm volatile("" ::: "memory");
  if (nst >= NS) wait_vm<(NA + NB) * (NS - 1)>();
  else wait_vm<0>();
  barrier();
  read(0, I0{});
  int kt = 0;
  // steps whose refill lies inside the k range, two at a time (one per register set)
  for (; kt + 1 + NS < nst; kt += 2) {
    static_for<2>([&](auto S) {
      constexpr int cur = decltype(S)::value;
      const int k = kt + cur;
      asm volatile("" ::: "memory");
      wait_vm<(NA + NB) * (NS - 2)>();
      barrier();
      read(k + 1, std::integral_constant<int, cur ^ 1>{});
      __builtin_amdgcn_sched_barrier(0);
      mma(0, S);
      __builtin_amdgcn_sched_barrier(0);
      load(k + NS);
      __builtin_amdgcn_sched_barrier(0);
      mma(1, S);
    });
  }
  for (; kt < nst; kt += 2) {
    static_for<2>([&](auto S) {
      constexpr int cur = decltype(S)::value;
      const int k = kt + cur;
      if (k >= nst) return;
      if (k + 1 < nst) {
        asm volatile("" ::: "memory");
        if (k + NS - 1 < nst) wait_vm<(NA + NB) * (NS - 2)>();
        else wait_vm<0>();
        barrier();
        read(k + 1, std::integral_constant<int, cur ^ 1>{});
        if (k + NS < nst) load(k + NS);
      }
      mma(0, S);
      if (!half_tail || k + 1 < nst) mma(1, S);
    });
  }

  // acc[i][j][r]: row 16 i + 4 kg + r, column 16 j + fr of the wave's tile
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row0 = m0 + (wave_m * TM + i) * 16 + kg * 4;
#pragma unroll
    for (int p = 0; p < TP; ++p) {
      const int group = wave_n * TP + p;              // 32-column group of the tile
      if constexpr (BMAP == FB_PLAIN) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int col = tile_n * BN + group * 32 + h * 16 + fr;
          float old[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            old[r] = a.add && row0 + r < M && col < a.N ? a.out[(size_t)(row0 + r) * a.ldo + col] : 0.f;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (row0 + r < M && col < a.N)
              a.out[(size_t)(row0 + r) * a.ldo + col] = a.add ? old[r] + acc[i][2 * p + h][r] : acc[i][2 * p + h][r];
        }
      } else if constexpr (BMAP == FB_GU) {
        const int col = tile_n * (BN / 2) + group * 16 + fr;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row0 + r < M && col < a.split) {
            const float g = acc[i][2 * p][r];
            a.out[(size_t)(row0 + r) * a.split + col] = g / (1.0f + __expf(-g)) * acc[i][2 * p + 1][r];
          }
      } else {
        const int pc = tile_n * BN + group * 32;
        if (pc >= a.N) continue;
        const int which = pc / a.d, hc = pc - which * a.d, pp = hc & (a.dh - 1), half = a.dh >> 1;
        const int head = hc / a.dh, fi = (pp >> 1) + fr;   // rotary index
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = row0 + r;
          if (row >= M) continue;
          float x1 = acc[i][2 * p][r], x2 = acc[i][2 * p + 1][r];
          const int pos = a.rows.pos[row];
          if (which < 2) {
            const float c = a.cosT[(size_t)pos * half + fi], s = a.sinT[(size_t)pos * half + fi];
            // explicit fma of a rounded product: the same arithmetic in every tile shape
            // (free contraction may differ between instantiations)
            const float p1 = x2 * s, p2 = x1 * s;
            x1 = __builtin_fmaf(x1, c, -p1);
            x2 = __builtin_fmaf(x2, c, p2);
          }
          float* dst;
          if (which == 0) {
            dst = a.q + (size_t)row * a.d + head * a.dh;
          } else {
            dst = which == 1 ? a.kdst : a.vdst;
            dst += a.kv_mode == 0 ? (((size_t)a.rows.user[row] * a.H + head) * a.Pmax + pos) * a.dh
                                  : (size_t)a.rows.slot[row] * a.d + head * a.dh;
          }
          dst[fi] = x1;
          dst[half + fi] = x2;
        }
      }
    }
  }
}

template <int WM, int WN, int TM, int TP, int NS, bool DMA = true>
hipError_t launch_f32(const GemmCall& g, const F32Args& in, hipStream_t st) {
  constexpr int BM = WM * TM * 16, BN = WN * TP * 32;
  F32Args a = in;
  a.Mt = std::max(1, (g.Mmax + BM - 1) / BM);
  const int Nt = (g.N + BN - 1) / BN;
  const dim3 grid(8 * ((a.Mt * Nt + 7) / 8)), block(64 * WM * WN);
  if (g.kind == GEMM_QKV) hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, TM, TP, NS, FB_QKV, DMA>), grid, block, 0, st, a);
  else if (g.kind == GEMM_GU) hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, TM, TP, NS, FB_GU, DMA>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, TM, TP, NS, FB_PLAIN, DMA>), grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace

// d_model and d_ffn are multiples of 16 and d_head is 32, 64 or 128 (checked at
// create), so k-ranges are whole halves of a k-tile and no 32-column group of
// q/k/v straddles two matrices.
hipError_t gemm_f32(const GemmCall& g, hipStream_t st) {
  F32Args a{};
  a.A = (const float*)g.A; a.lda = g.lda; a.Mdev = g.Mdev; a.N = g.N; a.K = g.K;
  a.w0 = (const float*)g.w0; a.w1 = (const float*)g.w1; a.w2 = (const float*)g.w2; a.split = g.split;
  a.out = g.kind == GEMM_GU ? (float*)g.hout : g.out; a.ldo = g.ldo; a.add = g.kind == GEMM_RESID;
  a.q = (float*)g.q; a.kdst = (float*)g.kdst; a.vdst = (float*)g.vdst; a.cosT = g.cosT; a.sinT = g.sinT;
  a.rows = g.rows; a.kv_mode = g.kv_mode; a.Pmax = g.Pmax; a.d = g.d; a.dh = g.dh; a.H = g.H;
  if (g.K % 16 != 0) return hipErrorInvalidValue;
  // The DMA takes 16-byte chunks; matrices that do not start at a multiple of 16 bytes
  // (views into larger buffers) go through registers, which a k-tile's copy waits for:
  // a forward of 930 rows of d 1024 in two layers 756 us instead of 651, 117 rows of d
  // 128 185 instead of 142 (2,425 and 454 with vector FMAs).
  if ((((uintptr_t)g.w0 | (uintptr_t)g.w1 | (uintptr_t)g.w2) & 15) != 0)
    return launch_f32<2, 2, 2, 1, 3, false>(g, a, st);
  // Tile by the time of a k-tile on the fullest CU, us, with n workgroups there:
  // fitted at d 512 and 1,024, f 1,408 and 2,816, 10 to 1,900 rows (within 6% of the
  // measured times).  A tile's own latency rules at few rows, where 32x64 has the
  // shortest chain; with CUs full the fuller last round decides.
  const long M = std::max(1, g.Mmax);
  auto time = [&](int bm, int bn, float t0, float t1) {
    const long n = (((M + bm - 1) / bm) * ((g.N + bn - 1) / bn) + 255) / 256;
    return t0 + t1 * (float)n;
  };
  const float t32 = time(32, 64, 0.07f, 0.29f), t64 = time(64, 64, 0.08f, 0.53f), t128 = time(128, 64, 0.10f, 1.03f);
  if (t32 <= t64 && t32 <= t128) return launch_f32<2, 2, 1, 1, 4>(g, a, st);
  if (t64 <= t128) return launch_f32<2, 2, 2, 1, 3>(g, a, st);
  return launch_f32<4, 2, 2, 1, 3>(g, a, st);
}

}  // namespace atspeed
