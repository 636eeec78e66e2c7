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
// hundreds of rows, the serial chain of k-tiles at a few rows.  The kernel this
// one replaced (64x64 tiles of vector FMAs, one LDS buffer, the product stored
// and read back by an elementwise kernel) took, 960 rows at d 1024, f 2816:
// q/k/v 163 us, gate/up 257, down 166 plus 10 per epilogue; this one 66 and
// 120 us (92 TFLOP/s, the epilogue included).  At 60 rows of d 128, f 512 (one
// user's tree) 10-64 us fell to 4.5-5.2.
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

// At most N vector loads outstanding, and no LDS read.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N < 64, "vmcnt holds 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (((N >> 4) & 3) << 14) | (0x7 << 4));
}

template <int WM, int WN, int TM, int TP, int NS, int BMAP>
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
#pragma unroll
    for (int j = 0; j < NA; ++j)
      dma_rows(st + (wave * NA + j) * 1024, abase, aoff[j] + kb - (tail && ((chi >> j) & 1) ? 64u : 0u));
#pragma unroll
    for (int j = 0; j < NB; ++j)
      dma_rows(st + BM * 128 + (wave * NB + j) * 1024, bbase[j],
               boff[j] + kb - (tail && ((chi >> (NA + j)) & 1) ? 64u : 0u));
  };

  f32x4_t acc[TM][2 * TP];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < 2 * TP; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, kg = lane >> 4;

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nst) load(s);
  for (int kt = 0; kt < nst; ++kt) {
    // k-tile kt has landed when at most the loads of the NS - 2 tiles after it
    // are outstanding; the barrier makes every wave's share visible, and tells
    // that all have finished reading the stage that the next load overwrites
    if (kt + NS - 2 < nst) wait_vm<(NA + NB) * (NS - 2)>();
    else wait_vm<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + NS - 1 < nst) load(kt + NS - 1);
    const unsigned char* st = lds + (kt % NS) * STAGE;
    const int nkk = half_tail && kt == nst - 1 ? 1 : 2;
    auto step = [&](int kk) {
      f32x4_t af[TM], bf[2 * TP];
      const int ch = kk * 4 + kg;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = (wave_m * TM + i) * 16 + fr;
        af[i] = *reinterpret_cast<const f32x4_t*>(st + r * 128 + ((ch ^ swz32(r)) << 4));
      }
#pragma unroll
      for (int j = 0; j < 2 * TP; ++j) {
        const int r = (wave_n * 2 * TP + j) * 16 + fr;
        bf[j] = *reinterpret_cast<const f32x4_t*>(st + BM * 128 + r * 128 + ((ch ^ swz32(r)) << 4));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < 2 * TP; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i][e], bf[j][e], acc[i][j], 0, 0, 0);
    };
    step(0);
    if (nkk == 2) step(1);
    asm volatile("" ::: "memory");
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
            const float y1 = x1 * c - x2 * s;
            x2 = x2 * c + x1 * s;
            x1 = y1;
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

template <int WM, int WN, int TM, int TP, int NS>
hipError_t launch_f32(const GemmCall& g, const F32Args& in, hipStream_t st) {
  constexpr int BM = WM * TM * 16, BN = WN * TP * 32;
  F32Args a = in;
  a.Mt = std::max(1, (g.Mmax + BM - 1) / BM);
  const int Nt = (g.N + BN - 1) / BN;
  const dim3 grid(8 * ((a.Mt * Nt + 7) / 8)), block(64 * WM * WN);
  if (g.kind == GEMM_QKV) hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, TM, TP, NS, FB_QKV>), grid, block, 0, st, a);
  else if (g.kind == GEMM_GU) hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, TM, TP, NS, FB_GU>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((gemm_f32_kernel<WM, WN, TM, TP, NS, FB_PLAIN>), grid, block, 0, st, a);
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
  // Large tiles read fewer LDS bytes per MFMA, but only pay once there are enough
  // of them for every CU to hold work; below that 64x64 tiles (three workgroups
  // fit a CU), and at a few rows 32x64 tiles, whose serial chain is the shortest.
  const long M = std::max(1, g.Mmax);
  auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((g.N + bn - 1) / bn); };
  if (tiles(128, 128) >= 384) return launch_f32<2, 2, 4, 2, 3>(g, a, st);
  if (tiles(64, 64) >= 192) return launch_f32<2, 2, 2, 1, 3>(g, a, st);
  return launch_f32<2, 2, 1, 1, 4>(g, a, st);
}

}  // namespace atspeed
