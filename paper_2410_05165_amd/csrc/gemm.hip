// Dense projections of the decoder block: Y[M, N] = X[M, K] · W[N, K]^T.
//
// bf16 path: MFMA v_mfma_f32_32x32x16_bf16 (fp32 accumulate), block tile
// BM x BN x 64, wave tile TM x TN blocks of 32x32, operands through LDS in
// XOR-swizzled 16-byte chunks.  Four pipelines, by the wave tile and the number
// of LDS stages NS: k-tiles staged through registers (four waves, one per SIMD,
// TM + TN >= 6), two stages fed by global->LDS DMA, three or four
// stages fed by it, and three to six with the next k-tile's fragments in
// registers (TM + TN <= 4).  The shape is the one that a fitted
// model of the call's time prefers (gemm() below).  Epilogues are fused:
//   QKV   rotary embedding on q and k, rounding to bf16, q to its row buffer,
//         k/v scattered into the prefix cache or the tree KV buffer.  The tile's
//         weight rows are interleaved (qkv_logical) so that a column's
//         rotate-half partner is in the same MFMA block, and with the operands
//         swapped in the same lane, whatever the tile width;
//   GU    gate and up columns share a tile (first/second half of each wave's
//         blocks), out = bf16(SiLU(gate) * up);
//   RESID residual stream x += acc (fp32); with a partial buffer the k range
//         is split at K/2 into two workgroups per tile, the first adding its
//         product into x and the second storing its own into the buffer (the
//         following RMSNorm adds it), so the o and down projections fill the
//         CUs with 256x256 tiles;
//   STORE fp32 logits.
// M is read from device memory; the grid covers the caller's row count or
// bound (GemmCall::Mmax), and tiles past M exit at once.
// fp32 models take the kernels of gemm_f32.hip.
#include <algorithm>
#include "common.h"
#include "kernels.h"

namespace atspeed {

enum { EPI_STORE = 0, EPI_RESID = 1, EPI_GU = 2, EPI_QKV = 3 };
enum { BMAP_PLAIN = 0, BMAP_QKV = 1, BMAP_GU = 2 };

struct EpiArgs {
  float* out;        // STORE: [M, ldo] fp32; RESID: residual [M, ldo] fp32
  int ldo;
  float* part;       // RESID split in k: the second half's product [M, ldo] fp32 (null: no split)
  bf16_t* hout;      // GU: [M, f] bf16
  // QKV
  bf16_t* q;         // [M, d]
  bf16_t* kdst;      // prefix cache or tree KV base of this layer
  bf16_t* vdst;
  const float* ropeT; // [max_pos][d_head / 2] (cos, sin)
  Rows rows;
  int kv_mode;       // 0 prefix cache [B][H][Pmax][dh], 1 tree [slot][d]
  int Pmax;
  int d, dh;
};

struct BArgs {
  const bf16_t* w0;
  const bf16_t* w1;
  const bf16_t* w2;
  int split;         // QKV: d; GU: f
};

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

template <int WM, int WN, int TM, int TN>
struct Tile {
  static constexpr int NT = 64 * WM * WN;
  static constexpr int BM = WM * TM * 32;
  static constexpr int BN = WN * TN * 32;
  static constexpr int BK = 64;
  static constexpr int A_BYTES = BM * 128;
  static constexpr int B_BYTES = BN * 128;
  static constexpr int STAGE = A_BYTES + B_BYTES;
};

typedef __attribute__((address_space(3))) void lds_void_t;

// LDS swizzle of the 128-byte tile rows: logical 16-byte chunk c of row r sits
// at physical chunk c ^ swz(r).  A fragment read has 16 lanes on 16 consecutive
// rows in one LDS cycle, and a row covers half of the 64 banks, so the 8 even
// rows must use 8 distinct chunks and so must the 8 odd ones: (r >> 1) & 7
// does that (r & 7 would put rows r and r + 8 on the same banks).
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Column order of the q/k/v product (bf16 path).  Within each head, the 32
// columns of MFMA block b hold rotary indices 16b .. 16b+15 of the head's first
// half at 0..15 and the same indices of its second half at 16..31, so every
// column's rotate-half partner is 16 away in the same block.  Maps a
// column's place pp within its head (as the tile holds it) to its column in
// the head (d_head 64 or 128); a bijection on 0 .. d_head-1 that keeps runs of
// 16 columns, and so 16-byte chunks of the bf16 output, contiguous.
__device__ __forceinline__ int qkv_logical(int pp, int halfdh) {
  return ((pp >> 5) << 4) + (pp & 15) + ((pp & 16) ? halfdh : 0);
}

// One k-tile (64 columns of A and W) into an LDS stage with direct global->LDS
// DMA (global_load_lds_dwordx4): each wave instruction fills 1 KB = 8 rows of
// 128 B; lane i lands at byte 16*i, i.e. row i/8, physical chunk i%8, and so
// fetches logical chunk (i%8) ^ swz(row) -- the XOR swizzle the fragment reads
// undo.  No VGPRs hold the tile.  Each address is a wave-uniform base plus an
// unsigned 32-bit byte offset per lane, so the instruction takes its scalar-base
// form (one VGPR per address instead of a 64-bit pair: fewer live registers,
// measured 3-7% faster on the 7B projections); the byte offsets stay below 2^32
// (activation and weight buffers are below 2^31 elements).
template <int NA, int NB>
__device__ __forceinline__ void load_stage(unsigned char* stage, int wave, const bf16_t* A, const int* a_off,
                                           const bf16_t* const* Bp, const int* b_off, int k0, int a_bytes) {
#pragma unroll
  for (int j = 0; j < NA; ++j)
    __builtin_amdgcn_global_load_lds((void*)(reinterpret_cast<const unsigned char*>(A) + (uint32_t)(a_off[j] + k0) * 2u),
                                     (lds_void_t*)(stage + (wave * NA + j) * 1024), 16, 0, 0);
#pragma unroll
  for (int j = 0; j < NB; ++j)
    __builtin_amdgcn_global_load_lds(
        (void*)(reinterpret_cast<const unsigned char*>(Bp[j]) + (uint32_t)(b_off[j] + k0) * 2u),
        (lds_void_t*)(stage + a_bytes + (wave * NB + j) * 1024), 16, 0, 0);
}

// The same stage load as untracked inline-asm DMA, for the pipelines with more
// than two stages: the compiler counts only a few LDS-DMA stores in flight and
// would drain all of them once per round, so these loads are issued where it
// does not see them and the pipeline waits with an explicit vmcnt.  The asm
// writes M0 (the LDS address) itself.  M0 is a reserved register, so the
// compiler ignores its clobber (and warns); that is safe because the kernels
// that use these loads contain no M0 use of the compiler's own (the two-stage
// kernels, whose builtin DMA sets M0, contain no such asm).  Binding the
// address to M0 as an asm operand instead was tried and faulted the GPU.
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const void*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void dma_to_lds(uint32_t lds, uint32_t off, const void* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
               : "memory", "m0");
}
template <int NA, int NB>
__device__ __forceinline__ void load_stage_u(unsigned char* stage, int wave, const bf16_t* A, const int* a_off,
                                             const bf16_t* const* Bp, const int* b_off, int k0, int a_bytes) {
  const void* Au = uniform_ptr(A);
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)(stage + (wave * NA + j) * 1024));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"((uint32_t)(a_off[j] + k0) * 2u),
                 "s"(Au) : "memory", "m0");
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)(stage + a_bytes + (wave * NB + j) * 1024));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"((uint32_t)(b_off[j] + k0) * 2u),
                 "s"(uniform_ptr(Bp[j])) : "memory", "m0");
  }
}

// acc + A W^T of one 32x32 block.  Swapped, the block's transpose: each lane then
// holds four consecutive output columns of a row at a time instead of one column
// of many rows (the same products in the same order, so the same bits).
template <bool SWAP>
__device__ __forceinline__ f32x16_t mfma(bf16x8_t a, bf16x8_t w, f32x16_t acc) {
  return SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a, acc, 0, 0, 0)
              : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w, acc, 0, 0, 0);
}

// One LDS stage (64 columns of k) through the MFMAs.  Fragments of k-step kk+1
// are read into a second register set while the MFMAs of step kk issue, so the
// LDS latency hides behind matrix work instead of stalling every step.
template <int TM, int TN, bool SWAP>
__device__ __forceinline__ void mma_stage(const unsigned char* stage, int wave_m, int wave_n, int fr, int fc,
                                          f32x16_t (&acc)[TM][TN], int a_bytes) {
  bf16x8_t af[2][TM], bfr[2][TN];
  auto read = [&](int kk, bf16x8_t (&a)[TM], bf16x8_t (&b)[TN]) {
    const int ch = kk * 2 + fc;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = wave_m * TM * 32 + i * 32 + fr;
      a[i] = *reinterpret_cast<const bf16x8_t*>(stage + r * 128 + ((ch ^ swz(r)) << 4));
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int r = wave_n * TN * 32 + j * 32 + fr;
      b[j] = *reinterpret_cast<const bf16x8_t*>(stage + a_bytes + r * 128 + ((ch ^ swz(r)) << 4));
    }
  };
  read(0, af[0], bfr[0]);
  // the scheduling groups below describe the whole stage in order: these reads,
  // then per k-step an MFMA / next-step-read alternation (mask 0x008 = MFMA,
  // 0x100 = DS read), then the last step's MFMAs
  __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
  static_for<4>([&](auto KK) {
    constexpr int kk = decltype(KK)::value;
    constexpr int cur = kk & 1, nxt = cur ^ 1;
    if constexpr (kk + 1 < 4) read(kk + 1, af[nxt], bfr[nxt]);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = mfma<SWAP>(af[cur][i], bfr[cur][j], acc[i][j]);
    if constexpr (kk + 1 < 4) {
      static_for<TM + TN>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      });
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - (TM + TN), 0);
    } else {
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
    }
  });
}

template <int WM, int WN, int TM, int TN, int BMAP, int EPI, int NS>
__global__ void __launch_bounds__(64 * WM * WN)
gemm_bf16_kernel(const bf16_t* __restrict__ A, int lda, const int* __restrict__ Mdev, int Mt, int N, int K,
                 BArgs b, EpiArgs e) {
  using T = Tile<WM, WN, TM, TN>;
  constexpr int NW = WM * WN;
  constexpr bool SWAP = EPI == EPI_GU || EPI == EPI_QKV;   // the outputs that are written in bf16
  static_assert(NW == 1 || NW == 2 || NW == 4 || NW == 8, "one, two, four or eight waves");
  static_assert(NS >= 2 && NS <= 8, "two to eight LDS stages");
  constexpr int NA = T::BM / (8 * NW);   // wave instructions per stage for A (8 rows of 128 B each)
  constexpr int NB = T::BN / (8 * NW);
  constexpr bool WIDE = NS == 2 && NW == 4 && TM + TN >= 6;   // one wave per SIMD
  // two stages: two named arrays (see the pipeline below); more: one array of NS
  constexpr bool ONE = NS > 2 || WIDE;
  __shared__ size_t kvrow[EPI == EPI_QKV ? T::BM : 1];   // K/V destination of each tile row (its head 0)
  __shared__ __align__(1024) unsigned char st0[ONE ? 16 : T::STAGE];
  __shared__ __align__(1024) unsigned char st1[ONE ? 16 : T::STAGE];
  __shared__ __align__(1024) unsigned char stn[ONE ? NS : 1][ONE ? T::STAGE : 16];
  const int M = *Mdev;
  // XCD-aware tile order: workgroup L is dispatched to XCD L % 8; XCD x owns the
  // contiguous range x*per .. x*per+per-1 of the tiles.  Tiles are numbered in
  // groups of GM M-tiles, N-major inside a group, so the workgroups that run at
  // once on an XCD cover a few M-tiles times a few N-tiles and share both their
  // activation and their weight slices in its L2 (numbering all M-tiles first
  // gives each running workgroup its own activation slice once M is large: at
  // 38,400 rows that fetched 28 GB per gate/up launch).  GM = 4 measured best
  // over 1,920-38,400 rows: with many rows the activations, not the weights,
  // fall out of the Infinity Cache, so an activation slice should serve more
  // N-tiles than a weight slice serves M-tiles.  The last group takes the
  // remainder (GM to 2 GM - 1 M-tiles): a group of one or two M-tiles would
  // spread over all N-tiles and make its XCDs stream the whole weight matrix
  // for a few rows (with five 64-row tiles that cost the 320-row step 4%).
  // A RESID call with e.part splits k in two halves at K/2 for every row count
  // (so a row's arithmetic never depends on the batch): workgroups of the
  // first half add their product into the residual, those of the second store
  // theirs into e.part, and the next row kernel adds the two.
  const int kparts = (EPI == EPI_RESID && e.part != nullptr) ? 2 : 1;
  const int Nt = (N + T::BN - 1) / T::BN;
  const int tiles1 = Mt * Nt, ntiles = tiles1 * kparts, per = (ntiles + 7) >> 3;
  const int L = blockIdx.x;
  const int tk = (L & 7) * per + (L >> 3);
  if (tk >= ntiles) return;
  const int ks = tk / tiles1, t = tk - ks * tiles1;
  const int kbase = ks * (K / kparts);
  constexpr int GM = 4;
  const int ngrp = Mt / GM > 0 ? Mt / GM : 1;                 // the last group takes the remainder
  const int g0 = t / (GM * Nt), grp = g0 < ngrp - 1 ? g0 : ngrp - 1;
  const int gm0 = grp * GM, gsz = grp == ngrp - 1 ? Mt - gm0 : GM;
  const int tr = t - gm0 * Nt;
  const int tile_n = tr / gsz, tile_m = gm0 + tr - tile_n * gsz;
  const int m0 = tile_m * T::BM;
  if (m0 >= M) return;
  // wave index in a scalar register: the DMA row bases and the weight choice
  // derived from it are then wave-uniform
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave / WN, wave_n = wave % WN;
  const int lrow = lane >> 3;

  // per-lane element offsets of the 16-byte chunks this lane fetches
  int a_off[NA], b_off[NB];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    int r = (wave * NA + j) * 8 + lrow;
    int gr = m0 + r;
    gr = gr < M ? gr : M - 1;
    a_off[j] = gr * lda + kbase + ((lane & 7) ^ swz(r)) * 8;
  }
  // Weight rows of the B tile.  DMA instruction j fills tile rows r0 .. r0+7
  // (r0 = (wave*NB + j)*8), all from one weight matrix Bp[j], chosen from r0
  // alone so that its base stays wave-uniform (d_model and d_ffn are multiples
  // of 8, so no instruction straddles two matrices).
  const bf16_t* Bp[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int r0 = (wave * NB + j) * 8, r = r0 + lrow;
    int row;
    if (BMAP == BMAP_GU) {
      // gate rows in the first half of each wave's blocks, the matching up rows in the second
      constexpr int half = TN / 2;
      const int wn = r / (TN * 32), blk = (r / 32) % TN, cc = r % 32;
      row = tile_n * (T::BN / 2) + wn * (half * 32) + (blk % half) * 32 + cc;
      row = row < b.split ? row : b.split - 1;
      Bp[j] = (r0 / 32) % TN >= half ? b.w1 : b.w0;
    } else if (BMAP == BMAP_QKV) {
      // tile row = column of [q | k | v] (3 d_model), rows past it clamped to the last
      int p = tile_n * T::BN + r;
      p = p < N ? p : N - 1;
      const int p0 = tile_n * T::BN + r0;
      const int which = (p0 < N ? p0 : N - 1) / b.split;
      const int hc = p - which * b.split, pp = hc & (e.dh - 1);
      row = hc - pp + qkv_logical(pp, e.dh >> 1);
      Bp[j] = which == 0 ? b.w0 : (which == 1 ? b.w1 : b.w2);
    } else {
      row = tile_n * T::BN + r;
      row = row < N ? row : N - 1;
      Bp[j] = b.w0;
    }
    b_off[j] = row * K + kbase + ((lane & 7) ^ swz(r)) * 8;
  }

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = K / kparts / T::BK;
  const int fr = lane & 31, fc = lane >> 5;
  // Two-stage pipeline: while the MFMAs consume one LDS stage, the DMA of the
  // next k-tile fills the other.  Each stage is its own LDS array, named at
  // compile time, so the compiler sees that a step's DMA and fragment reads
  // touch different objects and inserts no waits between them.
  // nk is even (each k-range is a multiple of 128, checked on the host)
  if constexpr (WIDE) {
  // The largest tiles: four waves of up to 128x128, one per SIMD with its 512
  // registers, which reads the fewest LDS bytes per MFMA.  Nothing else hides a
  // wave's waits, so every instruction has a place between two MFMAs:
  //  - a k-step's fragments are read during the step before it, also across
  //    k-tiles: the barrier stands before a k-tile's last step, once every wave has
  //    read its fragments and written its share of the next k-tile;
  //  - k-tiles come through registers, a 16-byte chunk at a time, its LDS write
  //    and the load that refills its register spread evenly over the MFMAs, so a
  //    load has a whole k-tile's time to arrive.  Six loads in a row keep the
  //    vector memory path busy longer than the MFMAs between them (2,610 instead
  //    of 2,320 cycles a k-tile at 256x256, 2,048 of them MFMA); direct
  //    global->LDS DMA, which must wait for the stage to be free, took 3,000-4,000
  //    where the lines miss L2.
  constexpr int NLOADS = NA + NB, SLOTS = TM * TN;
  // chunk w goes after MFMA slot_of(w) of the 4 SLOTS from a barrier to the next
  constexpr auto slot_of = [](int w) constexpr { return w * 4 * SLOTS / NLOADS + 2; };
  static_assert(slot_of(NLOADS - 1) < 4 * SLOTS, "every chunk of a k-tile has an MFMA to follow");
  static_assert(TM + TN <= SLOTS, "every fragment of a k-step has an MFMA to follow");
  constexpr int EARLY = [=]() constexpr { int n = 0; while (n < NLOADS && slot_of(n) < SLOTS) ++n; return n; }();
  uint32_t off[NLOADS];
#pragma unroll
  for (int j = 0; j < NLOADS; ++j)
    off[j] = (uint32_t)(j < NA ? a_off[j < NA ? j : 0] : b_off[j < NA ? 0 : j - NA]) * 2u;
  u32x4_t stg[NLOADS];
  const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, -1, 0x00020000);
  __amdgpu_buffer_rsrc_t brs[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
    brs[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(uniform_ptr(Bp[j])), 0, -1, 0x00020000);
  auto gload = [&](int j, int kt) {
    stg[j] = __builtin_amdgcn_raw_buffer_load_b128(j < NA ? ars : brs[j < NA ? 0 : j - NA], (int)off[j], kt * 128, 0);
  };
  auto swrite = [&](int j, int buf) {
    unsigned char* const d = j < NA ? stn[buf] + wave * NA * 1024 + lane * 16 + j * 1024
                                    : stn[buf] + T::A_BYTES + wave * NB * 1024 + lane * 16 + (j - NA) * 1024;
    *reinterpret_cast<u32x4_t*>(d) = stg[j];
  };
  const int ra = wave_m * TM * 32 + fr, rb = wave_n * TN * 32 + fr;
  const unsigned char* ap[2][4];
  const unsigned char* bp[2][4];
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      ap[b2][kk] = stn[b2] + ra * 128 + (((kk * 2 + fc) ^ swz(ra)) << 4);
      bp[b2][kk] = stn[b2] + T::A_BYTES + rb * 128 + (((kk * 2 + fc) ^ swz(rb)) << 4);
    }
  bf16x8_t fa[2][TM], fb[2][TN];
  // fragment q of a k-step, in the order its MFMAs need them
  auto read1 = [&](int q, int buf, int kk, int set) {
    if (q == 0) fa[set][0] = *reinterpret_cast<const bf16x8_t*>(ap[buf][kk]);
    else if (q <= TN) fb[set][q - 1] = *reinterpret_cast<const bf16x8_t*>(bp[buf][kk] + (q - 1) * 4096);
    else fa[set][q - TN] = *reinterpret_cast<const bf16x8_t*>(ap[buf][kk] + (q - TN) * 4096);
  };
  auto barrier = [] {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
#pragma unroll
  for (int j = 0; j < NLOADS; ++j) gload(j, 0);
#pragma unroll
  for (int j = 0; j < NLOADS; ++j) {
    swrite(j, 0);
    gload(j, 1);
  }
#pragma unroll
  for (int j = 0; j < EARLY; ++j) {
    swrite(j, 1);
    if (nk > 2) gload(j, 2);
  }
  barrier();
  static_for<TM + TN>([&](auto Q) { read1(decltype(Q)::value, 0, 0, 0); });
  // k-tile kt; Left: k-tiles after it, at most 3 (more make no difference)
  auto ktile = [&](auto Buf, auto Left, int kt) {
    constexpr int buf = decltype(Buf)::value, left = decltype(Left)::value;
    static_for<4>([&](auto KK) {
      constexpr int kk = decltype(KK)::value, cur = kk & 1, nxt = cur ^ 1;
      if constexpr (kk == 3 && left > 0) barrier();
      static_for<SLOTS>([&](auto Q) {
        constexpr int q = decltype(Q)::value, i = q / TN, j = q % TN;
        acc[i][j] = mfma<SWAP>(fa[cur][i], fb[cur][j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (q < TM + TN) {
          if constexpr (kk < 3) read1(q, buf, kk + 1, nxt);
          else if constexpr (left > 0) read1(q, buf ^ 1, 0, nxt);
        }
        // after the barrier k-tile kt + 2's first chunks go to the stage this
        // k-tile has left, before it k-tile kt + 1's others to the other one
        constexpr int slot = ((kk + 1) & 3) * SLOTS + q;
        static_for<NLOADS>([&](auto W) {
          constexpr int w = decltype(W)::value;
          if constexpr (slot_of(w) == slot) {
            if constexpr (left > (kk < 3 ? 0 : 1)) {
              swrite(w, kk < 3 ? buf ^ 1 : buf);
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (left > (kk < 3 ? 1 : 2)) gload(w, kt + (kk < 3 ? 2 : 3));
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
  int kt = 0;
  for (; kt + 4 < nk; kt += 2) {
    ktile(I0{}, I3{}, kt);
    ktile(I1{}, I3{}, kt + 1);
  }
  if (kt + 4 == nk) {
    ktile(I0{}, I3{}, kt);
    ktile(I1{}, I2{}, kt + 1);
  }
  ktile(I0{}, I1{}, nk - 2);
  ktile(I1{}, I0{}, nk - 1);
  __syncthreads();
  } else if constexpr (NS > 2 && TM + TN <= 4) {
  // Register-ahead pipeline (wave tiles small enough to hold two k-tiles of
  // fragments): while a k-tile's MFMAs issue from registers, the next one's
  // fragments are on their way from LDS and the NS - 1 after it from memory, so
  // a step costs its MFMA chain and one barrier instead of the sum of the
  // barrier, the LDS latency and the chain.  Stage kt % NS is free once every
  // wave holds k-tile kt's fragments, which the barrier of step kt tells; the
  // DMA that refills it issues between the MFMAs.
  constexpr int NLOADS = NA + NB;                 // DMA instructions per stage per lane
  static_assert(NLOADS * (NS - 1) < 64, "vmcnt holds 6 bits");
  constexpr auto vm_lgkm0 = [](int n) constexpr { return (n & 0xF) | (((n >> 4) & 3) << 14) | (0x7 << 4); };
  const void* base[NLOADS];
  uint32_t off[NLOADS];                           // byte offset of this lane's next chunk
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)stn[0]);
#pragma unroll
  for (int j = 0; j < NLOADS; ++j) {
    base[j] = uniform_ptr(j < NA ? A : Bp[j < NA ? 0 : j - NA]);
    off[j] = (uint32_t)(j < NA ? a_off[j < NA ? j : 0] : b_off[j < NA ? 0 : j - NA]) * 2u;
  }
  auto load1 = [&](int j, uint32_t stage) {       // DMA instruction j of the next k-tile
    dma_to_lds(lds0 + stage + (j < NA ? (wave * NA + j) * 1024 : T::A_BYTES + (wave * NB + j - NA) * 1024), off[j],
               base[j]);
    off[j] += 128u;
  };
  // fragment address: rows 32 apart share their swizzle, so one offset per
  // k-step serves every block of the wave
  const int ra = wave_m * TM * 32 + fr, rb = wave_n * TN * 32 + fr;
  int ao[4], bo[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    ao[kk] = ra * 128 + (((kk * 2 + fc) ^ swz(ra)) << 4);
    bo[kk] = T::A_BYTES + rb * 128 + (((kk * 2 + fc) ^ swz(rb)) << 4);
  }
  bf16x8_t fa[2][4][TM], fb[2][4][TN];
  auto read = [&](uint32_t stage, auto Set) {
    constexpr int set = decltype(Set)::value;
    const unsigned char* st = stn[0] + stage;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[set][kk][i] = *reinterpret_cast<const bf16x8_t*>(st + ao[kk] + i * 4096);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[set][kk][j] = *reinterpret_cast<const bf16x8_t*>(st + bo[kk] + j * 4096);
    }
  };
  auto mma = [&](int kk, auto Set) {
    constexpr int set = decltype(Set)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = mfma<SWAP>(fa[set][kk][i], fb[set][kk][j], acc[i][j]);
  };
  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nk)
#pragma unroll
      for (int j = 0; j < NLOADS; ++j) load1(j, s * T::STAGE);
  asm volatile("" ::: "memory");
  if (nk >= NS) __builtin_amdgcn_s_waitcnt(vm_lgkm0(NLOADS * (NS - 1)));
  else __builtin_amdgcn_s_waitcnt(vm_lgkm0(0));
  barrier();
  read(0, std::integral_constant<int, 0>{});
  uint32_t st_cur = 0, st_next = T::STAGE;        // stages of k-tiles kt and kt + 1
  auto advance = [&]() {
    st_cur = st_next;
    st_next = st_next + T::STAGE == (uint32_t)NS * T::STAGE ? 0u : st_next + T::STAGE;
  };
  int kt = 0;
  // steps whose refill lies inside the k range, two at a time (one per register set)
  for (; kt + 1 + NS < nk; kt += 2) {
    static_for<2>([&](auto S) {
      constexpr int cur = decltype(S)::value;
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(vm_lgkm0(NLOADS * (NS - 2)));
      barrier();
      read(st_next, std::integral_constant<int, cur ^ 1>{});
      __builtin_amdgcn_sched_barrier(0);
      static_for<4>([&](auto KK) {
        constexpr int kk = decltype(KK)::value;
        mma(kk, S);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = kk * NLOADS / 4; j < (kk + 1) * NLOADS / 4; ++j) load1(j, st_cur);
        __builtin_amdgcn_sched_barrier(0);
      });
      advance();
    });
  }
  for (; kt < nk; kt += 2) {
    static_for<2>([&](auto S) {
      constexpr int cur = decltype(S)::value;
      const int k = kt + cur;
      if (k + 1 < nk) {
        asm volatile("" ::: "memory");
        if (k + NS - 1 < nk) __builtin_amdgcn_s_waitcnt(vm_lgkm0(NLOADS * (NS - 2)));
        else __builtin_amdgcn_s_waitcnt(vm_lgkm0(0));
        barrier();
        read(st_next, std::integral_constant<int, cur ^ 1>{});
        if (k + NS < nk)
#pragma unroll
          for (int j = 0; j < NLOADS; ++j) load1(j, st_cur);
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) mma(kk, S);
      advance();
    });
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  } else if constexpr (NS > 2) {
  // NS-stage pipeline (small row counts, where each k-tile's weights arrive
  // cold from HBM): stage s of round kt0 computes k-tile kt0+s while the DMA of
  // k-tiles up to kt0+s+NS-1 is in flight; at each stage end the wave waits
  // until only the newest NS-2 stages' loads are outstanding, then a bare
  // barrier makes every wave's share of the next stage visible.  Empty asm with
  // a memory clobber on both sides keeps fragment reads and DMA issue from
  // moving across the barrier (the barrier intrinsic does not order memory).
  auto stage = [&](auto S) -> unsigned char* { return stn[decltype(S)::value % NS]; };
  constexpr int NLOADS = NA + NB;                 // DMA instructions per stage per lane
  constexpr int ALLOW = NLOADS * (NS - 2);        // loads that may stay in flight at a stage boundary
  constexpr int WAITCNT = (ALLOW & 0xF) | (((ALLOW >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8);
  constexpr int WAITALL = (0x7 << 4) | (0xF << 8);  // vmcnt(0)
  static_assert(ALLOW < 64, "vmcnt holds 6 bits");
  static_for<NS - 1>([&](auto S) {
    constexpr int s_ = decltype(S)::value;
    if (s_ < nk) load_stage_u<NA, NB>(stage(S), wave, A, a_off, Bp, b_off, s_ * 64, T::A_BYTES);
  });
  asm volatile("" ::: "memory");
  if (NS - 2 < nk) __builtin_amdgcn_s_waitcnt(WAITCNT);
  else __builtin_amdgcn_s_waitcnt(WAITALL);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  for (int kt0 = 0; kt0 < nk; kt0 += NS) {
    static_for<NS>([&](auto S) {
      constexpr int s_ = decltype(S)::value;
      const int kt = kt0 + s_;
      if (kt < nk) {
        if (kt + NS - 1 < nk)
          load_stage_u<NA, NB>(stage(std::integral_constant<int, s_ + NS - 1>{}), wave, A, a_off, Bp, b_off,
                               (kt + NS - 1) * 64, T::A_BYTES);
        __builtin_amdgcn_sched_barrier(0);
        mma_stage<TM, TN, SWAP>(stage(S), wave_m, wave_n, fr, fc, acc, T::A_BYTES);
        asm volatile("" ::: "memory");
        if (kt + NS - 1 < nk) __builtin_amdgcn_s_waitcnt(WAITCNT);
        else __builtin_amdgcn_s_waitcnt(WAITALL);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
    });
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  } else {
  load_stage<NA, NB>(st0, wave, A, a_off, Bp, b_off, 0, T::A_BYTES);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // sched_barrier(0) after each DMA issue: left free, the scheduler sinks the
  // DMA below the stage's MFMAs, right before the wait that ends the stage,
  // and the load latency is exposed instead of hidden
  for (int kt = 0; kt < nk; kt += 2) {
    load_stage<NA, NB>(st1, wave, A, a_off, Bp, b_off, (kt + 1) * 64, T::A_BYTES);
    __builtin_amdgcn_sched_barrier(0);
    mma_stage<TM, TN, SWAP>(st0, wave_m, wave_n, fr, fc, acc, T::A_BYTES);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (kt + 2 < nk) load_stage<NA, NB>(st0, wave, A, a_off, Bp, b_off, (kt + 2) * 64, T::A_BYTES);
    __builtin_amdgcn_sched_barrier(0);
    mma_stage<TM, TN, SWAP>(st1, wave_m, wave_n, fr, fc, acc, T::A_BYTES);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
  }

  // ---- epilogue.  acc[i][j][r] is row (r/4)*8 + (lane/32)*4 + r%4, column lane%32 of block (i, j).
  const int row0 = m0 + wave_m * TM * 32;
  const int col0 = tile_n * T::BN + wave_n * TN * 32;
  if constexpr (EPI == EPI_STORE || EPI == EPI_RESID) {
    // Branch-free: the accesses go through a buffer resource spanning this
    // tile's valid rows, so the hardware drops stores past it (rows >= M, and
    // columns >= N, which get an out-of-range offset) and returns 0 for such
    // loads.  Guarding each access with a branch instead makes the compiler
    // wait for every store before the next one.  RESID loads all TN x 16
    // residual values of a 32-row block before it adds and stores them.
    const int mrows = M - m0 < T::BM ? M - m0 : T::BM;
    const bool add_old = EPI == EPI_RESID && ks == 0;   // the k-split's second half stores its product alone
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (ks == 0 ? e.out : e.part) + (size_t)m0 * e.ldo, 0, mrows * e.ldo * (int)sizeof(float), 0x00020000);
    const int lrow0 = wave_m * TM * 32;
    // byte offset = row part + column part; a column >= N gets a 1 GiB column
    // part, past the range of any tile's rows
    int coff[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = col0 + j * 32 + fr;
      coff[j] = col < N ? col * (int)sizeof(float) : (1 << 30);
    }
    static_for<TM>([&](auto I) {
      constexpr int i = decltype(I)::value;
      int roff[16];
      static_for<16>([&](auto R) {
        constexpr int r = decltype(R)::value;
        roff[r] = (lrow0 + i * 32 + (r >> 2) * 8 + fc * 4 + (r & 3)) * e.ldo * (int)sizeof(float);
      });
      // residual values loaded for half a 32-row block at a time, all issued
      // before any is used
      static_for<2>([&](auto Hh) {
        constexpr int h0 = decltype(Hh)::value * 8;
        float old[TN][8];
        if (add_old) {
          static_for<8>([&](auto R) {
            constexpr int r = decltype(R)::value;
#pragma unroll
            for (int j = 0; j < TN; ++j)
              old[j][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, roff[h0 + r] + coff[j], 0, 0));
          });
        }
        static_for<8>([&](auto R) {
          constexpr int r = decltype(R)::value;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float v = add_old ? old[j][r] + acc[i][j][h0 + r] : acc[i][j][h0 + r];
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, roff[h0 + r] + coff[j], 0, 0);
          }
        });
      });
    });
  } else {
    // Results are rounded to bf16 into an LDS copy of the output tile (the stage
    // buffers are free now), then written out in 16-byte chunks along rows.  With
    // swapped operands acc[i][j][4 g + r] is row lane % 32, column 8 g + 4 (lane /
    // 32) + r of block (i, j), so four values make one 8-byte LDS write.  Chunk c of
    // row r sits at c ^ osw(r), which spreads the 32 rows of a write over the banks.
    constexpr int OUTC = EPI == EPI_GU ? T::BN / 2 : T::BN;  // output columns of the tile
    constexpr int OROW = OUTC * 2;                            // bytes per LDS row
    constexpr int CPRW = OUTC / 8;                            // 16-byte chunks per output row
    constexpr int RSH = OROW >= 256 ? 0 : (OROW == 128 ? 1 : 2);   // rows per 256 bytes, log2
    constexpr int CMASK = (CPRW % 16 == 0 ? 16 : CPRW % 8 == 0 ? 8 : 4) - 1;
    static_assert(CPRW % 4 == 0, "whole groups of swizzled chunks");
    auto osw = [](int r) { return (r >> RSH) & CMASK; };
    // The whole output tile in the first stage buffer (one array, in the multi-stage
    // kernels) when it fits; otherwise its first half of rows there and the second
    // in the next one.
    constexpr bool ONEBUF = T::BM * OROW <= (ONE ? NS : 1) * T::STAGE;
    constexpr int HROWS = ONEBUF ? T::BM : T::BM / 2;
    constexpr int WMH = ONEBUF ? WM : WM / 2;       // wave rows per buffer
    static_assert(ONEBUF || (HROWS * OROW <= T::STAGE && WM % 2 == 0), "each half of the output tile fits a stage");
    unsigned char* const ob0 = ONE ? stn[0] : st0;
    unsigned char* const ob1 = ONE ? stn[0] : st1;
    unsigned char* const ob = wave_m < WMH ? ob0 : ob1;
    auto put = [&](int lr, int col, float v0, float v1, float v2, float v3) {   // 4 values at (row of this buffer, column)
      uint2 w;
      w.x = (uint32_t)f2bf(v0) | ((uint32_t)f2bf(v1) << 16);
      w.y = (uint32_t)f2bf(v2) | ((uint32_t)f2bf(v3) << 16);
      *reinterpret_cast<uint2*>(ob + lr * OROW + (((col >> 3) ^ osw(lr)) << 4) + (col & 4) * 2) = w;
    };
    const int hrow0 = (wave_m % WMH) * TM * 32 + fr;          // this lane's row of block 0 in its buffer
    if constexpr (EPI == EPI_GU) {
      constexpr int half = TN / 2;
      static_for<TM>([&](auto I) {
        constexpr int i = decltype(I)::value;
        static_for<half * 4>([&](auto G) {
          constexpr int j = decltype(G)::value / 4, g = decltype(G)::value % 4;
          float v[4];
          static_for<4>([&](auto R) {
            constexpr int r = decltype(R)::value;
            v[r] = silu(acc[i][j][4 * g + r]) * acc[i][j + half][4 * g + r];
          });
          put(hrow0 + i * 32, wave_n * (half * 32) + j * 32 + 8 * g + 4 * fc, v[0], v[1], v[2], v[3]);
        });
      });
    } else {  // EPI_QKV: rotary embedding on q and k (column order of qkv_logical)
      // per block (wave-uniform; d_model and d_head are multiples of 32): which of
      // q, k, v it lies in, and its first rotary index; columns 0..15 of a block
      // and their partners 16..31 are groups g and g + 2 of the same lane
      for (int r = tid; r < T::BM; r += T::NT) {
        const int row = m0 + r < M ? m0 + r : M - 1;
        kvrow[r] = e.kv_mode == 0 ? (size_t)e.rows.user[row] * e.d * e.Pmax + (size_t)e.rows.pos[row] * e.dh
                                  : (size_t)e.rows.slot[row] * e.d;
      }
      int pos[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m0 + (wave_m * TM + i) * 32 + fr;
        pos[i] = e.rows.pos[row < M ? row : M - 1];
      }
      const int halfdh = e.dh >> 1;
      static_for<TN>([&](auto J) {
        constexpr int j = decltype(J)::value;
        int pc = col0 + j * 32;
        pc = pc < N ? pc : N - 32;
        const bool rot = pc < 2 * e.d;
        const int idx0 = ((pc & (e.dh - 1)) >> 1) + 4 * fc;      // d_model is a multiple of d_head
        static_for<TM>([&](auto I) {
          constexpr int i = decltype(I)::value;
          const int lr = hrow0 + i * 32, lc = wave_n * TN * 32 + j * 32 + 4 * fc;
          if (rot) {
            // (cos, sin) of the lane's 2 x 4 consecutive rotary indices
            const float* t = e.ropeT + ((size_t)pos[i] * halfdh + idx0) * 2;
            f32x4_t cs[4];
#pragma unroll
            for (int h = 0; h < 4; ++h)
              cs[h] = *reinterpret_cast<const f32x4_t*>(t + (h >> 1) * 16 + (h & 1) * 4);
            static_for<2>([&](auto G) {
              constexpr int g = decltype(G)::value;
              float y1[4], y2[4];
              static_for<4>([&](auto R) {
                constexpr int r = decltype(R)::value;
                const float x1 = acc[i][j][4 * g + r], x2 = acc[i][j][4 * (g + 2) + r];
                const float c = cs[2 * g + r / 2][(r & 1) * 2], sn = cs[2 * g + r / 2][(r & 1) * 2 + 1];
                // explicit fma of a rounded product: the same arithmetic in every
                // tile shape (free contraction may differ between instantiations,
                // and rows must not depend on the shape their batch got)
                const float p1 = x2 * sn, p2 = x1 * sn;
                y1[r] = __builtin_fmaf(x1, c, -p1);
                y2[r] = __builtin_fmaf(x2, c, p2);
              });
              put(lr, lc + 8 * g, y1[0], y1[1], y1[2], y1[3]);
              put(lr, lc + 8 * (g + 2), y2[0], y2[1], y2[2], y2[3]);
            });
          } else {
            static_for<4>([&](auto G) {
              constexpr int g = decltype(G)::value;
              put(lr, lc + 8 * g, acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
            });
          }
        });
      });
    }
    __syncthreads();
#pragma unroll 2
    for (int c = tid; c < T::BM * CPRW; c += T::NT) {
      const int lr = c / CPRW, cc = c % CPRW;
      const int row = m0 + lr;
      if (row >= M) continue;
      const int br = lr < HROWS ? lr : lr - HROWS;    // row in its buffer
      const unsigned char* src = (lr < HROWS ? ob0 : ob1) + br * OROW + ((cc ^ osw(br)) << 4);
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(src);
      if constexpr (EPI == EPI_GU) {
        const int fcol = tile_n * (T::BN / 2) + cc * 8;
        if (fcol < b.split) *reinterpret_cast<u32x4_t*>(e.hout + (size_t)row * b.split + fcol) = v;
      } else {
        const int col = tile_n * T::BN + cc * 8;   // 8 columns of the tile's order, one run of qkv_logical
        if (col >= N) continue;
        const int which = (col >= e.d) + (col >= 2 * e.d), pc = col - which * e.d, pp = pc & (e.dh - 1);
        const int hbase = pc - pp, in = qkv_logical(pp, e.dh >> 1);   // first column of the head, column in it
        if (which == 0) {
          *reinterpret_cast<u32x4_t*>(e.q + (size_t)row * e.d + hbase + in) = v;
        } else {
          // prefix cache: heads Pmax x d_head apart; tree K/V: a row's heads side by side
          const size_t off = kvrow[lr] + (size_t)hbase * (e.kv_mode == 0 ? e.Pmax : 1) + in;
          *reinterpret_cast<u32x4_t*>((which == 1 ? e.kdst : e.vdst) + off) = v;
        }
      }
    }
  }
}

// ------------------------------------------------------------------ launchers
// Launch of one instantiation over the tiles of a call.
template <int BMAP, int EPI, int WMW, int WNW, int TMW, int TNW, int NS = 2>
static hipError_t launch_bf16(const GemmCall& g, hipStream_t st) {
  using T = Tile<WMW, WNW, TMW, TNW>;
  BArgs b{(const bf16_t*)g.w0, (const bf16_t*)g.w1, (const bf16_t*)g.w2, g.split};
  EpiArgs e{};
  e.out = g.out; e.ldo = g.ldo; e.hout = (bf16_t*)g.hout;
  e.part = EPI == EPI_RESID ? g.part : nullptr;
  e.q = (bf16_t*)g.q; e.kdst = (bf16_t*)g.kdst; e.vdst = (bf16_t*)g.vdst;
  e.ropeT = g.ropeT; e.rows = g.rows; e.kv_mode = g.kv_mode; e.Pmax = g.Pmax;
  e.d = g.d; e.dh = g.dh;
  const int kparts = e.part ? 2 : 1;
  // each k-range is an even number of k-tiles of 64 (two stages)
  if (g.K % (kparts * 128) != 0) return hipErrorInvalidValue;
  const int Mt = (g.Mmax + T::BM - 1) / T::BM, Nt = (g.N + T::BN - 1) / T::BN;
  const int per = (kparts * Mt * Nt + 7) / 8;
  dim3 grid(8 * per);
  auto kern = gemm_bf16_kernel<WMW, WNW, TMW, TNW, BMAP, EPI, NS>;
  hipLaunchKernelGGL(kern, grid, dim3(T::NT), 0, st, (const bf16_t*)g.A, g.lda, g.Mdev, Mt, g.N, g.K, b, e);
  return hipGetLastError();
}

// Tile shape of a call, by a model of its time: with n workgroups of a shape on
// the fullest CU (at most `cap` at once, more take further rounds), a round of
// nk k-tiles costs nk * max(lat, thr * n) + epi us and the launch t0 once.  lat
// is a k-tile's own latency (barrier, LDS, MFMA chain), which few rows or few
// columns are bound by: small tiles spread those calls over more CUs; thr is a
// k-tile's share of a full CU, where large tiles move fewer bytes per MFMA.  With
// cap 1 only the larger of the two counts, and the other is whatever the fit left.
//
// The constants are fitted to measurements on MI355X, weights cold in L2: d 256,
// 768, 1,024, 2,048, 4,096 with f 1,024 to 11,008, 25 row counts from 10 to 4,800
// (7,744 at d 4,096), about 17 shapes a call.  The model's picks are on average
// within 0.3% (q/k/v, gate/up), 2.1% (o, down) and 1.3% (head) of the
// fastest shape measured.  The rule before it (fixed row thresholds, and rounds
// fitted at d 4,096 alone) was 14-21% off on the same grid: at 640 rows of
// d 768, f 3,072 q/k/v took 13.3 instead of 9.2 us, gate/up 14.3 (10.9), o 7.2
// (4.7) and down 16.0 (8.4); the head of 640 rows at d 4,096 33 (16).
// The shape does not change any element's k-order, so results do not depend on
// it.  g.Mmax is the row count of the call when the caller knows it, else an
// upper bound.
namespace {
constexpr int kCUs = 256;
struct Shape {
  int bm, bn, cap;
  float t0, lat, thr, epi;
  hipError_t (*launch)(const GemmCall&, hipStream_t);
};
const Shape kQkvShapes[] = {
    {32, 64, 2, 2.77f, 0.239f, 0.173f, 1.18f, launch_bf16<BMAP_QKV, EPI_QKV, 1, 2, 1, 1, 6>},
    {64, 64, 2, 2.49f, 0.268f, 0.204f, 1.23f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 1, 1, 4>},
    {64, 64, 3, 3.37f, 0.308f, 0.233f, 0.18f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 1, 1, 3>},
    {128, 64, 1, 1.68f, 0.339f, 0.049f, 2.40f, launch_bf16<BMAP_QKV, EPI_QKV, 4, 2, 1, 1, 4>},
    {64, 256, 1, 2.68f, 0.614f, 0.296f, 2.75f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 4, 1, 2, 3>},
    {128, 128, 1, 1.31f, 0.165f, 0.502f, 4.38f, launch_bf16<BMAP_QKV, EPI_QKV, 4, 2, 1, 2, 4>},
    {128, 128, 2, 4.05f, 0.754f, 0.505f, 1.83f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 2, 2, 2>},
    {128, 256, 1, 2.48f, 0.832f, 0.446f, 6.31f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 2, 4, 2>},
    {256, 128, 1, 0.00f, 0.775f, 0.755f, 11.42f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 4, 2, 2>},
    {192, 192, 1, 0.08f, 0.842f, 0.548f, 10.29f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 3, 3, 2>},
    {192, 256, 1, 0.00f, 1.063f, 0.098f, 11.64f, launch_bf16<BMAP_QKV, EPI_QKV, 2, 2, 3, 4, 2>},
    {256, 256, 1, 0.61f, 1.371f, 0.795f, 10.08f, launch_bf16<BMAP_QKV, EPI_QKV, 4, 2, 2, 4, 2>},
};
const Shape kGuShapes[] = {
    {64, 64, 2, 2.61f, 0.307f, 0.238f, 0.50f, launch_bf16<BMAP_GU, EPI_GU, 2, 1, 1, 2, 4>},
    {64, 128, 1, 2.37f, 0.402f, 0.374f, 0.80f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 1, 2, 4>},
    {64, 128, 2, 1.65f, 0.493f, 0.317f, 1.16f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 1, 2, 3>},
    {128, 64, 1, 1.67f, 0.388f, 0.042f, 1.68f, launch_bf16<BMAP_GU, EPI_GU, 4, 1, 1, 2, 4>},
    {128, 128, 1, 1.82f, 0.530f, 0.405f, 2.60f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 2, 2, 4>},
    {128, 128, 1, 1.84f, 0.559f, 0.436f, 1.84f, launch_bf16<BMAP_GU, EPI_GU, 4, 2, 1, 2, 3>},
    {128, 128, 2, 2.51f, 0.790f, 0.509f, 1.90f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 2, 2, 2>},
    {192, 128, 1, 0.00f, 0.738f, 0.399f, 5.33f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 3, 2, 4>},
    {128, 256, 1, 0.00f, 0.904f, 0.046f, 6.57f, launch_bf16<BMAP_GU, EPI_GU, 4, 2, 1, 4, 3>},
    {256, 128, 1, 0.00f, 0.806f, 0.154f, 5.24f, launch_bf16<BMAP_GU, EPI_GU, 4, 2, 2, 2, 3>},
    {192, 256, 1, 0.00f, 1.050f, 0.901f, 8.69f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 3, 4, 2>},
    {256, 256, 1, 0.00f, 1.204f, 1.320f, 10.15f, launch_bf16<BMAP_GU, EPI_GU, 2, 2, 4, 4, 2>},
    {256, 256, 1, 0.00f, 1.462f, 1.044f, 7.46f, launch_bf16<BMAP_GU, EPI_GU, 4, 2, 2, 4, 2>},
};
const Shape kResidShapes[] = {
    {64, 32, 2, 1.09f, 0.195f, 0.160f, 1.51f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 1, 1, 1, 6>},
    {64, 64, 1, 2.23f, 0.014f, 0.221f, 0.48f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 1, 1, 4>},
    {64, 64, 2, 1.96f, 0.269f, 0.197f, 0.66f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 1, 1, 3>},
    {64, 128, 1, 1.06f, 0.362f, 0.007f, 2.01f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 1, 2, 4>},
    {128, 64, 1, 0.40f, 0.351f, 0.297f, 2.73f, launch_bf16<BMAP_PLAIN, EPI_RESID, 4, 2, 1, 1, 4>},
    {128, 128, 1, 0.00f, 0.527f, 0.237f, 4.91f, launch_bf16<BMAP_PLAIN, EPI_RESID, 4, 2, 1, 2, 4>},
    {128, 128, 1, 0.42f, 0.161f, 0.550f, 3.50f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 2, 2, 3>},
    {128, 128, 2, 1.49f, 0.747f, 0.533f, 2.71f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 2, 2, 2>},
    {128, 256, 1, 0.00f, 0.860f, 0.547f, 6.35f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 2, 4, 2>},
    {256, 128, 1, 0.00f, 0.831f, 0.736f, 7.36f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 4, 2, 2>},
    {192, 256, 1, 0.00f, 1.061f, 0.378f, 9.12f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 3, 4, 2>},
    {256, 256, 1, 0.00f, 1.391f, 0.316f, 10.91f, launch_bf16<BMAP_PLAIN, EPI_RESID, 2, 2, 4, 4, 2>},
};
// the item rows of the output head (at most 1,024 columns)
const Shape kHeadShapes[] = {
    {64, 32, 2, 0.99f, 0.130f, 0.115f, 1.82f, launch_bf16<BMAP_PLAIN, EPI_STORE, 2, 1, 1, 1, 6>},
    {64, 64, 1, 1.96f, 0.012f, 0.166f, 0.74f, launch_bf16<BMAP_PLAIN, EPI_STORE, 2, 2, 1, 1, 4>},
    {64, 64, 3, 1.03f, 0.226f, 0.183f, 1.60f, launch_bf16<BMAP_PLAIN, EPI_STORE, 2, 2, 1, 1, 3>},
    {128, 64, 1, 0.00f, 0.202f, 0.250f, 2.97f, launch_bf16<BMAP_PLAIN, EPI_STORE, 2, 2, 2, 1, 4>},
    {128, 128, 1, 1.51f, 0.435f, 0.340f, 2.85f, launch_bf16<BMAP_PLAIN, EPI_STORE, 2, 2, 2, 2, 3>},
};

template <int NSH>
const Shape& pick_shape(const Shape (&sh)[NSH], int M, int N, int K, int kparts) {
  const float nk = (float)(K / kparts) / 64.f;
  int best = 0;
  float best_time = 0.f;
  for (int i = 0; i < NSH; ++i) {
    const Shape& s = sh[i];
    const long tiles = (long)kparts * ((M + s.bm - 1) / s.bm) * ((N + s.bn - 1) / s.bn), slots = (long)kCUs * s.cap;
    const long full = tiles / slots, rest = tiles - full * slots;
    float time = s.t0 + (float)full * (nk * std::max(s.lat, s.thr * (float)s.cap) + s.epi);
    if (rest) time += nk * std::max(s.lat, s.thr * (float)((rest + kCUs - 1) / kCUs)) + s.epi;
    if (i == 0 || time < best_time) { best = i; best_time = time; }
  }
  return sh[best];
}
}  // namespace

hipError_t gemm(const GemmCall& g, hipStream_t st) {
  if (!g.bf16) return gemm_f32(g, st);
  const int M = g.Mmax > 0 ? g.Mmax : 1;
  switch (g.kind) {
    case GEMM_QKV: return pick_shape(kQkvShapes, M, g.N, g.K, 1).launch(g, st);
    case GEMM_GU: return pick_shape(kGuShapes, M, g.N, g.K, 1).launch(g, st);
    case GEMM_RESID: return pick_shape(kResidShapes, M, g.N, g.K, g.part ? 2 : 1).launch(g, st);
    default: return pick_shape(kHeadShapes, M, g.N, g.K, 1).launch(g, st);
  }
}

}  // namespace atspeed
