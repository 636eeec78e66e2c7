// Tree attention (tree-based attention of Sec. 3.3 and its implementation
// appendix, restated): a query row of user u attends to the first nctx keys of
// u's prefix KV cache and to its own tree keys (ancestors and itself, at most L).
// The same kernel runs causal prefill (nctx = position + 1, no tree keys).
//
// One workgroup handles (user, head, 64 query rows of that user): the user's
// prefix K/V are streamed once per workgroup in 64-key tiles through LDS and
// shared by all its queries (the prefix is read once per user per layer, not
// once per tree token).  Softmax is online (running max and sum) in fp32.
// Workgroup L runs on XCD L % 8: the (user, head) pairs are dealt round-robin
// over the XCDs, a pair's query blocks on one of them.
#include "common.h"
#include "kernels.h"

namespace atspeed {

// ---------------------------------------------------------------- fp32 kernel
// Per workgroup: (head, user, 64 query rows); wave w owns queries 16w..16w+15.
// S^T = K Q^T with v_mfma_f32_16x16x4_f32, a lane's 16-byte K and Q fragments
// feeding four of them (MFMA e takes dims 16 ks + 4 (lane / 16) + e).  Lane l
// then holds S^T[key 4g+i][query l%16] (g = l/16), which is the B operand of
// O^T = V^T P^T for the MFMA over keys {i, 4+i, 8+i, 12+i}, so probabilities stay
// in registers.  Each query's tree keys (ancestors and itself) follow, one dot
// product split over the 4 lanes of the query.
//
// Bound by latency at the sizes fp32 models run (tens of rows, a few key tiles):
// the next tile's loads are in flight during the current tile's MFMAs, and the
// key range is the last row's, so nothing is exchanged before the first tile.
// One user's 30-60 rows over 80 keys at d_head 32 took 18-21 us with vector FMAs
// over LDS and take 7-9; 120 rows x 8 users over 120 keys at d_head 64, 41 -> 15.
template <int DH>
__global__ void __launch_bounds__(256)
attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ pk, const float* __restrict__ pv,
                const float* __restrict__ tk, const float* __restrict__ tv, float* __restrict__ out, Rows rows,
                int H, int Pmax, float qscale, int nusers, int nqblk) {
  constexpr int KT = 64;          // keys per tile
  constexpr int NKS = DH / 16;    // 16-dim groups of S^T
  constexpr int NDB = DH / 16;    // 16-dim blocks of O^T
  constexpr int CPR = DH / 4;     // 16-byte chunks per row
  __shared__ __align__(16) float Ks[KT * DH];
  __shared__ __align__(16) float Vs[KT * DH];
  // chunk swizzles: K fragments are read 16 rows at one chunk, V 4 rows (4 apart)
  // at one 16-dim block
  auto kswz = [](int key) { return CPR >= 16 ? key & 15 : (key >> 1) & 7; };
  auto vswz = [](int key) { return ((key >> 2) & (NDB >= 4 ? 3 : 1)) << 2; };

  const int Lw = blockIdx.x, xcd = Lw & 7, qi8 = Lw >> 3, Z = nqblk;
  const int pair = (qi8 / Z) * 8 + xcd, zb = qi8 % Z;
  if (pair >= H * nusers) return;
  const int u = pair / H, h = pair % H;
  const int ubeg = rows.user_off[u], uend = rows.user_off[u + 1];
  const int r0 = ubeg + zb * 64;
  if (r0 >= uend) return;
  const int nq = min(64, uend - r0);
  const int kmax = rows.nctx[r0 + nq - 1];   // never decreases along a user's rows
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, ql = lane & 15;
  const int qi = wave * 16 + ql;
  const bool valid = qi < nq;
  const int row = r0 + (valid ? qi : 0);
  const int d = H * DH;
  const size_t kvbase = ((size_t)u * H + h) * Pmax * DH;

  constexpr int NC = KT * CPR / 256;         // chunks per thread of a K (or V) tile
  f32x4_t kreg[NC], vreg[NC];
  auto fetch = [&](int k0) {
    const int nk = min(KT, kmax - k0);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int idx = tid + c * 256, key = idx / CPR, j = idx % CPR;
      const size_t o = kvbase + (size_t)(k0 + key) * DH + j * 4;
      kreg[c] = key < nk ? *reinterpret_cast<const f32x4_t*>(pk + o) : f32x4_t{0.f, 0.f, 0.f, 0.f};
      vreg[c] = key < nk ? *reinterpret_cast<const f32x4_t*>(pv + o) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  };
  if (kmax > 0) fetch(0);
  const int nctx = valid ? rows.nctx[row] : 0;
  f32x4_t qf[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    qf[ks] = valid ? *reinterpret_cast<const f32x4_t*>(q + (size_t)row * d + h * DH + ks * 16 + g * 4)
                   : f32x4_t{0.f, 0.f, 0.f, 0.f};
  f32x4_t o[NDB];
#pragma unroll
  for (int i = 0; i < NDB; ++i) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;

  for (int k0 = 0; k0 < kmax; k0 += KT) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int idx = tid + c * 256, key = idx / CPR, j = idx % CPR;
      *reinterpret_cast<f32x4_t*>(Ks + key * DH + (j ^ kswz(key)) * 4) = kreg[c];
      *reinterpret_cast<f32x4_t*>(Vs + key * DH + (j ^ vswz(key)) * 4) = vreg[c];
    }
    __syncthreads();
    if (k0 + KT < kmax) fetch(k0 + KT);
    f32x4_t sc[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) sc[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      f32x4_t kf[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        const int key = kb * 16 + ql;
        kf[kb] = *reinterpret_cast<const f32x4_t*>(Ks + key * DH + ((ks * 4 + g) ^ kswz(key)) * 4);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
          sc[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kb][e], qf[ks][e], sc[kb], 0, 0, 0);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = k0 + kb * 16 + g * 4 + i;
        const float v = key < nctx ? sc[kb][i] * qscale : -INFINITY;
        sc[kb][i] = v;
        mx = fmaxf(mx, v);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mnew = fmaxf(m, mx);
    const float alpha = (m == -INFINITY) ? 0.f : exp2f(m - mnew);
    float ps = 0.f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = (sc[kb][i] == -INFINITY) ? 0.f : exp2f(sc[kb][i] - mnew);
        sc[kb][i] = p;
        ps += p;
      }
    lsum = lsum * alpha + ps;
    m = mnew;
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] *= alpha;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = kb * 16 + 4 * g + i;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const int dim = db * 16 + ql;
          const float vf = Vs[key * DH + (((dim >> 2) ^ vswz(key)) << 2) + (dim & 3)];
          o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf, sc[kb][i], o[db], 0, 0, 0);
        }
      }
    __syncthreads();
  }

  if (tk != nullptr && valid) {  // tree keys: ancestors and self
    const int na = rows.nanc[row];
    int slot[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) slot[a] = a < na ? rows.anc[row * 4 + a] : 0;
    float sa[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      float part = 0.f;
      if (a < na) {
        const float* kp = tk + (size_t)slot[a] * d + h * DH + g * 4;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          const f32x4_t kf = *reinterpret_cast<const f32x4_t*>(kp + ks * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) part += qf[ks][e] * kf[e];
        }
      }
      part += __shfl_xor(part, 16);
      part += __shfl_xor(part, 32);
      sa[a] = a < na ? part * qscale : -INFINITY;
    }
    const float mx = fmaxf(fmaxf(sa[0], sa[1]), fmaxf(sa[2], sa[3]));
    const float mnew = fmaxf(m, mx);
    const float alpha = (m == -INFINITY) ? 0.f : exp2f(m - mnew);
    float ps = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      sa[a] = a < na ? exp2f(sa[a] - mnew) : 0.f;
      ps += sa[a];
    }
    lsum = lsum * alpha + (g == 0 ? ps : 0.f);
    // lane (query, g) holds dims db*16 + 4g .. +3 of O
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] *= alpha;
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (a < na) {
        const float* vp = tv + (size_t)slot[a] * d + h * DH + g * 4;
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] += sa[a] * *reinterpret_cast<const f32x4_t*>(vp + db * 16);
      }
  }
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  if (valid) {
    const float inv = 1.f / lsum;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      *reinterpret_cast<f32x4_t*>(out + (size_t)row * d + h * DH + db * 16 + g * 4) = o[db] * inv;
  }
}

// ---------------------------------------------------------------- bf16 kernel
// Per workgroup: (head, user, 64 query rows); wave w owns queries 16w..16w+15.
// S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (A = K rows from LDS, B = Q from
// registers): lane l holds S^T[key 4g+i][query l%16] (g = l/16) of each 16-key
// block, so the probabilities of its query sit in registers in exactly the
// B-operand layout of O^T = V^T P^T, with the 32 keys of a k-step ordered
// {4g..4g+3, 16+4g..16+4g+3} on both operands.  V rows sit in LDS as they are; a
// transposing read (4 keys x 16 dims per 16 lanes) gives V^T's fragments.
// Each query's tree keys (ancestors and itself) follow, one dot product split
// over the 4 lanes of the query.
//
// Bound by vector instructions around the MFMAs at long contexts and by the chain
// of dependent loads at short ones, so a tile whose keys every query of the wave
// sees carries no mask, the accumulators are rescaled only when a maximum moved,
// waves without queries only help to stage, and nothing is exchanged before the
// first tile.  With V transposed by shifts on the way into LDS, masks on every tile
// and range-checked exponentials, at 16 users x ~230 rows over 1,024 keys of d_head
// 128 a layer took 285 us (199 now), 16 users x 960 causal rows 799 (560), and 640
// rows over 144 keys at 12 heads of 64 13.6 (11.9).
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// a - b of the rounded a: not to be contracted with the product a may be, so that
// a score's distance from the maximum does not depend on the branch it came by.
__device__ __forceinline__ float sub_rn(float a, float b) {
#pragma clang fp contract(off)
  return a - b;
}

template <int DH>
__global__ void __launch_bounds__(256)
attn_mfma_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ pk, const bf16_t* __restrict__ pv,
                 const bf16_t* __restrict__ tk, const bf16_t* __restrict__ tv, bf16_t* __restrict__ out, Rows rows,
                 int H, int Pmax, float qscale, int nusers, int nqblk) {
  constexpr int KT = 64;          // keys per tile
  constexpr int NKS = DH / 32;    // k-steps of S^T
  constexpr int NDB = DH / 16;    // 16-dim blocks of O^T
  constexpr int CPR = DH / 8;     // 16-byte chunks per row
  constexpr bool EARLY = DH == 64;   // tree K/V loaded before the tiles (at d_head 128 they would cost a wave per SIMD)
  __shared__ __align__(16) bf16_t Ks[KT * DH];
  __shared__ __align__(16) bf16_t Vs[KT * DH];
  // K fragments are read 16 rows at one chunk; V 8 rows at one 16-dim block (two chunks)
  auto vswz = [](int key) { return (DH == 128 ? key & 7 : (key >> 1) & 3) << 1; };

  // Workgroup L runs on XCD L % 8.  The Z query blocks of one (user, head) pair
  // get consecutive indices on one XCD, so they run together and share the
  // pair's prefix tiles in that XCD's L2; the pairs are dealt round-robin over
  // the XCDs.
  const int Lw = blockIdx.x, xcd = Lw & 7, qi8 = Lw >> 3, Z = nqblk;
  const int pair = (qi8 / Z) * 8 + xcd, zb = qi8 % Z;
  if (pair >= H * nusers) return;
  const int u = pair / H, h = pair % H;
  const int ubeg = rows.user_off[u], uend = rows.user_off[u + 1];
  const int r0 = ubeg + zb * 64;
  if (r0 >= uend) return;
  const int nq = min(64, uend - r0);
  const int kmax = rows.nctx[r0 + nq - 1];   // never decreases along a user's rows
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, ql = lane & 15;
  const int qi = wave * 16 + ql;
  const bool valid = qi < nq, active = wave * 16 < nq;
  const int row = r0 + (valid ? qi : 0);
  const int d = H * DH;
  const size_t kvbase = ((size_t)u * H + h) * Pmax * DH;

  // Tile staging: 16-byte chunks, NKC of K and of V per thread.  The next tile's
  // global loads are issued into registers before the current tile's matrix work.
  constexpr int NKC = KT * CPR / 256;
  u32x4_t kreg[NKC], vreg[NKC];
  auto fetch = [&](int k0) {
    const int nk = min(KT, kmax - k0);
#pragma unroll
    for (int c = 0; c < NKC; ++c) {
      const int idx = tid + c * 256, key = idx / CPR, j = idx % CPR;
      const size_t o = kvbase + (size_t)(k0 + key) * DH + j * 8;
      kreg[c] = key < nk ? *reinterpret_cast<const u32x4_t*>(pk + o) : u32x4_t{0u, 0u, 0u, 0u};
      vreg[c] = key < nk ? *reinterpret_cast<const u32x4_t*>(pv + o) : u32x4_t{0u, 0u, 0u, 0u};
    }
  };
  if (kmax > 0) fetch(0);
  const int nctx = valid ? rows.nctx[row] : 0;
  const int seen = active ? rows.nctx[r0 + wave * 16] : 0;   // keys every query of the wave sees
  bf16x8_t qf[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    if (valid) qf[ks] = *reinterpret_cast<const bf16x8_t*>(q + (size_t)row * d + h * DH + ks * 32 + g * 8);
    else qf[ks] = bf16x8_t{};
  }
  // tree keys of this query: slots, and at d_head 64 their K and V already
  const bool tree = tk != nullptr && valid;
  const int na = tree ? rows.nanc[row] : 0;
  int slot[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) slot[a] = a < na ? rows.anc[row * 4 + a] : 0;
  bf16x8_t tkf[EARLY ? 4 : 1][NKS];
  uint2 tvf[EARLY ? 4 : 1][NDB];
  auto load_k = [&](int a, bf16x8_t (&f)[NKS]) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      f[ks] = *reinterpret_cast<const bf16x8_t*>(tk + (size_t)slot[a] * d + h * DH + ks * 32 + g * 8);
  };
  auto load_v = [&](int a, uint2 (&f)[NDB]) {   // lane (query, g) takes dims db*16 + 4g .. +3
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      f[db] = *reinterpret_cast<const uint2*>(tv + (size_t)slot[a] * d + h * DH + g * 4 + db * 16);
  };
  if constexpr (EARLY) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (a < na) load_k(a, tkf[a]);
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (a < na) load_v(a, tvf[a]);
  }
  f32x4_t o[NDB];
#pragma unroll
  for (int i = 0; i < NDB; ++i) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;

  for (int k0 = 0; k0 < kmax; k0 += KT) {
#pragma unroll
    for (int c = 0; c < NKC; ++c) {
      const int idx = tid + c * 256, key = idx / CPR, j = idx % CPR;
      *reinterpret_cast<u32x4_t*>(Ks + key * DH + ((j ^ (key & (CPR - 1))) * 8)) = kreg[c];
      *reinterpret_cast<u32x4_t*>(Vs + key * DH + ((j ^ vswz(key)) * 8)) = vreg[c];
    }
    __syncthreads();
    if (k0 + KT < kmax) fetch(k0 + KT);
    if (active) {
      // S^T for 4 blocks of 16 keys
      f32x4_t sc[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        sc[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        const int key = kb * 16 + ql;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          const int j = ks * 4 + g;
          const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(Ks + key * DH + ((j ^ (key & (CPR - 1))) * 8));
          sc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[ks], sc[kb], 0, 0, 0);
        }
      }
      const bool full = k0 + KT <= seen;
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) sc[kb] *= qscale;
      if (!full) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (k0 + kb * 16 + g * 4 + i >= nctx) sc[kb][i] = -INFINITY;
      }
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sc[kb][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mnew = fmaxf(m, mx);
      float alpha = 1.f;
      if (__any(mnew > m)) {   // else every factor is 1
        alpha = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mnew);
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] *= alpha;
        m = mnew;
      }
      // probabilities; below 2^-126 of the largest they are zero.  A query that has
      // seen no key yet (m is -inf) takes 0 in place of -inf - -inf.
      const float mref = m != -INFINITY ? m : 0.f;
      float ps = 0.f;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f(sub_rn(sc[kb][i], mref));
          sc[kb][i] = p;
          ps += p;
        }
      lsum = __builtin_fmaf(lsum, alpha, ps);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        // P as the sum of two bf16 parts (hi + lo ~ 16 significant bits), so the
        // probabilities keep near-fp32 precision through the bf16 MFMA.
        bf16x8_t pf, pl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pf[i] = (__bf16)sc[2 * kk][i];
          pf[4 + i] = (__bf16)sc[2 * kk + 1][i];
          pl[i] = (__bf16)(sc[2 * kk][i] - (float)pf[i]);
          pl[4 + i] = (__bf16)(sc[2 * kk + 1][i] - (float)pf[4 + i]);
        }
        // lane (g, ql) addresses 4 dims of key 4g + ql / 4 and receives its own dim
        // of keys 4g .. 4g + 3
        const int key = kk * 32 + 4 * g + (ql >> 2);
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const int j = db * 2 + ((ql >> 1) & 1);
          const bf16_t* v0 = Vs + key * DH + ((j ^ vswz(key)) << 3) + (ql & 1) * 4;
          const bf16_t* v1 = Vs + (key + 16) * DH + ((j ^ vswz(key + 16)) << 3) + (ql & 1) * 4;
          const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)v0);
          const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)v1);
          const auto w8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, w8);
          o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[db], 0, 0, 0);
          o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl, o[db], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }

  if (tree) {  // tree keys: ancestors and self
    float sa[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      float part = 0.f;
      if (a < na) {
        if constexpr (!EARLY) load_k(a, tkf[0]);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) part += (float)qf[ks][e] * (float)tkf[EARLY ? a : 0][ks][e];
      }
      part += __shfl_xor(part, 16);
      part += __shfl_xor(part, 32);
      sa[a] = a < na ? part * qscale : -INFINITY;
    }
    const float mx = fmaxf(fmaxf(sa[0], sa[1]), fmaxf(sa[2], sa[3]));
    const float mnew = fmaxf(m, mx);
    const float alpha = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mnew);
    float ps = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      sa[a] = a < na ? __builtin_amdgcn_exp2f(sa[a] - mnew) : 0.f;
      ps += sa[a];
    }
    lsum = lsum * alpha + (g == 0 ? ps : 0.f);
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] *= alpha;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      if (a < na) {
        if constexpr (!EARLY) load_v(a, tvf[0]);
        const float p = sa[a];
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const uint2 w = tvf[EARLY ? a : 0][db];
          o[db][0] += p * __uint_as_float(w.x << 16);
          o[db][1] += p * __uint_as_float(w.x & 0xffff0000u);
          o[db][2] += p * __uint_as_float(w.y << 16);
          o[db][3] += p * __uint_as_float(w.y & 0xffff0000u);
        }
      }
    }
  }
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  if (valid) {
    const float inv = 1.f / lsum;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      uint2 w;
      w.x = (uint32_t)f2bf(o[db][0] * inv) | ((uint32_t)f2bf(o[db][1] * inv) << 16);
      w.y = (uint32_t)f2bf(o[db][2] * inv) | ((uint32_t)f2bf(o[db][3] * inv) << 16);
      *reinterpret_cast<uint2*>(out + (size_t)row * d + h * DH + db * 16 + g * 4) = w;
    }
  }
}

// One-dimensional grid: ceil(pairs / 8) groups of 8 (user, head) pairs x Z query blocks.
template <class T, class F>
static hipError_t launch(const AttnCall& a, F kern, int dh, hipStream_t st) {
  const float qscale = 1.4426950408889634f / sqrtf((float)dh);   // log2(e) / sqrt(d_head)
  const int Z = std::max(1, (a.Tq + 63) / 64);
  const long pairs = (long)a.H * a.B;
  const long nwg = (pairs + 7) / 8 * 8 * Z;
  if (nwg > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)nwg), dim3(256), 0, st, (const T*)a.q, (const T*)a.pk, (const T*)a.pv,
                     (const T*)a.tk, (const T*)a.tv, (T*)a.out, a.rows, a.H, a.Pmax, qscale, a.B, Z);
  return hipGetLastError();
}

hipError_t attention(const AttnCall& a, hipStream_t st) {
  if (a.bf16) {
    if (a.dh == 64) return launch<bf16_t>(a, attn_mfma_kernel<64>, 64, st);
    if (a.dh == 128) return launch<bf16_t>(a, attn_mfma_kernel<128>, 128, st);
  } else {
    if (a.dh == 32) return launch<float>(a, attn_f32_kernel<32>, 32, st);
    if (a.dh == 64) return launch<float>(a, attn_f32_kernel<64>, 64, st);
    if (a.dh == 128) return launch<float>(a, attn_f32_kernel<128>, 128, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace atspeed
