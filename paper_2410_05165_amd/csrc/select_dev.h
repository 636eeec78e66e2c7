// Device helpers shared by the selection kernels: path keys, selection keys,
// trie lookup, candidate generation and TopK (one workgroup per user).
#pragma once
#include "common.h"
#include "select.h"

namespace atspeed {

__device__ __forceinline__ uint32_t path_with(uint32_t path, int level0, int code) {
  return path | ((uint32_t)code << (8 * (3 - level0)));
}
__device__ __forceinline__ int path_code(uint32_t path, int level0) { return (path >> (8 * (3 - level0))) & 0xFF; }

__device__ __forceinline__ uint64_t make_key(float score, uint32_t path) {
  return ((uint64_t)(~float_order_key(score)) << 32) | path;
}
__device__ __forceinline__ float key_score(uint64_t key) {
  uint32_t k = ~(uint32_t)(key >> 32);
  uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
  return __uint_as_float(u);
}

// Child of `node` with this code, or -1.  A node's children have distinct
// ascending codes below 256, so child i has a code of at least i and at most
// 256 - cnt + i, which bounds where the code can sit; what is left is narrowed
// eightfold a round by loads that do not wait for each other (a binary search's
// eight dependent loads per level made a tree walk's latency).
__device__ inline int trie_child(const TrieDev& t, int node, int code) {
  const int first = t.first[node], cnt = t.cnt[node];
  const int* c = t.code + first;
  int lo = max(0, code - (256 - cnt)), hi = min(cnt - 1, code);
  while (hi - lo > 7) {
    const int step = (hi - lo + 8) >> 3;      // at least 2; eight runs cover lo .. hi
    int n = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) {
      const int p = lo + k * step;
      n += p <= hi && c[min(p, hi)] <= code;
    }
    lo += n * step;
    hi = min(hi, lo + step - 1);
  }
  int found = -1;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int p = lo + k;
    if (p <= hi && c[min(p, hi)] == code) found = first + p;
  }
  return found;
}

// ---------------------------------------------------------------- selection core
constexpr int kList = 256;    // keys that select_smallest ranks against each other
struct SelShared {
  int hist[256];
  unsigned long long prefix, mask;
  int need, done, count;
  int par_off[kMaxPar + 1], par_first[kMaxPar];
  unsigned long long list[kList];
  __align__(16) uint32_t least[256];
  uint32_t bound;
};

// Where each parent's children start in the level's candidate list (sh.par_off)
// and in the trie (sh.par_first); returns the number of candidates.  A parent per
// thread and a prefix sum in one wave (a single thread adding up the counts waited
// for each parent's load in turn).
__device__ inline int list_parents(const TrieDev& trie, int npar, const int* par_trie, SelShared& sh) {
  static_assert(kMaxPar == 128, "two parents a lane");
  const int tid = threadIdx.x;
  for (int i = tid; i < kMaxPar; i += blockDim.x) {
    const int node = i < npar ? par_trie[i] : -1;
    sh.par_off[i + 1] = node >= 0 ? trie.cnt[node] : 0;
    sh.par_first[i] = node >= 0 ? trie.first[node] : 0;
  }
  __syncthreads();
  if (tid < 64) {
    const int a = sh.par_off[2 * tid + 1], b = sh.par_off[2 * tid + 2];
    int incl = a + b;
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, 64);
      if (tid >= o) incl += y;
    }
    sh.par_off[2 * tid + 1] = incl - b;
    sh.par_off[2 * tid + 2] = incl;
    if (tid == 0) sh.par_off[0] = 0;
  }
  __syncthreads();
  return sh.par_off[npar];
}

// Keys of all trie-valid one-code extensions of the parents, into keys[].
// par_lp[i] is the log-prob row of parent i; codes of item level lvl0 (0-based).
// Bound by the chain parent -> trie code -> log-prob, so a thread walks it for
// four candidates at once.
__device__ inline int gen_candidates(const TrieDev& trie, int npar, const uint32_t* par_path, const float* par_score,
                              const int* par_trie, const float* const* par_lp, int lvl0, int codebook,
                              unsigned long long* keys, SelShared& sh) {
  constexpr int U = 4;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int n = list_parents(trie, npar, par_trie, sh);
  int top = 1;
  while (2 * top < npar) top *= 2;
  for (int c0 = tid; c0 < n; c0 += U * nt) {
    int par[U], code[U];
    float lp[U];
#pragma unroll
    for (int j = 0; j < U; ++j) par[j] = 0;
    for (int step = top; step > 0; step >>= 1)   // last parent whose offset <= c
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int c = min(c0 + j * nt, n - 1), q = par[j] + step;
        if (q < npar && sh.par_off[min(q, kMaxPar)] <= c) par[j] = q;
      }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int c = min(c0 + j * nt, n - 1);
      code[j] = trie.code[sh.par_first[par[j]] + (c - sh.par_off[par[j]])];
    }
#pragma unroll
    for (int j = 0; j < U; ++j) lp[j] = par_lp[par[j]][codebook * lvl0 + code[j]];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int c = c0 + j * nt;
      if (c < n) keys[c] = make_key(par_score[par[j]] + lp[j], path_with(par_path[par[j]], lvl0, code[j]));
    }
  }
  __syncthreads();
  return n;
}

// Radix select: the nsel smallest of n keys, unsorted, into sh.list (8 bits of the
// key a pass, a 256-bin histogram in LDS).  sh.count holds their number.
__device__ inline void radix_smallest(const unsigned long long* keys, int n, int nsel, SelShared& sh) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (tid == 0) { sh.prefix = 0; sh.mask = 0; sh.need = nsel; sh.done = (nsel == n); sh.count = 0; }
  __syncthreads();
  for (int shift = 56; shift >= 0 && !sh.done; shift -= 8) {
    for (int i = tid; i < 256; i += nt) sh.hist[i] = 0;
    __syncthreads();
    const unsigned long long pf = sh.prefix, mk = sh.mask;
    for (int c = tid; c < n; c += nt) {
      unsigned long long k = keys[c];
      if ((k & mk) == pf) atomicAdd(&sh.hist[(k >> shift) & 255], 1);
    }
    __syncthreads();
    if (tid < 64) {
      // wave 0 finds the bucket b where the running count first reaches need:
      // a prefix sum over 4 buckets per lane, then the one lane holding the
      // crossing (below b < need <= below b + hist[b]) records it
      const int h[4] = {sh.hist[4 * tid], sh.hist[4 * tid + 1], sh.hist[4 * tid + 2], sh.hist[4 * tid + 3]};
      const int s4 = h[0] + h[1] + h[2] + h[3];
      int incl = s4;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (tid >= o) incl += y;
      }
      const int need = sh.need;
      int below = incl - s4, b = -1, bbelow = 0, hb = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (b < 0 && below < need && below + h[q] >= need) { b = 4 * tid + q; bbelow = below; hb = h[q]; }
        below += h[q];
      }
      if (b >= 0) {
        sh.need = need - bbelow;
        sh.prefix |= (unsigned long long)b << shift;
        sh.mask |= 0xFFull << shift;
        if (hb == need - bbelow) sh.done = 1;
      }
    }
    __syncthreads();
  }
  const unsigned long long pf = sh.prefix, mk = sh.mask;
  const bool all = (nsel == n);
  for (int c = tid; c < n; c += nt) {
    unsigned long long k = keys[c];
    if (all || (k & mk) <= pf) {
      int slot = atomicAdd(&sh.count, 1);
      if (slot < kList) sh.list[slot] = k;
    }
  }
  __syncthreads();
}

// The nsel smallest keys, ascending, into out[]; returns their number.  Equal keys
// (a beam that the caller's state holds twice, a path that its tree holds twice) each
// take a place of their own, so every one of the nsel entries is written; at most
// kMaxPar copies of the nsel-th key and fewer than kMaxSel keys before it fit the list.
// Bound by latency (one workgroup, a few thousand keys at most): up to kList keys are ranked
// against each other at once.  More are first cut down to those whose score is at
// least the nsel-th best of the threads' own best scores: nsel threads hold a key
// that good, so none of the nsel best is lost, and about as many keys pass as are
// wanted (two passes over the keys; a radix select alone took up to nine).  Only
// where more than kList keys pass, as with many equal scores, does the radix select
// cut them down.  Drafting 40 of 20 parents' or 40 drafted nodes' extensions for 16
// users, level by level: 13.2 -> 9.0 us a level.
__device__ inline int select_smallest(const unsigned long long* keys, int n, int nsel, unsigned long long* out, SelShared& sh) {
  static_assert(kMaxSel + kMaxPar <= kList, "every selection fits the list");
  const int tid = threadIdx.x, nt = blockDim.x;
  if (nsel > n) nsel = n;
  int m = n;
  if (n <= kList) {
    for (int c = tid; c < n; c += nt) sh.list[c] = keys[c];
    __syncthreads();
  } else {
    uint32_t mine = ~0u;
#pragma unroll 4
    for (int c = tid; c < n; c += nt) mine = min(mine, (uint32_t)(keys[c] >> 32));
    sh.least[tid] = mine;
    if (tid == 0) { sh.count = 0; sh.bound = 0; }
    __syncthreads();
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < nt; i += 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(&sh.least[i]);
      rank += (v.x < mine) + (v.y < mine) + (v.z < mine) + (v.w < mine);
    }
    if (rank < nsel) atomicMax(&sh.bound, mine);
    __syncthreads();
    const uint32_t bound = sh.bound;
#pragma unroll 4
    for (int c = tid; c < n; c += nt) {
      const unsigned long long k = keys[c];
      if ((uint32_t)(k >> 32) <= bound) {
        const int slot = atomicAdd(&sh.count, 1);
        if (slot < kList) sh.list[slot] = k;
      }
    }
    __syncthreads();
    if (sh.count > kList) {
      __syncthreads();                       // every thread has read sh.count
      radix_smallest(keys, n, nsel, sh);
    }
    m = min(sh.count, kList);
  }
  for (int i = tid; i < m; i += nt) {
    const unsigned long long k = sh.list[i];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < m; ++j) rank += sh.list[j] < k || (sh.list[j] == k && j < i);
    if (rank < nsel) out[rank] = k;
  }
  __syncthreads();
  return nsel;
}

}  // namespace atspeed
