// Decode-time constraint filter (CD + GTM) and trie step (GRACE, Sec. 4, Sec. 5.4,
// App. A) for gfx950.
//
// gtm_mask: the child entries (CSR ranges) of a workgroup's beams are dealt out
//   evenly over its threads.  A thread reads an entry's two matcher rows in one
//   go, tests them against the request's bitmask and locations, and ORs the
//   surviving token into its beam's filter words in LDS, which the workgroup
//   then stores whole.  The request-side matchers are shared by the beams of a
//   request and wait in LDS where the workgroup's beams belong to one request.
// trie_advance: one lane per new beam: binary search of its token among the
//   parent node's child tokens (ascending within a node's range).
#include "common.hpp"
#include "kernels.hpp"

namespace grace {

constexpr int kGtmThreads = 256;
constexpr int kMaxBm = 8, kMaxBl = 4, kMaxLocs = 64;
static_assert(kMaxLocs * kMaxBl <= kGtmThreads, "one word of a request's locations per thread");

struct GtmDev {
  const int32_t* off;
  const int32_t* child;
  const int16_t* tok;
  const int32_t* bmi;
  const int32_t* bli;
  const uint64_t* bmt;
  const uint64_t* blt;
  int32_t nodes, entries, V, wbm, wbl, bm_rows, bl_rows;
};

struct UserDev {
  const uint64_t* bm;
  const uint64_t* bl;
  const int32_t* nloc;
  int32_t lmax;
};

// Bound by latency: node -> range -> entry -> matcher rows is a chain of four
// dependent loads, so everything that can be in flight at once is: the ranges of
// all the workgroup's beams with the request's matchers, then all their entries,
// each with both matcher rows whole (16-byte loads) instead of word by word up to
// the first miss.  64 x 4096 beams with 2.5 children each: 16 lanes per beam and
// early exits 106 us, this 26 us; eight beams at the root, 512 children: 46 and
// 7 us.  At 64 x 4096 with 30 children each it is the vector ALU: 263 and 120 us.
constexpr int kGtmMaxBeams = 128;     // per workgroup
constexpr int kGtmWordsCap = 4096;    // filter words per workgroup (16 KiB of LDS)
constexpr int32_t kGtmLongRange = 1 << 22;   // 256 ranges of this length sum to 2^30

// n 64-bit words (n <= N, uniform) of a matcher row, zero beyond: 16-byte loads
// of two (the row is 8-byte aligned).
template <int N>
__device__ __forceinline__ void load_words(const uint64_t* p, int n, uint32_t (&w)[2 * N]) {
#pragma unroll
  for (int j = 0; j < N; j += 2) {
    u32x4 q = {0u, 0u, 0u, 0u};
    if (j + 1 < n) {
      typedef u32x4 __attribute__((aligned(8))) u32x4_a8;
      q = *(const u32x4_a8*)(p + j);
    } else if (j < n) {
      const u32x2 h = *(const u32x2*)(p + j);
      q = u32x4{h.x, h.y, 0u, 0u};
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) w[2 * j + e] = q[e];
  }
}

// Bits of want[0..n) that have does not hold (0: all are there).
template <int N>
__device__ __forceinline__ uint32_t missing(const uint32_t* want, const uint32_t (&absent)[N]) {
  uint32_t acc = 0u;
#pragma unroll
  for (int j = 0; j < N; ++j) acc |= want[j] & absent[j];
  return acc;
}

// A request's matchers, zero beyond its words and locations.
struct GtmUser {
  uint32_t bm[2 * kMaxBm];
  uint32_t bl[kMaxLocs][2 * kMaxBl];
};

// beams: beam rows per workgroup, a power of two up to kGtmMaxBeams with
// beams * ceil(V/32) <= kGtmWordsCap (dynamic LDS).
__global__ void __launch_bounds__(kGtmThreads)
gtm_mask_kernel(GtmDev ix, UserDev us, const int32_t* __restrict__ node_ids, int32_t R, FastDiv per_request,
                int32_t beams, uint32_t* __restrict__ mask, int32_t* __restrict__ err_flag) {
  extern __shared__ uint32_t words[];
  // first entry of beam i; entries of beams 0 .. i (of beam i alone where by_beam)
  __shared__ int32_t first[kGtmMaxBeams], upto[kGtmMaxBeams];
  __shared__ uint32_t wave_total[kGtmThreads / 64];
  const int tid = threadIdx.x;
  const int32_t r0 = (int32_t)((int64_t)blockIdx.x * beams);
  const int32_t nb = min(beams, R - r0);
  const int W = (ix.V + 31) >> 5;
  const int32_t b0 = (int32_t)per_request.div((uint32_t)r0);
  const bool one = (int32_t)per_request.div((uint32_t)(r0 + nb - 1)) == b0;
  __shared__ __attribute__((aligned(16))) GtmUser user;
  int32_t nloc0 = 0;
  if (one) {   // the request's matchers, on the way while the ranges are looked up
    nloc0 = us.nloc[b0];
    nloc0 = nloc0 < 0 ? 0 : (nloc0 > us.lmax ? us.lmax : nloc0);
    if (tid < kMaxBm) {
      const uint64_t w = tid < ix.wbm ? us.bm[(int64_t)b0 * ix.wbm + tid] : 0ull;
      user.bm[2 * tid] = (uint32_t)w;
      user.bm[2 * tid + 1] = (uint32_t)(w >> 32);
    }
    const int q = tid / kMaxBl, j = tid % kMaxBl;   // one word of a location per thread
    const uint64_t w = q < us.lmax && j < ix.wbl ? us.bl[((int64_t)b0 * us.lmax + q) * ix.wbl + j] : 0ull;
    user.bl[q][2 * j] = (uint32_t)w;
    user.bl[q][2 * j + 1] = (uint32_t)(w >> 32);
  }
  for (int i = tid; i < nb * W; i += kGtmThreads) words[i] = 0u;
  bool bad = false;
  // the beams' child ranges and their running total
  int32_t e0 = 0, n = 0;
  if (tid < nb) {
    const int32_t node = node_ids[r0 + tid];
    if (node >= 0 && node < ix.nodes) {
      int32_t e1 = ix.off[node + 1];
      e0 = ix.off[node];
      e0 = e0 < 0 ? 0 : (e0 > ix.entries ? ix.entries : e0);
      e1 = e1 < e0 ? e0 : (e1 > ix.entries ? ix.entries : e1);
      n = e1 - e0;
    } else {
      bad = node >= ix.nodes;   // negative ids are dead beams; ids past the trie are errors
    }
  }
  // a node has at most 4096 distinct tokens; ranges so long that their sum
  // could overflow (bad data) are taken beam by beam below, as are beams with so
  // many children that a whole workgroup finds enough in each (the root's 512:
  // 64 x 4096 beams there 1063 us dealt out, 862 beam by beam)
  bool by_beam = __syncthreads_or(n > kGtmLongRange) != 0;
  const uint32_t sum = wave_scan((uint32_t)n);
  if ((tid & 63) == 63) wave_total[tid >> 6] = sum;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kGtmThreads / 64; ++w) {
    before += w < (tid >> 6) ? wave_total[w] : 0u;
    all += wave_total[w];
  }
  by_beam = by_beam || all >= (uint32_t)(nb * kGtmThreads);
  if (tid < kGtmMaxBeams) {
    first[tid] = e0;
    upto[tid] = by_beam ? n : (int32_t)(before + sum);
  }
  __syncthreads();
  uint32_t u_one[2 * kMaxBm];   // the request's bitmask, in scalar registers
#pragma unroll
  for (int j = 0; j < 2 * kMaxBm; ++j) u_one[j] = one ? __builtin_amdgcn_readfirstlane(user.bm[j]) : 0u;
  // entry e of beam `slot` (none where !live); called by whole waves
  auto entry = [&](int slot, int32_t e, bool live) {
    int32_t v = 0, bi = 0, li = 0;
    if (live) {
      v = ix.tok[e];
      bi = ix.bmi[e];
      li = ix.bli[e];
      if (v < 0 || v >= ix.V || bi < 0 || bi >= ix.bm_rows || li < 0 || li >= ix.bl_rows) {
        bad = true;
        live = false;
      }
    }
    // what the entry's matchers lack: every user attribute bit has to be in the
    // bitmask, and some location's filter in the Bloom row
    uint32_t nbm[2 * kMaxBm] = {}, nbl[2 * kMaxBl] = {};
    if (live) {
      load_words<kMaxBm>(ix.bmt + (int64_t)bi * ix.wbm, ix.wbm, nbm);
      load_words<kMaxBl>(ix.blt + (int64_t)li * ix.wbl, ix.wbl, nbl);
    }
#pragma unroll
    for (int j = 0; j < 2 * kMaxBm; ++j) nbm[j] = ~nbm[j];
#pragma unroll
    for (int j = 0; j < 2 * kMaxBl; ++j) nbl[j] = ~nbl[j];
    bool ok = false;
    if (one) {
      live = live && missing(u_one, nbm) == 0u;
      // four locations per step, the last repeated past the end
      for (int32_t q = 0; q < nloc0 && __any(live && !ok); q += 4) {
        uint32_t lacks[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) lacks[i] = missing(user.bl[min(q + i, nloc0 - 1)], nbl);
        ok = ok || min(min(lacks[0], lacks[1]), min(lacks[2], lacks[3])) == 0u;
      }
      ok = ok && live;
    } else if (live) {
      const int64_t b = per_request.div((uint32_t)(r0 + slot));
      int32_t nloc = us.nloc[b];
      nloc = nloc < 0 ? 0 : (nloc > us.lmax ? us.lmax : nloc);
      uint32_t u[2 * kMaxBm], l[2 * kMaxBl];
      load_words<kMaxBm>(us.bm + b * ix.wbm, ix.wbm, u);
      if (missing(u, nbm) == 0u)
        for (int32_t q = 0; q < nloc && !ok; ++q) {
          load_words<kMaxBl>(us.bl + (b * us.lmax + q) * ix.wbl, ix.wbl, l);
          ok = missing(l, nbl) == 0u;
        }
    }
    if (ok) atomicOr(&words[slot * W + (v >> 5)], 1u << (v & 31));
  };
  if (!by_beam) {
    const int32_t total = upto[nb - 1];
    for (int32_t i0 = 0; i0 < total; i0 += kGtmThreads) {
      const int32_t i = i0 + tid;
      // the beam: the first whose running total exceeds i
      int slot = 0;
      for (int step = beams >> 1; step > 0; step >>= 1)
        if (upto[slot + step - 1] <= i) slot += step;
      entry(slot, first[slot] + i - (slot > 0 ? upto[slot - 1] : 0), i < total);
    }
  } else {
    for (int slot = 0; slot < nb; ++slot)
      for (int64_t i0 = 0; i0 < upto[slot]; i0 += kGtmThreads)
        entry(slot, first[slot] + (int32_t)(i0 + tid), i0 + tid < upto[slot]);
  }
  __syncthreads();
  uint32_t* out = mask + (int64_t)r0 * W;
  for (int i = tid; i < nb * W; i += kGtmThreads) out[i] = words[i];
  if (bad && err_flag) *err_flag = 1;
}

__global__ void __launch_bounds__(kGtmThreads)
trie_advance_kernel(GtmDev ix, const int32_t* __restrict__ node_prev,
                    const int32_t* __restrict__ parents, const int32_t* __restrict__ tokens,
                    int32_t n, int32_t M_prev, int32_t k, int32_t* __restrict__ node_next,
                    int32_t* __restrict__ err_flag) {
  const int32_t i = (int32_t)blockIdx.x * kGtmThreads + (int32_t)threadIdx.x;
  if (i >= n) return;
  const int32_t b = i / k, p = parents[i], v = tokens[i];
  int32_t out = -1;
  if (p < 0 || p >= M_prev) {
    if (err_flag) *err_flag = 1;
  } else {
    const int32_t node = node_prev[(int64_t)b * M_prev + p];
    if (node >= ix.nodes) {
      if (err_flag) *err_flag = 1;
    } else if (node >= 0) {
      int32_t lo = ix.off[node], end = ix.off[node + 1];
      lo = lo < 0 ? 0 : (lo > ix.entries ? ix.entries : lo);
      end = end < lo ? lo : (end > ix.entries ? ix.entries : end);
      int32_t hi = end;
      while (lo < hi) {   // first entry with token >= v
        const int32_t mid = (lo + hi) >> 1;
        if (ix.tok[mid] < v) lo = mid + 1;
        else hi = mid;
      }
      if (lo < end && ix.tok[lo] == v) out = ix.child[lo];
    }
  }
  node_next[i] = out;
}

static GtmDev to_dev(const grace_gtm_index& x) {
  return GtmDev{x.node_offsets, x.child_nodes, x.tokens, x.bitmask_index, x.bloom_index,
                x.bitmask_table, x.bloom_table, x.num_nodes, x.num_entries, x.vocab,
                x.bitmask_words, x.bloom_words, x.bitmask_rows, x.bloom_rows};
}

hipError_t launch_gtm_mask(const grace_gtm_index& index, const grace_gtm_user& user,
                           const int32_t* node_ids, int32_t R, int32_t M, uint32_t* mask,
                           int32_t* err_flag, hipStream_t stream) {
  const UserDev us{user.bitmask, user.bloom, user.num_locations, user.max_locations};
  // Beams per workgroup, as many as leave a chip full of workgroups: 2048 (eight
  // per CU), or 1024 of few beams, where starting a workgroup (5 ns) counts (8 x
  // 1024 beams at level 2: 7.4 us with 1024, 10.8 with 2048; 64 x 1024 at level 1:
  // 58 and 38), or 640 of fewer still, which keeps the grid within 1280 (3300 and
  // 1561 beams at level 3: 8.9 and 8.6 us with 1024, 6.4 and 6.0 with 640; 13000 at
  // level 1: 15.7 and 28).  Their filter words have to fit.
  const int32_t W = (index.vocab + 31) / 32, fill = R >= 32768 ? 2048 : (R >= 4096 ? 1024 : 640);
  int32_t beams = 1;
  while (beams < kGtmMaxBeams && R / (2 * beams) >= fill && 2 * beams * W <= kGtmWordsCap) beams *= 2;
  const int64_t blocks = ((int64_t)R + beams - 1) / beams;
  hipLaunchKernelGGL(gtm_mask_kernel, dim3((unsigned)blocks), dim3(kGtmThreads), (size_t)beams * W * 4, stream,
                     to_dev(index), us, node_ids, R, FastDiv((uint32_t)M), beams, mask, err_flag);
  return hipGetLastError();
}

hipError_t launch_trie_advance(const grace_gtm_index& index, const int32_t* node_prev,
                               const int32_t* parents, const int32_t* tokens, int32_t B,
                               int32_t M_prev, int32_t k, int32_t* node_next, int32_t* err_flag,
                               hipStream_t stream) {
  const int32_t n = B * k;
  hipLaunchKernelGGL(trie_advance_kernel, dim3((unsigned)((n + kGtmThreads - 1) / kGtmThreads)),
                     dim3(kGtmThreads), 0, stream, to_dev(index), node_prev, parents, tokens, n,
                     M_prev, k, node_next, err_flag);
  return hipGetLastError();
}

}  // namespace grace
