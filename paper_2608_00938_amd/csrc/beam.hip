// Beam score update and per-request top-k (GRACE, Sec. 3.1, Sec. 3.3) for gfx950.
//
// scores: one wave per beam row (or several rows), the row in registers.  The
//   row's log-softmax over the vocabulary is added to the beam's accumulated
//   score; filtered tokens score -inf.  The kernel also writes each row's best
//   candidate score.
// top-k:  candidates are totally ordered by an order-preserving 32-bit key of
//   the score (descending; -0 == +0; NaN below -inf), then by flat index
//   m*V + v (ascending), so the selection is unique.
//   N <= 65536 candidates per request: one workgroup per request holds them all
//   in registers, finds by a histogram of the 64-unit window below the best
//   score the bin with the k-th candidate, and ranks that bin and above.
//   More: a sample of the candidates picks a threshold above which somewhat
//   more than k are expected (select), one pass over the candidates gathers
//   everything at or above it (gather), and the gathered set, which holds the k
//   best exactly when it has at least k members, is ranked (final).  A set that
//   does not fit the list, of crowded scores or from a coarse sample, goes on
//   behind the sample and is narrowed to the list by digits of its entries.
//   When fewer than k candidates are above -inf (dead beams), the rest are the
//   -inf candidates of lowest index.  When the gathered set is too small or
//   does not fit the workspace, an exact radix select on the key (digits of 12, 12
//   and 8 bits) and an index-ordered collection of the tied candidates take over.
//   Ranking: a counting sort over bins of the gathered range and a comparison
//   inside each bin, or a bitonic sort in LDS when a bin is crowded.
#include <float.h>
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace grace {

// ---------------------------------------------------------------------------
// wave reductions over 64 lanes, every lane gets the result.  Partners are
// lanes l ^ 32, 16, 8, 4, 2, 1 in that order; all six steps stay in the vector
// ALU (half and row swaps, row rotations, quad permutes) instead of going
// through LDS.  A rotation by 4 within 16 lanes reaches l ^ 4 because lanes l
// and l ^ 8 already agree.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// The six steps for NR values of each lane at once (NR = 1, 2 or 4), sharing
// the swaps and all later steps: row j's result ends in the lanes of group
// lane_of_row<NR>(j) (all lanes for NR = 1, a half for 2, 16 lanes for 4).  Each
// row's order of operations is that of NR = 1.
template <int NR>
__device__ __forceinline__ constexpr int lane_of_row(int j) {
  return NR == 1 ? 0 : (NR == 2 ? 32 * j : 32 * (j & 1) + 16 * (j >> 1));
}
template <int NR>
__device__ __forceinline__ int row_of_lane(int lane) {
  return NR == 1 ? 0 : (NR == 2 ? lane >> 5 : (lane >> 5) + 2 * ((lane >> 4) & 1));
}
template <class Op>
__device__ __forceinline__ float swap_halves(float a, float b, Op op) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return op(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
template <int NR, class Op>
__device__ __forceinline__ float reduce_rows(const float (&v)[NR], Op op) {
  static_assert(NR == 1 || NR == 2 || NR == 4, "rows per wave");
  const float y = swap_halves(v[0], v[NR > 1 ? 1 : 0], op);
  float w = y;
  if constexpr (NR == 4) w = swap_halves(v[2], v[3], op);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(w), false, false);
  float x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  x = op(x, dpp<0x128>(x));   // row_ror:8
  x = op(x, dpp<0x124>(x));   // row_ror:4
  x = op(x, dpp<0x4E>(x));    // quad_perm 2,3,0,1
  return op(x, dpp<0xB1>(x)); // quad_perm 1,0,3,2
}
template <int NR>
__device__ __forceinline__ float max_rows(const float (&v)[NR]) {
  return reduce_rows<NR>(v, [](float a, float b) { return max3(a, b, b); });
}
template <int NR>
__device__ __forceinline__ float sum_rows(const float (&v)[NR]) {
  return reduce_rows<NR>(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float x) { return max_rows<1>({x}); }
__device__ __forceinline__ float wave_sum(float x) { return sum_rows<1>({x}); }
// x of lane l, in a scalar register
__device__ __forceinline__ float lane_value(float x, int l) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), l));
}

template <class T>
__device__ __forceinline__ float load_logit(const T* p);
template <>
__device__ __forceinline__ float load_logit<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float load_logit<uint16_t>(const uint16_t* p) {
  return __uint_as_float((uint32_t)*p << 16);
}

// x where bit e of `bits` is set, else -inf (one bit-field extract, one bit select)
__device__ __forceinline__ float keep_bit(float x, uint32_t bits, int e) {
  const uint32_t m = (uint32_t)((int32_t)(bits << (31 - e)) >> 31);
  return __uint_as_float((__float_as_uint(x) & m) | (0xff800000u & ~m));
}

constexpr int kHistBins = 4096;    // bins of the threshold and ranking histograms
constexpr int kGatherCap = 8192;   // gathered candidates a request can rank

// Workspace of one call.  Per request: the gathered list [kGatherCap] of
// composites, S sample areas of kSampleArea fp16 (the last one doubles as the
// select workgroups' common histogram; what the sample leaves of them takes the
// gathered composites past the list), info [kInfo] = {threshold (float bits),
// gathered count, how the selection ended (kRanked, kNarrowed, kExact), workgroups
// done, unused...}.  S grows with the candidates of a request, one area per 32768
// up to 64.
constexpr int kMaxSlices = 64;
constexpr uint32_t kSliceTarget = 32768;
constexpr int kInfo = 8;
constexpr int kSampleArea = 2 * kHistBins;
constexpr int32_t kRanked = 0, kNarrowed = 1, kExact = 2;

__host__ __device__ inline int topk_slices(uint32_t N) {
  const uint32_t s = (N + kSliceTarget - 1) / kSliceTarget;
  return (int)(s < 1 ? 1 : (s > (uint32_t)kMaxSlices ? (uint32_t)kMaxSlices : s));
}

struct TopkWs {
  uint64_t* list = nullptr;
  uint16_t* sample = nullptr;
  int32_t* info = nullptr;
  int S = 0;
  int32_t spill = 0;   // fp16 of the sample areas that the sample takes, a multiple of 4
  TopkWs() = default;
  __host__ __device__ TopkWs(void* ws, int B, int S_) : S(S_) {
    char* p = (char*)ws;
    list = (uint64_t*)p;
    p += (size_t)B * kGatherCap * 8;
    sample = (uint16_t*)p;
    p += (size_t)B * S_ * kHistBins * 4 + (size_t)B * S_ * 4;
    info = (int32_t*)p;
  }
  __host__ __device__ static size_t bytes(int B, int S_) {
    return (size_t)B * kGatherCap * 8 + (size_t)B * S_ * kHistBins * 4 + (size_t)B * S_ * 4 +
           (size_t)B * kInfo * 4;
  }
  __host__ __device__ int64_t sample_stride() const { return (int64_t)S * kSampleArea; }
  __host__ __device__ int64_t sample_room() const { return (int64_t)(S - 1) * kSampleArea; }
  // composites a request can hold: the list and behind the sample
  __host__ __device__ uint32_t gather_room() const {
    return (uint32_t)kGatherCap + (uint32_t)(sample_stride() - spill) / 4;
  }
  __device__ __forceinline__ uint32_t* hist(int64_t b) const {
    return (uint32_t*)(sample + b * sample_stride() + sample_room());
  }
};

// Clears what several workgroups of a request's selection share (the score pass
// does it where there is one).
__device__ __forceinline__ void clear_shared(const TopkWs& ws, int64_t b, uint32_t first, uint32_t step) {
  uint32_t* sum = ws.hist(b);
  for (uint32_t i = first; i < (uint32_t)kHistBins; i += step) sum[i] = 0u;
  if (first == 0) ws.info[b * kInfo + 1] = ws.info[b * kInfo + 3] = 0;
}

// How the workgroups of one request hand what they share (counts, list entries)
// to the last of them to finish; nobody waits for anybody.  Writers use relaxed
// agent-scope read-modify-writes only, which every XCD sees in one order per
// location.  Then every wave waits until its own are performed (publish_shared,
// in the place of a release: no plain store is handed over, and a release fence
// writes back the whole L2, 170 against 11 us for the threshold kernel in 512
// workgroups), and one thread takes a ticket.  The thread with the last ticket
// acquires at agent scope, so that what its workgroup reads after the next
// barrier is read after all the tickets and from no older copy in a cache of its
// XCD; those reads are relaxed agent-scope loads.
__device__ __forceinline__ void publish_shared() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}
// One thread, after publish_shared: 1 in the last of n workgroups, else 0.
__device__ __forceinline__ int32_t last_to_finish(int32_t* done, int32_t n) {
  if (__hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != n - 1) return 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return 1;
}
template <class T>
__device__ __forceinline__ T load_shared(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// candidate scores
// ---------------------------------------------------------------------------
constexpr int kScoreThreads = 256;

// A score pass that keeps no candidate array writes a sample of it instead: of
// every 2^lp consecutive tokens of a row the one at an offset that changes from
// row to row (so that no token order biases it), ceil(V / 2^lp) per row, -inf
// past the row's end and in three places behind a request's last row; 3 <= lp
// <= 9.  Stored as fp16 differences from a score
// near the request's best prefix (sample_ref): the sample only has to place a
// threshold, which a difference of up to 16 gets to 1/128.
struct SampleOut {
  uint16_t* p = nullptr;     // [B][stride], request b's rows in order; null: no sample
  int64_t stride = 0;
  TopkWs ws;                 // what the selection's workgroups share is cleared too
  uint32_t per_row = 0;
  int32_t lp = 0, M = 1;
  FastDiv per_request{1};    // row -> request
};
__device__ __forceinline__ uint32_t sample_offset(uint32_t row, int lp) {
  return (row * 0x9E3779B1u) >> (32 - lp);
}
// The best of up to 64 of the request's prefix scores, 0 if none is finite;
// called by a whole wave.
__device__ __forceinline__ float sample_ref(const float* prev, int32_t M) {
  const int lane = threadIdx.x & 63;
  const float p = prev[(int64_t)M * lane / 64];
  const float m = wave_max(fabsf(p) < INFINITY ? p : -INFINITY);
  return m > -INFINITY ? m : 0.f;
}
// Two fp32 values as fp16, rounded toward zero (monotonic; beyond the range to
// its end, infinities kept).
__device__ __forceinline__ uint32_t pack_f16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Generic row kernel (any V): lanes stride over the row.  CAND = false writes
// only the row's log-sum-exp (lse_out) and an upper bound of its candidates
// (row_max), for a top-k that recomputes each candidate from the logits.
template <class T, bool CAND = true>
__global__ void __launch_bounds__(kScoreThreads)
beam_scores_kernel(const T* __restrict__ logits, const float* __restrict__ prev,
                   const uint32_t* __restrict__ mask, float* __restrict__ cand,
                   float* __restrict__ row_max, float* __restrict__ lse_out, int32_t R, int32_t V,
                   SampleOut smp) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * (kScoreThreads / 64) + (threadIdx.x >> 6);
  if (r >= R) return;   // whole waves
  const T* x = logits + r * V;
  float mx = -INFINITY;
  for (int v = lane; v < V; v += 64) mx = fmaxf(mx, load_logit(x + v));
  mx = wave_max(mx);
  float z = 0.f;
  for (int v = lane; v < V; v += 64) z += fast_exp2((load_logit(x + v) - mx) * kLog2e);
  z = wave_sum(z);
  const float lse = mx + logf(z);
  const float p = prev[r];
  const int32_t words = (V + 31) >> 5;
  auto score = [&](int v) {
    const bool ok = mask == nullptr || ((mask[r * words + (v >> 5)] >> (v & 31)) & 1u);
    return ok ? p + (load_logit(x + v) - lse) : -INFINITY;
  };
  if constexpr (CAND) {
    float best = -INFINITY;
    float* out = cand + r * V;
    for (int v = lane; v < V; v += 64) {
      const float s = score(v);
      out[v] = s;
      best = fmaxf(best, s);
    }
    best = wave_max(best);
    if (row_max != nullptr && lane == 0) row_max[r] = best;
  } else {
    if (lane == 0) {
      row_max[r] = p + (mx - lse);
      lse_out[r] = lse;
    }
    if (smp.p == nullptr) return;
    const uint32_t b = smp.per_request.div((uint32_t)r), m = (uint32_t)r - b * (uint32_t)smp.M;
    const uint32_t h = sample_offset(m, smp.lp);
    const float ref = sample_ref(prev + (int64_t)b * smp.M, smp.M);
    uint16_t* out = smp.p + b * smp.stride + (int64_t)m * smp.per_row;
    for (uint32_t i = lane; i < smp.per_row; i += 64) {
      const uint32_t v = (i << smp.lp) + h;
      out[i] = (uint16_t)pack_f16x2(v < (uint32_t)V ? score((int)v) - ref : -INFINITY, 0.f);
    }
    if (m == (uint32_t)smp.M - 1 && lane < 3) out[smp.per_row + lane] = 0xfc00u;
    clear_shared(smp.ws, b, m * 64 + lane, (uint32_t)smp.M * 64);
  }
}

// Row kernel with the row in registers across the max, sum and output passes:
// NCH runs of 8 tokens per lane, V <= 512*NCH.  RUN = true (V a multiple of 8,
// 16-byte aligned logits): a run is 8 consecutive tokens, one 16-byte bf16 load
// or two fp32 loads; else its tokens are 64 apart, so that a wave's loads cover
// consecutive tokens.  The sums of exp run over a lane's tokens in order and
// then over the lanes as in the generic kernel.
//
// The row sums of exp take the hardware exp2 of a log2(e)-scaled argument
// (relative error about 1e-6 per term against 2^-24 for expf), which keeps
// the pass from being bound by the vector ALU.
//
// CAND = false: the candidates' upper bound prev + (max - lse) holds for every
// token, as rounding is monotonic, so neither the filter nor the candidates are
// needed for it.
// Rows per wave.  A pass that writes the candidates is bound by those writes and
// takes one (64 x 4096 x 512 bf16: 135 us with one row, 153 with two, 191 with
// four, whose stores leave in bursts); without them the vector ALU counts, and
// the reductions of four rows at once take it from 88 to 60 us.
template <int NCH, bool CAND>
constexpr int score_rows_per_wave() { return CAND ? 1 : (NCH == 1 ? 4 : (NCH == 2 ? 2 : 1)); }

template <class T, int NCH, bool RUN, bool CAND>
__global__ void __launch_bounds__(kScoreThreads)
beam_scores_reg_kernel(const T* __restrict__ logits, const float* __restrict__ prev,
                       const uint32_t* __restrict__ mask, float* __restrict__ cand,
                       float* __restrict__ row_max, float* __restrict__ lse_out, int32_t R,
                       int32_t V, SampleOut smp) {
  // RPW rows per wave, all their loads issued before the first reduction, which
  // runs over all of them at once
  constexpr int RPW = score_rows_per_wave<NCH, CAND>();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = ((int64_t)blockIdx.x * (kScoreThreads / 64) + wave) * RPW;
  if (r0 >= R) return;   // whole waves
  const int32_t words = (V + 31) >> 5;
  const bool sampled = !CAND && smp.p != nullptr;
  auto token = [&](int c, int e) { return RUN ? c * 512 + 8 * lane + e : (c * 8 + e) * 64 + lane; };
  // rows past the last repeat it and are not written
  auto row = [&](int j) { return min(r0 + j, (int64_t)R - 1); };
  float f[RPW][NCH][8];
  uint32_t bits[RPW][NCH];
#pragma unroll
  for (int j = 0; j < RPW; ++j) {
    const int64_t r = row(j);
    const T* x = logits + r * V;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if constexpr (RUN) {
        const int v0 = token(c, 0);
        if (v0 < V) {
          if constexpr (sizeof(T) == 2) {
            Chunk<BF16>::unpack(*(const u32x4*)(x + v0), f[j][c]);
          } else {
            Chunk<F32>::unpack(*(const u32x4*)(x + v0), f[j][c]);
            Chunk<F32>::unpack(*(const u32x4*)(x + v0 + 4), f[j][c] + 4);
          }
          if (CAND || sampled)
            bits[j][c] = mask == nullptr ? 0xffu : mask[r * words + (v0 >> 5)] >> (v0 & 31);
        }
      } else {
        bits[j][c] = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int v = token(c, e);
          if (v < V) {
            f[j][c][e] = load_logit(x + v);
            if constexpr (CAND)
              bits[j][c] |= (mask == nullptr ? 1u : (mask[r * words + (v >> 5)] >> (v & 31)) & 1u) << e;
          }
        }
      }
    }
  }
  const int64_t r_lane = row(row_of_lane<RPW>(lane));   // the row whose results this lane gets
  const float p_lane = prev[r_lane];
  const bool writes = (lane & (64 / RPW - 1)) == 0 && r0 + row_of_lane<RPW>(lane) < R;
  float part[RPW];
#pragma unroll
  for (int j = 0; j < RPW; ++j) {
    float mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if constexpr (RUN) {
        if (token(c, 0) < V) {
#pragma unroll
          for (int e = 0; e < 8; e += 2) mx = max3(mx, f[j][c][e], f[j][c][e + 1]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (token(c, e) < V) mx = fmaxf(mx, f[j][c][e]);
      }
    }
    part[j] = mx;
  }
  const float mx_lane = max_rows<RPW>(part);
#pragma unroll
  for (int j = 0; j < RPW; ++j) {
    const float mx = lane_value(mx_lane, lane_of_row<RPW>(j));
    float z = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if constexpr (RUN) {
        if (token(c, 0) < V) {
#pragma unroll
          for (int e = 0; e < 8; ++e) z += fast_exp2((f[j][c][e] - mx) * kLog2e);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (token(c, e) < V) z += fast_exp2((f[j][c][e] - mx) * kLog2e);
      }
    }
    part[j] = z;
  }
  const float lse_lane = mx_lane + logf(sum_rows<RPW>(part));
  if constexpr (CAND) {
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
      part[j] = -INFINITY;
      if (r0 + j >= R) continue;   // whole waves
      const float lse = lane_value(lse_lane, lane_of_row<RPW>(j));
      const float p = lane_value(p_lane, lane_of_row<RPW>(j));
      float best = -INFINITY;
      float* out = cand + (r0 + j) * V;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        float o[8];
        // streamed past the caches: the array is larger than L2 and MALL, and
        // the top-k reads it back with streaming loads as well
        if constexpr (RUN) {
          const int v0 = token(c, 0);
          if (v0 >= V) continue;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = keep_bit(p + (f[j][c][e] - lse), bits[j][c], e);
#pragma unroll
          for (int e = 0; e < 8; e += 2) best = fmaxf(best, fmaxf(o[e], o[e + 1]));
          __builtin_nontemporal_store(Chunk<F32>::pack(o), (u32x4*)(out + v0));
          __builtin_nontemporal_store(Chunk<F32>::pack(o + 4), (u32x4*)(out + v0 + 4));
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int v = token(c, e);
            if (v < V) {
              o[e] = keep_bit(p + (f[j][c][e] - lse), bits[j][c], e);
              best = fmaxf(best, o[e]);
              __builtin_nontemporal_store(o[e], out + v);
            }
          }
        }
      }
      part[j] = best;
    }
    const float best_lane = max_rows<RPW>(part);
    if (row_max != nullptr && writes) row_max[r_lane] = best_lane;
  } else {
    if (writes) {
      row_max[r_lane] = p_lane + (mx_lane - lse_lane);
      lse_out[r_lane] = lse_lane;
    }
    if (!sampled) return;
    uint32_t b_ref = 0xffffffffu;
    float ref = 0.f;
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
      if (r0 + j >= R) continue;
      const uint32_t r = (uint32_t)(r0 + j);
      const uint32_t b = smp.per_request.div(r), m = r - b * (uint32_t)smp.M;
      if (b != b_ref) ref = sample_ref(prev + (int64_t)b * smp.M, smp.M);   // whole waves
      b_ref = b;
      const float lse = lane_value(lse_lane, lane_of_row<RPW>(j));
      const float p = lane_value(p_lane, lane_of_row<RPW>(j));
      const uint32_t h = sample_offset(m, smp.lp);
      uint16_t* out = smp.p + b * smp.stride + (int64_t)m * smp.per_row;
      if (m == (uint32_t)smp.M - 1 && lane < 3) out[smp.per_row + lane] = 0xfc00u;
      clear_shared(smp.ws, b, m * 64 + lane, (uint32_t)smp.M * 64);
      if constexpr (RUN) {
        // one element of every 2^(lp-3)-th run; the RPW rows of a wave share
        // out the eight elements, so that two (four, eight) remain to pick from
        constexpr int kPick = 8 / RPW;
        const uint32_t runs = 1u << (smp.lp - 3), q = h & (kPick - 1);
        const auto pick = [](bool hi, float x, float y) { return hi ? y : x; };   // by value
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          float t[kPick];
#pragma unroll
          for (int e = 0; e < kPick; ++e) t[e] = f[j][c][j * kPick + e];
#pragma unroll
          for (int w = 1; w < kPick; w *= 2)
#pragma unroll
            for (int e = 0; e + w < kPick; e += 2 * w) t[e] = pick(q & w, t[e], t[e + w]);
          const uint32_t e = j * kPick + q, run = c * 64 + lane;
          if ((run & (runs - 1)) == (h >> 3) && 8 * (run & ~(runs - 1)) < (uint32_t)V) {
            const bool ok = 8 * run < (uint32_t)V && ((bits[j][c] >> e) & 1u);
            out[(8 * run) >> smp.lp] =
                (uint16_t)pack_f16x2(ok ? p + (t[0] - lse) - ref : -INFINITY, 0.f);
          }
        }
      } else {
        // from memory again: at most an eighth of the row, in cache
        for (uint32_t i = lane; i < smp.per_row; i += 64) {
          const uint32_t v = (i << smp.lp) + h;
          float sc = -INFINITY;
          if (v < (uint32_t)V && (mask == nullptr || ((mask[r * (int64_t)words + (v >> 5)] >> (v & 31)) & 1u)))
            sc = p + (load_logit(logits + (int64_t)r * V + v) - lse) - ref;
          out[i] = (uint16_t)pack_f16x2(sc, 0.f);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// top-k
// ---------------------------------------------------------------------------
constexpr int kTopkThreads = 1024;
constexpr float kWindow = 64.0f;        // small requests: threshold window below the best score
constexpr uint32_t kSmallN = 65536;     // candidates one workgroup holds in registers

// Order-preserving key: larger key = better candidate.  -0 maps to +0's key,
// NaN to 0 (below -inf, whose key is 0x007fffff).
__device__ __forceinline__ uint32_t order_key(float x) {
  uint32_t u = __float_as_uint(x);
  if (x != x) return 0u;
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Sort key: key in the high word, inverted index in the low word, so that a
// descending sort puts better scores first and the lower index first on ties.
__device__ __forceinline__ uint64_t composite(uint32_t key, uint32_t idx) {
  return ((uint64_t)key << 32) | (uint64_t)(~idx);
}

// Bin of x in kHistBins equal steps of 1/inv_w up from lo; bin 0 also takes
// everything below (and -inf and NaN).  Monotonic in x.
__device__ __forceinline__ int step_bin(float x, float lo, float inv_w) {
  const float t = (x - lo) * inv_w;
  return t > 0.f ? (int)fminf(t, (float)(kHistBins - 1)) : 0;
}

// Add 1 to hist[bin] for every lane with pred set: one LDS atomic for the
// whole wave when all those lanes agree on the bin (crowded bins), else one
// per lane.  Called by the whole wave.
__device__ __forceinline__ void hist_add(uint32_t* hist, int bin, bool pred) {
  const uint64_t active = __ballot(pred);
  if (active == 0) return;
  const int lead = (int)__builtin_ctzll(active);
  const int b0 = __shfl(bin, lead);
  if (__ballot(pred && bin == b0) == active) {
    if ((int)(threadIdx.x & 63) == lead) atomicAdd(&hist[b0], (uint32_t)__popcll(active));
  } else if (pred) {
    atomicAdd(&hist[bin], 1u);
  }
}

// Bitonic sort of list[0, n) descending; n a power of two <= capacity.
__device__ void bitonic_desc(uint64_t* list, int n) {
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < (n >> 1); i += kTopkThreads) {
        const int lo = 2 * i - (i & (stride - 1));
        const int hi = lo + stride;
        const bool desc = (lo & size) == 0;
        const uint64_t a = list[lo], b = list[hi];
        if ((a < b) == desc) {
          list[lo] = b;
          list[hi] = a;
        }
      }
      __syncthreads();
    }
  }
}

// Exclusive prefix of one uint32 per thread over the block (1024 threads);
// *total receives the sum.  Every wave scans the wave totals for itself.
__device__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* scratch, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t v = wave_scan(x);
  if (lane == 63) scratch[wave] = v;
  __syncthreads();
  const uint32_t w = wave_scan(scratch[lane & (kTopkThreads / 64 - 1)]);   // lanes 0-15: the sums
  *total = (uint32_t)__builtin_amdgcn_readlane((int)w, kTopkThreads / 64 - 1);
  const uint32_t before = wave == 0 ? 0u : (uint32_t)__shfl((int)w, wave - 1);
  __syncthreads();
  return before + v - x;
}

// Where the top-k reads candidate scores: the array the score kernel wrote,
// or each score recomputed from the logits with the same operations and the
// row's stored log-sum-exp, so that both give the same bits.
struct CandArray {
  const float* cand;
  struct Row {   // one request's candidates
    const float* p;
    __device__ __forceinline__ float operator[](uint32_t i) const { return p[i]; }
    __device__ __forceinline__ float nt(uint32_t i) const { return __builtin_nontemporal_load(&p[i]); }
    // candidates i .. i+7 (i and N multiples of 8, p 16-byte aligned)
    __device__ __forceinline__ void load8(uint32_t i, float (&x)[8]) const {
      Chunk<F32>::unpack(*(const u32x4*)(p + i), x);
      Chunk<F32>::unpack(*(const u32x4*)(p + i + 4), x + 4);
    }
  };
  __device__ __forceinline__ Row request(int64_t b, uint32_t N) const {
    return Row{cand + b * (int64_t)N};
  }
};

template <class T>
struct CandFromLogits {
  const T* logits;
  const float* prev;
  const uint32_t* mask;   // NULL: every token allowed
  const float* lse;       // per row
  int32_t M, V;
  FastDiv per_row;        // request-local candidate index -> beam
  struct Row {
    const T* logits;
    const float* prev;
    const uint32_t* mask;
    const float* lse;
    int64_t r0;
    int32_t V;
    FastDiv per_row;
    __device__ __forceinline__ float operator[](uint32_t i) const {
      const uint32_t m = per_row.div(i), v = i - m * (uint32_t)V;
      const int64_t r = r0 + m;
      const int32_t words = (V + 31) >> 5;
      const bool ok = mask == nullptr || ((mask[r * words + (v >> 5)] >> (v & 31)) & 1u);
      return ok ? prev[r] + (load_logit(logits + r * V + v) - lse[r]) : -INFINITY;
    }
    __device__ __forceinline__ float nt(uint32_t i) const { return (*this)[i]; }
    // what the E candidates from flat index i on, of beam m, are made of: their
    // logits as stored, the row's prefix score and log-sum-exp
    template <int E>
    struct Raw {
      u32x4 w[E > 1 ? E * sizeof(T) / 16 : 1];
      float p, l;
      __device__ __forceinline__ void logits(float (&f)[E]) const {
        if constexpr (E == 1) {
          f[0] = __uint_as_float(w[0].x);
        } else if constexpr (sizeof(T) == 2) {
          Chunk<BF16>::unpack(w[0], f);
        } else {
          Chunk<F32>::unpack(w[0], f);
          Chunk<F32>::unpack(w[1], f + 4);
        }
      }
    };
    template <int E>
    __device__ __forceinline__ void load_raw(uint32_t i, uint32_t m, Raw<E>& raw) const {
      const T* x = logits + r0 * V + i;
      if constexpr (E == 1) {
        raw.w[0].x = __float_as_uint(load_logit(x));
      } else {
        raw.w[0] = *(const u32x4*)x;
        if constexpr (sizeof(T) == 4) raw.w[1] = *(const u32x4*)(x + 4);
      }
      raw.p = prev[r0 + m];
      raw.l = lse[r0 + m];
    }
    // and their scores
    template <int E>
    __device__ __forceinline__ void finish(uint32_t i, uint32_t m, const Raw<E>& raw, float (&x)[E]) const {
      float f[E];
      raw.logits(f);
      const uint32_t v = i - m * (uint32_t)V;
      const int32_t words = (V + 31) >> 5;
      const uint32_t bits = mask == nullptr ? 0xffu : mask[(r0 + m) * words + (v >> 5)] >> (v & 31);
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] = keep_bit(raw.p + (f[e] - raw.l), bits, e);
    }
    // candidates i .. i+7 (i and V multiples of 8, so one row): one 16-byte
    // run of logits, as the score kernel's 8-token runs
    __device__ __forceinline__ void load8(uint32_t i, float (&x)[8]) const {
      const uint32_t m = per_row.div(i), v = i - m * (uint32_t)V;
      const int64_t r = r0 + m;
      const T* row = logits + r * V + v;
      float f[8];
      if constexpr (sizeof(T) == 2) {
        Chunk<BF16>::unpack(*(const u32x4*)row, f);
      } else {
        Chunk<F32>::unpack(*(const u32x4*)row, f);
        Chunk<F32>::unpack(*(const u32x4*)(row + 4), f + 4);
      }
      const int32_t words = (V + 31) >> 5;
      const uint32_t bits =
          mask == nullptr ? 0xffu : (mask[r * words + (v >> 5)] >> (v & 31)) & 0xffu;
      const float p = prev[r], l = lse[r];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = ((bits >> e) & 1u) ? p + (f[e] - l) : -INFINITY;
    }
  };
  __device__ __forceinline__ Row request(int64_t b, uint32_t) const {
    return Row{logits, prev, mask, lse, b * M, V, per_row};
  }
};

struct TopkShared {
  uint64_t list[kGatherCap];
  // members per bin (counted from the top bin down), then the first position
  // of each bin in the bin-ordered list; the threshold histograms use the first
  uint32_t bin_count[kHistBins];
  uint32_t bin_start[kHistBins];
  uint32_t scan[64];
  float fscan[2 * kTopkThreads / 64];
  int32_t ipar[4];
  uint32_t max_count, n_list;
};

// Bins at most this full are ranked by comparing a candidate with the other
// members of its bin; fuller bins take the bitonic sort.
constexpr uint32_t kRankBinCap = 512;

// The score a fast-path key came from (finite scores only; -0 is read back
// from the candidates because its key is +0's).
__device__ __forceinline__ float key_score(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

__device__ __forceinline__ float block_max(float x, float* scratch) {
  x = wave_max(x);
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = x;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  x = wave_max(lane < kTopkThreads / 64 ? scratch[lane] : -INFINITY);
  __syncthreads();
  return x;
}

__device__ __forceinline__ void clear_bins(uint32_t* bins) {
  for (int i = threadIdx.x; i < kHistBins; i += kTopkThreads) bins[i] = 0u;
}

// The highest bin b >= 1 of hist with at least `want` counts in bins >= b, or 0
// when bins >= 1 hold fewer; ipar[1] gets the counts in the bins above it, ipar[2]
// its own.  hist is complete (a barrier since its last update).  Ends with a barrier.
__device__ int boundary_bin(const uint32_t* hist, uint32_t want, uint32_t* scan, int32_t* ipar) {
  const int tid = threadIdx.x;
  if (tid == 0) ipar[0] = 0;
  // thread 0 owns the top 4 bins, in descending order
  const int t_rev = kTopkThreads - 1 - tid;
  uint32_t own[4], s4 = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    own[e] = 4 * t_rev + 3 - e > 0 ? hist[4 * t_rev + 3 - e] : 0u;
    s4 += own[e];
  }
  uint32_t total;
  const uint32_t before = block_exclusive_scan(s4, scan, &total);
  if (before < want && before + s4 >= want) {
    uint32_t run = before;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (run < want && run + own[e] >= want) {
        ipar[0] = 4 * t_rev + 3 - e;
        ipar[1] = (int32_t)run;
        ipar[2] = (int32_t)own[e];
      }
      run += own[e];
    }
  }
  if (tid == 0 && total < want) {
    ipar[1] = (int32_t)total;
    ipar[2] = (int32_t)hist[0];
  }
  __syncthreads();
  const int b = ipar[0];
  __syncthreads();
  return b;
}

// Calls put(composite) for each of a lane's candidates x[0..7] (flat indices
// i ..) at or above thr: few lanes have any, and most of those one.
template <int E, class Put>
__device__ __forceinline__ void for_hits(const float (&x)[E], uint32_t i, float thr, Put put) {
  uint32_t hits = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) hits |= x[e] >= thr ? 1u << e : 0u;
  if (hits == 0) return;
  put.reserve((uint32_t)__popc(hits));
  do {
    const int e = __ffs(hits) - 1;
    hits &= hits - 1;
    float y = x[0];
#pragma unroll
    for (int q = 1; q < E; ++q) y = e == q ? x[q] : y;
    put(composite(order_key(y), i + e));
  } while (hits != 0);
}

// To a list in LDS: one LDS atomic per lane with candidates.
struct PutList {
  uint64_t* list;
  uint32_t* count;
  uint32_t cap, pos = 0;
  __device__ __forceinline__ void reserve(uint32_t n) { pos = atomicAdd(count, n); }
  __device__ __forceinline__ void operator()(uint64_t v) {
    if (pos < cap) list[pos] = v;
    ++pos;
  }
};

struct TopkOut {
  int32_t* parents;
  int32_t* tokens;
  float* scores;
  FastDiv per_row;   // flat index -> beam
  int32_t V;
  __device__ __forceinline__ void put(int64_t at, uint32_t idx, float score) const {
    const uint32_t m = per_row.div(idx);
    parents[at] = (int32_t)m;
    tokens[at] = (int32_t)(idx - m * (uint32_t)V);
    scores[at] = score;
  }
};

// The selected composites sh.list[0, n), n >= k or all there are, sorted best
// first; the first min(n, k) are emitted.
template <class Row>
__device__ __forceinline__ void sort_and_emit(TopkShared& sh, uint32_t n, int32_t k, int64_t out0, const Row& c,
                              const TopkOut& out) {
  uint32_t n2 = 1;
  while (n2 < n) n2 <<= 1;
  for (uint32_t i = n + threadIdx.x; i < n2; i += kTopkThreads) sh.list[i] = 0ull;
  __syncthreads();
  bitonic_desc(sh.list, (int)n2);
  for (uint32_t j = threadIdx.x; j < min(n, (uint32_t)k); j += kTopkThreads) {
    const uint32_t idx = ~(uint32_t)(sh.list[j] & 0xffffffffull);
    out.put(out0 + j, idx, c[idx]);
  }
}

// Bound by the chain of LDS passes of one workgroup per request (64 requests,
// 6144 gathered, k = 4096: 26 us with bins of 1/64 in a 64-unit window and
// scattered outputs, 15 us with bins of the gathered range and whole lines).
// Ranks n <= kGatherCap gathered candidates above -inf (thread t holds numbers
// t, t + 1024, ... in v) and emits the first min(n, k): a counting sort over
// equal steps of their range, then each candidate's place inside its bin from
// the bin's other members.  Where a bin is too full for that, those of the bins that
// hold the k best are sorted (130 beams x 46 tokens, one beam in ten live over dead
// ones at -1e4, which stretch the range and fill the last bin, k = 46: all of them
// sorted 83 us, these 21).
template <class Row>
__device__ __forceinline__ void rank_and_emit(TopkShared& sh, uint64_t (&v)[kGatherCap / kTopkThreads], uint32_t n,
                              int32_t k, int64_t out0, const Row& c, const TopkOut& out) {
  constexpr int kPer = kGatherCap / kTopkThreads;
  const int tid = threadIdx.x;
  float hi = -INFINITY, lo_neg = -INFINITY;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if ((uint32_t)(tid + j * kTopkThreads) < n) {
      const float x = key_score((uint32_t)(v[j] >> 32));
      hi = fmaxf(hi, x);
      lo_neg = fmaxf(lo_neg, -x);
    }
  clear_bins(sh.bin_count);
  if (tid == 0) sh.max_count = sh.n_list = 0u;
  // both maxima at once
  const float m2 = max_rows<2>({hi, lo_neg});
  if ((tid & 31) == 0) sh.fscan[tid >> 5] = m2;
  __syncthreads();
  {
    const float y = sh.fscan[tid & 31];   // waves' hi at even, lo_neg at odd places
    const bool odd = tid & 1;
    const float both = max_rows<2>({odd ? -INFINITY : y, odd ? y : -INFINITY});
    hi = lane_value(both, 0);
    lo_neg = lane_value(both, 32);
  }
  const float lo = -lo_neg;
  // an infinite range or a single value: one bin
  const float range = hi - lo;
  const float inv_w = range > 0.f && range < INFINITY ? (float)kHistBins / range : 0.f;
  uint32_t rb[kPer], slot[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if ((uint32_t)(tid + j * kTopkThreads) < n) {
      rb[j] = (uint32_t)(kHistBins - 1 -
                         step_bin(key_score((uint32_t)(v[j] >> 32)), lo, inv_w));
      slot[j] = atomicAdd(&sh.bin_count[rb[j]], 1u);
    }
  }
  __syncthreads();
  {
    uint32_t c4[4], s4 = 0, mx = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c4[e] = sh.bin_count[4 * tid + e];
      s4 += c4[e];
      mx = max(mx, c4[e]);
    }
    if (mx > 1) atomicMax(&sh.max_count, mx);
    uint32_t total;
    uint32_t run = block_exclusive_scan(s4, sh.scan, &total);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sh.bin_start[4 * tid + e] = run;
      run += c4[e];
    }
  }
  __syncthreads();
  const bool crowded = sh.max_count > kRankBinCap;
  // members of a bin that starts at or past k are not among the k best
  if (__builtin_expect(crowded, 0)) {
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if ((uint32_t)(tid + j * kTopkThreads) < n && sh.bin_start[rb[j]] < (uint32_t)k)
        sh.list[atomicAdd(&sh.n_list, 1u)] = v[j];
    __syncthreads();
    sort_and_emit(sh, sh.n_list, k, out0, c, out);   // all n, or k of them and more
    return;
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if ((uint32_t)(tid + j * kTopkThreads) < n && sh.bin_start[rb[j]] < (uint32_t)k)
      sh.list[sh.bin_start[rb[j]] + slot[j]] = v[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    slot[j] = 0xffffffffu;
    if ((uint32_t)(tid + j * kTopkThreads) >= n) continue;
    const uint32_t s0 = sh.bin_start[rb[j]], nb = sh.bin_count[rb[j]];
    if (s0 >= (uint32_t)k) continue;
    uint32_t pos = s0;
    for (uint32_t e = 0; e < nb; ++e) pos += sh.list[s0 + e] > v[j] ? 1u : 0u;
    slot[j] = pos;
  }
  // back to LDS in rank order, so that the outputs leave as whole lines
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (slot[j] < (uint32_t)k) sh.list[slot[j]] = v[j];
  __syncthreads();
  for (uint32_t j = tid; j < min(n, (uint32_t)k); j += kTopkThreads) {
    const uint32_t key = (uint32_t)(sh.list[j] >> 32), idx = ~(uint32_t)(sh.list[j] & 0xffffffffull);
    // the key is the score, but for -0, which has +0's key
    out.put(out0 + j, idx, key == 0x80000000u ? c[idx] : key_score(key));
  }
}

// Candidates i .. i+7 of a request (-inf past N; i a multiple of 8).
template <bool VEC8, class Row>
__device__ __forceinline__ void load_run(const Row& c, uint32_t i, uint32_t N, float (&x)[8]) {
  if constexpr (VEC8) {
    if (i < N) {   // N is a multiple of 8
      c.load8(i, x);
      return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = -INFINITY;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = i + e < N ? c[i + e] : -INFINITY;
  }
}

// Fills positions n .. k-1 with the candidates that are not above -inf: the
// -inf ones by index, then the NaN ones by index.
template <bool VEC8, class Row>
__device__ __forceinline__ void fill_dead(TopkShared& sh, uint32_t n, int32_t k, uint32_t N, int64_t out0,
                          const Row& c, const TopkOut& out) {
  for (int pass = 0; pass < 2 && n < (uint32_t)k; ++pass) {
    for (uint32_t i0 = 0; i0 < N && n < (uint32_t)k; i0 += 8 * kTopkThreads) {
      const uint32_t i = i0 + 8 * threadIdx.x;
      float x[8];
      load_run<VEC8>(c, i, N, x);
      uint32_t cnt = 0;
      bool hit[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        hit[e] = i + e < N && (pass == 0 ? x[e] == -INFINITY : x[e] != x[e]);
        cnt += hit[e] ? 1u : 0u;
      }
      uint32_t total;
      uint32_t pos = n + block_exclusive_scan(cnt, sh.scan, &total);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (hit[e]) {
          if (pos < (uint32_t)k) out.put(out0 + pos, i + e, x[e]);
          ++pos;
        }
      n += total;
    }
  }
}

// The digit (bin of sh.bin_count, complete) that holds the `want`-th best, counted
// from the highest digit down: ipar[0]; ipar[1] gets the counts of the higher
// digits, ipar[2] its own.  Ends with a barrier.
__device__ __forceinline__ void digit_of_rank(TopkShared& sh, uint32_t want) {
  // 4 digits per thread, thread 0 owns the highest
  uint32_t own[4], s4 = 0, total;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    own[j] = sh.bin_count[kHistBins - 1 - 4 * threadIdx.x - j];
    s4 += own[j];
  }
  const uint32_t before = block_exclusive_scan(s4, sh.scan, &total);
  if (before < want && before + s4 >= want) {
    uint32_t run = before;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (run < want && run + own[j] >= want) {
        sh.ipar[0] = kHistBins - 1 - 4 * (int)threadIdx.x - j;
        sh.ipar[1] = (int32_t)run;
        sh.ipar[2] = (int32_t)own[j];
      }
      run += own[j];
    }
  }
  __syncthreads();
}

// More gathered composites than the list holds (k < n <= entry.room): brings those
// down to the digit of 12 bits that holds the k-th, taken from the top until they
// fit, into sh.list and returns their number.  Composites differ, so at the
// latest the last digit does.  Bound by reading the entries, eight in flight per
// thread, once per digit (at most six; crowded scores need two or three).
template <class Entries>
__device__ __forceinline__ uint32_t narrow(TopkShared& sh, uint32_t n, int32_t k, const Entries& entry) {
  constexpr int U = 8;
  constexpr uint32_t kStep = U * kTopkThreads;
  const int tid = threadIdx.x;
  uint64_t prefix = 0;
  uint32_t above = 0, fit;
  int shift = 64;
  do {
    const int top = shift, bits = min(12, shift);
    shift -= bits;
    __syncthreads();
    clear_bins(sh.bin_count);
    if (tid == 0) sh.n_list = 0u;
    __syncthreads();
    for (uint32_t i0 = 0; i0 < n; i0 += kStep) {
      uint64_t v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = i0 + u * kTopkThreads + tid < n ? entry(i0 + u * kTopkThreads + tid) : 0ull;
#pragma unroll
      for (int u = 0; u < U; ++u)
        hist_add(sh.bin_count, (int)(v[u] >> shift) & ((1 << bits) - 1),
                 i0 + u * kTopkThreads + tid < n && (top == 64 || (v[u] >> top) == (prefix >> top)));
    }
    __syncthreads();
    digit_of_rank(sh, (uint32_t)k - above);
    prefix |= (uint64_t)(uint32_t)sh.ipar[0] << shift;
    above += (uint32_t)sh.ipar[1];
    fit = above + (uint32_t)sh.ipar[2];
  } while (fit > (uint32_t)kGatherCap);
  for (uint32_t i0 = 0; i0 < n; i0 += kStep) {
    uint64_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i0 + u * kTopkThreads + tid < n ? entry(i0 + u * kTopkThreads + tid) : 0ull;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * kTopkThreads + tid < n && v[u] >= prefix) sh.list[atomicAdd(&sh.n_list, 1u)] = v[u];
  }
  __syncthreads();
  return fit;
}

// sh.list[0, n), n <= kGatherCap, into registers, number t + 1024 j to thread t.
__device__ __forceinline__ void take_list(const TopkShared& sh, uint32_t n,
                                          uint64_t (&v)[kGatherCap / kTopkThreads]) {
#pragma unroll
  for (int j = 0; j < kGatherCap / kTopkThreads; ++j) {
    const uint32_t i = (uint32_t)(threadIdx.x + j * kTopkThreads);
    v[j] = i < n ? sh.list[i] : 0ull;
  }
  __syncthreads();
}

// Exact selection of any request: a radix select on the key (digits of 12, 12
// and 8 bits) over all the candidates, an index-ordered collection of the ties with
// the k-th, and a bitonic sort.  Eight candidates per thread and step.
template <bool VEC8, class Row>
__device__ __forceinline__ void exact_select(TopkShared& sh, int32_t k, uint32_t N, int64_t out0, const Row& c,
                             const TopkOut& out) {
  const int tid = threadIdx.x;
  uint32_t* hist = sh.bin_count;
  constexpr uint32_t kStep = 8 * kTopkThreads;
  uint32_t prefix = 0, remaining = (uint32_t)k;
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 20 : (pass == 1 ? 8 : 0), bits = pass == 2 ? 8 : 12;
    const uint32_t pmask = pass == 0 ? 0u : 0xffffffffu << (shift + bits);
    __syncthreads();
    clear_bins(hist);
    __syncthreads();
    for (uint32_t i0 = 0; i0 < N; i0 += kStep) {
      const uint32_t i = i0 + 8 * tid;
      float x[8];
      load_run<VEC8>(c, i, N, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t key = order_key(x[e]);
        hist_add(hist, (int)((key >> shift) & ((1u << bits) - 1u)), i + e < N && (key & pmask) == prefix);
      }
    }
    __syncthreads();
    digit_of_rank(sh, remaining);
    prefix |= (uint32_t)sh.ipar[0] << shift;
    remaining -= (uint32_t)sh.ipar[1];
  }
  __syncthreads();
  // prefix is the k-th key T; `remaining` candidates equal to T are taken,
  // lowest index first, after the k - remaining candidates above T.
  const uint32_t T = prefix, need = remaining, gt_total = (uint32_t)k - remaining;
  uint32_t gt_base = 0, eq_base = 0;
  for (uint32_t i0 = 0; i0 < N && (gt_base < gt_total || eq_base < need); i0 += kStep) {
    const uint32_t i = i0 + 8 * tid;
    float x[8];
    load_run<VEC8>(c, i, N, x);
    uint32_t keys[8], ngt = 0, neq = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = i + e < N;
      keys[e] = order_key(x[e]);
      ngt += in && keys[e] > T;
      neq += in && keys[e] == T;
    }
    // at most 8192 of either in a step: two 16-bit counts in one scan
    uint32_t total;
    const uint32_t pre = block_exclusive_scan((neq << 16) | ngt, sh.scan, &total);
    uint32_t pg = gt_base + (pre & 0xffffu), pe = eq_base + (pre >> 16);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (i + e >= N) continue;
      if (keys[e] > T) {
        sh.list[pg++] = composite(keys[e], i + e);
      } else if (keys[e] == T) {
        if (pe < need) sh.list[gt_total + pe] = composite(keys[e], i + e);
        ++pe;
      }
    }
    gt_base += total & 0xffffu;
    eq_base += total >> 16;
  }
  __syncthreads();
  sort_and_emit(sh, (uint32_t)k, k, out0, c, out);
}

// ---- N <= kSmallN: one workgroup per request ----
// Bound by latency: one read of the candidates (from L2: at most 128 KiB of
// bf16 logits), then a chain of LDS passes.  RUNS runs of 8 per thread.
template <class Src, bool VEC8, int RUNS>
__global__ void __launch_bounds__(kTopkThreads)
topk_small_kernel(Src src, uint32_t N, int32_t k, TopkOut out) {
  __shared__ TopkShared sh;
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.x, out0 = b * k;
  const auto c = src.request(b, N);
  float x[RUNS][8];
#pragma unroll
  for (int j = 0; j < RUNS; ++j) load_run<VEC8>(c, (uint32_t)(j * kTopkThreads + tid) * 8, N, x[j]);
  float thr = -FLT_MAX;
  bool exact = false;
  if (tid == 0) sh.n_list = 0u;
  if (N > (uint32_t)kGatherCap) {
    clear_bins(sh.bin_count);
    float mx = -INFINITY;
    uint32_t live = 0;
#pragma unroll
    for (int j = 0; j < RUNS; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        mx = fmaxf(mx, x[j][e]);
        live += x[j][e] > -INFINITY ? 1u : 0u;
      }
    const float best = block_max(mx, sh.fscan);
    uint32_t n_live;
    block_exclusive_scan(live, sh.scan, &n_live);
    // fewer than k above -inf: all of them are gathered (k <= kGatherCap)
    if (n_live >= (uint32_t)k) {
      const float lo = best - kWindow, inv_w = (float)kHistBins / kWindow;
      // the k-th best of the threads' own best is at or below the k-th best of
      // all (if there are k threads): only what is above enters the histogram
      int first = 1;
      const int own = step_bin(mx, lo, inv_w);
      if (k <= kTopkThreads) {
        if (own > 0) atomicAdd(&sh.bin_count[own], 1u);
        __syncthreads();
        first = max(1, boundary_bin(sh.bin_count, (uint32_t)k, sh.scan, sh.ipar));
        clear_bins(sh.bin_count);
        __syncthreads();
      }
      if (own >= first) {
#pragma unroll
        for (int j = 0; j < RUNS; ++j)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int bin = step_bin(x[j][e], lo, inv_w);
            if (bin >= first) atomicAdd(&sh.bin_count[bin], 1u);
          }
      }
      __syncthreads();
      const int bin = boundary_bin(sh.bin_count, (uint32_t)k, sh.scan, sh.ipar);
      exact = bin == 0 || !(best < INFINITY);   // also NaN
      // the lowest score of the bin and above, to the exact bin
      if (!exact) {
        float low_neg = -INFINITY;
#pragma unroll
        for (int j = 0; j < RUNS; ++j)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (step_bin(x[j][e], lo, inv_w) >= bin) low_neg = fmaxf(low_neg, -x[j][e]);
        thr = -block_max(low_neg, sh.fscan);
      }
    }
  }
  __syncthreads();
  if (!exact) {
#pragma unroll
    for (int j = 0; j < RUNS; ++j)
      for_hits<8>(x[j], (uint32_t)(j * kTopkThreads + tid) * 8, thr,
                  PutList{sh.list, &sh.n_list, (uint32_t)kGatherCap});
    __syncthreads();
    const uint32_t n = sh.n_list;
    if (n <= (uint32_t)kGatherCap) {
      uint64_t v[kGatherCap / kTopkThreads];
      take_list(sh, n, v);
      rank_and_emit(sh, v, n, k, out0, c, out);
      if (n < (uint32_t)k) fill_dead<VEC8>(sh, n, k, N, out0, c, out);
      return;
    }
    __syncthreads();
  }
  exact_select<VEC8>(sh, k, N, out0, c, out);
}

// ---- more candidates: select, gather, final ----

// Threshold of each request: the score above which about `want` samples lie, by
// a histogram of the differences from ref in [-kBelow, kAbove).  A workgroup
// takes kSelectSamples samples (one CU reads from beyond its L2 at some 20 GB/s,
// so a sample of 256 KiB takes 27 us on one CU and 8 us on eight); the last one
// of a request to finish sums the workgroups' histograms.  The want-th best of
// the threads' own best samples bounds the threshold from below, so that only
// the few samples above that are counted.  A request with fewer than `want`
// samples in the window gathers everything above -inf, if that can fit.
constexpr float kBelow = 112.0f, kAbove = 16.0f;
constexpr uint32_t kSelectSamples = 16384;

constexpr float kSelectInvW = (float)kHistBins / (kBelow + kAbove);
// Bin of a sample.  A sample v below 0 was rounded up, from (v - q, v], q its fp16
// step; bins that take their upper edge in and not their lower one hold that whole
// range above the edge below, as edges are fp16 values from -64 up.
constexpr float kEdge = 0x1p-14f;
__device__ __forceinline__ int sample_bin(float x) { return step_bin(x, kEdge - kBelow, kSelectInvW); }
__device__ __forceinline__ bool in_top_bin(float x) { return sample_bin(x) == kHistBins - 1; }

// Samples of a request, four at a time as packed fp16 differences from ref(b):
// as the score pass stored them, or one 32-candidate chunk of every 2^lp
// consecutive ones (picked by a hash of the group index, so that neither a
// row's token order nor the row length biases it), read from the candidates.
// scores4: the scores of samples j .. j+3, -inf past the last, for samples that lie
// so far above ref(b) that they meet in the top bin; the stored ones' may be those
// of a neighbour, and are -inf below that bin (their scattered reads of the logits
// are what such a pass costs).
template <class Src>
struct StoredSample {
  Src src;
  const uint16_t* p;
  int64_t stride;
  uint32_t n;
  int32_t lp;
  FastDiv per_row;   // sample -> beam
  struct Row {
    typename Src::Row c;
    const u32x2* p;
    uint32_t n, samples_per_row;
    int32_t lp;
    FastDiv per_row;
    __device__ __forceinline__ float at(uint32_t j) const {
      if (j >= n) return -INFINITY;
      const uint32_t m = per_row.div(j), v = ((j - m * samples_per_row) << lp) + sample_offset(m, lp);
      return v < (uint32_t)c.V ? c[m * (uint32_t)c.V + v] : -INFINITY;
    }
    __device__ __forceinline__ void scores4(uint32_t j, float (&x)[4]) const {
      const u32x2 w = load4(j, 0.f);
      const f16x2 lo = __builtin_bit_cast(f16x2, w.x), hi = __builtin_bit_cast(f16x2, w.y);
      const bool top[4] = {in_top_bin((float)lo.x), in_top_bin((float)lo.y), in_top_bin((float)hi.x),
                           in_top_bin((float)hi.y)};
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = top[e] ? at(j + e) : -INFINITY;
    }
    // the score pass put -inf behind the last sample, up to a whole four
    __device__ __forceinline__ u32x2 load4(uint32_t j, float) const {
      const u32x2 w = p[min(j, n - 1) >> 2];
      return j < n ? w : u32x2{0xfc00fc00u, 0xfc00fc00u};   // -inf
    }
  };
  __device__ __forceinline__ Row request(int64_t b, uint32_t N) const {
    return Row{src.request(b, N), (const u32x2*)(p + b * stride), n, ((uint32_t)src.V + (1u << lp) - 1) >> lp,
               lp, per_row};
  }
  __device__ __forceinline__ float ref(const Row&, int64_t b, float*) const {
    return sample_ref(src.prev + b * src.M, src.M);
  }
};
template <class Src>
struct ChunkSample {
  Src src;
  int32_t lp;
  uint32_t n;   // a multiple of 32
  struct Row {
    typename Src::Row c;
    int32_t lp;
    uint32_t n, N;
    // flat index of sample j (past 2^32: past any candidate)
    __device__ __forceinline__ uint64_t index(uint32_t j) const {
      const uint32_t g = j >> 5, chunk = (g << lp) + ((g * 0x9E3779B1u) >> (32 - lp));
      return 32ull * chunk + (j & 31);
    }
    __device__ __forceinline__ float at(uint32_t j) const {
      const uint64_t i = index(j);
      return j < n && i < N ? c.nt((uint32_t)i) : -INFINITY;
    }
    __device__ __forceinline__ void scores4(uint32_t j, float (&x)[4]) const {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = at(j + e);
    }
    __device__ __forceinline__ u32x2 load4(uint32_t j, float ref) const {
      const uint64_t i = index(j);   // j a multiple of 4: one chunk
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = j < n && i + e < N ? c.nt((uint32_t)i + e) - ref : -INFINITY;
      return u32x2{pack_f16x2(x[0], x[1]), pack_f16x2(x[2], x[3])};
    }
  };
  __device__ __forceinline__ Row request(int64_t b, uint32_t N) const {
    return Row{src.request(b, N), lp, n, N};
  }
  // the best of 8 samples each from 128 chunks all over the request, 0 if none is
  // finite
  __device__ __forceinline__ float ref(const Row& row, int64_t, float* scratch) const {
    const uint32_t chunk = (uint32_t)((uint64_t)(threadIdx.x >> 3) * (n >> 5) / 128);
    const float x = row.at(32 * chunk + (threadIdx.x & 7));
    const float m = block_max(fabsf(x) < INFINITY ? x : -INFINITY, scratch);
    return m > -INFINITY ? m : 0.f;
  }
};

// Samples j0 .. j0 + kSelectSamples - 1 (-inf past the last), kSampleLoads loads of
// four per thread.
constexpr int kSampleLoads = kSelectSamples / (4 * kTopkThreads);
template <class Row>
__device__ __forceinline__ void load_samples(const Row& sample, uint32_t j0, float ref,
                                             float (&x)[kSampleLoads][4]) {
  u32x2 w[kSampleLoads];
#pragma unroll
  for (int u = 0; u < kSampleLoads; ++u) w[u] = sample.load4(j0 + 4 * (u * kTopkThreads + threadIdx.x), ref);
#pragma unroll
  for (int u = 0; u < kSampleLoads; ++u) {
    const f16x2 lo = __builtin_bit_cast(f16x2, w[u].x), hi = __builtin_bit_cast(f16x2, w[u].y);
    x[u][0] = (float)lo.x;
    x[u][1] = (float)lo.y;
    x[u][2] = (float)hi.x;
    x[u][3] = (float)hi.y;
  }
}

// hist: the counts of samples j0 .. j0 + kSelectSamples - 1 in the bins from the
// want-th best of the threads' own best samples up; where those are all the
// window's, bin 0 counts the finite samples below it.
template <class Row>
__device__ __forceinline__ void sample_hist(const Row& sample, uint32_t j0, float ref, uint32_t want,
                                            uint32_t* hist, uint32_t* scan, int32_t* ipar) {
  constexpr int U = kSampleLoads;
  const int tid = threadIdx.x;
  float x[U][4];
  load_samples(sample, j0, ref, x);
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) mx = fmaxf(mx, x[u][e]);
  clear_bins(hist);
  __syncthreads();
  const int own = sample_bin(mx);
  if (own > 0) atomicAdd(&hist[own], 1u);
  __syncthreads();
  const int first = max(1, boundary_bin(hist, want, scan, ipar));   // 1: the whole window
  clear_bins(hist);
  __syncthreads();
  if (own >= first) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int bin = sample_bin(x[u][e]);
        if (bin >= first) atomicAdd(&hist[bin], 1u);
      }
  }
  if (first == 1) {
    uint32_t low = 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        low += x[u][e] > -INFINITY && sample_bin(x[u][e]) == 0 ? 1u : 0u;
    low = wave_scan(low);
    if ((tid & 63) == 63 && low != 0u) atomicAdd(&hist[0], low);
  }
  __syncthreads();
}
// Calls f(difference from ref) for all of a request's samples, a whole wave at a
// time: in fp16, or (SCORES) of their scores in fp32.
template <bool SCORES, class Row, class F>
__device__ __forceinline__ void for_samples(const Row& sample, float ref, const F& f) {
  if constexpr (SCORES) {
    const uint32_t own = 4 * threadIdx.x;
#pragma unroll 1
    for (uint32_t j0 = 0; j0 < sample.n; j0 += 4 * kTopkThreads) {
      float x[4];
      sample.scores4(j0 + own, x);
#pragma unroll 1
      for (int e = 0; e < 4; ++e) f((e == 0 ? x[0] : e == 1 ? x[1] : e == 2 ? x[2] : x[3]) - ref);
    }
  } else {
    for (uint32_t j0 = 0; j0 < sample.n; j0 += kSelectSamples) {
      float x[kSampleLoads][4];
      load_samples(sample, j0, ref, x);
#pragma unroll
      for (int u = 0; u < kSampleLoads; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) f(x[u][e]);
    }
  }
}

// The threshold of a request whose samples, one of 2^lp, hist counts (complete):
// the lower edge of the bin with the `want`-th best.  Where that bin is so crowded
// that what is expected at or above it comes near the room for gathered candidates,
// it is cut in 4096 by reading all the samples again; a smaller crowd costs less to
// gather and narrow (64 x 4096 x 512, k = 4096: the cut 13-47 us, 15000 candidates
// past the list 10).  Where even one value's crowd would not fit, what is above it
// may still be k: 5000 allowed tokens over a floor of equal scores.  That shape with
// equal prefixes and N(0, s^2) logits, against the exact selection by one workgroup
// for everything past the list: s = 0.3 3189 and 139 us, 0.1 2075 and 149, 0.02 2211
// and 155; 5000 tokens over a floor 2222 and 270.
// Scores far above ref (a few live beams, that ref's few prefixes missed, over dead
// ones at -1e9) meet in the top bin's last cut, and the slack of so large a ref may
// reach below all the bins: the differences are then taken anew, from the best
// sample, for the samples of the top bin, which are enough.  16 x 1000 x 509 fp32, k = 1024, one beam in 20 live: 1218 us by the exact
// selection, 49 so; two calls at 4 x 4096 x 4096, k = 4096: 13679 and 185.
template <class Row>
__device__ __forceinline__ float threshold(const Row& sample, uint32_t* hist, uint32_t want, int32_t lp,
                                           float ref, uint32_t room, uint32_t* scan, float* fscan,
                                           int32_t* ipar) {
  constexpr int kTop = kHistBins - 1;
  for (bool anew = false;; anew = true) {
    const int bin = boundary_bin(hist, want, scan, ipar);
    uint32_t above = (uint32_t)ipar[1];
    const bool crowded = ((uint64_t)(above + (uint32_t)ipar[2]) << lp) > min(room / 4 * 3, 3u * kGatherCap);
    float edge = (float)bin / kSelectInvW - kBelow;
    const float slack = fabsf(ref) * 0x1p-22f;   // the rounding of the differences
    bool far = !anew && bin == kTop && slack > 1.0f;
    if (__builtin_expect(!crowded && !far, 1))   // below -64 an fp16 step is wider than a bin
      return bin == 0 ? -FLT_MAX : ref + (edge < -64.f ? edge - 1.0f / kSelectInvW : edge) - slack;
    if (!far) {
      // the outer bins, open below and above, in as many steps of a bin's width
      const float inv_w = bin == 0 || bin == kTop ? kSelectInvW : kSelectInvW * (float)kHistBins;
      if (bin == 0) edge -= kBelow + kAbove;
      __syncthreads();
      clear_bins(hist);
      __syncthreads();
      const auto cut = [&](float x) __attribute__((always_inline)) {
        hist_add(hist, step_bin(x, edge, inv_w), x > -INFINITY && sample_bin(x) == bin);
      };
      if (anew) for_samples<true>(sample, ref, cut);
      else for_samples<false>(sample, ref, cut);
      __syncthreads();
      const int part = boundary_bin(hist, want - above, scan, ipar);
      far = !anew && bin == kTop && part == kTop;
      if (!far) {
        above += (uint32_t)ipar[1];
        const bool fits = ((uint64_t)(above + (uint32_t)ipar[2]) << lp) <= room || above == 0u;
        if (fits && bin == 0 && part == 0) return -FLT_MAX;
        // a sample v < 0 stands for (v - q, v], one of 0 and above for [v, v + q)
        edge += (float)part / inv_w;
        const float q = fmaxf(__uint_as_float(__float_as_uint(edge) & 0x7f800000u) * 0x1p-10f, 0x1p-24f);
        return fits ? ref + edge - (edge < 0.f ? q : 0.f) - slack
                    : ref + edge + 1.0f / inv_w + (edge < 0.f ? 0.f : q) + slack;
      }
    }
    float best = -INFINITY;
    for_samples<true>(sample, 0.f, [&](float x) __attribute__((always_inline)) {
      best = fmaxf(best, fabsf(x) < INFINITY ? x : -INFINITY);
    });
    best = block_max(best, fscan);
    if (!(best > -INFINITY)) return -FLT_MAX;
    ref = best;
    clear_bins(hist);
    __syncthreads();
    for_samples<true>(sample, ref, [&](float x) __attribute__((always_inline)) {
      hist_add(hist, sample_bin(x), x > -INFINITY);
    });
    __syncthreads();
  }
}

// Two workgroups per CU.
template <class Smp>
__global__ void __launch_bounds__(kTopkThreads, 8)
topk_select_kernel(Smp smp, uint32_t N, uint32_t want, int32_t lp, TopkWs ws) {
  __shared__ uint32_t hist[kHistBins];
  __shared__ uint32_t scan[64];
  __shared__ float fscan[kTopkThreads / 64];
  __shared__ int32_t ipar[4];
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.y;
  const auto sample = smp.request(b, N);
  const float ref = smp.ref(sample, b, fscan);
  sample_hist(sample, blockIdx.x * kSelectSamples, ref, want, hist, scan, ipar);
  int32_t* info = ws.info + b * kInfo;
  if (gridDim.x > 1) {
    // every workgroup's bins from the request's threshold up are complete, as
    // its `first` is at or below the threshold
    uint32_t* sum = ws.hist(b);
    for (int i = tid; i < kHistBins; i += kTopkThreads)
      if (hist[i] != 0u)
        (void)__hip_atomic_fetch_add(&sum[i], hist[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    publish_shared();
    if (tid == 0) ipar[0] = last_to_finish(&info[3], (int32_t)gridDim.x);
    __syncthreads();
    if (ipar[0] == 0) return;   // whole workgroup
    for (int i = tid; i < kHistBins; i += kTopkThreads) hist[i] = load_shared(&sum[i]);
    __syncthreads();
  }
  const float thr = threshold(sample, hist, want, lp, ref, ws.gather_room(), scan, fscan, ipar);
  if (tid == 0) {
    info[0] = __float_as_int(thr);
    info[1] = 0;   // gathered count
  }
}

__global__ void __launch_bounds__(kTopkThreads) topk_clear_kernel(TopkWs ws) {
  clear_shared(ws, blockIdx.x, threadIdx.x, kTopkThreads);
}

constexpr int kGatherThreads = 256;
constexpr int kStage = 1024;   // LDS entries of a gather workgroup

// A request's gathered composites: kGatherCap in the list, the rest behind the
// sample.  SHARED: other workgroups of this launch read them.
template <bool SHARED>
struct Gathered {
  uint64_t *list, *more;   // more: where number 0 would lie, if it were there
  uint32_t* count;
  uint32_t room;
  __device__ __forceinline__ Gathered(const TopkWs& ws, int64_t b)
      : list(ws.list + b * (int64_t)kGatherCap),
        more((uint64_t*)(ws.sample + b * ws.sample_stride() + ws.spill) - kGatherCap),
        count((uint32_t*)&ws.info[b * kInfo + 1]), room(ws.gather_room()) {}
  __device__ __forceinline__ uint64_t* at(uint32_t i) const {
    return (i < (uint32_t)kGatherCap ? list : more) + i;
  }
  __device__ __forceinline__ static void store(uint64_t* p, uint64_t v) {
    if constexpr (SHARED)
      (void)__hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      *p = v;
  }
  __device__ __forceinline__ void put(uint32_t i, uint64_t v) const {
    if (i < room) store(at(i), v);
  }
  __device__ __forceinline__ static uint64_t load(const uint64_t* p) {
    if constexpr (SHARED) return load_shared(p);
    else return *p;
  }
  __device__ __forceinline__ uint64_t operator()(uint32_t i) const { return load(at(i)); }
  __device__ __forceinline__ uint64_t in_list(uint32_t i) const { return load(list + i); }   // i < kGatherCap
};

// A workgroup's staged candidates: flushed with one global atomic (same-address
// global atomics serialise); what does not fit the stage goes to the list directly.
template <int STAGE>
struct GatherStage {
  uint64_t entry[STAGE];
  uint32_t n, base;
};
template <int STAGE, bool SHARED>
struct PutStage {
  GatherStage<STAGE>& st;
  const Gathered<SHARED>& to;
  uint32_t pos = 0, direct = 0;
  __device__ __forceinline__ void reserve(uint32_t n) {
    pos = atomicAdd(&st.n, n);
    const uint32_t first = max(pos, (uint32_t)STAGE);
    if (__builtin_expect(pos + n > first, 0)) direct = atomicAdd(to.count, pos + n - first);
  }
  __device__ __forceinline__ void operator()(uint64_t v) {
    if (__builtin_expect(pos < (uint32_t)STAGE, 1)) {
      st.entry[pos] = v;
    } else {
      to.put(direct++, v);
    }
    ++pos;
  }
};
template <int THREADS, bool SHARED, int STAGE>
__device__ __forceinline__ void gather_flush(GatherStage<STAGE>& st, const Gathered<SHARED>& to) {
  __syncthreads();
  const uint32_t n = min(st.n, (uint32_t)STAGE);
  if (n == 0) return;   // whole workgroup
  if (threadIdx.x == 0) st.base = atomicAdd(to.count, n);
  __syncthreads();
  const uint32_t b0 = st.base;
  if (__builtin_expect(b0 + n <= (uint32_t)kGatherCap, 1)) {
    for (uint32_t j = threadIdx.x; j < n; j += THREADS) to.store(to.list + b0 + j, st.entry[j]);
  } else {
    for (uint32_t j = threadIdx.x; j < n; j += THREADS) to.put(b0 + j, st.entry[j]);
  }
}

// Gather over a written candidate array (16 x 1000 x 509 fp32, 33 MB: 31 -> 12
// us, the former form had a barrier per step and 256 workgroups): workgroup s of request b takes
// candidates [s * per, (s + 1) * per), per a multiple of 1024.  Bound by the
// read of the array: VEC (16-byte aligned requests, N a multiple of 8) four
// candidates per load, four loads in flight; else eight single ones.
template <bool VEC>
__global__ void __launch_bounds__(kGatherThreads)
topk_gather_array_kernel(CandArray src, uint32_t N, uint32_t per, TopkWs ws) {
  __shared__ GatherStage<kStage> st;
  const int64_t b = blockIdx.y;
  const float thr = __int_as_float(ws.info[b * kInfo]);
  const auto c = src.request(b, N);
  const Gathered<false> to(ws, b);
  if (threadIdx.x == 0) st.n = 0u;
  __syncthreads();
  const uint64_t i0 = (uint64_t)blockIdx.x * per;
  const uint64_t i1 = min((uint64_t)N, i0 + per);
  if constexpr (VEC) {
    for (uint64_t j0 = i0; j0 < i1; j0 += 16 * kGatherThreads) {
      float x[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t i = j0 + 4 * (u * kGatherThreads + threadIdx.x);
        u32x4 q = {0xff800000u, 0xff800000u, 0xff800000u, 0xff800000u};
        if (i < i1) q = __builtin_nontemporal_load((const u32x4*)(c.p + i));   // N is a multiple of 4
        Chunk<F32>::unpack(q, x[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        for_hits<4>(x[u], (uint32_t)(j0 + 4 * (u * kGatherThreads + threadIdx.x)), thr,
                    PutStage<kStage, false>{st, to});
    }
  } else {
    for (uint64_t j0 = i0; j0 < i1; j0 += 8 * kGatherThreads) {
      float x[8][1];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint64_t i = j0 + u * kGatherThreads + threadIdx.x;
        x[u][0] = i < i1 ? c.nt((uint32_t)i) : -INFINITY;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        for_hits<1>(x[u], (uint32_t)(j0 + u * kGatherThreads + threadIdx.x), thr,
                    PutStage<kStage, false>{st, to});
    }
  }
  gather_flush<kGatherThreads>(st, to);
}

// Gather over candidates recomputed from the logits.  A wave takes up to 64
// rows and reads only those whose upper bound reaches the threshold: at 64
// requests x 4096 beams x 512 tokens 31 % of the rows hold all of the 6144 best
// candidates.  2^ll lanes per row (RUN: runs of 8 tokens per lane, else single
// tokens), 4 row pieces in flight.  Few lanes hold a candidate: the lanes whose
// best logit, filtered or not, reaches the threshold queue their run, and the
// workgroup then takes the queued runs apart with all lanes busy (64 x 4096 x
// 512: reading every row 136 us, these rows 51, with the queue 27).
constexpr int kQueue = 2048;

// rows: 64 bytes of LDS of the wave's own; m0, bound: the wave's first row, the
// lane's row's upper bound.  Ends without a barrier, st ready to be flushed.
template <bool RUN, int THREADS, int QUEUE, bool SHARED, int STAGE, class Row>
__device__ __forceinline__ void gather_rows(const Row& c, int64_t m0, float bound, float thr, int32_t ll,
                                            GatherStage<STAGE>& st, uint32_t* queue, uint32_t& n_queue,
                                            uint8_t* rows, const Gathered<SHARED>& to) {
  constexpr int E = RUN ? 8 : 1, U = 4;
  const int lane = threadIdx.x & 63;
  if (threadIdx.x == 0) st.n = n_queue = 0u;
  const uint64_t act = __ballot(bound >= thr);
  if (bound >= thr) rows[__popcll(act & ((1ull << lane) - 1ull))] = (uint8_t)lane;
  __syncthreads();
  const int n_act = (int)__popcll(act);
  const int32_t V = c.V;
  const int lpr = 1 << ll, rpp = 64 >> ll;             // lanes per row, rows per piece
  const int sub = lane >> ll, sl = lane & (lpr - 1);
  int idx0 = 0, v0 = 0;   // the next piece: first row (index into rows), first token
  while (idx0 < n_act) {
    typename Row::template Raw<E> raw[U];
    uint32_t at[U], m[U];
    bool live[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = idx0 + sub, v = v0 + sl * E;
      live[u] = idx < n_act && v < V;
      if (live[u]) {
        m[u] = (uint32_t)m0 + rows[idx];
        at[u] = m[u] * (uint32_t)V + (uint32_t)v;
        c.template load_raw<E>(at[u], m[u], raw[u]);
      }
      v0 += lpr * E;
      if (v0 >= V) {
        v0 = 0;
        idx0 += rpp;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!live[u]) continue;
      float f[E];
      raw[u].logits(f);
      float top = f[0];
      if constexpr (E > 1) {
        top = max3(top, f[1], f[2]);
        top = max3(top, f[3], f[4]);
        top = max3(top, f[5], f[6]);
        top = max3(top, f[7], f[7]);
      }
      if (!(raw[u].p + (top - raw[u].l) >= thr)) continue;
      if constexpr (RUN) {
        const uint32_t pos = atomicAdd(&n_queue, 1u);
        if (pos < (uint32_t)QUEUE) {
          queue[pos] = at[u];
          continue;
        }
      }
      float x[E];
      c.template finish<E>(at[u], m[u], raw[u], x);
      for_hits<E>(x, at[u], thr, PutStage<STAGE, SHARED>{st, to});
    }
  }
  if constexpr (RUN) {
    __syncthreads();
    const uint32_t n = min(n_queue, (uint32_t)QUEUE);
    for (uint32_t j = threadIdx.x; j < n; j += THREADS) {
      float x[8];
      c.load8(queue[j], x);
      for_hits<8>(x, queue[j], thr, PutStage<STAGE, SHARED>{st, to});
    }
  }
}

template <class T, bool RUN>
__global__ void __launch_bounds__(kGatherThreads)
topk_gather_rows_kernel(CandFromLogits<T> src, const float* __restrict__ row_max, int32_t rows_per_wave,
                        int32_t ll, uint32_t N, TopkWs ws) {
  constexpr int kWaves = kGatherThreads / 64;
  __shared__ GatherStage<kStage> st;
  __shared__ uint32_t queue[RUN ? kQueue : 1];
  __shared__ uint32_t n_queue;
  __shared__ uint8_t rows[kWaves][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = blockIdx.y;
  const int64_t m0 = ((int64_t)blockIdx.x * kWaves + wave) * rows_per_wave;
  const float bound = lane < rows_per_wave && m0 + lane < src.M ? row_max[b * src.M + m0 + lane] : -INFINITY;
  const float thr = __int_as_float(ws.info[b * kInfo]);
  const Gathered<false> to(ws, b);
  gather_rows<RUN, kGatherThreads, kQueue, false>(src.request(b, N), m0, bound, thr, ll, st, queue, n_queue,
                                                  rows[wave], to);
  gather_flush<kGatherThreads>(st, to);
}

// Final selection from the n gathered candidates at or above thr, or the exact
// selection over all the request's candidates; *how says which it was.
template <bool VEC8, class Row, class Entries>
__device__ __forceinline__ void final_select(TopkShared& sh, float thr, uint32_t n, uint32_t N, int32_t k,
                                             int64_t out0, const Row& c, const TopkOut& out,
                                             const Entries& entry, int32_t* how) {
  constexpr int kPer = kGatherCap / kTopkThreads;
  // all candidates at or above thr are gathered; the k best are among them when
  // they are at least k, or when they are all there are above -inf
  const bool enough = n >= (uint32_t)k || thr == -FLT_MAX;
  const int32_t way = !enough || n > entry.room ? kExact : (n > (uint32_t)kGatherCap ? kNarrowed : kRanked);
  if (threadIdx.x == 0) *how = way;
  if (__builtin_expect(way == kExact, 0)) {
    exact_select<VEC8>(sh, k, N, out0, c, out);
    return;
  }
  uint64_t v[kPer];
  if (__builtin_expect(way == kRanked, 1)) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t i = (uint32_t)(threadIdx.x + j * kTopkThreads);
      v[j] = i < n ? entry.in_list(i) : 0ull;
    }
  } else {
    n = narrow(sh, n, k, entry);
    take_list(sh, n, v);
  }
  rank_and_emit(sh, v, n, k, out0, c, out);
  if (n < (uint32_t)k) fill_dead<VEC8>(sh, n, k, N, out0, c, out);
}

template <class Src, bool VEC8>
__global__ void __launch_bounds__(kTopkThreads)
topk_final_kernel(Src src, uint32_t N, int32_t k, TopkWs ws, TopkOut out) {
  __shared__ TopkShared sh;
  const int64_t b = blockIdx.x;
  int32_t* info = ws.info + b * kInfo;
  final_select<VEC8>(sh, __int_as_float(info[0]), (uint32_t)info[1], N, k, b * k, src.request(b, N), out,
                     Gathered<false>(ws, b), &info[2]);
}

// Select, gather and final in one launch, for few rows: bound by the latency of
// each stage's chain and by the launches between them.  Every workgroup derives the
// threshold from the whole sample (at most kSelectSamples, 32 KiB), gathers its
// rows, one per wave, and the last of a request to finish ranks the list.  12 x 300
// x 500 tokens, k = 1000: score pass and selection 33.7 us with three launches of
// the selection, 26.2 with one; 8 x 512 x 1024, k = 1024: 30.7 and 26.0; 1 x 300 x 509,
// k = 100: 23.3 and 22.6; 1 x 16 x 20000, k = 50: 110 and 95.
// Only where the workgroups (one fits a CU, by its LDS) all run at once: with two
// rows per wave 16 x 1000 x 509, k = 1000 took 39.5 against 37.5.  And up to 32 of
// them per request, which all read its sample: 1 x 1024 x 512 25.9 against 25.6, 2 x
// 2048 x 512 26.7 against 26.6.
constexpr int kFusedStage = 4096, kFusedQueue = 4096;
constexpr uint32_t kFusedRows = kTopkThreads / 64;     // beam rows per workgroup, one per wave
constexpr uint32_t kFusedMaxPerRequest = 32, kFusedMaxBlocks = 256;

template <class T, bool RUN>
__global__ void __launch_bounds__(kTopkThreads)
topk_fused_rows_kernel(StoredSample<CandFromLogits<T>> smp, const float* __restrict__ row_max,
                       int32_t ll, uint32_t N, uint32_t want, int32_t lp, int32_t k, TopkWs ws, TopkOut out) {
  constexpr int kWaves = kTopkThreads / 64;
  __shared__ TopkShared sh;
  __shared__ uint32_t n_queue;
  __shared__ uint8_t rows[kWaves][64];
  typedef GatherStage<kFusedStage> Stage;
  static_assert(sizeof(Stage) + kFusedQueue * sizeof(uint32_t) <= sizeof(sh.list), "in the ranking's list");
  const CandFromLogits<T>& src = smp.src;
  Stage& st = *(Stage*)sh.list;
  uint32_t* const queue = (uint32_t*)((char*)sh.list + sizeof(Stage));
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = blockIdx.y;
  const int64_t m0 = (int64_t)blockIdx.x * kWaves + wave;
  const float bound = lane == 0 && m0 < src.M ? row_max[b * src.M + m0] : -INFINITY;
  const auto sample = smp.request(b, N);
  const float ref = smp.ref(sample, b, nullptr);
  sample_hist(sample, 0, ref, want, sh.bin_count, sh.scan, sh.ipar);
  const float thr = threshold(sample, sh.bin_count, want, lp, ref, ws.gather_room(), sh.scan, sh.fscan, sh.ipar);
  const Gathered<true> to(ws, b);
  const auto c = src.request(b, N);
  gather_rows<RUN, kTopkThreads, kFusedQueue, true>(c, m0, bound, thr, ll, st, queue, n_queue, rows[wave], to);
  gather_flush<kTopkThreads>(st, to);
  publish_shared();
  if (tid == 0) sh.ipar[0] = last_to_finish(&ws.info[b * kInfo + 3], (int32_t)gridDim.x);
  __syncthreads();
  if (sh.ipar[0] == 0) return;   // whole workgroup
  const uint32_t n = load_shared(to.count);
  __syncthreads();
  final_select<RUN>(sh, thr, n, N, k, b * k, c, out, to, &ws.info[b * kInfo + 2]);
}

// The score kernels; with CAND = false they write lse_out, the rows' upper
// bounds and the sample instead of cand.  Both modes pick the same kernel for a
// given V, so the log-sum-exp (and so every recomputed candidate) matches the
// written candidates bit for bit.
template <bool CAND>
static void launch_scores_mode(const void* logits, const float* prev, const uint32_t* mask,
                               float* cand, float* row_max, float* lse_out, int32_t R, int32_t V,
                               bool bf16, const SampleOut& smp, hipStream_t stream) {
  constexpr int64_t kWaves = kScoreThreads / 64;
#define GRACE_SC(TT, NCH, RUN)                                                                  \
  hipLaunchKernelGGL((beam_scores_reg_kernel<TT, NCH, RUN, CAND>),                              \
                     dim3((unsigned)(((int64_t)R + kWaves * score_rows_per_wave<NCH, CAND>() - 1) /    \
                                     (kWaves * score_rows_per_wave<NCH, CAND>()))),                    \
                     dim3(kScoreThreads), 0, stream, (const TT*)logits, prev, mask, cand,        \
                     row_max, lse_out, R, V, smp)
#define GRACE_SC_NCH(TT, RUN)               \
  do {                                      \
    if (nch == 1) GRACE_SC(TT, 1, RUN);     \
    else if (nch == 2) GRACE_SC(TT, 2, RUN); \
    else if (nch <= 4) GRACE_SC(TT, 4, RUN); \
    else GRACE_SC(TT, 8, RUN);              \
  } while (0)
  // rows of up to 4096 tokens fit the registers; 16-byte runs need V a
  // multiple of 8 and 16-byte aligned logits
  const bool run = V % 8 == 0 && ((uintptr_t)logits & 15) == 0;
  const int nch = (V + 511) / 512;
  if (V <= 4096) {
    if (bf16) {
      if (run) GRACE_SC_NCH(uint16_t, true);
      else GRACE_SC_NCH(uint16_t, false);
    } else {
      if (run) GRACE_SC_NCH(float, true);
      else GRACE_SC_NCH(float, false);
    }
    return;
  }
  const int64_t blocks = ((int64_t)R + kWaves - 1) / kWaves;
  if (bf16) {
    hipLaunchKernelGGL((beam_scores_kernel<uint16_t, CAND>), dim3((unsigned)blocks), dim3(kScoreThreads),
                       0, stream, (const uint16_t*)logits, prev, mask, cand, row_max, lse_out, R, V, smp);
  } else {
    hipLaunchKernelGGL((beam_scores_kernel<float, CAND>), dim3((unsigned)blocks), dim3(kScoreThreads), 0,
                       stream, (const float*)logits, prev, mask, cand, row_max, lse_out, R, V, smp);
  }
#undef GRACE_SC_NCH
#undef GRACE_SC
}

hipError_t launch_beam_scores(const void* logits, const float* prev, const uint32_t* mask,
                              float* cand, float* row_max, int32_t R, int32_t V, bool bf16,
                              hipStream_t stream) {
  launch_scores_mode<true>(logits, prev, mask, cand, row_max, nullptr, R, V, bf16, SampleOut{}, stream);
  return hipGetLastError();
}

size_t beam_topk_workspace_bytes(int32_t B, int32_t M, int32_t V) {
  return TopkWs::bytes(B, topk_slices((uint32_t)M * (uint32_t)V));
}

// N <= kSmallN
template <class Src, bool VEC8>
static hipError_t launch_topk_small(const Src& src, int32_t B, uint32_t N, int32_t k,
                                    const TopkOut& out, hipStream_t stream) {
  const dim3 grid((unsigned)B), block(kTopkThreads);
  const uint32_t runs = (N + 8 * kTopkThreads - 1) / (8 * kTopkThreads);
  if (runs <= 1)
    hipLaunchKernelGGL((topk_small_kernel<Src, VEC8, 1>), grid, block, 0, stream, src, N, k, out);
  else if (runs <= 4)
    hipLaunchKernelGGL((topk_small_kernel<Src, VEC8, 4>), grid, block, 0, stream, src, N, k, out);
  else
    hipLaunchKernelGGL((topk_small_kernel<Src, VEC8, 8>), grid, block, 0, stream, src, N, k, out);
  return hipGetLastError();
}

// Candidates to expect above the threshold, from samples of one in 2^lp: k and
// eight standard deviations of a sampled count of k, at most 3/4 of the list (as
// many deviations are left above that).  From lp = 5 on that is fewer than six for
// k = 4096, so there it is six deviations and the rest of the workspace takes
// what the list does not: reading all candidates again in one workgroup, which a set
// short of k needs, takes 14 ms for 16.8e6 of them.
static double gather_target(int32_t k, int lp, double deviations = 8.0) {
  return (double)k + deviations * sqrt((double)k * (double)(1u << lp));
}
static uint32_t samples_wanted(int32_t k, int lp) {
  const uint32_t t = (uint32_t)fmin(gather_target(k, lp), fmax(0.75 * kGatherCap, gather_target(k, lp, 6.0)));
  const uint32_t w = (t + (1u << lp) - 1) >> lp;
  return w < 1 ? 1 : w;
}
// A sample of one in 2^lp is as good as a larger one while the expected
// candidates stay within 2.5 k and the list: fewer samples to read cost less than
// the few more candidates to rank.
static bool sample_suffices(int32_t k, int lp) {
  const double t = gather_target(k, lp);
  return t <= 0.75 * kGatherCap && t <= fmax(2.5 * k, 1024.0);
}

constexpr uint32_t kSampleTarget = 131072;   // samples per request: eight select workgroups

static unsigned select_blocks(uint32_t n) { return (n + kSelectSamples - 1) / kSelectSamples; }

template <class Smp>
static void launch_select(const Smp& smp, int32_t B, uint32_t N, int32_t k, int lp, const TopkWs& ws,
                          hipStream_t stream) {
  hipLaunchKernelGGL(topk_select_kernel<Smp>, dim3(select_blocks(smp.n), (unsigned)B), dim3(kTopkThreads),
                     0, stream, smp, N, samples_wanted(k, lp), lp, ws);
}

template <class Src>
static void launch_select_chunks(const Src& src, int32_t B, uint32_t N, int32_t k, const TopkWs& ws,
                                 hipStream_t stream) {
  int lp = 3;
  while (lp < 8 && ((N >> lp) > kSampleTarget ||
                    ((N >> lp) > kSelectSamples && sample_suffices(k, lp + 1))))
    ++lp;
  const uint32_t group = 32u << lp, groups = (uint32_t)(((uint64_t)N + group - 1) / group);
  if (select_blocks(32u * groups) > 1)
    hipLaunchKernelGGL(topk_clear_kernel, dim3((unsigned)B), dim3(kTopkThreads), 0, stream, ws);
  launch_select(ChunkSample<Src>{src, lp, 32u * groups}, B, N, k, lp, ws, stream);
}

template <bool VEC8>
static hipError_t launch_topk_array(const CandArray& src, int32_t B, uint32_t N, int32_t k,
                                    void* workspace, const TopkOut& out, hipStream_t stream) {
  if (N <= kSmallN) return launch_topk_small<CandArray, VEC8>(src, B, N, k, out, stream);
  const TopkWs ws(workspace, B, topk_slices(N));
  launch_select_chunks(src, B, N, k, ws, stream);
  // 16384 candidates (64 KiB) per workgroup, fewer while the chip is not full
  uint32_t per = 16384;
  while (per > 4096 && (uint64_t)B * N / per < 2048) per >>= 1;
  hipLaunchKernelGGL(topk_gather_array_kernel<VEC8>, dim3((N + per - 1) / per, (unsigned)B),
                     dim3(kGatherThreads), 0, stream, src, N, per, ws);
  hipLaunchKernelGGL((topk_final_kernel<CandArray, VEC8>), dim3((unsigned)B), dim3(kTopkThreads), 0,
                     stream, src, N, k, ws, out);
  return hipGetLastError();
}

hipError_t launch_beam_topk(const float* cand, const float*, int32_t B, int32_t M, int32_t V,
                            int32_t k, void* workspace, int32_t* parents, int32_t* tokens,
                            float* scores, hipStream_t stream) {
  const uint32_t N = (uint32_t)M * (uint32_t)V;
  const CandArray src{cand};
  const TopkOut out{parents, tokens, scores, FastDiv((uint32_t)V), V};
  // 16-byte loads need every request's candidates on a 16-byte boundary
  if (N % 8 == 0 && ((uintptr_t)cand & 15) == 0)
    return launch_topk_array<true>(src, B, N, k, workspace, out, stream);
  return launch_topk_array<false>(src, B, N, k, workspace, out, stream);
}

size_t beam_step_workspace_bytes(int32_t B, int32_t M, int32_t V) {
  return beam_topk_workspace_bytes(B, M, V) + (size_t)B * M * 8;
}

template <class T, bool RUN>
static hipError_t launch_step(const void* logits, const float* prev, const uint32_t* mask, int32_t B,
                              int32_t M, int32_t V, int32_t k, void* workspace,
                              const TopkOut& out, hipStream_t stream) {
  const int32_t R = B * M;
  const uint32_t N = (uint32_t)M * (uint32_t)V;
  const int S = topk_slices(N);
  TopkWs ws(workspace, B, S);
  // after the top-k workspace: the rows' log-sum-exp and upper bounds
  float* lse = (float*)((char*)workspace + TopkWs::bytes(B, S));
  float* row_max = lse + R;
  const CandFromLogits<T> src{(const T*)logits, prev, mask, lse, M, V, FastDiv((uint32_t)V)};
  constexpr bool bf16 = sizeof(T) == 2;
  if (N <= kSmallN) {
    launch_scores_mode<false>(logits, prev, mask, nullptr, row_max, lse, R, V, bf16, SampleOut{}, stream);
    return launch_topk_small<CandFromLogits<T>, RUN>(src, B, N, k, out, stream);
  }
  // the sample of the score pass: one token in eight, or in more where that
  // does not fit its area or the target, or where fewer do
  SampleOut smp;
  for (int lp = 3; lp <= 9 && V >= (1 << lp); ++lp) {
    const uint64_t per_row = ((uint64_t)V + (1u << lp) - 1) >> lp, n = per_row * M;
    if (n + 3 > (uint64_t)ws.sample_room()) continue;
    smp = SampleOut{ws.sample, ws.sample_stride(), ws, (uint32_t)per_row, lp,
                    M, FastDiv((uint32_t)M)};
    if (n <= kSelectSamples || (n <= kSampleTarget && !sample_suffices(k, lp + 1))) break;
  }
  if (smp.p != nullptr) ws.spill = (int32_t)(((uint64_t)smp.per_row * (uint32_t)M + 3 + 3) / 4 * 4);
  // lanes per row: as many as its runs (tokens) need, at most a wave
  constexpr int E = RUN ? 8 : 1;
  int ll = 0;
  while (ll < 6 && (E << ll) < V) ++ll;
  launch_scores_mode<false>(logits, prev, mask, nullptr, row_max, lse, R, V, bf16, smp, stream);
  const StoredSample<CandFromLogits<T>> stored{src, smp.p, smp.stride, smp.per_row * (uint32_t)M, smp.lp,
                                               FastDiv(smp.p != nullptr ? smp.per_row : 1u)};
  const uint32_t fused_blocks = ((uint32_t)M + kFusedRows - 1) / kFusedRows;
  if (smp.p != nullptr && stored.n <= kSelectSamples && fused_blocks <= kFusedMaxPerRequest &&
      fused_blocks * (uint32_t)B <= kFusedMaxBlocks) {
    hipLaunchKernelGGL((topk_fused_rows_kernel<T, RUN>), dim3(fused_blocks, (unsigned)B), dim3(kTopkThreads),
                       0, stream, stored, row_max, ll, N, samples_wanted(k, smp.lp), smp.lp, k, ws, out);
    return hipGetLastError();
  }
  if (smp.p != nullptr)
    launch_select(stored, B, N, k, smp.lp, ws, stream);
  else
    launch_select_chunks(src, B, N, k, ws, stream);
  // rows per wave: up to 64, fewer while that leaves the chip without waves
  int32_t rpw = 64;
  while (rpw > 4 && (int64_t)B * ((M + rpw - 1) / rpw) < 8192) rpw >>= 1;
  const int32_t per_block = rpw * (kGatherThreads / 64);
  hipLaunchKernelGGL((topk_gather_rows_kernel<T, RUN>), dim3((unsigned)((M + per_block - 1) / per_block), (unsigned)B),
                     dim3(kGatherThreads), 0, stream, src, row_max, rpw, ll, N, ws);
  hipLaunchKernelGGL((topk_final_kernel<CandFromLogits<T>, RUN>), dim3((unsigned)B), dim3(kTopkThreads), 0,
                     stream, src, N, k, ws, out);
  return hipGetLastError();
}

hipError_t launch_beam_step(const void* logits, const float* prev, const uint32_t* mask,
                            int32_t B, int32_t M, int32_t V, int32_t k, bool bf16, void* workspace,
                            int32_t* parents, int32_t* tokens, float* scores,
                            hipStream_t stream) {
  const TopkOut out{parents, tokens, scores, FastDiv((uint32_t)V), V};
  // runs of eight: V a multiple of 8 and 16-byte aligned logits
  const bool run = V % 8 == 0 && ((uintptr_t)logits & 15) == 0;
#define GRACE_STEP(TT, RUN) return launch_step<TT, RUN>(logits, prev, mask, B, M, V, k, workspace, out, stream)
  if (bf16) {
    if (run) GRACE_STEP(uint16_t, true);
    GRACE_STEP(uint16_t, false);
  }
  if (run) GRACE_STEP(float, true);
  GRACE_STEP(float, false);
#undef GRACE_STEP
}

int32_t beam_topk_max_k() { return kGatherCap / 2; }

}  // namespace grace
