// Top-K keep (gfx950): Eq. (topk_selection) of ParallelVLM Sec. 4.1, keeping
// the top 1 - alpha fraction of visual tokens (Sec. 4.2).
//
// Ranking: larger score first, lower index first among equal scores, -0.0
// equal to +0.0, NaN below every number.  Each score maps to a 32-bit key
// whose unsigned order is that ranking (ties aside); the K-th largest key is
// found by an MSB-first radix select (four 8-bit digits), and one ordered
// pass then emits, in ascending index order, every index whose key is above
// the threshold plus the lowest-indexed ones equal to it.  The whole
// selection is integer work, so the result is bit-exact.
//
// Rows of up to 16384 scores take one 1024-thread workgroup each, the keys in
// registers.  Longer rows are split over NW workgroups and five ordinary
// launches: every launch sums the slices' histograms of the digit before,
// picks that digit and histograms its own slice's next one; the last emits.
// Each workgroup also counts its slice's keys above each digit, so the last
// launch knows where every slice's output starts.  No workgroup waits for
// another.  131072 scores from two criteria, us: one launch with five waits 51.1
// eagerly (cooperative) and 38.0 captured, these 32.4 and 36.8; plain scores
// 47.7 and 34.9, 31.6 and 36.9.  (The slice requested before the digit is known
// was slower: its loads delay the histograms'.)
#include "common.h"

namespace pvlm {
namespace {

constexpr int kTopkThreads = 256;
constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kPerThread = 16;   // consecutive scores per thread (register slice, ordered pass)
constexpr int kSlice = kTopkThreads * kPerThread;  // scores per workgroup unless B*NW would exceed the CUs
constexpr int kCopies = 8;       // counters per histogram bin: scores share few top digits, and LDS
                                 // atomics of one instruction to one address serialise
static_assert(kTopkThreads == 256, "one histogram bin per thread");

__device__ __forceinline__ uint32_t rank_key(float f) {
  if (f != f) return 0u;                 // NaN: lowest
  uint32_t u = __float_as_uint(f);
  if (f == 0.f) u = 0u;                  // -0.0 ranks as +0.0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix sum over a workgroup of WAVES waves; returns the exclusive
// prefix of this thread and writes the total to *total.
template <int WAVES = kTopkWaves>
__device__ __forceinline__ int block_exclusive_scan(int v, int* s_warp, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_warp[w] = x;
  __syncthreads();
  int before = 0;
#pragma unroll
  for (int ww = 0; ww < WAVES; ++ww) before += ww < w ? s_warp[ww] : 0;
  int tot = 0;
#pragma unroll
  for (int ww = 0; ww < WAVES; ++ww) tot += s_warp[ww];
  *total = tot;
  __syncthreads();
  return before + x - v;
}

// One wave (lanes 0-63): the digit of a 256-bin histogram (counts of the
// keys in the current prefix range, by next digit) that holds the need-th
// largest key, scanning digits from the top.  Lane l owns digits 255 - 4l ..
// 252 - 4l.  The lane that finds it calls found(digit, keys above the digit).
template <typename F>
__device__ __forceinline__ void find_digit(const int* hist, int need, F found) {
  const int lane = threadIdx.x & 63;
  int c[4], own = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    c[q] = hist[255 - 4 * lane - q];
    own += c[q];
  }
  int incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  const int excl = incl - own;
  if (excl < need && need <= incl) {
    int acc = excl;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (acc + c[q] >= need) {
        found(255 - 4 * lane - q, acc);
        break;
      }
      acc += c[q];
    }
  }
}

struct TArgs {
  const float* score;    // scores, or (fused MASS form) crit^L
  const float* sub;      // fused MASS form: crit^0, subtracted from crit^L; else NULL
  float* score_out;      // fused MASS form: the scores written out (nullable)
  const int32_t* m;
  const int32_t* k;
  int32_t* idx;
  int32_t* status;
  int* hist;       // [4][B][NW][256] per-slice histograms of each digit
  int2* state;     // [4][B]: the prefix up to a digit, keys above its range
  int* cnt;        // [3][B][NW]: a slice's keys above the prefix range by a digit
  int64_t m_cap;
  int k_cap, NW, slice;
};

// Entry i of a row (row offset `off`): the score, or in the fused MASS form
// the UV-Prune variation crit^L - crit^0 of Eq. (average_similarity),
// rounded exactly as pvlm_uvprune_score(MASS) rounds it (one fp32 subtraction).
template <bool FUSED>
__device__ __forceinline__ float score_at(const TArgs& a, size_t off, int64_t i) {
  if constexpr (FUSED) return a.score[off + i] - a.sub[off + i];
  else return a.score[off + i];
}

__device__ __forceinline__ int sum256(int x, int* s_warp) {
  int tot;
  block_exclusive_scan(x, s_warp, &tot);
  return tot;
}

// Launch `pass` of a long row: 0 .. 3 histogram that digit of the slice, 4
// emits.  Bound by the launch and one round trip each for the histograms and
// the slice (131072 scores: 32 slices of 4096).
template <bool FUSED>
__global__ void __launch_bounds__(kTopkThreads) topk_kernel(TArgs a, int pass) {
  constexpr int kChunk = kTopkThreads * kPerThread;
  __shared__ int hist[256 * kCopies];
  __shared__ int s_warp[kTopkWaves];
  __shared__ int s_res[3];
  const int b = blockIdx.x / a.NW, j = blockIdx.x % a.NW;
  const int tid = threadIdx.x, B = gridDim.x / a.NW;
  const size_t roff = (size_t)b * a.m_cap;
  int32_t* out = a.idx + (size_t)b * a.k_cap;

  int mb = a.m[b], kb = a.k[b];
  bool bad = false;
  if (mb < 0 || mb > a.m_cap) {
    bad = true;
    mb = mb < 0 ? 0 : (int)a.m_cap;
  }
  const int kmax = mb < a.k_cap ? mb : a.k_cap;
  if (kb < 0 || kb > kmax) {
    bad = true;
    kb = kb < 0 ? 0 : kmax;
  }
  if (pass == 0 && j == 0) {
    if (bad && tid == 0) dev_flag(a.status, PVLM_DEV_RANGE);
    for (int r = kb + tid; r < a.k_cap; r += kTopkThreads) out[r] = -1;
  }
  const int s0 = min(mb, j * a.slice), s1 = min(mb, s0 + a.slice);
  if constexpr (FUSED) {  // the scores of this workgroup's share of the row (0 past m[b])
    if (a.score_out && pass == 0) {
      const int64_t e1 = min((int64_t)(j + 1) * a.slice, a.m_cap);
      for (int64_t i = max((int64_t)j * a.slice, (int64_t)mb) + tid; i < e1; i += kTopkThreads)
        a.score_out[roff + i] = 0.f;
    }
  }
  if (kb == 0 && (!FUSED || !a.score_out || pass > 0)) return;

  // the digit before: every slice's histogram, and the keys of earlier slices
  uint32_t prefix = 0, mask = 0;
  int above = 0, gt_before = 0, eq_before = 0;
  if (pass > 0) {
    const int* hrow = a.hist + ((size_t)(pass - 1) * B + b) * a.NW * 256;
    int t = 0, before = 0, own = 0;
    for (int j0 = 0; j0 < a.NW; j0 += 16) {
      int v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = hrow[(size_t)min(j0 + q, a.NW - 1) * 256 + tid];  // in flight together
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int x = j0 + q < a.NW ? v[q] : 0;
        t += x;
        before += j0 + q < j ? x : 0;
        own = j0 + q == j ? x : own;
      }
    }
    const int2 st = pass > 1 ? a.state[(size_t)(pass - 1) * B + b] : make_int2(0, 0);
    hist[tid] = t;
    __syncthreads();
    if (tid < 64)
      find_digit(hist, kb - st.y, [&](int digit, int acc) {
        s_res[0] = digit;
        s_res[1] = st.y + acc;
      });
    __syncthreads();
    const int digit = s_res[0];
    above = s_res[1];
    prefix = (uint32_t)st.x | (uint32_t)digit << (32 - 8 * pass);
    mask = ~0u << (32 - 8 * pass);
    if (pass < 4) {
      const int g = sum256(tid > digit ? own : 0, s_warp);
      if (tid == 0) {
        a.cnt[((size_t)(pass - 1) * B + b) * a.NW + j] = g;
        if (j == 0) a.state[(size_t)pass * B + b] = make_int2((int)prefix, above);
      }
    } else {
      int g = tid > digit ? before : 0;
      for (int q = tid; q < 3 * j; q += kTopkThreads)
        g += a.cnt[((size_t)(q / j) * B + b) * a.NW + q % j];
      gt_before = sum256(g, s_warp);
      if (tid == digit) s_res[2] = before;
      __syncthreads();
      eq_before = s_res[2];
    }
    __syncthreads();  // hist and s_res are reused below
  }

  if (pass < 4) {
    const int shift = 24 - 8 * pass, copy = tid % kCopies;
    for (int i = tid; i < 256 * kCopies; i += kTopkThreads) hist[i] = 0;
    __syncthreads();
    for (int base = s0; base < s1; base += kChunk) {
      float v[kPerThread];
#pragma unroll
      for (int e = 0; e < kPerThread; ++e)  // clamped loads, all in flight together
        v[e] = score_at<FUSED>(a, roff, min(base + e * kTopkThreads + tid, s1 - 1));
#pragma unroll
      for (int e = 0; e < kPerThread; ++e) {
        const int i = base + e * kTopkThreads + tid;
        if (i < s1) {
          if constexpr (FUSED) {
            if (pass == 0 && a.score_out) a.score_out[roff + i] = v[e];
          }
          const uint32_t key = rank_key(v[e]);
          if ((key & mask) == prefix) atomicAdd(&hist[((key >> shift) & 255) * kCopies + copy], 1);
        }
      }
    }
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int c = 0; c < kCopies; ++c) t += hist[tid * kCopies + c];
    a.hist[(((size_t)pass * B + b) * a.NW + j) * 256 + tid] = t;
    return;
  }

  const uint32_t tau = prefix;
  const int need_eq = kb - above;  // keys equal to tau to keep, lowest indices first
  int carry_out = gt_before + min(eq_before, need_eq);
  int carry_eq = eq_before;

  // ---- ordered emission of the slice in ascending index order
  for (int base = s0; base < s1; base += kChunk) {
    const int i0 = base + tid * kPerThread;
    uint32_t keys[kPerThread];
    int g = 0, e_ = 0;
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
      const bool valid = i0 + e < s1;
      const float x = score_at<FUSED>(a, roff, min(i0 + e, s1 - 1));  // clamped (s1 > base >= 0)
      keys[e] = valid ? rank_key(x) : 0u;
      g += valid && keys[e] > tau;
      e_ += valid && keys[e] == tau;
    }
    int tot_eq;
    const int eq_before = carry_eq + block_exclusive_scan(e_, s_warp, &tot_eq);
    int take_eq = need_eq - eq_before;
    take_eq = take_eq < 0 ? 0 : (take_eq > e_ ? e_ : take_eq);
    int tot_sel;
    int pos = carry_out + block_exclusive_scan(g + take_eq, s_warp, &tot_sel);
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
      if (i0 + e < s1) {
        bool sel = keys[e] > tau;
        if (keys[e] == tau && take_eq > 0) {
          sel = true;
          --take_eq;
        }
        if (sel && pos < kb) out[pos++] = i0 + e;
      }
    }
    carry_eq += tot_eq;
    carry_out += tot_sel;
  }
}

// Rows of at most kSmallMax scores: one 1024-thread workgroup per row, no
// inter-workgroup exchange.  Thread t holds the keys of entries e * 1024 + t
// (coalesced loads) in registers.  The radix select takes three digits of
// 12, 10 and 10 bits: float keys of real data share few values of their top
// 8 bits (sign and exponent), and a first digit that wide spreads them over
// enough histogram bins that the LDS atomics rarely collide.  The ordered
// emission computes every selected entry's output position directly from
// per-(entry round, wave) counts, so no thread needs a contiguous range.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallMaxPer = 16;  // beyond 16384 scores, several workgroups per row are faster
constexpr int kSmallMax = kSmallThreads * kSmallMaxPer;
constexpr int kSmallBins = 4096;
// Every histogram bin has kHistCopies counters, lane l adding to copy l % 8:
// scores concentrate in few top digits (the UV-Prune scores of a 72B layer
// fill 29 of the 4096 first-pass bins), and LDS atomics of one instruction to
// one address serialise.
constexpr int kHistCopies = 8;
constexpr int kSmallLds = kSmallBins * (kHistCopies + 1) * 4;  // the copies, then the bin totals

template <int PER, bool FUSED>
__global__ void __launch_bounds__(kSmallThreads) topk_small_kernel(TArgs a) {
  extern __shared__ __align__(16) int hist[];  // [kSmallBins][kHistCopies], then [kSmallBins] totals
  int* bins = hist + kSmallBins * kHistCopies;
  __shared__ int s_warp[kSmallWaves];
  __shared__ int s_res[2];
  __shared__ int s_cnt[2][PER][kSmallWaves];  // per (round e, wave): keys above tau, equal to tau
  const int b = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const size_t roff = (size_t)b * a.m_cap;
  int32_t* out = a.idx + (size_t)b * a.k_cap;
  int mb = a.m[b], kb = a.k[b];
  bool bad = false;
  if (mb < 0 || mb > a.m_cap) {
    bad = true;
    mb = mb < 0 ? 0 : (int)a.m_cap;
  }
  const int kmax = mb < a.k_cap ? mb : a.k_cap;
  if (kb < 0 || kb > kmax) {
    bad = true;
    kb = kb < 0 ? 0 : kmax;
  }
  if (bad && tid == 0) dev_flag(a.status, PVLM_DEV_RANGE);
  for (int r = kb + tid; r < a.k_cap; r += kSmallThreads) out[r] = -1;
  if (!FUSED && kb == 0) return;  // uniform across the workgroup
  // unconditional loads (indices clamped into the row, or to entry 0 of an
  // empty row) so that all PER are in flight together, then the entries past
  // the row are zeroed
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) v[e] = score_at<FUSED>(a, roff, min(e * kSmallThreads + tid, max(mb - 1, 0)));
  // the first digit's histogram (every copy) is cleared while the keys load
  __builtin_amdgcn_sched_barrier(0);
  for (int i = tid; i < kSmallBins * kHistCopies / 4; i += kSmallThreads)
    reinterpret_cast<int4*>(hist)[i] = make_int4(0, 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (FUSED) {  // the scores written out (0 past m[b]), then the selection
    if (a.score_out)
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int i = e * kSmallThreads + tid;
        if (i < a.m_cap) a.score_out[roff + i] = i < mb ? v[e] : 0.f;
      }
    if (kb == 0) return;
  }
  uint32_t kr[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) kr[e] = e * kSmallThreads + tid < mb ? rank_key(v[e]) : 0u;

  // ---- radix select of the kb-th largest key: digits [31:20], [19:10], [9:0].
  // The first digit's keys crowd into few bins (the sign and exponent of
  // real scores), so its histogram has kHistCopies counters per bin; the later
  // digits count only the keys left in the chosen bin, one counter per bin.
  uint32_t prefix = 0, mask = 0;
  int above = 0;
#pragma unroll 1
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
    const int nb = pass == 0 ? 4096 : 1024;
    const int copies = pass == 0 ? kHistCopies : 1;
    if (pass > 0)
      for (int i = tid; i < nb / 4; i += kSmallThreads) reinterpret_cast<int4*>(hist)[i] = make_int4(0, 0, 0, 0);
    __syncthreads();
    const int copy = pass == 0 ? (lane & (kHistCopies - 1)) : 0;
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (e * kSmallThreads + tid < mb && (kr[e] & mask) == prefix)
        atomicAdd(&hist[((kr[e] >> shift) & (uint32_t)(nb - 1)) * copies + copy], 1);
    __syncthreads();
    if (pass == 0) {
      // each bin's copies summed, consecutive threads on consecutive bins
      for (int i = tid; i < nb; i += kSmallThreads) {
        const int4* h = reinterpret_cast<const int4*>(hist + i * kHistCopies);
        const int4 x = h[0], y = h[1];
        bins[i] = x.x + x.y + x.z + x.w + y.x + y.y + y.z + y.w;
      }
      __syncthreads();
    }
    const int* totals = pass == 0 ? bins : hist;
    // bins in descending order: thread t owns q = nb / 1024 consecutive ones
    const int q = nb / kSmallThreads;
    const int top = nb - 1 - tid * q;
    int cnt[kSmallBins / kSmallThreads];
    int own = 0;
#pragma unroll
    for (int j = 0; j < kSmallBins / kSmallThreads; ++j) {
      cnt[j] = j < q ? totals[top - j] : 0;
      own += cnt[j];
    }
    int tot;
    const int excl = block_exclusive_scan<kSmallWaves>(own, s_warp, &tot);
    const int need = kb - above;
    if (excl < need && need <= excl + own) {
      int acc = excl;
#pragma unroll
      for (int j = 0; j < kSmallBins / kSmallThreads; ++j) {
        if (j < q) {
          if (acc + cnt[j] >= need) {
            s_res[0] = top - j;
            s_res[1] = above + acc;
            break;
          }
          acc += cnt[j];
        }
      }
    }
    __syncthreads();
    prefix |= (uint32_t)s_res[0] << shift;
    mask |= (uint32_t)(nb - 1) << shift;
    above = s_res[1];
  }
  const uint32_t tau = prefix;
  const int need_eq = kb - above;  // keys equal to tau to keep, lowest indices first

  // ---- emission: output position of entry (e, w, lane) = keys above tau
  //      before it + min(keys equal to tau before it, need_eq)
  uint64_t bg[PER], be[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const bool valid = e * kSmallThreads + tid < mb;
    bg[e] = __ballot(valid && kr[e] > tau);
    be[e] = __ballot(valid && kr[e] == tau);
    if (lane == 0) {
      s_cnt[0][e][w] = __popcll(bg[e]);
      s_cnt[1][e][w] = __popcll(be[e]);
    }
  }
  __syncthreads();
  // exclusive prefix over (e, w) in that order, by one wave: lane l takes
  // PER * kSmallWaves / 64 consecutive slots
  if (w == 0) {
    constexpr int kSlots = PER * kSmallWaves;
    constexpr int kPerLane = (kSlots + 63) / 64;
    int* cg = &s_cnt[0][0][0];
    int* ce = &s_cnt[1][0][0];
    int sg = 0, se = 0;
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
      const int sl = lane * kPerLane + j;
      if (sl < kSlots) {
        sg += cg[sl];
        se += ce[sl];
      }
    }
    int ig = sg, ie = se;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int yg = __shfl_up(ig, o, 64), ye = __shfl_up(ie, o, 64);
      if (lane >= o) {
        ig += yg;
        ie += ye;
      }
    }
    int rg = ig - sg, re = ie - se;
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
      const int sl = lane * kPerLane + j;
      if (sl < kSlots) {
        const int g = cg[sl], q = ce[sl];
        cg[sl] = rg;
        ce[sl] = re;
        rg += g;
        re += q;
      }
    }
  }
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const bool gt = (bg[e] >> lane) & 1ull, eq = (be[e] >> lane) & 1ull;
    if (gt || eq) {
      const int gt_before = s_cnt[0][e][w] + __popcll(bg[e] & below);
      const int eq_before = s_cnt[1][e][w] + __popcll(be[e] & below);
      if (gt || eq_before < need_eq) {
        const int pos = gt_before + min(eq_before, need_eq);
        if (pos < kb) out[pos] = e * kSmallThreads + tid;
      }
    }
  }
}

struct TPlan {
  int NW, slice;
  size_t off_hist, off_state, off_cnt, bytes;
};

// stream / with_stream: as for verify's plan (the stream's compute-unit budget).
pvlm_status plan_topk(int B, int64_t m_cap, TPlan* p, hipStream_t stream, bool with_stream) {
  if (B < 1 || m_cap < 1 || m_cap > ((int64_t)1 << 30)) return PVLM_ERR_SHAPE;
  if (m_cap <= kSmallMax) {  // one workgroup per row, no workspace
    p->NW = 1;
    p->slice = (int)m_cap;
    p->bytes = 0;
    return PVLM_OK;
  }
  DeviceInfo di;
  pvlm_status st = with_stream ? device_info(&di, stream) : device_info(&di);
  if (st != PVLM_OK) return st;
  if (B > di.cus) return PVLM_ERR_UNSUPPORTED;  // the documented limit: long rows for every compute unit
  const int nw_max = di.cus / B;  // every workgroup sums the others' histograms: no more than fill the device
  int64_t nw = (m_cap + kSlice - 1) / kSlice;
  if (nw > nw_max) nw = nw_max;
  if (nw < 1) nw = 1;
  p->NW = (int)nw;
  p->slice = (int)((m_cap + nw - 1) / nw);
  size_t off = kSyncRegion;
  p->off_hist = off;
  off = align_up(off + sizeof(int) * 4 * (size_t)B * p->NW * 256, 256);
  p->off_state = off;
  off = align_up(off + sizeof(int2) * 4 * (size_t)B, 256);
  p->off_cnt = off;
  off = align_up(off + sizeof(int) * 3 * (size_t)B * p->NW, 256);
  p->bytes = off;
  return PVLM_OK;
}

}  // namespace
}  // namespace pvlm

using namespace pvlm;

extern "C" size_t pvlm_topk_workspace_size(int B, int64_t m_cap) {
  TPlan p;
  if (plan_topk(B, m_cap, &p, nullptr, false) != PVLM_OK) return 0;
  return p.bytes;
}

namespace {
// score: the scores, or with sub the fused MASS form (score = crit^L,
// sub = crit^0, optional score_out).
pvlm_status topk_run(int B, int64_t m_cap, const int32_t* m, const int32_t* k, int32_t k_cap,
                     const float* score, const float* sub, float* score_out, int32_t* idx,
                     void* ws, size_t ws_bytes, int32_t* status, hipStream_t stream) {
  if (!m || !k || !score || (k_cap > 0 && !idx)) return PVLM_ERR_NULL;
  if (B < 1 || m_cap < 1 || k_cap < 0 || m_cap > ((int64_t)1 << 30)) return PVLM_ERR_SHAPE;
  if (k_cap == 0 && !score_out) return PVLM_OK;
  TPlan p;
  pvlm_status st = plan_topk(B, m_cap, &p, stream, true);
  if (st != PVLM_OK) return st;
  if (p.bytes > 0 && (!ws || ws_bytes < p.bytes)) return PVLM_ERR_WORKSPACE;
  TArgs a = {};
  a.score = score;
  a.sub = sub;
  a.score_out = score_out;
  a.m = m;
  a.k = k;
  a.idx = idx;
  a.status = status;
  a.m_cap = m_cap;
  a.k_cap = k_cap;
  a.NW = p.NW;
  a.slice = p.slice;
  void* args[] = {&a};
  const bool fused = sub != nullptr;
  if (m_cap <= kSmallMax) {
    const int per = m_cap <= kSmallThreads * 4 ? 4 : (m_cap <= kSmallThreads * 8 ? 8 : kSmallMaxPer);
    const void* kern =
        per == 4 ? (fused ? reinterpret_cast<const void*>(topk_small_kernel<4, true>)
                          : reinterpret_cast<const void*>(topk_small_kernel<4, false>))
        : per == 8 ? (fused ? reinterpret_cast<const void*>(topk_small_kernel<8, true>)
                            : reinterpret_cast<const void*>(topk_small_kernel<8, false>))
                   : (fused ? reinterpret_cast<const void*>(topk_small_kernel<kSmallMaxPer, true>)
                            : reinterpret_cast<const void*>(topk_small_kernel<kSmallMaxPer, false>));
    PVLM_HIP(allow_dynamic_lds(kern, kSmallLds));
    PVLM_HIP(hipLaunchKernel(kern, dim3(B), dim3(kSmallThreads), args, kSmallLds, stream));
    return PVLM_OK;
  }
  char* wsb = static_cast<char*>(ws);
  a.hist = reinterpret_cast<int*>(wsb + p.off_hist);
  a.state = reinterpret_cast<int2*>(wsb + p.off_state);
  a.cnt = reinterpret_cast<int*>(wsb + p.off_cnt);
  for (int pass = 0; pass < 5; ++pass) {
    // The fused form writes the scores in its first launch and reads them in
    // the others: half the bytes of the criteria, which may be gone by then
    // (the caller may have the scores written over them).
    const bool crit = fused && (pass == 0 || !score_out);
    if (fused && !crit) a.score = score_out;
    void* pargs[] = {&a, &pass};
    const void* kern = crit ? reinterpret_cast<const void*>(topk_kernel<true>) : reinterpret_cast<const void*>(topk_kernel<false>);
    PVLM_HIP(hipLaunchKernel(kern, dim3(B * p.NW), dim3(kTopkThreads), pargs, 0, stream));
  }
  return PVLM_OK;
}
}  // namespace

extern "C" pvlm_status pvlm_topk_select(int B, int64_t m_cap, const int32_t* m, const int32_t* k,
                                        int32_t k_cap, const float* score, int32_t* idx, void* ws,
                                        size_t ws_bytes, int32_t* status, hipStream_t stream) {
  return topk_run(B, m_cap, m, k, k_cap, score, nullptr, nullptr, idx, ws, ws_bytes, status,
                  stream);
}

extern "C" pvlm_status pvlm_uvprune_topk_mass(int B, int L, int64_t m_cap, const int32_t* m,
                                              const float* crit_stack, const int32_t* k,
                                              int32_t k_cap, float* score, int32_t* idx, void* ws,
                                              size_t ws_bytes, int32_t* status,
                                              hipStream_t stream) {
  if (!crit_stack) return PVLM_ERR_NULL;
  if (B < 1 || L < 1 || m_cap < 1 || m_cap > ((int64_t)1 << 30)) return PVLM_ERR_SHAPE;
  return topk_run(B, m_cap, m, k, k_cap, crit_stack + (size_t)L * B * m_cap, crit_stack, score, idx,
                  ws, ws_bytes, status, stream);
}
