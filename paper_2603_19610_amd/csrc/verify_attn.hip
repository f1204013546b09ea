// Verify attention with fused per-token attention mass (gfx950).
//
// Computes the target's verification forward over the video KV cache
// (ParallelVLM Sec. 2.2; Sec. 4.2 Parallel Decoding) for the gamma + 1 verify
// rows, fused with the per-token attention mass that attention-guided pruning
// ranks visual tokens by (Sec. 3, Challenge 2; Suppl. D, attention criterion).
// The paper notes that pruning by attention needs explicit scores, which
// block-wise attention kernels never materialise (Sec. 3; Sec. 5.3,
// FlashAttention compatibility): here the mass is produced block by block,
// with no score matrix in memory.
//
// Design:
//  * Partial kernel.  The (Hq/Hkv) * T query rows of a KV head are packed as
//    the N side of 16-row MFMA tiles, tokens are the M side.  A workgroup
//    takes one KV head's row tiles (up to 9) and one chunk of its tokens: one
//    wave per tile (two below three tiles) and two waves that only load.
//    Those stream the chunk through an LDS ring of four stages (two blocks of
//    K and of V each), so every cache row is fetched once for all its query
//    rows and loads stay in flight behind the arithmetic; a tile's statistics
//    and O never leave its wave.  One barrier per stage hands a landed slot
//    over and an emptied one back.  The wave writes the chunk's (max,
//    exp-sum) per row and its unnormalised O.
//  * The mass needs every row's log-sum-exp over all chunks before any
//    probability.  Outside a stream capture the mass kernel streams K through
//    the same units a second time: no workgroup waits for another, so the
//    launches are ordinary ones, free to run beside any other stream's work.
//    Under capture, chunks of up to a few stages keep their scores in
//    registers and the partial kernel waits for the statistics itself; both
//    forms run the same arithmetic in the same order (bit-equal results).
//  * Finish kernel.  One wave per query row sums the chunks' O with the
//    weights exp2(chunk max - row max) / row sum; the mass is the sum of the
//    KV heads' partials.  Every order of summation is fixed.
//  * fp32 inputs run the same kernels on v_mfma_f32_16x16x4_f32.
//
// What bounds it (one MI355X; a large copy streams at 5.1 TB/s): long contexts
// are bound by HBM, K read twice (batch of four at 16-33K tokens: partial kernel
// 80 us for 419 MB, which the copy's rate takes 81; mass kernel 46), 136 rows
// per KV head by the waves' LDS reads and issue (131K tokens: partial 124-128 us
// where the copy's rate takes 105, mass 74-75), short ones by the launches' own
// chain of memory round trips (~1.7 us a launch, ~1 us a trip).  Rotary append
// and verify, us a layer, against one waiting launch per call with statistics
// and O exchanges, both timed in turn:
//   64 x 8 heads, 9 rows, 12.8K tokens (captured)  30.7 -> 27.7
//   28 x 4 heads, 6 rows, 6.4K (captured)          20.2 -> 18.5
//   28 x 4 heads, 1 row, 0.8K, no mass (captured)  14.0 -> 11.6
//   40 x 8 heads, 9 rows, batch 4, 16-33K (eager)   154 -> 141
//   64 x 8 heads, 17 rows, 131K (eager)             214 -> 208
//   4 x 1 heads, fp32, 5 rows, 1K (eager)            54 -> 33
// Past seven stages a chunk (three to six row tiles) a captured call reads K
// twice as well: the first line's layer takes 25.3 us without its append at
// 14300 tokens, 30.5 at 14400.
#include <mutex>
#include <type_traits>

#include "common.h"
#include "verify_plan.h"

namespace pvlm {
namespace {

constexpr int kLoaders = 2;      // its loading waves: one for K, one for V
constexpr int kSlots = 4;        // LDS slots of its ring, a stage of K and V rows each
constexpr int kFinWaves = kFinThreads / 64;  // waves of a finish workgroup
constexpr int kPageSlots = 512;  // page-table entries a workgroup stages in LDS
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kNegInf = -__builtin_huge_valf();
// A wave's running reference may trail its row maximum by this much (log2
// domain): probabilities then reach 2^8, far inside the range of bf16 and
// fp32, and O is rescaled only when a block's maximum exceeds it.
constexpr float kRefSlack = 8.f;

struct VArgs {
  const void* q;
  const void* k;
  const void* v;
  const int32_t* ctx_len;
  const int32_t* table;  // paged caches: [B][max_pages] pool page of each logical page; NULL: padded
  int64_t n_pages;       // pool pages
  int max_pages, page_shift;
  int64_t n_cap;
  int B, T, Hq, Hkv, G, R;
  unsigned g_magic; // row / G == row * g_magic >> 20 for row < 640 (2^20 / G + 1; G <= 640)
  int RTT, RG;      // 16-row tiles of a KV head's G * T rows, and workgroups sharing them
  int max_ctx;
  int splits, chunk, units;
  float sl2;        // scale * log2(e)
  float* mpart;     // [B][Hkv * RG][n_cap] mass of one workgroup row group
  float2* stats;    // [B * Hkv * RTT][splits][16] (log2-domain max, exp-sum) of a chunk's rows
  void* opart;      // [B * Hkv * RTT][splits][16][D] chunk sums relative to that max (fp32 or storage type)
  void* out;
  float* lse;
  float* mass;
  int32_t* status;
  int mass_wgs;     // finish kernel: workgroups that sum the mass,
  int mass_per;     // ... those of one sequence,
  int mass_rows;    // ... and the cache rows of one
  bool o32;                // O partials are fp32
  bool clear;              // ... which also clears the statistics
};

// Three 64-byte lines: a fourth costs every launch's waves a scalar load more
// before they start (208 bytes: 28 layers of one row over 0.8K tokens 333 us, 192: 324).
static_assert(sizeof(VArgs) <= 192, "kernel arguments fit three lines");

struct Unit {
  int split, bg, b, g, rg, ctx, N, c0, c1;
};

__device__ __forceinline__ int seq_ctx(const VArgs& a, int b, bool flag) {
  const int ctx = a.ctx_len[b];
  if (ctx >= 0 && ctx <= a.max_ctx) return ctx;
  if (flag) dev_flag(a.status, PVLM_DEV_RANGE);
  return ctx < 0 ? 0 : a.max_ctx;
}

// Workgroup i runs on XCD i % 8, so consecutive units, whose row groups read
// the same cache rows, are given to one XCD and share its L2 (a matter of
// speed only).
__device__ __forceinline__ bool decode_unit(const VArgs& a, Unit& u) {
  const int per = gridDim.x / 8;
  const int lg = ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8;
  if (lg >= a.units) return false;
  u.rg = lg % a.RG;
  const int cs = lg / a.RG;
  u.split = cs % a.splits;
  u.bg = cs / a.splits;
  u.g = u.bg % a.Hkv;
  u.b = u.bg / a.Hkv;
  u.ctx = seq_ctx(a, u.b, u.split == 0 && threadIdx.x == 0);
  u.N = u.ctx + a.T;
  u.c0 = u.split * a.chunk;
  u.c1 = min(u.c0 + a.chunk, u.N);
  return u.c0 < u.N;
}

// exp2 on the hardware transcendental unit (v_exp_f32).  It flushes results
// below 2^-126 to zero, which only drops probabilities under the mass
// tolerance's absolute floor.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ void lse_combine(float& m, float& z, float m2, float z2) {
  const float M = fmaxf(m, m2);
  if (M == kNegInf) {
    m = kNegInf;
    z = 0.f;
    return;
  }
  z = z * fast_exp2(m - M) + z2 * fast_exp2(m2 - M);
  m = M;
}

// ---------------------------------------------------------- element types --
// Both types put tokens on the M side and query rows on the N side of 16-row
// score tiles (lane (n, gq) = (lane & 15, lane >> 4) owns row n and tokens
// 4 gq .. 4 gq + 3 of each tile), which is the layout P.V needs as its A
// operand.  O keeps column DPL * n + jd of rows 4 gq + i.
template <int D_>
struct Bf16 {
  typedef uint16_t E;
  static constexpr int D = D_, BLK = 32, TT = 2, DPL = D / 16, CH = D / 8;
  static constexpr int KS = D / 32;  // 16-byte chunks of a row per lane (chunk 4 ks + gq)
  // B operands of P.V: element s of r[jd] is V[token(s)][16 jd + n], tokens
  // {4 gq .. +3, 16 + 4 gq .. +3}
  struct V {
    bf16x8 r[DPL];
  };
  static constexpr bool kSwizzleV = true;
  // cache row te, from which rows te .. te + BLK - 1 are contiguous (rows of the block at tb)
  static __device__ __forceinline__ const E* block(const KvRows& kv, int tb, int c1, int& te) {
    return kv_block<D>(kv, tb, c1, te);
  }
  // Transposed LDS reads: each 16 lanes fetch 16 columns of four rows (lane n
  // the 8 bytes of row n / 4, columns 4 (n % 4) on) and lane n receives
  // column n of the four.  Building the operands from row-major reads took 32
  // v_perm_b32 per block and row tile, a quarter of a wave's vector work.
  static __device__ __forceinline__ void read_v(const char* blk, int n, int gq, V& v) {
    typedef short s4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s4* lds_s4;
    const int row = 4 * gq + n / 4;
    const uint32_t at = lds_addr(blk) + row * D * 2 + (n & 1) * 8;
#pragma unroll
    for (int jd = 0; jd < DPL; ++jd) {
      const uint32_t p = at + ((2 * jd + ((n >> 1) & 1)) ^ (row % CH)) * 16;
      const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)p);
      const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(p + 16 * D * 2));
      typedef short s8 __attribute__((ext_vector_type(8)));
      v.r[jd] = __builtin_bit_cast(bf16x8, (s8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
  // column of O that value `idx` of a stored partial row holds
  static __device__ __forceinline__ int column(int idx) { return 16 * (idx % DPL) + idx / DPL; }
  // Q operand of k-step ks from its 16-byte chunk
  static __device__ __forceinline__ floatx4 qk(const uint4& k, const uint4& q, floatx4 s) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, q),
                                                   s, 0, 0, 0);
  }
  static __device__ __forceinline__ void pv(const floatx4 (&P)[TT], const V& v, floatx4 (&O)[DPL]) {
    bf16x8 pa;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) pa[4 * tt + i] = static_cast<__bf16>(P[tt][i]);
#pragma unroll
    for (int jd = 0; jd < DPL; ++jd) O[jd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, v.r[jd], O[jd], 0, 0, 0);
  }
  static __device__ __forceinline__ void store_out(E* row, int idx, float x) { row[column(idx)] = f32_to_bf16(x); }
};

template <int D_>
struct F32 {
  typedef float E;
  static constexpr int D = D_, BLK = 16, TT = 1, DPL = D / 16, CH = D / 4;
  static constexpr int KS = D / 16;
  struct V {
    float4 r[4][DPL / 4];
  };
  static constexpr bool kSwizzleV = false;
  static __device__ __forceinline__ const E* block(const KvRows& kv, int tb, int c1, int& te) {
    te = 0;
    return reinterpret_cast<const float*>(kv.base);
  }
  static __device__ __forceinline__ void read_v(const char* blk, int n, int gq, V& v) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < DPL / 4; ++j)
        v.r[s][j] = *reinterpret_cast<const float4*>(blk + ((4 * gq + s) * D + DPL * n + 4 * j) * sizeof(E));
  }
  // the four values of a lane's chunk are k indices 4 apart in four steps: the
  // same assignment on both sides, so the sum over d is complete
  static __device__ __forceinline__ floatx4 qk(const uint4& k, const uint4& q, floatx4 s) {
    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k.x), __uint_as_float(q.x), s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k.y), __uint_as_float(q.y), s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k.z), __uint_as_float(q.z), s, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k.w), __uint_as_float(q.w), s, 0, 0, 0);
  }
  static __device__ __forceinline__ void pv(const floatx4 (&P)[TT], const V& v, floatx4 (&O)[DPL]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int jd = 0; jd < DPL; ++jd) {
        const float4& x = v.r[i][jd / 4];
        const float b = jd % 4 == 0 ? x.x : jd % 4 == 1 ? x.y : jd % 4 == 2 ? x.z : x.w;
        O[jd] = __builtin_amdgcn_mfma_f32_16x16x4f32(P[0][i], b, O[jd], 0, 0, 0);
      }
  }
  static __device__ __forceinline__ void store_out(E* row, int idx, float x) { row[idx] = x; }
};

// Chunk partials of O: four consecutive values, and the PC values of a
// 16-byte piece.
__device__ __forceinline__ void store4(float* p, const float (&x)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(x[0], x[1], x[2], x[3]);
}
__device__ __forceinline__ void store4(uint16_t* p, const float (&x)[4]) {
  *reinterpret_cast<uint64_t*>(p) = pack_bf16x4(x[0], x[1], x[2], x[3]);
}
__device__ __forceinline__ void unpack(const uint4& u, float (&x)[4]) {
  x[0] = __uint_as_float(u.x);
  x[1] = __uint_as_float(u.y);
  x[2] = __uint_as_float(u.z);
  x[3] = __uint_as_float(u.w);
}
__device__ __forceinline__ void unpack(const uint4& u, float (&x)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[2 * j] = __uint_as_float(w[j] << 16);
    x[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
  }
}

// The row views of (b, g): a padded cache's base, or the pool through the
// page table, with the entries of rows [c0, c1) checked against the pool,
// clamped into it and staged in LDS when they fit (every thread takes part).
template <typename M>
__device__ __forceinline__ void kv_rows_setup(const VArgs& a, int b, int g, int c0, int c1, int32_t* s_pages,
                                              KvRows& kg, KvRows& vg) {
  constexpr int D = M::D;
  if (a.table) {
    const size_t hoff = ((size_t)g << a.page_shift) * D;
    const int32_t* tab = a.table + (size_t)b * a.max_pages;
    const int64_t pe = ((int64_t)a.Hkv << a.page_shift) * D;
    const int p0 = c0 >> a.page_shift, p1 = (c1 - 1) >> a.page_shift;
    const bool fit = p1 - p0 < kPageSlots;
    for (int pg = p0 + threadIdx.x; pg <= p1; pg += (int)blockDim.x) {
      int e = tab[pg];
      if (e < 0 || e >= a.n_pages) {
        dev_flag(a.status, PVLM_DEV_RANGE);
        e = e < 0 ? 0 : (int)(a.n_pages - 1);
      }
      if (fit) s_pages[pg - p0] = e;
    }
    __syncthreads();
    kg = {static_cast<const uint16_t*>(a.k) + hoff, tab, s_pages, pe, a.n_pages, a.page_shift, p0, true, fit};
    vg = {static_cast<const uint16_t*>(a.v) + hoff, tab, s_pages, pe, a.n_pages, a.page_shift, p0, true, fit};
  } else {
    const size_t off = ((size_t)b * a.Hkv + g) * a.n_cap * D * sizeof(typename M::E);
    kg = {reinterpret_cast<const uint16_t*>(static_cast<const char*>(a.k) + off), a.ctx_len, s_pages, 0, 1, 5, 0,
          false, false};
    vg = {reinterpret_cast<const uint16_t*>(static_cast<const char*>(a.v) + off), a.ctx_len, s_pages, 0, 1, 5, 0,
          false, false};
  }
}

__device__ __forceinline__ int row_t(const VArgs& a, int row) { return (int)((unsigned)row * a.g_magic >> 20); }

// Q row r of KV head g (rows are (t, head of the group), t slowest; padding
// rows repeat the last real one)
template <typename M>
__device__ __forceinline__ const typename M::E* q_row(const VArgs& a, int b, int g, int r) {
  const int row = min(r, a.R - 1), t = row_t(a, row), h = g * a.G + row - t * a.G;
  return static_cast<const typename M::E*>(a.q) + (((size_t)b * a.T + t) * a.Hq + h) * M::D;
}

// -------------------------------------------------------- partial kernel --
// One 32-row (fp32: 16-row) block of K or V into LDS by global->LDS loads of
// 1 KB per instruction.  K's 16-byte chunk c of row r lands at position
// c ^ (r mod CH) of the row (the lanes fetch permuted chunks), so the 16 rows
// of an operand read fall on distinct banks; V stays row-major.  Rows past
// the chunk fetch its last row again (their probabilities are 0).  The loads
// are inline asm, so the compiler neither counts them nor waits for them: the
// loading wave, which issues no other vector memory operation in its loop,
// counts them itself (wait_stage).  Nor does it look for hazards inside the
// asm: an LDS load may not directly follow the scalar write of M0 that gives
// its LDS address (one wait state), hence the s_nop.
template <typename M, bool SWIZZLE>
__device__ __forceinline__ void issue_block(const KvRows& kv, int tb, int c1, char* lds, int lane) {
  constexpr int D = M::D, CH = M::CH, RPI = 64 / CH, NI = M::BLK / RPI;
  int te;
  const typename M::E* r0 = M::block(kv, tb, c1, te);
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    const int row = k * RPI + lane / CH, c = lane % CH;
    const typename M::E* src = r0 + (size_t)(min(tb + row, c1 - 1) - te) * D +
                               (16 / sizeof(typename M::E)) * (SWIZZLE ? c ^ (row % CH) : c);
    const uint32_t at = __builtin_amdgcn_readfirstlane(lds_addr(lds + k * 1024));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"(src) : "memory", "m0");
  }
}
// Wait until at most `stages` later stages' loads (N per stage) are in flight.
template <int N>
__device__ __forceinline__ void wait_stage(int stages) {
  static_assert((kSlots - 2) * N < 64, "vmcnt holds 6 bits");
  if (stages <= 0)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else if (stages == 1)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * N) : "memory");
}

// log2-sum-exp of row n of a row tile over its nsp chunks, the lane groups
// taking the chunks in turn (+inf for padding rows and rows whose sum is not
// positive: their probabilities are then 0).
//
// WAIT: the records come from workgroups of the same launch.  A record's row
// is 0 until it is written (the finish kernel clears it again; a written one
// never is: its sum is positive, or its maximum -inf), so polling the records
// themselves is the exchange: no counter, no second round trip for the data.
template <bool WAIT>
__device__ __forceinline__ float tile_lse(const VArgs& a, int tile, bool real, int nsp, int n, int gq) {
  constexpr int kU = 8;
  const float2* st = a.stats + (size_t)tile * a.splits * 16 + n;
  float Mx = kNegInf, Z = 0.f;
  for (int s0 = 0; s0 < nsp; s0 += 4 * kU) {
    float2 v[kU];
    if constexpr (WAIT) {
      for (int spins = 0;; ++spins) {
        bool here = true;
#pragma unroll
        for (int j = 0; j < kU; ++j) v[j] = ld_agent(st + (size_t)min(s0 + gq + 4 * j, nsp - 1) * 16);
#pragma unroll
        for (int j = 0; j < kU; ++j) here &= __builtin_bit_cast(uint64_t, v[j]) != 0;
        if (__all(here)) break;
        if (spins > kSpinLimit) {
          dev_flag(a.status, PVLM_DEV_TIMEOUT);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    } else {
#pragma unroll
      for (int j = 0; j < kU; ++j) v[j] = st[(size_t)min(s0 + gq + 4 * j, nsp - 1) * 16];
    }
    float bm = kNegInf;
#pragma unroll
    for (int j = 0; j < kU; ++j) bm = fmaxf(bm, s0 + gq + 4 * j < nsp ? v[j].x : kNegInf);
    const float bref = bm == kNegInf ? 0.f : bm;
    float bz = 0.f;
#pragma unroll
    for (int j = 0; j < kU; ++j) bz += s0 + gq + 4 * j < nsp ? v[j].y * fast_exp2(v[j].x - bref) : 0.f;
    lse_combine(Mx, Z, bm, bz);
  }
  lse_combine(Mx, Z, lane_xor16(Mx), lane_xor16(Z));
  lse_combine(Mx, Z, lane_xor32(Mx), lane_xor32(Z));
  return real && Z > 0.f ? Mx + __log2f(Z) : __builtin_huge_valf();
}

// Sums of a block's probabilities over the 16 rows (lanes n) of a tile, one
// per token, into dst[token of the block].
__device__ __forceinline__ void rows_to_lds(const floatx4 (&p)[2], float* dst, int n, int gq) {
  // transpose-reduce: each step a lane keeps half of its values (chosen by
  // one bit of n) and adds the partner's copy of that half
  const bool h8 = n & 8, h4 = n & 4, h2 = n & 2;
  float a8[4], a4[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) a8[k] = (h8 ? p[1][k] : p[0][k]) + lane_xor8(h8 ? p[0][k] : p[1][k]);
#pragma unroll
  for (int k = 0; k < 2; ++k) a4[k] = (h4 ? a8[2 + k] : a8[k]) + lane_mirror8(h4 ? a8[k] : a8[2 + k]);
  float a2 = (h2 ? a4[1] : a4[0]) + lane_xor2(h2 ? a4[0] : a4[1]);
  a2 += lane_xor1(a2);
  if (!(n & 1)) dst[16 * (h8 ? 1 : 0) + 4 * gq + (h4 ? 2 : 0) + (h2 ? 1 : 0)] = a2;
}
__device__ __forceinline__ void rows_to_lds(const floatx4 (&p)[1], float* dst, int n, int gq) {
  const bool h8 = n & 8, h4 = n & 4;
  float a8[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) a8[k] = (h8 ? p[0][2 + k] : p[0][k]) + lane_xor8(h8 ? p[0][k] : p[0][2 + k]);
  float a4 = (h4 ? a8[1] : a8[0]) + lane_mirror8(h4 ? a8[0] : a8[1]);
  a4 += lane_xor2(a4);
  a4 += lane_xor1(a4);
  if (!(n & 3)) dst[4 * gq + (h8 ? 2 : 0) + (h4 ? 1 : 0)] = a4;
}

template <typename M, int RT>
struct PartShape {
  static constexpr int TW = RT <= 2 ? 2 : 1;            // waves sharing a row tile's tokens
  static constexpr int ST = 2 * M::BLK, NBW = 2 / TW;   // tokens of a stage, blocks of it per wave
  static constexpr int kThreads = (RT * TW + kLoaders) * 64;
  static constexpr int kHalf = ST * M::D * (int)sizeof(typename M::E);  // bytes of a stage's K (or V)
  static constexpr int kLds = kSlots * 2 * kHalf;
  static constexpr int kWpe = (kPerCu * (RT * TW + kLoaders) + 3) / 4;  // waves per SIMD
};

template <typename M, int RT, int RES>
__global__ void __launch_bounds__((PartShape<M, RT>::kThreads))
__attribute__((amdgpu_waves_per_eu(PartShape<M, RT>::kWpe, PartShape<M, RT>::kWpe))) verify_part_kernel(VArgs a) {
  typedef PartShape<M, RT> S_;
  constexpr int D = M::D, DPL = M::DPL, TT = M::TT, CH = M::CH, BLK = M::BLK, KS = M::KS;
  constexpr int TW = S_::TW, ST = S_::ST, NBW = S_::NBW, kHalf = S_::kHalf;
  __shared__ int32_t s_pages[kPageSlots];
  __shared__ float s_sum[RES ? RES : 1][RES ? RT : 1][ST];
  extern __shared__ __align__(1024) char s_ring[];  // [kSlots][K, V][ST][D]

  Unit u;
  if (!decode_unit(a, u)) return;
  const int lane = threadIdx.x & 63, n = lane & 15, gq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  KvRows kg, vg;
  kv_rows_setup<M>(a, u.b, u.g, u.c0, u.c1, s_pages, kg, vg);
  const int nst = (u.c1 - u.c0 + ST - 1) / ST;

  if (w >= RT * TW) {  // the loading waves
    const bool is_k = w == RT * TW;
    char* base = s_ring + (is_k ? 0 : kHalf);
    auto issue = [&](int s) {
      char* dst = base + (s % kSlots) * 2 * kHalf;
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        if (is_k) issue_block<M, true>(kg, u.c0 + s * ST + x * BLK, u.c1, dst + x * (kHalf / 2), lane);
        else issue_block<M, M::kSwizzleV>(vg, u.c0 + s * ST + x * BLK, u.c1, dst + x * (kHalf / 2), lane);
      }
    };
    __builtin_amdgcn_s_setprio(3);  // the loads go out before the other waves' arithmetic
    __builtin_amdgcn_s_waitcnt(0);  // the counts start from zero
    for (int s = 0; s < kSlots - 1 && s < nst; ++s) issue(s);
    for (int s = 0; s < nst; ++s) {
      wait_stage<kHalf / 1024>(min(kSlots - 2, nst - 1 - s));
      lds_sync();  // stage s has landed; every wave is done with stage s - 1
      if (s + kSlots - 1 < nst) issue(s + kSlots - 1);
    }
    if constexpr (TW > 1) {
      lds_sync();
      lds_sync();
    }
    if constexpr (RES > 0) {  // the loading waves sum the rows' mass and write it
      lds_sync();
      float* mp = a.mpart + ((size_t)u.bg * a.RG + u.rg) * a.n_cap;
      for (int s = is_k ? 0 : 1; s < nst; s += 2) {
        const int t = u.c0 + s * ST + lane;
        if (lane < ST && t < u.c1) {
          float sum = s_sum[s][0][lane];
#pragma unroll
          for (int r = 1; r < RT; ++r) sum += s_sum[s][r][lane];
          mp[t] = sum;
        }
      }
    }
    return;
  }

  const int rt = w / TW, tw = w % TW, gt = u.rg * RT + rt;  // row tile of the KV head
  const bool live = gt < a.RTT;
  const int row = gt * 16 + n;
  const int lim = row < a.R ? min(u.c1 - 1, u.ctx + row_t(a, row)) : -1;  // last token the lane's row sees
  const int vis_all = min(u.c1 - 1, u.ctx);                          // row 0 sees the least
  uint4 q[KS];
  {
    const uint4* p = reinterpret_cast<const uint4*>(q_row<M>(a, u.b, u.g, row));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = p[4 * ks + gq];
  }
  float ref = kNegInf, z = 0.f;
  floatx4 O[DPL];
#pragma unroll
  for (int jd = 0; jd < DPL; ++jd) O[jd] = floatx4{0.f, 0.f, 0.f, 0.f};
  // one stage: its raw (masked) scores, then the running statistics and O
  auto stage = [&](int s, auto& S) {
    lds_sync();
    const char* kb = s_ring + (s % kSlots) * 2 * kHalf + tw * NBW * (kHalf / 2);
    const char* vb = kb + kHalf;
    const int tb = u.c0 + s * ST + tw * NBW * BLK;
    if (tb >= u.c1 || !live) return;
    // every operand read of the stage before its first use (the compiler
    // would otherwise wait out one LDS latency per matrix instruction)
    uint4 kr[NBW][TT][KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const int r = 16 * tt + n;
          kr[x][tt][ks] =
              *reinterpret_cast<const uint4*>(kb + x * (kHalf / 2) + (r * CH + ((4 * ks + gq) ^ (r % CH))) * 16);
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < NBW; ++x)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) S[x][tt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) S[x][tt] = M::qk(kr[x][tt][ks], q[ks], S[x][tt]);
    typename M::V V[NBW];
#pragma unroll
    for (int x = 0; x < NBW; ++x) M::read_v(vb + x * (kHalf / 2), n, gq, V[x]);
    __builtin_amdgcn_sched_barrier(0);
    if (tb + NBW * BLK - 1 > vis_all) {
      const int off = lim - tb - 4 * gq;  // element (x, tt, i) visible iff BLK x + 16 tt + i <= off
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (BLK * x + 16 * tt + i > off) S[x][tt][i] = kNegInf;
    }
    float mx = kNegInf;
#pragma unroll
    for (int x = 0; x < NBW; ++x)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
        mx = fmaxf(fmaxf(mx, fmaxf(S[x][tt][0], S[x][tt][1])), fmaxf(S[x][tt][2], S[x][tt][3]));
    mx = rows4_max(mx) * a.sl2;
    if (__any(mx > ref + kRefSlack)) {  // the first stage, and seldom after it
      const float nm = fmaxf(ref, mx);
      const float al = ref == kNegInf ? 0.f : fast_exp2(ref - nm);
      z *= al;
      ref = nm;
      floatx4 f;
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = __shfl(al, 4 * gq + i, 64);
#pragma unroll
      for (int jd = 0; jd < DPL; ++jd) O[jd] = O[jd] * f;
    }
    floatx4 P[NBW][TT];
    const float r0 = ref == kNegInf ? 0.f : ref;  // no visible token yet: P = 0
#pragma unroll
    for (int x = 0; x < NBW; ++x)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = fast_exp2(fmaf(S[x][tt][i], a.sl2, -r0));
          P[x][tt][i] = p;
          z += p;
        }
#pragma unroll
    for (int x = 0; x < NBW; ++x) M::pv(P[x], V[x], O);
  };
  floatx4 Sr[RES ? RES : 1][NBW][TT];
  if constexpr (RES > 0) {
#pragma unroll
    for (int s = 0; s < RES; ++s) {
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) Sr[s][x][tt] = floatx4{kNegInf, kNegInf, kNegInf, kNegInf};
      if (s < nst) stage(s, Sr[s]);
    }
  } else {
    for (int s = 0; s < nst; ++s) stage(s, Sr[0]);
  }

  z = rows4_sum(z);
  if constexpr (TW > 1) {  // the second token wave's sums join the first's
    floatx4* xo = reinterpret_cast<floatx4*>(s_ring) + rt * (DPL * 64 + 64);
    lds_sync();
    if (tw == 1) {
#pragma unroll
      for (int jd = 0; jd < DPL; ++jd) xo[jd * 64 + lane] = O[jd];
      xo[DPL * 64 + lane] = floatx4{ref, z, 0.f, 0.f};
    }
    lds_sync();
    if (RES == 0 && tw == 1) return;
    if (tw == 0) {
      const floatx4 o = xo[DPL * 64 + lane];
      const float Mx = fmaxf(ref, o[0]);
      const float f0 = ref == kNegInf ? 0.f : fast_exp2(ref - Mx);
      const float f1 = o[0] == kNegInf ? 0.f : fast_exp2(o[0] - Mx);
      z = z * f0 + o[1] * f1;
      ref = Mx;
      floatx4 g0, g1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        g0[i] = __shfl(f0, 4 * gq + i, 64);
        g1[i] = __shfl(f1, 4 * gq + i, 64);
      }
#pragma unroll
      for (int jd = 0; jd < DPL; ++jd) O[jd] = O[jd] * g0 + xo[jd * 64 + lane] * g1;
    }
  }
  const int tile = u.bg * a.RTT + gt;
  const size_t rec = (size_t)tile * a.splits + u.split;
  if (live && tw == 0) {
    if (gq == 0) {
      if constexpr (RES > 0) st_agent(a.stats + rec * 16 + n, make_float2(ref, z));
      else a.stats[rec * 16 + n] = make_float2(ref, z);
    }
    auto store_o = [&](auto* op) {
      op += rec * 16 * D;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < DPL / 4; ++h) {
          const float x[4] = {O[4 * h][i], O[4 * h + 1][i], O[4 * h + 2][i], O[4 * h + 3][i]};
          store4(op + (4 * gq + i) * D + DPL * n + 4 * h, x);
        }
    };
    if (a.o32) store_o(static_cast<float*>(a.opart));
    else store_o(static_cast<typename M::E*>(a.opart));
  }
  if constexpr (RES > 0) {
    // the rows' log-sum-exp over the launch's chunks, then the exact
    // probabilities of the resident scores
    const float lse = live ? tile_lse<true>(a, tile, row < a.R, (u.N + a.chunk - 1) / a.chunk, n, gq)
                           : __builtin_huge_valf();
#pragma unroll
    for (int s = 0; s < RES; ++s)
      if (s < nst) {
#pragma unroll
        for (int x = 0; x < NBW; ++x) {
#pragma unroll
          for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) Sr[s][x][tt][i] = fast_exp2(fmaf(Sr[s][x][tt][i], a.sl2, -lse));
          rows_to_lds(Sr[s][x], &s_sum[s][rt][(tw * NBW + x) * BLK], n, gq);
        }
      }
    lds_sync();
  }
}

// ----------------------------------------------------------- mass kernel --
// The partial kernel's units again, with every row's log-sum-exp known: the
// chunk's K passes through the ring once more, a wave per row tile forms the
// exact probabilities, and the tokens' sums over the workgroup's rows meet in
// LDS, from where the last wave writes them.  The stages go backwards: the
// rows the partial kernel read last are the ones still cached.
template <typename M, int RT>
__global__ void __launch_bounds__((PartShape<M, RT>::kThreads))
__attribute__((amdgpu_waves_per_eu(PartShape<M, RT>::kWpe, PartShape<M, RT>::kWpe))) verify_mass_kernel(VArgs a) {
  typedef PartShape<M, RT> S_;
  constexpr int D = M::D, TT = M::TT, CH = M::CH, BLK = M::BLK, KS = M::KS;
  constexpr int TW = S_::TW, ST = S_::ST, NBW = S_::NBW, kHalf = S_::kHalf;
  __shared__ int32_t s_pages[kPageSlots];
  __shared__ float s_sum[2][RT][ST];
  extern __shared__ __align__(1024) char s_ring[];  // [kSlots][ST][D]

  Unit u;
  if (!decode_unit(a, u)) return;
  const int lane = threadIdx.x & 63, n = lane & 15, gq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  KvRows kg, vg;
  kv_rows_setup<M>(a, u.b, u.g, u.c0, u.c1, s_pages, kg, vg);
  const int nst = (u.c1 - u.c0 + ST - 1) / ST;
  if (w == RT * TW) {  // the loading wave
    auto issue = [&](int s) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
        issue_block<M, true>(kg, u.c0 + (nst - 1 - s) * ST + x * BLK, u.c1, s_ring + (s % kSlots) * kHalf + x * (kHalf / 2), lane);
    };
    __builtin_amdgcn_s_setprio(3);  // the loads go out before the other waves' arithmetic
    __builtin_amdgcn_s_waitcnt(0);  // the counts start from zero
    for (int s = 0; s < kSlots - 1 && s < nst; ++s) issue(s);
    for (int s = 0; s < nst; ++s) {
      wait_stage<kHalf / 1024>(min(kSlots - 2, nst - 1 - s));
      lds_sync();
      if (s + kSlots - 1 < nst) issue(s + kSlots - 1);
    }
    lds_sync();
    return;
  }
  if (w > RT * TW) {  // the summing wave: stage s - 1's sums after stage s's barrier
    float* mp = a.mpart + ((size_t)u.bg * a.RG + u.rg) * a.n_cap;
    lds_sync();
    for (int s = 0; s < nst; ++s) {
      lds_sync();
      const int t = u.c0 + (nst - 1 - s) * ST + lane;
      if (lane < ST && t < u.c1) {
        float sum = s_sum[s & 1][0][lane];
#pragma unroll
        for (int r = 1; r < RT; ++r) sum += s_sum[s & 1][r][lane];
        mp[t] = sum;
      }
    }
    return;
  }

  const int rt = w / TW, tw = w % TW, gt = u.rg * RT + rt;
  const int row = gt * 16 + n;
  const int lim = row < a.R ? min(u.c1 - 1, u.ctx + row_t(a, row)) : -1;
  const int vis_all = min(u.c1 - 1, u.ctx);
  uint4 q[KS];
  {
    const uint4* p = reinterpret_cast<const uint4*>(q_row<M>(a, u.b, u.g, row));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = p[4 * ks + gq];
  }
  const float lse = tile_lse<false>(a, u.bg * a.RTT + min(gt, a.RTT - 1), row < a.R, (u.N + a.chunk - 1) / a.chunk, n, gq);
  for (int s = 0; s < nst; ++s) {
    lds_sync();
    const char* kb = s_ring + (s % kSlots) * kHalf + tw * NBW * (kHalf / 2);
    const int tb = u.c0 + (nst - 1 - s) * ST + tw * NBW * BLK;
    uint4 kr[NBW][TT][KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const int r = 16 * tt + n;
          kr[x][tt][ks] =
              *reinterpret_cast<const uint4*>(kb + x * (kHalf / 2) + (r * CH + ((4 * ks + gq) ^ (r % CH))) * 16);
        }
    __builtin_amdgcn_sched_barrier(0);
    floatx4 S[NBW][TT];
#pragma unroll
    for (int x = 0; x < NBW; ++x)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) S[x][tt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) S[x][tt] = M::qk(kr[x][tt][ks], q[ks], S[x][tt]);
    if (tb + NBW * BLK - 1 > vis_all) {
      const int off = lim - tb - 4 * gq;
#pragma unroll
      for (int x = 0; x < NBW; ++x)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (BLK * x + 16 * tt + i > off) S[x][tt][i] = kNegInf;
    }
#pragma unroll
    for (int x = 0; x < NBW; ++x) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[x][tt][i] = fast_exp2(fmaf(S[x][tt][i], a.sl2, -lse));
      rows_to_lds(S[x], &s_sum[s & 1][rt][(tw * NBW + x) * BLK], n, gq);
    }
  }
  lds_sync();
}

// --------------------------------------------------------- finish kernel --
// One row of O: the sum over its chunks of the partials weighted by
// exp2(chunk max - row max) / row sum, and the row's log-sum-exp.  64 / LPR
// lane sets take the chunks in turn, 16 bytes per lane and chunk.
template <typename M, typename PT>
__device__ void combine_row(const VArgs& a, int64_t id) {
  constexpr int D = M::D, PC = 16 / sizeof(PT), LPR = D / PC, SG = 64 / LPR, kU = 8;
  static_assert(64 % (kU * SG) == 0, "a batch of chunks shares one weight register");
  if (id >= (int64_t)a.B * a.Hkv * a.R) return;
  const int lane = threadIdx.x & 63, sg = lane / LPR, col = lane % LPR;
  const int bg = (int)(id / a.R), row = (int)(id - (int64_t)bg * a.R);
  const int b = bg / a.Hkv, g = bg - b * a.Hkv;
  const int N = seq_ctx(a, b, false) + a.T;
  const int nsp = (N + a.chunk - 1) / a.chunk;
  const size_t rec = ((size_t)bg * a.RTT + row / 16) * a.splits * 16 + row % 16;
  const float2* st = a.stats + rec;
  const uint4* op = reinterpret_cast<const uint4*>(static_cast<const PT*>(a.opart) + rec * D) + col;
  const size_t os = (size_t)16 * LPR;  // 16-byte pieces between chunks
  // the first kU pieces load together with the statistics
  uint4 v[kU];
#pragma unroll
  for (int j = 0; j < kU; ++j) v[j] = op[min(sg + j * SG, nsp - 1) * os];
  // the statistics of 256 chunks at a time, all in flight together: few rows
  // over many chunks are bound by this wave's round trips (18 rows over 247
  // chunks, us a layer with the rotary append: 24.1 with 64 at a time and a
  // second read, 22.0 this way)
  constexpr int kC = 4;
  float2 x[kC];
  auto load_stats = [&](int s0) {
#pragma unroll
    for (int c = 0; c < kC; ++c)
      if (c == 0 || s0 + 64 * c < nsp) x[c] = st[(size_t)min(s0 + 64 * c + lane, nsp - 1) * 16];
#pragma unroll
    for (int c = 0; c < kC; ++c)
      if (s0 + 64 * c + lane >= nsp) x[c] = make_float2(kNegInf, 0.f);
  };
  float Mx = kNegInf, Z = 0.f;
  for (int s0 = 0; s0 < nsp; s0 += 64 * kC) {
    load_stats(s0);
    float m = x[0].x;
#pragma unroll
    for (int c = 1; c < kC; ++c) m = fmaxf(m, x[c].x);
    const float bm = warp_max(m);
    float e = 0.f;
#pragma unroll
    for (int c = 0; c < kC; ++c) e += x[c].x == kNegInf ? 0.f : x[c].y * fast_exp2(x[c].x - bm);
    lse_combine(Mx, Z, bm, warp_sum(e));
  }
  const bool ok = Z > 0.f;
  const float inv = ok ? 1.f / Z : 0.f;
  float acc[PC];
#pragma unroll
  for (int c = 0; c < PC; ++c) acc[c] = 0.f;
  for (int s0 = 0; s0 < nsp; s0 += 64 * kC) {
    if (nsp > 64 * kC) load_stats(s0);
    float wt[kC];
#pragma unroll
    for (int c = 0; c < kC; ++c) wt[c] = x[c].x == kNegInf ? 0.f : fast_exp2(x[c].x - Mx) * inv;
    const int cnt = min(64 * kC, nsp - s0);
    for (int k0 = 0; k0 < cnt; k0 += kU * SG) {  // kU * SG divides 64
      if (s0 + k0 > 0) {
#pragma unroll
        for (int j = 0; j < kU; ++j) v[j] = op[min(s0 + k0 + sg + j * SG, nsp - 1) * os];
      }
      const int kc = k0 / 64;  // uniform
      const float w = kc == 0 ? wt[0] : kc == 1 ? wt[1] : kc == 2 ? wt[2] : wt[3];
#pragma unroll
      for (int j = 0; j < kU; ++j) {
        const int s = k0 + sg + j * SG;
        const float f = __shfl(w, s & 63, 64);
        float p[PC];
        unpack(v[j], p);
#pragma unroll
        for (int c = 0; c < PC; ++c) acc[c] = s < cnt ? fmaf(f, p[c], acc[c]) : acc[c];
      }
    }
  }
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
    for (int c = 0; c < PC; ++c) acc[c] += __shfl_xor(acc[c], o, 64);
  const int t = row_t(a, row), h = g * a.G + row - t * a.G;
  if (a.clear) {  // the records' rows (the tile's last real row also clears the padding rows)
    const int rows = row == a.R - 1 ? 16 - row % 16 : 1;
    for (int r = 0; r < rows; ++r)
      for (int s = lane; s < nsp; s += 64) a.stats[rec + (size_t)s * 16 + r] = make_float2(0.f, 0.f);
  }
  if (sg == 0) {
    typename M::E* o = static_cast<typename M::E*>(a.out) + (((size_t)b * a.T + t) * a.Hq + h) * D;
#pragma unroll
    for (int c = 0; c < PC; ++c) M::store_out(o, PC * col + c, acc[c]);
  }
  if (a.lse && lane == 0)
    a.lse[((size_t)b * a.Hq + h) * a.T + t] = ok ? (Mx + __log2f(Z)) * kLn2 : __builtin_huge_valf();
}

// The mass of every cache row: the sum of its KV heads' and row groups'
// partials in order (0 past the sequence).
__device__ __forceinline__ void sum_mass(const VArgs& a, int id) {
  constexpr int kP = 8;
  const int P = a.Hkv * a.RG;
  const int b = id / a.mass_per;
  const int64_t t0 = (int64_t)(id - b * a.mass_per) * a.mass_rows;
  const int N = seq_ctx(a, b, false) + a.T;
  const float* mp = a.mpart + (size_t)b * P * a.n_cap;
  float* mass = a.mass + (size_t)b * a.n_cap;
  for (int64_t t = t0 + threadIdx.x; t < min(t0 + a.mass_rows, a.n_cap); t += kFinThreads) {
    float sum = 0.f;
    if (t < N)
      for (int p0 = 0; p0 < P; p0 += kP) {
        float v[kP];
#pragma unroll
        for (int j = 0; j < kP; ++j) v[j] = mp[(size_t)min(p0 + j, P - 1) * a.n_cap + t];
#pragma unroll
        for (int j = 0; j < kP; ++j)
          if (p0 + j < P) sum += v[j];
      }
    mass[t] = sum;
  }
}

template <typename M>
__global__ void __launch_bounds__(kFinThreads) verify_finish_kernel(VArgs a) {
  const int id = blockIdx.x;
  if (id < a.mass_wgs) sum_mass(a, id);
  else if (a.o32) combine_row<M, float>(a, (int64_t)(id - a.mass_wgs) * kFinWaves + (threadIdx.x >> 6));
  else combine_row<M, typename M::E>(a, (int64_t)(id - a.mass_wgs) * kFinWaves + (threadIdx.x >> 6));
}

// -------------------------------------------------- allocation-free entry --
// The scratch buffer of pvlm_verify_attn_noalloc: a file-scope device array
// that every call on a device shares (each device holds its own copy for the
// life of the process).  Host code never uses this name as an address: the
// device address comes from hipGetSymbolAddress, once per device.
constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

__global__ void __launch_bounds__(256) zero_words_kernel(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

// ------------------------------------------------------------------ host --
typedef void (*VKernel)(VArgs);

struct VPlan : VSplit {
  int threads, lds, mass_lds;  // partial and mass kernels
  VKernel part, fused, mass, finish;  // fused: NULL if the chunk is not resident
};

// Most stages of a chunk whose scores a wave keeps in registers: 16 per stage
// and lane (8 where two waves share a row tile) beside the ~130 of the stage
// itself, out of 512 (one wave per SIMD), 256 or 168.
template <int RT>
struct Resident {
  static constexpr int stages = RT == 1 ? 20 : RT == 2 ? 12 : RT <= 6 ? 7 : 0;
};

template <typename M, int RT>
void set_part(VPlan* p) {
  p->part = verify_part_kernel<M, RT, 0>;
  const int st = p->chunk / PartShape<M, RT>::ST;
  p->fused = nullptr;
  constexpr int kRes = Resident<RT>::stages;
  if constexpr (kRes > 0) {
    if (st <= 2) p->fused = verify_part_kernel<M, RT, 2>;
    else if (st <= 7) p->fused = verify_part_kernel<M, RT, 7>;
    else if constexpr (kRes > 7) {
      if (st <= kRes) p->fused = verify_part_kernel<M, RT, kRes>;
    }
  }
  p->threads = PartShape<M, RT>::kThreads;
  p->lds = PartShape<M, RT>::kLds;
  p->mass = verify_mass_kernel<M, RT>;
  p->mass_lds = p->lds / 2;
}
template <typename M>
void pick_kernels(VPlan* p) {
  switch (p->RT) {
    case 1: set_part<M, 1>(p); break;
    case 2: set_part<M, 2>(p); break;
    case 3: set_part<M, 3>(p); break;
    case 4: set_part<M, 4>(p); break;
    case 5: set_part<M, 5>(p); break;
    case 6: set_part<M, 6>(p); break;
    case 7: set_part<M, 7>(p); break;
    case 8: set_part<M, 8>(p); break;
    default: set_part<M, 9>(p); break;
  }
  p->finish = verify_finish_kernel<M>;
}

// stream: the launch's stream, whose compute-unit budget bounds the plan;
// with_stream false plans for the whole device (workspace sizes, enough for
// every budget).
pvlm_status plan_verify(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D, int64_t n_cap,
                        int64_t max_ctx, VPlan* p, hipStream_t stream, bool with_stream) {
  pvlm_status st = check_verify(dt, B, T, Hq, Hkv, D, n_cap, max_ctx);
  if (st != PVLM_OK) return st;
  DeviceInfo whole, di;
  st = device_info(&whole);
  if (st != PVLM_OK) return st;
  di = whole;
  if (with_stream) st = device_info(&di, stream);
  if (st != PVLM_OK) return st;
  st = split_verify(dt, B, T, Hq, Hkv, D, n_cap, max_ctx, whole, di, p);
  if (st != PVLM_OK) return st;
  if (dt == PVLM_BF16) {
    if (D == 128) pick_kernels<Bf16<128>>(p);
    else pick_kernels<Bf16<64>>(p);
  } else {
    if (D == 128) pick_kernels<F32<128>>(p);
    else pick_kernels<F32<64>>(p);
  }
  return PVLM_OK;
}

}  // namespace
}  // namespace pvlm

using namespace pvlm;

extern "C" size_t pvlm_verify_attn_workspace_size(pvlm_dtype dt, int B, int T, int Hq, int Hkv,
                                                  int D, int64_t n_cap, int64_t max_ctx) {
  VPlan p;
  if (plan_verify(dt, B, T, Hq, Hkv, D, n_cap, max_ctx, &p, nullptr, false) != PVLM_OK) return 0;
  return p.bytes;
}

namespace {
// The cache rows come from a padded cache (table == NULL) or through a page
// table into a page pool (logical capacity n_cap = max_pages << page_shift).
pvlm_status verify_run(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D, int64_t n_cap,
                       int64_t max_ctx, float scale, const void* q, const void* k_cache,
                       const void* v_cache, const int32_t* table, int64_t n_pages, int max_pages,
                       int page_shift, const int32_t* ctx_len, void* out, float* mass, float* lse,
                       void* ws, size_t ws_bytes, int32_t* status, hipStream_t stream) {
  if (!q || !k_cache || !v_cache || !ctx_len || !out) return PVLM_ERR_NULL;
  if (!(scale > 0.f) || !std::isfinite(scale)) return PVLM_ERR_SHAPE;
  VPlan p;
  pvlm_status st = plan_verify(dt, B, T, Hq, Hkv, D, n_cap, max_ctx, &p, stream, true);
  if (st != PVLM_OK) return st;
  if (!ws) return PVLM_ERR_WORKSPACE;
  if (ws_bytes < p.bytes) return PVLM_ERR_WORKSPACE;
  char* wsb = static_cast<char*>(ws);
  VArgs a;
  a.q = q;
  a.k = k_cache;
  a.v = v_cache;
  a.ctx_len = ctx_len;
  a.table = table;
  a.n_pages = n_pages;
  a.max_pages = max_pages;
  a.page_shift = page_shift;
  a.stats = reinterpret_cast<float2*>(wsb + p.off_stats);
  a.mpart = reinterpret_cast<float*>(wsb + p.off_mpart);
  a.opart = wsb + p.off_opart;
  a.out = out;
  a.lse = lse;
  a.mass = mass;
  a.status = status;
  a.n_cap = n_cap;
  a.B = B;
  a.T = T;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.G = p.G;
  a.g_magic = (1u << 20) / (unsigned)p.G + 1u;
  a.R = p.R;
  a.RG = p.RG;
  a.RTT = p.RTT;
  a.max_ctx = (int)max_ctx;
  a.splits = p.splits;
  a.chunk = p.chunk;
  a.units = B * Hkv * p.RG * p.splits;
  a.sl2 = scale * kLog2e;
  a.o32 = p.o32;
  a.mass_rows = (int)mass_rows(B, n_cap);
  a.mass_per = (int)mass_workgroups(n_cap, a.mass_rows);
  a.mass_wgs = mass ? B * a.mass_per : 0;
  const int comb_wgs = (B * Hkv * p.R + kFinWaves - 1) / kFinWaves;
  // While a stream is captured, a call whose chunks' scores stay in registers
  // is one waiting launch; otherwise the mass is a second pass over K.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  PVLM_HIP(hipStreamIsCapturing(stream, &cap));
  const dim3 grid((a.units + 7) / 8 * 8), block(p.threads);
  const int64_t records = (int64_t)B * Hkv * p.RTT * p.splits;
  a.clear = false;
  void* args[] = {&a};
  if (mass && p.fused && cap != hipStreamCaptureStatusNone && 128 * records <= (int64_t)(kSyncTopkOff - kSyncVerifyOff)) {
    const void* k = reinterpret_cast<const void*>(p.fused);
    PVLM_HIP(allow_dynamic_lds(k, p.lds));
    if (check_coresident(k, (int)grid.x, p.threads, p.lds, kPerCu, stream) == PVLM_OK) {
      a.clear = true;
      a.stats = reinterpret_cast<float2*>(wsb + kSyncVerifyOff);
      PVLM_HIP(hipLaunchKernel(k, grid, block, args, p.lds, stream));
    }
  }
  if (!a.clear) {
    const void* part = reinterpret_cast<const void*>(p.part);
    PVLM_HIP(allow_dynamic_lds(part, p.lds));
    PVLM_HIP(hipLaunchKernel(part, grid, block, args, p.lds, stream));
    if (mass) {
      const void* mk = reinterpret_cast<const void*>(p.mass);
      PVLM_HIP(allow_dynamic_lds(mk, p.mass_lds));
      PVLM_HIP(hipLaunchKernel(mk, grid, block, args, p.mass_lds, stream));
    }
  }
  PVLM_HIP(hipLaunchKernel(reinterpret_cast<const void*>(p.finish), dim3(a.mass_wgs + comb_wgs),
                           dim3(kFinThreads), args, 0, stream));
  return PVLM_OK;
}
}  // namespace

extern "C" pvlm_status pvlm_verify_attn(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D,
                                        int64_t n_cap, int64_t max_ctx, float scale, const void* q,
                                        const void* k_cache, const void* v_cache,
                                        const int32_t* ctx_len, void* out, float* mass, float* lse,
                                        void* ws, size_t ws_bytes, int32_t* status,
                                        hipStream_t stream) {
  return verify_run(dt, B, T, Hq, Hkv, D, n_cap, max_ctx, scale, q, k_cache, v_cache, nullptr, 0, 0,
                    0, ctx_len, out, mass, lse, ws, ws_bytes, status, stream);
}

extern "C" pvlm_status pvlm_verify_attn_paged(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D,
                                              int page_size, int max_pages, int64_t n_pages,
                                              int64_t max_ctx, float scale, const void* q,
                                              const void* k_pool, const void* v_pool,
                                              const int32_t* page_table, const int32_t* ctx_len,
                                              void* out, float* mass, float* lse, void* ws,
                                              size_t ws_bytes, int32_t* status,
                                              hipStream_t stream) {
  if (!page_table) return PVLM_ERR_NULL;
  const int shift = page_shift_of(page_size);
  if (shift < 0 || max_pages < 1 || n_pages < 1 || n_pages > INT32_MAX) return PVLM_ERR_SHAPE;
  if (dt != PVLM_BF16) return PVLM_ERR_UNSUPPORTED;
  return verify_run(dt, B, T, Hq, Hkv, D, (int64_t)max_pages << shift, max_ctx, scale, q, k_pool,
                    v_pool, page_table, n_pages, max_pages, shift, ctx_len, out, mass, lse, ws,
                    ws_bytes, status, stream);
}

namespace {
std::mutex g_scratch_mu;
void* g_scratch[64] = {nullptr};  // device address of `scratch` per device
}  // namespace

extern "C" size_t pvlm_verify_attn_noalloc_max_bytes(void) { return kScratchBytes; }

extern "C" pvlm_status pvlm_verify_attn_noalloc(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D,
                                                int64_t n_cap, int64_t max_ctx, float scale,
                                                const void* q, const void* k_cache,
                                                const void* v_cache, const int32_t* ctx_len,
                                                void* out, float* mass, float* lse, int32_t* status,
                                                hipStream_t stream) {
  if (!q || !k_cache || !v_cache || !ctx_len || !out) return PVLM_ERR_NULL;
  if (!(scale > 0.f) || !std::isfinite(scale)) return PVLM_ERR_SHAPE;
  VPlan p;
  pvlm_status st = plan_verify(dt, B, T, Hq, Hkv, D, n_cap, max_ctx, &p, stream, true);
  if (st != PVLM_OK) return st;
  if (p.bytes > kScratchBytes) return PVLM_ERR_WORKSPACE;  // beyond the fixed scratch
  int dev = 0;
  PVLM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return PVLM_ERR_UNSUPPORTED;
  void* ptr = nullptr;
  bool first = false;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
      void* a = nullptr;
      PVLM_HIP(hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)));
      if (!a) return PVLM_ERR_HIP;
      g_scratch[dev] = a;
      first = true;
    }
    ptr = g_scratch[dev];
  }
  if (first) {  // the synchronisation region starts at zero (a fill kernel, so
                // a capturing caller records no memset node)
    hipLaunchKernelGGL(zero_words_kernel, dim3(256), dim3(256), 0, stream, static_cast<uint32_t*>(ptr),
                       kSyncRegion / sizeof(uint32_t));
    PVLM_LAUNCHED();
  }
  return pvlm_verify_attn(dt, B, T, Hq, Hkv, D, n_cap, max_ctx, scale, q, k_cache, v_cache, ctx_len,
                          out, mass, lse, ptr, kScratchBytes, status, stream);
}
