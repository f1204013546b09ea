// Launch plan of verify attention: how its row tiles and tokens are split over
// workgroups, and where the workspace's areas lie.  Plain C++, so that the plan
// can be run over all sizes without a GPU.
#pragma once

#include <cstddef>
#include <cstdint>

#include "layout.h"
#include "pvlm.h"

namespace pvlm {

constexpr int kMaxRT = 9;  // 16-row tiles per workgroup of the partial kernel
// Workgroups of the partial and mass kernels that a compute unit holds, at
// either head dim: their waves-per-SIMD bound makes them reserve a unit's
// registers (two tiles reserve 176 of a lane's 512 for each of six waves), and
// at D = 128 their ring takes its LDS.  The runtime's occupancy figure counts
// the registers they use, so a launch that waits has to go by this one.  With
// two planned at D = 64 a call ran in two rounds (18 rows over 63K tokens,
// captured, us a layer: 18.7 without mass, against 14.6 with one).
constexpr int kPerCu = 1;

struct VSplit {
  int G, R, RTT, RG, RT;
  int splits, chunk;
  int slots;  // workgroups of the partial kernel that run at once
  bool o32;
  size_t off_stats, off_opart, off_mpart, bytes;
};

// The workspace size that callers are told (for the whole device): a bound
// that every plan below keeps within, a function of the sizes and the compute units alone, so that
// buffers sized by it and the fixed scratch take the same calls whatever the
// split.  Per group one statistics record and one fp32-sized partial for
// each of `splits` chunks, and one mass row per KV head and row group.
inline size_t workspace_bound(bool bf16, int B, int Hkv, int D, int RTT, int64_t n_cap, int64_t n_plan,
                              const DeviceInfo& di, bool* ok) {
  int RG = (RTT + 4) / 5;
  if (bf16 && B * Hkv * RG < di.xcds && RTT > RG) {
    const int want = (di.xcds + B * Hkv - 1) / (B * Hkv);
    RG = want < RTT ? want : RTT;
  }
  int RT = (RTT + RG - 1) / RG, W = di.cus;
  int64_t groups, chunk, splits;
  auto layout = [&]() {
    groups = (int64_t)B * Hkv * RG;
    splits = W / (groups < W ? groups : W);
    if (!bf16 && splits > (n_plan + 63) / 64) splits = (n_plan + 63) / 64;
    chunk = ((n_plan + splits - 1) / splits + 31) / 32 * 32;
    splits = (n_plan + chunk - 1) / chunk;
  };
  layout();
  if (bf16 && chunk > 512 && RTT > 5 && RTT <= 9 && B * Hkv >= di.xcds) {
    RG = 1;
    RT = 9;
    if (!di.budgeted) W = 2 * di.cus;
    layout();
  }
  // the limits of earlier plans, which kept a line of counters per group and
  // per chunk in the fixed region: no call is taken beyond them
  *ok = 3 * kSyncLine * (size_t)groups <= kSyncTopkOff - kSyncVerifyOff &&
        kSyncLine * (size_t)B * splits <= kSyncVerifyOff;
  const size_t rows = (size_t)RT * 16;
  size_t bytes = kSyncRegion;
  bytes = align_up(bytes + 8 * (size_t)groups * splits * ((rows + 16) / 16 * 16), 256);
  bytes = align_up(bytes + 4 * (size_t)groups * splits * rows * D, 256);
  return align_up(bytes + 4 * (size_t)B * Hkv * RG * n_cap, 256);
}

// The sizes that no device takes, before the device is asked for.
inline pvlm_status check_verify(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D, int64_t n_cap,
                                int64_t max_ctx) {
  if (dt != PVLM_F32 && dt != PVLM_BF16) return PVLM_ERR_UNSUPPORTED;
  if (B < 1 || T < 1 || Hq < 1 || Hkv < 1 || n_cap < 1) return PVLM_ERR_SHAPE;
  if (T > 32 || Hq % Hkv != 0 || (D != 64 && D != 128)) return PVLM_ERR_UNSUPPORTED;
  if (max_ctx < 0 || max_ctx + T > n_cap || n_cap > (int64_t)1 << 30) return PVLM_ERR_SHAPE;
  return (int64_t)(Hq / Hkv) * T > 640 ? PVLM_ERR_UNSUPPORTED : PVLM_OK;
}

// Finish kernel: cache rows whose mass one workgroup sums, and the workgroups of
// a sequence.  kFinThreads rows each, unless that takes more workgroups than
// kMassWgs in all: a launch holds fewer than 2^32 threads.
constexpr int kFinThreads = 256;
constexpr int64_t kMassWgs = 1 << 16;
inline int64_t mass_rows(int B, int64_t n_cap) {
  const int64_t wgs = B < kMassWgs ? kMassWgs / B : 1, rows = (n_cap + wgs - 1) / wgs;
  return (rows + kFinThreads - 1) / kFinThreads * kFinThreads;
}
inline int64_t mass_workgroups(int64_t n_cap, int64_t rows) { return (n_cap + rows - 1) / rows; }

// The plan on a device, or on a stream's budget `di` of a device `whole`, for
// arguments that check_verify takes.
inline pvlm_status split_verify(pvlm_dtype dt, int B, int T, int Hq, int Hkv, int D, int64_t n_cap, int64_t max_ctx,
                                const DeviceInfo& whole, const DeviceInfo& di, VSplit* p) {
  p->G = Hq / Hkv;
  p->R = p->G * T;
  const bool bf16 = dt == PVLM_BF16;
  const int64_t n_plan = max_ctx + T;
  p->RTT = (p->R + 15) / 16;
  bool ok;
  p->bytes = workspace_bound(bf16, B, Hkv, D, p->RTT, n_cap, n_plan, di, &ok);
  if (!ok) return PVLM_ERR_UNSUPPORTED;
  if (di.budgeted) {
    // callers size a workspace for the whole device, whose bound can be the
    // smaller one (six to nine tiles in chunks that only the budget makes long)
    bool whole_ok;
    const size_t sized = workspace_bound(bf16, B, Hkv, D, p->RTT, n_cap, n_plan, whole, &whole_ok);
    if (whole_ok && sized < p->bytes) p->bytes = sized;
  }
  p->RG = (p->RTT + kMaxRT - 1) / kMaxRT;
  p->RT = (p->RTT + p->RG - 1) / p->RG;
  const int blk = bf16 ? 32 : 16, e = bf16 ? 2 : 4;
  const int64_t tiles = (int64_t)B * Hkv * p->RTT;
  // chunks of whole stages (two blocks)
  const int64_t nst = (n_plan + 2 * blk - 1) / (2 * blk), slots = (int64_t)di.cus * kPerCu;
  p->slots = (int)slots;
  // One workgroup per compute unit, all of them in one round (as many chunks as
  // every group has compute units for: one workgroup more runs alone in a
  // second round; batch of three, 8 KV heads, 16K tokens: 264 workgroups 82 us a
  // layer, 240 68), and at least two stages each: fewer only add partials.
  auto chunk_stages = [&](int64_t groups) {
    const int64_t most = slots > groups ? slots / groups : 1, cs = (nst + most - 1) / most;
    return cs < 2 ? (int64_t)2 : cs;
  };
  const int64_t heads = (int64_t)B * Hkv;
  const size_t per_split = (size_t)tiles * 16 * (8 + (size_t)D * e);
  const int rg6 = (p->RTT + 5) / 6;
  if (p->RT > 6 && heads * rg6 <= slots && chunk_stages(heads * rg6) <= 7) {
    // Seven row tiles or more leave a wave 168 registers: no room for resident
    // scores.  Chunks that stay within seven stages with up to six tiles go to
    // more workgroups (K and V read again, from L2); longer ones would pay for
    // that (131K tokens, 9 tiles as 5 and 4: 256 us against 209).
    const int64_t cs = chunk_stages(heads * rg6);
    if (kSyncRegion + 256 + 4 * (size_t)(heads * rg6) * n_cap + per_split * ((nst + cs - 1) / cs) <= p->bytes) {
      p->RG = rg6;
      p->RT = (p->RTT + p->RG - 1) / p->RG;
    }
  }
  const int64_t groups = heads * p->RG;
  int64_t cs = chunk_stages(groups);
  // within the workspace bound
  p->off_mpart = kSyncRegion;
  p->off_stats = align_up(p->off_mpart + 4 * (size_t)groups * n_cap, 256);
  const int64_t most = p->bytes > p->off_stats ? (int64_t)((p->bytes - p->off_stats) / per_split) : 1;
  const int64_t least = most < 1 ? nst : (nst + most - 1) / most;
  if (cs < least) cs = least;
  p->chunk = (int)(cs * 2 * blk);
  p->splits = (int)((n_plan + p->chunk - 1) / p->chunk);
  p->off_opart = p->off_stats + 128 * (size_t)tiles * p->splits;
  // A bf16 partial's rounding averages out over many chunks; over few it would
  // show beside the result's own (1.7e-3), so few chunks keep fp32 partials.
  p->o32 = !bf16 || (p->splits < 24 && p->off_opart + 64 * (size_t)tiles * p->splits * D <= p->bytes);
  return PVLM_OK;
}

}  // namespace pvlm
