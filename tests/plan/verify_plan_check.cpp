// Runs verify attention's plan over its sizes without a GPU.
//   verify_plan_check resident WG   no plan counts on more than WG workgroups
//                                   of a compute unit at once
//   verify_plan_check round         a plan's workgroups run in one round
//                                   wherever its groups of row tiles do
//   verify_plan_check areas         the areas follow each other inside the
//                                   workspace, every cache row in one chunk
//   verify_plan_check finish        the finish kernel's grid within a launch's
//                                   limit, to the longest cache
//   verify_plan_check sized         a workspace sized for the whole device is
//                                   enough under every budget
//   verify_plan_check show DT B T HQ HKV D N_CAP CTX
//                                   prints a call's row tiles, row groups,
//                                   chunks and tokens of a chunk
// Prints the first failures and their number.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "verify_plan.h"

using namespace pvlm;

struct Call {
  pvlm_dtype dt;
  int B, T, Hq, Hkv, D;
  int64_t n_cap, ctx;
};

template <typename F>
static void each_call(F f) {
  const int64_t ctxs[] = {0,    1,    62,   63,   64,    127,   333,   787,   1300,  1919,  4096,   6432,
                          8192, 9000, 12800, 14300, 14400, 16384, 20000, 32768, 63000, 70000, 131072, 500000};
  for (int dt = 0; dt < 2; ++dt)
    for (int D : {64, 128})
      for (int Hkv : {1, 2, 3, 4, 5, 7, 8, 12, 16})
        for (int G : {1, 4, 5, 7, 8, 16, 32})
          for (int T : {1, 2, 4, 6, 9, 12, 17, 32})
            for (int B : {1, 2, 3, 4, 5, 6, 7, 8, 40})
              for (int64_t ctx : ctxs) {
                const Call c{dt ? PVLM_BF16 : PVLM_F32, B, T, G * Hkv, Hkv, D, ctx + T + (ctx % 3) * 50, ctx};
                if (check_verify(c.dt, c.B, c.T, c.Hq, c.Hkv, c.D, c.n_cap, c.ctx) == PVLM_OK) f(c);
              }
}

template <typename F>
static long failures(F bad) {
  long n = 0, fail = 0;
  DeviceInfo whole;
  whole.cus = 256;
  whole.xcds = 8;
  each_call([&](const Call& c) {
    for (int cus : {256, 248, 224, 128, 104, 40, 32, 8}) {
      DeviceInfo di = whole;
      di.cus = cus;
      di.budgeted = cus != whole.cus;
      VSplit p;
      if (split_verify(c.dt, c.B, c.T, c.Hq, c.Hkv, c.D, c.n_cap, c.ctx, whole, di, &p) != PVLM_OK) continue;
      ++n;
      if (bad(c, di, p) && fail++ < 10)
        std::printf("%s B %d T %d heads %d/%d D %d ctx %lld on %d: %d x %d tiles, %d chunks of %d, slots %d\n",
                    c.dt == PVLM_BF16 ? "bf16" : "fp32", c.B, c.T, c.Hq, c.Hkv, c.D, (long long)c.ctx, cus, p.RG,
                    p.RT, p.splits, p.chunk, p.slots);
    }
  });
  std::printf("%ld of %ld plans fail\n", fail, n);
  return n == 0 ? 1 : fail;
}

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "resident")) {
    const int wg = std::atoi(argv[2]);
    return failures([&](const Call&, const DeviceInfo& di, const VSplit& p) { return p.slots > wg * di.cus; }) != 0;
  }
  if (argc == 2 && !std::strcmp(argv[1], "round"))
    return failures([&](const Call& c, const DeviceInfo&, const VSplit& p) {
             const int64_t groups = (int64_t)c.B * c.Hkv * p.RG;
             return groups * p.splits > p.slots && (groups <= p.slots || p.splits > 1);
           }) != 0;
  if (argc == 2 && !std::strcmp(argv[1], "areas"))
    return failures([&](const Call& c, const DeviceInfo&, const VSplit& p) {
             const size_t tiles = (size_t)c.B * c.Hkv * p.RTT, e = p.o32 ? 4 : 2;
             const int64_t n = c.ctx + c.T;
             return p.RT > kMaxRT || p.RT * p.RG < p.RTT || p.off_mpart < kSyncRegion ||
                    p.off_stats < p.off_mpart + 4 * (size_t)c.B * c.Hkv * p.RG * c.n_cap ||
                    p.off_opart < p.off_stats + 128 * tiles * p.splits ||
                    p.bytes < p.off_opart + tiles * p.splits * 16 * c.D * e ||
                    (int64_t)p.chunk * p.splits < n || (int64_t)p.chunk * (p.splits - 1) >= n;
           }) != 0;
  if (argc == 2 && !std::strcmp(argv[1], "finish")) {
    long fail = 0;
    for (int B : {1, 3, 4, 64, 2048})
      for (int64_t n_cap : {(int64_t)1, (int64_t)256, (int64_t)257, (int64_t)1 << 24, ((int64_t)1 << 30) - 1, (int64_t)1 << 30}) {
        const int64_t per = mass_rows(B, n_cap), wgs = mass_workgroups(n_cap, per);
        const int64_t rows = (int64_t)640 * 2048;  // rows of O, four a workgroup
        fail += per % kFinThreads != 0 || per * wgs < n_cap || per * (wgs - 1) >= n_cap ||
                (n_cap * B <= kMassWgs * kFinThreads && per != kFinThreads) ||
                (B * wgs + rows / 4) * kFinThreads >= (int64_t)1 << 32;
      }
    std::printf("%ld grids fail\n", fail);
    return fail != 0;
  }
  if (argc == 2 && !std::strcmp(argv[1], "sized")) {
    DeviceInfo whole;
    whole.cus = 256;
    whole.xcds = 8;
    return failures([&](const Call& c, const DeviceInfo&, const VSplit& p) {
             VSplit w;
             return split_verify(c.dt, c.B, c.T, c.Hq, c.Hkv, c.D, c.n_cap, c.ctx, whole, whole, &w) == PVLM_OK && p.bytes > w.bytes;
           }) != 0;
  }
  if (argc == 10 && !std::strcmp(argv[1], "show")) {
    int64_t v[8];
    for (int i = 0; i < 8; ++i) v[i] = std::atoll(argv[2 + i]);
    DeviceInfo di;
    di.cus = 256;
    di.xcds = 8;
    VSplit p;
    if (split_verify((pvlm_dtype)v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], di, di, &p) != PVLM_OK) return 1;
    std::printf("%d %d %d %d\n", p.RT, p.RG, p.splits, p.chunk);
    return 0;
  }
  return 2;
}
