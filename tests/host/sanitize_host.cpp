// Host-only exercise of the library's host logic (instance search, reduction choice, leader rule, time models,
// least-loaded routing, error paths that return before any device call) for a build with AddressSanitizer and
// UndefinedBehaviorSanitizer on the host side.  No GPU is touched.  Exit code 0 = all checks passed.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "../../include/gmidrl.h"
#include "../../paper_2206_08482_amd/csrc/internal.h"
#include "../../paper_2206_08482_amd/csrc/rollout.h"

static int fails = 0;
#define CHECK(c) do { if (!(c)) { std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #c); ++fails; } } while (0)

struct Table { int calls = 0; };
// throughput grows with the env count and saturates; memory grows linearly
static int profile(int32_t k, int32_t n, int32_t* runnable, double* top, double* mem, void* user) {
  static_cast<Table*>(user)->calls++;
  *runnable = k <= 8;
  *top = 1000.0 * n / (n + 2048.0) / k;
  *mem = 1e6 * n + 5e7;
  return 0;
}

int main() {
  {
    Table t;
    const int32_t ks[] = {8, 4, 2, 1, 16}, ns[] = {128, 512, 2048, 8192};
    int32_t n_out = -1, k_out = -1;
    double proj = -1.0;
    const int rc = gmi_explore(profile, &t, nullptr, nullptr, 1, 0.05, ks, 5, ns, 4, &n_out, &k_out, &proj);
    CHECK(rc == GMI_OK);
    CHECK(t.calls > 0 && t.calls <= 20);
    CHECK(n_out > 0 && k_out > 0 && proj > 0.0);
    CHECK(gmi_explore(nullptr, &t, nullptr, nullptr, 1, 0.05, ks, 5, ns, 4, &n_out, &k_out, &proj) != GMI_OK);
    CHECK(std::strlen(gmi_last_error()) > 0);
    // an empty grid records no point: the documented answer is the pair (0, 0)
    CHECK(gmi_explore(profile, &t, nullptr, nullptr, 1, 0.05, ks, 0, ns, 4, &n_out, &k_out, &proj) == GMI_OK && n_out == 0 && k_out == 0);
  }
  {
    const int64_t load[] = {50, 20, 20, 70};
    int32_t best = -1;
    CHECK(gmi_route_least_loaded(load, 4, &best) == GMI_OK && best == 1);
    CHECK(gmi_route_least_loaded(load, 0, &best) != GMI_OK);
    CHECK(gmi_route_least_loaded(nullptr, 4, &best) != GMI_OK);
  }
  {
    // Algorithm 1's three exits, the leader rule and the time models (Table 2)
    int32_t strat = -1;
    const int32_t one[] = {4}, even[] = {2, 2, 2, 2}, uneven[] = {2, 3}, many[] = {4, 4};
    CHECK(gmi_select_reduction(one, 1, &strat) == GMI_OK && strat == GMI_REDUCE_MULTI_PROCESS);
    CHECK(gmi_select_reduction(even, 4, &strat) == GMI_OK && strat == GMI_REDUCE_MULTI_RING);
    CHECK(gmi_select_reduction(uneven, 2, &strat) == GMI_OK && strat == GMI_REDUCE_HIERARCHICAL);
    CHECK(gmi_select_reduction(many, 2, &strat) == GMI_OK && strat == GMI_REDUCE_HIERARCHICAL);
    CHECK(gmi_select_reduction(nullptr, 2, &strat) != GMI_OK);
    const int32_t ids[] = {0, 1, 2, 3, 4, 5}, start[] = {0, 3, 6};
    int32_t leaders[2] = {-2, -2};
    CHECK(gmi_har_leaders(ids, start, 2, 1, leaders) == GMI_OK && leaders[0] == 1 && leaders[1] == 4);
    double sec[3] = {0, 0, 0};
    for (int st = 0; st < 3; ++st) CHECK(gmi_reduction_time(st, 4, 2, 1e6, 1e9, 1e10, &sec[st]) == GMI_OK && sec[st] > 0.0);
    CHECK(gmi_reduction_time(7, 4, 2, 1e6, 1e9, 1e10, &sec[0]) != GMI_OK);
  }
  {
    // bad handles are reported before anything touches a device
    CHECK(gmi_sync(nullptr) == GMI_ERR_BAD_HANDLE);
    CHECK(gmi_destroy(nullptr) == GMI_ERR_BAD_HANDLE);
    CHECK(gmi_channels_drop(nullptr, 1) == GMI_ERR_BAD_HANDLE);
    CHECK(gmi_stream(nullptr) == nullptr);
  }
  {
    // what a kernel has been allowed on one device says nothing about another; devices may be added by several threads
    gmi::DeviceSet done;
    CHECK(!done.has(0) && !done.has(-1) && !done.has(64));
    done.add(3);
    CHECK(done.has(3) && !done.has(0) && !done.has(2) && !done.has(4) && !done.has(35));
    done.add(-1);
    done.add(64);
    CHECK(!done.has(-1) && !done.has(64) && !done.has(0));
    std::vector<std::thread> ts;
    for (int i = 0; i < 8; ++i) ts.emplace_back([&done, i]() { for (int d = i; d < 64; d += 8) done.add(d); });
    for (std::thread& t : ts) t.join();
    for (int d = 0; d < 64; ++d) CHECK(done.has(d));
  }
  {
    // a collection's simulator waves read inside every row of the matrix (the last one ends where the allocation does) and of the
    // states, and every group of the product that they do not take in order is among the ones read ahead
    int outside = 0, missed = 0;
    for (int O = 1; O <= 700; ++O)
      for (int A = 1; A <= 64; ++A) {
        const SimGroups s = sim_groups_ahead(O, A);
        const int last = (s.g0 > s.g1 ? s.g0 : s.g1) > s.gt ? (s.g0 > s.g1 ? s.g0 : s.g1) : s.gt;
        outside += 4 * last + 4 > ((O + A + 3) & ~3) || 4 * last + 4 > gmi::env_row_stride(O, A) || 4 * last + 4 > split_stride(O, A);
        const int gs = O / 4, ng = (O + A) / 4;
        missed += (gs < ng && s.g0 != gs) || (gs + 1 < ng && s.g1 != gs + 1) || ((O + A) % 4 && s.gt != ng);
      }
    CHECK(outside == 0);
    CHECK(missed == 0);
  }
  {
    // a weight gradient's rows: at least as many partial sums for every layer as the same number of splits for all would give, and
    // no more workgroups than one per compute unit where that is possible
    const int shapes[][6] = {{64, 256, 128, 64, 32, 0},    {128, 416, 224, 128, 32, 0},  {224, 512, 512, 256, 128, 32}, {224, 512, 512, 512, 256, 32},
                             {256, 512, 512, 512, 512, 32}, {224, 512, 416, 416, 320, 32}, {64, 416, 320, 32, 0, 0},      {32, 320, 224, 64, 32, 0},
                             {32, 32, 32, 0, 0, 0},        {160, 512, 512, 320, 320, 32}, {320, 1120, 1120, 64, 32, 0},  {256, 256, 192, 192, 32, 0}};
    for (const auto& s : shapes) {
      int out[12], in[12], n = 0, tiles = 0, groups = 0;
      for (int net = 0; net < 2; ++net)
        for (int l = 0; l < 5 && s[l + 1]; ++l) { out[n] = s[l + 1]; in[n++] = s[l]; }
      const gmi::WgradSplits p = gmi::plan_wgrad(out, in, n);
      for (int i = 0; i < n; ++i) { tiles += gmi::wgrad_tiles(out[i], in[i]); groups += gmi::wgrad_tiles(out[i], in[i]) * p.n[i]; }
      const int even = 256 / tiles / 4 * 4, same = even < 8 ? 8 : even > 32 ? 32 : even;
      for (int i = 0; i < n; ++i) CHECK(p.n[i] * gmi::wgrad_sums(out[i], in[i]) >= same);
      CHECK(groups <= 256 || tiles > 32);
    }
  }
  {
    // the quotient and the root of a draw: for every radius and every estimate within an ulp what IEEE division and square root give (at the
    // theorem's exception with the reciprocal unit's own, see quotient_from)
    const auto ulps = [](float v, int d) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) + (uint32_t)d); };
    int64_t quotients = 0, roots = 0;
    for (uint32_t j = 1; j < 1u << 24; j += 2) {
      int e;
      const float f = 2.0f * frexpf((float)j, &e), m = f > 0x1.6a09e6p+0f ? f * 0.5f : f, num = m - 1.0f, den = m + 1.0f;
      const float t = num / den, y = (float)(1.0 / (double)den);
      for (int d = -1; d <= 1; ++d)
        if (j == 8388607 ? d == 0 : fabs((double)ulps(y, d) * den - 1.0) <= (double)(ulps(y, 1) - y) * den)
          quotients += gmi::quotient_from(ulps(y, d), num, den) != t;
    }
    for (uint32_t bits = 0x3F800000u; bits < 0x40800000u; ++bits) {      // [1, 4): every mantissa under an even and an odd exponent
      const float x = __builtin_bit_cast(float, bits), r = sqrtf(x);
      for (int d = -1; d <= 1; ++d) roots += gmi::root_from(ulps(r, d), x) != r;
    }
    CHECK(quotients == 0);
    CHECK(roots == 0);
  }
  std::printf(fails ? "host checks: %d failed\n" : "host checks passed\n", fails);
  return fails ? 1 : 0;
}
