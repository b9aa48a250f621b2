// Host-only check of which forms of the kernels a list of matrices is launched in.  The library's host code (csrc/fira.hip) is
// compiled into this program with a stand-in for the HIP runtime below it (host_hip.h), which records every launch.  Built and
// run on the CPU by tests/test_host_launch.py.
#include "../paper_2410_01623_amd/csrc/fira.hip"

#include "host_hip.h"

namespace {

std::vector<const void*> launched;

template <typename K>
int times(K kernel) { return (int)std::count(launched.begin(), launched.end(), (const void*)kernel); }

// A context over `descs` whose matrices have projectors and gates that let the Gram route through, and the step of some of them.
struct Case {
  std::vector<fira_matrix_desc> descs;
  fira_ctx* ctx = nullptr;
  void* slab = nullptr;
  explicit Case(std::vector<fira_matrix_desc> d) : descs(std::move(d)) {
    const int n = (int)descs.size();
    const fira_hparams hp = {1e-3, 0.9, 0.999, 1e-8, 1.0, 1.01};
    const size_t bytes = fira_state_bytes(descs.data(), n);
    slab = std::aligned_alloc(256, align_up(bytes));
    CHECK(fira_init_state(&ctx, descs.data(), n, &hp, slab, bytes, nullptr) == FIRA_OK);
    for (int i = 0; i < n; ++i) {
      const int idx[1] = {i};
      const void* const P[1] = {(const void*)0x5000};
      CHECK(fira_set_projectors(ctx, 1, idx, P, (fira_dtype)descs[i].wg_dtype) == FIRA_OK);
      CHECK(fira_set_gate(ctx, i, 1e-3f, 1e-4f) == FIRA_OK);
    }
  }
  ~Case() { fira_destroy(ctx); std::free(slab); }
  void step(const std::vector<int>& idx) {
    std::vector<void*> W(idx.size(), (void*)0x1000);
    std::vector<const void*> G(idx.size(), (const void*)0x3000);
    launched.clear();
    CHECK(fira_step(ctx, (int)idx.size(), idx.data(), W.data(), G.data()) == FIRA_OK);
  }
};

fira_matrix_desc desc(long long m, long long n, int r, int dtype) { return {m, n, n, r, dtype}; }

}  // namespace

int main() {
  on_launch = [](const void* kernel, dim3, void**) { launched.push_back(kernel); };
  auto whole = fira_backproject_kernel<1, bf16_raw, 4, 2>;
  auto quarter = fira_backproject_kernel<1, bf16_raw, 2, 1>;

  {   // bf16 lists of 512 tiles: quarter tiles up to rank 256, whole ones above, by the ranks of the bf16 matrices alone
    Case c({desc(4096, 4096, 128, FIRA_BF16), desc(320, 400, 300, FIRA_F32), desc(300, 300, 260, FIRA_BF16)});
    c.step({0});
    CHECK(times(quarter) == 1 && times(whole) == 0);
    c.step({0, 1});
    CHECK(times(quarter) == 1 && times(whole) == 0);
    c.step({0, 2});
    CHECK(times(quarter) == 0 && times(whole) == 1);
  }
  {   // ranks whose R stays in memory: the fused kernel from 200 tiles of 128 factors on, two kernels below and beside ranks whose R does not
    Case c({desc(128, 128 * 199, 96, FIRA_BF16), desc(128, 128 * 200, 96, FIRA_BF16), desc(200, 128, 68, FIRA_BF16), desc(160, 256, 160, FIRA_BF16),
            desc(300, 200, 40, FIRA_BF16), desc(128, 128 * 200, 97, FIRA_BF16)});
    struct { std::vector<int> idx; int fused; } lists[] = {{{0}, 0}, {{1}, 1}, {{0, 2}, 1}, {{4, 1}, 1}, {{1, 3}, 0}, {{3}, 1}, {{3, 4}, 0}, {{1, 5}, 0}};
    for (auto& l : lists) {
      c.step(l.idx);
      CHECK(times(fira_project_adam_kernel<1>) == l.fused && times(fira_adam_kernel<1, false>) == 1 - l.fused);
    }
  }
  {   // ranks that all leave R in memory, on the residual route, in two planes and right after an installation: one kernel where its launch fills enough of a round
    auto one = fira_fused_leave_r_kernel<1>;
    auto two = fira_fused_leave_r_kernel<2>;
    struct L { std::vector<fira_matrix_desc> d; int one, two; };
    auto copies = [](fira_matrix_desc d, int n, std::vector<fira_matrix_desc> more = {}) { more.insert(more.begin(), n, d); return more; };
    auto wide = [](int S, long long tiles, int r) { return desc(S, 128 * tiles, r, FIRA_BF16); };
    const std::vector<L> lists = {
        // both sides of the line: whole ranks, 3/4 of a round of 512 workgroups (r > 256: of 256), of two rounds, and just above one
        {{wide(128, 376, 128)}, 0, 0}, {{wide(128, 377, 128)}, 1, 0}, {{wide(128, 512, 128)}, 1, 0}, {{wide(128, 513, 128)}, 0, 0}, {{wide(128, 769, 128)}, 1, 0},
        {{wide(256, 376, 256)}, 0, 0}, {{wide(256, 377, 256)}, 1, 0}, {{wide(256, 513, 256)}, 0, 0},
        {{wide(512, 184, 512)}, 0, 0}, {{wide(512, 185, 512)}, 0, 1}, {{wide(512, 256, 512)}, 0, 1}, {{wide(512, 257, 512)}, 0, 0},
        // narrower ones, 15/16; from r = 128 on 15/16 of the tile's width as well
        {{wide(128, 472, 96)}, 0, 0}, {{wide(128, 473, 96)}, 1, 0}, {{wide(256, 473, 240)}, 1, 0}, {{wide(256, 472, 240)}, 0, 0}, {{wide(256, 512, 236)}, 0, 0},
        {{wide(512, 233, 480)}, 0, 1}, {{wide(512, 232, 480)}, 0, 0}, {{wide(512, 256, 476)}, 0, 0}, {{wide(384, 256, 260)}, 0, 0},
        // the lists of test_gpu_fused_every_route.py and test_gpu_list_independence.py
        {copies(desc(130, 1700, 68, FIRA_BF16), 35, {desc(300, 260, 40, FIRA_BF16)}), 1, 0}, {copies(desc(200, 1537, 128, FIRA_BF16), 38), 1, 0},
        {copies(desc(1665, 300, 252, FIRA_BF16), 35), 1, 0}, {copies(desc(259, 1700, 256, FIRA_BF16), 35), 1, 0}, {copies(desc(1665, 520, 508, FIRA_BF16), 17), 0, 1},
        {copies(desc(520, 1536, 512, FIRA_BF16), 20), 0, 1}, {copies(desc(1665, 129, 124, FIRA_BF16), 35), 1, 0}, {copies(desc(161, 1600, 96, FIRA_BF16), 38), 1, 0},
        {copies(desc(1665, 256, 128, FIRA_BF16), 35), 1, 0}, {copies(desc(1665, 300, 240, FIRA_BF16), 35), 1, 0}, {copies(desc(320, 1536, 256, FIRA_BF16), 41), 1, 0},
        {copies(desc(520, 1700, 484, FIRA_BF16), 17), 0, 1}, {copies(desc(620, 1536, 512, FIRA_BF16), 20), 0, 1},
        // the two parts of a launch start anew on every XCD
        {copies(desc(128, 128, 128, FIRA_BF16), 256, {desc(128 * 256, 128, 128, FIRA_BF16)}), 1, 0}, {copies(desc(256, 256, 256, FIRA_BF16), 121, {desc(128 * 265, 256, 256, FIRA_BF16)}), 0, 0},
        // what else is listed: a rank that asks for more, another width, a small rank (a kernel of its own), and what cannot take it
        {{wide(256, 416, 256), wide(128, 24, 96)}, 0, 0}, {{wide(256, 416, 256), wide(128, 60, 96)}, 1, 0}, {{wide(256, 416, 256), wide(512, 200, 512)}, 1, 1},
        {{wide(256, 416, 256), wide(512, 20, 512)}, 0, 0}, {{wide(256, 416, 256), desc(300, 200, 40, FIRA_BF16)}, 1, 0},
        {{wide(256, 416, 256), desc(300, 200, 97, FIRA_BF16)}, 0, 0}, {{wide(256, 416, 256), desc(600, 700, 516, FIRA_BF16)}, 0, 0},
        {{wide(256, 416, 256), desc(300, 200, 96, FIRA_F32)}, 0, 0}, {{desc(300, 200, 40, FIRA_BF16)}, 0, 0},
    };
    for (const L& l : lists) {
      Case c(l.d);
      const int n = (int)l.d.size();
      std::vector<int> all(n);
      for (int i = 0; i < n; ++i) all[i] = i;
      auto check = [&](const char* route, bool expected) {
        const int fused = expected ? 1 : 0;
        // the other matrices' projection and Adam run if and only if the fused kernel does not
        bool general = false;
        for (const fira_matrix_desc& d : l.d) general = general || (d.wg_dtype == FIRA_BF16 && d.r > 64);
        const int others = general && !(fused && (l.one || l.two)) ? 1 : 0;
        if (times(one) != fused * l.one || times(two) != fused * l.two || times(fira_project_kernel) != others ||
            times(fira_adam_kernel<1, false>) + times(fira_adam_kernel<1, true>) != others) {
          ++failures;
          std::printf("FAIL: %s, %d matrices, first %lld x %lld, r = %d: %d %d\n", route, n, (long long)l.d[0].m, (long long)l.d[0].n, (int)l.d[0].r, times(one), times(two));
        }
        CHECK(!expected || fira_last_step_fused(c.ctx) == 0);
      };
      c.step(all);                                   // the Gram route has forms of its own
      CHECK(times(one) == 0 && times(two) == 0);
      CHECK(fira_set_z_planes(c.ctx, 2) == FIRA_OK);
      c.step(all);
      check("two planes, Gram route", true);
      for (int i = 0; i < n; ++i) CHECK(fira_set_gate(c.ctx, i, 1.0f, 1.0f) == FIRA_OK);
      c.step(all);
      check("two planes, residual route", true);
      CHECK(fira_set_z_planes(c.ctx, 1) == FIRA_OK);
      c.step(all);
      check("gates closed", true);
      CHECK(fira_set_fusion(c.ctx, 0) == FIRA_OK);
      c.step(all);
      check("fusion off", false);
      CHECK(fira_set_fusion(c.ctx, 1) == FIRA_OK);
      for (int i = 0; i < n; ++i) CHECK(fira_set_gate(c.ctx, i, 1e-3f, 1e-4f) == FIRA_OK);
      CHECK(fira_set_options(c.ctx, FIRA_SCALE_COLUMN, FIRA_NORM_RESIDUAL) == FIRA_OK);
      c.step(all);
      check("residual norm", true);
      CHECK(fira_set_options(c.ctx, FIRA_SCALE_MATRIX, FIRA_NORM_RESIDUAL) == FIRA_OK);
      c.step(all);
      check("a factor per matrix", false);
      CHECK(fira_set_options(c.ctx, FIRA_SCALE_COLUMN, FIRA_NORM_GRAM) == FIRA_OK);
      for (int i = 0; i < n; ++i) {
        const int idx[1] = {i};
        const void* const P[1] = {(const void*)0x5000};
        CHECK(fira_set_projectors(c.ctx, 1, idx, P, (fira_dtype)l.d[i].wg_dtype) == FIRA_OK);
      }
      c.step(all);
      check("right after an installation", true);
    }
    // one matrix on the Gram route beside others that are not: as on that route, where R does not stay
    Case c({wide(256, 416, 256), wide(256, 8, 256)});
    CHECK(fira_set_gate(c.ctx, 0, 1.0f, 1.0f) == FIRA_OK);
    c.step({0, 1});
    CHECK(times(one) == 0 && times(fira_project_adam_kernel<1>) == 1 && times(fira_project_kernel) == 1);
  }
  {   // fp32 projection: whole panels where all of the list's run at once, tiles otherwise and for wider matrices
    Case c({desc(128, 256, 64, FIRA_F32), desc(2, 64 * 2600, 1, FIRA_F32), desc(417, 500, 64, FIRA_F32)});
    c.step({0});
    CHECK(times(fira_panel_project_kernel) == 1 && times(fira_fp32_project_kernel) == 0);
    c.step({0, 1});
    CHECK(times(fira_panel_project_kernel) == 0 && times(fira_fp32_project_kernel) == 1);
    c.step({0, 2});
    CHECK(times(fira_panel_project_kernel) == 1 && times(fira_fp32_project_kernel) == 1);
  }
  {   // ... "at once" counts the workgroups that are launched, two a CU at most, and ranks above 256 take tiles
    auto copies = [](fira_matrix_desc d, int n) { return std::vector<fira_matrix_desc>(n, d); };
    auto all = [](int n) { std::vector<int> v(n); for (int i = 0; i < n; ++i) v[i] = i; return v; };
    struct { fira_matrix_desc d; int n; bool panels; } lists[] = {
        {desc(400, 800, 256, FIRA_F32), 18, true},    {desc(400, 800, 256, FIRA_F32), 19, false},   // 252 and 266 workgroups, one a CU
        {desc(800, 400, 256, FIRA_F32), 18, true},    {desc(800, 400, 256, FIRA_F32), 19, false},
        {desc(400, 800, 257, FIRA_F32), 1, false},    {desc(400, 800, 400, FIRA_F32), 18, false},
        {desc(64, 32768, 64, FIRA_F32), 1, true},     {desc(64, 32769, 64, FIRA_F32), 1, false},    // 512 and 514, of which LDS alone would take five a CU
        {desc(16, 32768, 16, FIRA_F32), 1, true},     {desc(16, 150000, 16, FIRA_F32), 1, false},
        {desc(64, 64, 16, FIRA_F32), 256, true},      {desc(64, 64, 16, FIRA_F32), 257, false},     // every second workgroup has a panel
    };
    for (auto& l : lists) {
      Case c(copies(l.d, l.n));
      c.step(all(l.n));
      const bool panels = times(fira_panel_project_kernel) == 1, tiles = times(fira_fp32_project_kernel) == 1;
      if (panels != l.panels || tiles == l.panels) { ++failures; std::printf("FAIL: %d matrices of %lld x %lld, r = %d\n", l.n, (long long)l.d.m, (long long)l.d.n, (int)l.d.r); }
    }
  }
  std::printf("%d failure(s)\n", failures);
  return failures ? 1 : 0;
}
