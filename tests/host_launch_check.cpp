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
