// Host-only check of the gate values of the Gram route as the host keeps them: memory that the kernels write while the host only
// waits for an event.  The library's host code (csrc/fira.hip) is compiled into this program with a stand-in for the HIP runtime
// below it (host_hip.h).  Built and run on the CPU by tests/test_host_gate.py.
#include "../paper_2410_01623_amd/csrc/fira.hip"

#include "host_hip.h"

int main() {
  const fira_matrix_desc descs[2] = {{96, 160, 160, 16, FIRA_BF16}, {160, 96, 96, 16, FIRA_F32}};
  const fira_hparams hp = {1e-3, 0.9, 0.999, 1e-8, 1.0, 1.01};
  const size_t bytes = fira_state_bytes(descs, 2);
  void* slab = std::aligned_alloc(256, bytes);
  fira_ctx* ctx = nullptr;
  CHECK(fira_init_state(&ctx, descs, 2, &hp, slab, bytes, nullptr) == FIRA_OK);
  if (!ctx) return 1;

  // What kernels store is the host's to see once the event has passed, whatever the environment makes of memory without a flag.
  CHECK(made_with[ctx->h_gate] & hipHostMallocCoherent);
  CHECK(made_with[ctx->h_gate] & hipHostMallocMapped);
  CHECK(made_with[ctx->ortho_event] & hipEventReleaseToSystem);

  // An installation that fails leaves the old projector and its gate in force, if nothing of it was launched, or no projector: never an old
  // projector's gate on the device and none on the host, which would send a matrix two ways in one step.
  const int idx[2] = {0, 1};
  const void* const P[2] = {(const void*)0x5000, (const void*)0x6000};
  auto one = [&] { return fira_set_projector(ctx, 0, P[0], FIRA_F32); };
  auto list = [&] { return fira_set_projectors(ctx, 2, idx, P, FIRA_F32); };
  auto install = [&] {
    CHECK(list() == FIRA_OK);
    for (int i = 0; i < 2; ++i) CHECK(fira_set_gate(ctx, i, 1e-3f, 1e-4f) == FIRA_OK);
  };
  auto as_before = [&](int i) {
    return ctx->plan.mats[i].has_projector && !ctx->unmeasured[i] && ctx->h_gate[i].ortho_err == ctx->d_scal[i].ortho_err && ctx->h_gate[i].gram_err == ctx->d_scal[i].gram_err;
  };
  auto gone = [&](int i) { return !ctx->plan.mats[i].has_projector; };
  install();
  uploads_fail = true;
  CHECK(list() == FIRA_ERR_HIP);
  uploads_fail = false;
  CHECK(as_before(0) && as_before(1));
  failing_event = ctx->install_event;
  CHECK(list() == FIRA_ERR_HIP);
  CHECK(as_before(0) && as_before(1));
  failing_event = ctx->ortho_event;
  CHECK(list() == FIRA_ERR_HIP);
  CHECK(gone(0) && gone(1));
  failing_event = nullptr;
  install();
  failing_event = ctx->ortho_event;
  CHECK(one() == FIRA_ERR_HIP);
  CHECK(gone(0) && as_before(1));
  failing_event = nullptr;
  install();
  launches_fail = true;
  CHECK(one() == FIRA_ERR_HIP);
  CHECK(gone(0) && as_before(1));
  CHECK(list() == FIRA_ERR_HIP);
  CHECK(gone(0) && gone(1));
  launches_fail = false;
  install();
  CHECK(as_before(0) && as_before(1));

  // ... and a refresh likewise
  const void* const G[2] = {(const void*)0x3000, (const void*)0x4000};
  const size_t wsb = fira_refresh_workspace_bytes(ctx, 2, idx);
  void* ws = std::aligned_alloc(256, align_up(wsb));
  auto refresh = [&] { return fira_refresh_projectors(ctx, 2, idx, G, 2, 7, ws, wsb); };
  uploads_fail = true;
  CHECK(refresh() == FIRA_ERR_HIP);
  uploads_fail = false;
  CHECK(as_before(0) && as_before(1));
  launches_fail = true;
  CHECK(refresh() == FIRA_ERR_HIP);
  launches_fail = false;
  CHECK(gone(0) && gone(1));
  install();
  failing_event = ctx->ortho_event;
  CHECK(refresh() == FIRA_ERR_HIP);
  failing_event = nullptr;
  CHECK(gone(0) && gone(1));
  CHECK(refresh() == FIRA_OK && !gone(0) && !gone(1));

  fira_destroy(ctx);
  std::free(ws);
  std::free(slab);
  std::printf("%d failure(s)\n", failures);
  return failures ? 1 : 0;
}
