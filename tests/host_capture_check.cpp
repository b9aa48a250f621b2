// Host-only check of which calls a capturing stream refuses.  The library's host code (csrc/fira.hip) is compiled into this
// program with a stand-in for the HIP runtime below it: device memory is host memory, copies happen at once, kernels do
// nothing, everything that would be enqueued is counted, and the stream is "captured" while `capturing` is set.  Built and
// run on the CPU by tests/test_host_capture.py.
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
  const int idx[2] = {0, 1};
  void* const W[2] = {(void*)0x1000, (void*)0x2000};
  const void* const G[2] = {(const void*)0x3000, (const void*)0x4000};
  const size_t wsb = fira_refresh_workspace_bytes(ctx, 2, idx);
  void* ws = std::aligned_alloc(256, align_up(wsb));
  const size_t image = [&] { RefreshPlan rp; make_refresh_plan(ctx->plan, 2, idx, &rp); return rp.top_begin; }();

  // The measured gate of a matrix: what the kernels of a first step would have written (they do nothing here).
  auto set_gates = [&](float gram_err) { for (int i = 0; i < 2; ++i) { ctx->d_scal[i].ortho_err = 1e-3f; ctx->d_scal[i].gram_err = gram_err; } };
  // `call` is refused while the stream is captured: an error, nothing enqueued, the context as it was.
  auto refused = [&](auto call) {
    std::vector<char> img(ctx->h_refresh, ctx->h_refresh + image), un = ctx->unmeasured;
    const bool rp = ctx->refresh_pending, op = ctx->ortho_pending, p0 = ctx->plan.mats[0].has_projector, p1 = ctx->plan.mats[1].has_projector;
    const long before = enqueued;
    capturing = true;
    const fira_status st = call();
    capturing = false;
    return st == FIRA_ERR_HIP && enqueued == before && rp == ctx->refresh_pending && op == ctx->ortho_pending && un == ctx->unmeasured &&
           p0 == ctx->plan.mats[0].has_projector && p1 == ctx->plan.mats[1].has_projector &&
           std::memcmp(img.data(), ctx->h_refresh, image) == 0;
  };
  auto accepted = [&](auto call) {
    const long before = enqueued;
    const fira_status st = call();
    return st == FIRA_OK && enqueued > before;
  };
  auto captured = [&](auto call) { capturing = true; const bool ok = accepted(call); capturing = false; return ok; };
  auto refresh = [&] { return fira_refresh_projectors(ctx, 2, idx, G, 2, 7, ws, wsb); };
  auto refresh_static = [&] { return fira_refresh_projectors_static(ctx, 2, idx, G, 2, 7); };
  auto step = [&] { return fira_step(ctx, 2, idx, W, G); };
  auto step0 = [&] { return fira_step(ctx, 1, idx, W, G); };

  // The projector refresh, as a context's first one (nothing pending that a capture would trip over) and later.
  CHECK(refused(refresh));
  CHECK(refused(refresh_static));
  CHECK(accepted(refresh));
  CHECK(refused(refresh));
  CHECK(refused(refresh_static));
  CHECK(accepted(refresh_static));

  // The step that measures the Gram route's gate; the next ones are captured as documented.
  set_gates(INFINITY);
  CHECK(refused(step));
  CHECK(accepted(step0));                 // measures matrix 0; matrix 1 still waits for its first step
  CHECK(refused(step));
  CHECK(captured(step0));
  CHECK(accepted(step));
  set_gates(1e-4f);
  CHECK(accepted(step));
  CHECK(captured(step));

  // Steps that measure nothing are captured from the first one on.
  const void* const P[2] = {(const void*)0x5000, (const void*)0x6000};
  CHECK(accepted([&] { return fira_set_projectors(ctx, 2, idx, P, FIRA_F32); }));
  CHECK(refused(step));
  CHECK(fira_set_options(ctx, FIRA_SCALE_COLUMN, FIRA_NORM_RESIDUAL) == FIRA_OK);
  CHECK(captured(step));
  CHECK(fira_set_options(ctx, FIRA_SCALE_COLUMN, FIRA_NORM_GRAM) == FIRA_OK);
  CHECK(fira_set_variant(ctx, FIRA_VARIANT_ONLY_SCALING) == FIRA_OK);
  CHECK(captured(step));
  CHECK(fira_set_variant(ctx, FIRA_VARIANT_FULL) == FIRA_OK);
  CHECK(refused(step));
  for (int i = 0; i < 2; ++i) CHECK(fira_set_gate(ctx, i, 1e-3f, 1e-4f) == FIRA_OK);   // restored gates: nothing to measure
  CHECK(captured(step));

  fira_destroy(ctx);
  std::free(slab);
  std::free(ws);
  std::printf("%d failure(s)\n", failures);
  return failures ? 1 : 0;
}
