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

  fira_destroy(ctx);
  std::free(slab);
  std::printf("%d failure(s)\n", failures);
  return failures ? 1 : 0;
}
