// Encoder instantiations for the token norm over all kv heads (App. "Fused Hadamard-Norm
// Kernel").  -ffp-contract=off, as for every user of the encoder header.
//
// Two launches: oscar_token_norm_kernel computes the norms of the new tokens (it reads every head of a
// token once), then the encoder kernel runs as usual and takes those norms from the pages' norm slots
// and the residual window.  In an append of few tokens the first launch computes those of tokens that
// move into a page only (a rare case), and the encoder the others'.  A single-token decode append never
// moves a new token into a page (a deferred flush holds residual tokens only), so it skips the first launch.
#include "oscar_append_kernel.h"

namespace {
template <bool WINDOW> int launch_norms_of_type(const AppendParams& P, hipStream_t st) {
  switch (P.c.cfg.io_dtype) {
    case OSCAR_F32: return launch_token_norms<float, WINDOW>(P, st);
    case OSCAR_BF16: return launch_token_norms<__hip_bfloat16, WINDOW>(P, st);
    case OSCAR_F16: return launch_token_norms<__half, WINDOW>(P, st);
    default: return OSCAR_ERR_UNSUPPORTED;
  }
}
}  // namespace

int oscar_launch_append_all_heads(const AppendParams& P, dim3 grid, hipStream_t st) {
  if (P.T <= kFewTokens) {
    if (P.T > 1 || (P.flags & OSCAR_APPEND_EAGER)) {
      const int rc = launch_norms_of_type<false>(P, st);
      if (rc != OSCAR_OK) return rc;
    }
    return launch_append<XF_ALL_HEADS_FEW>(P, grid, st);
  }
  const int rc = launch_norms_of_type<true>(P, st);
  return rc != OSCAR_OK ? rc : launch_append<XF_ALL_HEADS>(P, grid, st);
}
