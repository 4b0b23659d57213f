// The encoder's form for the smallest launches, norm over all kv heads.  -ffp-contract=off, as for every user of the
// encoder header.
#include "oscar_append_sides.h"

int oscar_launch_append_sides_all_heads(const AppendParams& P, dim3 grid, hipStream_t st) {
  return launch_sides_all_types<XF_ALL_HEADS>(P, grid, st);
}
