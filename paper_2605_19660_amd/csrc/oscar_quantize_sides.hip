// The encoder's form for the smallest launches, published transform.  -ffp-contract=off, as for every user of the
// encoder header.
#include "oscar_append_sides.h"

int oscar_launch_append_sides(const AppendParams& P, bool all_heads, dim3 grid, hipStream_t st) {
  return all_heads ? oscar_launch_append_sides_all_heads(P, grid, st) : launch_sides_all_types<XF_PUBLISHED>(P, grid, st);
}
