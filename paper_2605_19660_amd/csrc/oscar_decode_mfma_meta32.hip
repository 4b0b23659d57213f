// The matrix-core decode kernel for fp32 metadata (step sizes, zero-points, norms): the same
// source as oscar_decode_mfma.hip with the metadata type fixed at compile time.
#define OSCAR_MFMA_META32 1
#include "oscar_decode_mfma.hip"
