// The matrix-core decode kernel for fp32 metadata and the float zero-point form: the same source
// as oscar_decode_mfma.hip with both fixed at compile time.
#define OSCAR_MFMA_META32 1
#define OSCAR_MFMA_ZPMIN 1
#include "oscar_decode_mfma.hip"
