// The decode step's kernel (append of one token per sequence, then attention) for the float
// zero-point form: the source of oscar_decode_mfma.hip with both fixed at compile time.
#define OSCAR_MFMA_STEP 1
#define OSCAR_MFMA_ZPMIN 1
#include "oscar_decode_mfma.hip"
