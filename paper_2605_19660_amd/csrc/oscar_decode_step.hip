// The decode step's kernel (append of one token per sequence, then attention) for the integer
// zero-point: the source of oscar_decode_mfma.hip with the append switched in at compile time.
#define OSCAR_MFMA_STEP 1
#include "oscar_decode_mfma.hip"
