// The key-stationary pass for short sequences (dkdv32_kernel with the queries split over pairs
// of waves), in an object of its own so that the long-sequence instances keep their code.
#define LAGA_SHORT_SEQ
#include "attn_bwd.hip"
