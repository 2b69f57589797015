// The 64/32/64-wide heads of the attention forward, in an object of their own: instantiated
// beside the 128/64/128 ones they changed the inlining order of the helpers that both use,
// and with it the register allocation of those tuned kernels.
#define LAGA_HALF_WIDTHS
#include "attn_fwd.hip"
