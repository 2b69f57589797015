// The 64/32/64-wide heads of the dQ pass, in an object of their own (as attn_fwd_half.hip).
#define LAGA_HALF_WIDTHS
#include "attn_bwd_dq.hip"
