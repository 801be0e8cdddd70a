// The kernels of attn_fwd_wide.hip for head dimension 64.
#define PDA_SP_HEAD_DIM 64
#include "attn_fwd_wide.hip"
