// Decode-attention kernel variant: mixed family (KIVI keys, RTN values),
// up to 4 query heads per kv-head, bit-widths up to 4.
#include "rq_attn_impl.h"

RQ_DEFINE_ATTN_LAUNCHER(RQ_KIVI_RTN, 1, 4, launch_attn_kivirtn_n1_b4)
