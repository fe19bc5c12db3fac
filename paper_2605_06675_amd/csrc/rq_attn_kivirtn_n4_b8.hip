// Decode-attention kernel variant: mixed family (KIVI keys, RTN values),
// more than 8 query heads per kv-head, bit-widths up to 8.
#include "rq_attn_impl.h"

RQ_DEFINE_ATTN_LAUNCHER(RQ_KIVI_RTN, 4, 8, launch_attn_kivirtn_n4_b8)
