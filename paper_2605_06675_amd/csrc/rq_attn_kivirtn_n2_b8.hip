// Decode-attention kernel variant: mixed family (KIVI keys, RTN values),
// 5 to 8 query heads per kv-head, bit-widths up to 8.
#include "rq_attn_impl.h"

RQ_DEFINE_ATTN_LAUNCHER(RQ_KIVI_RTN, 2, 8, launch_attn_kivirtn_n2_b8)
