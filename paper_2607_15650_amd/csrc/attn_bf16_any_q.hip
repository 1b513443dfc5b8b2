// attn_bf16_any_q.hip - the hand-scheduled bf16 attention kernel for query
// tensors that are not 16-byte aligned: the same source, its query rows staged
// through registers.  A file of its own so that the two compile side by side
// (a minute each).
#define DITANGO_ANY_Q
#include "attn_bf16.hip"
