// The matrix-core decode kernel with two pairs of waves per work-group, for launches of few work-groups.
#define KVQ_DECODE_PAIRS 2
#include "kvq_decode_mfma.hip"
