// All bins in one launch: the plane families that the default and the autotuned
// packings of uneven robots use (8 contacts in registers).
#define SIMK_MULTI_SET 0
#define SIMK_MULTI_FAMILIES(X)                                                                 \
  X(8, 1, 8) X(12, 1, 8) X(16, 1, 8) X(16, 2, 8) X(16, 2, 16) X(20, 1, 4) X(20, 1, 8) X(20, 2, 8)  \
  X(24, 1, 8) X(24, 2, 8) X(28, 2, 8)
#include "../rollout_multi.inc"
