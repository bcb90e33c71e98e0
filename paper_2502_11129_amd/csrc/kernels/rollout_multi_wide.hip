// All bins in one launch, 16 contacts in registers for the families of up to 16
// DoFs (the tuned packing's 8 for its 16-DoF bin as well).
#define SIMK_MULTI_SET 1
#define SIMK_MULTI_FAMILIES(X)                                                                 \
  X(8, 1, 16) X(12, 1, 16) X(16, 1, 8) X(16, 1, 16) X(16, 2, 16) X(20, 1, 4) X(20, 1, 8) X(20, 2, 8)  \
  X(24, 1, 8) X(24, 2, 8) X(28, 2, 8)
#include "../rollout_multi.inc"
