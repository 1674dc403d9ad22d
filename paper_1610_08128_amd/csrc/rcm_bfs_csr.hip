// The team kernel's instance for graphs without a fixed-stride row copy.
#define RCM_ORDER_CSR
#include "rcm_bfs.hip"
