// The team kernel's instance for work-groups of 512 threads.
#define RCM_ORDER_WIDE
#include "rcm_bfs.hip"
