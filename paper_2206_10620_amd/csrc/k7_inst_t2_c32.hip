// Row-stacked matrix-core kernel, two rows per wavefront, tiles of 32 columns.
#define PPC_T 2
#define PPC_TC 32
#define PPC_FN k7_lookup_t2_c32
#define PPC_ONE
#define PPC_TWO
#include "k7_inst.inc"
