// Row-stacked matrix-core kernel, two rows per wavefront, tiles of 16 columns.
#define PPC_T 2
#define PPC_TC 16
#define PPC_FN k7_lookup_t2_c16
#define PPC_TWO
#include "k7_inst.inc"
