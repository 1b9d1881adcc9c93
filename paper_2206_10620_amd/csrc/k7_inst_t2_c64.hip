// Row-stacked matrix-core kernel, two rows per wavefront, tiles of 64 columns.
#define PPC_T 2
#define PPC_TC 64
#define PPC_FN k7_lookup_t2_c64
#define PPC_ONE
#define PPC_TWO
#include "k7_inst.inc"
