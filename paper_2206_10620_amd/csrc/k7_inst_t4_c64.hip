// Row-stacked matrix-core kernel, four rows per wavefront, tiles of 64 columns.
#define PPC_T 4
#define PPC_TC 64
#define PPC_FN k7_lookup_t4_c64
#define PPC_ONE
#include "k7_inst.inc"
