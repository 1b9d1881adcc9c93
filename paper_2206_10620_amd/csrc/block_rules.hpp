// Which 16-byte pieces of x the binary16 block product may fetch with one direct load: shared by the kernels and by the host
// test that walks every piece of small matrices.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define PPC_BOTH __host__ __device__ __forceinline__
#else
#define PPC_BOTH inline
#endif

namespace ppc {

// A piece at byte offset `off` of a matrix of `x_bytes` bytes reaches behind its end (a matrix shorter than a piece: every piece
// does) and is fetched element by element.
PPC_BOTH bool k4_piece_ends_behind(uint32_t off, uint32_t x_bytes) { return x_bytes < 16u || off > x_bytes - 16u; }

// Rows that start before this offset have no such piece: their last one starts at most 2 bytes before the row's end.
PPC_BOTH uint32_t k4_edge_from(uint32_t x_bytes, uint32_t row_bytes) { return x_bytes > row_bytes + 14u ? x_bytes - row_bytes - 14u : 0u; }

}  // namespace ppc
