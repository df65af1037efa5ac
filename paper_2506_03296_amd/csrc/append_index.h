// append_index.h -- where the rows of a paged KV append lie: vectors of eight
// fp16 values in the new-row buffer and in a cache.  Compiled for the device
// (the kernel) and the host (tests).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace apex {

// The shape of a call: vectors per row, rows per pass of a work group, and
// (kPow2 builds) the logarithms of vectors per row, kv-heads and block size.
struct AppendShape {
    int rows, Hkv, row_vecs, rows_per_pass, block_size;
    int vec_shift, head_shift, block_shift;
    int64_t token_vecs, capacity;
};

// Vector c of kv-head g's row of token t.  (Hkv row_vecs may pass 2^32: a
// token's row of 2^29 kv-heads of d = 64 is that long.)
__host__ __device__ inline int64_t append_source(const AppendShape& s, unsigned t, unsigned g, unsigned c)
{
    return (int64_t)t * s.token_vecs + (int64_t)g * s.row_vecs + c;
}

// Vector c of kv-head g's row at `slot` (in the pool).
template <bool kPow2>
__host__ __device__ inline int64_t append_target(const AppendShape& s, int64_t slot, unsigned g, unsigned c)
{
    int64_t block, pos;
    if (kPow2) {
        block = slot >> s.block_shift;
        pos = slot & (s.block_size - 1);
    } else if (((uint64_t)slot >> 32) == 0) {
        block = (unsigned)slot / (unsigned)s.block_size;
        pos = slot - block * s.block_size;
    } else {
        block = slot / s.block_size;
        pos = slot - block * s.block_size;
    }
    return ((block * s.Hkv + g) * s.block_size + pos) * s.row_vecs + c;
}

}  // namespace apex
