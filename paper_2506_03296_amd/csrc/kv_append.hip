// kv_append.hip -- paged KV-cache append (include/apex_kv_append.h).
//
// Each new token owns Hkv rows of d fp16 values in K and in V; each row is
// moved by d / 8 lanes with one 16-byte load and one 16-byte store per lane
// per cache.  A pass of a 256-lane work group covers 256 / (d / 8)
// consecutive (token, kv-head) rows, so the reads of a wave are contiguous in
// the new-row buffer and every write is a whole 16-byte-aligned piece of one
// cache row; a work group makes two passes.  Both rows' slots are asked for
// first, then the rows, and only those whose slot is in the pool: a padding or
// out-of-pool token costs its slot and nothing else.
//
// A decode step's append (a few hundred rows) is bound by the launch and one
// chain of instructions and round trips: divisions in 64 bits and one row after
// the other made it 3.7 us for 32 tokens of 8 kv-heads (back to back in a
// graph); with shifts (kPow2: vectors per row, kv-heads and block size are
// powers of two, else 32-bit divisions where they hold the slot) it takes 2.06.
// Asking for the rows together with the slots takes 1.98, but then padding is
// read too, which a bucketed prompt pays for: 54777 tokens, of them no, half,
// 95 % padding: 69.9, 50.9, 34.1 us that way, 70.9, 36.7, 7.9 this way (the
// divisions' kernel: 81.3, 37.5, 14.5).  A call without padding is bound by
// HBM, reads and writes together.  Rows per thread (one, two, four): 70.8, 70.9,
// 74.7 us there.
#include <hip/hip_runtime.h>

#include <limits.h>
#include <stdint.h>

#include "apex_kv_append.h"
#include "append_index.h"
#include "status.h"

namespace {

using apex::AppendShape;
using apex::fail;

constexpr int kAppendThreads = 256;
constexpr int kMaxRowVecs = kAppendThreads;   // d <= 2048
constexpr int kRows = 2;                      // rows per thread
constexpr int64_t kMaxGridX = 1 << 23;        // 2^31 threads
// The cache rows are written non-temporally: the attention that reads them
// streams past the caches.  The new rows come out of a projection that has
// just written them, so up to half the 256 MB Infinity Cache they are read
// through it (30082 tokens, 123 MB: 37.0 us, 45.1 non-temporally); larger ones
// cannot have stayed there and are read past it (224 MB: 84.2 against 82.7).
constexpr int64_t kCachedNewBytes = (int64_t)128 << 20;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <bool kPow2, bool kStream>
__global__ __launch_bounds__(kAppendThreads) void kv_append_kernel(
    const u32x4* __restrict__ k_new, const u32x4* __restrict__ v_new, u32x4* __restrict__ k_cache,
    u32x4* __restrict__ v_cache, const int64_t* __restrict__ slots, AppendShape s)
{
    const unsigned local_row = kPow2 ? threadIdx.x >> s.vec_shift : threadIdx.x / (unsigned)s.row_vecs;
    const unsigned c = threadIdx.x - local_row * (unsigned)s.row_vecs;
    if (local_row >= (unsigned)s.rows_per_pass) return;
    const int64_t group = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t base = group * s.rows_per_pass * kRows + local_row;
    u32x4 kv[kRows], vv[kRows];
    int64_t slot[kRows];
    unsigned t[kRows], g[kRows];
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int64_t r64 = base + (int64_t)i * s.rows_per_pass;
        const unsigned r = (unsigned)(r64 < s.rows ? r64 : s.rows - 1);
        t[i] = kPow2 ? r >> s.head_shift : r / (unsigned)s.Hkv;
        g[i] = r - t[i] * (unsigned)s.Hkv;
        const int64_t at = slots[t[i]];   // every row's slot is in flight before the first is needed
        slot[i] = r64 < s.rows && at < s.capacity ? at : -1;
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        if (slot[i] < 0) continue;
        const int64_t src = apex::append_source(s, t[i], g[i], c);
        kv[i] = kStream ? __builtin_nontemporal_load(&k_new[src]) : k_new[src];
        vv[i] = kStream ? __builtin_nontemporal_load(&v_new[src]) : v_new[src];
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        if (slot[i] < 0) continue;
        const int64_t dst = apex::append_target<kPow2>(s, slot[i], g[i], c);
        __builtin_nontemporal_store(kv[i], &k_cache[dst]);
        __builtin_nontemporal_store(vv[i], &v_cache[dst]);
    }
}

int log2_exact(int x)
{
    return x > 0 && (x & (x - 1)) == 0 ? __builtin_ctz((unsigned)x) : -1;
}

template <bool kPow2, bool kStream>
void launch_append(const void* k_new, const void* v_new, void* k_cache, void* v_cache, const int64_t* slots,
                   const AppendShape& s, hipStream_t stream)
{
    // a grid dimension holds fewer than 2^32 threads: a longer one wraps without
    // an error, so more groups than kMaxGridX go into a second dimension (an
    // even cut; the last row's surplus groups find no rows)
    const int64_t per_group = (int64_t)s.rows_per_pass * kRows;
    const int64_t groups = (s.rows + per_group - 1) / per_group;
    const int64_t y = (groups + kMaxGridX - 1) / kMaxGridX, x = (groups + y - 1) / y;
    kv_append_kernel<kPow2, kStream><<<dim3((unsigned)x, (unsigned)y), kAppendThreads, 0, stream>>>(
        (const u32x4*)k_new, (const u32x4*)v_new, (u32x4*)k_cache, (u32x4*)v_cache, slots, s);
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

bool overlaps(const void* a, size_t na, const void* b, size_t nb)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

}  // namespace

extern "C" int apex_kv_append(const void* k_new, const void* v_new, int64_t new_token_stride,
                              void* k_cache, void* v_cache, const int64_t* slot_mapping, int T,
                              int Hkv, int d, int block_size, int64_t num_blocks, void* stream)
{
    apex::clear_error();
    if (T < 0) return fail(APEX_ERR_INVALID_ARG, "T = %d is negative", T);
    if (Hkv <= 0 || block_size <= 0)
        return fail(APEX_ERR_INVALID_ARG, "Hkv = %d and block_size = %d must be positive", Hkv, block_size);
    if (num_blocks < 0) return fail(APEX_ERR_INVALID_ARG, "num_blocks is negative");
    if (d <= 0 || d % 8 != 0 || d / 8 > kMaxRowVecs)
        return fail(APEX_ERR_UNSUPPORTED, "head dim %d unsupported (a multiple of 8 up to %d)", d,
                    8 * kMaxRowVecs);
    const int64_t row_elems = (int64_t)Hkv * d;
    const int64_t stride = new_token_stride == 0 ? row_elems : new_token_stride;
    if (stride < row_elems || stride % 8 != 0)
        return fail(APEX_ERR_INVALID_ARG, "new_token_stride %lld must be 0 or a multiple of 8 >= Hkv * d",
                    (long long)new_token_stride);
    if ((int64_t)T * Hkv > INT_MAX) return fail(APEX_ERR_UNSUPPORTED, "T * Hkv exceeds 2^31 - 1");
    if (num_blocks > INT64_MAX / ((int64_t)Hkv * block_size * d * 2))
        return fail(APEX_ERR_INVALID_ARG, "cache size overflows");
    if (T == 0) return APEX_OK;
    if (!k_new || !v_new || !k_cache || !v_cache || !slot_mapping)
        return fail(APEX_ERR_INVALID_ARG, "a tensor pointer is NULL");
    if (!aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(k_cache, 16) || !aligned(v_cache, 16))
        return fail(APEX_ERR_INVALID_ARG, "k_new, v_new, k_cache and v_cache must be 16-byte aligned");
    if (!aligned(slot_mapping, 8)) return fail(APEX_ERR_INVALID_ARG, "slot_mapping must be 8-byte aligned");
    const size_t cache_bytes = (size_t)num_blocks * Hkv * block_size * d * 2;
    const size_t new_bytes = ((size_t)(T - 1) * stride + row_elems) * 2;
    if (overlaps(k_cache, cache_bytes, v_cache, cache_bytes))
        return fail(APEX_ERR_INVALID_ARG, "k_cache overlaps v_cache");
    const void* inputs[3] = {k_new, v_new, slot_mapping};
    const size_t input_bytes[3] = {new_bytes, new_bytes, (size_t)T * 8};
    for (int i = 0; i < 3; ++i)
        if (overlaps(inputs[i], input_bytes[i], k_cache, cache_bytes) ||
            overlaps(inputs[i], input_bytes[i], v_cache, cache_bytes))
            return fail(APEX_ERR_INVALID_ARG, "an input overlaps a cache");
    if (num_blocks == 0) return APEX_OK;   // every slot is out of the pool

    AppendShape s;
    s.rows = T * Hkv;
    s.Hkv = Hkv;
    s.row_vecs = d / 8;
    s.rows_per_pass = kAppendThreads / s.row_vecs;
    s.block_size = block_size;
    s.token_vecs = stride / 8;
    s.capacity = num_blocks * block_size;
    s.vec_shift = log2_exact(s.row_vecs);
    s.head_shift = log2_exact(Hkv);
    s.block_shift = log2_exact(block_size);
    const bool pow2 = s.vec_shift >= 0 && s.head_shift >= 0 && s.block_shift >= 0;
    const bool stream_in = 2 * (int64_t)s.rows * d * 2 > kCachedNewBytes;
    const auto launch = pow2 ? (stream_in ? launch_append<true, true> : launch_append<true, false>)
                             : (stream_in ? launch_append<false, true> : launch_append<false, false>);
    launch(k_new, v_new, k_cache, v_cache, slot_mapping, s, (hipStream_t)stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(APEX_ERR_HIP, "kv_append launch failed: %s", hipGetErrorString(e));
    return APEX_OK;
}
