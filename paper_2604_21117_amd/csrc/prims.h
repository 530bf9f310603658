// Device-wide primitives used by the build and insert paths: exclusive scans
// and a stable (key, index) sort.  Wave64 block helpers live here too.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gt {

// Inclusive scan over the 64 lanes of a wave (every lane active).  32-bit
// integers use DPP moves, which stay in the vector ALU: within each row of
// 16 lanes, steps adding the value 1, 2, 4 and 8 lanes below (a lane whose
// source lies outside its row adds 0), then row 0's total into row 1 and
// row 2's into row 3 (row broadcast of lane 15), then the total of rows 0-1
// into rows 2 and 3 (row broadcast of lane 31).  Other types shift with
// cross-lane reads, one LDS-path round trip per step, in the same order as
// before for floating point.
template <class T>
__device__ __forceinline__ T wave_incl_scan(T x) {
    if constexpr (sizeof(T) == 4 && static_cast<T>(-1) > static_cast<T>(0)) {
        int v = static_cast<int>(x);
        v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
        v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
        v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
        v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
        v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15, rows 1 and 3
        v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31, rows 2 and 3
        return static_cast<T>(v);
    } else {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            T y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        return x;
    }
}

// Exclusive scan across the block (blockDim.x a multiple of 64, <= 2048).
// `sh` needs 33 entries of shared memory.  All threads must call it.
template <class T>
__device__ __forceinline__ T block_excl_scan(T v, T* sh, T* total) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nw = blockDim.x >> 6;
    T inc = wave_incl_scan(v);
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    if (w == 0) {
        T s = lane < nw ? sh[lane] : T(0);
        T si = wave_incl_scan(s);
        if (lane < nw) sh[lane] = si - s;
        if (lane == nw - 1) sh[32] = si;
    }
    __syncthreads();
    T res = inc - v + sh[w];
    *total = sh[32];
    __syncthreads();
    return res;
}

// ------------------------------------------------------------ host side

// Largest batch rank_sort_small takes (all keys sit in each workgroup's LDS);
// up to kRankSortMax keys callers need no other buffer for a sort.
constexpr uint32_t kRankSortTop = 8192;
constexpr uint32_t kRankSortMax = 2048;

// Stable sort of B <= kRankSortTop keys by rank: sk[r] = keys[i] and
// si[r] = i, where r is the number of pairs (keys[j], j) before (keys[i], i)
// in (key, index) order.
template <class K>
void rank_sort_small(const K* keys, uint32_t B, K* sk, uint32_t* si, hipStream_t s);

// Scratch bytes needed by scan_exclusive for up to n elements.
uint64_t scan_tmp_bytes(uint64_t n);

// out[i] = sum of in[0..i) for i < n, where n = *n_dev if n_dev is given
// (n_max is then an upper bound used to size the grid), else n_max.  If
// `total` is non-null it receives the sum of all n inputs.  in == out is
// allowed.
template <class T>
void scan_exclusive(const T* in, T* out, T* total, const uint32_t* n_dev, uint64_t n_max,
                    void* tmp, hipStream_t s);

// Scratch bytes needed by sort_from for n elements.
uint64_t sort_tmp_bytes(uint64_t n, int key_bytes);

// Stable sort of (src[i], i) by key, n host-known: src is read, keys/idx
// receive the result, keys_alt/idx_alt are ping-pong buffers of n entries.  If
// the sort fails (never expected), err_bit is or-ed into *err (a device word,
// optional) and the result is every key 0, index i at position i.
template <class K>
void sort_from(const K* src, K* keys, uint32_t* idx, K* keys_alt, uint32_t* idx_alt, uint64_t n, void* tmp,
               hipStream_t s, uint32_t* err = nullptr, uint32_t err_bit = 1u);

// The sample sort (sample_sort.hip), which sort_from takes up to
// sample_sort_max() elements: a stable sort of (src[i], i) as sort_from
// describes it; tmp holds sample_sort_tmp_bytes, which is less than
// sort_tmp_bytes.  force_fail makes it report a
// failure (testing hook).
uint64_t sample_sort_max();
uint64_t sample_sort_tmp_bytes(uint64_t n, int key_bytes);
template <class K>
void sample_sort_from(const K* src, K* keys, uint32_t* idx, K* keys_alt, uint32_t* idx_alt, uint64_t n, void* tmp,
                      hipStream_t s, uint32_t* err, uint32_t err_bit, bool force_fail);

// Testing hooks of the sample sort: the largest input it takes (larger ones are
// radix-sorted) and the largest group it sorts in LDS (larger ones in device
// memory); each returns the previous value.
uint64_t set_sample_sort_max(uint64_t n);
uint32_t set_sample_sort_group(uint32_t pairs);

// Whether the testing hook makes a sort of n elements fail.
bool sort_forced_to_fail(uint64_t n);

// Empty look-back steps after which a sort gives up (process-wide; 0 makes
// every tile after the first give up at once).  Returns the previous value.
uint32_t set_sort_spin_limit(uint32_t limit);

}  // namespace gt
