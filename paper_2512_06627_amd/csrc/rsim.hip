// Signature hashing for random-pattern simulation (gfx950).
//
// A sweeping flow proposes potentially equivalent node pairs from simulation
// signatures (paper, Section 2.3, step 1); a node and its complement are the
// same candidate, so each row is normalised to start with a 0 before it is
// hashed.  Row r of the signature matrix is hashed as
//     sum over words k of word'_k * (fmix32(k) | 1)   (mod 2^64)
// with word' = word XOR (all ones if bit 0 of word 0 is 1), fmix32 the
// MurmurHash3 32-bit finaliser (keys use k mod 2^32), and each product the
// exact 64-bit product of two 32-bit values.  The sum is order-free, so each
// lane accumulates its own words and one wave reduction finishes the row.
// The row's number of ones (before normalisation) is summed alongside; the
// paper's stability and entropy features (Section 3.2) derive from it.
//
// Work decomposition: a workgroup takes a group of one or two rows and its waves the 256-word
// chunks of their columns in turn; a lane reads four consecutive words of each row (1 KB per wave and
// row), the next chunk's while it works on one.  The keys depend on the column alone and are made
// once for the group: the finaliser's two multiplications and the 64-bit product run at a quarter of
// the vector rate, so that one row at a time asks for about 90 issue cycles per 64 words, 60% of the
// time that HBM takes to deliver them, and two rows for about 55.  The complement is taken out of the
// sum: sum (~w) * key = (2^32 - 1) * sum key - sum w * key.
//
// Bound by HBM reads: 3,111 x 100,003 words 209 us, 6.0 TB/s (a wave per row with 1 KB of loads in
// flight: 292 us, 4.3 TB/s), 1,870 x 131,706 165 us (308), 1,631 x 155,733 174 (369), 300 x 250,000 74 us
// (473: a row's chain of loads); matrices that stay in the memory-side cache 3,055 x 12,511 24 (27).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"

namespace fes {
namespace {

__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

constexpr int kMaxSplit = 16;  // waves a row group's columns are shared among

// Four words of R rows, their keys, into the sums.
template <int R>
__device__ __forceinline__ void accumulate(const uint32_t (&w)[R][4], const uint32_t (&key)[4], uint64_t (&sum)[2 * R],
                                           uint64_t& keys) {
#pragma unroll
    for (int u = 0; u < 4; ++u) keys += key[u];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        uint32_t bits = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            sum[j] += (uint64_t)w[j][u] * key[u];
            bits += (uint32_t)__builtin_popcount(w[j][u]);
        }
        sum[R + j] += bits;
    }
}

template <int R>
__device__ __forceinline__ void load_chunk(uint32_t (&w)[R][4], const uint32_t* const (&row)[R], uint64_t k) {
#pragma unroll
    for (int j = 0; j < R; ++j) __builtin_memcpy(w[j], row[j] + k, 16);
}

template <int R>
__global__ void __launch_bounds__(64 * kMaxSplit) signature_hash_kernel(const uint32_t* __restrict__ sig,
                                                                        uint64_t rows, uint64_t W,
                                                                        uint64_t* __restrict__ hash,
                                                                        uint64_t* __restrict__ ones,
                                                                        unsigned long long* __restrict__ start) {
    if (start && blockIdx.x == 0 && threadIdx.x == 0) *start = __builtin_amdgcn_s_memrealtime();
    constexpr int N = 2 * R;  // sums of a wave: of w * key for each row, of ones for each row
    __shared__ uint64_t part[kMaxSplit][N + 1];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), split = blockDim.x >> 6;
    const uint64_t full = W / 256u;
    for (uint64_t r0 = (uint64_t)blockIdx.x * R; r0 < rows; r0 += (uint64_t)gridDim.x * R) {
        const uint32_t* row[R];
#pragma unroll
        for (int j = 0; j < R; ++j) row[j] = sig + min(r0 + j, rows - 1) * W;  // past the last: again the last

        uint64_t sum[N] = {}, keys = 0;
        uint32_t next[R][4];
        if (wave < full) load_chunk<R>(next, row, wave * 256u + 4u * lane);
        for (uint64_t c = wave; c < full; c += split) {
            const uint64_t k = c * 256u + 4u * lane;
            uint32_t w[R][4], key[4];
            __builtin_memcpy(w, next, sizeof w);
            if (c + split < full) load_chunk<R>(next, row, k + split * 256u);
#pragma unroll
            for (int u = 0; u < 4; ++u) key[u] = fmix32((uint32_t)k + u) | 1u;
            accumulate<R>(w, key, sum, keys);
        }
        if (W % 256u && wave == full % split) {
            const uint64_t k = full * 256u + 4u * lane;
            uint32_t w[R][4], key[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = k + u < W;
                const uint64_t at = in ? k + u : W - 1;
#pragma unroll
                for (int j = 0; j < R; ++j) w[j][u] = row[j][at];
                key[u] = in ? fmix32((uint32_t)k + u) | 1u : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int j = 0; j < R; ++j) w[j][u] = k + u < W ? w[j][u] : 0u;
            }
            accumulate<R>(w, key, sum, keys);
        }

        // Each step of the first ones leaves a lane half of the sums to go on with.
        uint32_t off = 32;
#pragma unroll
        for (int half = N / 2; half > 0; half >>= 1, off >>= 1) {
            const bool upper = lane & off;
#pragma unroll
            for (int i = 0; i < half; ++i) {
                const uint64_t give = upper ? sum[i] : sum[i + half];
                sum[i] = (upper ? sum[i + half] : sum[i]) + __shfl_xor(give, off, 64);
            }
        }
#pragma unroll
        for (; off > 0; off >>= 1) sum[0] += __shfl_xor(sum[0], off, 64);
#pragma unroll
        for (uint32_t o = 32; o > 0; o >>= 1) keys += __shfl_xor(keys, o, 64);
        if (lane % (64u / N) == 0) part[wave][lane / (64u / N)] = sum[0];
        if (lane == 0) part[wave][N] = keys;
        __syncthreads();
        if (threadIdx.x < (uint32_t)R && r0 + threadIdx.x < rows) {
            const uint64_t r = r0 + threadIdx.x;
            uint64_t acc = 0, cnt = 0, all = 0;
            for (uint32_t v = 0; v < split; ++v) {
                acc += part[v][threadIdx.x];
                cnt += part[v][R + threadIdx.x];
                all += part[v][N];
            }
            hash[r] = sig[r * W] & 1u ? all * 0xFFFFFFFFu - acc : acc;
            ones[r] = cnt;
        }
        __syncthreads();
    }
}

}  // namespace

// Rows per group: two where that leaves a group per CU (600 x 250,000 words: 136 us, one at a time
// 186; with groups of four the latency of their reduction shows on short rows, 6,000 x 300: 8.7 us
// against 6.8, and long ones gain nothing).  Then up to 16 waves a CU (with a chunk in hand and one on
// the way that is 64 KB per CU in flight; 3,055 x 12,511: 29 us, with 32 waves 34), the same number on
// each SIMD where a group has more than four: 1,631 x 155,733 in groups of five waves 251 us, of four
// 174; 600 x 250,000 in thirteens 134, in eights 107.  A group's waves share its chunks out evenly.
hipError_t launch_signature_hash_from(const uint32_t* sig, uint64_t rows, uint64_t words, uint64_t* hash,
                                      uint64_t* ones, int cus, unsigned long long* start, hipStream_t stream) {
    if (!sig || !hash || !ones || rows == 0 || words == 0 || cus <= 0) return hipErrorInvalidValue;
    const uint64_t per = rows >= 2ull * cus ? 2 : 1;
    const uint64_t groups = (rows + per - 1) / per, chunks = (words + 255) / 256;
    const uint64_t room = std::clamp<uint64_t>(16ull * cus / groups, 1, kMaxSplit);
    const uint64_t most = room >= 16 ? 16 : room >= 8 ? 8 : std::min<uint64_t>(room, 4);
    const uint64_t turns = (chunks + most - 1) / most, split = (chunks + turns - 1) / turns;
    const dim3 grid((uint32_t)std::min<uint64_t>(groups, 1u << 20)), block((uint32_t)(64 * split));
    if (per == 2) hipLaunchKernelGGL(signature_hash_kernel<2>, grid, block, 0, stream, sig, rows, words, hash, ones, start);
    else hipLaunchKernelGGL(signature_hash_kernel<1>, grid, block, 0, stream, sig, rows, words, hash, ones, start);
    return hipGetLastError();
}

hipError_t launch_signature_hash(const uint32_t* sig, uint64_t rows, uint64_t words, uint64_t* hash, uint64_t* ones,
                                 int cus, hipStream_t stream) {
    return launch_signature_hash_from(sig, rows, words, hash, ones, cus, nullptr, stream);
}

namespace {
const bool g_registered = (register_hash(&launch_signature_hash_from), true);
}

}  // namespace fes
