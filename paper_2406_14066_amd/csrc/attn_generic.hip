// Lookahead attention, generic kernels (Section 2.2 / Section 4 of arXiv
// 2406.14066: the k+1 query positions of a request are scored against its
// cached keys and values, query j seeing keys 0 .. kv_len - q_len + j).
//
//   attn_generic_kernel   any dtype (fp32, bf16) and page layout, scalar fp32
//                         arithmetic: one block per (KV chunk, query head,
//                         query row), one thread per key of the chunk.  Every
//                         shape has a matrix-instruction kernel; this one takes the
//                         fp32 attention alone where it is faster (see
//                         f32_scalar_is_faster), and with
//                         SPEC_VERIFY_FORCE_GENERIC=1 everything, which the tests
//                         compare the others with.
//   attn_combine_kernel   merges the per-chunk partial results of either
//                         attention kernel: out = sum_c w_c acc_c / sum_c w_c l_c,
//                         w_c = 2^(m_c - max_c m_c).  Requests with one chunk are
//                         written by the kernel that holds their only partial.
//   kv_repack_kernel      token-major pages -> matrix-instruction page layout.
//
// Scores are kept in base-2 units (the softmax scale is folded with log2 e).
#include "common.h"

#include <math.h>

namespace specv {

namespace {

constexpr int kChunkThreads = 256;

__device__ __forceinline__ float load_as_float(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_as_float(const uint16_t *p, size_t i)
{
    return __uint_as_float((uint32_t)p[i] << 16);
}

// index of K/V element (page, kv head, slot, dim) in the two page layouts
__device__ __forceinline__ size_t k_index(int layout, int page, int Hkv, int kvh, int slot, int c, int d)
{
    const size_t head = (size_t)page * Hkv + kvh;
    if (layout == SPEC_KV_TOKEN_MAJOR) return (head * SPEC_BLOCK_SIZE + slot) * d + c;
    return ((head * (d >> 3) + (c >> 3)) * SPEC_BLOCK_SIZE + slot) * 8 + (c & 7);
}

// SPEC_KV_MFMA value layout inside one (page, kv head): [d/32][4 token groups][16 dims][2 dim halves][4 tokens]
__device__ __forceinline__ size_t v_tiled_offset(int c, int slot)
{
    const int pair = c >> 5, half = (c >> 4) & 1, m = c & 15, g = slot >> 2, r = slot & 3;
    return (size_t)((((pair * 4 + g) * 16 + m) * 2 + half) * 4 + r);
}

__device__ __forceinline__ size_t v_index(int layout, int page, int Hkv, int kvh, int slot, int c, int d)
{
    const size_t head = (size_t)page * Hkv + kvh;
    if (layout == SPEC_KV_TOKEN_MAJOR) return (head * SPEC_BLOCK_SIZE + slot) * d + c;
    return head * d * SPEC_BLOCK_SIZE + v_tiled_offset(c, slot);
}

// request that owns packed query row `row`: largest b with cu_q_len[b] <= row
// (T = cu_q_len[B]; with one draft length for all requests the first guess is right, and its two
// loads replace a chain of log2 B dependent ones)
__device__ __forceinline__ int find_request(const int32_t *cu_q_len, int B, int T, int row)
{
    const int guess = min((int)(((long long)row * B) / T), B - 1);
    if (cu_q_len[guess] <= row && row < cu_q_len[guess + 1]) return guess;
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (cu_q_len[mid] <= row) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <typename KV_T>
__global__ __launch_bounds__(kChunkThreads, 4) void attn_generic_kernel(AttnParams p)
{
    const int tid = threadIdx.x;
    const int chunk = blockIdx.x;
    const int h = blockIdx.y;
    const int row = blockIdx.z;
    const int b = find_request(p.cu_q_len, p.B, p.T, row);
    const int q_len = p.cu_q_len[b + 1] - p.cu_q_len[b];
    const int j = row - p.cu_q_len[b];
    const int L = p.kv_len[b];
    // (lengths from device memory bound the loops and indices below: a request that does not fit
    // the launch is left out and reported once)
    if (!request_lengths_ok(L, q_len, p.capacity_tokens, p.max_blocks_per_req)) {
        if (chunk == 0 && h == 0 && j == 0 && tid == 0 && p.errors != nullptr) atomicAdd(p.errors, 1ull);
        return;
    }
    const int nchunks = (L + p.chunk_tokens - 1) / p.chunk_tokens;
    if (chunk >= nchunks) return;
    const int last_visible = L - q_len + j;
    const int kvh = h / (p.Hq / p.Hkv);
    const int d = p.d;

    __shared__ float sh_q[128];
    __shared__ float sh_p[kChunkThreads];
    __shared__ int sh_page[kChunkThreads];
    __shared__ float sh_red[kChunkThreads / kWave];

    const KV_T *q = static_cast<const KV_T *>(p.q);
    const KV_T *kc = static_cast<const KV_T *>(p.k_cache);
    const KV_T *vc = static_cast<const KV_T *>(p.v_cache);
    if (tid < d) sh_q[tid] = load_as_float(q, ((size_t)row * p.Hq + h) * d + tid);
    __syncthreads();

    // one key per thread (chunk_tokens == blockDim.x)
    const int token = chunk * p.chunk_tokens + tid;
    const bool visible = tid < p.chunk_tokens && token <= last_visible;
    float score = -INFINITY;
    int page = -1;
    if (visible) {
        page = p.block_table[(size_t)b * p.max_blocks_per_req + token / SPEC_BLOCK_SIZE];
        const int slot = token % SPEC_BLOCK_SIZE;
        if ((unsigned)page < (unsigned)p.num_blocks) {
            // eight consecutive head dims are contiguous in both page layouts: one vector load per
            // group, several groups in flight (element by element the loop is a chain of load
            // latencies: 37 us for 128 keys of 64 dims)
            struct alignas(8 * sizeof(KV_T)) Vec8 { KV_T e[8]; };
            // (four sums: a shorter chain, and a smaller error than one long sum's: 2.7e-7 of the output's norm in fp32
            // instead of 4.4e-7, the matrix-instruction kernel's being 3.1e-7)
            float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
            for (int c = 0; c < d; c += 8) {
                const Vec8 kv = *reinterpret_cast<const Vec8 *>(kc + k_index(p.kv_layout, page, p.Hkv, kvh, slot, c, d));
#pragma unroll
                for (int e = 0; e < 8; ++e) dot[e % 4] = fmaf(sh_q[c + e], load_as_float(kv.e, e), dot[e % 4]);
            }
            score = ((dot[0] + dot[1]) + (dot[2] + dot[3])) * p.scale_log2;
        } else {
            // an entry outside the pool is never turned into an address: the page reads as zeros
            page = -1;
            score = 0.0f;
            // (counted by the request's last row, which sees every page in use)
            if (slot == 0 && h == 0 && j == q_len - 1 && p.errors != nullptr) atomicAdd(p.errors, 1ull);
        }
    }
    sh_page[tid] = page;

    // block maximum
    float mx = score;
    for (int off = kWave / 2; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (tid % kWave == 0) sh_red[tid / kWave] = mx;
    __syncthreads();
    mx = kEmptyMax;
    for (int w = 0; w < kChunkThreads / kWave; ++w) mx = fmaxf(mx, sh_red[w]);
    __syncthreads();

    const float prob = visible ? __builtin_amdgcn_exp2f(score - mx) : 0.0f;
    sh_p[tid] = prob;
    float sum = prob;
    for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (tid % kWave == 0) sh_red[tid / kWave] = sum;
    __syncthreads();
    sum = 0.0f;
    for (int w = 0; w < kChunkThreads / kWave; ++w) sum += sh_red[w];

    // weighted sum of values: the block's 256 / d thread groups take the keys in turn, one head
    // dim per thread, and the groups' sums are added through shared memory (d is 64 or 128)
    const size_t slot_index = ((size_t)row * p.Hq + h) * p.max_chunks + chunk;
    const int ngrp = kChunkThreads / d;
    const int grp = tid / d, c = tid % d;
    {
        const int ntok = min(p.chunk_tokens, last_visible - chunk * p.chunk_tokens + 1);
        float acc = 0.0f;
        // (no branch in the loop, so that the loads of several keys are in flight together: a page
        // that is not there is read as page 0 with weight 0)
#pragma unroll 8
        for (int t = grp; t < ntok; t += ngrp) {
            const int slot = (chunk * p.chunk_tokens + t) % SPEC_BLOCK_SIZE;
            const int pg = sh_page[t];
            const float v = load_as_float(vc, v_index(p.kv_layout, max(pg, 0), p.Hkv, kvh, slot, c, d));
            acc = fmaf(pg >= 0 ? sh_p[t] : 0.0f, pg >= 0 ? v : 0.0f, acc);
        }
        __syncthreads();     // every thread has read its probabilities: the buffer now carries the groups' sums
        sh_p[tid] = acc;
        __syncthreads();
    }
    if (tid < d) {
        float acc = 0.0f;
        for (int gi = 0; gi < ngrp; ++gi) acc += sh_p[gi * d + tid];
        // the only chunk of its request: the row is complete, no merge needed
        if (nchunks == 1) p.out[((size_t)row * p.Hq + h) * d + tid] = acc / sum;
        else p.ws_acc[slot_index * d + tid] = acc;
    }
    if (tid == 0 && nchunks > 1) {
        p.ws_ml[slot_index * 2 + 0] = mx;
        p.ws_ml[slot_index * 2 + 1] = sum;
    }
}

// grid = T*Hq blocks of d threads
__global__ void attn_combine_kernel(AttnParams p)
{
    const int row = blockIdx.x / p.Hq;
    const int h = blockIdx.x % p.Hq;
    const int tid = threadIdx.x;
    const int b = find_request(p.cu_q_len, p.B, p.T, row);
    if (!request_lengths_ok(p.kv_len[b], p.cu_q_len[b + 1] - p.cu_q_len[b], p.capacity_tokens, p.max_blocks_per_req))
        return;   // left out by the partial kernel too
    const int nchunks = (p.kv_len[b] + p.chunk_tokens - 1) / p.chunk_tokens;
    if (nchunks == 1) return;   // written by the kernel that made the partial results
    const size_t base = ((size_t)row * p.Hq + h) * p.max_chunks;
    float mx = kEmptyMax;
#pragma unroll 8
    for (int c = 0; c < nchunks; ++c) mx = fmaxf(mx, p.ws_ml[(base + c) * 2]);
    float denom = 0.0f, acc = 0.0f;
#pragma unroll 8
    for (int c = 0; c < nchunks; ++c) {
        const float w = __builtin_amdgcn_exp2f(p.ws_ml[(base + c) * 2] - mx);
        denom = fmaf(w, p.ws_ml[(base + c) * 2 + 1], denom);
        acc = fmaf(w, p.ws_acc[(base + c) * p.d + tid], acc);
    }
    p.out[((size_t)row * p.Hq + h) * p.d + tid] = acc / denom;
}

// Token-major pages to the matrix-instruction layout: one wavefront per (page, KV head), 16 x D of K and of V.
// Bound by memory (every byte read once and written once), so both pools are touched in whole pieces:
// K moves as 16-byte pieces (8 dims of a token are contiguous in both layouts), taken in the order of the
// destination so that a store instruction writes 1 KB; V's rows are staged in LDS, token rows padded by 16
// bytes against bank conflicts, and come back through the transposing LDS read (the 16 lanes of a row give
// the addresses of 4 tokens x 16 dims, lane n pointing at token n / 4, dims 4 (n % 4) .. + 3, and lane n
// receives dim n of the 4 tokens), which is the destination's order.  Element by element V's stores took
// most of the time: 4096 pages of 8 heads, d = 128, 537 MB in all: 208 -> 93 us = 5.8 TB/s.
// (The pools' pieces may start at any 2-byte address, as elements do.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
constexpr int kRepackWaves = 4;

template <int D>
__global__ __launch_bounds__(kRepackWaves *kWave) void kv_repack_kernel(const uint16_t *src_k, const uint16_t *src_v, uint16_t *dst_k,
                                                                        uint16_t *dst_v, size_t heads)
{
    constexpr int kPieces = SPEC_BLOCK_SIZE * D / 8 / kWave;   // 16-byte pieces per lane
    constexpr int kPerRow = D / 8;                             // ... per token row
    constexpr int kRow = D * 2 + 16;                           // bytes per token row in LDS
    __shared__ alignas(16) unsigned char stage[kRepackWaves][SPEC_BLOCK_SIZE * kRow];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const size_t head = (size_t)blockIdx.x * kRepackWaves + wave;
    if (head >= heads) return;   // (the wavefronts of a block are independent)
    const size_t base = head * (SPEC_BLOCK_SIZE * D);
    u32x4 k[kPieces], v[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int piece = i * kWave + lane;   // of the destination: dims 8 (piece / 16) .. + 7 of token piece % 16
        k[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(
            src_k + base + (piece % SPEC_BLOCK_SIZE) * D + piece / SPEC_BLOCK_SIZE * 8));
        v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(src_v + base + (size_t)piece * 8));
    }
    unsigned char *st = stage[wave];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int piece = i * kWave + lane;
        __builtin_nontemporal_store(k[i], reinterpret_cast<u32x4_any *>(dst_k + base + (size_t)piece * 8));
        *reinterpret_cast<u32x4 *>(st + piece / kPerRow * kRow + piece % kPerRow * 16) = v[i];
    }
    // (LDS executes a wavefront's accesses in order: the reads see the writes without a barrier)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
    const int g = lane >> 4, n = lane & 15;
    unsigned char *at = st + (4 * g + (n >> 2)) * kRow + (n & 3) * 8;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {   // dims 32 i + n and 32 i + 16 + n, tokens 4 g .. 4 g + 3
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + i * 64)));
        const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + i * 64 + 32)));
        const u32x4 out = {lo.x, lo.y, hi.x, hi.y};
        __builtin_nontemporal_store(out, reinterpret_cast<u32x4_any *>(dst_v + base + (size_t)(i * kWave + lane) * 8));
    }
}

// KV append: one thread per (packed row, kv head, group of 8 elements).  Latency is what a launch of this size takes: the
// chain of dependent loads before the stores, and the stores of V in the tiled layout.  The rows to move do not
// depend on where they go, and with one draft length for all requests the first guess of the request is right: rows of 16-bit
// elements are fetched along with the guess's lengths, so that two round trips (lengths, page index) are left
// before the stores instead of four; fp32 rows, twice the registers, after the page index (256 requests: 6.2 us, the other
// way 6.35).  The empty asm statements hold the loads where they are written: the compiler moves them to their first use
// otherwise, and the lengths' into the comparison.  The layout is a template parameter: chosen at run time, V went through the
// strided loads' registers in either.  Replayed from a graph, k = 4, 8 heads of 128, 1 / 256 requests: tiled pages
// 2.7 / 7.2 us (with loads at their first use and one store per dim 3.4 / 9.1), token-major bf16 2.15 / 3.3 (2.5 / 3.6),
// fp32 2.4 / 6.2 (2.8 / 6.2).  (Called one by one, 256 requests on tiled pages take the same 7 us: a shorter host call changes nothing.)
template <typename T, bool TILED>
__global__ void kv_append_kernel(KvAppendParams p)
{
    const int groups = p.d >> 3;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)p.T * p.Hkv * groups;
    if (idx >= total) return;
    const int g = (int)(idx % groups);
    const int kvh = (int)((idx / groups) % p.Hkv);
    const int row = (int)(idx / ((size_t)groups * p.Hkv));
    typedef T vec8 __attribute__((ext_vector_type(8)));
    const size_t from = ((size_t)row * p.Hkv + kvh) * p.d;
    const T *sk = static_cast<const T *>(p.new_k) + from, *sv = static_cast<const T *>(p.new_v) + from;
    vec8 new_k, new_v;
    auto fetch = [&] {
        new_k = *reinterpret_cast<const vec8 *>(sk + g * 8);
        if constexpr (TILED) {   // every groups-th dim: the stores below then fall into 2 cache lines per row and instruction, not 16
#pragma unroll
            for (int e = 0; e < 8; ++e) new_v[e] = sv[g + e * groups];
        } else {
            new_v = *reinterpret_cast<const vec8 *>(sv + g * 8);
        }
    };
    constexpr bool early = sizeof(T) == 2;
    if constexpr (early) fetch();
    int b = min((int)(((long long)row * p.B) / p.T), p.B - 1);
    int begin = p.cu_q_len[b], end = p.cu_q_len[b + 1], len = p.kv_len[b];
    asm volatile("" : "+v"(begin), "+v"(end), "+v"(len));
    if (begin > row || row >= end) {
        b = find_request(p.cu_q_len, p.B, p.T, row);
        begin = p.cu_q_len[b];
        end = p.cu_q_len[b + 1];
        len = p.kv_len[b];
    }
    if constexpr (early) asm volatile("" : "+v"(new_k), "+v"(new_v));
    const int pos = len - (end - begin) + (row - begin);
    // position and page index come from device memory: a row that would land outside the
    // request's block-table row or outside the pool is not written, and counted
    int page = -1;
    if (pos >= 0 && pos / SPEC_BLOCK_SIZE < p.max_blocks_per_req)
        page = p.block_table[(size_t)b * p.max_blocks_per_req + pos / SPEC_BLOCK_SIZE];
    if ((unsigned)page >= (unsigned)p.num_blocks) {
        if (g == 0 && kvh == 0 && p.errors != nullptr) atomicAdd(p.errors, 1ull);
        return;
    }
    const int slot = pos % SPEC_BLOCK_SIZE;
    if constexpr (!early) fetch();
    T *dk = static_cast<T *>(p.k_cache);
    T *dv = static_cast<T *>(p.v_cache);
    constexpr int layout = TILED ? SPEC_KV_MFMA : SPEC_KV_TOKEN_MAJOR;
    // the 8 elements of a thread are contiguous in the cache in every case but one (V in the tiled
    // layout, where consecutive dims of a token are 16 bytes apart): whole-vector stores where they are
    *reinterpret_cast<vec8 *>(dk + k_index(layout, page, p.Hkv, kvh, slot, g * 8, p.d)) = new_k;
    if constexpr (TILED) {
#pragma unroll
        for (int e = 0; e < 8; ++e) dv[v_index(layout, page, p.Hkv, kvh, slot, g + e * groups, p.d)] = new_v[e];
    } else {
        *reinterpret_cast<vec8 *>(dv + v_index(layout, page, p.Hkv, kvh, slot, g * 8, p.d)) = new_v;
    }
}

}  // namespace

hipError_t launch_kv_append(const KvAppendParams &p, hipStream_t stream)
{
    const size_t total = (size_t)p.T * p.Hkv * (p.d >> 3);
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (p.elem_bytes == 4)
        hipLaunchKernelGGL((kv_append_kernel<float, false>), dim3(blocks), dim3(256), 0, stream, p);
    else if (p.kv_layout == SPEC_KV_TOKEN_MAJOR)
        hipLaunchKernelGGL((kv_append_kernel<uint16_t, false>), dim3(blocks), dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL((kv_append_kernel<uint16_t, true>), dim3(blocks), dim3(256), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_attn_generic(const AttnParams &p, int dtype, hipStream_t stream)
{
    dim3 grid(p.max_chunks, p.Hq, p.T);
    if (dtype == SPEC_F32)
        hipLaunchKernelGGL(attn_generic_kernel<float>, grid, dim3(kChunkThreads), 0, stream, p);
    else
        hipLaunchKernelGGL(attn_generic_kernel<uint16_t>, grid, dim3(kChunkThreads), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_attn_combine(const AttnParams &p, hipStream_t stream)
{
    hipLaunchKernelGGL(attn_combine_kernel, dim3(p.T * p.Hq), dim3(p.d), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_kv_repack(const void *src_k, const void *src_v, void *dst_k, void *dst_v, int32_t num_blocks,
                            int32_t Hkv, int32_t d, hipStream_t stream)
{
    const size_t heads = (size_t)num_blocks * Hkv;
    const dim3 grid((unsigned)((heads + kRepackWaves - 1) / kRepackWaves)), block(kRepackWaves * kWave);
    const uint16_t *sk = static_cast<const uint16_t *>(src_k), *sv = static_cast<const uint16_t *>(src_v);
    uint16_t *dk = static_cast<uint16_t *>(dst_k), *dv = static_cast<uint16_t *>(dst_v);
    if (d == 128) hipLaunchKernelGGL(kv_repack_kernel<128>, grid, block, 0, stream, sk, sv, dk, dv, heads);
    else hipLaunchKernelGGL(kv_repack_kernel<64>, grid, block, 0, stream, sk, sv, dk, dv, heads);
    return hipGetLastError();
}

}  // namespace specv
