// The speculative-verification step as ONE kernel launch (arXiv 2406.14066:
// "score" = lookahead attention of the k+1 query positions against the paged KV
// cache, Section 2.2 / Section 4; "accept" = rejection sampling with bonus token,
// Section 4; the accept rule is the cited speculative-sampling method's).
//
// The grid is a list of work items; a block's index selects its role:
//
//   statistics   one (logit row, vocabulary segment) each: offset and sum of
//                exponentials, published with the call's generation tag.
//   race         one (request, vocabulary segment) each: computes its random variates, recomputes the
//                request's (cheap) accept chain from the published statistics, then races
//                its segment for the next token.
//   final        one per group of requests: picks the race winners, writes the requests'
//                outputs and adds up their counters.
//   attention    one (request, KV head, KV chunk) each; the block that completes
//                the LAST chunk of a (request, KV head) merges the chunk partials
//                and writes the output.
// Other acceptance rules reuse the stages: greedy acceptance computes (largest logit,
// lowest id) per (target row, segment) in the statistics stage and has no race; a
// point-mass draft needs statistics of the target rows only and leaves the rejected
// token out of the race.
// Large batches take the statistics items in position order and skip the rows after a request's
// first rejection (stats_role): the accept chain of a request stops there (Section 4), so those rows
// decide nothing.  A block finds out by waiting for the earlier positions or by looking at what they
// have published (kStopWait, kStopPeek; 96 requests on 64/8 heads, k = 7, V = 32000: 97.7 us with all rows read,
// 93.3 waiting, 86.7 looking; the planner says which).
// The rejection items keep that order among themselves and are mixed into the first part
// of the attention items (see GridSplit), so that the rejection half, whose stages depend
// on each other, runs underneath the attention stream and is done before it.
//
// Attention blocks never wait: "last one out merges" is decided with one atomic
// ticket per (request, KV head).  Race and final items consume what earlier items
// of the grid published (tagged with the call's generation).  The producers precede
// the consumers in the grid, so they were dispatched before them, and they wait for
// nothing: the bounded wait that checks for the data always ends.  (Same-address atomic
// tickets cost about 0.3 us per arrival here, so they are kept for the attention chunks,
// which arrive spread out in time, and avoided for the hundreds of statistics blocks of a
// request, which arrive together.)  Tickets and records carry the call's generation tag
// in their high half, so a workspace needs no zero-initialisation and a call that never
// finished cannot poison the next; the last user also resets them, so a replayed HIP
// graph (same tag) works too.
//
// Attention arithmetic, per 16-token page and 16-row tile (lane = 16*g + n):
//   S^T[token][row] = K[token][:] . Q[row][:]        4 x v_mfma_f32_16x16x32_bf16
//   base-2 online softmax on the lane's tokens 4g..4g+3 of query row n
//   O^T[dim][row] += V^T[dim][token] . P^T[token][row]   8 x v_mfma_f32_16x16x16_bf16,
//   P^T being S^T's own accumulator layout; P is fed as bf16 high + low parts so
//   that its rounding does not limit the result.  All q_len * (Hq/Hkv) query rows
//   sharing a KV head are fused into the N dimension: K and V are read once.
//
// fp32 caches take a kernel of their own with the same grid (f32_step_kernel, attn_f32_role).
//
// Rejection arithmetic: the streaming part is fp32; what happens once per row or
// per decision (segment sums, log-sum-exp, p/q of the draft token, the comparison
// with u) is fp64.
#include "common.h"
#include "bounded_wait.h"
#include "grid_split.h"

#include <hip/hip_ext.h>

#include <float.h>
#include <math.h>
#include <stddef.h>
#include <string.h>

#include <type_traits>

namespace specv {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kD = 128;   // head dim of the main variants (those for 64: see head_dim_of)
constexpr int kBufferFlags = 0x00020000;   // raw 32-bit buffer descriptor, word 3
// Cache policy of the loads that stream data read once (KV pages, the race's logit rows):
// non-temporal, i.e. the lines are first in line for replacement in the L2.  Without it the
// stream pushes out what the blocks do come back to (code, block tables, queries, hand-off
// words); measured on the four large workloads the hint alone takes 8-10% off the step.
constexpr int kStreamPolicy = 2;           // "nt" bit of a raw buffer load
constexpr float kRescaleSlack = 8.0f;      // see the online softmax of the attention role
constexpr int kXcds = kXcdCount;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Exchanges between the four 16-lane rows of a wavefront with the gfx950 row-swap instructions
// (vector ALU, a few cycles) instead of a round trip through the LDS crossbar, which is what a
// generic lane shuffle by 16 or 32 compiles to: v_permlane16_swap trades the odd rows of its
// first operand with the even rows of its second, v_permlane32_swap the upper half of the first
// with the lower half of the second.  Fed the same value twice, the two results hold, in every
// lane l, the values of lanes l and l ^ 16 (l ^ 32).
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float max_across_xor16(float v)
{
    const u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_across_xor32(float v)
{
    const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_across_rows(float v)   // over lanes l, l ^ 16, l ^ 32, l ^ 48
{
    u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One gfx950 transposing LDS read: the 16 lanes of a row give the addresses of a 4 x 16 block of 16-bit
// elements, 8 bytes each (lane n: block row n / 4, elements 4 (n % 4) .. + 3), and lane n receives block
// column n.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 read_transposed(const unsigned char *src)
{
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)src));
}

// ---------------------------------------------------------------------------
// Tickets.  Word = generation << 32 | arrivals.  Returns how many blocks arrived
// before this one.  The common case is one atomic add: the word carries this call's
// generation already.  The first arrivals of a call find something else (garbage, the
// zero its last user left, or either plus what other early arrivals added) and replace
// it; the last arrival, which is the one the merge waits for, is never among them.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t ticket_arrive(unsigned long long *ticket, uint32_t generation)
{
    const unsigned long long got = atomicAdd(ticket, 1ull);
    if ((uint32_t)(got >> 32) == generation) return (uint32_t)got;
    unsigned long long cur = got + 1ull;
    for (;;) {
        const unsigned long long first = ((unsigned long long)generation << 32) | 1ull;
        const unsigned long long seen = atomicCAS(ticket, cur, first);
        if (seen == cur) return 0u;
        if ((uint32_t)(seen >> 32) == generation) return (uint32_t)atomicAdd(ticket, 1ull);
        cur = seen;
    }
}

__device__ __forceinline__ void ticket_reset(unsigned long long *ticket)
{
    __hip_atomic_store(ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Data handed from one block to another inside the launch (chunk partials, row
// statistics) is written and read with relaxed agent-scope atomic accesses, which
// go past the non-coherent cache levels, and published by waiting for the
// writes to complete before the ticket is taken.  A full agent-scope fence would
// also write back and invalidate the whole L2 of the XCD on every block; that is
// far too slow for thousands of blocks.
__device__ __forceinline__ void publish_u64(unsigned long long *dst, unsigned long long v)
{
    __hip_atomic_store(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long fetch_u64(const unsigned long long *src)
{
    return __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long pack_f32x2(float a, float b)
{
    return (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
}

// A 32-bit payload and the call's generation tag in one 8-byte word: written and read
// atomically, so a reader that finds this call's tag also has the payload, with no
// ordering needed between the words of a record.
__device__ __forceinline__ void publish_tagged(unsigned long long *dst, uint32_t payload, uint32_t generation)
{
    publish_u64(dst, (unsigned long long)payload | ((unsigned long long)generation << 32));
}

__device__ __forceinline__ bool tagged_ok(unsigned long long word, uint32_t generation)
{
    return (uint32_t)(word >> 32) == generation;
}

__device__ __forceinline__ void writes_complete()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);  // every outstanding store of this wavefront has been acknowledged
}

__device__ __forceinline__ void order_after_ticket()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Read-only inputs indexed by a block-uniform value (lengths, row offsets) are read through
// the constant address space, which makes them scalar loads: they are served by the scalar
// cache (these arrays are small and every block reads them) instead of a round trip to
// the L2 under load, and they have a wait counter of their own.
typedef const int32_t __attribute__((address_space(4))) *uniform_i32_ptr;
__device__ __forceinline__ int uniform_load(const int32_t *base, int index)
{
    return ((uniform_i32_ptr)(uintptr_t)base)[__builtin_amdgcn_readfirstlane(index)];
}

// ===========================================================================
// Rejection half
// ===========================================================================

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies,
// a word permutation with key xor, and a Weyl sequence on the key.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // full 64-bit products: one multiply instruction each instead of a high and a low one
        const unsigned long long pa = (unsigned long long)0xD2511F53u * (unsigned long long)c.x;
        const unsigned long long pb = (unsigned long long)0xCD9E8D57u * (unsigned long long)c.z;
        c = make_uint4((uint32_t)(pb >> 32) ^ c.y ^ k0, (uint32_t)pb, (uint32_t)(pa >> 32) ^ c.w ^ k1, (uint32_t)pa);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// The step counter of the random numbers: the launch's own, or, if the caller gave a device word
// (a captured launch that draws fresh numbers on every replay), what that word holds now.
struct StepWords {
    uint32_t lo, hi24;
};
typedef const unsigned long long __attribute__((address_space(4))) *uniform_u64_ptr;
__device__ __forceinline__ StepWords philox_step_words(const RejectParams &p)
{
    StepWords w = {p.step_lo, p.step_hi24};
    if (p.step_device != nullptr) {
        const unsigned long long s = *((uniform_u64_ptr)(uintptr_t)p.step_device);
        w.lo = (uint32_t)s;
        w.hi24 = (uint32_t)(s >> 32) & 0xFFFFFFu;
    }
    return w;
}

constexpr int kMaxStatSegments = 32;
constexpr int kMaxFinalGroup = 1 << kMaxFinalShift;
constexpr int kRaceVec = 8;                      // see the race
constexpr int kRacePart = kRaceVec * kThreads;   // vectors of 4 ids per part of the race
constexpr float kLog2eHi = 1.4426950216293335f;     // fp32(log2 e)
constexpr float kLog2eLo = 1.9259629911266175e-8f;  // log2 e - kLog2eHi

struct RejectShared {
    float red_f[kWaves];
    double red_d[kWaves];
    // target rows 0..k, then draft rows 0..k-1: sum_v 2^(x_v * log2(e) - row_off), row_off a whole number
    double row_sum[2 * SPEC_K_MAX + 1];
    float row_off[2 * SPEC_K_MAX + 1];
    double u[SPEC_K_MAX], ratio[SPEC_K_MAX];
    int accept[SPEC_K_MAX];
    int m, near;
    float best_score[kWaves];
    int best_id[kWaves];
    double seg_sum[2 * SPEC_K_MAX + 1][kMaxStatSegments];
    float seg_off[2 * SPEC_K_MAX + 1][kMaxStatSegments];
    // final stage: per request of the block
    int fin_ready[kMaxFinalGroup], fin_need[kMaxFinalGroup], fin_id[kMaxFinalGroup];
    int pos_count[SPEC_K_MAX + 2][kWaves], pos_request;   // see position_item
    uint32_t fin_count[2];
    f32x4 variates[kRaceVec][kThreads];   // 1 / e_v of a race block's part, each thread its own
};

// Streams one segment of a logit row through the block: `use(batch, x)` is called for each batch of
// kBatch vectors per thread, the vectors of thread t of batch i being (i * kBatch + u) * kThreads + t.
// DEPTH batches are in flight per thread: as soon as one is used its registers are refilled, so
// the memory system stays busy during the arithmetic (a pass that loads a whole batch of rows, waits
// and then computes leaves it idle in between, all blocks of a rejection-only launch in step: greedy
// acceptance of 256 requests, k = 3, V = 32000, 131 MB: 44.9 -> 35.7 us with the arg-max below).
// Vectors past the end read as zeros without touching memory (the descriptor ends with the segment).
constexpr int kBatch = 4;
template <int DEPTH, int POLICY, typename F>
__device__ __forceinline__ void stream_segment(const float *seg, int nvec, F use)
{
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(seg), 0, (uint32_t)nvec * 16u, kBufferFlags);
    f32x4 ring[DEPTH][kBatch];
    auto fetch = [&](int batch, f32x4(&x)[kBatch]) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            x[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                rsrc, (int)(((uint32_t)(batch * kBatch + u) * kThreads + threadIdx.x) * 16u), 0, POLICY));
    };
    const int nbatch = (nvec + kBatch * kThreads - 1) / (kBatch * kThreads);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        fetch(d, ring[d]);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay in ring order: a wait for one batch is not a wait for later ones
    }
    for (int i = 0; i < nbatch; i += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (i + d < nbatch) use(i + d, ring[d]);
            fetch(i + d + DEPTH, ring[d]);
        }
    }
}

// Sets what a batch holds past the end of the segment (zeros) to -inf.
__device__ __forceinline__ void mask_past_end(int batch, int nvec, f32x4 (&x)[kBatch])
{
    if ((batch + 1) * kBatch * kThreads <= nvec) return;   // the same for the whole block
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
        if ((batch * kBatch + u) * kThreads + (int)threadIdx.x >= nvec) x[u] = (f32x4){-INFINITY, -INFINITY, -INFINITY, -INFINITY};
}

__device__ __forceinline__ float max_of(const f32x4 &x) { return fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])); }

// One (row, segment): offset and sum of 2^(x*log2e - offset) over the segment.
// The running offset is integer-valued in base-2 units, so every rescale is an
// exact power of two and x*log2(e) - offset is rounded once (log2 e enters as an
// fp32 hi/lo pair inside fused multiply-adds).
template <int DEPTH>   // batches in flight per thread (these blocks share the attention role's register budget)
__device__ __forceinline__ void stats_block(const RejectParams &p, int row, int seg, RejectShared &sh)
{
    const int tid = threadIdx.x;
    const float *base = row < p.T ? p.target_logits + (size_t)row * p.V
                                  : p.draft_logits + (size_t)(row - p.T) * p.V;
    const int v0 = seg * p.stat_seg_len;
    const int v1 = min(p.V, v0 + p.stat_seg_len);
    const int nvec = (v1 - v0) >> 2;

    float m = -FLT_MAX;   // largest logit seen
    float off = kEmptyMax;
    float s = 0.0f;
    stream_segment<DEPTH, 0>(base + v0, nvec, [&](int batch, f32x4(&x)[kBatch]) {
        mask_past_end(batch, nvec, x);
        float cm = m;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) cm = fmaxf(cm, max_of(x[u]));
        if (cm > m) {
            const float new_off = ceilf(cm * kLog2eHi);
            s *= fast_exp2(off - new_off);
            off = new_off;
            m = cm;
        }
        const float noff = -off;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s += fast_exp2(fmaf(x[u][e], kLog2eHi, fmaf(x[u][e], kLog2eLo, noff)));
        }
    });

    const int wave = tid / kWave, lane = tid % kWave;
    float wm = off;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) wm = fmaxf(wm, __shfl_xor(wm, o));
    if (lane == 0) sh.red_f[wave] = wm;
    __syncthreads();
    float boff = sh.red_f[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) boff = fmaxf(boff, sh.red_f[w]);
    // one exact power-of-two rescale per thread, then the cross-thread sum in fp64
    double sd = (double)s * (double)fast_exp2(off - boff);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) sd += __shfl_xor(sd, o);
    if (lane == 0) sh.red_d[wave] = sd;
    __syncthreads();
    if (tid == 0) {
        double total = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) total += sh.red_d[w];
        // three tagged words: low and high half of the fp64 sum, and the offset
        unsigned long long *dst = p.stats + 3 * ((size_t)row * p.stat_segments + seg);
        const unsigned long long bits = (unsigned long long)__double_as_longlong(total);
        publish_tagged(dst + 0, (uint32_t)bits, p.generation);
        publish_tagged(dst + 1, (uint32_t)(bits >> 32), p.generation);
        publish_tagged(dst + 2, __float_as_uint(boff), p.generation);
    }
}

// Greedy mode: one (target row, segment): the largest logit and the lowest id that has it.
template <int DEPTH>
__device__ __forceinline__ void argmax_block(const RejectParams &p, int row, int seg, RejectShared &sh)
{
    const int tid = threadIdx.x;
    const float *base = p.target_logits + (size_t)row * p.V;
    const int v0 = seg * p.stat_seg_len;
    const int v1 = min(p.V, v0 + p.stat_seg_len);
    const int nvec = (v1 - v0) >> 2;
    // Per element only a maximum is taken (of three operands per instruction); the id is looked up when a
    // batch raises a thread's maximum, which gets rare after the first few.  Ids rise from batch to
    // batch and within one, so the first batch with the maximum and its lowest match are the answer.
    // (Nothing but -inf: the lowest id.)
    float best = -INFINITY;
    int best_id = tid < nvec ? v0 + 4 * tid : 0x7FFFFFFF;
    stream_segment<DEPTH, kStreamPolicy>(base + v0, nvec, [&](int batch, f32x4(&x)[kBatch]) {
        mask_past_end(batch, nvec, x);
        float cm = best;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) cm = fmaxf(cm, max_of(x[u]));
        if (cm > best) {
            best = cm;
#pragma unroll
            for (int u = kBatch - 1; u >= 0; --u) {
                const int id0 = v0 + 4 * ((batch * kBatch + u) * kThreads + tid);
#pragma unroll
                for (int e = 3; e >= 0; --e) best_id = x[u][e] == cm ? id0 + e : best_id;
            }
        }
    });
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o);
        const int oi = __shfl_xor(best_id, o);
        if (ov > best || (ov == best && oi < best_id)) { best = ov; best_id = oi; }
    }
    const int wave = tid / kWave, lane = tid % kWave;
    if (lane == 0) { sh.best_score[wave] = best; sh.best_id[wave] = best_id; }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            const float ov = sh.best_score[w];
            const int oi = sh.best_id[w];
            if (ov > best || (ov == best && oi < best_id)) { best = ov; best_id = oi; }
        }
        unsigned long long *dst = p.stats + 3 * ((size_t)row * p.stat_segments + seg);
        publish_tagged(dst + 0, __float_as_uint(best), p.generation);
        publish_tagged(dst + 1, (uint32_t)best_id, p.generation);
    }
}

__device__ __forceinline__ float race_exponential(uint32_t word)
{
    // U' = n * 2^-24 with n = (word >> 8) + 1 in [1, 2^24]; e = -log(U').
    const uint32_t n = (word >> 8) + 1u;
    const uint32_t j = 16777216u - n;  // U' = 1 - j * 2^-24
    if (j < 4096u) {
        // -log(1 - x) = x + x^2/2 + x^3/3 + ..., x < 2^-12: three terms are exact to fp32
        const float x = (float)j * 5.9604644775390625e-8f;
        return x * fmaf(x, fmaf(x, 0.33333334f, 0.5f), 1.0f);
    }
    const float u = (float)n * 5.9604644775390625e-8f;
    return -__builtin_amdgcn_logf(u) * kLn2;   // v_log_f32 is log2
}

// The race over vocabulary ids of one request: best r_v / e_v, e_v = -log(U'_v).
// It goes by parts of kRaceVec vectors of 4 ids per thread.  The variates of a part depend on the
// random numbers only, so a race block computes those of its first part before it waits for the
// statistics: the Philox rounds and the logarithms, three quarters of the race's arithmetic, then run under
// the streams of the statistics instead of after them (48 requests, V = 128256, rejection alone: 56.0 -> 50.1 us;
// 96 requests of a 70B-shaped step at k = 7: 123.6 -> 119.9 us, both with fewer or more segments as planned).
// (They wait in LDS: kept in registers across the accept chain they cost the kernel an occupancy step.)
__device__ __forceinline__ void race_variates(const RejectParams &p, const StepWords &step, int b, int g0, int g_end, RejectShared &sh)
{
    const int nu = min((g_end - g0 + kThreads - 1) / kThreads, kRaceVec);
    const uint32_t c3 = (step.hi24 << 8) | 1u;
#pragma unroll 2
    for (int u = 0; u < nu; ++u) {
        const int g = g0 + u * kThreads + (int)threadIdx.x;
        const uint4 w = philox4x32_10(make_uint4((uint32_t)g, (uint32_t)b, step.lo, c3), p.seed_lo, p.seed_hi);
        sh.variates[u][threadIdx.x] =   // (e_v == 0: +inf)
            (f32x4){__builtin_amdgcn_rcpf(race_exponential(w.x)), __builtin_amdgcn_rcpf(race_exponential(w.y)),
                    __builtin_amdgcn_rcpf(race_exponential(w.z)), __builtin_amdgcn_rcpf(race_exponential(w.w))};
    }
}

// Offsets of the race rows of request b after accept_phase.
struct RaceRows {
    const float *trow, *drow;
    float off_t, corr_t, off_d, corr_d;
    int m;
    int exclude;   // point-mass draft: the rejected token takes no part in the race
};

// One part (vectors g0 .. of [g0, g_end)): the thread's best (score, id) so far is carried along.
// drow == nullptr: weights are the target probabilities (bonus token), with `exclude` left out (point-mass
// draft: the rejected token; -1: none); otherwise the positive part of p - q.
//   p_v = corr_t * 2^(x_v * log2e + off_t), off_t = -(the row's offset, a whole number), corr_t =
//   1 / (its sum).  Ties keep the lowest id; weights <= 0 never win.
__device__ __forceinline__ void race_part(const RaceRows &rr, int g0, int g_end, const RejectShared &sh, float &best_score, int &best_id)
{
    // The loads run kRaceDepth vectors ahead.  Descriptors end with the part (past it the loads read zeros
    // without touching memory, and the ids take no part); without a draft row its descriptor is empty and
    // corr_d is 0, so that r - 0 is left.
    constexpr int kRaceDepth = 4;
    const int nvec = min(g_end - g0, kRacePart);
    const __amdgpu_buffer_rsrc_t td =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(rr.trow + 4 * (size_t)g0), 0, nvec * 16, kBufferFlags);
    const __amdgpu_buffer_rsrc_t dd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>((rr.drow != nullptr ? rr.drow : rr.trow) + 4 * (size_t)g0), 0, rr.drow != nullptr ? nvec * 16 : 0, kBufferFlags);
    f32x4 xt[kRaceDepth], xd[kRaceDepth];
    auto fetch = [&](int u) {
        const int at = (u * kThreads + (int)threadIdx.x) * 16;
        xt[u % kRaceDepth] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(td, at, 0, kStreamPolicy));
        xd[u % kRaceDepth] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(dd, at, 0, kStreamPolicy));
    };
#pragma unroll
    for (int u = 0; u < kRaceDepth; ++u) fetch(u);
#pragma unroll
    for (int u = 0; u < kRaceVec; ++u) {
        if (u * kThreads >= nvec) break;   // the same for the whole block
        const int i = u * kThreads + (int)threadIdx.x;
        const int v = 4 * (g0 + i);
        const f32x4 t = xt[u % kRaceDepth], d = xd[u % kRaceDepth], inv = sh.variates[u][threadIdx.x];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float r = rr.corr_t * fast_exp2(fmaf(t[e], kLog2eHi, fmaf(t[e], kLog2eLo, rr.off_t))) -
                            rr.corr_d * fast_exp2(fmaf(d[e], kLog2eHi, fmaf(d[e], kLog2eLo, rr.off_d)));
            const float score = r * inv[e];
            // ids rise within a thread: strict > keeps the lowest
            if (i < nvec && r > 0.0f && v + e != rr.exclude && score > best_score) {
                best_score = score;
                best_id = v + e;
            }
        }
        if (u + kRaceDepth < kRaceVec) fetch(u + kRaceDepth);
        __builtin_amdgcn_sched_barrier(0);   // (the scheduler would move all loads to the front, at twice the registers)
    }
}

// The block's best (score, id), to every thread.
__device__ __forceinline__ void race_winner(float &best_score, int &best_id, RejectShared &sh)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const float os = __shfl_xor(best_score, o);
        const int oi = __shfl_xor(best_id, o);
        if (os > best_score || (os == best_score && oi < best_id)) { best_score = os; best_id = oi; }
    }
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    __syncthreads();
    if (lane == 0) { sh.best_score[wave] = best_score; sh.best_id[wave] = best_id; }
    __syncthreads();
    best_score = sh.best_score[0];
    best_id = sh.best_id[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
        const float os = sh.best_score[w];
        const int oi = sh.best_id[w];
        if (os > best_score || (os == best_score && oi < best_id)) { best_score = os; best_id = oi; }
    }
    __syncthreads();
}

// Bounded wait until `ready` holds for every thread of the block (block-wide AND).
// `probe` re-evaluates the condition; returns false if the limit ran out.
// FEW: see nap_length.
template <bool FEW = false, typename F>
__device__ __forceinline__ bool wait_all(const RejectParams &p, F probe)
{
    for (int spin = 0; spin < p.spin_limit; ++spin) {
        if (__syncthreads_and(probe() ? 1 : 0)) return true;
        switch (nap_length(spin, FEW, p.short_naps != 0)) {   // (the instruction takes a constant)
            case 2: __builtin_amdgcn_s_sleep(2); break;
            case 8: __builtin_amdgcn_s_sleep(8); break;
            default: __builtin_amdgcn_s_sleep(32); break;
        }
    }
    return false;
}

// Accept chain of request b from the published row statistics.  Cheap (a few
// hundred loads and fp64 operations), so every block that needs its result just
// recomputes it.  Waits (bounded) until all of the request's statistics carry this
// call's tag.  Leaves the rows' offsets and sums in sh.row_off and sh.row_sum, m in sh.m, the near-tie count
// in sh.near.  Returns false if the statistics never arrived.
__device__ __forceinline__ bool accept_phase(const RejectParams &p, int b, RejectShared &sh, bool write_debug, int npos = -1)
{
    const int tid = threadIdx.x;
    const int row_t0 = uniform_load(p.cu_q_len, b);
    const int k = uniform_load(p.cu_q_len, b + 1) - row_t0 - 1;
    const int row_d0 = row_t0 - b;
    const bool has_draft_rows = p.mode == SPEC_ACCEPT_SAMPLE;
    const int nrows = has_draft_rows ? 2 * k + 1 : k + 1;
    const int nstat = nrows * p.stat_segments;
    // npos >= 0: only the first npos positions (their target and draft rows) are looked at, and
    // sh.m counts the leading accepts among them
    const int npos_eval = npos < 0 ? k : npos;

    // the draft tokens' logits and the uniforms do not depend on the statistics: fetch and draw them first
    // (a token outside the vocabulary is never used as an index: it has probability 0 under the
    // target, so its test rejects; the final stage counts it among the input errors)
    float tx = -INFINITY, dx = 0.0f;
    if (tid < npos_eval) {
        const int x = p.draft_tokens[row_d0 + tid];
        if ((unsigned)x < (unsigned)p.V) {
            tx = p.target_logits[(size_t)(row_t0 + tid) * p.V + x];
            if (has_draft_rows) dx = p.draft_logits[(size_t)(row_d0 + tid) * p.V + x];
        }
    }

    double u = 0.0;
    if (tid < npos_eval) {
        const StepWords step = philox_step_words(p);
        const uint4 w = philox4x32_10(make_uint4((uint32_t)tid, (uint32_t)b, step.lo, (step.hi24 << 8) | 0u),
                                      p.seed_lo, p.seed_hi);
        u = (double)(w.x >> 8) * (1.0 / 16777216.0);
    }

    // poll and fetch in one: every word carries its own tag
    const bool ok = wait_all(p, [&] {
        bool mine = true;
        for (int i = tid; i < nstat; i += kThreads) {
            const int ri = i / p.stat_segments;
            const int sg = i - ri * p.stat_segments;
            if (npos >= 0 && (ri <= k ? ri : ri - k - 1) >= npos) continue;   // a row of a later position
            const int row = ri <= k ? row_t0 + ri : p.T + row_d0 + (ri - k - 1);
            const unsigned long long *st = p.stats + 3 * ((size_t)row * p.stat_segments + sg);
            const unsigned long long w0 = fetch_u64(st), w1 = fetch_u64(st + 1), w2 = fetch_u64(st + 2);
            mine = mine && tagged_ok(w0, p.generation) && tagged_ok(w1, p.generation) && tagged_ok(w2, p.generation);
            sh.seg_sum[ri][sg] = __longlong_as_double((long long)((w0 & 0xFFFFFFFFull) | (w1 << 32)));
            sh.seg_off[ri][sg] = __uint_as_float((uint32_t)w2);
        }
        return mine;
    });
    if (!ok) return false;
    if (tid < nrows && (npos < 0 || (tid <= k ? tid : tid - k - 1) < npos)) {
        float mx = kEmptyMax;
        for (int sg = 0; sg < p.stat_segments; ++sg) mx = fmaxf(mx, sh.seg_off[tid][sg]);
        double total = 0.0;
        for (int sg = 0; sg < p.stat_segments; ++sg)
            // an exact power of two (the offsets are whole numbers; an empty segment's -1e30 gives 0): one instruction
            // instead of a call in a chain of as many calls as there are segments (this, the series below and the
            // uniforms drawn before the wait: tiny fp32 step 13.05 -> 12.64 us, 48 requests of V = 128256 alone 47.2 -> 46.4)
            total += ldexp(sh.seg_sum[tid][sg], (int)fmaxf(sh.seg_off[tid][sg] - mx, -4000.0f));
        sh.row_sum[tid] = total;
        sh.row_off[tid] = mx;
    }
    __syncthreads();

    // accept tests, all evaluated in parallel; the chain is resolved below
    if (tid < npos_eval) {
        // p/q = 2^(difference of the exponents) * (ratio of the sums): no logarithm in the chain (rejection alone, 48 requests,
        // V = 128256 46.5 -> 46.0 us; 128 at k = 3, V = 4096 17.0 -> 16.4)
        double e = (double)tx * kLog2eD - (double)sh.row_off[tid], ratio = 1.0 / sh.row_sum[tid];
        if (has_draft_rows) {   // (a point mass: q(x) = 1)
            e -= (double)dx * kLog2eD - (double)sh.row_off[k + 1 + tid];
            ratio = sh.row_sum[k + 1 + tid] / sh.row_sum[tid];
        }
        ratio *= exp2(e);   // p = 0 -> 0, q = 0 < p -> inf, both 0 -> NaN (rejects)
        sh.u[tid] = u;
        sh.ratio[tid] = ratio;
        sh.accept[tid] = (u < ratio) ? 1 : 0;
    }
    __syncthreads();
    if (tid == 0) {
        int m = 0;
        while (m < npos_eval && sh.accept[m]) ++m;
        int near = 0;
        const int evaluated = m + 1 < npos_eval ? m + 1 : npos_eval;
        for (int i = 0; i < evaluated; ++i)
            if (fabs(sh.u[i] - sh.ratio[i]) < 1e-6) ++near;
        sh.m = m;
        sh.near = near;
    }
    __syncthreads();
    if (write_debug && p.debug_u_ratio != nullptr && tid < k) {
        const bool evaluated = tid <= sh.m;
        p.debug_u_ratio[2 * (size_t)(row_d0 + tid) + 0] = evaluated ? sh.u[tid] : (double)NAN;
        p.debug_u_ratio[2 * (size_t)(row_d0 + tid) + 1] = evaluated ? sh.ratio[tid] : (double)NAN;
    }
    return true;
}

// Greedy mode: how many of the first npos draft tokens of request b equal their row's arg-max
// (a leading run), from the arg-max records of the target rows 0 .. npos-1.  Waits (bounded)
// for those records; the result is left in sh.m.  Returns false if they never arrived.
__device__ __forceinline__ bool greedy_prefix(const RejectParams &p, int b, int npos, RejectShared &sh)
{
    const int tid = threadIdx.x;
    const int row_t0 = uniform_load(p.cu_q_len, b);
    const int row_d0 = row_t0 - b;
    const int nstat = npos * p.stat_segments;
    const bool ok = wait_all(p, [&] {
        bool mine = true;
        for (int i = tid; i < nstat; i += kThreads) {
            const int ri = i / p.stat_segments;
            const int sg = i - ri * p.stat_segments;
            const unsigned long long *st = p.stats + 3 * ((size_t)(row_t0 + ri) * p.stat_segments + sg);
            const unsigned long long w0 = fetch_u64(st), w1 = fetch_u64(st + 1);
            mine = mine && tagged_ok(w0, p.generation) && tagged_ok(w1, p.generation);
            sh.seg_off[ri][sg] = __uint_as_float((uint32_t)w0);
            sh.seg_sum[ri][sg] = (double)(uint32_t)w1;   // the id, exactly
        }
        return mine;
    });
    if (!ok) return false;
    if (tid < npos) {
        float best = -INFINITY;
        int best_id = 0x7FFFFFFF;
        for (int sg = 0; sg < p.stat_segments; ++sg) {
            const float v = sh.seg_off[tid][sg];
            const int id = (int)sh.seg_sum[tid][sg];
            if (v > best || (v == best && id < best_id)) { best = v; best_id = id; }
        }
        sh.accept[tid] = p.draft_tokens[row_d0 + tid] == (best_id == 0x7FFFFFFF ? 0 : best_id) ? 1 : 0;
    }
    __syncthreads();
    if (tid == 0) {
        int m = 0;
        while (m < npos && sh.accept[m]) ++m;
        sh.m = m;
    }
    __syncthreads();
    return true;
}

// The row of a statistics item in position order: the target and draft rows (the target rows, if the draft
// is a point mass or the mode is greedy) of position 0 of all requests, then those of position 1, ...; a request's
// bonus row counts as a target row of position k.
struct PositionItem {
    int j, b, row;
};
static_assert(kMaxOwnLengths <= kThreads, "a thread per request");
template <bool PEEK>
__device__ __forceinline__ bool position_item(const RejectParams &p, int rec, RejectShared &sh, PositionItem &at)
{
    const bool has_draft_rows = p.mode == SPEC_ACCEPT_SAMPLE;
    bool is_draft = false;
    if (!PEEK || p.uniform_k >= 0) {   // one draft length: the bonus rows make up the last position
        const int k = p.uniform_k;
        const int per_position = has_draft_rows ? 2 * p.B : p.B;
        if (rec < per_position * k) {
            at.j = rec / per_position;
            const int w = rec - at.j * per_position;
            at.b = has_draft_rows ? w >> 1 : w;
            is_draft = has_draft_rows && (w & 1) != 0;
        } else {
            at.j = k;
            at.b = rec - per_position * k;
        }
        const int row_t0 = at.b * (k + 1);
        at.row = is_draft ? p.T + (row_t0 - at.b) + at.j : row_t0 + at.j;
        return true;
    }
    // Draft lengths of their own (up to kMaxOwnLengths requests): thread t looks at request t, and the counts of requests with
    // k >= 0, 1, ... say which position the item is in and which of its requests it belongs to.
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int row_t0 = tid < p.B ? p.cu_q_len[tid] : 0;
    const int k = tid < p.B ? p.cu_q_len[tid + 1] - row_t0 - 1 : -1;
#pragma unroll
    for (int i = 0; i < SPEC_K_MAX + 2; ++i) {
        const unsigned long long has = __builtin_amdgcn_ballot_w64(k >= i);
        if (lane == 0) sh.pos_count[i][wave] = __builtin_popcountll(has);
    }
    if (tid == 0) sh.pos_request = -1;
    __syncthreads();
    int j = 0, n_draft = 0;
    for (;; ++j) {
        if (j > SPEC_K_MAX) return false;   // (lengths on the device that are not the host's)
        int n_target = 0;
        n_draft = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            n_target += sh.pos_count[j][w];
            n_draft += sh.pos_count[j + 1][w];
        }
        const int n = n_target + (has_draft_rows ? n_draft : 0);
        if (rec < n) break;
        rec -= n;
    }
    // the rank-th request, in the given order, of those with k > j (target and draft row side by side), k == j
    // (bonus rows, after them), or, with target rows only, k >= j
    const bool bonus = has_draft_rows && rec >= 2 * n_draft;
    const int rank = !has_draft_rows ? rec : (bonus ? rec - 2 * n_draft : rec >> 1);
    is_draft = has_draft_rows && !bonus && (rec & 1) != 0;
    const bool mine = !has_draft_rows ? k >= j : (bonus ? k == j : k > j);
    int before = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int above = sh.pos_count[j + 1][w], from = sh.pos_count[j][w];
        if (w < wave) before += !has_draft_rows ? from : (bonus ? from - above : above);
    }
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(mine);
    if (mine && before + __builtin_popcountll(mask & ((1ull << lane) - 1ull)) == rank) sh.pos_request = tid;
    __syncthreads();
    at.j = j;
    at.b = __builtin_amdgcn_readfirstlane(sh.pos_request);
    if (at.b < 0) return false;
    const int t0 = uniform_load(p.cu_q_len, at.b);
    at.row = is_draft ? p.T + (t0 - at.b) + j : t0 + j;
    __syncthreads();   // (the statistics use the same memory)
    return true;
}

// Do the records that have been published so far show that one of the first j accept tests of request b fails?  Does
// not wait: a test whose records are not all there yet, or that is closer than a hundredth to its threshold, shows nothing
// (the exact decision is the accept chain's; this one only says which rows need not be read).  Half a wavefront
// looks at one position, a lane at one segment of its rows.
static_assert(SPEC_K_MAX * 32 <= kThreads && kMaxStatSegments <= 32, "half a wavefront per position, a lane per segment");
__device__ __forceinline__ bool rejected_before(const RejectParams &p, int b, int j)
{
    const int i = threadIdx.x >> 5, sg = threadIdx.x & 31;
    const bool greedy = p.mode == SPEC_ACCEPT_GREEDY, has_draft_rows = p.mode == SPEC_ACCEPT_SAMPLE;
    const int row_t0 = uniform_load(p.cu_q_len, b);
    const int row_d0 = row_t0 - b;
    bool reject = false;
    if (i < j) {
        const int x = p.draft_tokens[row_d0 + i];
        bool here = true;
        if (greedy) {
            float best = -INFINITY;
            int id = 0x7FFFFFFF;
            if (sg < p.stat_segments) {
                const unsigned long long *st = p.stats + kStatWords * ((size_t)(row_t0 + i) * p.stat_segments + sg);
                const unsigned long long w0 = fetch_u64(st), w1 = fetch_u64(st + 1);
                here = tagged_ok(w0, p.generation) && tagged_ok(w1, p.generation);
                const float v = __uint_as_float((uint32_t)w0);
                if (v >= best) { best = v; id = (int)(uint32_t)w1; }
            }
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) {
                const float ov = __shfl_xor(best, o);
                const int oi = __shfl_xor(id, o);
                if (ov > best || (ov == best && oi < id)) { best = ov; id = oi; }
            }
            reject = x != (id == 0x7FFFFFFF ? 0 : id);
        } else {
            unsigned long long t[kStatWords], d[kStatWords];
            float off_t = kEmptyMax, off_d = kEmptyMax, sum_t = 0.0f, sum_d = 0.0f, tx = -INFINITY, dx = 0.0f;
            if (sg < p.stat_segments) {
                const unsigned long long *st = p.stats + kStatWords * ((size_t)(row_t0 + i) * p.stat_segments + sg);
                const unsigned long long *sd = p.stats + kStatWords * ((size_t)(p.T + row_d0 + i) * p.stat_segments + sg);
#pragma unroll
                for (int w = 0; w < kStatWords; ++w) {
                    t[w] = fetch_u64(st + w);
                    d[w] = has_draft_rows ? fetch_u64(sd + w) : 0ull;
                }
            }
            if ((unsigned)x < (unsigned)p.V) {
                tx = p.target_logits[(size_t)(row_t0 + i) * p.V + x];
                if (has_draft_rows) dx = p.draft_logits[(size_t)(row_d0 + i) * p.V + x];
            }
            const StepWords step = philox_step_words(p);
            const uint4 w = philox4x32_10(make_uint4((uint32_t)i, (uint32_t)b, step.lo, (step.hi24 << 8) | 0u), p.seed_lo, p.seed_hi);
            if (sg < p.stat_segments) {
#pragma unroll
                for (int u = 0; u < kStatWords; ++u)
                    here = here && tagged_ok(t[u], p.generation) && (!has_draft_rows || tagged_ok(d[u], p.generation));
                off_t = __uint_as_float((uint32_t)t[2]);
                sum_t = (float)__longlong_as_double((long long)((t[0] & 0xFFFFFFFFull) | (t[1] << 32)));
                if (has_draft_rows) {
                    off_d = __uint_as_float((uint32_t)d[2]);
                    sum_d = (float)__longlong_as_double((long long)((d[0] & 0xFFFFFFFFull) | (d[1] << 32)));
                }
            }
            float mt = off_t, md = off_d;
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) {
                mt = fmaxf(mt, __shfl_xor(mt, o));
                md = fmaxf(md, __shfl_xor(md, o));
            }
            sum_t *= fast_exp2(off_t - mt);
            sum_d *= fast_exp2(off_d - md);
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) {
                sum_t += __shfl_xor(sum_t, o);
                sum_d += __shfl_xor(sum_d, o);
            }
            // log2 of p/q: the offsets, which may be large, are taken off in fp64
            float lr = (float)((double)tx * kLog2eD - (double)mt) - __builtin_amdgcn_logf(sum_t);
            if (has_draft_rows) lr = (float)((double)tx * kLog2eD - (double)mt - ((double)dx * kLog2eD - (double)md)) -
                                     (__builtin_amdgcn_logf(sum_t) - __builtin_amdgcn_logf(sum_d));
            const float u = (float)(w.x >> 8) * 5.9604644775390625e-8f;
            reject = __builtin_amdgcn_logf(u) > lr + 0.015f;
        }
        const unsigned long long missing = __builtin_amdgcn_ballot_w64(!here);
        reject = reject && ((missing >> (threadIdx.x & 32)) & 0xFFFFFFFFull) == 0;
    }
    return __syncthreads_or(reject ? 1 : 0) != 0;
}

// Statistics items are ordered by request (its target rows, then its draft rows), so that
// the first requests' statistics are complete early and their races can start while
// later requests' rows are still being read.
template <int DEPTH, bool PEEK>
__device__ __forceinline__ void stats_role(const RejectParams &p, int item, RejectShared &sh)
{
    const int rec = item / p.stat_segments;          // (request, row of the request)
    const int seg = item - rec * p.stat_segments;
    if (p.early_stop != kReadAll) {
        // Position order: the rows of a position are only needed if the request's earlier positions were all
        // accepted, and by the time a block of position j starts, those of positions < j were dispatched
        // long before.  A row that is not needed gets a placeholder record, so that later stages, which
        // poll all of a request's records and use those up to the first rejection, find it.
        PositionItem at;
        if (!position_item<PEEK>(p, rec, sh, at)) return;
        const int j = at.j, b = at.b, row = at.row;
        const bool greedy = p.mode == SPEC_ACCEPT_GREEDY;
        bool skip = false;
        if (PEEK && j > 0 && p.early_stop == kStopPeek) skip = rejected_before(p, b, j);
        else if (j > 0) skip = (greedy ? greedy_prefix(p, b, j, sh) : accept_phase(p, b, sh, false, j)) && sh.m < j;
        if (skip) {
            if (threadIdx.x == 0) {
                unsigned long long *dst = p.stats + 3 * ((size_t)row * p.stat_segments + seg);
                if (greedy) {   // (largest logit, id) of nothing
                    publish_tagged(dst + 0, __float_as_uint(-INFINITY), p.generation);
                    publish_tagged(dst + 1, 0x7FFFFFFFu, p.generation);
                } else {        // sum 1, offset 0
                    const unsigned long long bits = (unsigned long long)__double_as_longlong(1.0);
                    publish_tagged(dst + 0, (uint32_t)bits, p.generation);
                    publish_tagged(dst + 1, (uint32_t)(bits >> 32), p.generation);
                    publish_tagged(dst + 2, __float_as_uint(0.0f), p.generation);
                }
            }
            return;
        }
        if (greedy) argmax_block<DEPTH>(p, row, seg, sh);
        else stats_block<DEPTH>(p, row, seg, sh);
        return;
    }
    if (p.mode != SPEC_ACCEPT_SAMPLE) {   // target rows only: rec is the row
        if (p.mode == SPEC_ACCEPT_GREEDY) argmax_block<DEPTH>(p, rec, seg, sh);
        else stats_block<DEPTH>(p, rec, seg, sh);
        return;
    }
    // largest b with 2 * cu_q_len[b] - b <= rec (rows of the requests before b).  Start from
    // where b would be if all requests had equally many rows, and walk: with equal draft
    // lengths that is one round of loads instead of the log2(B) dependent ones of a bisection.
    const int nrec = 2 * p.T - p.B;
    int lo = (int)(((long long)rec * p.B) / nrec);
    if (lo > p.B - 1) lo = p.B - 1;
    while (lo > 0 && 2 * uniform_load(p.cu_q_len, lo) - lo > rec) --lo;
    while (lo < p.B - 1 && 2 * uniform_load(p.cu_q_len, lo + 1) - (lo + 1) <= rec) ++lo;
    const int b = lo;
    const int row_t0 = uniform_load(p.cu_q_len, b);
    const int k = uniform_load(p.cu_q_len, b + 1) - row_t0 - 1;
    const int ri = rec - (2 * row_t0 - b);
    const int row = ri <= k ? row_t0 + ri : p.T + (row_t0 - b) + (ri - k - 1);
    stats_block<DEPTH>(p, row, seg, sh);
}

__device__ __forceinline__ RaceRows race_rows(const RejectParams &p, int b, const RejectShared &sh)
{
    RaceRows rr;
    const int row_t0 = uniform_load(p.cu_q_len, b);
    const int k = uniform_load(p.cu_q_len, b + 1) - row_t0 - 1;
    const int row_d0 = row_t0 - b;
    rr.m = sh.m;
    rr.off_t = -sh.row_off[rr.m];
    rr.corr_t = (float)(1.0 / sh.row_sum[rr.m]);
    rr.off_d = 0.0f;
    rr.corr_d = 0.0f;
    rr.trow = p.target_logits + (size_t)(row_t0 + rr.m) * p.V;
    rr.drow = nullptr;
    rr.exclude = -1;
    if (rr.m < k && p.mode == SPEC_ACCEPT_POINT_DRAFT) rr.exclude = p.draft_tokens[row_d0 + rr.m];
    if (rr.m < k && p.mode == SPEC_ACCEPT_SAMPLE) {
        rr.off_d = -sh.row_off[k + 1 + rr.m];
        rr.corr_d = (float)(1.0 / sh.row_sum[k + 1 + rr.m]);
        rr.drow = p.draft_logits + (size_t)(row_d0 + rr.m) * p.V;
    }
    return rr;
}

// One (request, vocabulary segment) of the race.  Race items follow all statistics
// items in the grid, so the statistics blocks they wait for (inside accept_phase, with
// a bound) were scheduled before them and never wait themselves: the wait ends.
// Should the bound ever run out, the block publishes nothing and the request's final stage,
// whose own wait then runs out too, abandons the request.
__device__ __forceinline__ void race_role(const RejectParams &p, int item, RejectShared &sh)
{
    const int tid = threadIdx.x;
    const int b = item / p.race_segments;
    const int seg = item - b * p.race_segments;
    const int g_begin = seg * p.race_seg_len >> 2;
    const int g_end = min(p.V, (seg + 1) * p.race_seg_len) >> 2;
    const StepWords step = philox_step_words(p);
    race_variates(p, step, b, g_begin, g_end, sh);
    if (!accept_phase(p, b, sh, seg == 0)) return;
    const RaceRows rr = race_rows(p, b, sh);
    float win_score = -1.0f;
    int win_id = 0x7FFFFFFF;
    race_part(rr, g_begin, g_end, sh, win_score, win_id);
    for (int g0 = g_begin + kRacePart; g0 < g_end; g0 += kRacePart) {
        race_variates(p, step, b, g0, g_end, sh);
        race_part(rr, g0, g_end, sh, win_score, win_id);
    }
    race_winner(win_score, win_id, sh);
    if (tid == 0) {
        unsigned long long *dst = p.race_partial + 2 * ((size_t)b * p.race_segments + seg);
        publish_tagged(dst + 0, __float_as_uint(win_score), p.generation);
        publish_tagged(dst + 1, (uint32_t)win_id, p.generation);
        if (seg == 0)   // the accept chain's result, for the final stage
            publish_tagged(p.race_info + b, (uint32_t)rr.m | ((uint32_t)sh.near << 16), p.generation);
    }
}

// Last stage: one item per group of 2^final_shift requests (after all race items), 2^(8 - final_shift)
// threads each.  Waits (bounded) for what the group's requests need, writes their outputs, adds up
// their counters, and clears their tags so that a replay of the same launch (HIP graph) starts
// clean.  Requests are grouped because of the counters: all blocks add to the same few words, and
// such adds are taken one after the other, some 14 ns each (one block per request and seven adds: the last
// of 256 blocks ended 10 us after the race; the adds of a block of 16 requests are made once:
// greedy acceptance of 256 requests, k = 3: 35.1 -> 29.0 us; a 70B-shaped step of 256: 155.6 -> 150.3 us).
//   Sampling: the requests' race segments and accept results; the best segment wins.
//   Greedy acceptance (there is no race): the arg-max records of the k+1 target rows; the leading run
//   of draft tokens that equal their row's arg-max is accepted, the arg-max after it emitted.
__device__ __forceinline__ void final_role(const RejectParams &p, int item, RejectShared &sh)
{
    const int tid = threadIdx.x;
    const int group = kThreads >> p.final_shift;   // threads per request
    const int local = tid / group;                 // request of the block
    const int li = tid % group;
    const int b = (item << p.final_shift) + local;
    const bool valid = b < p.B;
    const bool greedy = p.mode == SPEC_ACCEPT_GREEDY;
    const int segs = p.stat_segments;

    // what does not depend on the other stages is fetched before the wait
    const int row_t0 = valid ? p.cu_q_len[b] : 0;
    const int k = valid ? p.cu_q_len[b + 1] - row_t0 - 1 : 0;
    const int row_d0 = row_t0 - b;
    const int token = li < k ? p.draft_tokens[row_d0 + li] : 0;
    const int kv_len = (valid && li == 0 && p.new_kv_len != nullptr) ? p.kv_len[b] : 0;
    if (tid < kMaxFinalGroup) {
        sh.fin_ready[tid] = 1;
        sh.fin_need[tid] = 0;
    }
    if (tid < 2) sh.fin_count[tid] = 0;
    __syncthreads();

    // poll and fetch in one: every word carries its own tag
    unsigned long long *part = p.race_partial + 2 * (size_t)b * p.race_segments;
    unsigned long long *rec_t = p.stats + kStatWords * ((size_t)row_t0 * segs);   // target rows, then (sampling) draft rows
    float best_score = -1.0f;
    int best_id = 0x7FFFFFFF;
    uint32_t info = 0;
    float *rec_value = &sh.seg_off[0][0] + local * (SPEC_K_MAX + 1) * segs;   // (2^final_shift * segs <= kMaxStatSegments)
    double *rec_id = &sh.seg_sum[0][0] + local * (SPEC_K_MAX + 1) * segs;
    bool mine = true;
    const bool ok = wait_all<true>(p, [&] {
        mine = true;
        if (!valid) return true;
        if (greedy) {
            for (int i = li; i < (k + 1) * segs; i += group) {
                const unsigned long long w0 = fetch_u64(rec_t + kStatWords * i), w1 = fetch_u64(rec_t + kStatWords * i + 1);
                mine = mine && tagged_ok(w0, p.generation) && tagged_ok(w1, p.generation);
                rec_value[i] = __uint_as_float((uint32_t)w0);
                rec_id[i] = (double)(uint32_t)w1;   // the id, exactly
            }
            return mine;
        }
        best_score = -1.0f;
        best_id = 0x7FFFFFFF;
        for (int i = li; i < p.race_segments; i += group) {   // segments in rising id order: > keeps the lowest id
            const unsigned long long w0 = fetch_u64(part + 2 * i), w1 = fetch_u64(part + 2 * i + 1);
            mine = mine && tagged_ok(w0, p.generation) && tagged_ok(w1, p.generation);
            const float score = __uint_as_float((uint32_t)w0);
            if (score > best_score) {
                best_score = score;
                best_id = (int)(uint32_t)w1;
            }
        }
        if (li <= SPEC_K_MAX) {
            const unsigned long long wi = fetch_u64(p.race_info + b);
            mine = mine && tagged_ok(wi, p.generation);
            info = (uint32_t)wi;
        }
        return mine;
    });
    if (!ok) {   // the same for the whole block: find the requests that are complete all the same
        if (!mine) sh.fin_ready[local] = 0;
        __syncthreads();
    }

    // the first lanes of a request's threads (all in one wavefront) hold its result
    const int lane = tid % kWave;
    int m, near = 0, win_id;
    if (greedy) {
        int id = 0;
        if (valid && li <= k) {
            float best = -INFINITY;
            id = 0x7FFFFFFF;
            for (int sg = 0; sg < segs; ++sg) {   // segments in rising id order: > keeps the lowest id
                const float v = rec_value[li * segs + sg];
                const int vid = (int)rec_id[li * segs + sg];
                if (v > best || (v == best && vid < id)) { best = v; id = vid; }
            }
            if (id == 0x7FFFFFFF) id = 0;
        }
        const int first = lane - li;   // (meaningful in the wavefront that holds li = 0 .. k)
        const unsigned long long equal = __builtin_amdgcn_ballot_w64(li < k && token == id);
        m = __builtin_ctzll(~(equal >> (first & (kWave - 1))));   // (bit k of the request is clear)
        win_id = __shfl(id, (first + m) & (kWave - 1));
    } else {
        const int width = group < kWave ? group : kWave;
        for (int o = width / 2; o > 0; o >>= 1) {
            const float os = __shfl_xor(best_score, o);
            const int oi = __shfl_xor(best_id, o);
            if (os > best_score || (os == best_score && oi < best_id)) { best_score = os; best_id = oi; }
        }
        m = (int)(info & 0xFFu);
        near = (int)(info >> 16);
        win_id = best_id;
        // p - q has no positive entry (p == q to rounding): draw from p instead
        const bool need = valid && li == 0 && sh.fin_ready[local] && !(best_score > 0.0f);
        if (need) sh.fin_need[local] = 1;
        if (__syncthreads_or(need ? 1 : 0)) {
            for (int r = 0; r < (1 << p.final_shift); ++r) {
                if (!sh.fin_need[r]) continue;   // (the same for the whole block)
                const int rb = (item << p.final_shift) + r;
                if (!accept_phase(p, rb, sh, false)) {
                    if (tid == 0) sh.fin_ready[r] = 0;
                    __syncthreads();
                    continue;
                }
                RaceRows rr = race_rows(p, rb, sh);
                rr.drow = nullptr;
                rr.corr_d = rr.off_d = 0.0f;
                rr.exclude = -1;
                const StepWords step = philox_step_words(p);
                float score = -1.0f;
                int id = 0x7FFFFFFF;
                for (int g0 = 0; g0 < p.V >> 2; g0 += kRacePart) {
                    race_variates(p, step, rb, g0, p.V >> 2, sh);
                    race_part(rr, g0, p.V >> 2, sh, score, id);
                }
                race_winner(score, id, sh);
                if (tid == 0) sh.fin_id[r] = id;
                __syncthreads();
            }
            if (sh.fin_need[local]) win_id = sh.fin_id[local];
        }
    }

    // (The outputs before the counters' sums and their barrier: behind it, where it would not wait for their stores, a step of four requests of 2470
    // tokens on 32/8 heads of 64, k = 0, V = 65292 takes 15.45 us and not 14.95, three greedy ones of 9 to 161, k = 8 7.6 and not
    // 7.45; seven of 20 to 381, k = 0 11.85 and not 12.0; eighteen others are the same.)
    const bool ready = sh.fin_ready[local] != 0;
    if (valid && li <= SPEC_K_MAX) {
        if (p.out_tokens != nullptr)
            p.out_tokens[(size_t)b * (SPEC_K_MAX + 1) + li] = !ready ? -1 : (li < m ? token : (li == m ? win_id : -1));
        if (ready && li < k && (unsigned)token >= (unsigned)p.V) atomicAdd(&sh.fin_count[1], 1u << 8);   // an input error
        if (li == 0) {
            p.accepted_len[b] = ready ? m : -1;
            p.next_token[b] = ready ? win_id : -1;
            if (p.new_kv_len != nullptr) p.new_kv_len[b] = ready ? kv_len - (k - m) : -1;
            if (p.draft_next_len != nullptr) p.draft_next_len[b] = !ready ? -1 : ((k > 0 && m == k) ? 2 : 1);
            if (ready) {   // four sums of at most 16 * 8 in one word
                atomicAdd(&sh.fin_count[0], (uint32_t)k | (uint32_t)m << 8 | (uint32_t)(m + 1 < k ? m + 1 : k) << 16 | (uint32_t)near << 24);
                atomicAdd(&sh.fin_count[1], 1u);
            } else {       // a wait ran out (never in a healthy launch): the request is counted here only
                atomicAdd(&p.counters[7], 1ull);
            }
        }
    }
    __syncthreads();
    if (tid < 7) {
        const uint32_t sums = sh.fin_count[0], n = sh.fin_count[1] & 0xFFu;
        uint32_t add = tid == 5 ? n : sh.fin_count[1] >> 8;
        if (tid < 3) add = (sums >> (8 * tid)) & 0xFFu;
        if (tid == 3) add = ((sums >> 8) & 0xFFu) + n;
        if (tid == 4) add = sums >> 24;
        if (add != 0) atomicAdd(&p.counters[tid], (unsigned long long)add);
    }
    if (!valid || !ready) return;
    // clear the request's tags
    for (int i = li; i < kStatWords * (k + 1) * segs; i += group) publish_u64(rec_t + i, 0ull);
    if (greedy) return;
    if (p.mode == SPEC_ACCEPT_SAMPLE) {
        unsigned long long *rec_d = p.stats + kStatWords * ((size_t)(p.T + row_d0) * segs);
        for (int i = li; i < kStatWords * k * segs; i += group) publish_u64(rec_d + i, 0ull);
    }
    for (int i = li; i < 2 * p.race_segments; i += group) publish_u64(part + i, 0ull);
    if (li == 0) publish_u64(p.race_info + b, 0ull);
}

// ===========================================================================
// Attention half
// ===========================================================================
template <int D>
struct PageRegs {
    u32x4 k[D / 32];  // k[kk]: token n, dims 32*kk + 8g .. +7
    u32x4 v[D / 32];  // v[pp]: dims 32*pp + n (low half) and 32*pp + 16 + n (high half), tokens 4g .. 4g+3
};

// The query rows and the output tile pass through LDS so that global memory sees them as
// whole rows (full cache lines, each once per block) instead of the 64-byte pieces of the
// matrix-operand layout, once per wavefront: with 32 to 48 query rows per KV head (grouped
// heads) these requests were a fifth of all the block's memory requests, and the launch is
// bound by requests as much as by bytes.  Rows are padded against bank conflicts.
constexpr int q_stride(int D) { return D * 2 + 16; }   // bytes per bf16 query row in LDS
constexpr int o_stride(int D) { return D * 4 + 16; }   // bytes per fp32 output row in LDS

// Wave groups.  A block's four wavefronts form WG groups of PW = 4 / WG wavefronts.  Each group
// owns NT 16-row tiles of the query rows of one (request, KV head) and walks ALL pages of the
// block's chunk, its PW wavefronts taking them in turn.  WG = 1 is the common case (up to 48
// fused rows).  With more rows per KV head (long drafts on wide query groups: up to 9 x 16 = 144
// rows) the groups of one block read the same pages at the same time, so the pages cross the
// memory interface once and the groups find each other's loads in the compute unit's cache or
// in flight.
// Token-major pages ([16 tokens][D dims] per page and KV head).  The matrix operands want, per lane, 8
// consecutive dims of one token (K) and four consecutive tokens of one dim (V).  Each wavefront loads its page as
// whole rows (1 KB per load, 16 bytes per lane), stages it in a region of its own in LDS and reads it back in operand
// order, V through the transposing read.  (K can be loaded in operand order directly, but each load then
// touches 16 half cache lines, and the other halves have often left the cache by the time the next load wants
// them.  Attention alone: 64 requests on 32/8 heads of 64, k = 3: 31.3 -> 28.7 us; 24 on 64/8 heads, k = 4:
// 62.6 -> 58.1; four of 20 to 28 k tokens on 32/8 heads, k = 8: 95.0 -> 87.7; 256 on 64/8 heads, k = 2, which the
// memory system bounds already: 120.5 -> 119.7.)  Token rows are padded by 16 bytes
// (272 at D = 128) so that neither the row writes nor the operand reads have bank conflicts.
constexpr int vt_row_bytes(int D) { return D * 2 + 16; }
constexpr int vt_wave_bytes(int D) { return SPEC_BLOCK_SIZE * vt_row_bytes(D); }
// Which blocks walk their pages staged (see the staged walk in attn_role).
constexpr bool staged_walk(int WG, bool TM, bool K_DIRECT) { return WG > 1 && TM && !K_DIRECT; }

template <int NT, int WG, bool TM = false, int D = kD, bool K_DIRECT = false>
struct AttnShared {
    static constexpr int kRowsMax = WG * NT * 16;
    static constexpr bool kStaged = staged_walk(WG, TM, K_DIRECT);
    union {
        // staged walk: two rounds of a page per wavefront, K and V
        unsigned char ring[kStaged ? 2 : 1][kStaged ? kWaves : 1][2][kStaged ? vt_wave_bytes(D) : 16];
        alignas(16) unsigned char vt[TM && !kStaged ? 2 * kWaves * vt_wave_bytes(D) : 16];   // token-major pages: K and V staged per wavefront
        f32x4 acc[2][NT][D / 16][kWave];          // epilogue: partial results of the wavefronts being merged
        unsigned char q[kRowsMax * q_stride(D)];  // prologue: the block's query rows
        unsigned char o[WG == 1 ? NT * 16 * o_stride(D) : 16];   // epilogue of an unsplit request (one group): the output tile
    };
    float m[2][NT][kWave];
    float l[2][NT][kWave];
    int last;
};

// The order in which the attention items take the requests (longest first), as the kernel
// sees it: a pointer into the kernel-argument segment, read with scalar loads (taking the
// address of the by-value argument instead would make the compiler copy the table to
// private memory).  Two 16-bit entries per word; n == 0: the given order.
typedef const uint32_t __attribute__((address_space(4))) *uniform_u32_ptr;
struct OrderTable {
    int n;
    uniform_u32_ptr pairs;
};

// VAR: 0 = pages in the matrix-operand layout, softmax weights fed as bf16 high + low parts;
//      1 = the same with the weights as one bf16 (an experiment switch);
//      2 = token-major pages (K and V staged through LDS, which gives V transposed; K_DIRECT: V alone), weights as
//          high + low parts;
//      3 = as 0 with a head dim of 64, 4 = as 2 with a head dim of 64 (all others: 128).
constexpr int head_dim_of(int VAR) { return (VAR == 3 || VAR == 4) ? 64 : kD; }
constexpr bool token_major_of(int VAR) { return VAR == 2 || VAR == 4; }

// What one attention block works on, and each thread's place in it (see attn_begin).
struct AttnWork {
    int tid, wave, lane, n16, g;   // lane = 16 g + n16
    int grp, pw;                   // this wavefront's row group, and its place in the page walk of the group
    int kvh, unit, chunk, nchunks;
    int L, row0, q_len, group;     // group: query heads per KV head
    int rows, row_lo, grp_rows;    // fused query rows of the block; first row and number of rows of this wavefront's group
    int tok0, npages;
    int bt;                        // block-table entries of this wavefront's pages, one per lane (-1: outside the pool)
    int my_pages;
};

// The block's place in the work: request, KV head, chunk, rows, pages.  False: nothing to do.
// (STAGED: the wavefronts of all groups share the page loads between them, see the staged walk.)
template <int NT, int WG, bool STAGED>
__device__ __forceinline__ bool attn_begin(const AttnParams &p, OrderTable order, int item, AttnWork &w)
{
    constexpr int PW = kWaves / WG;   // wavefronts that share the pages of a group between them
    constexpr int STEP = STAGED ? kWaves : PW;   // a wavefront loads every STEP-th page
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / PW;        // this wavefront's row group
    const int pw = wave % PW;         // ... and its place in the page walk of the group
    const int lane = tid & 63;
    const int n16 = lane & 15;
    const int g = lane >> 4;
    const int first = STAGED ? wave : pw;   // ... from this one on
    // Items are chunk-major: all first chunks (requests longest first, KV heads innermost),
    // then all second chunks, ...  Consecutive blocks go to different XCDs, so every XCD
    // gets the same mix of chunk indices; the chunk indices that only the longest requests
    // have come last (blocks of the others for these indices exit at once), instead of
    // always falling on the same XCDs.
    // With split requests a row of items (one chunk index) is padded to whole rows of kXcds blocks, so
    // that all chunks of a (request, KV head) run on one XCD and find its query rows, table entries,
    // partial results and ticket in that XCD's L2 (spread over the XCDs the ragged long-context
    // workload takes 4% longer).
    // Where the order table lists chunks there is one such row: only the chunks that exist, request by request (no
    // holes between blocks that have work: the dispatcher deals the blocks out in turn, and empty ones leave their compute
    // units idle while others get two).
    const int n_units = p.ranks * p.Hkv;
    const int row_items = attn_row_items(p);
    int chunk = item / row_items;
    const int place = item - chunk * row_items;
    if (place >= n_units) return false;   // padding
    const int kvh = place % p.Hkv;
    int b = place / p.Hkv;   // rank in the order of the attention items
    int capacity = p.capacity_tokens, listed = p.max_chunks;
    if (order.n > 0) {
        const uint32_t pair = order.pairs[b >> 1];
        b = (int)((b & 1) ? pair >> 16 : pair & 0xFFFFu);
        if (p.spread) {
            // A request that has grown on the device past its listed chunks takes longer ones, as far as a wavefront's table
            // entries go.  (Beyond that it is left out by all of its blocks: a ticket taken for a merge that no block
            // makes would still be there in the next replay of the launch.)
            listed = (b >> (kListRequestBits + kListChunkBits)) + 1;
            capacity = min(capacity, listed * (kWave * PW * SPEC_BLOCK_SIZE));
            chunk = b >> kListRequestBits & (kMaxListedChunks - 1);
            b &= kMaxListedRequests - 1;
        }
    }
    const int unit = b * p.Hkv + kvh;

    // When no request is split, a wavefront's block-table entries do not depend on kv_len:
    // fetch them alongside it (entries past the request's pages are never used).
    int bt = 0;
    if (p.max_chunks == 1 && first + STEP * lane < p.max_blocks_per_req)
        bt = p.block_table[(size_t)b * p.max_blocks_per_req + first + STEP * lane];
    const int L = uniform_load(p.kv_len, b);
    const int row0 = uniform_load(p.cu_q_len, b);
    const int q_len = uniform_load(p.cu_q_len, b + 1) - row0;
    // The lengths come from device memory and bound every loop and index below: a request
    // whose lengths do not fit the launch (longer than planned for, beyond its block-table row,
    // shorter than its own query rows) is left out and reported.
    if (!request_lengths_ok(L, q_len, capacity, p.max_blocks_per_req)) {
        if (chunk == 0 && kvh == 0 && tid == 0 && p.errors != nullptr) atomicAdd(p.errors, 1ull);
        return false;
    }
    const int nchunks = min((L + p.chunk_tokens - 1) / p.chunk_tokens, listed);   // (<= max_chunks in any case, since L <= capacity_tokens)
    if (chunk >= nchunks) return false;
    // even chunks per request, page aligned (never longer than chunk_tokens, unless there are too few listed)
    const int C = ((L + nchunks - 1) / nchunks + SPEC_BLOCK_SIZE - 1) & ~(SPEC_BLOCK_SIZE - 1);
    const int group = p.Hq / p.Hkv;
    // (the plan sized WG and NT for the longest draft of the host copy of cu_q_len; should the device
    // copy disagree, the rows beyond that are left out rather than staged out of bounds)
    const int rows = min(q_len * group, WG * NT * 16);
    const int row_lo = grp * (NT * 16);          // first row of this wavefront's group
    const int grp_rows = min(max(rows - row_lo, 0), NT * 16);
    const int tok0 = chunk * C;
    const int tok1 = min(L, tok0 + C);
    const int npages = (tok1 - tok0 + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE;  // <= 64 * PW
    const int page0 = tok0 / SPEC_BLOCK_SIZE;

    // block-table entries of this wavefront's pages (every STEP-th), one per lane
    if (p.max_chunks != 1 && first + STEP * lane < npages)
        bt = p.block_table[(size_t)b * p.max_blocks_per_req + page0 + first + STEP * lane];
    {
        // an entry outside the pool is never turned into an address: the page reads as zeros
        const bool bad = first + STEP * lane < npages && (unsigned)bt >= (unsigned)p.num_blocks;
        if (bad) bt = -1;
        const unsigned long long bad_lanes = __builtin_amdgcn_ballot_w64(bad);
        if (bad_lanes != 0 && kvh == 0 && (STAGED || grp == 0) && p.errors != nullptr && lane == 0)
            atomicAdd(p.errors, (unsigned long long)__builtin_popcountll(bad_lanes));
    }

    w.tid = tid; w.wave = wave; w.lane = lane; w.n16 = n16; w.g = g; w.grp = grp; w.pw = pw;
    w.kvh = kvh; w.unit = unit; w.chunk = chunk; w.nchunks = nchunks;
    w.L = L; w.row0 = row0; w.q_len = q_len; w.group = group;
    w.rows = rows; w.row_lo = row_lo; w.grp_rows = grp_rows; w.tok0 = tok0; w.npages = npages; w.bt = bt;
    // (none for a group that has no rows of this request, unless it loads for the others)
    w.my_pages = (npages > first && (STAGED || grp_rows > 0)) ? (npages - first + STEP - 1) / STEP : 0;
    return true;
}

// The merge of a request's chunks, in chunk order: half a wavefront takes RB query rows at a time (four head dims per lane) and
// GROUP chunks of each per pass.
template <int GROUP, int RB, int D>
__device__ __forceinline__ void merge_chunks(const AttnParams &p, const AttnWork &w)
{
    const int lane = w.lane, wave = w.wave, rows = w.rows, group = w.group, row0 = w.row0, kvh = w.kvh, nchunks = w.nchunks;
    const int half = lane >> 5, l32 = lane & 31;
    const bool dims_on = 4 * l32 < D;   // (a head dim of 64 keeps half of the lanes busy)
    for (int r0 = 2 * wave + half; r0 < rows; r0 += 2 * kWaves * RB) {
        bool rv[RB];
        size_t rh[RB];
        const unsigned long long *ml[RB], *pa[RB];
        float mx[RB], denom[RB];
        f32x4 o[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            const int r = r0 + 2 * kWaves * j;
            rv[j] = r < rows;
            const int rr = rv[j] ? r : 0;
            rh[j] = (size_t)(row0 + rr / group) * p.Hq + kvh * group + rr % group;
            const size_t base = rh[j] * p.max_chunks;
            ml[j] = reinterpret_cast<const unsigned long long *>(p.ws_ml) + base;
            pa[j] = reinterpret_cast<const unsigned long long *>(p.ws_acc) + base * (D / 2) + 2 * (l32 % (D / 4));
            mx[j] = kEmptyMax;
            denom[j] = 0.0f;
            o[j] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int c0 = 0; c0 < nchunks; c0 += GROUP) {
            unsigned long long mlv[RB][GROUP], a0[RB][GROUP], a1[RB][GROUP];
#pragma unroll
            for (int j = 0; j < RB; ++j) {
#pragma unroll
                for (int c = 0; c < GROUP; ++c) {
                    const unsigned long long *al = pa[j] + (size_t)(c0 + c) * (D / 2);
                    if constexpr (RB == 1 || D < 4 * 32) {
                        mlv[j][c] = pack_f32x2(kEmptyMax, 0.0f);
                        a0[j][c] = a1[j][c] = 0ull;
                        // the same for the whole wavefront: one branch for the three
                        if (c0 + c < nchunks && (RB == 1 || __builtin_amdgcn_readfirstlane(r0) + 2 * kWaves * j < rows)) {
                            mlv[j][c] = fetch_u64(ml[j] + c0 + c);
                            a0[j][c] = fetch_u64(al);
                            a1[j][c] = fetch_u64(al + 1);
                        }
                    } else {
                        const bool on = rv[j] && c0 + c < nchunks;
                        mlv[j][c] = on ? fetch_u64(ml[j] + c0 + c) : pack_f32x2(kEmptyMax, 0.0f);
                        a0[j][c] = on ? fetch_u64(al) : 0ull;
                        a1[j][c] = on ? fetch_u64(al + 1) : 0ull;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                float gmx = mx[j];
#pragma unroll
                for (int c = 0; c < GROUP; ++c) gmx = fmaxf(gmx, __uint_as_float((uint32_t)mlv[j][c]));
                const float keep = fast_exp2(mx[j] - gmx);   // rescale of what earlier passes summed
                denom[j] *= keep;
                o[j] *= keep;
                mx[j] = gmx;
#pragma unroll
                for (int c = 0; c < GROUP; ++c) {
                    const float w = fast_exp2(__uint_as_float((uint32_t)mlv[j][c]) - gmx);
                    denom[j] = fmaf(w, __uint_as_float((uint32_t)(mlv[j][c] >> 32)), denom[j]);
                    o[j][0] = fmaf(w, __uint_as_float((uint32_t)a0[j][c]), o[j][0]);
                    o[j][1] = fmaf(w, __uint_as_float((uint32_t)(a0[j][c] >> 32)), o[j][1]);
                    o[j][2] = fmaf(w, __uint_as_float((uint32_t)a1[j][c]), o[j][2]);
                    o[j][3] = fmaf(w, __uint_as_float((uint32_t)(a1[j][c] >> 32)), o[j][3]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < RB; ++j)
            if (rv[j] && dims_on) *reinterpret_cast<f32x4 *>(p.out + rh[j] * D + 4 * l32) = o[j] * (1.0f / denom[j]);
    }
}

// The end of an attention block: merges its wavefronts, and writes the output rows (a request that is not
// split) or publishes the chunk's partial results and, as the last chunk to finish, merges all of them.
// acc[nt][mt] holds, per lane, four consecutive head dims of query row n16 of tile nt, the first of which
// is dim_base(mt, g).
template <int NT, int WG, int D, bool FEW_CHUNKS, typename Shared, typename DimBase>
__device__ __forceinline__ void attn_end(const AttnParams &p, const AttnWork &w, f32x4 (&acc)[NT][D / 16], float (&m_run)[NT],
                                         float (&l_run)[NT], const int (&out_row)[NT], DimBase dim_base, Shared &sh)
{
    constexpr int MT = D / 16;
    constexpr int kOStride = o_stride(D);
    const int tid = w.tid, wave = w.wave, lane = w.lane, n16 = w.n16, g = w.g, grp = w.grp, pw = w.pw;
    const int kvh = w.kvh, unit = w.unit, chunk = w.chunk, nchunks = w.nchunks, row0 = w.row0, group = w.group;
    const int rows = w.rows, grp_rows = w.grp_rows;
    // each lane summed its own four tokens per page: finish the row sums
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        l_run[nt] = sum_across_rows(l_run[nt]);
    }

    // merge the wavefronts of each group into the group's first one
    auto put = [&](int buf) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) sh.acc[buf][nt][mt][lane] = acc[nt][mt];
            sh.m[buf][nt][lane] = m_run[nt];
            sh.l[buf][nt][lane] = l_run[nt];
        }
    };
    auto merge = [&](int buf) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const float mo = sh.m[buf][nt][lane];
            const float lo = sh.l[buf][nt][lane];
            const float mn = fmaxf(m_run[nt], mo);
            const float wa = fast_exp2(m_run[nt] - mn);
            const float wb = fast_exp2(mo - mn);
            l_run[nt] = l_run[nt] * wa + lo * wb;
            m_run[nt] = mn;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = acc[nt][mt] * wa + sh.acc[buf][nt][mt][lane] * wb;
        }
    };
    if constexpr (WG == 1) {          // 2,3 -> 0,1 then 1 -> 0 (the last step below, by wavefront 0)
        if (wave >= 2) put(wave - 2);
        __syncthreads();
        if (wave < 2) merge(wave);
        __syncthreads();
        if (wave == 1) put(0);
        __syncthreads();
    } else if constexpr (WG == 2) {   // 1 -> 0 and 3 -> 2
        if (pw == 1) put(grp);
        __syncthreads();
        if (pw == 0) merge(grp);
        __syncthreads();
    }
    const bool lead = pw == 0 && grp_rows > 0;   // this wavefront holds its group's result

    if (nchunks == 1) {
        if constexpr (WG == 1) {
            // the only chunk of this (request, KV head): normalise, lay the tile out by rows in
            // LDS, and let the whole block write the rows (16 bytes per thread, consecutive
            // threads along a row)
            if (wave == 0) {
                merge(0);   // (its reads of the shared partials precede the writes below in program order)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const float inv = 1.0f / l_run[nt];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        *reinterpret_cast<f32x4 *>(sh.o + (nt * 16 + n16) * kOStride + dim_base(mt, g) * 4) = acc[nt][mt] * inv;
                }
            }
            __syncthreads();
            constexpr int OP = D / 4;   // 16-byte pieces of an fp32 output row
            for (int piece = tid; piece < rows * OP; piece += kThreads) {
                const int r = piece / OP, c = piece % OP;
                const size_t rh = (size_t)(row0 + r / group) * p.Hq + kvh * group + r % group;
                __builtin_nontemporal_store(*reinterpret_cast<const f32x4 *>(sh.o + r * kOStride + c * 16),
                                            reinterpret_cast<f32x4 *>(p.out + rh * D + c * 4));
            }
        } else if (lead) {
            // several groups: each group's first wavefront writes its rows itself (a lane holds four
            // consecutive head dims of one row per 16-dim slice)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (out_row[nt] < 0) continue;
                const float inv = 1.0f / l_run[nt];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    __builtin_nontemporal_store(acc[nt][mt] * inv,
                                                reinterpret_cast<f32x4 *>(p.out + (size_t)out_row[nt] * D + dim_base(mt, g)));
            }
        }
        return;
    }

    if (WG == 1 ? wave == 0 : lead) {
        if constexpr (WG == 1) merge(0);
        // one partial per query row: acc[dim], running max, running sum
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (out_row[nt] < 0) continue;
            const size_t slot = (size_t)out_row[nt] * p.max_chunks + chunk;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                unsigned long long *dst = reinterpret_cast<unsigned long long *>(p.ws_acc + slot * D + dim_base(mt, g));
                publish_u64(dst + 0, pack_f32x2(acc[nt][mt][0], acc[nt][mt][1]));
                publish_u64(dst + 1, pack_f32x2(acc[nt][mt][2], acc[nt][mt][3]));
            }
            if (g == 0)
                publish_u64(reinterpret_cast<unsigned long long *>(p.ws_ml + slot * 2), pack_f32x2(m_run[nt], l_run[nt]));
        }
        writes_complete();  // the partials are in memory before the ticket is taken
    }
    if (!p.fused_combine) return;   // a separate combine launch merges the partials
    if constexpr (WG > 1) __syncthreads();   // ... those of every group
    if (tid == 0) {
        unsigned long long *ticket = &p.tickets[unit];
        const uint32_t before = ticket_arrive(ticket, p.generation);
        const int last = (before + 1u == (uint32_t)nchunks) ? 1 : 0;
        if (last) ticket_reset(ticket);
        sh.last = last;
    }
    __syncthreads();
    if (!sh.last) return;
    order_after_ticket();

    // Last chunk of this (request, KV head) to finish: merge all chunks in chunk order.
    // Half a wavefront takes two query rows at a time (four head dims per lane) and eight
    // chunks of each per pass; every load of a pass is issued before the first is used, so
    // a pass costs one memory round trip.  (Lanes past the last row or past a head dim of 64 load what the
    // first ones do and store nothing: with conditions of their own the loads took a branch each.  Eight requests on
    // 64/8 heads of 128, k = 1, two chunks: 10.94 -> 10.75 us; 16 on 32/8 heads of 64, k = 8: 15.8 -> 14.7.  With two
    // rows in flight of 128 dims, where those loads are too many, it costs 2%: 75.1 / 77.3 us for four of 6000
    // tokens on 64/4 heads, k = 8.)
    // FEW_CHUNKS: with four chunks or fewer, half as many chunks and twice as many rows per pass, so that 17 to 32 rows take one
    // pass (attention alone, 64/8 heads, k = 7, one request of 1000 tokens 19.5 -> 18.5 us; fp32, 32/8 heads, k = 4, four of 500 19.5 -> 19.0, eight
    // of 256 to 1024 24.45 -> 24.0).  For two row tiles of 128 dims in wave groups or fp32 only: three tiles spill.
    if constexpr (FEW_CHUNKS && NT == 2 && D == 128) {
        if (nchunks <= 4) {
            merge_chunks<4, 4, D>(p, w);
            return;
        }
    }
    constexpr int GROUP = 8;   // chunks merged per pass (16 per pass spill 200 to 340 bytes per lane)
    constexpr int RB = NT >= 2 ? 2 : 1;   // rows in flight per half wavefront (one row tile: at most two passes anyway, and registers are tight)
    merge_chunks<GROUP, RB, D>(p, w);
}

// (K_DIRECT: see attn_k_direct_kernel)
template <int NT, int WG, int VAR, bool K_DIRECT = false>
__device__ __forceinline__ void attn_role(const AttnParams &p, OrderTable order, int item,
                                          AttnShared<NT, WG, token_major_of(VAR), head_dim_of(VAR), K_DIRECT> &sh)
{
    constexpr bool SPLIT_P = VAR != 1;
    constexpr bool TM = token_major_of(VAR);
    constexpr bool STAGED = staged_walk(WG, TM, K_DIRECT);
    constexpr int D = head_dim_of(VAR);
    // Which walks take two pages at a time (consume_pair).  The staged one, up to two row tiles or a head dim of 64 (three of
    // 128 leave no registers for a second page's operands): attention alone, 64/8 heads, k = 7, 96 / 256 requests of 256 to
    // 1024 tokens 63.1 -> 61.0 / 138.6 -> 135.9 us; head dim 64, 64/4 heads, 32 requests of 300 to 2900, k = 3 35.1 -> 31.3, k = 5 42.9 ->
    // 40.4.  A wavefront's own walk on token-major pages of 64 dims with two or three row tiles: 32/8 heads, 64 requests of
    // 200 to 1900 tokens, k = 7 / 8 31.0 -> 30.0 / 33.0 -> 31.4; four of 9000 to 18000, k = 8 37.5 -> 34.4; 128 of 100, k = 5 14.9 -> 14.2.
    // (Not elsewhere: one row tile of 64 dims 28.5 -> 28.3 and, 256 short requests, 38.5 -> 38.8; tiled pages of 64 dims 28.0 ->
    // 28.4; 128 dims, one tile, 43.9 -> 50.5 at an occupancy step less, two tiles 41.1 -> 42.9.  With K straight into operand
    // order, two groups of two tiles take the staged walk's pairs, whose sums they have to equal.  Staged, requests of one
    // page or two lose: 130 of 9 to 16 tokens on 64/8 heads, k = 7 22.5 -> 23.8 us, of 33 to 48 25.05 -> 24.5.)
    constexpr bool PAIRS_STAGED = STAGED && (NT <= 2 || D == 64);
    constexpr bool PAIR_WALK = !STAGED && TM && ((D == 64 && NT >= 2) || (K_DIRECT && NT == 2 && WG == 2));
    constexpr int KK = D / 32;                        // 32-dim steps of the score product = 1 KB loads per K or V page
    constexpr int MT = D / 16;                        // 16-dim slices of the output
    constexpr int kQStride = q_stride(D);
    constexpr int kPageHeadBytes = SPEC_BLOCK_SIZE * D * 2;   // one (page, KV head) of K or of V: 4096 at D = 128
    constexpr int QP = D / 8;                         // 16-byte pieces of a bf16 query row
    constexpr int QI = (NT * WG * 16 * QP + kThreads - 1) / kThreads;   // ... of all the block's rows, per thread
    constexpr int kVtRowBytes = vt_row_bytes(D), kVtWaveBytes = vt_wave_bytes(D);
    constexpr int PW = kWaves / WG;   // wavefronts that share the pages of a group between them
    AttnWork w;
    if (!attn_begin<NT, WG, STAGED>(p, order, item, w)) return;
    const int tid = w.tid, wave = w.wave, lane = w.lane, n16 = w.n16, g = w.g, pw = w.pw;
    const int kvh = w.kvh, L = w.L, row0 = w.row0, q_len = w.q_len, group = w.group, rows = w.rows, row_lo = w.row_lo;
    const int grp_rows = w.grp_rows, tok0 = w.tok0, bt = w.bt, my_pages = w.my_pages;

    // Q: the block fetches its query rows once, 16 bytes per thread and consecutive threads
    // along a row (the heads of a group are adjacent in memory), and leaves them in LDS
    u32x4 qpiece[QI];
#pragma unroll
    for (int i = 0; i < QI; ++i) {
        const int piece = tid + i * kThreads;   // QP pieces per row
        const int r = piece / QP, c = piece % QP;
        qpiece[i] = (u32x4){0u, 0u, 0u, 0u};
        if (r < rows) {
            const size_t rh = (size_t)(row0 + r / group) * p.Hq + kvh * group + r % group;
            qpiece[i] = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.q) + rh * (D * 2) + c * 16);
        }
    }
    bf16x8 qreg[NT][KK];   // filled from LDS below
    int limit[NT];     // each lane's last visible key
    int out_row[NT];   // packed (token row * Hq + head) of this lane's query row, -1 if padding
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int r = row_lo + nt * 16 + n16;
        const bool valid = r < rows;
        const int j = valid ? r / group : 0;
        const int gq = valid ? r % group : 0;
        limit[nt] = valid ? L - q_len + j : -1;
        out_row[nt] = valid ? (int)((size_t)(row0 + j) * p.Hq + kvh * group + gq) : -1;
    }

    // Pages are read with buffer loads through a descriptor that covers exactly one
    // (page, KV head): 4 KB of K or V.  A page index past the end gets a descriptor of
    // length 0, for which the hardware returns zeros without touching memory.  That
    // keeps every load unconditional, so the loads of later pages stay in flight across
    // the arithmetic of the current one (a branch around them would make the compiler
    // wait for all outstanding loads at every use).
    const char *khead = static_cast<const char *>(p.k_cache) + (size_t)kvh * kPageHeadBytes;
    const char *vhead = static_cast<const char *>(p.v_cache) + (size_t)kvh * kPageHeadBytes;
    const size_t page_stride = (size_t)p.Hkv * kPageHeadBytes;
    const int lane_off = lane * 16;

    auto load_page = [&](int it, PageRegs<D> &r) {   // it-th page of this wavefront
        const int entry = __builtin_amdgcn_readlane(bt, it < my_pages ? it : 0);
        const bool valid = it < my_pages && entry >= 0;
        const int page = valid ? entry : 0;
        const int bytes = valid ? kPageHeadBytes : 0;
        const __amdgpu_buffer_rsrc_t kd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(khead + (size_t)page * page_stride), 0, bytes, kBufferFlags);
        const __amdgpu_buffer_rsrc_t vd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(vhead + (size_t)page * page_stride), 0, bytes, kBufferFlags);
#pragma unroll
        for (int i = 0; i < KK; ++i)
            r.k[i] = K_DIRECT   // in operand order: token n16, dims 32 i + 8 g .. + 7 sit at n16 * 2 D + 64 i + 16 g (no streaming hint:
                                // half a cache line per load, see the fp32 role; 24 requests on 64/8 heads, k = 3 47.4 -> 40.7 us)
                         ? __builtin_amdgcn_raw_buffer_load_b128(kd, n16 * (D * 2) + g * 16, i * 64, 0)
                         : __builtin_amdgcn_raw_buffer_load_b128(kd, lane_off, i * 1024, kStreamPolicy);
        // V: in operand order already, or (token-major) as whole rows: with D / 8 lanes per row, lane L of load i holds
        // token (512 / D) i + 8 L / D, dims 8 (L % (D / 8)) .. + 7
#pragma unroll
        for (int i = 0; i < KK; ++i) r.v[i] = __builtin_amdgcn_raw_buffer_load_b128(vd, lane_off, i * 1024, kStreamPolicy);
    };

    // K or V of the it-th page of this wavefront
    auto load_half = [&](int it, const char *head, bool direct, u32x4(&r)[KK]) {
        const int entry = __builtin_amdgcn_readlane(bt, it < my_pages ? it : 0);
        const bool valid = it < my_pages && entry >= 0;
        const __amdgpu_buffer_rsrc_t desc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(head + (size_t)(valid ? entry : 0) * page_stride), 0, valid ? kPageHeadBytes : 0, kBufferFlags);
#pragma unroll
        for (int i = 0; i < KK; ++i)
            r[i] = direct ? __builtin_amdgcn_raw_buffer_load_b128(desc, n16 * (D * 2) + g * 16, i * 64, 0)
                          : __builtin_amdgcn_raw_buffer_load_b128(desc, lane_off, i * 1024, kStreamPolicy);
    };

    f32x4 acc[NT][MT];
    float m_run[NT], l_run[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_run[nt] = kEmptyMax;
        l_run[nt] = 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    }

    const int first_masked_token = L - q_len + 1;  // keys from here on are hidden from some row (or past the end)

    // The reference of the running sums follows the maximum lazily: it is raised only when
    // a score exceeds it by more than 8 (base-2 units), so weights reach at most 2^8 and
    // the accumulators are rescaled on few pages instead of on most early ones (the
    // result is the same up to rounding: numerator and denominator share the reference).
    // So a row's maximum over its four lanes is only taken when one of them exceeds the reference by that much: the exchange
    // between the lanes is no part of the chain from a page's scores to its weights (attention alone, 64/4
    // heads, k = 8, 64 requests of 300 to 900 tokens: 66.8 -> 63.5 us; 64/8 heads, k = 7, 96 requests 64.5 -> 63.7; memory-bound
    // launches unchanged).
    auto raise_reference = [&](int nt, float mx) {   // mx: largest unscaled score of this lane's tokens
        mx *= p.scale_log2;
        const float most = m_run[nt] + kRescaleSlack;
        if (__builtin_amdgcn_ballot_w64(mx > most) == 0) return;
        mx = max_across_xor32(max_across_xor16(mx));
        const float m_new = mx > most ? mx : m_run[nt];
        const float alpha = fast_exp2(m_run[nt] - m_new);
        l_run[nt] *= alpha;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] *= alpha;
        m_run[nt] = m_new;
    };

    auto consume = [&](PageRegs<D> &cur, int pi) {
        const int page_tok = tok0 + pi * SPEC_BLOCK_SIZE;
        const bool need_mask = page_tok + SPEC_BLOCK_SIZE > first_masked_token;
        const int tbase = page_tok + 4 * g;

        if constexpr (TM && !STAGED) {
            // through this wavefront's LDS region: rows in, operand order out (LDS executes a wavefront's
            // accesses in order, so the reads see the writes without a barrier)
            unsigned char *kl = sh.vt + wave * (2 * kVtWaveBytes), *vl = kl + kVtWaveBytes;
            constexpr int LR = D / 8;   // lanes per token row of a 1 KB load (16 bytes each)
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                const int at = ((kWave / LR) * i + lane / LR) * kVtRowBytes + (lane % LR) * 16;
                if constexpr (!K_DIRECT) *reinterpret_cast<u32x4 *>(kl + at) = cur.k[i];
                *reinterpret_cast<u32x4 *>(vl + at) = cur.v[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                if constexpr (!K_DIRECT) cur.k[i] = *reinterpret_cast<const u32x4 *>(kl + n16 * kVtRowBytes + i * 64 + g * 16);
                const unsigned char *src = vl + (4 * g + (n16 >> 2)) * kVtRowBytes + (n16 & 3) * 8 + i * 64;
                const u32x2 lo = read_transposed(src), hi = read_transposed(src + 32);
                cur.v[i] = (u32x4){lo.x, lo.y, hi.x, hi.y};
            }
        }

        if (page_tok + SPEC_BLOCK_SIZE > L) {
            // slots past kv_len in the request's last page may hold anything: clear their V
            // (the branch is the same for the whole wavefront and holds no loads)
            const int nvalid = min(max(L - tbase, 0), 4);
            const uint32_t lo = nvalid >= 2 ? 0xFFFFFFFFu : (nvalid == 1 ? 0x0000FFFFu : 0u);
            const uint32_t hi = nvalid >= 4 ? 0xFFFFFFFFu : (nvalid == 3 ? 0x0000FFFFu : 0u);
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                cur.v[i].x &= lo; cur.v[i].y &= hi;
                cur.v[i].z &= lo; cur.v[i].w &= hi;
            }
        }

#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt > 0 && nt * 16 >= grp_rows) continue;   // a tile this request has no rows for (the same for the whole wavefront)
            f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur.k[kk]), qreg[nt][kk], s, 0, 0, 0);
            // (the softmax scale, folded with log2 e, is applied inside the exponent's fused
            // multiply-add below; the maximum commutes with it, the scale being positive)
            if (need_mask) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (tbase + r > limit[nt]) s[r] = -INFINITY;
            }
            raise_reference(nt, fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
            f32x4 pr;
#pragma unroll
            for (int r = 0; r < 4; ++r) pr[r] = fast_exp2(fmaf(s[r], p.scale_log2, -m_run[nt]));
            l_run[nt] += (pr[0] + pr[1]) + (pr[2] + pr[3]);
            const bf16x4 p_hi = __builtin_convertvector(pr, bf16x4);
            bf16x4 p_lo;
            if (SPLIT_P) p_lo = __builtin_convertvector(pr - __builtin_convertvector(p_hi, f32x4), bf16x4);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const u32x4 vv = cur.v[mt >> 1];
                const u32x2 half = (mt & 1) ? (u32x2){vv.z, vv.w} : (u32x2){vv.x, vv.y};
                const bf16x4 va = __builtin_bit_cast(bf16x4, half);
                acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, p_hi, acc[nt][mt], 0, 0, 0);
                if (SPLIT_P) acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, p_lo, acc[nt][mt], 0, 0, 0);
            }
        }
    };

    // Two pages at a time: their scores are two independent chains, one look at the reference serves both, and the output
    // product contracts 32 tokens per instruction, which the matrix cores take at twice the rate of 16 (slots 8 g .. + 3 of
    // the contraction are the first page's tokens 4 g .. + 3, the other four the second's).  k0, k1: the pages' K operands;
    // then_values is called once they are used and gives V's: v[mt] for dims 16 mt .. + 15, the first page's tokens in x
    // and y, the second's in z and w.  has1 == false: there is no second page (its operands are finite).
    auto consume_pair = [&](const u32x4(&k0)[KK], const u32x4(&k1)[KK], auto then_values, int pi0, int pi1, bool has1) {
        const int tb0 = tok0 + pi0 * SPEC_BLOCK_SIZE + 4 * g, tb1 = tok0 + pi1 * SPEC_BLOCK_SIZE + 4 * g;
        const bool need_mask = !has1 || tok0 + (pi1 + 1) * SPEC_BLOCK_SIZE > first_masked_token;
        f32x4 s[NT][2];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            s[nt][0] = s[nt][1] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
            if (nt > 0 && nt * 16 >= grp_rows) continue;   // a tile this request has no rows for (the same for the whole wavefront)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                s[nt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k0[kk]), qreg[nt][kk], s[nt][0], 0, 0, 0);
                s[nt][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k1[kk]), qreg[nt][kk], s[nt][1], 0, 0, 0);
            }
        }
        u32x4 v[MT];
        then_values(v);
        if (!has1 || tok0 + (pi1 + 1) * SPEC_BLOCK_SIZE > L) {   // slots past kv_len may hold anything: clear their V
            const int n0 = L - tb0, n1 = has1 ? L - tb1 : 0;
            const u32x4 keep = {n0 >= 2 ? 0xFFFFFFFFu : (n0 == 1 ? 0x0000FFFFu : 0u), n0 >= 4 ? 0xFFFFFFFFu : (n0 == 3 ? 0x0000FFFFu : 0u),
                                n1 >= 2 ? 0xFFFFFFFFu : (n1 == 1 ? 0x0000FFFFu : 0u), n1 >= 4 ? 0xFFFFFFFFu : (n1 == 3 ? 0x0000FFFFu : 0u)};
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) v[mt] &= keep;
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt > 0 && nt * 16 >= grp_rows) continue;
            if (need_mask) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (tb0 + r > limit[nt]) s[nt][0][r] = -INFINITY;
                    if (!has1 || tb1 + r > limit[nt]) s[nt][1][r] = -INFINITY;
                }
            }
            float mx = fmaxf(fmaxf(s[nt][0][0], s[nt][0][1]), fmaxf(s[nt][0][2], s[nt][0][3]));
            mx = fmaxf(mx, fmaxf(fmaxf(s[nt][1][0], s[nt][1][1]), fmaxf(s[nt][1][2], s[nt][1][3])));
            raise_reference(nt, mx);
            bf16x8 p_hi, p_lo;
            float sum = 0.0f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 pr;
#pragma unroll
                for (int r = 0; r < 4; ++r) pr[r] = fast_exp2(fmaf(s[nt][h][r], p.scale_log2, -m_run[nt]));
                sum += (pr[0] + pr[1]) + (pr[2] + pr[3]);
                const bf16x4 hi = __builtin_convertvector(pr, bf16x4);
                const bf16x4 lo = __builtin_convertvector(pr - __builtin_convertvector(hi, f32x4), bf16x4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p_hi[4 * h + r] = hi[r];
                    p_lo[4 * h + r] = lo[r];
                }
            }
            l_run[nt] += sum;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const bf16x8 va = __builtin_bit_cast(bf16x8, v[mt]);
                acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, p_hi, acc[nt][mt], 0, 0, 0);
                acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, p_lo, acc[nt][mt], 0, 0, 0);
            }
        }
    };
    // Operands of a page out of LDS (token rows, padded): K as 16 bytes of a row, V through the transposing read.
    auto k_operand = [&](const unsigned char *page, int i) { return *reinterpret_cast<const u32x4 *>(page + n16 * kVtRowBytes + i * 64 + g * 16); };
    auto v_operands = [&](const unsigned char *page0, const unsigned char *page1, u32x4(&v)[MT]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int at = (4 * g + (n16 >> 2)) * kVtRowBytes + (n16 & 3) * 8 + mt * 32;
            const u32x2 v0 = read_transposed(page0 + at), v1 = read_transposed(page1 + at);
            v[mt] = (u32x4){v0.x, v0.y, v1.x, v1.y};
        }
    };

    // Q as the B operand of S^T = K Q^T, out of LDS (the first pages are on their way)
    auto stage_q = [&] {
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            const int piece = tid + i * kThreads;
            if (QI * kThreads == NT * WG * 16 * QP || piece < NT * WG * 16 * QP)
                *reinterpret_cast<u32x4 *>(sh.q + (piece / QP) * kQStride + (piece % QP) * 16) = qpiece[i];
        }
        __syncthreads();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                qreg[nt][kk] = *reinterpret_cast<const bf16x8 *>(sh.q + (row_lo + nt * 16 + n16) * kQStride + kk * 64 + g * 16);
        }
        __syncthreads();   // the epilogue reuses this memory
    };

    if constexpr (STAGED) {
        // The staged walk, for wave groups on token-major pages.  All groups need all pages, so the block loads each
        // page once, a page per wavefront and round, DEPTH rounds ahead in registers, and hands it to the groups
        // through LDS (two buffers, one barrier per round): whole rows go in, operands come out (K as 16
        // bytes of a token row, V through the transposing LDS read; rows padded as above).  When every group loaded
        // the pages for itself, half (three quarters) of the loads in flight were duplicates, K's came in
        // half cache lines, and V was transposed once per group.  Attention alone, 64/8 heads, k = 7, 96 / 256
        // requests of 256 to 1024 tokens: 82.8 -> 66.9 / 191.5 -> 145.2 us; 64/4 heads, k = 4 / 8: 81.3 -> 65.5 /
        // 124.8 -> 113.1 us.  Pages in the matrix-operand layout gain less and not always (the same shapes: 64.5
        // -> 65.6, 152.0 -> 143.6, 67.9 -> 65.0, 107.8 -> 109.4; two split requests 28.6 -> 30.0), so there every
        // group still loads its operands itself.
        // (The walk ends with its last round: rounds rounded up to DEPTH cost short contexts a store, a load and a
        // barrier for nothing.  64/8 heads, k = 7, four requests of 16 / 64 / 200 tokens: 7.4 / 8.2 / 12.35 us -> 6.8 / 7.75 / 12.3.)
        constexpr int DEPTH = NT >= 3 && D == 128 ? 1 : 2;   // (three row tiles leave no registers for a second round)
        constexpr int LR = D / 8;   // lanes per token row of a 1 KB load (16 bytes each)
        const int rounds = (w.npages + kWaves - 1) / kWaves;
        PageRegs<D> st[DEPTH];
        auto store_page = [&](int buf, const PageRegs<D> &r) {
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                const int at = ((kWave / LR) * i + lane / LR) * kVtRowBytes + (lane % LR) * 16;
                *reinterpret_cast<u32x4 *>(sh.ring[buf][wave][0] + at) = r.k[i];
                *reinterpret_cast<u32x4 *>(sh.ring[buf][wave][1] + at) = r.v[i];
            }
        };
        auto fetch_page = [&](int buf, int slot, PageRegs<D> &r) {
            const unsigned char *ks = sh.ring[buf][slot][0], *vs = sh.ring[buf][slot][1];
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                r.k[i] = *reinterpret_cast<const u32x4 *>(ks + n16 * kVtRowBytes + i * 64 + g * 16);
                const unsigned char *src = vs + (4 * g + (n16 >> 2)) * kVtRowBytes + (n16 & 3) * 8 + i * 64;
                const u32x2 lo = read_transposed(src), hi = read_transposed(src + 32);
                r.v[i] = (u32x4){lo.x, lo.y, hi.x, hi.y};
            }
        };
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) load_page(i, st[i]);
        stage_q();
        store_page(0, st[0]);
        load_page(DEPTH, st[0]);
        __syncthreads();
        [&] {
            for (int t = 0;; t += DEPTH) {
#pragma unroll
                for (int i = 0; i < DEPTH; ++i) {
                    const int round = t + i;
                    if (grp_rows > 0) {
#pragma unroll 1
                        for (int slot = pw; slot < kWaves; slot += PAIRS_STAGED ? 2 * PW : PW) {
                            const int page = round * kWaves + slot;
                            if (page < w.npages) {
                                if constexpr (PAIRS_STAGED) {
                                    const unsigned char(*ring0)[kVtWaveBytes] = sh.ring[round & 1][slot], (*ring1)[kVtWaveBytes] = sh.ring[round & 1][slot + PW];
                                    u32x4 k0[KK], k1[KK];
#pragma unroll
                                    for (int i = 0; i < KK; ++i) {
                                        k0[i] = k_operand(ring0[0], i);
                                        k1[i] = k_operand(ring1[0], i);
                                    }
                                    consume_pair(k0, k1, [&](u32x4(&v)[MT]) { v_operands(ring0[1], ring1[1], v); }, page, page + PW, page + PW < w.npages);
                                } else {
                                    PageRegs<D> cur;
                                    fetch_page(round & 1, slot, cur);
                                    consume(cur, page);
                                }
                            }
                        }
                    }
                    if (round + 1 >= rounds) return;
                    store_page((round + 1) & 1, st[(i + 1) % DEPTH]);
                    load_page(round + 1 + DEPTH, st[(i + 1) % DEPTH]);
                    __syncthreads();
                }
            }
        }();
        __syncthreads();   // every wavefront is done with the ring: the epilogue reuses the memory
    } else if constexpr (PAIR_WALK) {
        // Two pages at a time: the next pair's K is loaded once this pair's scores are done, its V once this pair's V is
        // in LDS, so that half a pair at least is always in flight.
        u32x4 k0[KK], k1[KK], v0[KK], v1[KK];
        auto load_k = [&](int it) { load_half(it, khead, K_DIRECT, k0); load_half(it + 1, khead, K_DIRECT, k1); };
        auto load_v = [&](int it) { load_half(it, vhead, false, v0); load_half(it + 1, vhead, false, v1); };
        load_k(0);
        load_v(0);
        stage_q();
        // this wavefront's LDS region: room for two pages, K's and then V's (LDS executes a wavefront's accesses in order,
        // so reads see the writes before them, and no write overtakes a read, without a barrier)
        unsigned char *const lds0 = sh.vt + wave * (2 * kVtWaveBytes), *const lds1 = lds0 + kVtWaveBytes;
        constexpr int LR = D / 8;   // lanes per token row of a 1 KB load (16 bytes each)
        auto to_lds = [&](const u32x4(&r0)[KK], const u32x4(&r1)[KK]) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                const int at = ((kWave / LR) * i + lane / LR) * kVtRowBytes + (lane % LR) * 16;
                *reinterpret_cast<u32x4 *>(lds0 + at) = r0[i];
                *reinterpret_cast<u32x4 *>(lds1 + at) = r1[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        // (A last page without a partner goes by itself, at half the work of a pair: 130 requests of 9 to 16 / 49 to 64 / 300 to 900
        // tokens on 32/8 heads, k = 7 15.8 -> 14.4 / 16.8 -> 15.1 / 39.2 -> 37.7 us.  Not with K straight into operand order,
        // whose sums have to equal the staged walk's, and there code for both spills or is slower: 25.2 -> 26.2 at 64 dims.)
        int it = 0;
        for (; it < (K_DIRECT ? my_pages : my_pages - 1); it += 2) {
            if constexpr (!K_DIRECT) {
                to_lds(k0, k1);
#pragma unroll
                for (int i = 0; i < KK; ++i) {
                    k0[i] = k_operand(lds0, i);
                    k1[i] = k_operand(lds1, i);
                }
            }
            consume_pair(k0, k1, [&](u32x4(&v)[MT]) {
                load_k(it + 2);
                to_lds(v0, v1);
                load_v(it + 2);
                v_operands(lds0, lds1, v);
            }, pw + PW * it, pw + PW * (it + 1), !K_DIRECT || it + 1 < my_pages);
        }
        if (!K_DIRECT && it < my_pages) {
            PageRegs<D> last;
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                last.k[i] = k0[i];
                last.v[i] = v0[i];
            }
            consume(last, pw + PW * it);
        }
    } else {
        // Two register batches of P pages each.  While one batch is consumed the loads of the
        // other are in flight.  The order inside a half-step matters: first wait for the batch
        // about to be consumed (at that point it is the only one outstanding, so the full
        // wait the compiler emits waits for nothing else), then issue the other batch's loads,
        // then do the arithmetic, which needs no further wait.
        // pages per batch: two bring nothing once the launch keeps the memory system busy, except with the
        // half-size pages of a head dim of 64 (the same bytes in flight per wavefront as at 128)
        constexpr int P = D == 64 ? 2 : 1;
        PageRegs<D> batch_a[P], batch_b[P];
        auto load_batch = [&](int it, PageRegs<D>(&r)[P]) {
#pragma unroll
            for (int j = 0; j < P; ++j) load_page(it + j, r[j]);
        };
        auto arrived = [&](PageRegs<D>(&r)[P]) {
#pragma unroll
            for (int j = 0; j < P; ++j) {
                if constexpr (KK == 4)
                    asm volatile("" ::"v"(r[j].k[0]), "v"(r[j].k[1]), "v"(r[j].k[2]), "v"(r[j].k[3]), "v"(r[j].v[0]),
                                 "v"(r[j].v[1]), "v"(r[j].v[2]), "v"(r[j].v[3])
                                 : "memory");
                else
                    asm volatile("" ::"v"(r[j].k[0]), "v"(r[j].k[1]), "v"(r[j].v[0]), "v"(r[j].v[1]) : "memory");
            }
        };
        auto consume_batch = [&](PageRegs<D>(&r)[P], int it) {
#pragma unroll
            for (int j = 0; j < P; ++j)
                if (it + j < my_pages) consume(r[j], pw + PW * (it + j));
        };
        load_batch(0, batch_a);
        stage_q();
        for (int it0 = 0; it0 < my_pages; it0 += 2 * P) {
            arrived(batch_a);
            load_batch(it0 + P, batch_b);
            consume_batch(batch_a, it0);
            arrived(batch_b);
            load_batch(it0 + 2 * P, batch_a);
            consume_batch(batch_b, it0 + P);
        }
    }

    if constexpr (TM && !STAGED) __syncthreads();   // every wavefront is done with its staging region: the epilogue reuses the memory
    attn_end<NT, WG, D, (WG > 1)>(p, w, acc, m_run, l_run, out_row, [](int mt, int gg) { return mt * 16 + 4 * gg; }, sh);
}

// ---------------------------------------------------------------------------
// The attention role in fp32 (token-major pages).  As above: one block per (request, KV head, chunk), all query
// rows of a KV head fused, K and V read once.  Per 16-token page and 16-row tile, lane = 16 g + n:
//   S^T[token][row] = K[token][:] . Q[row][:]     D / 4 x v_mfma_f32_16x16x4_f32
//   O^T[dim][row] += V^T[dim][token] . P^T[token][row]     D / 4 x v_mfma_f32_16x16x4_f32
// The order of a contraction and the numbering of output dims are free, so every operand comes straight
// out of 16-byte loads: lane (g, n) holds dims 16 i + 4 g + e of token n for K (and of row n for Q: its
// element e is step 4 i + e of the score product), and dims 64 h + 4 n + e of token 4 g + r for V (its element e
// is the A operand of output slice 4 h + e, step r, whose B operand is P^T in the scores' own layout).
// Two row tiles (32 rows, padding included) take 10.4 us of matrix instructions per 100 MB of pages at the 154 TFLOP/s
// of a large product (8 flops per byte and tile of 16 rows), against 15 us of reading: memory bounds one and two
// tiles, the matrix instructions three (15.6 us).  Q stays in LDS: its operands for three tiles would take 96 registers,
// and the 8 LDS reads per page and tile cost a thirtieth of the 64 matrix instructions they feed.
// One batch of registers each for K and V: the next page's K is loaded once this page's scores are done, its
// V once the output product is, so that half a page (8 KB, as much as the bf16 role has) is always in
// flight per wavefront.
// Before, fp32 ran on scalar kernels, one block per query row and head, which read K and V from the L2 once
// for each: eight requests of 256 to 1024 tokens, 32/8 heads, k = 4: 177.3 -> 24.5 us; a step of one request
// of 128 tokens, now one launch instead of two: 22.2 -> 13.2 us.  The error against 64 bits went from 4.5e-7
// to 2.8e-7 of the output's norm.
// ---------------------------------------------------------------------------
constexpr int f32_q_stride(int D) { return D * 4 + 16; }   // bytes per query row in LDS (padded: 16 rows cover all banks)

template <int NT, int WG, int D>
struct AttnF32Shared {
    union {
        f32x4 acc[2][NT][D / 16][kWave];                             // epilogue: partial results of the wavefronts being merged
        unsigned char q[WG * NT * 16 * f32_q_stride(D)];             // the block's query rows
        unsigned char o[WG == 1 ? NT * 16 * o_stride(D) : 16];       // epilogue of an unsplit request (one group): the output tile
    };
    float m[2][NT][kWave];
    float l[2][NT][kWave];
    int last;
};

// (K_POLICY: cache policy of the K loads)
template <int NT, int WG, int D, int K_POLICY>
__device__ __forceinline__ void attn_f32_role(const AttnParams &p, OrderTable order, int item, AttnF32Shared<NT, WG, D> &sh)
{
    constexpr int KI = D / 16;                        // 16-byte K loads per lane and page
    constexpr int VH = D / 64;                        // ... V loads per lane and token
    constexpr int MT = D / 16;
    constexpr int PW = kWaves / WG;
    constexpr int kQStride = f32_q_stride(D);
    constexpr int kPageHeadBytes = SPEC_BLOCK_SIZE * D * 4;
    AttnWork w;
    if (!attn_begin<NT, WG, false>(p, order, item, w)) return;
    const int n16 = w.n16, g = w.g, L = w.L, my_pages = w.my_pages, bt = w.bt;

    const char *khead = static_cast<const char *>(p.k_cache) + (size_t)w.kvh * kPageHeadBytes;
    const char *vhead = static_cast<const char *>(p.v_cache) + (size_t)w.kvh * kPageHeadBytes;
    const size_t page_stride = (size_t)p.Hkv * kPageHeadBytes;
    // (descriptors as in the bf16 role: exactly one (page, KV head), empty past the end)
    auto page_desc = [&](const char *head, int it) {
        const int entry = __builtin_amdgcn_readlane(bt, it < my_pages ? it : 0);
        const bool valid = it < my_pages && entry >= 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(head + (size_t)(valid ? entry : 0) * page_stride), 0,
                                                 valid ? kPageHeadBytes : 0, kBufferFlags);
    };
    f32x4 k[KI], v[4][VH];   // v[r][h]: token 4 g + r, dims 64 h + 4 n16 ..
    // (K without the streaming hint: a load takes 64 bytes of each token row, half a cache line, and the other half, which
    // the next load wants, is gone by then if the line is first in line for replacement.  Eight requests on 32/32 heads, k = 4: 39.8 -> 35.1
    // us; on 32/8, k = 2: 18.3 -> 17.4.  With it beside many rejection blocks, see launch_f32.)
    auto load_k = [&](int it) {
        const __amdgpu_buffer_rsrc_t d = page_desc(khead, it);
#pragma unroll
        for (int i = 0; i < KI; ++i)
            k[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(d, n16 * (D * 4) + g * 16, i * 64, K_POLICY));
    };
    auto load_v = [&](int it) {
        const __amdgpu_buffer_rsrc_t d = page_desc(vhead, it);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < VH; ++h)
                v[r][h] = __builtin_bit_cast(
                    f32x4, __builtin_amdgcn_raw_buffer_load_b128(d, g * (D * 16) + n16 * 16, r * (D * 4) + h * 256, kStreamPolicy));
    };
    load_k(0);
    load_v(0);

    // the block's query rows: 16 bytes per thread, consecutive threads along a row
    constexpr int QP = D / 4;
    for (int piece = w.tid; piece < NT * WG * 16 * QP; piece += kThreads) {
        const int r = piece / QP, c = piece % QP;
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
        if (r < w.rows) {
            const size_t rh = (size_t)(w.row0 + r / w.group) * p.Hq + w.kvh * w.group + r % w.group;
            x = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(p.q) + rh * D + c * 4);
        }
        *reinterpret_cast<f32x4 *>(sh.q + r * kQStride + c * 16) = x;
    }
    int limit[NT];     // each lane's last visible key
    int out_row[NT];   // packed (token row * Hq + head) of this lane's query row, -1 if padding
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int r = w.row_lo + nt * 16 + n16;
        const bool valid = r < w.rows;
        const int j = valid ? r / w.group : 0;
        limit[nt] = valid ? L - w.q_len + j : -1;
        out_row[nt] = valid ? (w.row0 + j) * p.Hq + w.kvh * w.group + r % w.group : -1;
    }
    __syncthreads();

    f32x4 acc[NT][MT];   // slice 4 h + e, element r of a lane: dim 64 h + 16 g + 4 r + e of query row n16
    float m_run[NT], l_run[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_run[nt] = kEmptyMax;
        l_run[nt] = 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    }
    const int first_masked_token = L - w.q_len + 1;

    for (int it = 0; it < my_pages; ++it) {
        const int page_tok = w.tok0 + (w.pw + PW * it) * SPEC_BLOCK_SIZE;
        const int tbase = page_tok + 4 * g;
        const bool need_mask = page_tok + SPEC_BLOCK_SIZE > first_masked_token;
        f32x4 pr[NT];   // scores, then softmax weights
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt > 0 && nt * 16 >= w.grp_rows) continue;   // a tile this request has no rows for (the same for the whole wavefront)
            const unsigned char *qrow = sh.q + (w.row_lo + nt * 16 + n16) * kQStride + g * 16;
            f32x4 s0 = {0.0f, 0.0f, 0.0f, 0.0f}, s1 = s0;   // (two chains: an instruction need not wait for the one before it)
#pragma unroll
            for (int i = 0; i < KI; ++i) {
                const f32x4 q = *reinterpret_cast<const f32x4 *>(qrow + i * 64);
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][0], q[0], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][1], q[1], s1, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][2], q[2], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][3], q[3], s1, 0, 0, 0);
            }
            pr[nt] = s0 + s1;
        }
        load_k(it + 1);

        bool odd_values = false;   // a value that is not finite in a page with hidden keys
        if (need_mask) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int h = 0; h < VH; ++h) {
                    // slots past kv_len may hold anything: clear their V
                    if (tbase + r >= L) v[r][h] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) odd_values = odd_values || !(fabsf(v[r][h][e]) < INFINITY);
                }
            odd_values = __builtin_amdgcn_ballot_w64(odd_values) != 0;
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt > 0 && nt * 16 >= w.grp_rows) continue;
            f32x4 s = pr[nt];
            if (need_mask) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (tbase + r > limit[nt]) s[r] = -INFINITY;
            }
            // online softmax with a lazily raised reference, see the bf16 role
            float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
            mx = max_across_xor32(max_across_xor16(mx)) * p.scale_log2;
            const float m_new = mx > m_run[nt] + kRescaleSlack ? mx : m_run[nt];
#pragma unroll
            for (int r = 0; r < 4; ++r) pr[nt][r] = fast_exp2(fmaf(s[r], p.scale_log2, -m_new));
            if (__builtin_amdgcn_ballot_w64(m_new != m_run[nt]) != 0) {
                const float alpha = fast_exp2(m_run[nt] - m_new);
                l_run[nt] *= alpha;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[nt][mt] *= alpha;
                m_run[nt] = m_new;
            }
            l_run[nt] += (pr[nt][0] + pr[nt][1]) + (pr[nt][2] + pr[nt][3]);
            if (!odd_values) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][mt / 4][mt % 4], pr[nt][r], acc[nt][mt], 0, 0, 0);
                continue;
            }
            // A hidden key's weight is 0, but 0 times infinity or NaN is not: token by token, and added only to the
            // rows that see the token.
#pragma unroll
            for (int r = 0; r < 4; ++r)
                for (int gt = 0; gt < 4; ++gt) {
                    const bool visible = page_tok + 4 * gt + r <= limit[nt];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const f32x4 one = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            g == gt ? v[r][mt / 4][mt % 4] : 0.0f, g == gt ? pr[nt][r] : 0.0f, (f32x4){0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[nt][mt][e] = visible ? acc[nt][mt][e] + one[e] : acc[nt][mt][e];
                    }
                }
        }
        load_v(it + 1);
    }
    __syncthreads();   // every wavefront is done with the query rows: the epilogue reuses their memory

    f32x4 out[NT][MT];   // slice 4 h + r: four consecutive dims from 64 h + 16 g + 4 r
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int e = 0; e < 4; ++e) out[nt][mt][e] = acc[nt][mt / 4 * 4 + e][mt % 4];
    attn_end<NT, WG, D, true>(p, w, out, m_run, l_run, out_row, [](int mt, int gg) { return mt / 4 * 64 + 16 * gg + mt % 4 * 4; }, sh);
}

// ===========================================================================
// The kernel
// ===========================================================================
// Grid order.  The hardware dispatcher places blocks strictly in grid order and waits for
// the slot it has chosen, so block slots sit idle when neighbouring blocks run for very
// different times.  The order keeps neighbours alike and ends on independent work.
// The rejection items always keep their own order (statistics, race, final).
//  - No more attention blocks than block slots: attention first.  All of them are
//    resident from the start (one per compute unit if there are few: two on one unit
//    would take twice as long as the rest), and the rejection items flow through the
//    slots that are left.
//  - More attention blocks: they take the requests longest first (so blocks that run at
//    the same time take about equally long), and the rejection items are mixed into the
//    first part of them (reject_span of the attention rows), so that the dependent
//    rejection stages are done before the attention items are and the tail of the launch
//    is short attention blocks.  The mixing is done per row of 8 consecutive blocks: the
//    hardware deals consecutive blocks to the 8 XCDs in turn, and a finer pattern would
//    alias with that (with equal counts, "every other block" would put all attention on
//    four XCDs and all rejection on the other four).  Within the mixed part, row r is an
//    attention row iff floor((r+1) * rows_attn / rows) > floor(r * rows_attn / rows).
struct GridSplit {
    int n_stat, n_reject, n_attn;
    int attn_first;        // 1: attention items first, 0: mixed (with no attention rows in the mixed part: rejection items first)
    int rows_attn_mixed;   // attention rows among which the rejection rows are spread; the other attention rows follow
    int reject_cols;       // positions of a row of 8 blocks that carry rejection items: all 8, or the 4 even ones
};

// All kernel arguments in one struct, so that the place of the order table inside the
// kernel-argument segment is known.
struct StepArgs {
    AttnParams ap;
    RejectParams rp;
    GridSplit gs;
    UnitOrder order;
};

// The work item of a block of a launch that holds both halves; false: a padding block.
__device__ __forceinline__ bool grid_item(const GridSplit &gs, int &item, bool &is_attn)
{
    item = blockIdx.x;
    if (gs.attn_first) {
        const int n_attn_rows8 = (gs.n_attn + kXcds - 1) / kXcds * kXcds;   // whole rows: positions keep their XCD
        is_attn = item < n_attn_rows8;
        if (is_attn) {
            if (item >= gs.n_attn) return false;   // padding of the last attention row
        } else {
            item -= n_attn_rows8;
            if (gs.reject_cols != kXcds) {
                if (item & 1) return false;
                item >>= 1;
            }
            if (item >= gs.n_reject) return false;
        }
    } else {
        // rows of kXcds consecutive blocks (one per XCD, the hardware deals blocks to the
        // XCDs round-robin) share a role, so every XCD sees the same mix
        const int row = item / kXcds, col = item % kXcds;
        const long long rows_attn = gs.rows_attn_mixed;
        const long long rows_all = rows_attn + (gs.n_reject + gs.reject_cols - 1) / gs.reject_cols;
        if (row < rows_all) {
            const int before = (int)((row * rows_attn) / rows_all);
            const int upto = (int)(((row + 1) * rows_attn) / rows_all);
            is_attn = upto > before;
            if (is_attn) {
                item = before * kXcds + col;
            } else if (gs.reject_cols == kXcds) {
                item = (row - before) * kXcds + col;
            } else {
                if (col & 1) return false;
                item = (row - before) * (kXcds / 2) + (col >> 1);
            }
        } else {   // the attention rows after the last rejection row
            is_attn = true;
            item = (int)(rows_attn + (row - rows_all)) * kXcds + col;
        }
        if (item >= (is_attn ? gs.n_attn : gs.n_reject)) return false;   // padding of the last row
    }
    return true;
}

// (PEEK: the kernel knows kStopPeek.  The fp32 kernel and the rejection half's do not: all code beside the stages costs the smallest
// launches, this one 0.9 of the smallest fp32 step's 12.7 us.)
template <int DEPTH, bool PEEK>
__device__ __forceinline__ void reject_item(const RejectParams &p, int n_stat, int item, RejectShared &sh)
{
    if (item < n_stat) {
        stats_role<DEPTH, PEEK>(p, item, sh);
        return;
    }
    const int after = item - n_stat;
    const int n_race = p.B * p.race_segments;
    if (after < n_race) race_role(p, after, sh);
    else final_role(p, after - n_race, sh);
}

__device__ __forceinline__ OrderTable order_table(int n)
{
    OrderTable order;
    order.n = n;
    order.pairs = (uniform_u32_ptr)((const char __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr() +
                                    offsetof(StepArgs, order) + offsetof(UnitOrder, request));
    return order;
}

// Blocks per compute unit the registers have to allow: two, and four where the attention variant needs
// no more registers than that (one row tile at a head dim of 64) or is absent, so that the race does not
// take more.
template <int NT, bool HAS_ATTN, int VAR>
constexpr int kMinBlocks = !HAS_ATTN || (NT == 1 && head_dim_of(VAR) == 64) ? 4 : 2;

template <int NT, int WG, bool HAS_ATTN, bool HAS_REJECT, int VAR>
__global__ __launch_bounds__(kThreads, (kMinBlocks<NT, HAS_ATTN, VAR>)) void spec_step_kernel(StepArgs args)
{
    const AttnParams &ap = args.ap;
    const RejectParams &rp = args.rp;
    int item = blockIdx.x;
    bool is_attn = HAS_ATTN;
    if constexpr (HAS_ATTN && HAS_REJECT)
        if (!grid_item(args.gs, item, is_attn)) return;
    // one piece of LDS for either role
    typedef AttnShared<NT, WG, token_major_of(VAR), head_dim_of(VAR)> AttnSh;
    constexpr size_t kSharedBytes = !HAS_REJECT ? sizeof(AttnSh)
                                    : (!HAS_ATTN || sizeof(RejectShared) > sizeof(AttnSh) ? sizeof(RejectShared) : sizeof(AttnSh));
    __shared__ alignas(16) unsigned char shared[kSharedBytes];
    if constexpr (HAS_REJECT) {
        if (!is_attn) {
            // a whole 32000-entry row per round trip where the registers allow it
            reject_item<(HAS_ATTN && NT >= 2) ? 8 : 4, HAS_ATTN>(rp, args.gs.n_stat, item, *reinterpret_cast<RejectShared *>(shared));
            return;
        }
    }
    if constexpr (HAS_ATTN) {
        AttnSh &ash = *reinterpret_cast<AttnSh *>(shared);
        attn_role<NT, WG, VAR>(ap, order_table(args.order.n), item, ash);
    }
}

// The attention alone on token-major pages of a head dim of 128, with K loaded straight into operand order
// (each load touches 16 half cache lines) and only V staged, every wave group reading its pages itself.  The chain from a
// page's arrival to its scores is shorter by a trip through LDS, which is what some launches wait for (the planner's
// k_direct says which, and what both measured); a kernel of its own, because the choice inside the other costs its launches 0.7%.
template <int NT, int WG>
__global__ __launch_bounds__(kThreads, 2) void attn_k_direct_kernel(StepArgs args)
{
    typedef AttnShared<NT, WG, true, kD, true> AttnSh;
    __shared__ alignas(16) unsigned char shared[sizeof(AttnSh)];
    attn_role<NT, WG, 2, true>(args.ap, order_table(args.order.n), blockIdx.x, *reinterpret_cast<AttnSh *>(shared));
}

// The step in fp32: the same grid and roles.  A launch of the attention alone has no rejection items.
// (Three row tiles take over 256 registers at a head dim of 128: 33 to 48 rows run as two wave groups of two
// tiles, and only the widest shapes, 129 to 144 rows, as four groups of three with one block per compute unit.)
template <int NT, int WG, int D, int K_POLICY = 0>
__global__ __launch_bounds__(kThreads, (NT == 3 ? 1 : 2)) void f32_step_kernel(StepArgs args)
{
    int item;
    bool is_attn;
    if (!grid_item(args.gs, item, is_attn)) return;
    typedef AttnF32Shared<NT, WG, D> AttnSh;
    __shared__ alignas(16) unsigned char shared[sizeof(RejectShared) > sizeof(AttnSh) ? sizeof(RejectShared) : sizeof(AttnSh)];
    if (is_attn) attn_f32_role<NT, WG, D, K_POLICY>(args.ap, order_table(args.order.n), item, *reinterpret_cast<AttnSh *>(shared));
    else reject_item<NT >= 2 ? 8 : 4, false>(args.rp, args.gs.n_stat, item, *reinterpret_cast<RejectShared *>(shared));
}

// The kernel arguments of a launch and its grid.
template <bool HAS_ATTN, bool HAS_REJECT>
dim3 fill_args(StepArgs &args, const AttnParams &ap, const RejectParams &rp, int n_stat, int n_attn, int n_race, const UnitOrder *order)
{
    args.ap = ap;
    args.rp = rp;
    args.order.n = 0;
    if (HAS_ATTN && order != nullptr && order->n > 0) {
        args.order.n = order->n;
        memcpy(args.order.request, order->request, sizeof(uint16_t) * (size_t)order->n);
    }
    GridSplit &gs = args.gs;
    gs.n_stat = n_stat;
    gs.n_reject = n_stat + n_race;
    gs.n_attn = n_attn;
    gs.attn_first = (n_attn <= ap.attn_first_limit) ? 1 : 0;
    const int n_reject = n_stat + n_race;
    // The rejection items are a chain of dependent stages that takes some 15 us whatever its size.
    // Beside an attention half that streams for no longer than that (the planner's estimate), the
    // chain is what the launch waits for: its items go first, ahead of the attention blocks, which
    // lose a few microseconds of dispatch to them.  (Four requests of 512 tokens: 21.2 -> 18.0 us;
    // sixteen with 64/8 heads: 28.3 -> 24.6 us; two of 2048 tokens: 22.4 -> 19.2 us.)
    // (In terms of the mixed order: no attention rows among the rejection rows.)
    const bool reject_first = HAS_ATTN && HAS_REJECT && n_reject <= ap.reject_first_limit;
    if (reject_first) gs.attn_first = 0;
    const bool mixed = HAS_ATTN && HAS_REJECT && !gs.attn_first;
    const int rows_attn_all = (n_attn + kXcds - 1) / kXcds;
    // XCDs 1, 3, 5, 7 of this device stream from memory some 6% slower than XCDs 0, 2, 4, 6 (block
    // traces of equal attention blocks), and a launch ends with its slowest XCD.  When there is at
    // most one attention block per compute unit (all resident from the start, the rejection blocks
    // beside them), the rejection blocks, which slow down the attention block they share a compute
    // unit with, go to the even XCDs only: even positions of a row of 8 blocks; the odd positions
    // of such rows exit at once.  (With more attention blocks it does not pay: measured 1% slower
    // with two per compute unit, 15% slower where the rejection half is a fifth of the step.  Nor where the
    // order table lists the chunks, whose blocks are all about equally long: even / all XCDs, 32/8 heads, ten requests of 500 to 8000
    // tokens, k = 4, V = 32000 38.1 / 33.0 us; 64/8, nine, k = 3, V = 128256 47.8 / 40.4; at best 2% faster.)
    gs.reject_cols = (HAS_ATTN && HAS_REJECT && ap.reject_even_xcds && !ap.spread && n_attn <= ap.reject_even_limit && !reject_first) ? kXcds / 2 : kXcds;
    const int rows_reject = (n_reject + gs.reject_cols - 1) / gs.reject_cols;
    gs.rows_attn_mixed = reject_first ? 0 : attention_rows_mixed(rows_attn_all, rows_reject, ap.reject_span);
    return dim3(mixed ? (rows_attn_all + rows_reject) * kXcds
                          : (HAS_ATTN && HAS_REJECT ? (rows_attn_all + rows_reject) * kXcds : n_reject + n_attn));
}

// (with events the extended launch attaches them to the kernel's own begin and end)
template <typename Kernel>
hipError_t launch_kernel(Kernel kernel, dim3 grid, const StepArgs &args, LaunchEvents ev, hipStream_t stream)
{
    if (ev.start != nullptr) hipExtLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, ev.start, ev.stop, 0, args);
    else hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, args);
    return hipGetLastError();
}

template <int NT, int WG, bool HAS_ATTN, bool HAS_REJECT>
hipError_t launch(const AttnParams &ap, const RejectParams &rp, int n_stat, int n_attn, int n_race,
                  const UnitOrder *order, LaunchEvents ev, hipStream_t stream)
{
    StepArgs args;
    const dim3 grid = fill_args<HAS_ATTN, HAS_REJECT>(args, ap, rp, n_stat, n_attn, n_race, order);
    auto go = [&](auto var) {
        return launch_kernel(spec_step_kernel<NT, WG, HAS_ATTN, HAS_REJECT, decltype(var)::value>, grid, args, ev, stream);
    };
    if constexpr (HAS_ATTN && !HAS_REJECT && WG <= 2 && NT >= 2)
        if (ap.k_direct && ap.kv_layout == SPEC_KV_TOKEN_MAJOR && ap.d == kD)
            return launch_kernel(attn_k_direct_kernel<NT, WG>, grid, args, ev, stream);
    if constexpr (HAS_ATTN) {
        if (ap.kv_layout == SPEC_KV_TOKEN_MAJOR)
            return ap.d == 64 ? go(std::integral_constant<int, 4>()) : go(std::integral_constant<int, 2>());
        if (ap.d == 64) return go(std::integral_constant<int, 3>());
        // (the single-bf16 experiment exists for one wave group only)
        if constexpr (WG == 1)
            if (!ap.split_p) return go(std::integral_constant<int, 1>());
    }
    return go(std::integral_constant<int, 0>());
}

template <int NT, int WG>
hipError_t launch_f32(const AttnParams &ap, const RejectParams &rp, int n_stat, int n_attn, int n_race, const UnitOrder *order,
                      LaunchEvents ev, hipStream_t stream)
{
    StepArgs args;
    const dim3 grid = fill_args<true, true>(args, ap, rp, n_stat, n_attn, n_race, order);
    // 64 dims, one wave group: K takes the streaming hint beside a race and more rejection blocks than the chip has slots, whose logits, part
    // of them read twice, then pass through the caches for most of the launch, and contexts that do not outlast them.  Without
    // / with it, steps in us: 16/16 heads, 243 requests of 10 to 199 tokens, k = 7, V = 16032 84.5 / 80.5, 173 of 60 to 113, k = 7 47.4 / 44.7,
    // 189 of 517, k = 2 147.8 / 146.0; 32/8, 164 of 212 to 395, k = 3 73.9 / 70.1, 97 of 662 to 1229, k = 4 109.4 / 107.9; longer ones, 73 of 1026 to
    // 1907, k = 6 154.1 / 163.9; fewer rejection blocks, 20 of 475 to 882, k = 0 24.3 / 28.4, 77 of 98 to 1863, k = 6 116.2 / 126.1.  Worst
    // for it, 148 of 57, k = 5, point-mass draft 43.5 / 44.4.  (128 dims: over 74 steps with more than 800 rejection blocks without it takes 0.86
    // to 1.05 of the time with it, 0.98 in the mean: 55 of 44 to 853 on 32/8 heads, k = 8 90.3 / 104.1, 57 of 233 on 64/8, k = 6 84.0 / 80.3, 133 of 6
    // to 127, k = 1 58.0 / 56.5; neither sizes nor blocks tell them apart.)
    if constexpr (WG == 1)
        if (ap.d == 64 && rp.race_segments > 0 && args.gs.n_reject > 4 * ap.reject_even_limit && ap.capacity_tokens <= 1536)
            return launch_kernel(f32_step_kernel<NT, WG, 64, kStreamPolicy>, grid, args, ev, stream);
    if (ap.d == 64) return launch_kernel(f32_step_kernel<NT, WG, 64>, grid, args, ev, stream);
    return launch_kernel(f32_step_kernel<NT, WG, 128>, grid, args, ev, stream);
}

}  // namespace

// The kernel variants of this file take over a minute to compile in one piece, so the build
// compiles the file several times, each time with SPEC_STEP_PART set to the part whose
// launchers it should hold (everything else of the file is shared, file-local code):
//   0: the dispatcher below, the rejection-only kernel, one row tile    1: two row tiles
//   2: three row tiles    3: two wave groups    4: four wave groups    5: fp32 (step_f32.hip)    (unset: all of it)
#ifndef SPEC_STEP_PART
#define SPEC_STEP_PART -1
#endif
#define SPEC_STEP_HAS_PART(k) (SPEC_STEP_PART < 0 || SPEC_STEP_PART == (k))

// launchers of the (row tiles, wave groups) variants, one function each
#define SPEC_STEP_LAUNCHER(NAME) \
    hipError_t NAME(const AttnParams &ap, const RejectParams &rp, bool with_reject, int n_stat, int n_attn, int n_race, \
                    const UnitOrder *order, LaunchEvents ev, hipStream_t stream)
SPEC_STEP_LAUNCHER(launch_step_tiles1);
SPEC_STEP_LAUNCHER(launch_step_tiles2);
SPEC_STEP_LAUNCHER(launch_step_tiles3);
SPEC_STEP_LAUNCHER(launch_step_tiles2_groups2);
SPEC_STEP_LAUNCHER(launch_step_tiles3_groups2);
SPEC_STEP_LAUNCHER(launch_step_tiles2_groups4);
SPEC_STEP_LAUNCHER(launch_step_tiles3_groups4);
SPEC_STEP_LAUNCHER(launch_step_f32);
#define SPEC_STEP_DEFINE(NAME, NT_, WG_)                                                                     \
    SPEC_STEP_LAUNCHER(NAME)                                                                                 \
    {                                                                                                        \
        return with_reject ? launch<NT_, WG_, true, true>(ap, rp, n_stat, n_attn, n_race, order, ev, stream) \
                           : launch<NT_, WG_, true, false>(ap, rp, 0, n_attn, 0, order, ev, stream);         \
    }
#if SPEC_STEP_HAS_PART(0)
SPEC_STEP_DEFINE(launch_step_tiles1, 1, 1)
#endif
#if SPEC_STEP_HAS_PART(1)
SPEC_STEP_DEFINE(launch_step_tiles2, 2, 1)
#endif
#if SPEC_STEP_HAS_PART(2)
SPEC_STEP_DEFINE(launch_step_tiles3, 3, 1)
#endif
#if SPEC_STEP_HAS_PART(3)
SPEC_STEP_DEFINE(launch_step_tiles2_groups2, 2, 2)
SPEC_STEP_DEFINE(launch_step_tiles3_groups2, 3, 2)
#endif
#if SPEC_STEP_HAS_PART(4)
SPEC_STEP_DEFINE(launch_step_tiles2_groups4, 2, 4)
SPEC_STEP_DEFINE(launch_step_tiles3_groups4, 3, 4)
#endif
#undef SPEC_STEP_DEFINE
#if SPEC_STEP_HAS_PART(5)
SPEC_STEP_LAUNCHER(launch_step_f32)
{
    (void)with_reject;
    switch (ap.row_groups * 10 + ap.row_tiles) {
        case 11: return launch_f32<1, 1>(ap, rp, n_stat, n_attn, n_race, order, ev, stream);
        case 12: return launch_f32<2, 1>(ap, rp, n_stat, n_attn, n_race, order, ev, stream);
        case 22: return launch_f32<2, 2>(ap, rp, n_stat, n_attn, n_race, order, ev, stream);
        case 42: return launch_f32<2, 4>(ap, rp, n_stat, n_attn, n_race, order, ev, stream);
        default: return launch_f32<3, 4>(ap, rp, n_stat, n_attn, n_race, order, ev, stream);
    }
}
#endif
#undef SPEC_STEP_LAUNCHER

#if SPEC_STEP_HAS_PART(0)
int step_attn_items(const AttnParams &ap)
{
    return attn_row_items(ap) * (ap.spread ? 1 : ap.max_chunks);
}

hipError_t launch_step_fused(const AttnParams *attn, const RejectParams *reject, const UnitOrder *order,
                             LaunchEvents ev, hipStream_t stream)
{
    AttnParams ap = {};
    RejectParams rp = {};
    int n_stat = 0, n_attn = 0, n_race = 0;
    if (reject != nullptr) {
        rp = *reject;
        if (rp.stat_segments > kMaxStatSegments || rp.race_segments > kWave || rp.spin_limit < 1 ||
            rp.final_shift < 0 || rp.final_shift > kMaxFinalShift || (rp.stat_segments << rp.final_shift) > kMaxStatSegments)
            return hipErrorInvalidValue;
        // early stop: a form that the kernel has, and one draft length unless each block finds its row from the lengths
        const bool can_peek = attn != nullptr && !attn->f32;
        if (rp.early_stop != kReadAll &&
            ((rp.early_stop == kStopPeek ? !can_peek : rp.early_stop != kStopWait) ||
             (rp.uniform_k >= 0 ? rp.T != rp.B * (rp.uniform_k + 1) : rp.early_stop != kStopPeek || rp.B > kMaxOwnLengths)))
            return hipErrorInvalidValue;
        if (rp.mode == SPEC_ACCEPT_GREEDY) rp.race_segments = 0;   // no race stage
        n_stat = (rp.mode == SPEC_ACCEPT_SAMPLE ? 2 * rp.T - rp.B : rp.T) * rp.stat_segments;
        n_race = rp.B * rp.race_segments + final_items(rp);   // race segments, then the final items
    }
    if (attn != nullptr) {
        ap = *attn;
        const int row_tiles = ap.row_tiles;
        // tiles per wave group and wave groups per block that the kernel is built for
        const bool shape_ok = ap.f32 ? (ap.row_groups == 1 && (row_tiles == 1 || row_tiles == 2)) ||
                                           ((ap.row_groups == 2 || ap.row_groups == 4) && row_tiles == 2) || (ap.row_groups == 4 && row_tiles == 3)
                                     : (ap.row_groups == 1 && row_tiles >= 1 && row_tiles <= 3) ||
                              ((ap.row_groups == 2 || ap.row_groups == 4) && (row_tiles == 2 || row_tiles == 3));
        // (a wavefront keeps the block-table entries of its pages one per lane)
        const bool dim_ok = ap.d == kD || ap.d == 64;
        if (!dim_ok || !shape_ok || ap.chunk_tokens > 4096 / ap.row_groups || ap.chunk_tokens % SPEC_BLOCK_SIZE != 0 ||
            ap.capacity_tokens > ap.chunk_tokens * ap.max_chunks ||
            (ap.f32 && ap.kv_layout != SPEC_KV_TOKEN_MAJOR) || (ap.fused_combine && ap.max_chunks > kMaxFusedChunks) || (order != nullptr && order->n != 0 && order->n != ap.ranks))
            return hipErrorInvalidValue;
        // listed chunks: a table with all of them, whole rows of blocks, and a merge inside the launch
        if (ap.spread ? (order == nullptr || order->n != ap.ranks || ap.B > kMaxListedRequests || ap.max_chunks > kMaxListedChunks || ap.Hkv % kXcds != 0 || !ap.fused_combine)
                      : ap.ranks != ap.B)
            return hipErrorInvalidValue;
        n_attn = step_attn_items(ap);
    }
    if (attn == nullptr) return launch<1, 1, false, true>(ap, rp, n_stat, 0, n_race, nullptr, ev, stream);
    const bool with_reject = reject != nullptr;
    if (ap.f32) return launch_step_f32(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
    switch (ap.row_groups * 10 + ap.row_tiles) {
        case 11: return launch_step_tiles1(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
        case 12: return launch_step_tiles2(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
        case 13: return launch_step_tiles3(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
        case 22: return launch_step_tiles2_groups2(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
        case 23: return launch_step_tiles3_groups2(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
        case 42: return launch_step_tiles2_groups4(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
        default: return launch_step_tiles3_groups4(ap, rp, with_reject, n_stat, n_attn, n_race, order, ev, stream);
    }
}
#endif   // part 0

}  // namespace specv
