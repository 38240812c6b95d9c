// C ABI of the speculative-verification library: host-side validation, launch
// planning and the exported entry points declared in spec_verify.h.
//
// A call costs the host: scalar checks of the argument structs, one hash over the host
// copies of the lengths, a look-up of the launch plan under that hash (the per-request
// checks, the split of the KV length, the order table and the grid layout are computed when a
// shape is seen for the first time), and the launch.  The tuning switches are read from the
// environment once.
#include "common.h"

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

// ---------------------------------------------------------------------------
// Scratch memory for callers that cannot allocate (spec_verify_step_static): one file-scope
// device array per GPU, held until the process ends.  In host code the array's name is only
// a stand-in for the symbol; its device address is resolved once per device, with that device
// current, and kept.  Each GPU has its own copy of the array at its own address.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[SPEC_STATIC_SCRATCH_BYTES];

namespace specv {

namespace {

constexpr size_t kAlign = 256;

constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_ptr[kMaxDevices];

void *static_scratch_of_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    void *ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        // (two threads may both resolve it: they get the same address)
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return nullptr;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
    return ptr;
}

// ---------------------------------------------------------------------------
// Optional per-kernel timing with HIP events (spec_profile_begin / spec_profile_end).
// Off by default; when on, every kernel launch is bracketed by two event records on
// the launch stream.  Not thread safe; meant for the benchmark.
// ---------------------------------------------------------------------------
struct KernelProfiler {
    bool on = false;
    std::vector<hipEvent_t> events;   // pairs: start, stop
    std::vector<int> kernel_of_pair;
    size_t capacity_pairs = 0;
};
KernelProfiler g_prof;

template <typename F>
hipError_t timed(int kernel_id, hipStream_t stream, F launch)
{
    const bool rec = g_prof.on && g_prof.kernel_of_pair.size() < g_prof.capacity_pairs;
    size_t pair = 0;
    if (rec) {
        pair = g_prof.kernel_of_pair.size();
        g_prof.kernel_of_pair.push_back(kernel_id);
        (void)hipEventRecord(g_prof.events[2 * pair], stream);
    }
    const hipError_t err = launch();
    if (rec) (void)hipEventRecord(g_prof.events[2 * pair + 1], stream);
    return err;
}
// The same for a launch that can carry its events itself.
template <typename F>
hipError_t timed_launch(int kernel_id, F launch)
{
    LaunchEvents ev = {nullptr, nullptr};
    if (g_prof.on && g_prof.kernel_of_pair.size() < g_prof.capacity_pairs) {
        const size_t pair = g_prof.kernel_of_pair.size();
        g_prof.kernel_of_pair.push_back(kernel_id);
        ev.start = g_prof.events[2 * pair];
        ev.stop = g_prof.events[2 * pair + 1];
    }
    return launch(ev);
}
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// ---------------------------------------------------------------------------
// Tuning switches (environment variables, for sweeps; none is needed in normal use).
// Read once; spec_verify_reload_env re-reads them.
// ---------------------------------------------------------------------------
struct Tuning {
    int force_generic = 0;        // SPEC_VERIFY_FORCE_GENERIC=1: every shape through the generic attention kernels
    long target_blocks = 0;       // SPEC_VERIFY_TARGET_BLOCKS: attention blocks to aim for when splitting requests (0: automatic)
    long chunk = 0;               // SPEC_VERIFY_CHUNK: tokens per chunk, multiple of 16 (0: automatic)
    int race_blocks = 0;          // SPEC_VERIFY_RACE_BLOCKS: race blocks to aim for (0: automatic)
    int early_stop = -1;          // SPEC_VERIFY_EARLY_STOP=0/1/2: all rows read / early stop that waits / that looks only (-1: automatic)
    float reject_span = 0.5f;     // SPEC_VERIFY_REJECT_SPAN: fraction of the attention items among which the rejection items are spread
    long attn_first_limit = -1;   // SPEC_VERIFY_ATTN_FIRST_LIMIT: attention blocks up to which they all precede the rejection blocks (-1: automatic)
    int reject_first_limit = 1024; // SPEC_VERIFY_REJECT_FIRST_LIMIT: rejection blocks up to which they precede the blocks of a short attention half
    int split_p = 1;              // SPEC_VERIFY_SPLIT_P=0: softmax weights as one bf16 instead of high + low parts
    int reject_even = 1;          // SPEC_VERIFY_REJECT_EVEN=0: rejection blocks on all XCDs
    int k_direct = -1;            // SPEC_VERIFY_K_DIRECT=0/1: the attention alone on token-major pages, K through LDS or straight into
                                  // operand order where there is a kernel for it (-1: automatic)
    int f32_scalar = -1;          // SPEC_VERIFY_F32_SCALAR=0/1: fp32 attention alone on the matrix-instruction / scalar kernel (-1: automatic)
    int spin_limit = 1 << 20;     // SPEC_VERIFY_SPIN_LIMIT: polls of a bounded wait (about two seconds at the default)
    uint32_t epoch = 1;           // changes with every reload: part of the plan cache's key
};
Tuning g_tuning;
std::once_flag g_tuning_once;
std::atomic<uint32_t> g_tuning_epoch{1};

void read_tuning()
{
    Tuning t;
    if (const char *e = getenv("SPEC_VERIFY_FORCE_GENERIC")) t.force_generic = e[0] == '1';
    if (const char *e = getenv("SPEC_VERIFY_TARGET_BLOCKS")) {
        const long v = strtol(e, nullptr, 10);
        if (v >= 1 && v <= (1 << 20)) t.target_blocks = v;
    }
    if (const char *e = getenv("SPEC_VERIFY_CHUNK")) {
        const long v = strtol(e, nullptr, 10);
        if (v >= 16 && v <= 4096 && v % SPEC_BLOCK_SIZE == 0) t.chunk = v;
    }
    if (const char *e = getenv("SPEC_VERIFY_RACE_BLOCKS")) {
        const int v = atoi(e);
        if (v >= 1 && v <= 65536) t.race_blocks = v;
    }
    if (const char *e = getenv("SPEC_VERIFY_EARLY_STOP")) t.early_stop = e[0] >= '0' && e[0] <= '2' ? e[0] - '0' : 1;
    if (const char *e = getenv("SPEC_VERIFY_REJECT_SPAN")) {
        const double v = strtod(e, nullptr);
        if (v > 0.0 && v <= 1.0) t.reject_span = (float)v;
    }
    if (const char *e = getenv("SPEC_VERIFY_ATTN_FIRST_LIMIT")) {
        const long v = strtol(e, nullptr, 10);
        if (v >= 0 && v <= (1 << 20)) t.attn_first_limit = v;
    }
    if (const char *e = getenv("SPEC_VERIFY_REJECT_FIRST_LIMIT")) {
        const long v = strtol(e, nullptr, 10);
        if (v >= 0 && v <= (1 << 20)) t.reject_first_limit = (int)v;
    }
    if (const char *e = getenv("SPEC_VERIFY_SPLIT_P")) t.split_p = e[0] != '0';
    if (const char *e = getenv("SPEC_VERIFY_REJECT_EVEN")) t.reject_even = e[0] != '0';
    if (const char *e = getenv("SPEC_VERIFY_K_DIRECT")) t.k_direct = e[0] != '0';
    if (const char *e = getenv("SPEC_VERIFY_F32_SCALAR")) t.f32_scalar = e[0] != '0';
    if (const char *e = getenv("SPEC_VERIFY_SPIN_LIMIT")) {
        const long v = strtol(e, nullptr, 10);
        if (v >= 1 && v <= (1 << 30)) t.spin_limit = (int)v;
    }
    t.epoch = g_tuning_epoch.fetch_add(1) + 1;
    g_tuning = t;
}

const Tuning &tuning()
{
    std::call_once(g_tuning_once, read_tuning);
    return g_tuning;
}

// Number of compute units of the current device (cached per process; one GPU).
int compute_units()
{
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;   // MI355X
        cached = n;
    }
    return cached;
}

// ---------------------------------------------------------------------------
// Validation.  The scalar part runs on every call; the per-request part (one pass over the
// host copies of the lengths) is what a cached plan vouches for.
// ---------------------------------------------------------------------------
spec_status validate_attn_scalars(const spec_attn_args *a)
{
    if (a == nullptr) return SPEC_EINVAL;
    if (a->B < 1 || a->Hq < 1 || a->Hkv < 1 || a->num_blocks < 1 || a->max_blocks_per_req < 1 || a->T < a->B)
        return SPEC_EINVAL;
    if (a->q == nullptr || a->k_cache == nullptr || a->v_cache == nullptr || a->block_table == nullptr ||
        a->kv_len == nullptr || a->cu_q_len == nullptr || a->out == nullptr || a->host_cu_q_len == nullptr)
        return SPEC_EINVAL;
    // (rows and pages move as vectors of up to 32 bytes)
    if (((reinterpret_cast<uintptr_t>(a->q) | reinterpret_cast<uintptr_t>(a->k_cache) | reinterpret_cast<uintptr_t>(a->v_cache) |
          reinterpret_cast<uintptr_t>(a->out)) & 31) != 0)
        return SPEC_EINVAL;
    if (a->max_kv_len < 0 || (a->max_kv_len == 0 && a->host_kv_len == nullptr)) return SPEC_EINVAL;
    if (a->Hq % a->Hkv != 0) return SPEC_EINVAL;
    if (!(a->softmax_scale >= 0.0f) || isinf(a->softmax_scale)) return SPEC_EINVAL;
    if (a->qkv_dtype != SPEC_F32 && a->qkv_dtype != SPEC_BF16) return SPEC_EINVAL;
    if (a->kv_layout != SPEC_KV_TOKEN_MAJOR && a->kv_layout != SPEC_KV_MFMA) return SPEC_EINVAL;
    if (a->validate != 0 && a->validate != 1) return SPEC_EINVAL;
    if (a->host_cu_q_len[0] != 0 || a->host_cu_q_len[a->B] != a->T) return SPEC_EINVAL;
    if (a->max_kv_len > 0 && (a->max_kv_len + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE > a->max_blocks_per_req)
        return SPEC_EINVAL;
    return SPEC_OK;
}

spec_status validate_attn_requests(const spec_attn_args *a)
{
    for (int b = 0; b < a->B; ++b) {
        const int q_len = a->host_cu_q_len[b + 1] - a->host_cu_q_len[b];
        if (q_len < 1 || q_len > SPEC_K_MAX + 1) return SPEC_EINVAL;
        if (a->host_kv_len == nullptr) continue;
        const int len = a->host_kv_len[b];
        if (len < q_len) return SPEC_EINVAL;
        if ((len + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE > a->max_blocks_per_req) return SPEC_EINVAL;
        if (a->max_kv_len > 0 && len > a->max_kv_len) return SPEC_EINVAL;
    }
    return SPEC_OK;
}

spec_status validate_attn_unsupported(const spec_attn_args *a)
{
    if (a->block_size != SPEC_BLOCK_SIZE) return SPEC_EUNSUPPORTED;
    if (a->d != 64 && a->d != 128) return SPEC_EUNSUPPORTED;
    if (a->Hq / a->Hkv > 16) return SPEC_EUNSUPPORTED;
    if (a->kv_layout == SPEC_KV_MFMA && a->qkv_dtype != SPEC_BF16) return SPEC_EUNSUPPORTED;
    if (a->T > 65535 || a->Hq > 65535) return SPEC_EUNSUPPORTED;
    return SPEC_OK;
}

// validate == 1: the host copy of the block table, every entry of a page in use
spec_status validate_attn_table(const spec_attn_args *a)
{
    if (a->validate != 1 || a->host_block_table == nullptr || a->host_kv_len == nullptr) return SPEC_OK;
    for (int b = 0; b < a->B; ++b) {
        const int pages = (a->host_kv_len[b] + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE;
        const int32_t *row = a->host_block_table + (size_t)b * a->max_blocks_per_req;
        for (int i = 0; i < pages; ++i)
            if (row[i] < 0 || row[i] >= a->num_blocks) return SPEC_EINVAL;
    }
    return SPEC_OK;
}

spec_status validate_attn(const spec_attn_args *a)
{
    spec_status st = validate_attn_scalars(a);
    if (st != SPEC_OK) return st;
    st = validate_attn_requests(a);
    if (st != SPEC_OK) return st;
    st = validate_attn_unsupported(a);
    if (st != SPEC_OK) return st;
    return validate_attn_table(a);
}

spec_status validate_reject_scalars(const spec_reject_args *r)
{
    if (r == nullptr) return SPEC_EINVAL;
    if (r->B < 1 || r->V < 1 || r->T < r->B) return SPEC_EINVAL;
    if (r->target_logits == nullptr || r->cu_q_len == nullptr || r->host_cu_q_len == nullptr ||
        r->accepted_len == nullptr || r->next_token == nullptr || r->counters == nullptr)
        return SPEC_EINVAL;
    if (r->accept_mode != SPEC_ACCEPT_SAMPLE && r->accept_mode != SPEC_ACCEPT_GREEDY &&
        r->accept_mode != SPEC_ACCEPT_POINT_DRAFT)
        return SPEC_EINVAL;
    if (r->validate != 0 && r->validate != 1) return SPEC_EINVAL;
    if (r->T > r->B && r->draft_tokens == nullptr) return SPEC_EINVAL;
    if (r->T > r->B && r->accept_mode == SPEC_ACCEPT_SAMPLE && r->draft_logits == nullptr) return SPEC_EINVAL;
    if (r->host_cu_q_len[0] != 0 || r->host_cu_q_len[r->B] != r->T) return SPEC_EINVAL;
    if ((r->new_kv_len != nullptr || r->draft_next_len != nullptr) && r->kv_len == nullptr) return SPEC_EINVAL;
    if ((reinterpret_cast<uintptr_t>(r->target_logits) & 15) != 0 ||
        (r->accept_mode == SPEC_ACCEPT_SAMPLE && (reinterpret_cast<uintptr_t>(r->draft_logits) & 15) != 0) ||
        (reinterpret_cast<uintptr_t>(r->philox_step_device) & 7) != 0)
        return SPEC_EINVAL;
    return SPEC_OK;
}

spec_status validate_reject_requests(const spec_reject_args *r)
{
    for (int b = 0; b < r->B; ++b) {
        const int q_len = r->host_cu_q_len[b + 1] - r->host_cu_q_len[b];
        if (q_len < 1 || q_len > SPEC_K_MAX + 1) return SPEC_EINVAL;
    }
    return SPEC_OK;
}

spec_status validate_reject_unsupported(const spec_reject_args *r)
{
    if (r->V % 4 != 0) return SPEC_EUNSUPPORTED;  // rows are read as 16-byte vectors
    if (r->B > 65535 || 2 * (int64_t)r->T - r->B > 65535) return SPEC_EUNSUPPORTED;
    return SPEC_OK;
}

// validate == 1: the host copy of the draft tokens
spec_status validate_reject_tokens(const spec_reject_args *r)
{
    if (r->validate != 1 || r->host_draft_tokens == nullptr) return SPEC_OK;
    for (int i = 0; i < r->T - r->B; ++i)
        if (r->host_draft_tokens[i] < 0 || r->host_draft_tokens[i] >= r->V) return SPEC_EINVAL;
    return SPEC_OK;
}

spec_status validate_reject(const spec_reject_args *r)
{
    spec_status st = validate_reject_scalars(r);
    if (st != SPEC_OK) return st;
    st = validate_reject_requests(r);
    if (st != SPEC_OK) return st;
    st = validate_reject_unsupported(r);
    if (st != SPEC_OK) return st;
    return validate_reject_tokens(r);
}

// ---------------------------------------------------------------------------
// Planning.
// ---------------------------------------------------------------------------
// The fp32 attention alone of a few short requests on wide query groups: is the scalar kernel (a block per query row and head)
// faster than the matrix-instruction kernel, whose few blocks walk their pages one after the other?  Both
// modelled from measurements, in us (matrix / scalar; 64/4 heads of 128, k = 4, tokens of each request: one request, 16
// 10.0 / 5.8, 48 14.6 / 8.2, 128 26.5 / 15.6, 256 45.9 / 27.0, 700 53.2 / 46.5; four 128 27.2 / 30.0; 16/1 heads, k = 8, eight
// requests, 128 45.1 / 32.0; 32/8 heads, k = 4, one request, 16 9.3 / 5.8, 128 12.9 / 15.7): of 1824 calls the rule takes
// 196, all of them 1.08 to 3 times as fast, 1.5 at the median, and leaves 20 that would be 1.2 times as fast or more.
bool f32_scalar_is_faster(const AttnPlan &pl, int d, int max_len, int64_t rows)
{
    if (pl.row_tiles < 2) return false;
    const bool wide = d == 128;
    const int pages = (std::min(max_len, pl.chunk_tokens) + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE;
    const int per_wave = (pages * pl.row_groups + 3) / 4;
    const double matrix_us = (4.0 + 1.2 * pl.row_tiles + 0.5 * (pl.row_groups - 1)) * (wide ? 1.0 : 0.8) +
                             per_wave * (0.4 + 1.25 * pl.row_tiles) * (wide ? 1.0 : 0.57) * (pl.row_groups > 1 && pl.row_tiles == 2 ? 0.9 : 1.0) +
                             (pl.max_chunks > 1 ? 3.0 : 0.0);
    const double blocks = rows * std::max(1.0, max_len / 256.0);
    const double load = blocks > 900.0 ? blocks / 450.0 : 1.0 + std::max(0.0, blocks - (max_len <= 64 ? 512.0 : 192.0)) / 900.0;
    const int keys = std::min(max_len, 256);
    const double scalar_us = (wide ? 4.6 + 0.087 * keys : 4.0 + 0.0445 * keys) * load + (max_len > 256 ? 3.0 : 0.0);
    return scalar_us <= 0.95 * matrix_us;
}

// Split of the KV length.  The matrix-instruction kernel runs one block per (request, KV head,
// chunk); the chunk is sized so that the launch has about one block per compute unit
// (two with three row tiles), in multiples of the 16 tokens of a page.  The longest length the
// plan allows for is the caller's bucket (max_kv_len) or, without one, the longest host length.
// (alone: no rejection half in the same call)
// (spread: the chunks may be sized from all lengths, see below, for this share of the blocks aimed for; 0: they may not, which needs
// the smaller workspace)
AttnPlan plan_attn(const spec_attn_args *a, const Tuning &tu, bool alone, double spread)
{
    AttnPlan pl;
    memset(&pl, 0, sizeof pl);
    int max_len = a->max_kv_len, max_q = 0;
    for (int b = 0; b < a->B; ++b) {
        if (a->max_kv_len == 0 && a->host_kv_len[b] > max_len) max_len = a->host_kv_len[b];
        const int q_len = a->host_cu_q_len[b + 1] - a->host_cu_q_len[b];
        if (q_len > max_q) max_q = q_len;
    }
    pl.max_q_len = max_q;
    const int group = a->Hq / a->Hkv;
    const int tiles = (max_q * group + 15) / 16;
    // both types run on matrix-instruction kernels, bf16 in either page layout (token-major pages pass
    // through LDS), fp32 on token-major pages, the only ones it has (a few calls excepted, see f32_scalar_is_faster)
    pl.use_mfma = tu.force_generic ? 0 : 1;
    pl.row_groups = 1;
    pl.row_tiles = tiles;
    if (pl.use_mfma) {
        // A wavefront holds up to three 16-row tiles of query rows in registers.  With up to 48 rows
        // per KV head the block's four wavefronts share the pages between them; with more (long
        // drafts on wide query groups) they form 2 or 4 groups that each own a share of the rows and
        // walk all pages, reading them side by side.
        const bool f32 = a->qkv_dtype == SPEC_F32;   // (twice the registers per tile: two tiles per wavefront)
        pl.row_groups = tiles <= (f32 ? 2 : 3) ? 1 : (tiles <= (f32 ? 4 : 6) ? 2 : 4);
        pl.row_tiles = (tiles + pl.row_groups - 1) / pl.row_groups;
        if (pl.row_groups > 1 && pl.row_tiles < 2) pl.row_tiles = 2;
        // Splitting costs (partials, a merge, more block start-ups), so the longest request is split
        // only as far as needed to give every compute unit a block.  With three row tiles the
        // wavefronts spend a larger share of their time on arithmetic and need a second block beside
        // them to keep loads in flight: then the target is two blocks per compute unit, less an
        // eighth of the slots, which the rejection items flow through while the attention blocks
        // (all resident from the start) stream (with a sixteenth the rejection items of the ragged
        // long-context workload ended after the attention: 90.0 against 88.2 us).
        const long cus = compute_units();
        long target_blocks = pl.row_tiles >= 3 ? 2 * cus - cus / 4 : cus;
        if (tu.target_blocks > 0) target_blocks = tu.target_blocks;
        const int64_t units = (int64_t)a->B * a->Hkv;
        int64_t nsplit = (target_blocks + units - 1) / units;
        if (nsplit < 1) nsplit = 1;
        // Few, short requests are bound by latencies, not by bytes: every further chunk adds block
        // start-ups and partials to merge (eight chunks per pass of the merge), and a chunk of
        // less than a few pages per wavefront does not repay its fixed cost.  So such requests get
        // at most 8 chunks (beyond that only chunks of 1024 tokens or more), of 256 tokens or more.
        // One request with 64/8 heads and 2749 tokens: 29 chunks 24.9 us, 8 chunks 15.8 us; four
        // of 204 tokens: 4 chunks 11.1 us, unsplit 7.9 us; 32/32 heads, 2048 tokens: 8 chunks
        // 13.6 us, 16 chunks 19.3 us, 2 chunks 17.2 us.
        int64_t min_chunk = 64;
        if (tu.target_blocks == 0) {
            // (fp32 takes about twice as long per token: chunks of 512 tokens. Two requests of 8000, 32/8 heads, k = 4:
            // 8 chunks 51.9 us, 16 chunks 38.9 us.)
            const int worth = a->qkv_dtype == SPEC_F32 ? 512 : 1024;
            const int64_t most = std::max<int64_t>(8, (max_len + worth - 1) / worth);
            if (nsplit > most) nsplit = most;
            min_chunk = 256;
        }
        int64_t chunk = (max_len + nsplit - 1) / nsplit;
        chunk = (chunk + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE * SPEC_BLOCK_SIZE;
        if (chunk < min_chunk) chunk = min_chunk;
        // a wavefront holds its pages' block-table entries one per lane, and takes every
        // (4 / row_groups)-th page of the chunk
        const int64_t chunk_cap = 4096 / pl.row_groups;
        if (chunk > chunk_cap) chunk = chunk_cap;
        if (tu.chunk > 0 && tu.chunk <= chunk_cap) chunk = tu.chunk;
        // Chunks sized from all lengths: the split above is the longest request's, and the shorter ones leave compute units
        // without a block, whose share the others' chunks could have.  So the chunk becomes the shortest with which the blocks
        // that have work are no more than aimed for, and the grid lists those only (empty blocks behind them, which the order of the
        // grid's halves then counts: three requests of 8000 and thirteen of 1000 tokens 34.6 -> 39.9 us, two of 16000 and fourteen
        // of 500 39.8 -> 42.5; steps, 32/8 heads, k = 3, V = 32000).  Before / after, in us, 32/8 heads, k = 3,
        // bf16: attention alone, eight requests of 500 to 8000 tokens (chunks of 1568 / 1040) 27.5 / 26.4, sixteen (3792 / 2992)
        // 59.3 / 55.9; their steps (V = 32000) 30.6 / 27.9 and 62.4 / 58.1.  Where that shortens the chunk by a fifth at least (3680 /
        // 3360 68.7 / 70.3, 2608 / 2240 40.2 / 40.3, 3392 / 3232 33.6 / 33.9), and not below 512 tokens (480 / 320: 13.9 / 13.8, 64/8
        // heads 16.0 / 16.3); not with three row tiles, which aim for two blocks per unit (a long-context step, k = 8: 71.2 / 73.9).
        // fp32 with two row tiles or more takes 3 us per page and wavefront, against which a merge of up to six chunks is cheap:
        // chunks of 128 tokens, or 192 where that makes more than six, unless they fill the chip (32/8 heads, k = 4, chunks of 256 /
        // 128: one request of 500 tokens 21.3 / 17.2 us, four 22.3 / 19.3; 256 / 192 / 128: four of 1000 24.3 / 21.4 / 24.0; 224 / 160,
        // eight of 640 22.7 / 23.6; one tile, k = 2, one of 250: 10.9 / 11.7).  Sixteen of 64 to 1000: 32.3 / 28.9.
        if (spread > 0.0 && tu.chunk == 0 && tu.target_blocks == 0 && a->max_kv_len == 0 && a->B <= kMaxListedRequests && a->Hkv % kXcdCount == 0 && units <= target_blocks &&
            (f32 || pl.row_tiles < 3)) {
            const int64_t least = !f32 ? 512 : (tiles >= 2 ? (max_len <= 768 ? 128 : 192) : 256);
            const int worth = f32 ? 512 : 1024;
            const int64_t most = std::max<int64_t>(8, (max_len + worth - 1) / worth);
            int64_t lo = (std::max(least, (max_len + most - 1) / most) + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE, hi = chunk / SPEC_BLOCK_SIZE;   // in pages
            while (lo < hi) {
                const int64_t mid = (lo + hi) / 2;
                int64_t blocks = 0;
                for (int b = 0; b < a->B; ++b) blocks += (a->host_kv_len[b] + mid * SPEC_BLOCK_SIZE - 1) / (mid * SPEC_BLOCK_SIZE);
                if (blocks * a->Hkv <= target_blocks * spread) hi = mid;
                else lo = mid + 1;
            }
            int64_t blocks = 0;
            for (int b = 0; b < a->B; ++b) blocks += (a->host_kv_len[b] + hi * SPEC_BLOCK_SIZE - 1) / (hi * SPEC_BLOCK_SIZE);
            const bool full = f32 && hi * SPEC_BLOCK_SIZE < 256 && blocks * a->Hkv > target_blocks * 4 / 5;
            if (hi * SPEC_BLOCK_SIZE <= chunk * 4 / 5 && !full && max_len <= hi * SPEC_BLOCK_SIZE * kMaxListedChunks) {
                chunk = hi * SPEC_BLOCK_SIZE;
                pl.spread = 1;
            }
        }
        pl.chunk_tokens = (int32_t)chunk;
        pl.max_chunks = (max_len + pl.chunk_tokens - 1) / pl.chunk_tokens;
        if (f32 && alone && (tu.f32_scalar >= 0 ? tu.f32_scalar != 0 : f32_scalar_is_faster(pl, a->d, max_len, (int64_t)a->T * a->Hq))) {
            pl.use_mfma = 0;
            pl.row_groups = 1;
            pl.row_tiles = tiles;
            pl.spread = 0;
        }
    }
    if (!pl.use_mfma) {
        pl.chunk_tokens = 256;  // one key per thread of the generic kernel
        pl.max_chunks = (max_len + pl.chunk_tokens - 1) / pl.chunk_tokens;
    }
    // Token-major pages of a head dim of 128, the attention alone, two or three row tiles per wavefront: K straight into
    // operand order where the launch waits for the chain from a page's arrival to its scores rather than for memory.
    // One wave group, unsplit, through LDS / direct in us (64/8 heads, k = 3; tokens of each request):
    //   more than two blocks per compute unit, about equal lengths, which do not all start at once, so that the last ones run thinly
    // spread: 768 blocks of 100 tokens 18.4 / 17.9, 250 27.8 / 26.1, 600 (memory) 50.0 / 51.6; 1024 of 250 32.2 / 29.9, 600 59.0 / 60.0; 1536 of
    // 100 30.3 / 28.3; 32/8 heads, k = 8, 768 of 250 30.8 / 28.5; lengths of a tenth to twice the mean 1 to 3% slower from 768 blocks on.
    //   one or two per unit, 400 to 700 tokens in the mean (below that the launch is start-up, above it memory): 512 of 600 30.3 / 29.4, of
    // 50 to 950 30.7 / 28.8, 384 of 600 25.1 / 24.5, 256 of 50 to 950 20.9 / 20.1; 512 of 250 16.5 / 16.3, of 1400 60.4 / 62.0.
    // Two wave groups: at most a block per compute unit, with 256 tokens or fewer.  Staged / direct, two row tiles (both in pairs of
    // pages): 64/8 heads, k = 7, 32 requests of 16 / 90 to 128 / 200 to 256 tokens 8.0 / 7.8, 10.45 / 9.7, 13.5 / 12.5 us; 64/4 heads,
    // k = 3, one of 256 10.9 / 10.6, eight of 500 to 2000 in chunks of 256 25.0 / 24.2.  More blocks: 48 requests on 64/8
    // heads, 90 to 128 tokens 13.6 / 14.8, 64 of 150 to 200 18.4 / 20.6; chunks of more tokens, 32 of 500 to 2000 46.0 / 47.4.  Three tiles:
    // 64/8 heads, four requests of 16 / 100 / 200 tokens direct 5, 4 and 6% faster; 64 requests of 100 / 200 tokens 0 and 6% slower.
    const int d_units = a->B * a->Hkv;
    pl.k_direct = 0;
    if (a->qkv_dtype == SPEC_BF16 && a->kv_layout == SPEC_KV_TOKEN_MAJOR && a->d == 128 && pl.use_mfma && pl.row_tiles >= 2) {
        const int cus = compute_units();
        if (pl.row_groups == 2) {
            pl.k_direct = pl.chunk_tokens <= 256 && (int64_t)d_units * pl.max_chunks <= cus;
        } else if (pl.row_groups == 1 && pl.max_chunks == 1 && a->host_kv_len != nullptr && d_units >= cus) {
            int64_t sum = 0;
            int longest = 0;
            for (int b = 0; b < a->B; ++b) {
                sum += a->host_kv_len[b];
                longest = std::max(longest, a->host_kv_len[b]);
            }
            const double mean = (double)sum / a->B;
            if (d_units > 2 * cus) pl.k_direct = mean >= 96.0 && mean <= (d_units > 4 * cus ? 512.0 : 320.0) && longest <= 1.35 * mean;
            else pl.k_direct = mean >= 400.0 && mean <= 700.0;
        }
        if (tu.k_direct >= 0) pl.k_direct = pl.row_groups <= 2 && tu.k_direct;
    }
    pl.capacity_tokens = pl.chunk_tokens * pl.max_chunks;
    pl.fused_combine = (pl.use_mfma && pl.max_chunks <= kMaxFusedChunks) ? 1 : 0;
    // (a request that is not split writes its output directly: the matrix kernel needs no partial
    // slots when no request can have a second chunk)
    // fp32 has room for the scalar kernels' chunks of 256 tokens: the workspace of a step, or of another batch, serves the calls they take
    const bool f32_type = a->qkv_dtype == SPEC_F32;
    const int slot_chunks = f32_type ? std::max(pl.max_chunks, (max_len + 255) / 256) : pl.max_chunks;
    const size_t slots = (pl.use_mfma && pl.max_chunks == 1 && !f32_type) ? 0 : (size_t)a->T * a->Hq * slot_chunks;
    pl.acc_bytes = align_up(slots * a->d * sizeof(float));
    pl.ml_bytes = align_up(slots * 2 * sizeof(float));
    pl.ticket_bytes = align_up((size_t)a->B * a->Hkv * sizeof(unsigned long long));
    pl.total_bytes = pl.acc_bytes + pl.ml_bytes + pl.ticket_bytes;
    pl.blocks = (int64_t)a->B * a->Hkv * pl.max_chunks;
    if (pl.spread) {
        pl.blocks = 0;
        for (int b = 0; b < a->B; ++b) pl.blocks += (int64_t)a->Hkv * ((a->host_kv_len[b] + pl.chunk_tokens - 1) / pl.chunk_tokens);
    }
    return pl;
}

// Rough duration of the attention half in microseconds (the KV bytes at 5.5 TB/s: what it takes
// when it streams well); from the host lengths, or from the bucket bound where there are none.
double attn_estimate_us(const spec_attn_args *a)
{
    double tokens = 0.0;
    for (int b = 0; b < a->B; ++b) tokens += a->host_kv_len != nullptr ? (double)a->host_kv_len[b] : 0.75 * a->max_kv_len;
    return tokens * 2.0 * a->Hkv * a->d * (a->qkv_dtype == SPEC_BF16 ? 2 : 4) / 5.5e6;
}

// attn_us: rough duration of the attention half that runs in the same launch (microseconds), or
// negative if the rejection half runs alone; attn_blocks: its blocks.  few_records: alone, but with no more statistics and race blocks than beside
// an attention half (at most two per compute unit), for a workspace that has no room for more.
RejectPlan plan_reject(const spec_reject_args *r, const Tuning &tu, double attn_us = -1.0, int64_t attn_blocks = 0, bool few_records = false,
                       bool peek = true)
{
    RejectPlan pl;
    memset(&pl, 0, sizeof pl);
    // logit rows that get a statistics pass: the draft rows only when there is a draft distribution
    const int rows = r->accept_mode == SPEC_ACCEPT_SAMPLE ? 2 * r->T - r->B : r->T;
    // statistics: segments of >= 8192 logits, at most 32 per row; about 4 blocks per compute unit (what one holds) when the
    // rejection half runs alone (with fewer, some units get two rows and others one: 48
    // requests, V = 128256, 256 / 1024 / 2048 blocks on 256 units 50.7 / 48.2 / 49.5 us, 16 of them at k = 4 29.1 / 26.7 / 29.2),
    // about one beside an attention half
    const int cus = compute_units();
    const bool many = attn_us < 0.0 && !few_records;
    int segs = ((many ? 4 * cus : cus) + rows - 1) / rows;
    const int max_by_len = (r->V + 8191) / 8192;
    if (segs > max_by_len) segs = max_by_len;
    if (segs > 32) segs = 32;
    if (segs < 1) segs = 1;
    int seg_len = (r->V + segs - 1) / segs;
    seg_len = (seg_len + 3) / 4 * 4;
    pl.stat_seg_len = seg_len;
    pl.stat_segments = (r->V + seg_len - 1) / seg_len;
    // (how long the launch streams when an attention half runs beside: KV and logit bytes at 5.5 TB/s)
    const double logits_us = (double)rows * r->V * 4.0 / 5.5e6;
    // race: segments of >= 2048 vocabulary ids, at most 64 per request; about 4 blocks per compute unit when the
    // rejection half runs alone (256 / 512 / 1024 / 1536 blocks on 256 units 59.3 / 53.8 /
    // 51.4 / 52.4 us for 256 requests, k = 2, V = 32000).  Beside an attention half, where every block
    // holds a slot of the attention's while it waits, about one (256 / 512 / 1024 blocks: 154.2 / 155.9 / 160.6 us for the
    // step of those requests on 64/8 heads, 119.5 / 122.2 / 130.6 us for 96 of them at k = 7), unless the segments are long
    // and the last request's race ends the launch.  How much of it a segment takes is estimated from a block's share of the
    // memory's rate (12.5 KB per microsecond); 256 / 512 blocks and that share:
    //   Attention blocks mixed with the others (more than two per unit): two race blocks per unit for segments above 16384 ids
    // and 0.18, or, with a vocabulary above 32768, of 16384 and 0.135.  64/8 heads, 400 tokens, k = 1: V = 64128,
    // 128 requests 70.3 / 59.2 us (0.36), 256 132.9 / 117.1 (0.37); V = 128256, 128 requests 118.7 / 89.6 (0.55); V = 32000, 256
    // 91.9 / 94.8 (0.22).  32/32 heads, k = 4: 500 tokens, V = 128256, 32 requests (16384) 81.8 / 71.9 (0.14); 200 tokens,
    // V = 64128, 96 requests 104.1 / 94.0 (0.14); V = 32000, 96 requests (11264) 71.0 / 72.9.
    //   Attention blocks first (up to two per unit), which leave few slots: one and a half per unit for segments above 24576 and
    // 0.18, if there is more than one attention block per unit.  V = 128256, 256 / 384 / 512 blocks: 64/8 heads, 64
    // requests, k = 1, 700 tokens 75.5 / 68.7 / 64.9; k = 4, 150 tokens 89.0 / 81.9 / 92.6; 64/4 heads, k = 4, 150 tokens, 64
    // requests (one attention block per unit) 86.5 / 81.3 / 109; k = 1, 700 tokens, 40 requests 39.0 / 42.9 / 42.9.
    const auto race_split = [&](int blocks, int multiple, int &segments, int &len) {
        int n = std::min({(blocks + r->B - 1) / r->B, (r->V + 2047) / 2048, 64});
        if (n < 1) n = 1;
        len = (int)std::min<int64_t>((((int64_t)r->V + n - 1) / n + multiple - 1) / multiple * multiple, INT32_MAX / 4 * 4);
        segments = (int)(((int64_t)r->V + len - 1) / len);
    };
    // (a block takes 1024 ids at a time)
    race_split(tu.race_blocks > 0 ? tu.race_blocks : (many ? 4 * cus : (few_records ? 2 * cus : cus)), 1024, pl.race_segments, pl.race_seg_len);
    if (tu.race_blocks == 0 && attn_us >= 0.0) {
        const double share = pl.race_seg_len * (r->accept_mode == SPEC_ACCEPT_SAMPLE ? 8.0 : 4.0) / 12500.0 / (attn_us + logits_us);
        if (attn_blocks > 2 * cus) {
            const bool large_v = r->V > 32768;   // (rows whose statistics take long)
            if ((pl.race_seg_len > 16384 && share > 0.18) || (large_v && pl.race_seg_len >= 16384 && share > 0.135))
                race_split(2 * cus, 1024, pl.race_segments, pl.race_seg_len);
        } else if (attn_blocks > cus && pl.race_seg_len > 24576 && share > 0.18) {
            race_split(3 * cus / 2, 1024, pl.race_segments, pl.race_seg_len);
        }
    }
    // requests per item of the final stage: as many as leave 8 items (the kernel says why they are grouped)
    pl.final_shift = 0;
    while (pl.final_shift < kMaxFinalShift && (16 << pl.final_shift) <= r->B && (pl.stat_segments << (pl.final_shift + 1)) <= 32)
        ++pl.final_shift;

    // Early stop: with one draft length for all requests the statistics items can be taken in
    // position order and the rows after a request's first rejection left unread.  That turns the
    // pass into a chain of k+1 dependent stages (then the race), which pays where it stays mostly hidden under the
    // attention's stream, or where the logits it saves are many.  Both are weighed by their streams (KV and logit
    // bytes at 5.5 TB/s) with weights fitted to measurements; the rejection half alone: see below.  Step without / with, in us:
    // 64/8 heads, B=96 k=7 102 / 94, k=3 64 / 64, B=128 L=512 k=4 87 / 80, B=256 k=2 156 / 149; 32/8 heads, B=128
    // L=512 k=2 64 / 61; 32/32 heads, L=1024, B=32 k=2 / 4 / 8 94 / 92, 97 / 95, 103 / 104, B=64 k=4 / 8 181 / 178,
    // 199 / 182.  Not where all attention blocks go first in the grid (two per compute unit or fewer): the chain then starts
    // late in few slots (64/8 heads, B=64, L=1000, k=1 / 2, V=8192: 54 / 57, 57 / 64; k=4, V=32000 67 / 84).  Over 407 steps (32 to 256
    // requests, k = 1 to 8, 150 to 1000 tokens, V = 8192, 32000 and 128256, acceptance rates of 0.5, 0.7 and 0.9) the rule
    // loses 0.4% against the better side on average; worst, at a rate of 0.5, a long chain that it leaves out (B=128 k=8 L=150
    // 92 / 82) and, at 0.9, one that it takes for few logits (V=8192, B=256 k=8 L=150 116 / 127).
    pl.early_stop = kReadAll;
    pl.uniform_k = 0;
    int uniform_q = r->T % r->B == 0 ? r->T / r->B : 0;   // every request's rows, 0: they differ
    for (int b = 0; b < r->B && uniform_q > 0; ++b)
        if (r->host_cu_q_len[b + 1] - r->host_cu_q_len[b] != uniform_q) uniform_q = 0;
    if (r->T > r->B && uniform_q > 0) {
        const int q = uniform_q;
        bool wanted;
        if (tu.early_stop >= 0) {
            wanted = tu.early_stop == 1;
        } else if (attn_us >= 0.0) {
            // a stage: a block reads its segment at its share of the memory's rate (12.5 KB per microsecond), and a hop
            const double chain_us = q * (2.0 + pl.stat_seg_len * 4.0 / 12500.0) + 30.0;
            wanted = r->B >= 32 && attn_blocks > 2 * cus && chain_us <= 0.9 * attn_us + 2.5 * logits_us;
        } else {
            // One stage per position: it streams what is still needed of its rows (at an acceptance rate of 0.7),
            // in 6 us at least, and has a block per compute unit.  Against all rows in one go, in one
            // launch: B=256 V=32000 k=1 / 2 / 7 +3 / -6 / -14%, B=128 k=4 +18%, B=512 V=8192 k=4 +4%; V=128256 B=256
            // k=1 -6%, B=128 k=2 -9%, B=40 k=7 (too few blocks per stage) +22%; greedy V=32000 k=3 B=256 / 512
            // +17 / -12%; the rule takes the better side in each.  (The rate only sizes the stages: over 413 random shapes at
            // rates of 0.5, 0.7 and 0.9 no call became slower with this rule and the split above than it was without both.)
            const int per_position = (r->accept_mode == SPEC_ACCEPT_SAMPLE ? 2 : 1) * r->B;
            double staged = 0.0, all = 0.0, needed = 1.0;
            for (int j = 0; j < q; ++j, needed *= 0.7) {
                const double us = (double)(j < q - 1 ? per_position : r->B) * r->V * 4.0 / 5.5e6;
                all += us;
                staged += std::max(6.0, needed * us);
            }
            wanted = staged <= 0.95 * all && (int64_t)per_position * pl.stat_segments >= compute_units();
        }
        if (wanted) { pl.early_stop = kStopWait; pl.uniform_k = q - 1; }
    }
    // The same without waiting, beside an attention half: a block looks at what its request's earlier positions have published
    // and skips its row if that shows a rejection.  Nothing waits for a chain of stages, so long drafts and draft lengths of
    // their own (up to a block's worth of requests) can have it, but the positions that are in flight at the same time do
    // not see each other: about a block per compute unit, or that many positions' worth of rows.  What is saved beyond
    // those, at an acceptance rate of 0.7, in us of logits at 5.5 TB/s, has to repay a look (3 us of a block's time) per row
    // and races that start later.  All rows read or waiting as chosen above / looking, in us: 64/8 heads, token-major, B=96 k=7 99 / 87,
    // tiles, B=48 k=8 88.4 / 80.9; 32/8 heads, B=86 k=7 L=1326 126 / 112; 64/4 heads, B=65 k=8 L=690 117 / 107; drafts of 1..k: 64/8
    // heads, B=200 k=3 93.7 / 90.0, B=64 k=5 (nothing is saved) 49.9 / 52.8.  Over 70 steps that stop early in either form (24 to
    // 256 requests, k = 2 to 8, V = 16000 to 128256, 60 to 2000 tokens, all modes) the time against all rows read is 0.98 at an acceptance
    // rate of 0.9, 0.94 at 0.7 and 0.90 at 0.45; best 0.78, 0.78 and 0.70; worst 1.15, 1.08 and 1.04 (64/4 heads, B=64 k=7,
    // V=16000, 16 to 97 tokens: the rate is not known here, nor how long a short launch takes to dispatch).  Not where the
    // rejection half runs alone: its blocks fill the chip at once (four per unit) and start together; 120 such calls -7 to +29%.
    // (peek: the kernel that takes the launch can.)
    if (peek && r->T > r->B && (uniform_q > 0 || r->B <= kMaxOwnLengths)) {
        const int sides = r->accept_mode == SPEC_ACCEPT_SAMPLE ? 2 : 1;
        const double in_flight = (double)cus / ((double)sides * r->B * pl.stat_segments);   // positions
        double saved_of_k[SPEC_K_MAX + 1] = {0.0}, before = 0.0;   // rows saved of a request with k draft tokens
        for (int k = 1; k <= SPEC_K_MAX; ++k) {
            const double skipped = 1.0 - pow(0.7, std::max(0.0, k - in_flight));   // ... of position k
            saved_of_k[k] = before + skipped;
            before += sides * skipped;
        }
        double saved_rows = 0.0;
        for (int b = 0; b < r->B; ++b) saved_rows += saved_of_k[r->host_cu_q_len[b + 1] - r->host_cu_q_len[b] - 1];
        const double saved_us = saved_rows * r->V * 4.0 / 5.5e6;
        // (a row's segment has to be worth the look at it, and the search for the item where draft lengths differ: V = 8016, drafts of
        // 1..8, 64/4 heads, B=255 65.8 / 72.3; V = 4736, k = 7, 32/8 heads of 64, B=194 52.8 / 55.2; V = 13792, k = 7, B=123 42.8 / 40.2)
        const bool long_enough = pl.stat_seg_len >= (uniform_q > 0 ? 8192 : 16384);
        if (tu.early_stop >= 0 ? tu.early_stop == 2 : attn_us >= 0.0 && long_enough && saved_us > (pl.early_stop == kStopWait ? 8.0 : 3.0)) {
            pl.early_stop = kStopPeek;
            pl.uniform_k = uniform_q > 0 ? uniform_q - 1 : -1;
        }
    }
    pl.stats_off = 0;
    pl.stats_bytes = align_up((size_t)rows * pl.stat_segments * kStatWords * sizeof(unsigned long long));
    pl.partial_off = pl.stats_off + pl.stats_bytes;
    // (room for the segments of 512 blocks at least, so that what fits the static scratch does not depend on the split)
    int room = 0, room_len = 0;
    race_split(tu.race_blocks > 0 ? tu.race_blocks : 512, 4, room, room_len);
    pl.partial_bytes = align_up(((size_t)r->B * std::max(pl.race_segments, room) * 2 + r->B) * sizeof(unsigned long long));
    pl.total_bytes = pl.stats_bytes + pl.partial_bytes;
    return pl;
}

// Blocks of the rejection half: statistics, race, final stage.
int64_t reject_blocks(const spec_reject_args *r, const RejectPlan &pl)
{
    const int64_t rows = r->accept_mode == SPEC_ACCEPT_SAMPLE ? 2 * (int64_t)r->T - r->B : r->T;
    const int64_t race = r->accept_mode == SPEC_ACCEPT_GREEDY ? 0 : (int64_t)r->B * pl.race_segments;
    return rows * pl.stat_segments + race + ((r->B + (1 << pl.final_shift) - 1) >> pl.final_shift);
}

// The most that the rejection half alone takes with this vocabulary, at this batch or any smaller one (fewer rows get more
// segments each, so the records of one batch alone would not do: an engine sizes its workspace once, for its largest).
size_t reject_room(const spec_reject_args *r, const Tuning &tu)
{
    const size_t rows = (size_t)(r->accept_mode == SPEC_ACCEPT_SAMPLE ? 2 * (int64_t)r->T - r->B : r->T), B = (size_t)r->B;
    const size_t slots = 4 * (size_t)compute_units();
    const size_t stat_most = std::min<size_t>(((size_t)r->V + 8191) / 8192, 32);
    const size_t race_most = std::min<size_t>(((size_t)r->V + 2047) / 2048, 64);
    const size_t race_blocks = tu.race_blocks > 0 ? (size_t)tu.race_blocks : std::max<size_t>(slots, 512);
    const size_t stats = std::min(rows * stat_most, rows + slots - 1);
    const size_t race = std::min(B * race_most, B + race_blocks - 1);
    return align_up(stats * kStatWords * sizeof(unsigned long long)) + align_up((race * 2 + B) * sizeof(unsigned long long));
}

// Requests by falling KV length (stable; from the host copy of kv_len).  The grid takes the
// attention items in this order: blocks that run at the same time then take about
// equally long, which the in-order hardware dispatcher needs to keep its block slots
// filled, and the short items even out the end of the launch.  Any order gives the same
// results, so under a length bucket the table made from the lengths at planning time stays
// valid (lengths that grow by a few tokens per step keep their ranks, more or less).  No table
// (given order) when all lengths are equal, unknown, or there are too many requests.
void make_order(const spec_attn_args *a, UnitOrder &order)
{
    order.n = 0;
    if (a->B > kMaxOrdered || a->host_kv_len == nullptr) return;
    bool equal = true;
    for (int b = 1; b < a->B; ++b)
        if (a->host_kv_len[b] != a->host_kv_len[0]) equal = false;
    if (equal) return;
    std::vector<int> idx(a->B);
    for (int b = 0; b < a->B; ++b) idx[b] = b;
    std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return a->host_kv_len[x] > a->host_kv_len[y]; });
    for (int b = 0; b < a->B; ++b) order.request[b] = (uint16_t)idx[b];
    order.n = a->B;
}

// The chunks that exist, request by request, for a plan whose chunks are sized from all lengths.
void list_chunks(const spec_attn_args *a, const AttnPlan &pl, UnitOrder &list)
{
    list.n = 0;
    for (int b = 0; b < a->B; ++b) {
        const int chunks = (a->host_kv_len[b] + pl.chunk_tokens - 1) / pl.chunk_tokens;
        for (int c = 0; c < chunks; ++c)
            list.request[list.n++] = (uint16_t)(b | c << kListRequestBits | (chunks - 1) << (kListRequestBits + kListChunkBits));
    }
}

// ---------------------------------------------------------------------------
// Plan cache: what one shape needs beyond the scalar checks, keyed by a hash of everything the
// plan depends on.  Per thread, sixteen entries (one per draft length and then some), replaced in turn.
// ---------------------------------------------------------------------------
struct StepPlan {
    uint64_t key = 0;
    bool used = false;
    spec_status status = SPEC_OK;   // of the per-request validation
    bool has_attn = false, has_reject = false;
    AttnPlan apl;
    AttnPlan apl_small;             // for workspaces without room for apl
    RejectPlan rpl;
    RejectPlan rpl_small;           // for workspaces without room for rpl (never larger than rpl)
    UnitOrder order, listed;        // apl's if its chunks are listed, apl_small's (and apl's otherwise)
    size_t workspace_bytes = 0;     // what callers are told: enough for this call, and for its rejection half alone at this batch or a smaller one
    // (for telling a hash collision from a hit)
    int32_t B = 0, T = 0, V = 0;
};

inline uint64_t mix(uint64_t h, uint64_t x)
{
    h ^= x;
    h *= 0x9E3779B97F4A7C15ull;
    return h ^ (h >> 29);
}

uint64_t hash_i32(uint64_t h, const int32_t *v, int n)
{
    int i = 0;
    for (; i + 1 < n; i += 2) h = mix(h, (uint64_t)(uint32_t)v[i] | ((uint64_t)(uint32_t)v[i + 1] << 32));
    if (i < n) h = mix(h, (uint64_t)(uint32_t)v[i]);
    return h;
}

uint64_t plan_key(const spec_attn_args *a, const spec_reject_args *r, const Tuning &tu)
{
    uint64_t h = mix(0x5EC0DEull, tu.epoch);
    if (a != nullptr) {
        h = mix(h, (uint64_t)(uint32_t)a->B | ((uint64_t)(uint32_t)a->Hq << 32));
        h = mix(h, (uint64_t)(uint32_t)a->Hkv | ((uint64_t)(uint32_t)a->d << 32));
        h = mix(h, (uint64_t)(uint32_t)a->T | ((uint64_t)(uint32_t)a->max_blocks_per_req << 32));
        h = mix(h, (uint64_t)(uint32_t)a->qkv_dtype | ((uint64_t)(uint32_t)a->kv_layout << 8) |
                       ((uint64_t)(uint32_t)a->block_size << 16) | ((uint64_t)(uint32_t)a->max_kv_len << 32));
        h = hash_i32(h, a->host_cu_q_len, a->B + 1);
        if (a->host_kv_len != nullptr) h = hash_i32(mix(h, 1), a->host_kv_len, a->B);
    }
    if (r != nullptr) {
        h = mix(h, 0xACCE97ull);
        h = mix(h, (uint64_t)(uint32_t)r->B | ((uint64_t)(uint32_t)r->V << 32));
        h = mix(h, (uint64_t)(uint32_t)r->T | ((uint64_t)(uint32_t)r->accept_mode << 32));
        if (a == nullptr || a->host_cu_q_len != r->host_cu_q_len) h = hash_i32(h, r->host_cu_q_len, r->B + 1);
    }
    return h | 1ull;
}

constexpr int kPlanCacheEntries = 16;
struct PlanCache {
    StepPlan entry[kPlanCacheEntries];
    int next = 0;
};

// The plan of (attn, reject); either may be null.  Scalar validation has passed.
const StepPlan &plan_for(const spec_attn_args *a, const spec_reject_args *r)
{
    thread_local PlanCache cache;
    const Tuning &tu = tuning();
    const uint64_t key = plan_key(a, r, tu);
    for (StepPlan &e : cache.entry)
        if (e.used && e.key == key && e.has_attn == (a != nullptr) && e.has_reject == (r != nullptr) &&
            e.B == (a != nullptr ? a->B : r->B) && e.T == (a != nullptr ? a->T : r->T) && e.V == (r != nullptr ? r->V : 0))
            return e;
    StepPlan &e = cache.entry[cache.next];
    cache.next = (cache.next + 1) % kPlanCacheEntries;
    e.key = key;
    e.used = true;
    e.has_attn = a != nullptr;
    e.has_reject = r != nullptr;
    e.B = a != nullptr ? a->B : r->B;
    e.T = a != nullptr ? a->T : r->T;
    e.V = r != nullptr ? r->V : 0;
    e.order.n = 0;
    e.status = SPEC_OK;
    if (a != nullptr) {
        e.status = validate_attn_requests(a);
        if (e.status == SPEC_OK) e.status = validate_attn_unsupported(a);
    }
    if (e.status == SPEC_OK && r != nullptr) {
        e.status = validate_reject_requests(r);
        if (e.status == SPEC_OK) e.status = validate_reject_unsupported(r);
    }
    if (e.status != SPEC_OK) return e;
    size_t base = 0;
    if (a != nullptr) {
        e.apl = plan_attn(a, tu, r == nullptr, 1.0);
        e.apl_small = plan_attn(a, tu, r == nullptr, 0.0);
        e.apl.short_attn = e.apl_small.short_attn = attn_estimate_us(a) <= 20.0 ? 1 : 0;
        make_order(a, e.order);
    }
    const double attn_us = (a != nullptr && e.apl.use_mfma) ? attn_estimate_us(a) : -1.0;
    const bool peek = attn_us >= 0.0 && a->qkv_dtype == SPEC_BF16;
    if (r != nullptr) {
        e.rpl = plan_reject(r, tu, attn_us, a != nullptr ? e.apl.blocks : 0, false, peek);
        // Rejection blocks that fill the chip and go first in the grid (see fill_args): the attention's get the slots that the statistics
        // leave, and the race's blocks, about one per compute unit, hold theirs to the end.  With a chunk's block for every compute
        // unit the last of them start when the race ends, so the split aims for an eighth less.  256 / 224 blocks, in us: 64/8
        // heads, k = 2, V = 128256, eight requests of 60 to 6000 tokens 41.3 / 36.2; 32/8, k = 1, twelve 33.8 / 28.9; fp32, 64/8, k = 3,
        // V = 32000, twelve of 60 to 3000 58.4 / 45.6.  With fewer rejection blocks (32/8, k = 1, V = 8192, 17 of 60 to 4000 26.6 / 28.4)
        // or a longer attention half (32/8, k = 4, V = 32000, eleven of 200 to 6000 31.7 / 38.2 with fewer) not.
        const int64_t n_reject = reject_blocks(r, e.rpl);
        if (a != nullptr && e.apl.spread && e.apl.short_attn && n_reject >= 2 * compute_units() && n_reject <= tu.reject_first_limit) {
            e.apl = plan_attn(a, tu, false, 0.875);
            e.apl.short_attn = 1;
            e.rpl = plan_reject(r, tu, attn_us, e.apl.blocks, false, peek);
        }
    }
    if (a != nullptr) {
        if (e.apl.spread) list_chunks(a, e.apl, e.listed);
        base = std::max(e.apl.total_bytes, e.apl_small.total_bytes);
    }
    e.workspace_bytes = base;
    if (r != nullptr) {
        e.rpl_small = attn_us < 0.0 ? plan_reject(r, tu, attn_us, a != nullptr ? e.apl.blocks : 0, true, peek) : e.rpl;
        if (e.rpl_small.total_bytes > e.rpl.total_bytes) e.rpl_small = e.rpl;
        e.workspace_bytes = std::max(base + e.rpl.total_bytes, (attn_us < 0.0 ? base : 0) + reject_room(r, tu));
    }
    return e;
}

// The plans on a workspace of `have` bytes.  The blocks of a rejection half that runs alone, and the chunks of requests of
// different lengths, are chosen for speed, and what they leave in the workspace takes more room than it would with few blocks or with
// chunks for the longest request: a workspace that holds only the latter (sized for another batch, say) still serves.
const AttnPlan &attn_plan_for(const StepPlan &plan, size_t have)
{
    const size_t rest = plan.has_reject ? plan.rpl_small.total_bytes : 0;
    return plan.apl.total_bytes + rest <= have ? plan.apl : plan.apl_small;
}
const RejectPlan &reject_plan_for(const StepPlan &plan, size_t have)   // have: after the attention's
{
    return plan.rpl.total_bytes <= have ? plan.rpl : plan.rpl_small;
}

// Tag of a call's tickets (see step_kernel.hip); unique per call within the process, never 0.
uint32_t next_generation()
{
    static std::atomic<uint32_t> counter{0x5EC0u};
    uint32_t g = ++counter;
    if (g == 0) g = ++counter;
    return g;
}

spec_status check_workspace(void *ws, size_t have, size_t need)
{
    if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & (kAlign - 1)) != 0 || have < need) return SPEC_EWORKSPACE;
    return SPEC_OK;
}

AttnParams attn_params(const spec_attn_args *a, const AttnPlan &pl, char *ws, int64_t *errors)
{
    const Tuning &tu = tuning();
    AttnParams p;
    memset(&p, 0, sizeof p);
    p.B = a->B; p.Hq = a->Hq; p.Hkv = a->Hkv; p.d = a->d;
    p.num_blocks = a->num_blocks; p.max_blocks_per_req = a->max_blocks_per_req; p.T = a->T;
    p.kv_layout = a->kv_layout;
    p.chunk_tokens = pl.chunk_tokens; p.max_chunks = pl.max_chunks;
    p.capacity_tokens = pl.capacity_tokens;
    p.row_groups = pl.row_groups;
    p.row_tiles = pl.row_tiles;
    p.k_direct = pl.k_direct;
    p.spread = (int8_t)pl.spread;
    p.ranks = pl.spread ? (int32_t)(pl.blocks / a->Hkv) : a->B;
    p.f32 = a->qkv_dtype == SPEC_F32 ? 1 : 0;
    const double scale = a->softmax_scale > 0.0f ? (double)a->softmax_scale : 1.0 / sqrt((double)a->d);
    p.scale_log2 = (float)(scale * kLog2eD);
    p.q = a->q; p.k_cache = a->k_cache; p.v_cache = a->v_cache;
    p.block_table = a->block_table; p.kv_len = a->kv_len; p.cu_q_len = a->cu_q_len;
    p.out = a->out;
    p.ws_acc = reinterpret_cast<float *>(ws);
    p.ws_ml = reinterpret_cast<float *>(ws + pl.acc_bytes);
    p.tickets = reinterpret_cast<unsigned long long *>(ws + pl.acc_bytes + pl.ml_bytes);
    p.errors = reinterpret_cast<unsigned long long *>(a->error_count != nullptr ? a->error_count : errors);
    p.generation = next_generation();
    p.fused_combine = pl.fused_combine;
    p.split_p = (int16_t)tu.split_p;
    p.reject_span = tu.reject_span;
    // as many attention blocks as there are block slots: all start at once
    p.attn_first_limit = tu.attn_first_limit >= 0 ? (int32_t)tu.attn_first_limit : 2 * compute_units();
    p.reject_even_xcds = tu.reject_even;
    p.reject_even_limit = compute_units();
    p.reject_first_limit = pl.short_attn ? tu.reject_first_limit : 0;
    return p;
}

RejectParams reject_params(const spec_reject_args *r, const RejectPlan &pl, char *ws)
{
    RejectParams p;
    memset(&p, 0, sizeof p);
    p.B = r->B; p.V = r->V; p.T = r->T;
    p.mode = r->accept_mode;
    p.target_logits = r->target_logits; p.draft_logits = r->draft_logits;
    p.draft_tokens = r->draft_tokens; p.cu_q_len = r->cu_q_len;
    p.seed_lo = (uint32_t)(r->philox_seed & 0xFFFFFFFFull);
    p.seed_hi = (uint32_t)(r->philox_seed >> 32);
    p.step_lo = (uint32_t)(r->philox_step & 0xFFFFFFFFull);
    p.step_hi24 = (uint32_t)((r->philox_step >> 32) & 0xFFFFFFull);
    p.step_device = reinterpret_cast<const unsigned long long *>(r->philox_step_device);
    p.accepted_len = r->accepted_len; p.next_token = r->next_token; p.out_tokens = r->out_tokens;
    p.counters = reinterpret_cast<unsigned long long *>(r->counters);
    p.debug_u_ratio = r->debug_u_ratio;
    p.kv_len = r->kv_len; p.new_kv_len = r->new_kv_len; p.draft_next_len = r->draft_next_len;
    p.stat_segments = pl.stat_segments; p.stat_seg_len = pl.stat_seg_len;
    p.race_segments = pl.race_segments; p.race_seg_len = pl.race_seg_len;
    p.early_stop = pl.early_stop; p.uniform_k = pl.uniform_k;
    p.final_shift = pl.final_shift;
    p.spin_limit = tuning().spin_limit;
    {
        // (a launch of at most one rejection block per compute unit counts as small)
        const int64_t rows = r->accept_mode == SPEC_ACCEPT_SAMPLE ? 2 * (int64_t)r->T - r->B : r->T;
        p.short_naps = rows * pl.stat_segments + (int64_t)r->B * pl.race_segments + final_items(p) <= compute_units() ? 1 : 0;
    }
    p.stats = reinterpret_cast<unsigned long long *>(ws + pl.stats_off);
    p.race_partial = reinterpret_cast<unsigned long long *>(ws + pl.partial_off);
    p.race_info = p.race_partial + (size_t)r->B * pl.race_segments * 2;
    p.generation = next_generation();
    return p;
}

spec_status run_attn_generic(const AttnParams &p, int dtype, hipStream_t stream)
{
    hipError_t err = timed(SPEC_KERNEL_ATTN_GENERIC, stream, [&] { return launch_attn_generic(p, dtype, stream); });
    if (err != hipSuccess) return SPEC_EHIP;
    if (p.max_chunks == 1) return SPEC_OK;   // no request is split: every row was written directly
    err = timed(SPEC_KERNEL_ATTN_COMBINE, stream, [&] { return launch_attn_combine(p, stream); });
    return err == hipSuccess ? SPEC_OK : SPEC_EHIP;
}

// Checks shared by the entry points that take both halves; leaves the plan in `plan`.
spec_status prepare_step(const spec_attn_args *attn, const spec_reject_args *reject, const StepPlan *&plan)
{
    spec_status st = validate_attn_scalars(attn);
    if (st != SPEC_OK) return st;
    st = validate_reject_scalars(reject);
    if (st != SPEC_OK) return st;
    if (attn->B != reject->B || attn->T != reject->T) return SPEC_EINVAL;
    plan = &plan_for(attn, reject);
    if (plan->status != SPEC_OK) return plan->status;
    st = validate_attn_table(attn);
    if (st != SPEC_OK) return st;
    return validate_reject_tokens(reject);
}

// The whole step on a given workspace (shared by spec_verify_step and spec_verify_step_static).
spec_status step_on_workspace(const spec_attn_args *attn, const spec_reject_args *reject, const StepPlan &plan,
                              void *workspace, size_t workspace_bytes, void *hip_stream)
{
    const AttnPlan &apl = attn_plan_for(plan, workspace_bytes);
    const RejectPlan &rpl = reject_plan_for(plan, workspace_bytes - std::min(workspace_bytes, apl.total_bytes));
    const spec_status st = check_workspace(workspace, workspace_bytes, apl.total_bytes + rpl.total_bytes);
    if (st != SPEC_OK) return st;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const AttnParams ap = attn_params(attn, apl, static_cast<char *>(workspace), reject->counters + 6);
    const RejectParams rp = reject_params(reject, rpl, static_cast<char *>(workspace) + apl.total_bytes);
    if (apl.use_mfma) {
        // the whole step in one launch
        hipError_t err = timed_launch(SPEC_KERNEL_STEP, [&](LaunchEvents ev) {
            return launch_step_fused(&ap, &rp, apl.spread ? &plan.listed : &plan.order, ev, stream);
        });
        if (err == hipSuccess && !apl.fused_combine && apl.max_chunks > 1)
            err = timed(SPEC_KERNEL_ATTN_COMBINE, stream, [&] { return launch_attn_combine(ap, stream); });
        return err == hipSuccess ? SPEC_OK : SPEC_EHIP;
    }
    const spec_status sa = run_attn_generic(ap, attn->qkv_dtype, stream);
    if (sa != SPEC_OK) return sa;
    const hipError_t err =
        timed_launch(SPEC_KERNEL_REJECT, [&](LaunchEvents ev) { return launch_step_fused(nullptr, &rp, nullptr, ev, stream); });
    return err == hipSuccess ? SPEC_OK : SPEC_EHIP;
}

}  // namespace

}  // namespace specv

using namespace specv;

extern "C" {

spec_status spec_validate_attn(const spec_attn_args *attn) { return validate_attn(attn); }

spec_status spec_validate_reject(const spec_reject_args *reject) { return validate_reject(reject); }

void spec_verify_reload_env(void)
{
    (void)tuning();   // the first read, if it has not happened yet
    read_tuning();
}

size_t spec_verify_workspace_bytes(const spec_attn_args *attn, const spec_reject_args *reject)
{
    if (attn == nullptr && reject == nullptr) return 0;
    if (attn != nullptr && validate_attn_scalars(attn) != SPEC_OK) return 0;
    if (reject != nullptr && validate_reject_scalars(reject) != SPEC_OK) return 0;
    if (attn != nullptr && reject != nullptr && (attn->B != reject->B || attn->T != reject->T)) return 0;
    const StepPlan &plan = plan_for(attn, reject);
    if (plan.status != SPEC_OK) return 0;
    return plan.workspace_bytes;
}

spec_status spec_verify_plan(const spec_attn_args *attn, const spec_reject_args *reject, spec_plan_info *info)
{
    if (info == nullptr || (attn == nullptr && reject == nullptr)) return SPEC_EINVAL;
    memset(info, 0, sizeof *info);
    spec_status st = attn != nullptr ? validate_attn_scalars(attn) : SPEC_OK;
    if (st != SPEC_OK) return st;
    st = reject != nullptr ? validate_reject_scalars(reject) : SPEC_OK;
    if (st != SPEC_OK) return st;
    if (attn != nullptr && reject != nullptr && (attn->B != reject->B || attn->T != reject->T)) return SPEC_EINVAL;
    const StepPlan &plan = plan_for(attn, reject);
    if (plan.status != SPEC_OK) return plan.status;
    if (attn != nullptr) {
        const AttnPlan &pl = plan.apl;
        info->attn_path = pl.use_mfma && attn->qkv_dtype == SPEC_BF16 ? SPEC_PATH_MFMA : SPEC_PATH_GENERIC;
        info->row_tiles = pl.row_tiles;
        info->row_groups = pl.row_groups;
        info->chunk_tokens = pl.chunk_tokens;
        info->max_chunks = pl.max_chunks;
        if (pl.use_mfma) {
            AttnParams ap;
            memset(&ap, 0, sizeof ap);
            ap.Hkv = attn->Hkv; ap.max_chunks = pl.max_chunks; ap.spread = (int8_t)pl.spread;
            ap.ranks = pl.spread ? (int32_t)(pl.blocks / attn->Hkv) : attn->B;
            info->attn_blocks = step_attn_items(ap);
            info->launches = 1 + ((!pl.fused_combine && pl.max_chunks > 1) ? 1 : 0);
        } else {
            info->attn_blocks = pl.max_chunks * attn->Hq * attn->T;
            info->launches = pl.max_chunks > 1 ? 2 : 1;
        }
    }
    if (reject != nullptr) {
        const RejectPlan &pl = plan.rpl;
        info->early_stop = pl.early_stop != kReadAll ? 1 : 0;
        info->stat_segments = pl.stat_segments;
        info->race_segments = reject->accept_mode == SPEC_ACCEPT_GREEDY ? 0 : pl.race_segments;
        info->reject_blocks = (int32_t)reject_blocks(reject, pl);
        if (attn == nullptr || !plan.apl.use_mfma) info->launches += 1;
    }
    info->workspace_bytes = plan.workspace_bytes;
    return SPEC_OK;
}

spec_status spec_verify_attn(const spec_attn_args *attn, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    spec_status st = validate_attn_scalars(attn);
    if (st != SPEC_OK) return st;
    const StepPlan &plan = plan_for(attn, nullptr);
    if (plan.status != SPEC_OK) return plan.status;
    st = validate_attn_table(attn);
    if (st != SPEC_OK) return st;
    const AttnPlan &pl = attn_plan_for(plan, workspace_bytes);
    st = check_workspace(workspace, workspace_bytes, pl.total_bytes);
    if (st != SPEC_OK) return st;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const AttnParams ap = attn_params(attn, pl, static_cast<char *>(workspace), nullptr);
    if (!pl.use_mfma) return run_attn_generic(ap, attn->qkv_dtype, stream);
    hipError_t err = timed_launch(SPEC_KERNEL_ATTN, [&](LaunchEvents ev) {
        return launch_step_fused(&ap, nullptr, pl.spread ? &plan.listed : &plan.order, ev, stream);
    });
    if (err == hipSuccess && !pl.fused_combine && pl.max_chunks > 1)
        err = timed(SPEC_KERNEL_ATTN_COMBINE, stream, [&] { return launch_attn_combine(ap, stream); });
    return err == hipSuccess ? SPEC_OK : SPEC_EHIP;
}

spec_status spec_reject_sample(const spec_reject_args *reject, void *workspace, size_t workspace_bytes,
                               void *hip_stream)
{
    spec_status st = validate_reject_scalars(reject);
    if (st != SPEC_OK) return st;
    const StepPlan &plan = plan_for(nullptr, reject);
    if (plan.status != SPEC_OK) return plan.status;
    st = validate_reject_tokens(reject);
    if (st != SPEC_OK) return st;
    const RejectPlan &pl = reject_plan_for(plan, workspace_bytes);
    st = check_workspace(workspace, workspace_bytes, pl.total_bytes);
    if (st != SPEC_OK) return st;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const RejectParams rp = reject_params(reject, pl, static_cast<char *>(workspace));
    const hipError_t err =
        timed_launch(SPEC_KERNEL_REJECT, [&](LaunchEvents ev) { return launch_step_fused(nullptr, &rp, nullptr, ev, stream); });
    return err == hipSuccess ? SPEC_OK : SPEC_EHIP;
}

spec_status spec_verify_step(const spec_attn_args *attn, const spec_reject_args *reject, void *workspace,
                             size_t workspace_bytes, void *hip_stream)
{
    const StepPlan *plan = nullptr;
    const spec_status st = prepare_step(attn, reject, plan);
    if (st != SPEC_OK) return st;
    return step_on_workspace(attn, reject, *plan, workspace, workspace_bytes, hip_stream);
}

spec_status spec_verify_step_static(const spec_attn_args *attn, const spec_reject_args *reject, void *hip_stream)
{
    // sizes first, on the host: a step that does not fit is refused before anything touches the GPU
    const StepPlan *plan = nullptr;
    const spec_status st = prepare_step(attn, reject, plan);
    if (st != SPEC_OK) return st;
    if (plan->apl_small.total_bytes + plan->rpl_small.total_bytes > SPEC_STATIC_SCRATCH_BYTES) return SPEC_EWORKSPACE;
    void *ws = static_scratch_of_current_device();
    if (ws == nullptr) return SPEC_EHIP;
    return step_on_workspace(attn, reject, *plan, ws, SPEC_STATIC_SCRATCH_BYTES, hip_stream);
}

spec_status spec_kv_append(const spec_kv_append_args *a, void *hip_stream)
{
    if (a == nullptr || a->B < 1 || a->Hkv < 1 || a->T < a->B || a->num_blocks < 1 || a->max_blocks_per_req < 1)
        return SPEC_EINVAL;
    if (a->new_k == nullptr || a->new_v == nullptr || a->k_cache == nullptr || a->v_cache == nullptr ||
        a->block_table == nullptr || a->kv_len == nullptr || a->cu_q_len == nullptr || a->host_kv_len == nullptr ||
        a->host_cu_q_len == nullptr)
        return SPEC_EINVAL;
    if (a->dtype != SPEC_F32 && a->dtype != SPEC_BF16) return SPEC_EINVAL;
    if (a->kv_layout != SPEC_KV_TOKEN_MAJOR && a->kv_layout != SPEC_KV_MFMA) return SPEC_EINVAL;
    // (rows and pools are moved as vectors of 8 elements)
    if (((reinterpret_cast<uintptr_t>(a->new_k) | reinterpret_cast<uintptr_t>(a->new_v) |
          reinterpret_cast<uintptr_t>(a->k_cache) | reinterpret_cast<uintptr_t>(a->v_cache)) & 31) != 0)
        return SPEC_EINVAL;
    if (a->d != 64 && a->d != 128) return SPEC_EUNSUPPORTED;
    if (a->kv_layout == SPEC_KV_MFMA && a->dtype != SPEC_BF16) return SPEC_EUNSUPPORTED;
    if (a->host_cu_q_len[0] != 0 || a->host_cu_q_len[a->B] != a->T) return SPEC_EINVAL;
    for (int b = 0; b < a->B; ++b) {
        const int q_len = a->host_cu_q_len[b + 1] - a->host_cu_q_len[b];
        if (q_len < 1 || q_len > SPEC_K_MAX + 1 || a->host_kv_len[b] < q_len) return SPEC_EINVAL;
        if ((a->host_kv_len[b] + SPEC_BLOCK_SIZE - 1) / SPEC_BLOCK_SIZE > a->max_blocks_per_req) return SPEC_EINVAL;
    }
    KvAppendParams p;
    memset(&p, 0, sizeof p);
    p.B = a->B; p.Hkv = a->Hkv; p.d = a->d; p.max_blocks_per_req = a->max_blocks_per_req; p.T = a->T;
    p.kv_layout = a->kv_layout;
    p.elem_bytes = a->dtype == SPEC_BF16 ? 2 : 4;
    p.num_blocks = a->num_blocks;
    p.new_k = a->new_k; p.new_v = a->new_v; p.k_cache = a->k_cache; p.v_cache = a->v_cache;
    p.block_table = a->block_table; p.kv_len = a->kv_len; p.cu_q_len = a->cu_q_len;
    p.errors = reinterpret_cast<unsigned long long *>(a->error_count);
    return launch_kv_append(p, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPEC_OK : SPEC_EHIP;
}

spec_status spec_kv_repack_mfma(const void *src_k, const void *src_v, void *dst_k, void *dst_v, int32_t num_blocks,
                                int32_t Hkv, int32_t d, void *hip_stream)
{
    if (src_k == nullptr || src_v == nullptr || dst_k == nullptr || dst_v == nullptr || num_blocks < 1 || Hkv < 1)
        return SPEC_EINVAL;
    if (src_k == dst_k || src_v == dst_v || src_k == dst_v || src_v == dst_k) return SPEC_EINVAL;
    if (d != 64 && d != 128) return SPEC_EUNSUPPORTED;
    const hipError_t err = launch_kv_repack(src_k, src_v, dst_k, dst_v, num_blocks, Hkv, d,
                                            static_cast<hipStream_t>(hip_stream));
    return err == hipSuccess ? SPEC_OK : SPEC_EHIP;
}

spec_status spec_profile_begin(int32_t max_launches)
{
    if (max_launches < 1 || max_launches > (1 << 20)) return SPEC_EINVAL;
    if (g_prof.on) return SPEC_EINVAL;
    g_prof.events.assign(2 * (size_t)max_launches, nullptr);
    for (auto &e : g_prof.events)
        if (hipEventCreate(&e) != hipSuccess) return SPEC_EHIP;
    g_prof.kernel_of_pair.clear();
    g_prof.kernel_of_pair.reserve(max_launches);
    g_prof.capacity_pairs = (size_t)max_launches;
    g_prof.on = true;
    return SPEC_OK;
}

spec_status spec_profile_end(float *total_ms, int32_t *launches)
{
    if (!g_prof.on || total_ms == nullptr || launches == nullptr) return SPEC_EINVAL;
    g_prof.on = false;
    for (int i = 0; i < SPEC_NUM_KERNELS; ++i) { total_ms[i] = 0.0f; launches[i] = 0; }
    spec_status st = SPEC_OK;
    for (size_t pair = 0; pair < g_prof.kernel_of_pair.size(); ++pair) {
        float ms = 0.0f;
        if (hipEventSynchronize(g_prof.events[2 * pair + 1]) != hipSuccess ||
            hipEventElapsedTime(&ms, g_prof.events[2 * pair], g_prof.events[2 * pair + 1]) != hipSuccess) {
            st = SPEC_EHIP;
            break;
        }
        total_ms[g_prof.kernel_of_pair[pair]] += ms;
        launches[g_prof.kernel_of_pair[pair]] += 1;
    }
    for (auto &e : g_prof.events) (void)hipEventDestroy(e);
    g_prof.events.clear();
    g_prof.kernel_of_pair.clear();
    g_prof.capacity_pairs = 0;
    return st;
}

const char *spec_status_string(spec_status status)
{
    switch (status) {
        case SPEC_OK: return "ok";
        case SPEC_EINVAL: return "invalid argument";
        case SPEC_EUNSUPPORTED: return "unsupported shape, dtype or layout";
        case SPEC_EWORKSPACE: return "workspace missing, misaligned or too small";
        case SPEC_EHIP: return "HIP call failed";
    }
    return "unknown status";
}

int32_t spec_verify_version(void) { return 200; }

}  // extern "C"
