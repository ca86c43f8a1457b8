// Host side of the C ABI declared in include/relay_attn.h: argument validation (before any
// HIP call), work decomposition, workspace layout and kernel launches.  Nothing here
// allocates, and nothing but relay_attn_debug_validate copies or synchronises.
#include "../../include/relay_attn.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "ra_kernels.h"

// Scratch of relay_attn_decode_static: the partial results between the partial-attention launch
// and the fusion launch, for callers that can neither allocate a workspace nor pass one.  Every
// device the library runs on holds its own copy of this array until the process ends.  In host
// code the name is only a handle for hipGetSymbolAddress, never an address to pass on.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int32_t kAbiVersion = 6;
constexpr int kWholeMinTokens = 32;   // new tokens per request, on average, from which the prompt phase is one launch

struct Plan {
    int group;            // query heads per kv head
    int rows;             // total_q * Hq output rows
    int n_mtiles;         // 32-row tiles of stacked queries per kv head
    int sys_chunk;        // system positions per work item
    int n_sys_chunks;
    int ctx_part;         // context positions per work item (prompt phase, per-request kernel)
    int n_ctx_parts;      // context partial slots per row
    int n_ctx_likely;     // of these, the ones that lengths near the bound take (0: all); see FuseArgs
    int ctx_wgs;          // decode: context workgroups (four wavefronts each) in the tile launch
    int ctx_t_floor;      // decode: least tiles per context wavefront, bounds the slots per row
    bool paired;          // decode: the launch is exactly two workgroups per compute unit
    bool whole;           // prompt phase: one launch of items that write the output themselves
    bool unsupported;
    int max_ctx;
    int block_size_log2;
    bool rows_path;       // system part (and prefill context part) through the many-rows kernel
    bool rows_sys;        // decode: system items of the many-rows kind inside the tile launch
    int n_sys_rowblocks;  // 128-row blocks of stacked queries per kv head
    int n_ctx_rowblocks;  // prefill: 128-row blocks per (request, kv head)
    // partial p of row r: o at off_o + (p*rows + r)*d*4, lse at off_lse + (p*rows + r)*4;
    // partials 0..n_sys_chunks-1 are system chunks, the rest context parts
    size_t off_o, off_lse, bytes;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

ra_status check_params(const ra_params *p, int32_t total_q) {
    if (!p) return RA_ERR_INVALID_ARG;
    if (p->batch < 0 || total_q < 0 || p->num_q_heads < 1 || p->num_kv_heads < 1 ||
        p->sys_len < 0 || p->block_size < 1 || p->num_blocks < 0 || p->max_blocks_per_seq < 0 ||
        p->max_context_len < 0 || p->sys_chunk_tokens < 0 || p->ctx_part_tokens < 0 ||
        p->reserved0 != 0)
        return RA_ERR_INVALID_ARG;
    if (p->num_q_heads % p->num_kv_heads != 0) return RA_ERR_INVALID_ARG;
    if ((p->block_size & (p->block_size - 1)) != 0) return RA_ERR_INVALID_ARG;
    if (!(p->softmax_scale == p->softmax_scale)) return RA_ERR_INVALID_ARG;  // NaN
    if (p->out_is_fp32 != 0 && p->out_is_fp32 != 1) return RA_ERR_INVALID_ARG;
    const int64_t strides[] = {p->q_stride_token, p->q_stride_head, p->o_stride_token,
                               p->o_stride_head, p->sys_stride_token, p->sys_stride_head};
    for (int64_t s : strides)
        if (s < 0 || (s % 8) != 0) return RA_ERR_INVALID_ARG;
    if (p->sys_chunk_tokens % 32 != 0 || p->ctx_part_tokens % 128 != 0) return RA_ERR_INVALID_ARG;
    if ((int64_t)p->max_blocks_per_seq * p->block_size > INT32_MAX) return RA_ERR_INVALID_ARG;
    if (p->max_context_len > (int64_t)p->max_blocks_per_seq * p->block_size)
        return RA_ERR_INVALID_ARG;
    if (p->head_dim != 64 && p->head_dim != 128) return RA_ERR_UNSUPPORTED;
    const int g = p->num_q_heads / p->num_kv_heads;
    if (g < 1 || g > 8) return RA_ERR_UNSUPPORTED;
    if ((int64_t)total_q * p->num_q_heads > (1 << 28)) return RA_ERR_UNSUPPORTED;
    return RA_OK;
}

enum PlanKind { kRelayDecode, kNaiveDecode, kPrefill };

// Compute units of the current device: asked once (an attribute query, no launch) and cached;
// 256, the MI355X's count, where no device answers (a machine without a GPU still sizes
// workspaces and reports plans).  The decomposition below is a pure function of the parameters
// and this number, so the workspace size a caller asked for and the launch always agree.
constexpr int kReferenceCus = 256;
int device_compute_units() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
            (void)hipGetLastError();         // leave no sticky error behind for the caller
            return kReferenceCus;
        }
        return n;
    }();
    return cus;
}

// Device address of this device's copy of `scratch`: looked up once per device, with that device
// current (each device has the array at an address of its own), and kept.
constexpr int kMaxDevices = 64;
ra_status static_scratch(void **ptr) {
    static std::mutex lock;
    static void *known[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return RA_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return RA_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> hold(lock);
    if (!known[dev]) {
        void *found = nullptr;
        if (hipGetSymbolAddress(&found, HIP_SYMBOL(scratch)) != hipSuccess || !found) {
            (void)hipGetLastError();
            return RA_ERR_HIP;
        }
        known[dev] = found;
    }
    *ptr = known[dev];
    return RA_OK;
}

// The longest context part whose block ids fit an item's table in LDS.
int longest_part(const ra_params *p) {
    int64_t cap = (int64_t)ra::kMaxPartBlocks * p->block_size;
    if (cap > 4096) cap = 4096;
    const int part = (int)(cap / 128 * 128);
    return part < 128 ? 128 : part;
}

// New tokens per request, on average, from which a block of 128 rows does not meet too many requests to
// go through their contexts one after the other.
bool many_new_tokens(const ra_params *p, int32_t total_q) {
    return total_q >= (int64_t)kWholeMinTokens * p->batch || (p->sys_len <= 1024 && total_q >= (int64_t)4 * p->batch);
}

// What the prefixes of a call are to an average query row: the length of its system prompt, and the requests that share it
// (negative: one prefix).  By rows and not by prefixes: several prompts are often one large application and some
// small ones, and a prefix that no request of the step uses counts for nothing.  (60 prompt-phase calls of
// such groups that choose another form so: 0.81 of the time by prefixes, eight of them slower, by up to 1.3.)
struct Groups {
    double sys_len = -1, requests = -1;
};

// How the prompt phase is cut, where the caller leaves it to the library.
struct PromptSplit {
    bool whole;          // one launch of items that go through prompt and contexts (see `run`)
    int chunk, part;     // otherwise: system positions and context positions of an item
};

// The fewest partials: about 400 workgroups of at least 512 system positions, the longest context parts;
// one launch where that is one chunk (see split_prompt for its limits).
PromptSplit coarse_split(const ra_params *p, int32_t total_q) {
    const int base = p->num_kv_heads * ceil_div(total_q * (p->num_q_heads / p->num_kv_heads), 128);
    const int most = ceil_div(p->sys_len, 512);
    int n = (400 + base / 2) / base;
    if (n > most) n = most;
    if (n < 1) n = 1;
    return {n == 1 && many_new_tokens(p, total_q), ceil_div(ceil_div(p->sys_len, n), 128) * 128, longest_part(p)};
}

// A prompt-phase launch takes about as long as the larger of its longest item and its work per
// compute unit, plus the thin end of the launch; a finer cut shortens the first and the last
// of these and costs partials, which are written, read again and fused.  The estimate below was
// fitted to measured cuts of 16 shapes (system prompts of 300 .. 12000, contexts up to 8000, 80 .. 14400
// stacked rows per kv head, 4 .. 40 kv heads, head_dim 64 and 128).  Over 478 cuts of 21 shapes, taken again
// with the present item order, its choice is 1 .. 12 % over the best cut of a shape, against up to 3.5 times for
// the fixed rule in front of it (coarse_split): 8 requests of 9 .. 75 tokens behind contexts of 300 ..
// 4000 118 -> 67 us, 4 requests of 10 .. 100 tokens behind 500 .. 2000 132 -> 37 us.
// Uses what the workspace size is computed from, and `groups` for the whole form only, which needs none of it.
PromptSplit split_prompt(const ra_params *p, int32_t total_q, int32_t max_ctx, const Groups &groups, bool tight) {
    const int64_t G = p->num_q_heads / p->num_kv_heads, hkv = p->num_kv_heads, batch = p->batch > 0 ? p->batch : 1;
    const int64_t s = p->sys_len, base = hkv * ((total_q * G + 127) / 128);
    const double row_bytes = (double)total_q * p->num_q_heads * p->head_dim * 4;
    const double step_us = p->head_dim == 128 ? 1.5 : 1.1;     // 64 keys by 128 rows, a compute unit to itself
    const double cus = device_compute_units();
    // The lengths live on the device.  Known of them is the bound, which may be a table's capacity, and
    // that the contexts of all requests together fit the cache (a num_blocks that does not even hold the
    // new tokens was not filled in; contexts that share blocks may be longer, which costs time only).
    // Going by the bound alone, a loose one took launches apart that are best left whole and left few
    // chunks to prompts that the launch then waited for: 32 requests of 32 heads with 40 .. 200 new
    // tokens, s = 600, in tables of 8192 positions 215 us against 126, 4 requests of 32/8 heads with
    // 10 .. 60 behind 100 .. 200, s = 1024, 40 against 25.
    const double mean_new = (double)total_q / batch;
    double held = (double)p->num_blocks * p->block_size;
    if (held < total_q) held = (double)batch * max_ctx;
    const double ctx = held / batch < 0.85 * max_ctx ? held / batch : 0.85 * max_ctx;
    double ctx_most = held < max_ctx ? held : max_ctx;      // (four times the mean: the longest of most batches)
    if (ctx_most > 4 * held / batch) ctx_most = 4 * held / batch;
    // items per context part: blocks of 128 stacked rows of an average request, times kv heads and requests
    const int64_t ctx_base = batch * hkv * (((total_q + batch - 1) / batch * G + 127) / 128);
    const double steps = ((double)base * s + ctx_base * ctx) / 64;
    auto launch_us = [&](double longest, double all, double items) {
        const double even = all / cus + 0.35 * longest;
        return step_us * (longest > even ? longest : even) + 2.0 * items / cus;
    };
    PromptSplit best{false, 128, longest_part(p)};
    double best_us = 1e300;
    const int longest = best.part;
    const int64_t most_chunks = s > 0 ? (s + 127) / 128 : 1;
    const int64_t most_parts = max_ctx > 0 ? (max_ctx + 127) / 128 : 1;
    const int64_t least_parts = max_ctx > 0 ? (max_ctx + longest - 1) / longest : 1;
    // (no more items than a launch index holds, whatever the longest request brings)
    const int64_t rb_most = batch * hkv * ((total_q * G + 127) / 128);
    // (and no more workspace than twice the coarsest cut's, or 64 MiB)
    int64_t most_partials = (int64_t)((64 << 20) / row_bytes);
    if (most_partials < 2 * (least_parts + 1)) most_partials = 2 * (least_parts + 1);
    for (int64_t nc = 1; nc <= most_chunks; nc += (nc + 1) / 2) {
        const int64_t chunk = (((s > 0 ? s : 1) + nc - 1) / nc + 127) / 128 * 128;
        const int64_t n_chunks = (s + chunk - 1) / chunk;
        for (int64_t np = least_parts; np <= most_parts; np += (np + 1) / 2) {
            int64_t part = (((max_ctx > 0 ? max_ctx : 1) + np - 1) / np + 127) / 128 * 128;
            if (part > longest) part = longest;
            if (np > least_parts && (rb_most * (np + 1) > (1 << 30) || base * n_chunks > (1 << 30))) break;
            if (np > least_parts && n_chunks + (max_ctx + part - 1) / part > most_partials) break;
            const double parts = max_ctx > 0 ? ceil(ctx / part) : 0;
            const double t_sys = (double)(chunk < s ? chunk : s) / 64, t_ctx = (part < ctx_most ? part : ctx_most) / 64;
            const double us = launch_us(t_sys > t_ctx ? t_sys : t_ctx, steps, base * n_chunks + ctx_base * parts) +
                              row_bytes * (n_chunks + parts) * (2 / 5e6) + 12;
            if (us < best_us) best_us = us, best.chunk = (int)chunk, best.part = (int)part;
        }
    }
    // Whole items or the cut, by an estimate of each.  Both forms of 480 drawn calls (4 .. 930 new tokens per
    // request, 1 .. 32 requests, 4 .. 52 kv heads, prompts of 100 .. 16000) were timed; the estimate of the whole form
    // is within 13 % of its time (one standard deviation): every request whose rows a block meets costs it a
    // range of keys of its own, and the longest context is taken as twice the mean.  The form it picks is 1.1 %
    // over the faster one in the mean.  The rule in front of it was 4.7 % over, and up to four times where a
    // short walk alone decided: 17 requests of 10 .. 13 tokens, 8 heads, s = 324, 66.1 us whole, 16.0 cut; one of
    // 57 tokens of 28/4 heads behind 1667, 57 and 20; the other way, 264 blocks of 5 prompts with s = 1726
    // 62 us whole, 81 cut.
    // With several prompts the requests of a block share one of them: no more meet than an average group has
    // (the workspace is sized without the groups, so they may only ever speak for the whole form, which needs none).
    const double met = mean_new > 0 ? 128.0 / G / mean_new + 1 : 1;     // requests with rows in a block
    const double reqs_any = met < batch ? met : batch, group = groups.requests < 0 ? (double)batch : ceil(groups.requests);
    const double sys_mean = groups.sys_len < 0 ? (double)s : groups.sys_len;
    const double reqs = reqs_any < group ? reqs_any : group;
    const double ctx_long = ctx_most < 2 * held / batch ? ctx_most : 2 * held / batch;
    const double walk = ceil(s / 64.0) + reqs * ceil(ctx_long / 64), walk_mean = ceil(sys_mean / 64) + reqs * (ctx / 64 + 0.5);
    const double blocks = base / cus, even = 0.8 * walk_mean * blocks + 0.55 * walk;
    const double whole_us = 8.6 + (p->head_dim == 128 ? 1.42 : 0.95) * (walk > even ? walk : even) + 0.8 * reqs + 4.3 * blocks;
    const double cut_us = 14 + (p->head_dim == 128 ? 0.85 : 0.75) * (best_us - 12);      // (as measured beside them)
    // Few blocks with a short walk stay whole without an estimate where the requests bring 32 tokens and
    // more: that form leaves the workspace alone (5 requests of 63 tokens, 8 heads, s = 493, 29.0 us, 19.8
    // cut, is the most it costs).
    const bool short_walk =
        s <= 512 && total_q >= (int64_t)kWholeMinTokens * batch && s + reqs_any * max_ctx <= 2048 - 28 * base;
    // Near the line the estimates err (the whole form's by 13 %).  A call that the cut's own estimate would not leave
    // whole is taken whole where that is a tenth faster, if cache or bound say how long the contexts are (4 requests of 8
    // heads, 104 .. 917 tokens: 52.2 us cut, 67.5 whole, estimates 70 and 65), and one that it would is cut, if the
    // bound leaves that open, where that is a fifth faster (11 of 32/8 heads of 64, 43 .. 76 tokens under 444: 21.7 whole,
    // 26.7 cut, 40 and 33).  Of 560 drawn calls nine were slower by the estimates alone than by that rule alone, by up to
    // 1.29, and four are with both, by up to 1.24; all together take 0.972 of the time by the rule, 0.8 % over the faster forms.
    const double walk_any = s + (reqs_any * ctx_most < held ? reqs_any * ctx_most : held);
    const bool few_blocks = (400 + base / 2) / base > 1 && s > 512;
    const bool by_cut = !few_blocks && (s + reqs_any * max_ctx <= 2048 ||
                                        launch_us(walk_any / 64, (s + reqs_any * ctx) / 64 * base, (double)base) + 4 + 2 * reqs_any <= best_us);
    const bool filled = held == (double)p->num_blocks * p->block_size;
    const bool known = (filled && held <= 1.5 * batch * max_ctx) || max_ctx <= 2 * mean_new;
    // (`tight`: a workspace too small for the cut.  The whole form needs none, so the estimates alone decide.)
    const double lead = tight ? 1 : by_cut ? (known ? 1 : 1.25) : (known ? 0.9 : 1);
    best.whole = many_new_tokens(p, total_q) && (short_walk || whole_us <= lead * cut_us);
    if (best.whole) best.chunk = (int)((s + 127) / 128 * 128), best.part = longest;
    if (best.chunk < 128) best.chunk = 128;
    return best;
}

// The least work worth giving a wavefront of the tile launch.
constexpr int kMinWaveTiles = 4;
// Row tiles (of 32 stacked query rows per kv head) from which a decode batch takes its system
// part through many-rows items.
constexpr int kRowsSysMinTiles = 8;

// How a decode step is planned, where a first plan shows what it comes to.
struct DecodeWay {
    bool by_bound = false;         // for contexts as long as the bound allows, whatever the cache holds
    bool rows_by_bound = false;    // the kind of its system items chosen so
    int64_t least_turns = 0;       // turns that a streaming system workgroup should at least have
    // (A workspace too small for the plan takes none of these refinements: they trade system chunks for context slots,
    // and some of the least workspaces that were accepted did not hold the slots, 6.1 MB of 6.6.)
};

// Work decomposition; a pure function of (params, total_q) so that the workspace size the
// caller asked for and the one the launch uses always agree.  A `budget` below that size asks for
// the fewest partials: the cut that a caller's workspace of fixed size, made for another batch, may
// still hold (the size does not only rise with the batch).  `way`: see DecodeWay.
Plan make_plan(const ra_params *p, int32_t total_q, PlanKind kind, int32_t max_q_len,
               int64_t sys_base_items = 0, bool allow_rows_sys = true, size_t budget = SIZE_MAX,
               const Groups &groups = {}, DecodeWay way = {}) {
    Plan pl{};
    const bool tight = budget != SIZE_MAX;
    const bool prefill = kind == kPrefill;
    // Wavefronts the chip holds at once with the tile kernel's two workgroups of four per
    // compute unit.
    const int kWorkgroupSlots = device_compute_units() * 2;
    const int kWaveSlots = kWorkgroupSlots * 4;
    pl.group = p->num_q_heads / p->num_kv_heads;
    pl.rows = total_q * p->num_q_heads;
    pl.n_mtiles = ceil_div(total_q * pl.group, 32);
    pl.block_size_log2 = 0;
    while ((1 << pl.block_size_log2) < p->block_size) ++pl.block_size_log2;
    pl.max_ctx = p->max_context_len > 0 ? p->max_context_len : p->max_blocks_per_seq * p->block_size;

    // Decode: the streaming tile kernel.  Prompt phase: the many-rows kernel, which fetches each
    // K/V tile once per 128 stacked rows.
    // (Wide GQA decode batches use many-rows items too, but inside the tile launch: rows_sys.)
    pl.rows_path = prefill;
    pl.n_sys_rowblocks = ceil_div(total_q * pl.group, 128);
    pl.n_ctx_rowblocks = prefill ? ceil_div(max_q_len * pl.group, 128) : 0;
    const size_t d = (size_t)p->head_dim;
    auto finish = [&]() {
        const size_t n_partials = (size_t)pl.n_sys_chunks + pl.n_ctx_parts;
        size_t at = 0;
        pl.off_o = at;   at = align_up(at + n_partials * pl.rows * d * 4, 256);
        pl.off_lse = at; at = align_up(at + n_partials * pl.rows * 4, 256);
        pl.bytes = at > 0 ? at : 256;
    };
    if (total_q == 0) {
        finish();
        return pl;
    }

    if (kind == kRelayDecode) {
        // One launch holds system workgroups (four wavefronts share a chunk of the prompt) and
        // context wavefronts (each takes an equal span of the stream of context tiles, see the
        // kernel).  The aim is that every wavefront of the launch moves about the same number of
        // 32-key tiles and that all of them are resident at once: t_star tiles each.  The context
        // side is sized from max_context_len (the lengths themselves live on the device); when
        // the real lengths are shorter its wavefronts simply finish earlier.
        const int64_t sys_tiles = ceil_div(p->sys_len, 32);               // per (kv head, row tile)
        const int64_t base_items = sys_base_items > 0 ? sys_base_items
                                                      : (int64_t)p->num_kv_heads * pl.n_mtiles;
        const int64_t t_max = pl.max_ctx > 0 ? ceil_div(pl.max_ctx, 32) : 0;   // tiles of one context
        const int64_t ctx_tiles = (int64_t)total_q * p->num_kv_heads * t_max;
        // What the launch is planned for: the contexts at the bound, or as many of their tiles as the cache can
        // hold where those are fewer (a num_blocks that does not even hold a token each was not filled in): a bound
        // twenty times the contexts had 7100 tiles planned for where 180 were there (18 requests of 32 heads, 3 .. 21
        // tokens behind s = 1008, 20.7 -> 14.8 us; contexts of 859 .. 1706 under a wider bound 23.3 -> 20.9).
        // Slots and the fewest workgroups stay those of the bound, so any lengths up to it are served.
        // Batches wide enough for many-rows items take it for short contexts only: with longer ones the even
        // launch that the bound leads to was faster (40 requests of 28/4 heads, contexts of 37 .. 310, 19.7 against 22.3
        // us; 153 of them, 425 .. 601, 47.5 against 52.7).
        int64_t ctx_like = ctx_tiles;
        if (!way.by_bound) {
            const int64_t held = (int64_t)p->num_blocks * p->block_size;
            const int64_t tiles = p->num_kv_heads * (held / 32 + (total_q + 1) / 2);
            const bool many_rows = pl.n_mtiles >= 4 && tiles >= 4 * (int64_t)total_q * p->num_kv_heads;
            if (held >= total_q && tiles < ctx_like && !many_rows) ctx_like = tiles;
        }
        const int64_t all_tiles = base_items * sys_tiles + ctx_like;
        if (ctx_tiles > INT32_MAX) {
            pl.unsupported = true;
            return pl;
        }
        // (in sixteenths of a tile, so that small launches are not rounded to whole tiles)
        int64_t t_star16 = (all_tiles * 16 + kWaveSlots - 1) / kWaveSlots;
        // (small launches: down to a tile and a half per wavefront rather than kMinWaveTiles, more
        // wavefronts in flight matter more than their length there: Llama-7B shape 25.7 -> 24.5 us,
        // batch 16 of the Llama-30B shape at s = 1024 24.0 -> 21.5 us, batch 8 at s = 512
        // 15.4 -> 14.4 us)
        if (t_star16 < 24) t_star16 = 24;
        const int64_t t_star = (t_star16 + 15) / 16;
        int64_t sys_wgs = 0, t_sys = 0, few_chunks = 0;
        const double t_item = ctx_tiles > 0 ? (double)ctx_like / ((double)total_q * p->num_kv_heads) : 0;   // tiles of a context
        // Wide grouped-query batches: with B*G stacked rows per kv head in many row tiles, every
        // 32-row streaming item would pull the system K/V of its chunk into its compute unit
        // (from L2, but what a unit can draw is capped there too: 87 us at the Llama-3-8B shape).
        // Many-rows items share each tile among 128 rows through LDS, a quarter of the draw.
        // (Measured against the streaming items over batch 32..512, 8..32 row tiles, prompts of
        // 512..16384: faster by 4..20 % where the system part is at least about half of the
        // context part, slower by up to 8 % in batches that are mostly context.)
        // From four row tiles (one full block of 128 rows) on it still pays when the system part
        // is both large (64 tiles per compute unit) and at least as large as the context part:
        // batch 128 of the Llama-30B shape at s = 8192 157 -> 128 us, batch 192 at 4096 163 -> 144 us.
        auto rows_pay = [&](int64_t ctx) {
            const int64_t sys_all = base_items * sys_tiles;
            const bool wide = pl.n_mtiles >= kRowsSysMinTiles && 2 * sys_all >= ctx;
            const bool full_block = pl.n_mtiles >= 4 && sys_all >= 64 * (kWorkgroupSlots / 2) && sys_all >= ctx;
            return allow_rows_sys && sys_base_items == 0 && p->sys_len > 0 && (wide || full_block);
        };
        pl.rows_sys = rows_pay(way.rows_by_bound ? ctx_tiles : ctx_like);
        if (pl.rows_sys) {
            const int64_t rb_items = (int64_t)p->num_kv_heads * pl.n_sys_rowblocks;
            int chunk = p->sys_chunk_tokens;
            if (chunk == 0) {
                // one workgroup per compute unit if the prompt is long enough (chunks of 256
                // positions or more: batch 64 of a 32/8-head model at s = 1024 34 -> 23 us against
                // chunks of 512), at most sixteen chunks (every chunk is one more partial per row
                // for the fusion to read)
                int64_t n_chunks = (kWorkgroupSlots / 2 + rb_items / 2) / rb_items;
                const int64_t most = ceil_div(p->sys_len, 256) < 16 ? ceil_div(p->sys_len, 256) : 16;
                if (n_chunks > most) n_chunks = most;
                if (n_chunks < 1) n_chunks = 1;
                chunk = (int)((sys_tiles + n_chunks - 1) / n_chunks) * 32;
            }
            pl.sys_chunk = chunk;
            pl.n_sys_chunks = ceil_div(p->sys_len, chunk);
            sys_wgs = rb_items * pl.n_sys_chunks;
            t_sys = chunk / 32;            // each of the four wavefronts walks every tile
        } else
        if (p->sys_len > 0) {
            int chunk = p->sys_chunk_tokens;
            if (chunk == 0) {
                auto chunks_of = [&](int64_t t16) {                     // nearest
                    const int64_t n = (sys_tiles * 16 + 2 * t16) / (4 * t16);
                    return n < 1 ? (int64_t)1 : n;
                };
                int64_t n_chunks = chunks_of(t_star16);
                // A plan for fewer tiles than the bound's comes to shorter chunks than that one.  They are taken as far
                // as they save a turn of the four wavefronts (25 requests of 40 heads, s = 645: four chunks of 6 tiles
                // 15.9 us, three of 7 13.3), and no shorter than `way` says.
                if (ctx_like < ctx_tiles) {
                    int64_t bound16 = ((base_items * sys_tiles + ctx_tiles) * 16 + kWaveSlots - 1) / kWaveSlots;
                    if (bound16 < 24) bound16 = 24;
                    few_chunks = chunks_of(bound16);
                    if (way.least_turns > 0 && n_chunks > few_chunks) {
                        const int64_t n = chunks_of(16 * way.least_turns);
                        n_chunks = n < few_chunks ? few_chunks : n < n_chunks ? n : n_chunks;
                    }
                    auto turns = [&](int64_t n) { return ((sys_tiles + n - 1) / n + 3) / 4; };
                    while (!tight && n_chunks > few_chunks && turns(n_chunks - 1) == turns(n_chunks)) --n_chunks;
                }
                // At most one system workgroup per compute unit: a compute unit cannot draw more
                // than about 1/256 of the memory bandwidth whatever it holds, so two long
                // workgroups on one unit finish last (measured: 208 system workgroups beat 312
                // and 416 at the 8192- and 16384-position prompts, 59 vs 63 us and 92 vs 95 us);
                // the context wavefronts fill the second slot of every unit.
                if (base_items * n_chunks > kWorkgroupSlots / 2) n_chunks = kWorkgroupSlots / 2 / base_items;
                if (n_chunks < 1) n_chunks = 1;
                chunk = (int)((sys_tiles + n_chunks - 1) / n_chunks) * 32;
                // Small launches (up to 2.5 tiles per wavefront) wait for units that got two workgroups
                // where most got one.  The four wavefronts take a chunk's tiles in turn, so up to the next
                // multiple of four a longer chunk takes as many turns; it is taken where it brings
                // the launch from above one workgroup per unit (by a quarter at most: beyond that the
                // second ones are spread anyway) down to it.  Both sides of 40 such launches, 1 .. 59
                // requests: 0.83 .. 1.00 of the time on 38 (two requests of 32 heads, s = 4152, 24.1 -> 19.9
                // us), 1.04 and 1.05 on two; without that effect 13.4 -> 14.0 (10 requests of 28/4 heads, s =
                // 1989).  Up to four tiles are one turn as they are.  (A multiple of four below, a turn
                // less, gives the context side shorter spans as well and was slower on 74 launches of 111,
                // by up to 21 %.)
                const int64_t tiles = chunk / 32, up = tiles / 4 * 4 + 4;
                if (t_star16 <= 40 && tiles > 4 && tiles % 4 != 0) {
                    const int64_t like16 = up * 4 > t_star16 ? up * 4 : t_star16;
                    const int64_t units = kWorkgroupSlots / 2, ctx_like_wgs = (ctx_like * 16 + 4 * like16 - 1) / (4 * like16);
                    auto wgs_at = [&](int64_t t) { return base_items * ((sys_tiles + t - 1) / t); };
                    const int64_t total = wgs_at(tiles) + ctx_like_wgs;
                    if (total > units && total <= units * 5 / 4 && wgs_at(up) + ctx_like_wgs <= units) chunk = (int)up * 32;
                }
            }
            pl.sys_chunk = chunk;
            pl.n_sys_chunks = ceil_div(p->sys_len, chunk);
            sys_wgs = base_items * pl.n_sys_chunks;
            t_sys = ceil_div(chunk / 32, 4);
        }
        if (ctx_tiles > 0) {
            // a span's block ids must fit the per-wavefront table in LDS
            int64_t t_cap = ((int64_t)ra::kMaxPartBlocks - 1) * p->block_size / 32;
            if (t_cap < 1) t_cap = 1;
            int64_t wgs;
            // Which workgroups share a compute unit (i and i + 256 of a 512-workgroup grid) was
            // measured on the 256-unit chip only; elsewhere every context wavefront gets an equal
            // span.
            const bool pairing_known = device_compute_units() == kReferenceCus;
            if (p->ctx_part_tokens > 0) {
                const int64_t t_fixed = p->ctx_part_tokens / 32;
                if (t_fixed > t_cap) {
                    pl.unsupported = true;
                    return pl;
                }
                wgs = (ctx_tiles + 4 * t_fixed - 1) / (4 * t_fixed);
                pl.ctx_t_floor = (int)t_fixed;
                pl.n_ctx_parts = (int)((t_max + t_fixed - 1) / t_fixed) + 1;
            } else {
                const int64_t least = (ctx_tiles + 4 * t_cap - 1) / (4 * t_cap);
                const int64_t t_like16 = t_sys * 16 > t_star16 ? t_sys * 16 : t_star16;
                wgs = (ctx_like * 16 + 4 * t_like16 - 1) / (4 * t_like16);
                // Short contexts: a wavefront of few tiles has as many contexts to begin, each with a chain of
                // trips of its own (length, block ids, rows: about 3 us next to 0.9 for a tile), so it takes
                // fewer of them than the turns of a system workgroup leave room for (a step of a many-rows item is
                // about half a turn), as long as the machine has places.  245 requests of 28/4 heads, contexts of
                // 21 .. 30, s = 437: 35.5 -> 21.2 us; 7 of 32 heads, 5 .. 17, s = 5429: 32.0 -> 24.2; 145 of 40 heads,
                // 30 .. 40, s = 162: 71 -> 47; longer contexts come out as before.
                if (!way.by_bound) {
                    const double turns = (pl.rows_sys ? 0.5 * t_sys : sys_wgs > 0 ? t_sys : t_star) + 2.5;
                    double per_wave = turns / (0.9 + 3.0 / (t_item > 1 ? t_item : 1));
                    if (per_wave < 1) per_wave = 1;
                    // (and no fewer workgroups than the bound would have, where there are places for them)
                    int64_t more = (int64_t)ceil(ctx_like / (4 * per_wave));
                    const int64_t bound = (ctx_tiles * 16 + 4 * t_like16 - 1) / (4 * t_like16);
                    if (bound > more) more = bound;
                    if (more > kWorkgroupSlots - sys_wgs) more = kWorkgroupSlots - sys_wgs;
                    if (more > wgs) wgs = more;
                }
                // when the launch is about one machine-full of equally long wavefronts, make it
                // exactly one
                if (all_tiles > (int64_t)kWaveSlots * kMinWaveTiles && sys_wgs <= kWorkgroupSlots * 7 / 8 &&
                    (sys_wgs == 0 || 4 * t_sys >= 3 * t_star) && sys_wgs + wgs <= kWorkgroupSlots * 3 / 2) {
                    wgs = kWorkgroupSlots - sys_wgs;
                    pl.paired = wgs >= least && sys_wgs > 0 && sys_wgs <= kWorkgroupSlots / 2 && pairing_known;
                }
                // a small launch that comes out just above one machine-full is cut back to it (the
                // overflow would run alone afterwards), if that leaves spans of two tiles or more
                else if (sys_wgs + wgs > kWorkgroupSlots && sys_wgs + wgs <= kWorkgroupSlots * 3 / 2 &&
                         sys_wgs < kWorkgroupSlots &&
                         ctx_tiles >= 2 * 4 * (kWorkgroupSlots - sys_wgs)) {
                    wgs = kWorkgroupSlots - sys_wgs;
                    pl.paired = wgs >= least && sys_wgs > 0 && sys_wgs <= kWorkgroupSlots / 2 && pairing_known;
                }
                if (wgs < least) wgs = least;
                if (wgs < 1) wgs = 1;
                // t_est: tiles per wavefront if every context had the maximum length.  Real
                // lengths are shorter and the spans shrink with them, down to the floor below; a
                // floor near t_est would leave most context wavefronts without work (a batch
                // with lengths uniform in [64, 1024] has half the tiles the plan assumed; one of
                // 1500 .. 15000 under a bound of 16400 has half of them as well).  So the floor is
                // an eighth of t_est.  Slots that the real lengths do not need cost workspace, and in
                // the fusion the log-sum-exps of a round (their payloads are left alone where they
                // would be many, see launch_fuse_d); the partials stay within the
                // static scratch unless even a floor of t_est itself takes more.
                // (12 requests, 8 kv heads, contexts 1500 .. 15000: 95.9 -> 73.5 us with
                // spans of 12 tiles on every wavefront instead of 24 on half of them)
                // (short contexts, up to 8 tiles, go by the tiles that are there: spans of one tile behind a loose
                // bound, 15.2 -> 10.9 us at 12 requests of 8 heads, 8 .. 76 tokens; for longer ones the partials
                // of so many spans cost more than they give, 17.0 -> 20.9 at 6 of 28/4 heads, 1240 .. 5082)
                auto parts = [&](int64_t t) { return (t_max + t - 1) / t + 1; };
                const int64_t t_bound = (ctx_tiles + 4 * wgs - 1) / (4 * wgs);
                const int64_t t_est = t_item < 8 ? (ctx_like + 4 * wgs - 1) / (4 * wgs) : t_bound;
                int64_t slots = parts(t_bound);
                int64_t t_low = (t_est + 7) / 8;
                if (t_low < kMinWaveTiles) t_low = kMinWaveTiles < t_est ? kMinWaveTiles : t_est;
                int64_t wide = parts(t_low);
                const size_t most = budget < kStaticScratchBytes ? budget : kStaticScratchBytes;
                const int64_t room = (int64_t)((most > 512 ? most - 512 : 0) / ((size_t)pl.rows * (d * 4 + 4))) -
                                     pl.n_sys_chunks;
                if (wide > room) wide = room;
                if (wide > slots) slots = wide;
                pl.n_ctx_parts = (int)slots;
                pl.ctx_t_floor = (int)((t_max + slots - 2) / (slots - 1));
                // The rule for even units gives what a unit without a system workgroup has left over to its context
                // wavefronts.  With short contexts the few such units can be what the launch waits for (50 requests
                // of 40 heads, contexts of 9 .. 56 behind s = 1792, 240 system workgroups: system parts done at 17 us,
                // the 32 other workgroups at 27).  An estimate of both sides in us (a tile's share of the memory a
                // unit can draw; a wavefront's own 1.2 a tile and 5 a context begun) takes equal spans then, where the
                // even units leave the others the longer spans, or spans below the floor (a part of those
                // wavefronts gets the floor, and the rest nothing): 76 requests of 40 heads, 11 .. 30, s = 3128 48.3 -> 31.9
                // us, 255 of 16 of 64, six prompts 36.1 -> 25.3, 58 of 52, s = 215 23.9 -> 20.8.  By the estimate alone
                // launches of many contexts and little else took it too: 122 of 52 heads, 14 .. 28, s = 190 31.8 -> 34.8,
                // 84 of 40, 13 .. 42, four prompts of 100 .. 153 24.3 -> 26.6.  With contexts of 30 tiles equal spans
                // lost as well: 71 -> 77.
                //   Beside many-rows items, which take a tile at about half of a streaming one's time, equal spans are for
                // plans by the cache (161 of 40 heads, s = 3558, bound 315 60.2 -> 54.1; 171, s = 2560 52.8 -> 46.4), where the
                // bound says little of the spans; at the bound they were no better (166 of 52, s = 4759 80.7 -> 85.9).
                if (pl.paired && t_item < 4 && !way.by_bound && pl.rows_sys) {
                    pl.paired = 2 * ctx_like >= ctx_tiles;
                } else if (pl.paired && t_item < 4 && !way.by_bound) {
                    const double step = (double)ceil_div(pl.sys_chunk, 32);
                    const double n = (double)ctx_like, even = n / (double)wgs;
                    const double draw = p->head_dim == 128 ? 0.59 : 0.3, each = 1.2 + 5.0 / (t_item > 1 ? t_item : 1);
                    auto longer = [](double a, double b) { return a > b ? a : b; };
                    const double light = longer(0, ((double)base_items * sys_tiles + n) / (kWorkgroupSlots / 2) - step);
                    const double heavy = wgs > sys_wgs ? (n - light * (double)sys_wgs) / (double)(wgs - sys_wgs) : 0;
                    const double by_unit = longer(longer(draw * (step + light), draw * 2 * heavy), each * longer(heavy, light) / 4);
                    const double equal = longer(longer(draw * (step + even), draw * 2 * even), each * even / 4);
                    if ((heavy > light || heavy < 4.2 * pl.ctx_t_floor) && equal < 0.995 * by_unit) pl.paired = false;
                }
                // What a row is likely to take of them: the contexts as they are planned for (short ones, the tiles that
                // are there) in spans as the device will cut them.  Counted with contexts at the bound, short
                // ones under a wide bound seemed to take every slot, and the fusion loaded the empty ones too (225
                // requests of 32/8 heads, contexts up to 70 under 2048 47.1 us so, 45.6 as here).
                const int64_t t_like = t_item < 8 ? (int64_t)ceil(t_item) : t_max;
                const int64_t span = pl.ctx_t_floor > t_est ? pl.ctx_t_floor : t_est;
                const int64_t likely = (t_like + span - 1) / span + 1;
                pl.n_ctx_likely = (int)(likely < slots ? likely : slots);
            }
            pl.ctx_wgs = (int)wgs;
        }
        finish();
        // Many-rows items because of what the cache holds, where the bound would not have them: with chunks of 12 tiles
        // and more, and spans short enough for half of the context wavefronts.  Their chunks take slots from the
        // contexts, whose spans get longer for it, and a short chunk leaves little to share.  Of 40 such steps that
        // were timed with either kind the rule takes the faster one or one within 13 %; always the many-rows kind
        // was up to twice as slow (173 requests of 32/8 heads, contexts of 19 .. 44, s = 1363, bound 3424, spans of 22
        // tiles: 108 us, 53 with the other kind; 84 of 32/8 heads of 64, s = 272, chunks of 5 tiles: 11.7 and 9.7), never
        // up to 1.5 times (99 of 40 heads, contexts of 78 .. 96, s = 8655: 122 us, 83 with chunks of 46 tiles).
        if (!tight && pl.rows_sys && !rows_pay(ctx_tiles) &&
            (pl.sys_chunk < 12 * 32 || (int64_t)pl.ctx_t_floor * pl.ctx_wgs * 4 > 2 * ctx_like)) {
            way.rows_by_bound = true;
            return make_plan(p, total_q, kind, max_q_len, sys_base_items, allow_rows_sys, budget, groups, way);
        }
        // Streaming chunks shorter than the bound's are no use where the launch waits for the contexts anyway: where a span
        // of the floor, in turns of a system workgroup (as estimated above), is longer than their turns.  Longer ones leave
        // the contexts more workgroups and more slots, and so shorter spans.  199 steps whose plan differs from the
        // bound's, with and without this: 0.98, up to 0.61 (6 requests of 32 heads, contexts of 126 .. 855 under 40032,
        // s = 6204: 69.7 -> 42.8 us; 6 of 52 heads, 156 .. 436, s = 768: 22.4 -> 18.9; 132 of 28/4, 9 .. 26 under 3280, s =
        // 1716: 36.2 -> 32.4), the worst 43.3 -> 47.1 (12 of 32/8, 571 .. 3904 under 40016, three prompts up to 5994).
        if (!tight && way.least_turns == 0 && !pl.rows_sys && pl.n_sys_chunks > few_chunks && few_chunks > 0 && p->ctx_part_tokens == 0) {
            double span = pl.ctx_t_floor * (0.9 + 3.0 / (t_item > 1 ? t_item : 1)) - 2.5;
            if (span < pl.ctx_t_floor) span = pl.ctx_t_floor;
            if (span > t_sys) {
                way.least_turns = (int64_t)ceil(span);
                return make_plan(p, total_q, kind, max_q_len, sys_base_items, allow_rows_sys, budget, groups, way);
            }
        }
        // A plan that outgrows the workspace or the static scratch takes no more than the bound's.
        if (!way.by_bound && pl.bytes > (budget < kStaticScratchBytes ? budget : kStaticScratchBytes)) {
            way.by_bound = true;
            const Plan bound = make_plan(p, total_q, kind, max_q_len, sys_base_items, allow_rows_sys, budget, groups, way);
            if (!bound.unsupported && bound.bytes < pl.bytes) return bound;
        }
        return pl;
    }

    const bool hand_set = p->sys_chunk_tokens != 0 || p->ctx_part_tokens != 0;
    PromptSplit split{false, 0, 256};
    if (prefill && !hand_set) split = split_prompt(p, total_q, pl.max_ctx, groups, tight);
    if ((!prefill && p->sys_len > 0) || (prefill && (hand_set || (tight && !split.whole)))) split = coarse_split(p, total_q);
    if (!prefill) split.part = 256;
    pl.whole = prefill && !hand_set && split.whole;
    if (p->sys_len > 0) {
        pl.sys_chunk = p->sys_chunk_tokens > 0 ? p->sys_chunk_tokens : split.chunk;
        pl.n_sys_chunks = ceil_div(p->sys_len, pl.sys_chunk);
    }
    if (pl.max_ctx > 0) {
        pl.ctx_part = p->ctx_part_tokens > 0 ? p->ctx_part_tokens : split.part;
        pl.n_ctx_parts = ceil_div(pl.max_ctx, pl.ctx_part);
        if (prefill) pl.n_ctx_likely = 1;       // (every context has a first part; many rows hide the trip)
        // a context part may touch at most kMaxPartBlocks blocks (the per-item block-id table in
        // LDS); parts start at multiples of ctx_part, which are block boundaries only when the
        // block size divides it
        const int touched = pl.ctx_part % p->block_size == 0
                                ? pl.ctx_part >> pl.block_size_log2
                                : ((pl.ctx_part - 1) >> pl.block_size_log2) + 2;
        if (touched > ra::kMaxPartBlocks) pl.unsupported = true;
    }
    finish();
    return pl;
}

// Decode launches of more than two workgroups per compute unit whose system workgroups all sit on units
// of their own: the context workgroups next to them are the last that should get work.
bool light_if_spare(int64_t sys_wgs, int64_t ctx_wgs) {
    const int cus = device_compute_units();
    return cus == kReferenceCus && sys_wgs > 0 && sys_wgs <= cus && sys_wgs + ctx_wgs > 2 * cus;
}

// A decode step small enough is one launch (decode_direct.hip): where the estimate of that form is below 14 us and
// below the two-launch form's, and no request takes too many rounds of its workgroup.  Both forms of 306 drawn
// steps (1 .. 64 requests and some to 256, 4 .. 52 query heads, prompts of 30 .. 3500 and some to 16000, contexts of 8 ..
// 3000 and some to 10000) were timed: 177 take this form, two of them at 1.04 and 1.05 of the two-launch time and
// the others faster (one request of 32/8 heads, s = 512, 10.2 -> 6.8 us; 16 of 16 heads of 64, s = 1000, contexts up to
// 255, 10.8 -> 7.8), and over all the choice is 1.7 % over the faster form.  The longest context is taken to be what
// the bound and the cache allow in the estimate, and half as long again as the cache makes likely in the rounds (4
// requests of 32 heads, s = 488, contexts of 353 .. 416 under 1072: 15.0 us in two launches, 11.1 in one).
//   Rounds: 16 wavefronts take 256 rows (head_dim 128; 512 at 64) of a request a round, and past the second a
// round costs 1.4 us (1 .. 2 rounds 5.3 us, 3 7.2, 4 8.8, 5 11, 6 12.3, 8 15.5).  So up to four are taken, up to six where
// three or fewer are context (those cost more, and the two-launch form spreads a context over the machine), and
// five where the two launches wait for memory.  Without these limits ten of the steps were more than 5 % slower in this
// form (10 requests of 8 heads, contexts of 287 .. 1540, 14.8 us in two launches and 19.3 in one).
//   Workgroups: 256 fit the machine.  As many again cost 1.3 us, and 1.8 without query groups, where two launches
// have no less to work on at once (50 requests of 16 heads of 64, s = 42, 7.9 us in two and 10.6 in one).
bool direct_form(const ra_params *p, int32_t total_q, int max_ctx, double sys_mean) {
    if (p->sys_chunk_tokens != 0 || p->ctx_part_tokens != 0 || total_q > 65535) return false;
    double held = (double)p->num_blocks * p->block_size;
    if (held < total_q) held = (double)total_q * max_ctx;            // (was not filled in)
    const double longest = held < max_ctx ? held : max_ctx, mean = held / total_q < max_ctx ? held / total_q : max_ctx;
    const double workgroups = (double)total_q * p->num_q_heads, row_bytes = 4.0 * p->head_dim;
    const int group = p->num_q_heads / p->num_kv_heads;
    const double tiles = ceil(total_q * (double)group / 32);
    const double mb = (tiles * sys_mean + total_q * mean) * p->num_kv_heads * row_bytes / 1e6;
    const double round = p->head_dim == 128 ? 256 : 512, reach = longest < 1.5 * mean ? longest : 1.5 * mean;
    if (p->sys_len + reach > (reach <= 3 * round ? 6 : mb > 60 ? 5 : 4) * round) return false;
    const double rate = p->head_dim == 128 ? 300 : 460;              // rows of a workgroup per us
    const double one = (p->sys_len + longest) / rate, even = (sys_mean + mean) / rate * workgroups / 256,
                 moved = workgroups * (sys_mean + mean) * row_bytes / 16.8e6;
    const double most = one > even ? (one > moved ? one : moved) : (even > moved ? even : moved);
    const double direct_us = 6.5 + most + (group > 1 ? 1.3 : 1.8) * (ceil(workgroups / 256) - 1);
    const double tile_us = 9.4 + mb / 8.9 + 0.34 * log2(1 + mb) + workgroups * 0.56e-3;
    return direct_us < 14 && direct_us < tile_us;
}

// Where the partial-attention launch records the begin and end of its wavefronts (measurement aid).
struct Timeline {
    unsigned long long *entries = nullptr;   // device, 2 per wavefront
    int waves = 0;
};

// The new key/value rows of a decode step that the attention launch writes into the cache itself.
struct NewRows {
    const void *k = nullptr, *v = nullptr;
    int64_t stride_token = 0, stride_head = 0;
};

ra_status run(const ra_params *p, const void *q, const int32_t *cu_seqlens_q, int32_t total_q,
              int32_t max_q_len,
              const void *k_sys, const void *v_sys, const void *k_cache, const void *v_cache,
              const int32_t *block_tables, const int32_t *context_lens, void *out,
              float *lse_out, void *workspace, size_t workspace_bytes, void *hip_stream,
              bool naive, int32_t num_prefixes = 0, const ra_prefix *prefixes = nullptr,
              int phases = 3, const NewRows *append = nullptr,
              const int32_t *req_order = nullptr, const int32_t *req_prefix = nullptr,
              const int32_t *prefix_num_tokens = nullptr, const Timeline *timeline = nullptr) {
    ra_status st = check_params(p, total_q);
    if (st != RA_OK) return st;
    if (naive && p->sys_len != 0) return RA_ERR_INVALID_ARG;
    if (append) {
        if (append->stride_token < 0 || append->stride_head < 0 || append->stride_token % 8 ||
            append->stride_head % 8)
            return RA_ERR_INVALID_ARG;
        if (total_q > 0 && (!append->k || !append->v || !aligned16(append->k) || !aligned16(append->v)))
            return RA_ERR_INVALID_ARG;
        if (append->stride_head < p->head_dim && p->num_kv_heads > 1) return RA_ERR_INVALID_ARG;
    }
    const int kWorkgroupSlots = device_compute_units() * 2;
    // Shared prefixes of the batch: one (the paper's setting) unless the caller lists several.
    ra_prefix one{k_sys, v_sys, p->sys_len, 0, total_q};
    if (!prefixes) {
        prefixes = &one;
        num_prefixes = 1;
    }
    // the run of tokens each prefix owns: its requests in a decode step, their new tokens in the
    // prompt phase (where the caller says how many those are)
    int tok0[ra::kMaxPrefixes], ntok[ra::kMaxPrefixes];
    for (int i = 0, at = 0; i < num_prefixes && i < ra::kMaxPrefixes; ++i) {
        tok0[i] = prefix_num_tokens ? at : prefixes[i].first_request;
        ntok[i] = prefix_num_tokens ? prefix_num_tokens[i] : prefixes[i].num_requests;
        at += ntok[i];
    }
    int64_t sys_base_items = 0;
    bool read_once = true;
    for (int i = 0; i < num_prefixes; ++i) {
        const int mt = ceil_div(prefixes[i].num_requests * (p->num_q_heads / p->num_kv_heads), 32);
        sys_base_items += (int64_t)p->num_kv_heads * mt;
        if (mt > 1) read_once = false;          // several row tiles re-read the same K/V
    }
    const PlanKind kind = cu_seqlens_q ? kPrefill : naive ? kNaiveDecode : kRelayDecode;
    // A caller sizes the workspace without knowing the grouping; should the grouping-aware plan
    // need more than that, a decode step takes the fewest slots with it (the blind plan does not count the
    // prefixes' workgroups and launched more than the machine holds: 19 requests of 40 heads, two prompts
    // of 1989 and 2830, 60.5 against 39.3 us), and otherwise the grouping-blind one (which is what the size
    // was computed from) is used.
    // Where the workspace is smaller than either, the cut with the fewest partials may still fit it.
    const bool multi = num_prefixes > 1;
    // (There the whole prompt form, which needs no workspace, is also taken where only the mean over the prefixes is for it.)
    Groups groups{0, 0}, by_prefix{0, (double)p->batch / (num_prefixes > 0 ? num_prefixes : 1)};
    for (int i = 0; i < num_prefixes && i < ra::kMaxPrefixes && total_q > 0; ++i) {
        groups.sys_len += (double)prefixes[i].sys_len * ntok[i] / total_q;
        groups.requests += (double)prefixes[i].num_requests * ntok[i] / total_q;
        by_prefix.sys_len += (double)prefixes[i].sys_len / num_prefixes;
    }
    Plan pl{};
    for (size_t budget : {SIZE_MAX, workspace_bytes}) {
        const Groups &shared = budget == SIZE_MAX ? groups : by_prefix;
        pl = make_plan(p, total_q, kind, max_q_len, multi ? sys_base_items : 0, true, budget, multi ? shared : Groups{});
        if (multi && kind == kRelayDecode && !pl.unsupported && pl.bytes > workspace_bytes)
            pl = make_plan(p, total_q, kind, max_q_len, sys_base_items, true, workspace_bytes);
        if (multi && !pl.unsupported && pl.bytes > workspace_bytes)
            pl = make_plan(p, total_q, kind, max_q_len, 0, false, budget);
        if (pl.unsupported || pl.bytes <= workspace_bytes) break;
    }
    if (pl.unsupported) return RA_ERR_UNSUPPORTED;
    if (total_q > 0) {
        if (!q || !out || !context_lens) return RA_ERR_INVALID_ARG;
        if (!aligned16(q) || !aligned16(out)) return RA_ERR_INVALID_ARG;
        if (p->sys_len > 0 && (!k_sys || !v_sys || !aligned16(k_sys) || !aligned16(v_sys)))
            return RA_ERR_INVALID_ARG;
        if (pl.max_ctx > 0 &&
            (!k_cache || !v_cache || !block_tables || !aligned16(k_cache) || !aligned16(v_cache)))
            return RA_ERR_INVALID_ARG;
        if (p->q_stride_head < p->head_dim || p->o_stride_head < p->head_dim ||
            (p->sys_len > 1 && p->sys_stride_token < p->head_dim))
            return RA_ERR_INVALID_ARG;
    }
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)
        return RA_ERR_INVALID_ARG;
    if (workspace_bytes < pl.bytes) return RA_ERR_WORKSPACE_TOO_SMALL;
    if (total_q == 0) return RA_OK;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    float *part_o = reinterpret_cast<float *>(ws + pl.off_o);
    float *part_lse = reinterpret_cast<float *>(ws + pl.off_lse);
    const float scale_log2 = p->softmax_scale * 1.4426950408889634f;
    const int mask = phases;

    // A per-request paged pass over a short sequence needs no workspace round trip.
    const bool direct = naive && pl.n_sys_chunks == 0 && pl.n_ctx_parts == 1;

    const bool prefill = cu_seqlens_q != nullptr;
    const int head_fastest = p->sys_stride_head < p->sys_stride_token ? 1 : 0;

    // A small decode step in one launch.  (A timeline is one of the two-launch form: it is taken of the partial
    // attention, and the result is this form's all the same.)
    const bool direct_step = !naive && !prefill && mask == 3 && direct_form(p, total_q, pl.max_ctx, groups.sys_len);
    auto launch_direct_step = [&]() -> ra_status {
        ra::DirectArgs d{};
        d.q = static_cast<const uint16_t *>(q);
        d.k_cache = static_cast<const uint16_t *>(k_cache);
        d.v_cache = static_cast<const uint16_t *>(v_cache);
        if (append) {
            d.k_new = static_cast<const uint16_t *>(append->k);
            d.v_new = static_cast<const uint16_t *>(append->v);
            d.new_stride_token = append->stride_token;
            d.new_stride_head = append->stride_head;
        }
        d.block_tables = block_tables;
        d.context_lens = context_lens;
        d.out = out;
        d.lse_out = lse_out;
        d.q_stride_token = p->q_stride_token;
        d.q_stride_head = p->q_stride_head;
        d.o_stride_token = p->o_stride_token;
        d.o_stride_head = p->o_stride_head;
        d.sys_stride_token = p->sys_stride_token;
        d.sys_stride_head = p->sys_stride_head;
        d.n_tokens = total_q;
        d.Hq = p->num_q_heads;
        d.Hkv = p->num_kv_heads;
        d.G = pl.group;
        d.max_ctx = pl.max_ctx;
        d.block_size_log2 = pl.block_size_log2;
        d.max_blocks_per_seq = p->max_blocks_per_seq;
        d.out_is_fp32 = p->out_is_fp32;
        d.scale_log2 = scale_log2;
        ra::DirectOne one{static_cast<const uint16_t *>(prefixes[0].k_sys),
                          static_cast<const uint16_t *>(prefixes[0].v_sys), prefixes[0].sys_len};
        ra::DirectMany many{};
        if (num_prefixes > 1) {
            many.n = num_prefixes;
            many.req_prefix = req_prefix;
            for (int i = 0; i < num_prefixes; ++i) {
                many.token_end[i] = tok0[i] + ntok[i];
                many.len[i] = prefixes[i].sys_len;
                many.k[i] = static_cast<const uint16_t *>(prefixes[i].k_sys);
                many.v[i] = static_cast<const uint16_t *>(prefixes[i].v_sys);
            }
        }
        return ra::launch_decode_direct(d, num_prefixes > 1 ? nullptr : &one, num_prefixes > 1 ? &many : nullptr,
                                        p->head_dim, stream) == hipSuccess ? RA_OK : RA_ERR_HIP;
    };
    if (direct_step && !timeline) return launch_direct_step();

    // Prompt phase in ONE launch: a work item carries its 128 rows through the system prompt and then
    // through the contexts of the requests they belong to, and writes the output itself; no
    // partials, no fusion launch.  split_prompt says when; the split form stays whenever the
    // caller tunes the decomposition by hand or asks for one phase only.
    const bool whole = prefill && !naive && pl.whole && mask == 3;
    // Many stacked rows per kv head (prompt phase; wide GQA decode batches): the many-rows kernel
    // takes the system part and, in the prompt phase, the causal context part as well.
    if ((mask & 1) && !naive && pl.rows_path) {
        ra::RowsArgs r{};
        r.q = static_cast<const uint16_t *>(q);
        r.k_sys = static_cast<const uint16_t *>(k_sys);
        r.v_sys = static_cast<const uint16_t *>(v_sys);
        r.k_cache = static_cast<const uint16_t *>(k_cache);
        r.v_cache = static_cast<const uint16_t *>(v_cache);
        r.block_tables = block_tables;
        r.context_lens = context_lens;
        r.cu_seqlens_q = cu_seqlens_q;
        r.part_o = part_o;
        r.part_lse = part_lse;
        r.q_stride_token = p->q_stride_token;
        r.q_stride_head = p->q_stride_head;
        r.sys_stride_token = p->sys_stride_token;
        r.sys_stride_head = p->sys_stride_head;
        r.n_tokens = total_q;
        r.Hq = p->num_q_heads;
        r.Hkv = p->num_kv_heads;
        r.G = pl.group;
        r.sys_len = p->sys_len;
        r.sys_chunk = pl.sys_chunk;
        r.n_sys_chunks = pl.n_sys_chunks;
        r.n_sys_rowblocks = pl.n_sys_rowblocks;
        r.n_sys_items = p->num_kv_heads * pl.n_sys_rowblocks * pl.n_sys_chunks;
        r.ctx_part = pl.ctx_part;
        r.n_ctx_parts = pl.n_ctx_parts;
        r.n_ctx_rowblocks = pl.n_ctx_rowblocks;
        r.n_ctx_items = prefill ? p->batch * p->num_kv_heads * pl.n_ctx_rowblocks * pl.n_ctx_parts : 0;
        r.block_size_log2 = pl.block_size_log2;
        r.max_blocks_per_seq = p->max_blocks_per_seq;
        r.rows = pl.rows;
        r.sys_head_fastest = head_fastest;
        r.scale_log2 = scale_log2;
        r.n_prefixes = num_prefixes;
        r.batch = p->batch;
        r.whole = whole ? 1 : 0;
        if (whole) {
            // one item per (kv head, block of 128 stacked rows) that goes through the system prompt
            // and the contexts and writes the output rows itself
            r.out = out;
            r.lse_out = lse_out;
            r.o_stride_token = p->o_stride_token;
            r.o_stride_head = p->o_stride_head;
            r.out_is_fp32 = p->out_is_fp32;
            r.n_sys_chunks = 1;
            r.sys_chunk = p->sys_len > 0 ? pl.sys_chunk : 1;
            r.n_sys_items = p->num_kv_heads * pl.n_sys_rowblocks;
            r.n_ctx_items = 0;
            if (r.n_ctx_parts < 1 || r.ctx_part < 1) r.n_ctx_parts = 0, r.ctx_part = 1;   // no context at all
        }
        if (num_prefixes > 1) {                    // system items prefix by prefix
            // Whole items start with the longest prompt's, which the launch would wait for, where there are more than the
            // machine holds at once (800 items of 1304 .. 1616 positions 0.93 of the time, 764 of 870 .. 2933 0.94) or
            // prompts are long (476 items of 2712 .. 10379 0.92, 296 of 3436 .. 8295 0.87).  Short ones that all start
            // together only change which of them share a unit: between 0.92 and 1.04 of 8 such launches, three
            // prompts of 300 .. 2000 68.0 us as given and 69.4 by length; the line lies between 2600 and 8300.
            int by_len[ra::kMaxPrefixes], whole_items = 0, longest = 0;
            for (int i = 0; whole && i < num_prefixes; ++i) {
                whole_items += p->num_kv_heads * ceil_div(ntok[i] * pl.group, 128);
                if (prefixes[i].sys_len > longest) longest = prefixes[i].sys_len;
            }
            const bool sorted = whole_items > 2 * device_compute_units() || longest >= 4096;
            for (int i = 0; i < num_prefixes; ++i) {
                int at = i;
                for (; sorted && at > 0 && prefixes[by_len[at - 1]].sys_len < prefixes[i].sys_len; --at) by_len[at] = by_len[at - 1];
                by_len[at] = i;
            }
            int items = 0;
            for (int at = 0; at < num_prefixes; ++at) {
                const int i = by_len[at];
                items += p->num_kv_heads * ceil_div(ntok[i] * pl.group, 128) *
                         (whole ? 1 : pl.sys_chunk > 0 ? ceil_div(prefixes[i].sys_len, pl.sys_chunk) : 0);
                r.pfx_item_end[at] = items;
                r.pfx_tok0[at] = tok0[i];
                r.pfx_ntok[at] = ntok[i];
                r.pfx_len[at] = prefixes[i].sys_len;
                r.pfx_k[at] = static_cast<const uint16_t *>(prefixes[i].k_sys);
                r.pfx_v[at] = static_cast<const uint16_t *>(prefixes[i].v_sys);
            }
            r.n_sys_items = items;
        }
        if (timeline && prefill) r.timeline = timeline->entries, r.timeline_waves = timeline->waves;
        if (ra::launch_relay_rows(r, p->head_dim, stream) != hipSuccess) return RA_ERR_HIP;
    }
    // Decode: system chunks (unless the many-rows kernel took them) and context parts in one
    // launch of the streaming tile kernel.
    if ((mask & 1) && !naive && !prefill) {
        ra::TileArgs t{};
        t.q = static_cast<const uint16_t *>(q);
        t.k_cache = static_cast<const uint16_t *>(k_cache);
        t.v_cache = static_cast<const uint16_t *>(v_cache);
        if (append) {
            t.k_new = static_cast<const uint16_t *>(append->k);
            t.v_new = static_cast<const uint16_t *>(append->v);
            t.new_stride_token = append->stride_token;
            t.new_stride_head = append->stride_head;
        }
        t.req_order = num_prefixes > 1 ? req_order : nullptr;
        t.block_tables = block_tables;
        t.context_lens = context_lens;
        t.part_o = part_o;
        t.part_lse = part_lse;
        t.q_stride_token = p->q_stride_token;
        t.q_stride_head = p->q_stride_head;
        t.sys_stride_token = p->sys_stride_token;
        t.sys_stride_head = p->sys_stride_head;
        t.n_tokens = total_q;
        t.Hq = p->num_q_heads;
        t.Hkv = p->num_kv_heads;
        t.G = pl.group;
        t.sys_chunk = pl.sys_chunk > 0 ? pl.sys_chunk : 128;
        t.n_sys_chunks = pl.n_sys_chunks;
        t.n_prefixes = num_prefixes;
        t.n_sys_rowblocks = pl.rows_sys ? pl.n_sys_rowblocks : 0;
        int items = 0;
        for (int i = 0; i < num_prefixes; ++i) {
            const int mt = pl.rows_sys ? pl.n_sys_rowblocks
                                       : ceil_div(prefixes[i].num_requests * pl.group, 32);
            items += p->num_kv_heads * mt * ceil_div(prefixes[i].sys_len, t.sys_chunk);
            t.pfx_item_end[i] = items;
            t.pfx_first[i] = prefixes[i].first_request;
            t.pfx_tokens[i] = prefixes[i].num_requests;
            t.pfx_len[i] = prefixes[i].sys_len;
            t.pfx_k[i] = static_cast<const uint16_t *>(prefixes[i].k_sys);
            t.pfx_v[i] = static_cast<const uint16_t *>(prefixes[i].v_sys);
        }
        t.n_sys_items = items;
        t.sys_read_once = read_once ? 1 : 0;
        t.ctx_waves = pl.ctx_wgs * 4;
        t.ctx_t_floor = pl.ctx_t_floor;
        {
            const int64_t cap = ((int64_t)ra::kMaxPartBlocks - 1) * p->block_size / 32;
            t.ctx_t_cap = (int)(cap < 1 ? 1 : cap > INT32_MAX / 2 ? INT32_MAX / 2 : cap);
        }
        t.n_ctx_slots = pl.n_ctx_parts;
        t.max_ctx = pl.max_ctx;
        // Workgroups i and i + 256 of a 512-workgroup grid share a compute unit: the context
        // workgroups 256 .. 256 + n_sys - 1 sit next to a system workgroup.
        if (pl.paired && items + pl.ctx_wgs == kWorkgroupSlots && items <= kWorkgroupSlots / 2) {
            t.ctx_light_begin = (kWorkgroupSlots / 2 - items) * 4;
            t.ctx_light_waves = items * 4;
            t.sys_wg_tiles = ceil_div(t.sys_chunk, 32);
            int64_t sum = 0;
            for (int i = 0; i < num_prefixes; ++i)      // (tiles fetched, once per workgroup)
                sum += (int64_t)p->num_kv_heads *
                       (pl.rows_sys ? pl.n_sys_rowblocks : ceil_div(prefixes[i].num_requests * pl.group, 32)) *
                       ceil_div(prefixes[i].sys_len, 32);
            t.sys_tiles_total = (int)(sum > INT32_MAX / 2 ? INT32_MAX / 2 : sum);
        } else if (light_if_spare(items, pl.ctx_wgs)) {
            t.ctx_light_begin = (kWorkgroupSlots / 2 - items) * 4;
            t.ctx_light_waves = items * 4;
            t.sys_wg_tiles = INT32_MAX / 2;             // (more than any unit: no light span)
            t.sys_tiles_total = 0;
        }
        t.block_size_log2 = pl.block_size_log2;
        t.max_blocks_per_seq = p->max_blocks_per_seq;
        t.rows = pl.rows;
        t.sys_head_fastest = head_fastest;
        t.scale_log2 = scale_log2;
        if (timeline) t.timeline = timeline->entries, t.timeline_waves = timeline->waves;
        if (ra::launch_relay_tiles(t, p->head_dim, stream) != hipSuccess) return RA_ERR_HIP;
        if (direct_step) return launch_direct_step();
    }
    // The per-request comparison path.
    if ((mask & 1) && naive) {
        if (pl.n_ctx_parts > 0) {
            ra::CtxArgs c{};
            c.q = static_cast<const uint16_t *>(q);
            c.k_cache = static_cast<const uint16_t *>(k_cache);
            c.v_cache = static_cast<const uint16_t *>(v_cache);
            c.block_tables = block_tables;
            c.context_lens = context_lens;
            c.cu_seqlens_q = nullptr;
            c.part_o = part_o + (size_t)pl.n_sys_chunks * pl.rows * p->head_dim;
            c.part_lse = part_lse + (size_t)pl.n_sys_chunks * pl.rows;
            c.out = out;
            c.lse_out = lse_out;
            c.q_stride_token = p->q_stride_token;
            c.q_stride_head = p->q_stride_head;
            c.o_stride_token = p->o_stride_token;
            c.o_stride_head = p->o_stride_head;
            c.batch = p->batch;
            c.n_tokens = total_q;
            c.Hq = p->num_q_heads;
            c.Hkv = p->num_kv_heads;
            c.block_size_log2 = pl.block_size_log2;
            c.max_blocks_per_seq = p->max_blocks_per_seq;
            c.part_tokens = pl.ctx_part;
            c.n_parts = pl.n_ctx_parts;
            c.rows = pl.rows;
            c.direct = direct ? 1 : 0;
            c.out_is_fp32 = p->out_is_fp32;
            c.scale_log2 = scale_log2;
            if (ra::launch_ctx_decode(c, p->head_dim, pl.group, stream) != hipSuccess)
                return RA_ERR_HIP;
        }
    }
    if ((mask & 2) && !direct && !whole) {
        ra::FuseArgs f{};
        f.part_o = part_o;
        f.part_lse = part_lse;
        f.out = out;
        f.lse_out = lse_out;
        f.o_stride_token = p->o_stride_token;
        f.o_stride_head = p->o_stride_head;
        f.rows = pl.rows;
        f.Hq = p->num_q_heads;
        f.n_partials = pl.n_sys_chunks + pl.n_ctx_parts;
        f.n_likely = pl.n_sys_chunks + (pl.n_ctx_likely > 0 ? pl.n_ctx_likely : pl.n_ctx_parts);
        f.n_sys_chunks = pl.n_sys_chunks;
        f.n_prefixes = num_prefixes;
        f.req_prefix = num_prefixes > 1 ? req_prefix : nullptr;
        for (int i = 0; i < num_prefixes; ++i) {
            f.pfx_token_end[i] = tok0[i] + ntok[i];
            f.pfx_chunks[i] = pl.sys_chunk > 0 ? ceil_div(prefixes[i].sys_len, pl.sys_chunk) : 0;
        }
        f.out_is_fp32 = p->out_is_fp32;
        if (ra::launch_fuse(f, p->head_dim, stream) != hipSuccess) return RA_ERR_HIP;
    }
    return RA_OK;
}

}  // namespace

extern "C" {

size_t relay_attn_workspace_bytes(const ra_params *p, int32_t total_q) {
    if (check_params(p, total_q) != RA_OK) return 0;
    // the caller does not say which entry point will use the workspace: cover both
    size_t most = 0;
    for (PlanKind kind : {kRelayDecode, kNaiveDecode, kPrefill}) {
        const Plan pl = make_plan(p, total_q, kind, kind == kPrefill ? total_q : 1);
        if (!pl.unsupported && pl.bytes > most) most = pl.bytes;
    }
    // (a call with several prefixes may fall back to the decode plan without many-rows items)
    const Plan blind = make_plan(p, total_q, kRelayDecode, 1, 0, false);
    if (!blind.unsupported && blind.bytes > most) most = blind.bytes;
    // (and a workspace serves calls over a cache of another size)
    for (const bool rows_sys : {true, false}) {
        const Plan bound = make_plan(p, total_q, kRelayDecode, 1, 0, rows_sys, SIZE_MAX, {}, DecodeWay{true});
        if (!bound.unsupported && bound.bytes > most) most = bound.bytes;
    }
    return most;
}

ra_status relay_attn_decode_plan(const ra_params *p, ra_decode_plan *plan) {
    if (!plan) return RA_ERR_INVALID_ARG;
    const ra_status st = check_params(p, p ? p->batch : 0);
    if (st != RA_OK) return st;
    const Plan pl = make_plan(p, p->batch, kRelayDecode, 1);
    if (pl.unsupported) return RA_ERR_UNSUPPORTED;
    plan->sys_chunk_tokens = pl.sys_chunk;
    plan->num_sys_chunks = pl.n_sys_chunks;
    plan->sys_rows_per_workgroup = pl.rows_sys ? 128 : 32;
    plan->num_sys_workgroups =
        p->num_kv_heads * (pl.rows_sys ? pl.n_sys_rowblocks : pl.n_mtiles) * pl.n_sys_chunks;
    plan->num_ctx_wavefronts = pl.ctx_wgs * 4;
    plan->min_tiles_per_ctx_wavefront = pl.ctx_t_floor;
    plan->num_ctx_slots = pl.n_ctx_parts;
    plan->max_blocks_per_span = ra::kMaxPartBlocks;
    plan->first_light_ctx_wavefront = 0;
    plan->num_light_ctx_wavefronts = 0;
    plan->compute_units = device_compute_units();
    const int kWorkgroupSlots = plan->compute_units * 2;
    plan->sys_workgroup_tiles = pl.sys_chunk > 0 ? ceil_div(pl.sys_chunk, 32) : 0;
    plan->sys_tiles_total = p->num_kv_heads * (pl.rows_sys ? pl.n_sys_rowblocks : pl.n_mtiles) *
                            ceil_div(p->sys_len, 32);
    if (pl.paired && plan->num_sys_workgroups + pl.ctx_wgs == kWorkgroupSlots &&
        plan->num_sys_workgroups <= kWorkgroupSlots / 2) {
        plan->first_light_ctx_wavefront = (kWorkgroupSlots / 2 - plan->num_sys_workgroups) * 4;
        plan->num_light_ctx_wavefronts = plan->num_sys_workgroups * 4;
    } else if (light_if_spare(plan->num_sys_workgroups, pl.ctx_wgs)) {
        plan->first_light_ctx_wavefront = (kWorkgroupSlots / 2 - plan->num_sys_workgroups) * 4;
        plan->num_light_ctx_wavefronts = plan->num_sys_workgroups * 4;
    }
    return RA_OK;
}

ra_status relay_attn_decode(const ra_params *p, const void *q, const void *k_sys,
                            const void *v_sys, const void *k_cache, const void *v_cache,
                            const int32_t *block_tables, const int32_t *context_lens, void *out,
                            float *lse_out, void *workspace, size_t workspace_bytes,
                            void *hip_stream) {
    if (!p) return RA_ERR_INVALID_ARG;
    return run(p, q, nullptr, p->batch, 1, k_sys, v_sys, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, workspace, workspace_bytes, hip_stream, false);
}

ra_status relay_attn_decode_append(const ra_params *p, const void *q, const void *k_new,
                                   const void *v_new, int64_t new_stride_token,
                                   int64_t new_stride_head, const void *k_sys, const void *v_sys,
                                   void *k_cache, void *v_cache, const int32_t *block_tables,
                                   const int32_t *context_lens, void *out, float *lse_out,
                                   void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!p) return RA_ERR_INVALID_ARG;
    NewRows rows;
    rows.k = k_new;
    rows.v = v_new;
    rows.stride_token = new_stride_token;
    rows.stride_head = new_stride_head;
    return run(p, q, nullptr, p->batch, 1, k_sys, v_sys, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, workspace, workspace_bytes, hip_stream, false, 0, nullptr,
               3, &rows);
}

size_t relay_attn_static_scratch_bytes(void) { return kStaticScratchBytes; }

ra_status relay_attn_decode_static(const ra_params *p, const void *q, const void *k_sys,
                                   const void *v_sys, const void *k_cache, const void *v_cache,
                                   const int32_t *block_tables, const int32_t *context_lens,
                                   void *out, float *lse_out, void *hip_stream) {
    if (!p) return RA_ERR_INVALID_ARG;
    ra_status st = check_params(p, p->batch);
    if (st != RA_OK) return st;
    // the same decomposition relay_attn_decode uses, so the same kernels and the same result
    const Plan pl = make_plan(p, p->batch, kRelayDecode, 1);
    if (pl.unsupported) return RA_ERR_UNSUPPORTED;
    if (pl.bytes > kStaticScratchBytes) return RA_ERR_WORKSPACE_TOO_SMALL;
    if (p->batch == 0) return RA_OK;
    void *ws = nullptr;
    st = static_scratch(&ws);
    if (st != RA_OK) return st;
    return run(p, q, nullptr, p->batch, 1, k_sys, v_sys, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, ws, kStaticScratchBytes, hip_stream, false);
}

ra_status relay_attn_debug_decode_phases(const ra_params *p, int32_t phases, const void *q,
                                         const void *k_sys, const void *v_sys, const void *k_cache,
                                         const void *v_cache, const int32_t *block_tables,
                                         const int32_t *context_lens, void *out, float *lse_out,
                                         void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!p || phases < 1 || phases > 3) return RA_ERR_INVALID_ARG;
    return run(p, q, nullptr, p->batch, 1, k_sys, v_sys, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, workspace, workspace_bytes, hip_stream, false, 0, nullptr,
               phases);
}

ra_status relay_attn_debug_timeline(const ra_params *p, const void *q, const int32_t *cu_seqlens_q,
                                    int32_t total_q, int32_t max_q_len, const void *k_sys,
                                    const void *v_sys, const void *k_cache, const void *v_cache,
                                    const int32_t *block_tables, const int32_t *context_lens,
                                    void *out, float *lse_out, void *workspace,
                                    size_t workspace_bytes, uint64_t *timeline,
                                    int32_t timeline_wavefronts, void *hip_stream) {
    if (!p || !timeline || timeline_wavefronts < 1 || (reinterpret_cast<uintptr_t>(timeline) & 7u))
        return RA_ERR_INVALID_ARG;
    if (!cu_seqlens_q && (total_q != p->batch || max_q_len != 1)) return RA_ERR_INVALID_ARG;
    Timeline tl;
    tl.entries = reinterpret_cast<unsigned long long *>(timeline);
    tl.waves = timeline_wavefronts;
    return run(p, q, cu_seqlens_q, total_q, max_q_len, k_sys, v_sys, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, workspace, workspace_bytes, hip_stream, false, 0, nullptr, 3,
               nullptr, nullptr, nullptr, nullptr, &tl);
}

ra_status relay_attn_decode_multi(const ra_params *p, int32_t num_prefixes,
                                  const ra_prefix *prefixes, const void *q, const void *k_cache,
                                  const void *v_cache, const int32_t *block_tables,
                                  const int32_t *context_lens, void *out, float *lse_out,
                                  void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!p || !prefixes || num_prefixes < 1) return RA_ERR_INVALID_ARG;
    if (num_prefixes > ra::kMaxPrefixes) return RA_ERR_UNSUPPORTED;
    int next = 0, longest = 0, longest_at = 0;
    for (int i = 0; i < num_prefixes; ++i) {           // groups tile the batch, in order
        const ra_prefix &f = prefixes[i];
        if (f.first_request != next || f.num_requests < 1 || f.sys_len < 0) return RA_ERR_INVALID_ARG;
        if (f.sys_len > 0 && (!f.k_sys || !f.v_sys || !aligned16(f.k_sys) || !aligned16(f.v_sys)))
            return RA_ERR_INVALID_ARG;
        next += f.num_requests;
        if (f.sys_len > longest) longest = f.sys_len, longest_at = i;
    }
    if (next != p->batch || longest != p->sys_len) return RA_ERR_INVALID_ARG;
    return run(p, q, nullptr, p->batch, 1, prefixes[longest_at].k_sys, prefixes[longest_at].v_sys,
               k_cache, v_cache,
               block_tables, context_lens, out, lse_out, workspace, workspace_bytes, hip_stream,
               false, num_prefixes, prefixes);
}

ra_status relay_attn_group_requests(const int32_t *sys_id, int32_t batch, int32_t num_prefixes,
                                    int32_t *request_order, int32_t *num_requests) {
    if (batch < 0 || num_prefixes < 1 || !num_requests || (batch > 0 && (!sys_id || !request_order)))
        return RA_ERR_INVALID_ARG;
    for (int i = 0; i < num_prefixes; ++i) num_requests[i] = 0;
    for (int r = 0; r < batch; ++r) {
        if (sys_id[r] < 0 || sys_id[r] >= num_prefixes) return RA_ERR_INVALID_ARG;
        ++num_requests[sys_id[r]];
    }
    // counting sort: the requests of prefix 0 in batch order, then those of prefix 1, ...
    int32_t at = 0;
    for (int i = 0; i < num_prefixes; ++i) {
        for (int r = 0; r < batch; ++r)
            if (sys_id[r] == i) request_order[at++] = r;
    }
    return RA_OK;
}

ra_status relay_attn_decode_grouped(const ra_params *p, int32_t num_prefixes,
                                    const ra_prefix *prefixes, const int32_t *sys_id,
                                    const int32_t *request_order, const void *q,
                                    const void *k_cache, const void *v_cache,
                                    const int32_t *block_tables, const int32_t *context_lens,
                                    void *out, float *lse_out, void *workspace,
                                    size_t workspace_bytes, void *hip_stream) {
    if (!p || !prefixes || num_prefixes < 1) return RA_ERR_INVALID_ARG;
    if (num_prefixes > ra::kMaxPrefixes) return RA_ERR_UNSUPPORTED;
    if (p->batch > 0 && (!sys_id || !request_order)) return RA_ERR_INVALID_ARG;
    // the same per-prefix table as relay_attn_decode_multi, with runs of request_order in place of
    // runs of the batch
    ra_prefix used[ra::kMaxPrefixes];
    int n_used = 0, next = 0, longest = 0, longest_at = -1;
    for (int i = 0; i < num_prefixes; ++i) {
        const ra_prefix &f = prefixes[i];
        if (f.num_requests < 0 || f.sys_len < 0) return RA_ERR_INVALID_ARG;
        if (f.sys_len > 0 && (!f.k_sys || !f.v_sys || !aligned16(f.k_sys) || !aligned16(f.v_sys)))
            return RA_ERR_INVALID_ARG;
        // (the fusion launch looks chunk counts up by sys_id, so the table keeps every prefix, with
        // zero requests where none uses it)
        used[n_used] = f;
        used[n_used].first_request = next;
        ++n_used;
        next += f.num_requests;
        if (f.num_requests > 0 && f.sys_len >= longest) {
            if (f.sys_len > longest || longest_at < 0) longest_at = i;
            longest = f.sys_len;
        }
    }
    if (next != p->batch || longest != p->sys_len) return RA_ERR_INVALID_ARG;
    if (p->batch == 0) longest_at = 0;
    return run(p, q, nullptr, p->batch, 1, prefixes[longest_at].k_sys, prefixes[longest_at].v_sys,
               k_cache, v_cache, block_tables, context_lens, out, lse_out, workspace,
               workspace_bytes, hip_stream, false, n_used, used, 3, nullptr, request_order, sys_id);
}

ra_status relay_attn_prefill(const ra_params *p, const void *q, const int32_t *cu_seqlens_q,
                             int32_t total_q, int32_t max_q_len, const void *k_sys,
                             const void *v_sys, const void *k_cache, const void *v_cache,
                             const int32_t *block_tables, const int32_t *context_lens, void *out,
                             float *lse_out, void *workspace, size_t workspace_bytes,
                             void *hip_stream) {
    if (!p || max_q_len < 0 || total_q < 0) return RA_ERR_INVALID_ARG;
    if (total_q > 0 && (!cu_seqlens_q || p->batch < 1)) return RA_ERR_INVALID_ARG;
    if ((int64_t)max_q_len * p->batch < total_q) return RA_ERR_INVALID_ARG;
    return run(p, q, cu_seqlens_q, total_q, max_q_len, k_sys, v_sys, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, workspace, workspace_bytes, hip_stream, false);
}

ra_status relay_attn_prefill_multi(const ra_params *p, int32_t num_prefixes,
                                   const ra_prefix *prefixes, const int32_t *prefix_num_tokens,
                                   const void *q, const int32_t *cu_seqlens_q, int32_t total_q,
                                   int32_t max_q_len, const void *k_cache, const void *v_cache,
                                   const int32_t *block_tables, const int32_t *context_lens,
                                   void *out, float *lse_out, void *workspace,
                                   size_t workspace_bytes, void *hip_stream) {
    if (!p || !prefixes || !prefix_num_tokens || num_prefixes < 1 || max_q_len < 0 || total_q < 0)
        return RA_ERR_INVALID_ARG;
    if (num_prefixes > ra::kMaxPrefixes) return RA_ERR_UNSUPPORTED;
    if (total_q > 0 && (!cu_seqlens_q || p->batch < 1)) return RA_ERR_INVALID_ARG;
    if ((int64_t)max_q_len * p->batch < total_q) return RA_ERR_INVALID_ARG;
    int next = 0, longest = 0, longest_at = 0;
    int64_t tokens = 0;
    for (int i = 0; i < num_prefixes; ++i) {           // groups tile the batch, in order
        const ra_prefix &f = prefixes[i];
        if (f.first_request != next || f.num_requests < 1 || f.sys_len < 0) return RA_ERR_INVALID_ARG;
        if (prefix_num_tokens[i] < 0 || (int64_t)prefix_num_tokens[i] > (int64_t)f.num_requests * max_q_len)
            return RA_ERR_INVALID_ARG;
        if (f.sys_len > 0 && (!f.k_sys || !f.v_sys || !aligned16(f.k_sys) || !aligned16(f.v_sys)))
            return RA_ERR_INVALID_ARG;
        next += f.num_requests;
        tokens += prefix_num_tokens[i];
        if (f.sys_len > longest) longest = f.sys_len, longest_at = i;
    }
    if (next != p->batch || tokens != total_q || longest != p->sys_len) return RA_ERR_INVALID_ARG;
    if (total_q == 0 && !cu_seqlens_q) {
        // (run() tells the prompt phase from decode by this pointer; an empty call has nothing to do)
        const ra_status st = check_params(p, 0);
        return st;
    }
    return run(p, q, cu_seqlens_q, total_q, max_q_len, prefixes[longest_at].k_sys,
               prefixes[longest_at].v_sys, k_cache, v_cache, block_tables, context_lens, out, lse_out,
               workspace, workspace_bytes, hip_stream, false, num_prefixes, prefixes, 3, nullptr,
               nullptr, nullptr, prefix_num_tokens);
}

ra_status paged_attn_decode_naive(const ra_params *p, const void *q, const void *k_cache,
                                  const void *v_cache, const int32_t *block_tables,
                                  const int32_t *context_lens, void *out, float *lse_out,
                                  void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!p) return RA_ERR_INVALID_ARG;
    return run(p, q, nullptr, p->batch, 1, nullptr, nullptr, k_cache, v_cache, block_tables,
               context_lens, out, lse_out, workspace, workspace_bytes, hip_stream, true);
}

ra_status relay_attn_cache_append(const ra_params *p, const void *k_new, const void *v_new,
                                  int64_t new_stride_token, int64_t new_stride_head,
                                  const int32_t *cu_seqlens_q, int32_t total_q, void *k_cache,
                                  void *v_cache, const int32_t *block_tables,
                                  const int32_t *context_lens, void *hip_stream) {
    ra_status st = check_params(p, total_q);
    if (st != RA_OK) return st;
    if (new_stride_token < 0 || new_stride_head < 0 || new_stride_token % 8 || new_stride_head % 8)
        return RA_ERR_INVALID_ARG;
    if (!cu_seqlens_q && total_q != p->batch) return RA_ERR_INVALID_ARG;
    if (total_q == 0) return RA_OK;
    if (p->batch < 1 || !k_new || !v_new || !k_cache || !v_cache || !block_tables || !context_lens)
        return RA_ERR_INVALID_ARG;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache))
        return RA_ERR_INVALID_ARG;
    if (new_stride_head < p->head_dim && p->num_kv_heads > 1) return RA_ERR_INVALID_ARG;
    ra::AppendArgs a{};
    a.k_new = static_cast<const uint16_t *>(k_new);
    a.v_new = static_cast<const uint16_t *>(v_new);
    a.k_cache = static_cast<uint16_t *>(k_cache);
    a.v_cache = static_cast<uint16_t *>(v_cache);
    a.block_tables = block_tables;
    a.context_lens = context_lens;
    a.cu_seqlens_q = cu_seqlens_q;
    a.new_stride_token = new_stride_token;
    a.new_stride_head = new_stride_head;
    a.batch = p->batch;
    a.total_q = total_q;
    a.Hkv = p->num_kv_heads;
    a.head_dim = p->head_dim;
    a.block_size_log2 = 0;
    while ((1 << a.block_size_log2) < p->block_size) ++a.block_size_log2;
    a.max_blocks_per_seq = p->max_blocks_per_seq;
    if (ra::launch_cache_append(a, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return RA_ERR_HIP;
    return RA_OK;
}

ra_status relay_attn_system_cache_layout(const ra_params *p, int64_t *stride_token_out,
                                         int64_t *stride_head_out, size_t *bytes_out) {
    if (!p || !stride_token_out || !stride_head_out || !bytes_out) return RA_ERR_INVALID_ARG;
    if (p->num_kv_heads < 1 || p->head_dim < 1 || p->head_dim % 8 || p->sys_len < 0)
        return RA_ERR_INVALID_ARG;
    // the smallest row stride >= the dense one that is 384 mod 1024 bytes (192 mod 512 elements)
    const int64_t dense = (int64_t)p->num_kv_heads * p->head_dim;
    int64_t stride = dense / 512 * 512 + 192;
    if (stride < dense) stride += 512;
    *stride_token_out = stride;
    *stride_head_out = p->head_dim;
    // (the last row needs no padding behind it)
    *bytes_out = p->sys_len > 0 ? (size_t)(((int64_t)p->sys_len - 1) * stride + dense) * 2 : 0;
    return RA_OK;
}

ra_status relay_attn_system_fill(const ra_params *p, const void *k_new, const void *v_new,
                                 int64_t new_stride_token, int64_t new_stride_head,
                                 int32_t first_pos, int32_t num_pos, void *k_sys, void *v_sys,
                                 void *hip_stream) {
    ra_status st = check_params(p, 0);
    if (st != RA_OK) return st;
    if (new_stride_token < 0 || new_stride_head < 0 || new_stride_token % 8 || new_stride_head % 8)
        return RA_ERR_INVALID_ARG;
    if (first_pos < 0 || num_pos < 0 || (int64_t)first_pos + num_pos > p->sys_len)
        return RA_ERR_INVALID_ARG;
    if (num_pos == 0) return RA_OK;
    if (!k_new || !v_new || !k_sys || !v_sys) return RA_ERR_INVALID_ARG;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_sys) || !aligned16(v_sys))
        return RA_ERR_INVALID_ARG;
    if (new_stride_head < p->head_dim && p->num_kv_heads > 1) return RA_ERR_INVALID_ARG;
    if (p->sys_stride_head < p->head_dim && p->num_kv_heads > 1) return RA_ERR_INVALID_ARG;
    if (p->sys_stride_token < p->head_dim && p->sys_len > 1) return RA_ERR_INVALID_ARG;
    ra::SysFillArgs a{};
    a.k_new = static_cast<const uint16_t *>(k_new);
    a.v_new = static_cast<const uint16_t *>(v_new);
    a.k_sys = static_cast<uint16_t *>(k_sys);
    a.v_sys = static_cast<uint16_t *>(v_sys);
    a.new_stride_token = new_stride_token;
    a.new_stride_head = new_stride_head;
    a.sys_stride_token = p->sys_stride_token;
    a.sys_stride_head = p->sys_stride_head;
    a.first_pos = first_pos;
    a.num_pos = num_pos;
    a.Hkv = p->num_kv_heads;
    a.head_dim = p->head_dim;
    if (ra::launch_system_fill(a, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return RA_ERR_HIP;
    return RA_OK;
}

ra_status relay_attn_debug_validate(const ra_params *p, const int32_t *block_tables,
                                    const int32_t *context_lens, const int32_t *cu_seqlens_q,
                                    int32_t total_q, void *workspace, size_t workspace_bytes,
                                    void *hip_stream, ra_validate_report *report) {
    const ra_status st = check_params(p, total_q);
    if (st != RA_OK) return st;
    if (!cu_seqlens_q && total_q != p->batch) return RA_ERR_INVALID_ARG;
    if (p->batch > 0 && (!context_lens || (!block_tables && p->max_blocks_per_seq > 0)))
        return RA_ERR_INVALID_ARG;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return RA_ERR_INVALID_ARG;
    if (workspace_bytes < 256) return RA_ERR_WORKSPACE_TOO_SMALL;
    ra::ValidateArgs a{};
    a.block_tables = block_tables;
    a.context_lens = context_lens;
    a.cu_seqlens_q = cu_seqlens_q;
    a.counters = static_cast<int32_t *>(workspace);
    a.batch = p->batch;
    a.total_q = total_q;
    a.num_blocks = p->num_blocks;
    a.block_size_log2 = 0;
    while ((1 << a.block_size_log2) < p->block_size) ++a.block_size_log2;
    a.max_blocks_per_seq = p->max_blocks_per_seq;
    a.max_len = p->max_context_len > 0 ? p->max_context_len : p->max_blocks_per_seq * p->block_size;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (ra::launch_validate(a, stream) != hipSuccess) return RA_ERR_HIP;
    int32_t host[4] = {0, 0, 0, 0};
    if (hipMemcpyAsync(host, a.counters, sizeof(host), hipMemcpyDeviceToHost, stream) != hipSuccess)
        return RA_ERR_HIP;
    if (hipStreamSynchronize(stream) != hipSuccess) return RA_ERR_HIP;
    const bool clean = host[0] == 0 && host[1] == 0 && host[2] == 0;
    if (report) {
        report->bad_context_lens = host[0];
        report->bad_block_ids = host[1];
        report->bad_query_lens = host[2];
        report->first_bad_request = clean ? -1 : host[3];
    }
    return clean ? RA_OK : RA_ERR_INVALID_ARG;
}

ra_status relay_attn_debug_stream_probe(const void *src, size_t bytes, int32_t nontemporal,
                                        void *sink, void *hip_stream) {
    if (!src || !sink || !aligned16(src) || (bytes % 16) != 0) return RA_ERR_INVALID_ARG;
    if (nontemporal != 0 && nontemporal != 1) return RA_ERR_INVALID_ARG;
    if (ra::launch_stream_probe(src, bytes, nontemporal, sink, static_cast<hipStream_t>(hip_stream)) !=
        hipSuccess)
        return RA_ERR_HIP;
    return RA_OK;
}

ra_status relay_attn_debug_launch_probe(void *sink, int32_t count, void *hip_stream) {
    if (!sink || count < 0 || count > (1 << 20)) return RA_ERR_INVALID_ARG;
    if (ra::launch_empty_probe(sink, count, static_cast<hipStream_t>(hip_stream)) != hipSuccess) return RA_ERR_HIP;
    return RA_OK;
}

const char *relay_attn_status_string(ra_status status) {
    switch (status) {
        case RA_OK: return "ok";
        case RA_ERR_INVALID_ARG: return "invalid argument";
        case RA_ERR_UNSUPPORTED: return "unsupported configuration";
        case RA_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case RA_ERR_HIP: return "HIP call failed";
    }
    return "unknown status";
}

int32_t relay_attn_abi_version(void) { return kAbiVersion; }

}  // extern "C"
