// Relay fusion (Alg. 1 "relay fusion"; App. A, Eq. 11-12).  With two partials the output is
//   out = alpha_sys * o_sys + (1 - alpha_sys) * o_ctx,  alpha_sys = 1 / (1 + exp(lse_ctx - lse_sys)).
// The system prompt is processed in several chunks and long contexts in several parts, so the
// same identity is applied to n partials in its max-shifted form: with M = max_p lse_p and
// w_p = exp(lse_p - M), out = sum_p w_p o_p / sum_p w_p and lse = M + log sum_p w_p.  For two
// partials w_sys / (w_sys + w_ctx) is exactly alpha_sys.  Log-sum-exps are kept in base 2
// internally and converted to natural log only for lse_out.
#include "ra_device.h"
#include "ra_kernels.h"

namespace ra {

// P groups of D/4 threads share an output row, group k taking every P-th batch of eight partials, and
// merge through LDS.  P = 1 where the rows alone fill the machine; with few rows that have many
// partials each (a few requests with long contexts: 384 rows of up to 40) the batches of one row
// would otherwise be one trip to memory after the other on a machine that is nearly empty.
// LATE: payloads behind the first `n_likely` partials are loaded once the log-sum-exps say that they are
// there.  One trip more than loading both together, but no bytes of slots that were never written: a
// bound far above the real lengths makes room for several times what a row uses.
template <int D, bool MULTI, int P, bool LATE>
__global__ __launch_bounds__(kThreads) void fuse_kernel(const FuseArgs a) {
    constexpr int TPR = D / 4;                  // threads per output row (4 elements each)
    constexpr int RPB = kThreads / (TPR * P);   // rows per block
    static_assert(P == 1 || RPB == 1, "the groups of a row are the whole workgroup");
    __shared__ int sm_end[2][P];
    const int part = P == 1 ? 0 : threadIdx.x / TPR;
    const int row = P == 1 ? blockIdx.x * RPB + threadIdx.x / TPR : blockIdx.x;
    const int e = (threadIdx.x % TPR) * 4;
    if (row >= a.rows) return;                  // (P > 1: uniform)

    // Loads are issued eight partials at a time before any of them is used: the partials were
    // written by other compute units, so each one costs a trip to L2 or memory, and a loop that
    // consumed them one by one would pay those trips back to back.  To keep the eight loads free of
    // branches a slot that does not exist is loaded from slot 0 and discarded by a select.
    constexpr int U = 8;
    // With several shared prefixes (App. D) a request whose prefix is shorter than the longest one
    // has fewer system chunks; the partial slots [n_sys, n_sys_chunks) of its rows were never
    // written, and the row's partials are numbered without them.
    int gap_at = 0, gap = 0;
    if (MULTI) {
        const int token = row / a.Hq;
        int pfx = 0;
        if (a.req_prefix) pfx = a.req_prefix[token];
        else
            while (pfx + 1 < a.n_prefixes && token >= a.pfx_token_end[pfx]) ++pfx;
        gap_at = a.pfx_chunks[pfx];
        gap = a.n_sys_chunks - gap_at;
    }
    const int n = a.n_partials - gap;
    [[maybe_unused]] const int likely = a.n_likely - gap;
    const int64_t oo = (int64_t)(row / a.Hq) * a.o_stride_token + (int64_t)(row % a.Hq) * a.o_stride_head + e;
    // One trip to memory per eight partials: log-sum-exps and payloads are loaded together and
    // merged with a running maximum (the same online rescaling the attention kernels use), rather
    // than reading all log-sum-exps first to find the maximum and then coming back for the rest.
    // The slots behind an end mark hold anything; those of the batch are discarded (and, LATE, not loaded:
    // there the log-sum-exps are fetched one round ahead, so that it stays one trip per round).
    // (v_exp_f32 as it is: a weight below the normal range cannot reach a sum that holds a 1.)
    float M = -INFINITY, W = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int end = INT_MAX;
    auto slot_of = [&](int p, bool read) -> int64_t {          // of the row's partial p; slot 0 if it is not read
        const int at = MULTI && p >= gap_at ? p + gap : p;
        return (int64_t)(read ? at : 0) * a.rows + row;
    };
    auto payload = [&](int64_t slot) { return *reinterpret_cast<const f32x4 *>(a.part_o + slot * D + e); };
    [[maybe_unused]] float l_next[U];
    if constexpr (LATE) {
#pragma unroll
        for (int j = 0; j < U; ++j) l_next[j] = a.part_lse[slot_of(part * U + j, part * U + j < n)];
    }
    for (int round = 0; round * (P * U) < n; ++round) {
        const int p0 = round * (P * U) + part * U;
        float l[U];
        f32x4 o[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const bool ok = p0 + j < n;
            if constexpr (LATE) {
                l[j] = l_next[j];
                if (round == 0) o[j] = payload(slot_of(p0 + j, p0 + j < likely));
            } else {
                const int64_t slot = slot_of(p0 + j, ok);
                l[j] = a.part_lse[slot];
                o[j] = payload(slot);
            }
            l[j] = ok ? l[j] : -INFINITY;
        }
#pragma unroll
        for (int j = U - 1; j >= 0; --j)
            if (__float_as_uint(l[j]) == kEndOfPartials) end = p0 + j;
        if constexpr (P > 1) {                  // the row's end is the first one that any group met
            if (e == 0) sm_end[round & 1][part] = end;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < P; ++k) end = min(end, sm_end[round & 1][k]);
        }
        if constexpr (LATE) {
            const int last = min(end, n), p1 = p0 + P * U;
#pragma unroll
            for (int j = 0; j < U; ++j)
                if ((round > 0 || p0 + j >= likely) && p0 + j < last) o[j] = payload(slot_of(p0 + j, true));
#pragma unroll
            for (int j = 0; j < U; ++j) l_next[j] = p1 < last ? a.part_lse[slot_of(p1 + j, p1 + j < n)] : 0.f;
        }
        float Mb = M;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            l[j] = p0 + j < end ? l[j] : -INFINITY;
            Mb = fmaxf(Mb, l[j]);
        }
        const float m_use = finite_or_zero(Mb);
        const float corr = __builtin_amdgcn_exp2f(M - m_use);      // M = -inf (nothing yet): 0, and acc, W are 0
        acc *= corr;
        W *= corr;
        M = Mb;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            // An empty or absent slot has w = 0; its payload may never have been written, so it is
            // dropped by a select.
            const float w = __builtin_amdgcn_exp2f(l[j] - m_use);
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            acc += (w > 0.f ? o[j] : zero) * w;
            W += w;
        }
        if (end <= (round + 1) * (P * U)) break;
    }
    if constexpr (P > 1) {
        __shared__ f32x4 sm_acc[P][TPR];
        __shared__ float sm_m[P], sm_w[P];
        sm_acc[part][e / 4] = acc;
        if (e == 0) sm_m[part] = M, sm_w[part] = W;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int k = 0; k < P; ++k) M = fmaxf(M, sm_m[k]);
        const float m_use = finite_or_zero(M);
        W = 0.f;
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const float f = __builtin_amdgcn_exp2f(sm_m[k] - m_use);
            acc += sm_acc[k][e / 4] * f;
            W = fmaf(sm_w[k], f, W);
        }
    }
    const float inv = W > 0.f ? 1.f / W : 0.f;
    acc *= inv;
    if (a.out_is_fp32) {
        *reinterpret_cast<f32x4 *>(static_cast<float *>(a.out) + oo) = acc;
    } else {
        u32x2 w2 = {pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
        *reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(a.out) + oo) = w2;
    }
    if (e == 0 && a.lse_out) a.lse_out[row] = W > 0.f ? (finite_or_zero(M) + log2f(W)) * kLn2 : -INFINITY;
}

// Cache append: a workgroup moves the rows of `tpw` consecutive tokens (K and V, all kv heads), a
// thread up to eight 16-byte pieces at a time.  Bound: HBM for many tokens (every byte in once and out
// once; one piece of K and V per thread, each with its own search for the request, ran 5222 tokens of 40
// heads in 43 us, this form in 33), the chain of dependent reads for few: the pieces are read before
// their place is known, and the request of a token is counted 64 requests at a time by the lanes of
// one wavefront instead of searched by halving.
constexpr int kAppendMaxTokens = 16;
__global__ __launch_bounds__(kThreads) void cache_append_kernel(const AppendArgs a, const int tpw) {
    __shared__ int64_t sm_dst[kAppendMaxTokens];         // element offset of (token, kv head 0), or -1
    const int token0 = (int)blockIdx.x * tpw;
    const int cpr_log2 = a.head_dim == 128 ? 4 : 3;       // 16-byte chunks per row
    const int per_token = a.Hkv << cpr_log2;
    const int n = min(tpw, a.total_q - token0) * per_token;
    const int64_t head_stride = (int64_t)a.head_dim << a.block_size_log2;
    constexpr int U = 4;
    u32x4 k[U], v[U];
    auto read = [&](int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kThreads;
            if (i >= n) continue;
            const int t = i / per_token, in_token = i - t * per_token;
            const int g = in_token >> cpr_log2, chunk = in_token & ((1 << cpr_log2) - 1);
            const int64_t src = (int64_t)(token0 + t) * a.new_stride_token + (int64_t)g * a.new_stride_head + chunk * 8;
            k[u] = *reinterpret_cast<const u32x4 *>(a.k_new + src);
            v[u] = *reinterpret_cast<const u32x4 *>(a.v_new + src);
        }
    };
    read(threadIdx.x);
    if (threadIdx.x < kWave) {
        const int lane = (int)threadIdx.x;
        const int token = token0 + lane;
        // The lanes hold the bounds and lengths of 64 requests at a time, so that a token's place is one trip
        // to its block id away once they are here (searched first and asked for then, the lengths were a
        // trip of their own).
        int req = token, pos = 0;
        if (a.cu_seqlens_q) {
            bool found = false;
            req = a.batch - 1;
            for (int base = 0; base < a.batch; base += kWave) {
                const int r = base + lane;
                const bool any = r < a.batch;
                const int first = any ? a.cu_seqlens_q[r] : 0, end = any ? a.cu_seqlens_q[r + 1] : INT_MAX;
                const int len = any ? a.context_lens[r] : 0;
                int owner = kWave;                        // requests of these that end at or before the token
                for (int t = 0; t < tpw; ++t) {
                    const int ended = __builtin_popcountll(__builtin_amdgcn_ballot_w64(end <= token0 + t));
                    if (lane == t) owner = ended;
                }
                // (a token that no request owns goes to the last one)
                const bool last = base + kWave >= a.batch;
                const int from = min(owner, min(a.batch - base, kWave) - 1);
                const int f = __shfl(first, from), e = __shfl(end, from), l = __shfl(len, from);
                if (!found && (owner < kWave || last)) {
                    found = true;
                    req = base + from;
                    pos = l - (e - f) + (token - f);
                }
            }
        }
        if (lane < tpw && token < a.total_q) {
            if (!a.cu_seqlens_q) pos = a.context_lens[req] - 1;
            int64_t dst = -1;                             // malformed lengths: write nothing
            if (pos >= 0) {
                const int64_t blk = a.block_tables[(int64_t)req * a.max_blocks_per_seq + (pos >> a.block_size_log2)];
                const int bmask = (1 << a.block_size_log2) - 1;
                dst = (((blk * a.Hkv) << a.block_size_log2) + (pos & bmask)) * (int64_t)a.head_dim;
            }
            sm_dst[lane] = dst;
        }
    }
    __syncthreads();
    for (int i0 = threadIdx.x; i0 < n; i0 += U * kThreads) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kThreads;
            if (i >= n) continue;
            const int t = i / per_token, in_token = i - t * per_token;
            const int g = in_token >> cpr_log2, chunk = in_token & ((1 << cpr_log2) - 1);
            if (sm_dst[t] < 0) continue;
            const int64_t to = sm_dst[t] + g * head_stride + chunk * 8;
            *reinterpret_cast<u32x4 *>(a.k_cache + to) = k[u];
            *reinterpret_cast<u32x4 *>(a.v_cache + to) = v[u];
        }
        read(i0 + U * kThreads);
    }
}

// System-cache fill: same 16-byte moves, destination addressed by (position, kv head) strides.
__global__ __launch_bounds__(kThreads) void system_fill_kernel(const SysFillArgs a) {
    const int cpr = a.head_dim / 8;
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t total = (int64_t)a.num_pos * a.Hkv * cpr;
    if (idx >= total) return;
    const int chunk = (int)(idx % cpr);
    const int g = (int)((idx / cpr) % a.Hkv);
    const int t = (int)(idx / ((int64_t)cpr * a.Hkv));
    const int64_t src = (int64_t)t * a.new_stride_token + (int64_t)g * a.new_stride_head + chunk * 8;
    const int64_t dst = (int64_t)(a.first_pos + t) * a.sys_stride_token +
                        (int64_t)g * a.sys_stride_head + chunk * 8;
    *reinterpret_cast<u32x4 *>(a.k_sys + dst) = *reinterpret_cast<const u32x4 *>(a.k_new + src);
    *reinterpret_cast<u32x4 *>(a.v_sys + dst) = *reinterpret_cast<const u32x4 *>(a.v_new + src);
}

hipError_t launch_system_fill(const SysFillArgs &a, hipStream_t stream) {
    const int64_t total = (int64_t)a.num_pos * a.Hkv * (a.head_dim / 8);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(system_fill_kernel, dim3((unsigned)((total + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_cache_append(const AppendArgs &a, hipStream_t stream) {
    if (a.total_q == 0) return hipSuccess;
    // about 1024 of the 16-byte chunks per workgroup (one round of U = 4), fewer where that would leave
    // compute units idle
    const int per_token = a.Hkv * (a.head_dim / 8);
    int tpw = 1024 / per_token;
    if (tpw > a.total_q / 512) tpw = a.total_q / 512;
    if (tpw > kAppendMaxTokens) tpw = kAppendMaxTokens;
    if (tpw < 1) tpw = 1;
    hipLaunchKernelGGL(cache_append_kernel, dim3((unsigned)((a.total_q + tpw - 1) / tpw)), dim3(kThreads), 0,
                       stream, a, tpw);
    return hipGetLastError();
}

template <int D, bool MULTI, int P>
static void launch_fuse_form(const FuseArgs &a, bool late, const dim3 &grid, hipStream_t stream) {
    if (late) hipLaunchKernelGGL((fuse_kernel<D, MULTI, P, true>), grid, dim3(kThreads), 0, stream, a);
    else hipLaunchKernelGGL((fuse_kernel<D, MULTI, P, false>), grid, dim3(kThreads), 0, stream, a);
}

constexpr int64_t kLateBytes = 12 << 20;
template <int D>
static void launch_fuse_d(const FuseArgs &a, hipStream_t stream) {
    constexpr int TPR = D / 4, P = kThreads / TPR;      // split form: one row per workgroup
    // More than two batches of eight partials and no more rows than the chip holds workgroups of
    // this kind at once: split (384 rows of up to 40 partials in
    // 131 slots take 5.2 us; three batches one after the other, 24 slots, took 5.1).
    const bool split = a.n_partials > 16 && a.rows <= 2048;
    // Late payloads where the first round would load more than 12 MiB beyond the likely partials, which
    // is about what the extra trip to memory costs.  Measured, whole call, early / late payloads: 1024
    // rows of 32 requests, bound 16128, one of them that long and the others 100 positions 37.4 / 32.5
    // us; 64 requests of 32/8 heads with contexts of 100 .. 1000 under a bound of 16400 48.6 / 46.1
    // us; but 256 rows that fill 130 slots (8 requests of 32/4 heads, one of 30000 positions) 30.1 / 33.0,
    // and one request of 90 positions 10.2 / 10.6.
    const int first = split ? 8 * P : 8;
    const int64_t beyond = (a.n_partials < first ? a.n_partials : first) - a.n_likely;
    const bool late = beyond * a.rows * D * 4 > kLateBytes;
    const bool multi = a.n_prefixes > 1;
    const dim3 grid(split ? a.rows : (a.rows + P - 1) / P);
    if (split && multi) launch_fuse_form<D, true, P>(a, late, grid, stream);
    else if (split) launch_fuse_form<D, false, P>(a, late, grid, stream);
    else if (multi) launch_fuse_form<D, true, 1>(a, late, grid, stream);
    else launch_fuse_form<D, false, 1>(a, late, grid, stream);
}

hipError_t launch_fuse(const FuseArgs &a, int head_dim, hipStream_t stream) {
    if (a.rows == 0) return hipSuccess;
    if (head_dim == 128) launch_fuse_d<128>(a, stream);
    else if (head_dim == 64) launch_fuse_d<64>(a, stream);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ra
