// A small decode step in one launch: one workgroup of 16 wavefronts per (request, query head) goes through
// the system prompt and the request's context and writes the output row (Eq. 7 as one softmax over
// [system ; context]; no partials, no fusion launch).
//
// Bound: the chain of dependent trips and then the rows, not bytes (one request of 32/8 heads, s = 512, 90 positions of
// context moves 2.5 MB).  The two-launch form needs arguments -> lengths -> block ids -> keys/values ->
// partials, then a second launch that reads the partials: 10.2 us for that call, 6.8 in this form (16 requests of
// 16 heads of 64, s = 1000, contexts of 16 .. 255: 10.8 and 7.8).  Here the trips are arguments -> length -> block
// ids -> keys/values (system rows do not wait for the two in the middle), and the wavefronts meet in LDS: 4.1 us of
// kernel time with one row and warm inputs, 4.7 with cold ones.  A round of 256 rows (head_dim 128) adds about 1.3 and
// 2.2: some 600 vector instructions a wavefront, four wavefronts a SIMD, are issued on the few units that have a
// workgroup.  16 wavefronts hold up to 16 (head_dim 128) or 32 rows each and ask for as many again while they work: 512
// rows of a call at head_dim 128, 1024 at 64.  (Block ids come back behind the rows that were asked for before them, so a
// second batch of context rows starts when the first has landed.)  The query heads of a kv head re-read its rows, from
// L2 where the kv head is the fastest grid index; what that and re-reading the system prompt per request costs
// is why the form is for small calls only (see direct_form in relay_attn.hip for the line).
// Vector arithmetic: with one query row there is no matrix product, and the row's 16 (head_dim 128) or 8
// lanes sum a score by data-parallel moves.
#include "ra_device.h"
#include "ra_kernels.h"

namespace ra {

constexpr int kDirectWaves = 16;
constexpr int kDirectThreads = kDirectWaves * kWave;

// Block-table slot to read for row `row` of [s system rows ; a context that is not empty]: the row's own, and the
// first one for a system row, so that no slot behind the ones in use is ever read.
__host__ __device__ constexpr int used_slot(int row, int s, int block_size_log2) {
    return row < s ? 0 : (row - s) >> block_size_log2;
}

template <int D, bool MULTI, bool APPEND>
__global__ __launch_bounds__(kDirectThreads, 4) void decode_direct_kernel(
    const DirectArgs a, const typename DirectPrefixes<MULTI>::type pfx) {
    constexpr int LPT = D / 8;                    // lanes per row, 8 elements (16 bytes) each
    constexpr int TPI = kWave / LPT;              // rows per load of a wavefront
    constexpr int U = 4;                          // rows per lane group in one batch
    constexpr int CH = TPI * U;                   // rows per batch of a wavefront
    constexpr int NG = kDirectWaves * TPI;        // lane groups of the workgroup
    constexpr int PITCH = D + 4;
    constexpr int PARTS = kDirectThreads / D;     // threads per element of the output row
    __shared__ __attribute__((aligned(16))) float sm_o[NG * PITCH];
    __shared__ float sm_m[NG], sm_l[NG];
    __shared__ float sm_part[PARTS * D];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int sub = lane % LPT, grp = lane / LPT;
    const int g = blockIdx.x, token = blockIdx.z;
    const int h = g * a.G + blockIdx.y;
    const int bsl = a.block_size_log2, bmask = (1 << bsl) - 1;
    const int32_t *bt = a.block_tables + (int64_t)token * a.max_blocks_per_seq;

    const uint16_t *k_sys, *v_sys;
    int s;
    if constexpr (MULTI) {
        int p = 0;
        if (pfx.req_prefix) p = pfx.req_prefix[token];
        else
            while (p + 1 < pfx.n && token >= pfx.token_end[p]) ++p;
        k_sys = pfx.k[p], v_sys = pfx.v[p], s = pfx.len[p];
    } else {
        k_sys = pfx.k, v_sys = pfx.v, s = pfx.len;
    }
    k_sys += (int64_t)g * a.sys_stride_head;
    v_sys += (int64_t)g * a.sys_stride_head;
    const int c = a.max_ctx > 0 ? max(0, min(a.context_lens[token], a.max_ctx)) : 0;
    const int total = s + c;

    const u32x4 qv = *reinterpret_cast<const u32x4 *>(a.q + (int64_t)token * a.q_stride_token +
                                                      (int64_t)h * a.q_stride_head + sub * 8);
    // Rows base .. base + CH - 1 of [system ; context]; rows behind the end re-load the last one.
    auto load = [&](int base, u32x4 (&k)[U], u32x4 (&v)[U]) {
        if (base + CH <= s) {                     // (uniform) system rows only
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t off = (int64_t)(base + u * TPI + grp) * a.sys_stride_token + sub * 8;
                k[u] = *reinterpret_cast<const u32x4 *>(k_sys + off);
                v[u] = *reinterpret_cast<const u32x4 *>(v_sys + off);
            }
            return;
        }
        // Every block id of the batch before its first row: an id asked for between the rows makes each row wait for
        // the ones before it (12 requests of 32/8 heads, s = 115, contexts of 144 .. 218: 10.5 us so, 9.4 as here).
        int row[U], blk[U] = {};
#pragma unroll
        for (int u = 0; u < U; ++u) row[u] = min(base + u * TPI + grp, total - 1);
        if (c > 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) blk[u] = bt[used_slot(row[u], s, bsl)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int pos = row[u] - s;
            const bool sys = pos < 0, fresh = APPEND && pos >= 0 && pos == c - 1;   // fresh: not in the cache yet
            int64_t off = sys ? (int64_t)row[u] * a.sys_stride_token
                              : ((((int64_t)blk[u] * a.Hkv + g) << bsl) + (pos & bmask)) * (int64_t)D;
            if (fresh) off = (int64_t)token * a.new_stride_token + (int64_t)g * a.new_stride_head;
            const uint16_t *kp = sys ? k_sys : fresh ? a.k_new : a.k_cache, *vp = sys ? v_sys : fresh ? a.v_new : a.v_cache;
            k[u] = *reinterpret_cast<const u32x4 *>(kp + off + sub * 8);
            v[u] = *reinterpret_cast<const u32x4 *>(vp + off + sub * 8);
        }
    };

    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = 0.f;
    auto attend = [&](int base, const u32x4 (&k)[U], const u32x4 (&v)[U]) {
        float sc[U], mx = m;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float dot = group_sum<LPT>(dot8_bf16(qv, k[u], 0.f));
            sc[u] = base + u * TPI + grp < total ? dot * a.scale_log2 : -INFINITY;
            mx = fmaxf(mx, sc[u]);
        }
        const float m_use = finite_or_zero(mx);
        const float corr = __builtin_amdgcn_exp2f(m - m_use);      // m = -inf: 0, and l, o are 0
        m = mx;
        l *= corr;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] *= corr;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float p = __builtin_amdgcn_exp2f(sc[u] - m_use);
            l += p;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t w = v[u][i];
                o[2 * i] = fmaf(p, bf16_lo(w), o[2 * i]);
                o[2 * i + 1] = fmaf(p, bf16_hi(w), o[2 * i + 1]);
            }
        }
    };

    constexpr int STRIDE = kDirectWaves * CH;
    u32x4 ka[U], va[U], kb[U], vb[U];
    int base = wave * CH;
    if (base < total) load(base, ka, va);
    while (base < total) {                        // the next batch is on its way while this one is worked off
        if (base + STRIDE < total) load(base + STRIDE, kb, vb);
        attend(base, ka, va);
        base += STRIDE;
        if (base >= total) break;
        if (base + STRIDE < total) load(base + STRIDE, ka, va);
        attend(base, kb, vb);
        base += STRIDE;
    }
    if (APPEND && c > 0 && blockIdx.y == 0 && wave == 0 && grp == 0) {
        const int64_t from = (int64_t)token * a.new_stride_token + (int64_t)g * a.new_stride_head + sub * 8;
        const int64_t to = ((((int64_t)bt[(c - 1) >> bsl] * a.Hkv + g) << bsl) + ((c - 1) & bmask)) * (int64_t)D + sub * 8;
        *reinterpret_cast<u32x4 *>(const_cast<uint16_t *>(a.k_cache) + to) = *reinterpret_cast<const u32x4 *>(a.k_new + from);
        *reinterpret_cast<u32x4 *>(const_cast<uint16_t *>(a.v_cache) + to) = *reinterpret_cast<const u32x4 *>(a.v_new + from);
    }

    // ---- the lane groups meet: weights by every wavefront for itself, PARTS threads per element
    const int mine = wave * TPI + grp;
#pragma unroll
    for (int i = 0; i < 8; i += 4)
        *reinterpret_cast<f32x4 *>(&sm_o[mine * PITCH + sub * 8 + i]) = f32x4{o[i], o[i + 1], o[i + 2], o[i + 3]};
    if (sub == 0) sm_m[mine] = m, sm_l[mine] = l;
    __syncthreads();
    constexpr int PER = NG / kWave;               // groups per lane
    float gm[PER], M = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; ++i) gm[i] = sm_m[i * kWave + lane], M = fmaxf(M, gm[i]);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float m_use = finite_or_zero(M);
    const int d = threadIdx.x % D, part = threadIdx.x / D;
    constexpr int GP = NG / PARTS;                // groups per part
    float acc = 0.f, W = 0.f;
#pragma unroll
    for (int i = 0; i < GP; ++i) {
        const int j = part * GP + i;
        const float w = __builtin_amdgcn_exp2f(sm_m[j] - m_use);
        acc = fmaf(w, sm_o[j * PITCH + d], acc);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) W = fmaf(__builtin_amdgcn_exp2f(gm[i] - m_use), sm_l[i * kWave + lane], W);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) W += __shfl_xor(W, off);
    sm_part[part * D + d] = acc;
    __syncthreads();
    if (part != 0) return;
#pragma unroll
    for (int i = 1; i < PARTS; ++i) acc += sm_part[i * D + d];
    acc *= W > 0.f ? 1.f / W : 0.f;
    const int64_t oo = (int64_t)token * a.o_stride_token + (int64_t)h * a.o_stride_head + d;
    if (a.out_is_fp32) static_cast<float *>(a.out)[oo] = acc;
    else static_cast<uint16_t *>(a.out)[oo] = (uint16_t)f32_to_bf16_bits(acc);
    if (d == 0 && a.lse_out) a.lse_out[(int64_t)token * a.Hq + h] = W > 0.f ? (m_use + log2f(W)) * kLn2 : -INFINITY;
}

template <int D, bool MULTI>
static void launch_direct(const DirectArgs &a, const typename DirectPrefixes<MULTI>::type &pfx, hipStream_t stream) {
    const dim3 grid((unsigned)a.Hkv, (unsigned)a.G, (unsigned)a.n_tokens), block(kDirectThreads);
    if constexpr (!MULTI) {                       // (no entry point appends with several prefixes)
        if (a.k_new) {
            hipLaunchKernelGGL((decode_direct_kernel<D, false, true>), grid, block, 0, stream, a, pfx);
            return;
        }
    }
    hipLaunchKernelGGL((decode_direct_kernel<D, MULTI, false>), grid, block, 0, stream, a, pfx);
}

hipError_t launch_decode_direct(const DirectArgs &a, const DirectOne *one, const DirectMany *many, int head_dim,
                                hipStream_t stream) {
    if (a.n_tokens == 0) return hipSuccess;
    if (a.n_tokens > 65535 || (!one && !many) || (!one && a.k_new)) return hipErrorInvalidValue;
    if (head_dim == 128 && one) launch_direct<128, false>(a, *one, stream);
    else if (head_dim == 128) launch_direct<128, true>(a, *many, stream);
    else if (head_dim == 64 && one) launch_direct<64, false>(a, *one, stream);
    else if (head_dim == 64) launch_direct<64, true>(a, *many, stream);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ra
