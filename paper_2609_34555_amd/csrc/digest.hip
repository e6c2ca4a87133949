// digest.hip -- per-block key digests of one KV head and the query-digest
// score of SoloHead selection, for gfx950.
//
// Digest (Sec. 2.1 Quest-style block digests; Sec. 4.4.1 digests kept for
// one KV head per layer): elementwise min and max of the head's keys over
// the valid tokens of each block, exact, in the KV dtype.
//
// Score (Sec. 4.4.1, query-digest score): for block b and the G query heads
// of the solo KV head,
//   s[b] = (1/G) * sum_g sum_c max(q_gc * mn_bc, q_gc * mx_bc).
// Since mn <= mx, max(q*mn, q*mx) = q * (q >= 0 ? mx : mn) exactly, so each
// channel costs one bit-select and half of a packed dot product.  Both
// kernels are HBM-bound streams over the digests (512 B per block); one
// 16-lane group owns one block, each lane 8 channels (one 16-byte load).
#include "pulse_internal.h"

namespace pulse {

// Largest r in [0, B) with blk_off[r] <= b (blk_off is non-decreasing).
__device__ inline int find_request(const int64_t* blk_off, int32_t B, int64_t b) {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (blk_off[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

typedef __attribute__((ext_vector_type(2))) int16_t s16x2;

// Two 16-bit float patterns as signed integers of the same order (-0 just below +0); its own inverse.
__device__ inline s16x2 order16(s16x2 x) { return x ^ ((x >> 15) & (int16_t)0x7FFF); }

// One wave per block, lane = (token group tg in 0..3, 8-channel slice).  Bound by HBM (or
// the host link): 256 bytes per token and 512 per block.  The keys' addresses do not depend
// on the request, so the whole block is loaded first (BS / 4 loads of 16 bytes in flight per
// lane) and the request is looked up meanwhile; rows past the context are left out of the
// minimum and maximum.  Both are taken on packed pairs: with one value per register the
// vector instructions bound the kernel.  8 x 32K tokens, 8 KV heads (73 MB), six batches in
// turn: 24.2 us with both the look-up first and single values, 17.6 now (4.2 TB/s).  One batch
// over and over, whose keys stay in the 256 MB Infinity Cache: 18.0 and 14.7.
template <int BS>
__global__ __launch_bounds__(256) void build_digests_kernel(const uint16_t* __restrict__ kv,
                                                            const int64_t* __restrict__ blk_off,
                                                            const int32_t* __restrict__ ctx_len, int32_t B,
                                                            int64_t total_blocks, int32_t Hkv, int32_t kv_head,
                                                            uint16_t* __restrict__ digests, int32_t* status) {
    constexpr int R = BS / 4;  // rows per lane
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (b >= total_blocks) return;
    const int c8 = (lane & 15) * 8;
    const int tg = lane >> 4;
    const size_t E = (size_t)2 * Hkv * BS * kHeadDim;
    const uint16_t* K = kv + (size_t)b * E + (size_t)kv_head * BS * kHeadDim + tg * kHeadDim + c8;
    u32x4 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = *reinterpret_cast<const u32x4*>(K + (size_t)4 * i * kHeadDim);
    const int r = find_request(blk_off, B, b);
    const int64_t j = b - blk_off[r];
    const int64_t nv64 = (int64_t)ctx_len[r] - j * BS;
    const int nv = nv64 >= BS ? BS : (int)nv64;
    u32x4* dst = reinterpret_cast<u32x4*>(digests + b * 2 * kHeadDim);
    if (j < 0 || b >= blk_off[r + 1] || nv <= 0) {
        if (lane == 0) report(status, PULSE_ERR_BAD_INDEX);
        if (tg == 0) {
            dst[c8 / 8] = u32x4{0, 0, 0, 0};
            dst[16 + c8 / 8] = u32x4{0, 0, 0, 0};
        }
        return;
    }
    s16x2 mn[4], mx[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) { mn[p] = (int16_t)0x7FFF; mx[p] = (int16_t)0x8000; }
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const bool in = nv == BS || tg + 4 * t < nv;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t two = v[t][p];  // (a bit cast of the element itself would read element 0)
            const s16x2 k = order16(__builtin_bit_cast(s16x2, two));
            mn[p] = __builtin_elementwise_min(mn[p], in ? k : mn[p]);
            mx[p] = __builtin_elementwise_max(mx[p], in ? k : mx[p]);
        }
    }
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            mn[p] = __builtin_elementwise_min(
                mn[p], __builtin_bit_cast(s16x2, __shfl_xor(__builtin_bit_cast(int, mn[p]), off)));
            mx[p] = __builtin_elementwise_max(
                mx[p], __builtin_bit_cast(s16x2, __shfl_xor(__builtin_bit_cast(int, mx[p]), off)));
        }
    if (tg == 0) {
        u32x4 omn, omx;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            omn[p] = __builtin_bit_cast(uint32_t, order16(mn[p]));
            omx[p] = __builtin_bit_cast(uint32_t, order16(mx[p]));
        }
        dst[c8 / 8] = omn;
        dst[16 + c8 / 8] = omx;
    }
}

// Sum of x over the 16 lanes of a group, in every lane: the additions of a butterfly (lane ^ 1,
// ^ 2, ^ 4, ^ 8) as register permutes.  After the first two a quad's lanes are equal, so mirroring
// the half row and the row brings the same values as exchanging with lane ^ 4 and lane ^ 8.
__device__ inline float row_sum(float x) {
    auto add = [&](int y) { x += __int_as_float(y); };
    add(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));   // quad_perm [1, 0, 3, 2]
    add(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, true));   // quad_perm [2, 3, 0, 1]
    add(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141, 0xF, 0xF, true));  // row_half_mirror
    add(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x140, 0xF, 0xF, true));  // row_mirror
    return x;
}

template <int DT>
__device__ inline float dot2(uint32_t a, uint32_t b, float acc) {
    if constexpr (DT == PULSE_BF16)
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b),
                                               acc, false);
    else
        return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b), acc, false);
}

// Two shapes of the score kernel, chosen by the number of digests read:
// small sets (up to kScoreLargeBlocks) take one 16-block iteration per
// workgroup, so more workgroups share the short stream; large ones take two
// iterations with non-temporal loads, which keep the once-read digests from
// displacing cached lines.  Both measured faster than the other's setting at
// their sizes (and than 4 or more iterations, or a grid-stride form).
constexpr int64_t kScoreLargeBlocks = 65536;

template <bool NT>
__device__ inline u32x4 score_load(const u32x4* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    return *p;
}

// Largest r in [0, B) with off[r] <= b, over an LDS copy of blk_off.
__device__ inline int find_request_lds(const int64_t* off, int32_t B, int64_t b) {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// 256 threads = 16 groups of 16 lanes; group gi handles blocks
// base + gi + 16*it so that consecutive groups stream consecutive digests.
// blockIdx.y selects the scoring KV head when several heads score at once
// (headwise selection); with one head it is `solo`.  blk_off is staged in LDS
// so the request of a block costs no dependent global loads.
template <int DT, int G, int ITERS, bool NT>
__global__ __launch_bounds__(256) void score_kernel(const uint16_t* __restrict__ q,
                                                    const uint16_t* __restrict__ digests,
                                                    const int64_t* __restrict__ blk_off, int32_t B,
                                                    int64_t total_blocks, int32_t Hq, int32_t solo,
                                                    int32_t n_sink, int32_t n_local, float* __restrict__ scores,
                                                    ReleaseArgs rel, int32_t do_release) {
    extern __shared__ int64_t s_off[];
    const int head = gridDim.y > 1 ? (int)blockIdx.y : solo;
    digests += (size_t)blockIdx.y * total_blocks * 2 * kHeadDim;
    scores += (size_t)blockIdx.y * total_blocks;
    const int sub = threadIdx.x & 15;
    const int gi = threadIdx.x >> 4;
    const int c8 = sub * 8;
    const int64_t base = (int64_t)blockIdx.x * (16 * ITERS) + gi;
    // digest loads first: their addresses do not depend on the request
    u32x4 dmn[ITERS], dmx[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int64_t b = base + 16 * it;
        if (b < total_blocks) {
            const u32x4* dg = reinterpret_cast<const u32x4*>(digests + (size_t)b * 2 * kHeadDim);
            dmn[it] = score_load<NT>(dg + sub);
            dmx[it] = score_load<NT>(dg + 16 + sub);
        }
    }
    // Up to G = 6, the query rows of the request that holds the first block if
    // every request had the same length (exact for equal contexts) are loaded
    // with the digests, and a wrong guess is reloaded once the offsets are
    // known.  Larger groups load them then: holding G x 4 more registers across
    // the barrier would take the kernel past 64 VGPRs (8 waves per SIMD).
    constexpr bool kEarlyQ = G <= 6;
    uint32_t qp[G][4];
    auto load_q = [&](int rq) {
        const uint16_t* qr = q + ((size_t)rq * Hq + (size_t)head * G) * kHeadDim + c8;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(qr + (size_t)g * kHeadDim);
#pragma unroll
            for (int p = 0; p < 4; ++p) qp[g][p] = v[p];
        }
    };
    int q_r = -1;
    if constexpr (kEarlyQ) {
        q_r = base < total_blocks ? (int)(base * B / total_blocks) : 0;
        q_r = q_r < B ? q_r : B - 1;
        load_q(q_r);
    }
    // the previous step's release, on the side (independent of the scores)
    if (do_release && blockIdx.y == 0)
        release_entries(rel, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256, true);
    for (int i = threadIdx.x; i <= B; i += 256) s_off[i] = blk_off[i];
    __syncthreads();
    int64_t r_lo = 0, r_hi = 0;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int64_t b = base + 16 * it;
        if (b >= total_blocks) break;
        if (b >= r_hi || b < r_lo) {
            const int cur_r = find_request_lds(s_off, B, b);
            r_lo = s_off[cur_r];
            r_hi = s_off[cur_r + 1];
            if (cur_r != q_r) {
                load_q(cur_r);
                q_r = cur_r;
            }
        }
        const int64_t j = b - r_lo;
        const int64_t n = r_hi - r_lo;
        if (j < n_sink || j >= n - n_local) continue;  // forced blocks are not scored
        float acc = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                // 0xFFFF in each half whose q is non-negative (sign bit clear), formed
                // here rather than kept: G x 4 fewer live registers
                const uint32_t qm = ~(((qp[g][p] & 0x80008000u) >> 15) * 0xFFFFu);
                const uint32_t sel = (dmx[it][p] & qm) | (dmn[it][p] & ~qm);
                acc = dot2<DT>(qp[g][p], sel, acc);
            }
        acc = row_sum(acc);
        if (sub == 0) scores[b] = acc / (float)G;
    }
}

// Scores averaged over the KV heads (Average selection), in one launch for small sets.  A
// workgroup scores every head of bpw consecutive blocks: its 16-lane groups take (block,
// head) pairs, block-major, with score_kernel's loads and sums, and the heads' scores of a
// block are added in ascending order from LDS.
template <int DT, int G>
__global__ __launch_bounds__(256) void score_average_kernel(const uint16_t* __restrict__ q,
                                                            const uint16_t* __restrict__ digests,
                                                            const int64_t* __restrict__ blk_off, int32_t B,
                                                            int64_t total_blocks, int32_t Hq, int32_t H, int32_t bpw,
                                                            int32_t n_sink, int32_t n_local,
                                                            float* __restrict__ scores) {
    extern __shared__ int64_t s_off[];                        // [B + 1]
    float* s_sc = reinterpret_cast<float*>(s_off + B + 1);   // [bpw][H]
    const int sub = threadIdx.x & 15;
    const int gi = threadIdx.x >> 4;
    const int64_t b0 = (int64_t)blockIdx.x * bpw;
    const int pairs = (int)min((int64_t)bpw, total_blocks - b0) * H;
    for (int p0 = 0; p0 < pairs; p0 += 16) {
        const int p = min(p0 + gi, pairs - 1);  // groups past the last pair repeat it
        const int h = p % H;
        const int64_t b = b0 + p / H;
        const u32x4* dg =
            reinterpret_cast<const u32x4*>(digests + ((size_t)h * total_blocks + (size_t)b) * 2 * kHeadDim);
        const u32x4 dmn = dg[sub], dmx = dg[16 + sub];
        u32x4 qv[G];
        auto load_q = [&](int r) {
            const uint16_t* qr = q + ((size_t)r * Hq + (size_t)h * G) * kHeadDim + sub * 8;
#pragma unroll
            for (int g = 0; g < G; ++g) qv[g] = *reinterpret_cast<const u32x4*>(qr + (size_t)g * kHeadDim);
        };
        // the rows of the request the block has if all are equally long, with the digests
        const int guess = min((int)(b * B / total_blocks), B - 1);
        load_q(guess);
        if (p0 == 0) {
            for (int i = threadIdx.x; i <= B; i += 256) s_off[i] = blk_off[i];
            __syncthreads();
        }
        if (b < s_off[guess] || b >= s_off[guess + 1]) load_q(find_request_lds(s_off, B, b));
        float acc = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t qw = qv[g][c];
                const uint32_t qm = ~(((qw & 0x80008000u) >> 15) * 0xFFFFu);
                acc = dot2<DT>(qw, (dmx[c] & qm) | (dmn[c] & ~qm), acc);
            }
        acc = row_sum(acc);
        if (sub == 0) s_sc[p] = acc / (float)G;
    }
    __syncthreads();
    const float inv = 1.f / (float)H;
    for (int t = threadIdx.x; t * H < pairs; t += 256) {
        const int64_t b = b0 + t;
        const int r = find_request_lds(s_off, B, b);
        const int64_t j = b - s_off[r], n = s_off[r + 1] - s_off[r];
        if (j < n_sink || j >= n - n_local) continue;  // forced blocks are not scored
        float s = 0.f;
        for (int h = 0; h < H; ++h) s += s_sc[t * H + h];
        scores[b] = s * inv;
    }
}

// avg[b] = (1/H) * sum_h sc[h][b], heads summed in ascending order, eight of them in flight
// at a time (with them one after the other the whole call on 16 x 64K tokens, 8 heads, took
// 53.4 us instead of 52.4).  Entries that were not scored (forced blocks) are not written.
__global__ __launch_bounds__(256) void average_scores_kernel(const float* __restrict__ sc,
                                                             const int64_t* __restrict__ blk_off, int32_t B,
                                                             int64_t total_blocks, int32_t H, int32_t n_sink,
                                                             int32_t n_local, float* __restrict__ avg) {
    extern __shared__ int64_t s_off[];
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float* p = sc + min(b, total_blocks - 1);
    float s = 0.f, v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[(size_t)min(i, H - 1) * total_blocks];
    for (int i = threadIdx.x; i <= B; i += 256) s_off[i] = blk_off[i];
    __syncthreads();
    for (int h0 = 0; h0 < H; h0 += 8) {
        if (h0 > 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p[(size_t)min(h0 + i, H - 1) * total_blocks];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (h0 + i < H) s += v[i];
    }
    if (b >= total_blocks) return;
    const int r = find_request_lds(s_off, B, b);
    const int64_t j = b - s_off[r], n = s_off[r + 1] - s_off[r];
    if (j >= n_sink && j < n - n_local) avg[b] = s * (1.f / (float)H);
}

hipError_t launch_build_digests(const pulse_shape& s, const void* kv, const int64_t* blk_off,
                                const int32_t* ctx_len, int32_t B, int64_t total_blocks, int32_t kv_head,
                                void* digests, int32_t* status, hipStream_t st) {
    if (total_blocks == 0) return hipSuccess;
#define PULSE_DIGEST(BS)                                                                                          \
    hipLaunchKernelGGL(build_digests_kernel<BS>, dim3((unsigned)((total_blocks + 3) / 4)), dim3(256), 0, st,     \
                       (const uint16_t*)kv, blk_off, ctx_len, B, total_blocks, s.num_kv_heads, kv_head,          \
                       (uint16_t*)digests, status)
    if (s.block_size == 16) PULSE_DIGEST(16);
    else if (s.block_size == 32) PULSE_DIGEST(32);
    else PULSE_DIGEST(64);
#undef PULSE_DIGEST
    return hipGetLastError();
}

template <int DT, int G>
static void launch_score_t(int32_t heads, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, const void* q,
                           const void* digests, const int64_t* blk_off, int32_t B, int64_t total, int32_t Hq,
                           int32_t solo, int32_t n_sink, int32_t n_local, float* scores, const ReleaseArgs* rel) {
    const uint32_t lds = (uint32_t)(sizeof(int64_t) * ((size_t)B + 1));
    const ReleaseArgs ra = rel ? *rel : ReleaseArgs{};
    const int32_t dr = rel != nullptr;
    if (total * heads > kScoreLargeBlocks) {
        const dim3 grid((unsigned)((total + 31) / 32), (unsigned)heads);
        launch_timed(score_kernel<DT, G, 2, true>, grid, dim3(256), lds, st, ev0, ev1, (const uint16_t*)q,
                     (const uint16_t*)digests, blk_off, B, total, Hq, solo, n_sink, n_local, scores, ra, dr);
    } else {
        const dim3 grid((unsigned)((total + 15) / 16), (unsigned)heads);
        launch_timed(score_kernel<DT, G, 1, false>, grid, dim3(256), lds, st, ev0, ev1, (const uint16_t*)q,
                     (const uint16_t*)digests, blk_off, B, total, Hq, solo, n_sink, n_local, scores, ra, dr);
    }
}

template <int DT, int G>
static void launch_average_t(hipStream_t st, const void* q, const void* digests, const int64_t* blk_off, int32_t B,
                             int64_t total, int32_t Hq, int32_t H, int32_t n_sink, int32_t n_local, float* scores) {
    const int32_t bpw = H < 16 ? 16 / H : 1;
    const uint32_t lds = (uint32_t)(sizeof(int64_t) * ((size_t)B + 1) + sizeof(float) * (size_t)bpw * H);
    hipLaunchKernelGGL((score_average_kernel<DT, G>), dim3((unsigned)((total + bpw - 1) / bpw)), dim3(256), lds, st,
                       (const uint16_t*)q, (const uint16_t*)digests, blk_off, B, total, Hq, H, bpw, n_sink, n_local,
                       scores);
}

template <int DT>
static void launch_score_dt(int G, int32_t heads, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, const void* q,
                            const void* digests, const int64_t* blk_off, int32_t B, int64_t total, int32_t Hq,
                            int32_t solo, int32_t n_sink, int32_t n_local, float* scores, const ReleaseArgs* rel) {
#define PULSE_SCORE_CASE(g)                                                                                    \
    case g:                                                                                                    \
        launch_score_t<DT, g>(heads, st, ev0, ev1, q, digests, blk_off, B, total, Hq, solo, n_sink, n_local,  \
                              scores, rel);                                                                    \
        break;
    switch (G) {
        PULSE_SCORE_CASE(1) PULSE_SCORE_CASE(2) PULSE_SCORE_CASE(3) PULSE_SCORE_CASE(4)
        PULSE_SCORE_CASE(5) PULSE_SCORE_CASE(6) PULSE_SCORE_CASE(7) PULSE_SCORE_CASE(8)
        PULSE_SCORE_CASE(9) PULSE_SCORE_CASE(10) PULSE_SCORE_CASE(11) PULSE_SCORE_CASE(12)
        PULSE_SCORE_CASE(13) PULSE_SCORE_CASE(14) PULSE_SCORE_CASE(15) PULSE_SCORE_CASE(16)
        default: break;
    }
#undef PULSE_SCORE_CASE
}

template <int DT>
static void launch_average_dt(int G, hipStream_t st, const void* q, const void* digests, const int64_t* blk_off,
                              int32_t B, int64_t total, int32_t Hq, int32_t H, int32_t n_sink, int32_t n_local,
                              float* scores) {
#define PULSE_AVERAGE_CASE(g)                                                                                  \
    case g:                                                                                                    \
        launch_average_t<DT, g>(st, q, digests, blk_off, B, total, Hq, H, n_sink, n_local, scores);            \
        break;
    switch (G) {
        PULSE_AVERAGE_CASE(1) PULSE_AVERAGE_CASE(2) PULSE_AVERAGE_CASE(3) PULSE_AVERAGE_CASE(4)
        PULSE_AVERAGE_CASE(5) PULSE_AVERAGE_CASE(6) PULSE_AVERAGE_CASE(7) PULSE_AVERAGE_CASE(8)
        PULSE_AVERAGE_CASE(9) PULSE_AVERAGE_CASE(10) PULSE_AVERAGE_CASE(11) PULSE_AVERAGE_CASE(12)
        PULSE_AVERAGE_CASE(13) PULSE_AVERAGE_CASE(14) PULSE_AVERAGE_CASE(15) PULSE_AVERAGE_CASE(16)
        default: break;
    }
#undef PULSE_AVERAGE_CASE
}

// One head: its scores are the average.  Up to kScoreLargeBlocks digests one launch scores and
// averages (8 heads x 256 blocks 15.5 -> 11.7 us with the selection, 2 heads x 8450 15.7 ->
// 12.3); larger sets stream better with neighbouring workgroups on one head's digests, so every
// head scores into ws first (8 heads x 65536 blocks: 43 us and 3 of averaging; in one launch
// 47 to 60, whether groups took heads in turn or pairs of up to 8 blocks and 8 heads).
hipError_t launch_average_scores(const pulse_shape& s, const void* q, const void* digests, const int64_t* blk_off,
                                 int32_t B, int64_t total_blocks, int32_t n_sink, int32_t n_local, float* scores,
                                 float* head_scores, hipStream_t st) {
    if (total_blocks == 0) return hipSuccess;
    if (s.num_kv_heads == 1)
        return launch_score(s, q, digests, blk_off, B, total_blocks, 0, n_sink, n_local, scores, 1, st);
    // (the one launch holds a block's scores of every head in LDS)
    if (total_blocks * s.num_kv_heads > kScoreLargeBlocks || s.num_kv_heads > 256) {
        hipError_t e = launch_score(s, q, digests, blk_off, B, total_blocks, 0, n_sink, n_local, head_scores,
                                    s.num_kv_heads, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(average_scores_kernel, dim3((unsigned)((total_blocks + 255) / 256)), dim3(256),
                           (uint32_t)(sizeof(int64_t) * ((size_t)B + 1)), st, head_scores, blk_off, B, total_blocks,
                           s.num_kv_heads, n_sink, n_local, scores);
        return hipGetLastError();
    }
    const int32_t H = s.num_kv_heads, G = s.num_q_heads / H;
    if (s.dtype == PULSE_BF16)
        launch_average_dt<PULSE_BF16>(G, st, q, digests, blk_off, B, total_blocks, s.num_q_heads, H, n_sink, n_local,
                                      scores);
    else
        launch_average_dt<PULSE_F16>(G, st, q, digests, blk_off, B, total_blocks, s.num_q_heads, H, n_sink, n_local,
                                     scores);
    return hipGetLastError();
}

hipError_t launch_score(const pulse_shape& s, const void* q, const void* digests, const int64_t* blk_off,
                        int32_t B, int64_t total_blocks, int32_t solo, int32_t n_sink, int32_t n_local,
                        float* scores, int32_t heads, hipStream_t st, const ReleaseArgs* rel, hipEvent_t start,
                        hipEvent_t stop) {
    if (total_blocks == 0) {  // no blocks: no recall to release either; requested events become markers
        hipError_t e = start ? hipEventRecord(start, st) : hipSuccess;
        if (e == hipSuccess && stop) e = hipEventRecord(stop, st);
        return e;
    }
    const int G = s.num_q_heads / s.num_kv_heads;
    if (s.dtype == PULSE_BF16)
        launch_score_dt<PULSE_BF16>(G, heads, st, start, stop, q, digests, blk_off, B, total_blocks, s.num_q_heads,
                                    solo, n_sink, n_local, scores, rel);
    else
        launch_score_dt<PULSE_F16>(G, heads, st, start, stop, q, digests, blk_off, B, total_blocks, s.num_q_heads,
                                   solo, n_sink, n_local, scores, rel);
    return hipGetLastError();
}

}  // namespace pulse
