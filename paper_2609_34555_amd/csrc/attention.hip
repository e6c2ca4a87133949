// attention.hip -- split-K sparse GQA decode attention over the selected
// blocks of the slot pool, for gfx950 (the attention that follows recall,
// Sec. 2.2 and Sec. 4.2.1).
//
// One wavefront owns (request r, KV head h, split s): a contiguous range of
// the request's selected blocks.  The G query heads of h share every K/V
// byte the wave reads, so the contraction is a batched GQA tile:
//   S^T[32 tokens x 16] = K[32 x 128] . Q^T[128 x 16]   (G <= 16 query columns)
//   O[16 x 128]        += P[16 x 32]  . V[32 x 128]
// both on v_mfma_f32_16x16x32_{bf16,f16}.  Each lane's MFMA operands are 16
// contiguous bytes in HBM: K is stored token-major and V channel-major, so
// neither operand needs an LDS transpose.  The S^T tile rows are assigned
// to tokens so that its accumulator layout is exactly the P operand layout
// of the P.V product (lane = query column, 8 consecutive tokens per lane
// group), so softmax probabilities never leave registers.
//
// Precision: K, V, q are consumed as stored (products exact in fp32, fp32
// accumulation).  P is split into hi + lo 16-bit parts (two MFMAs), which
// keeps the P.V product at ~2^-16 relative error instead of the 2^-9 of a
// single bf16 rounding.  Softmax is online per 32-token step in the log2
// domain.
//
// Merging the splits: a workgroup holds W waves = W consecutive splits of one
// (r, h) (W = 8 for G <= 8, else 4); they merge through LDS.  With one
// workgroup per (r, h) it writes the result directly.  Otherwise each workgroup writes one partial (m, l, O) to
// the workspace and a combine kernel merges those few partials, one thread
// per output element, with independent loads.  (Merging in the last workgroup
// to finish instead needs a device-scope release per workgroup, an L2
// write-back on gfx950 measured at about 9 ns per workgroup, plus a merge on
// the kernel's tail and counters that start at zero in the workspace: it would
// save well under the combine launch's 3.6 us.)
#include "pulse_internal.h"

namespace pulse {

#ifndef PULSE_ATTN_TARGET_WAVES
#define PULSE_ATTN_TARGET_WAVES 2048
#endif
constexpr int kCombineThreads = kHeadDim;

// Waves per workgroup (attn_waves): 8 while the LDS merge buffer (waves x G x
// 128 floats) stays within 32 KiB, else 4.  Fewer, wider workgroups leave
// fewer partials for the combine kernel.

// Entries of one 32-token step, and of the shortest split.
static int32_t split_step(int32_t bs) { return bs >= kChunkTokens ? 1 : kChunkTokens / bs; }
static int32_t split_least(int32_t bs) { return bs >= 2 * kChunkTokens ? 1 : 2 * kChunkTokens / bs; }

struct SplitArgs {
    int32_t eps, n_wg;    // host plan: entries per wave, workgroups per (request, KV head)
    int32_t step, least;  // granularity and least value of eps
    int32_t fit;          // pieces that a plan may have
    bool planned;         // share the grid out by the counts
    bool light_last;      // every (request, KV head)'s last workgroup has fewer waves: start those last
};

// ---- the split plan ----
// The host sizes the grid for requests of k_max selected blocks each: n_wg workgroups
// per (request, KV head), whose W waves take eps entries each.  Counts live on the
// device; where they differ, that leaves long requests few waves and short ones idle
// workgroups, so the kernels share the same grid out by the counts: the least eps with
// which ceil(cnt / (W * eps)) workgroups per request and head are no more than `fit`.
// Workgroup p is piece (p / Hkv, head p % Hkv) of the requests' pieces in order; its
// partial is number p.
//
// A CU takes a second workgroup only at the cost of both (their loads share its
// address path), so `fit` is one round of workgroups (2048 waves) where that leaves a
// quarter more pieces than requests, and the grid otherwise or where the host's own
// split takes more than a round.  Without a plan, where the grid takes more than a round
// and every last workgroup has fewer waves, splits are numbered slowest, so that those
// are the ones that come second.
// Finding and following a plan costs 1 to 2 us (two memory round trips), so it is for up to
// 64 requests (one lane each) whose eps may halve, or whose empty workgroups would make a
// second round.  In us, three batches in turn: the host's split alone (before the reductions
// in registers), a plan up to the whole grid wherever counts differ, and as it is.  Over 560
// calls drawn from 1 to 32 requests and budgets of 256 to 8192 tokens, lognormal or equal, the
// second was 1.08 and this is 1.13 times as fast as the first; 101 and 11 calls lost over 1%.
//   16 requests x 65K tokens, lognormal around 2048 tokens (188 MB)    58.0  42.9  43.0
//   7 requests x 120K tokens, blocks of 32, around 2705 (100 MB)       29.3  31.1  23.1
//   20 requests, 2 KV heads, all 387 blocks (280 workgroups)           34.9  39.2  29.5
//   5 requests, 3 KV heads, around 702 tokens                          11.3  12.1  10.9
constexpr int kPlanRequests = 64;

struct Piece {
    int eps, nwg, base;  // entries per wave, workgroups of the request, its first piece
    int r, wg;
    int32_t cnt;         // selected blocks of the request (0 if the count is invalid)
};

// Workgroups of a request of c blocks: at least one, which writes an empty request's output.
__device__ inline int pieces_of(int c, int per) { return max(1, (c + per - 1) / per); }

// The same for c below 2^23, by the reciprocal, whose quotient is at most one off.
__device__ inline int pieces_short(int c, int per) {
    const int n = c + per - 1;
    int q = (int)((float)n * __builtin_amdgcn_rcpf((float)per));
    const int rest = n - q * per;
    q += rest < 0 ? -1 : rest >= per ? 1 : 0;
    return max(1, q);
}

// Whether every request has k_max blocks (raw: sel_cnt of request `lane`): the host's split as it is.
__device__ inline bool equal_counts(int32_t raw, int32_t B, int32_t k_max, int lane) {
    return __ballot(lane < B && raw != k_max) == 0;
}

// Plan for piece index pr (of all heads of a request at once); all lanes of a wave take
// part.  raw: sel_cnt of request `lane` (B <= kPlanRequests).  r < 0: no such piece.
__device__ inline Piece plan_piece(int pr, int32_t raw, int32_t B, int32_t k_max, int32_t W, const SplitArgs& sp,
                                   int lane) {
    const int c = (lane < B && raw >= 0 && raw <= k_max) ? raw : 0;
    Piece p;
    auto pieces = [&](int eps) { return lane < B ? (uint32_t)pieces_short(c, W * eps) : 0u; };
    auto sum = [&](int eps) { return (int)last_lane(wave_scan(pieces(eps), 0u, OpAdd())); };
    const int fit = sum(sp.eps) <= sp.fit ? sp.fit : B * sp.n_wg;
    int lo = sp.least, hi = sp.eps;  // hi fits: no request has more than n_wg workgroups then
    while (lo < hi) {
        const int mid = (lo + hi) / 2 / sp.step * sp.step;
        if (sum(mid) <= fit) hi = mid;
        else lo = mid + sp.step;
    }
    p.eps = hi;
    const uint32_t np = pieces(p.eps);
    const uint32_t incl = wave_scan(np, 0u, OpAdd());
    const int before = __popcll(__ballot(lane < B && (int)(incl - np) <= pr));
    p.r = pr < (int)last_lane(incl) ? before - 1 : -1;
    const int at = max(p.r, 0);
    p.nwg = __builtin_amdgcn_readlane((int)np, at);
    p.base = __builtin_amdgcn_readlane((int)(incl - np), at);
    p.cnt = __builtin_amdgcn_readlane(c, at);
    p.wg = pr - p.base;
    return p;
}

// 2^x as the hardware has it (1 ulp; results below 2^-126 are 0, far below what a sum of
// probabilities with a largest one of 1 holds).
__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Combination of the four 16-lane groups' values, in every lane: rows and halves are exchanged
// between two copies in registers (v_permlane16_swap, v_permlane32_swap), no LDS round trip.
// With this, exp2_fast and the accumulators rescaled only when a maximum moved: 8 x 2048 tokens
// 16.2 -> 15.9 us, 4 x 8192 at G 8 30.2 -> 29.9, one request of 400 tokens 8.3 -> 7.8 in the kernel.
template <typename Op>
__device__ inline float across_groups(float x, Op op) {
    const uint32_t u = __float_as_uint(x);
    const u32x2 a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float y = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uint32_t w = __float_as_uint(y);
    const u32x2 b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Attention of one wave over entries [e0, e0 + ne) of request r, KV head h;
// j_lane is the selected block of entry e0 + lane (loaded by the caller).
// Leaves the running max (log2 domain) and the lane-group-reduced sum for
// query column `col` in m_run / l_run, and O rows g = 4*grp + v in acc.
template <int DT, int BS>
__device__ inline void attend_split(const uint16_t* __restrict__ q, const uint16_t* __restrict__ pool,
                                    int32_t n_slots, const int32_t* __restrict__ table, int32_t max_blocks,
                                    int32_t j_lane, const int32_t* __restrict__ ctx_len, int32_t Hq, int32_t Hkv,
                                    int32_t G, int r, int h, int ne, float scale_log2, int32_t* status, int lane,
                                    float& m_run, float& l_run, f32x4 (&acc)[8]) {
    using M = Mfma<DT>;
    using vec = typename M::vec;
    const int col = lane & 15;  // MFMA column: query head (QK^T), channel (PV)
    const int grp = lane >> 4;  // lane group: 8-channel / 8-token slice
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run = -INFINITY;
    l_run = 0.f;
    if (ne <= 0) return;
    // entry metadata, one entry per lane (ne <= 64); the table lookup does not wait for the context length
    const int32_t j = lane < ne ? j_lane : -1;
    const int32_t sl = (j >= 0 && j < max_blocks) ? table[(size_t)r * max_blocks + j] : -1;
    const int ctx = ctx_len[r];
    const int64_t n_r = ((int64_t)ctx + BS - 1) / BS;
    int my_slot = -1, my_nv = 0;
    if (lane < ne) {
        if (j < n_r && sl >= 0 && sl < n_slots) {
            my_slot = sl;
            const int64_t v = (int64_t)ctx - (int64_t)j * BS;
            my_nv = v >= BS ? BS : (int)v;
        }
        if (my_slot < 0) report(status, PULSE_ERR_BAD_INDEX);
    }
    // Q^T operand: lane holds q[g = col][8 channels of slice grp + 32 kc]
    vec qb[4];
    {
        const uint16_t* qr = q + ((size_t)r * Hq + (size_t)h * G + col) * kHeadDim + grp * 8;
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) qb[kc] = col < G ? load_vec<DT>(qr + 32 * kc) : zero_vec<DT>();
    }
    const size_t E = (size_t)2 * Hkv * BS * kHeadDim;
    const size_t k_head = (size_t)h * BS * kHeadDim;
    const size_t v_head = (size_t)Hkv * BS * kHeadDim + (size_t)h * kHeadDim * BS;
    const int tokens = ne * BS;

    // K and V operand loads of one 32-token step starting at sequence token t0
    // K: MFMA row m = col maps to token 8*(col/4) + 4*sub + col%4;
    // V: lane group grp holds tokens 8*grp .. 8*grp+7 of channel col + 16*tile.
    auto load_k = [&](int t0, vec (&ka)[2][4]) {
        const int ka_seq = t0 + 8 * (col >> 2);
        const int ka_e = ka_seq / BS;
        const int ka_slot = __shfl(my_slot, ka_e < ne ? ka_e : 0);
        const int ka_nv = __shfl(my_nv, ka_e < ne ? ka_e : 0);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const int row = ka_seq % BS + 4 * sub + (col & 3);
            const bool ok = ka_e < ne && ka_slot >= 0 && row < ka_nv;
            const uint16_t* kp = pool + (size_t)(ok ? ka_slot : 0) * E + k_head + (size_t)row * kHeadDim + grp * 8;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) ka[sub][kc] = ok ? load_vec<DT>(kp + 32 * kc) : zero_vec<DT>();
        }
    };
    auto load_v = [&](int t0, vec (&vb)[8]) {
        const int pv_seq = t0 + 8 * grp;
        const int pv_e = pv_seq / BS;
        const int pv_slot = __shfl(my_slot, pv_e < ne ? pv_e : 0);
        const bool pv_ok = pv_e < ne && pv_slot >= 0;
        const uint16_t* vp = pool + (size_t)(pv_ok ? pv_slot : 0) * E + v_head + (size_t)col * BS + pv_seq % BS;
#pragma unroll
        for (int t = 0; t < 8; ++t) vb[t] = pv_ok ? load_vec<DT>(vp + (size_t)16 * t * BS) : zero_vec<DT>();
    };

    // One 32-token step at a time: K is loaded first, V once the S tile is issued, so
    // the V loads overlap the softmax and fewer operands are live (121-128 VGPRs and 4
    // waves per SIMD with 8-wave workgroups, up to 130 and 3 with 4-wave ones).  The
    // other resident waves hide the load latency.  Measured slower:
    // loading K and V together (154 VGPRs; 2-5%), prefetching the next step into
    // registers as well (223 VGPRs; another 1-2%), and, for splits of two steps,
    // issuing all four loads before the first product (177 VGPRs; 11% slower on
    // 8 requests x 2048 selected tokens; no faster on one request either), and keys
    // loaded with neighbouring lanes on neighbouring pieces and staged through LDS,
    // pipelined by a step (2-4% slower on 8 x 2048, equal on larger calls).
#pragma unroll 1
    for (int t0 = 0; t0 < tokens; t0 += kChunkTokens) {
        vec ka[2][4], vb[8];
        load_k(t0, ka);
        const int pv_seq = t0 + 8 * grp;
        const int pv_e = pv_seq / BS;
        const int pv_slot = __shfl(my_slot, pv_e < ne ? pv_e : 0);
        const int pv_nv = __shfl(my_nv, pv_e < ne ? pv_e : 0);
        const int pv_row = pv_seq % BS;
        const bool pv_ok = pv_e < ne && pv_slot >= 0;
        // --- S^T = K . Q^T
        f32x4 s1 = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            s1 = M::mac(ka[0][kc], qb[kc], s1);
            s2 = M::mac(ka[1][kc], qb[kc], s2);
        }
        load_v(t0, vb);
        // lane (col, grp) now holds query col, tokens pv_seq + 0..7
        float x[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = s1[i] * scale_log2;
            x[4 + i] = s2[i] * scale_log2;
        }
        float cm = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (!pv_ok || pv_row + i >= pv_nv) x[i] = -INFINITY;
            cm = fmaxf(cm, x[i]);
        }
        cm = across_groups(cm, [](float a, float b) { return fmaxf(a, b); });
        const float m_new = fmaxf(m_run, cm);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = exp2_fast(m_run - m_use);
        float psum = 0.f;
        vec ph, pl;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float p = exp2_fast(x[i] - m_use);
            psum += p;
            typename M::elem hi, lo;
            M::split(p, hi, lo);
            ph[i] = hi;
            pl[i] = lo;
        }
        l_run = l_run * alpha + psum;
        m_run = m_new;
        // rescale accumulator rows g' = 4*grp + v by alpha of query g' (not while they are zero,
        // and not when no query's maximum moved)
        if (t0 > 0 && __ballot(alpha != 1.f)) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float av = __shfl(alpha, 4 * grp + v);
#pragma unroll
                for (int t = 0; t < 8; ++t) acc[t][v] *= av;
            }
        }
        // --- O += P . V  (hi and lo parts of P)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            acc[t] = M::mac(ph, vb[t], acc[t]);
            acc[t] = M::mac(pl, vb[t], acc[t]);
        }
    }
    l_run = across_groups(l_run, [](float a, float b) { return a + b; });
}

// grid = (Hkv, n_wg, B), or (Hkv, B, n_wg) with light_last; in either, workgroup p is piece p / Hkv of KV head
// p % Hkv of a plan; wave w of a request's workgroup wg owns split W * wg + w of eps entries.  Dynamic LDS:
// O [W][G][128] floats then (m, l) [W][G] float2.
template <int DT, int BS, int W>
__global__ __launch_bounds__(W * kWave) void attn_splitk_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ pool, int32_t n_slots,
    const int32_t* __restrict__ table, int32_t max_blocks, const int32_t* __restrict__ sel_idx,
    const int32_t* __restrict__ sel_cnt, int32_t k_max, const int32_t* __restrict__ ctx_len, int32_t B, int32_t Hq,
    int32_t Hkv, int32_t G, SplitArgs sp, float scale_log2, float* __restrict__ ws_o,
    float2* __restrict__ ws_ml, float* __restrict__ out, float* __restrict__ lse, __bf16* __restrict__ x,
    int32_t* status) {
    extern __shared__ float smem[];
    constexpr int kThreads = W * kWave;
    float* s_o = smem;                                                           // [W][G][128]
    float2* s_ml = reinterpret_cast<float2*>(smem + W * G * kHeadDim);  // [W][G]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int h = blockIdx.x;

    // this wave's selected blocks (one per lane) are loaded with the counts they depend on, at the place
    // they have when all counts are equal: one memory round trip fewer before the first K load
    Piece p;
    p.r = sp.light_last ? blockIdx.y : blockIdx.z;
    p.wg = sp.light_last ? blockIdx.z : blockIdx.y;
    p.eps = sp.eps;
    int piece = p.r * sp.n_wg + p.wg;
    const bool planned = sp.planned;
    auto load_j = [&]() {
        const int e = (p.wg * W + wave) * p.eps + lane;
        return (lane < p.eps && e < k_max) ? sel_idx[(size_t)p.r * k_max + e] : -1;
    };
    int32_t j_lane = load_j();
    if (planned) {
        const int32_t raw = lane < B ? sel_cnt[lane] : 0;
        if (piece == 0 && h == 0 && wave == 0 && (raw < 0 || raw > k_max)) report(status, PULSE_ERR_BAD_INDEX);
        p.cnt = k_max;
        p.nwg = sp.n_wg;
        if (!equal_counts(raw, B, k_max, lane)) {
            const int r0 = p.r, wg0 = p.wg;
            piece = (int)(blockIdx.z * gridDim.y + blockIdx.y);
            p = plan_piece(piece, raw, B, k_max, W, sp, lane);
            if (p.r < 0) return;  // fewer pieces than workgroups
            if (p.r != r0 || p.wg != wg0 || p.eps != sp.eps) j_lane = load_j();
        }
    } else {
        p.cnt = sel_cnt[p.r];
        if (p.cnt < 0 || p.cnt > k_max) {
            if (tid == 0) report(status, PULSE_ERR_BAD_INDEX);
            p.cnt = 0;
        }
        p.nwg = pieces_of(p.cnt, W * p.eps);
        if (p.wg >= p.nwg) return;
    }
    const int r = p.r;
    float* out_rh = out + ((size_t)r * Hq + (size_t)h * G) * kHeadDim;
    float* lse_rh = lse ? lse + (size_t)r * Hq + (size_t)h * G : nullptr;
    __bf16* x_rh = x ? x + ((size_t)r * Hq + (size_t)h * G) * kHeadDim : nullptr;
    if (p.cnt == 0) {  // empty selection: out = 0, lse = -inf
        for (int i = tid; i < G * kHeadDim; i += kThreads) {
            out_rh[i] = 0.f;
            if (x_rh) x_rh[i] = (__bf16)0.f;
        }
        if (lse_rh && tid < G) lse_rh[tid] = -INFINITY;
        return;
    }
    const int ne = min(p.eps, p.cnt - (p.wg * W + wave) * p.eps);
    float m_run, l_run;
    f32x4 acc[8];
    attend_split<DT, BS>(q, pool, n_slots, table, max_blocks, j_lane, ctx_len, Hq, Hkv, G, r, h, ne, scale_log2,
                         status, lane, m_run, l_run, acc);
    // wave partials to LDS
    if (grp == 0 && col < G) s_ml[wave * G + col] = make_float2(m_run, l_run);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int g = 4 * grp + v;
        if (g < G) {
            float* o = s_o + (wave * G + g) * kHeadDim + col;
#pragma unroll
            for (int t = 0; t < 8; ++t) o[16 * t] = acc[t][v];
        }
    }
    __syncthreads();
    // merge the W waves: thread handles outputs (g, c) = (idx / 128, idx % 128)
    const size_t unit = (size_t)piece * Hkv + h;
    for (int idx = tid; idx < G * kHeadDim; idx += kThreads) {
        const int g = idx / kHeadDim, c = idx % kHeadDim;
        float Mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) Mx = fmaxf(Mx, s_ml[w * G + g].x);
        float L = 0.f, a = 0.f;
        if (Mx != -INFINITY) {
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float2 ml = s_ml[w * G + g];
                const float wt = ml.x == -INFINITY ? 0.f : exp2_fast(ml.x - Mx);
                L += ml.y * wt;
                a += s_o[(w * G + g) * kHeadDim + c] * wt;
            }
        }
        if (p.nwg == 1) {
            const float o = Mx == -INFINITY ? 0.f : a / L;
            out_rh[idx] = o;
            if (x_rh) x_rh[idx] = (__bf16)o;
            if (lse_rh && c == 0) lse_rh[g] = Mx == -INFINITY ? -INFINITY : (Mx + log2f(L)) * 0.69314718055994531f;
        } else {
            ws_o[unit * G * kHeadDim + idx] = a;
            if (c == 0) ws_ml[unit * G + g] = make_float2(Mx, L);
        }
    }
}

// Merge the workgroup partials of one (request, KV head, query head):
// grid = (G, Hkv, B), 128 threads, thread c owns output channel c.  Partials
// are read 8 at a time (16 independent loads per thread) and merged online.
// Requests whose selection fits one workgroup were finished by the attention
// kernel.
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(
    const float* __restrict__ ws_o, const float2* __restrict__ ws_ml, const int32_t* __restrict__ sel_cnt,
    int32_t k_max, int32_t B, int32_t Hq, int32_t Hkv, int32_t G, SplitArgs sp, int32_t waves,
    float* __restrict__ out, float* __restrict__ lse, __bf16* __restrict__ x) {
    const int c = threadIdx.x, g = blockIdx.x, h = blockIdx.y, r = blockIdx.z;
    // piece i of this (request, head) is partial (base + i) * Hkv + h; with equal counts base = r * n_wg.
    // The first 8 are loaded there before the counts are known, and again if the base differs.
    const float2* ml = ws_ml + (size_t)h * G + g;
    const float* po = ws_o + ((size_t)h * G + g) * kHeadDim + c;
    float2 mlv[8];
    float ov[8];
    auto load8 = [&](int first, int n) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const size_t u = (size_t)(first + i) * Hkv * G;
            mlv[i] = i < n ? ml[u] : make_float2(-INFINITY, 0.f);
            ov[i] = i < n ? po[u * kHeadDim] : 0.f;
        }
    };
    load8(r * sp.n_wg, sp.n_wg);
    int nwg, base = r * sp.n_wg;
    if (sp.planned) {
        const int lane = c & 63;
        const int32_t raw = lane < B ? sel_cnt[lane] : 0;
        nwg = sp.n_wg;
        if (!equal_counts(raw, B, k_max, lane)) {
            const Piece p = plan_piece(0, raw, B, k_max, waves, sp, lane);
            // the request's own pieces: those of lane r
            const int cl = (raw >= 0 && raw <= k_max) ? raw : 0;
            const uint32_t np = (uint32_t)pieces_short(cl, waves * p.eps);
            nwg = __builtin_amdgcn_readlane((int)np, r);
            base = (int)last_lane(wave_scan(lane < r ? np : 0u, 0u, OpAdd()));
        }
    } else {
        const int32_t cnt = sel_cnt[r];
        nwg = (cnt < 0 || cnt > k_max) ? 1 : pieces_of(cnt, waves * sp.eps);
    }
    if (nwg <= 1) return;
    if (base != r * sp.n_wg || nwg > sp.n_wg) load8(base, nwg);
    float m_run = -INFINITY, L = 0.f, a = 0.f;
    for (int w0 = 0; w0 < nwg; w0 += 8) {
        if (w0 > 0) {
            load8(base + w0, nwg - w0);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i >= nwg) {  // not written by this call
                    mlv[i] = make_float2(-INFINITY, 0.f);
                    ov[i] = 0.f;
                }
        }
        float cm = m_run;
#pragma unroll
        for (int i = 0; i < 8; ++i) cm = fmaxf(cm, mlv[i].x);
        if (cm == -INFINITY) continue;
        const float alpha = m_run == -INFINITY ? 0.f : exp2f(m_run - cm);
        L *= alpha;
        a *= alpha;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float wt = mlv[i].x == -INFINITY ? 0.f : exp2f(mlv[i].x - cm);
            L += mlv[i].y * wt;
            a += ov[i] * wt;
        }
        m_run = cm;
    }
    const size_t at = ((size_t)r * Hq + (size_t)h * G + g) * kHeadDim + c;
    const float o = m_run == -INFINITY ? 0.f : a / L;
    out[at] = o;
    if (x) x[at] = (__bf16)o;
    if (lse && c == 0)
        lse[(size_t)r * Hq + (size_t)h * G + g] =
            m_run == -INFINITY ? -INFINITY : (m_run + log2f(L)) * 0.69314718055994531f;
}

AttnPlan attn_plan(int32_t B, int32_t Hkv, int32_t k_max, int32_t bs) {
    // a split covers whole 32-token steps, at least two, and at most 64 entries
    const int32_t step = split_step(bs);
    const int64_t units = (int64_t)B * Hkv;
    const int64_t target_waves = PULSE_ATTN_TARGET_WAVES;  // one round at 2 resident waves per SIMD on 256 CUs
    int64_t want = units > 0 ? (target_waves + units - 1) / units : 1;
    const int64_t min_entries = split_least(bs);
    int64_t max_split = (k_max + min_entries - 1) / min_entries;
    if (want > max_split) want = max_split;
    if (want < 1) want = 1;
    int64_t eps = (k_max + want - 1) / want;
    eps = ((eps + step - 1) / step) * step;
    if (eps > 64) eps = 64;
    if (eps < 1) eps = 1;
    AttnPlan p;
    p.entries_per_split = (int32_t)eps;
    p.n_split = (int32_t)((k_max + eps - 1) / eps);
    return p;
}

// `done` (optional): the kernel's stop event, carried by the launch.
template <int DT, int BS, int W>
static void launch_attn_t(dim3 grid, size_t lds, hipStream_t st, hipEvent_t done, const void* q, const void* pool,
                          int32_t n_slots, const int32_t* table, int32_t max_blocks, const int32_t* sel_idx,
                          const int32_t* sel_cnt, int32_t k_max, const int32_t* ctx_len, int32_t B, int32_t Hq,
                          int32_t Hkv, int32_t G, const SplitArgs& sp, float scale_log2, float* ws_o, float2* ws_ml,
                          float* out, float* lse, __bf16* x, int32_t* status) {
    launch_timed(attn_splitk_kernel<DT, BS, W>, grid, dim3(W * kWave), (uint32_t)lds, st, nullptr, done,
                 (const uint16_t*)q, (const uint16_t*)pool, n_slots, table, max_blocks, sel_idx, sel_cnt, k_max,
                 ctx_len, B, Hq, Hkv, G, sp, scale_log2, ws_o, ws_ml, out, lse, x, status);
}

hipError_t launch_attention(const pulse_shape& s, const void* q, const void* pool, int32_t n_slots,
                            const int32_t* table, int32_t max_blocks, const int32_t* sel_idx, const int32_t* sel_cnt,
                            int32_t k_max, const int32_t* ctx_len, int32_t B, float sm_scale, float* out, float* lse,
                            float* ws_o, float2* ws_ml, int32_t* status, hipStream_t st, hipEvent_t split_done,
                            hipEvent_t done, __bf16* x) {
    if (B == 0) return hipSuccess;
    const int32_t Hkv = s.num_kv_heads, Hq = s.num_q_heads, G = Hq / Hkv;
    const AttnPlan p = attn_plan(B, Hkv, k_max, s.block_size);
    const int W = attn_waves(G);
    const int32_t n_wg = (p.n_split + W - 1) / W;
    SplitArgs sp;
    sp.eps = p.entries_per_split;
    sp.n_wg = n_wg;
    sp.step = split_step(s.block_size);
    sp.least = split_least(s.block_size);
    const int64_t all = (int64_t)B * n_wg;
    const int32_t round = PULSE_ATTN_TARGET_WAVES / (W * Hkv);  // pieces of one round
    sp.fit = (int32_t)(4 * (int64_t)round >= 5 * (int64_t)B && round < all ? round : all);
    sp.planned = n_wg > 1 && B <= kPlanRequests && (sp.eps >= 2 * sp.least || all > round) && k_max <= (1 << 22);
    sp.light_last = p.n_split % W != 0 && all > round && n_wg <= 65535;
    const dim3 grid = sp.light_last ? dim3((unsigned)Hkv, (unsigned)B, (unsigned)n_wg)
                                    : dim3((unsigned)Hkv, (unsigned)n_wg, (unsigned)B);
    const size_t lds = sizeof(float) * W * G * kHeadDim + sizeof(float2) * W * G;
    const float scale_log2 = sm_scale * 1.4426950408889634f;
    // stop event of the split-K kernel: split_done, or `done` when no combine follows it
    const hipEvent_t splitk_stop = split_done ? split_done : (n_wg <= 1 ? done : nullptr);
#define PULSE_ATTN(DT, BS, W)                                                                                        \
    launch_attn_t<DT, BS, W>(grid, lds, st, splitk_stop, q, pool, n_slots, table, max_blocks, sel_idx, sel_cnt,     \
                             k_max, ctx_len, B, Hq, Hkv, G, sp, scale_log2, ws_o, ws_ml, out, lse, x, status)
#define PULSE_ATTN_W(DT, BS) \
    if (W == 8) PULSE_ATTN(DT, BS, 8); else PULSE_ATTN(DT, BS, 4)
    if (s.dtype == PULSE_BF16) {
        if (s.block_size == 16) PULSE_ATTN_W(PULSE_BF16, 16);
        else if (s.block_size == 32) PULSE_ATTN_W(PULSE_BF16, 32);
        else PULSE_ATTN_W(PULSE_BF16, 64);
    } else {
        if (s.block_size == 16) PULSE_ATTN_W(PULSE_F16, 16);
        else if (s.block_size == 32) PULSE_ATTN_W(PULSE_F16, 32);
        else PULSE_ATTN_W(PULSE_F16, 64);
    }
#undef PULSE_ATTN_W
#undef PULSE_ATTN
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (n_wg <= 1) return (done && split_done) ? hipEventRecord(done, st) : hipSuccess;
    launch_timed(attn_combine_kernel, dim3((unsigned)G, (unsigned)Hkv, (unsigned)B), dim3(kCombineThreads), 0u, st,
                 nullptr, done, (const float*)ws_o, (const float2*)ws_ml, sel_cnt, k_max, B, Hq, Hkv, G, sp, W, out, lse,
                 x);
    return hipGetLastError();
}

}  // namespace pulse
