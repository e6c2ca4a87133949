// variants.hip -- the selection strategies the paper compares SoloHead with,
// and the Middle Attention Mass that picks the solo head (Sec. 4.4.1, Eq. 2).
//
// Average selection: every KV head scores the blocks with its own digests,
// the scores are averaged over the heads (digest.hip), and one top-k on the
// average is shared by all heads.  Averaging the per-KV-head scores (each
// already the mean over its G query heads) is the mean over all query heads.
//
// MAM: for query head q, the softmax mass of its full attention that falls on
// middle tokens is (sum of exp(logit) over the middle tokens) / (the same sum
// over all tokens); a KV head's MAM is the mean over its G query heads.  One
// pass over the keys of the whole context accumulates both sums under one
// running maximum; values are not read.  Middle blocks are those that selection
// ranks: neither the first n_sink nor the last n_local.  The highest-MAM head
// is the SoloHead, the lowest the "reversed" choice.
#include "pulse_internal.h"

namespace pulse {

constexpr int kMamWaves = 4;
// Waves of a call: two per SIMD.  4 x 32K tokens took 58.0 / 59.1 / 58.1 us at 2048 / 4096 / 8192, one request
// of 55K tokens with 4 KV heads 19.0 / 20.6 / 20.6 (more partials to merge).
constexpr int64_t kMamTargetWaves = 2048;
constexpr int kMamStep = 32;  // tokens per MFMA step

// Softmax sums of one query column over part of the context.
struct MamSum {
    float m = -INFINITY, all = 0.f, mid = 0.f;  // running max (log2 domain), sums of exp2(x - m)
    __device__ void merge(float m2, float all2, float mid2) {
        const float mn = fmaxf(m, m2);
        // without a maximum on either side the sums are 0, or NaN where every logit is (a maximum skips NaN)
        if (mn == -INFINITY) {
            all += all2;
            mid += mid2;
            return;
        }
        const float a = exp2f(m - mn), b = exp2f(m2 - mn);
        all = all * a + all2 * b;
        mid = mid * a + mid2 * b;
        m = mn;
    }
    __device__ void merge_lanes(int off) {
        merge(__shfl_xor(m, off), __shfl_xor(all, off), __shfl_xor(mid, off));
    }
    // 0 where nothing was summed; a NaN among the logits reaches the mass
    __device__ float mass() const { return all == 0.f ? 0.f : mid / all; }
};

// Whether a request of n blocks has middle blocks; without any its mass is 0, whatever the logits are.
__device__ inline bool has_middle(int n, int n_sink, int n_local) { return n_sink < n - n_local; }

// Mean of the G heads' masses, summed in ascending order; lane g holds head g's.
__device__ inline float mean_mass(float mass, int G) {
    float s = 0.f;
    for (int g = 0; g < G; ++g) s += __shfl(mass, g);
    return s / (float)G;
}

// grid = (n_wg, Hkv, B); wave w of a workgroup owns the blocks [s * epw, (s + 1) * epw)
// of the request, s = blockIdx.x * kMamWaves + w.  Bound by HBM: 256 bytes per token and
// KV head, each read once.  A step is 32 tokens on v_mfma_f32_16x16x32 (S^T[tokens x heads] =
// K . Q^T, the operand layout of the attention kernel); the keys of the next step are loaded
// before this step's products.  Every lane keeps the sums of its own query column and token
// group, so the loop exchanges nothing between lanes.  Lanes, waves and workgroups are merged
// at the end; with one workgroup per (request, head) it writes the mean itself, otherwise
// partials [B][Hkv][n_wg][G] of (max, sum over all, sum over the middle).
template <int DT, int BS>
__global__ __launch_bounds__(kMamWaves * kWave) void mam_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ pool, int32_t n_slots,
    const int32_t* __restrict__ table, int32_t max_blocks, const int32_t* __restrict__ ctx_len, int32_t Hq,
    int32_t G, int32_t n_sink, int32_t n_local, int32_t epw, float scale_log2, float4* __restrict__ part,
    float* __restrict__ mam, int32_t* status) {
    using M = Mfma<DT>;
    using vec = typename M::vec;
    __shared__ float4 s_part[kMamWaves][kMaxGroup];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int wg = blockIdx.x, n_wg = gridDim.x, h = blockIdx.y, Hkv = gridDim.y, r = blockIdx.z;
    const int e0 = (wg * kMamWaves + wave) * epw;
    // the wave's table entries (one per lane) are loaded with the context length, not after it
    const int j = e0 + lane;
    const int32_t slot_any = (lane < epw && j < max_blocks) ? table[(size_t)r * max_blocks + j] : -1;
    const int64_t ctx = ctx_len[r];
    vec qb[4];
    {
        const uint16_t* qr = q + ((size_t)r * Hq + (size_t)h * G + col) * kHeadDim + grp * 8;
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) qb[kc] = col < G ? load_vec<DT>(qr + 32 * kc) : zero_vec<DT>();
    }
    int64_t n64 = ctx > 0 ? (ctx + BS - 1) / BS : 0;
    if (n64 > max_blocks) {  // the table row cannot hold this request
        if (wg == 0 && h == 0 && tid == 0) report(status, PULSE_ERR_BAD_INDEX);
        n64 = 0;
    }
    const int n = (int)n64;
    if (wg * kMamWaves * epw >= n && wg > 0) return;  // no block of this workgroup (workgroup 0 writes an empty request's 0)
    const int ne = min(epw, n - e0);  // may be negative
    int my_slot = -1, my_nv = 0;
    if (lane < ne) {
        my_slot = slot_any >= 0 && slot_any < n_slots ? slot_any : -1;
        if (my_slot < 0) {
            report(status, PULSE_ERR_BAD_INDEX);
        } else {
            const int64_t v = ctx - (int64_t)j * BS;
            my_nv = v >= BS ? BS : (int)v;
        }
    }
    const bool my_mid = j >= n_sink && j < n - n_local;
    const uint64_t mid_mask = __ballot(my_mid);
    const size_t E = (size_t)2 * Hkv * BS * kHeadDim;
    const uint16_t* head = pool + (size_t)h * BS * kHeadDim + (size_t)col * kHeadDim + grp * 8;
    const int steps = (max(ne, 0) * BS + kMamStep - 1) / kMamStep;
    // rows 16 * sub + col of step t: entry and row of each 16-token half are wave-uniform
    auto load_k = [&](int t, vec (&ka)[2][4]) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const int t16 = 2 * t + sub, e = t16 / (BS / 16);
            const int slot = e < ne ? __builtin_amdgcn_readlane(my_slot, e) : -1;
            const uint16_t* kp = head + (size_t)max(slot, 0) * E + (size_t)(t16 % (BS / 16)) * 16 * kHeadDim;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) ka[sub][kc] = slot >= 0 ? load_vec<DT>(kp + 32 * kc) : zero_vec<DT>();
        }
    };
    MamSum sum;
    auto accumulate = [&](int t, const vec (&ka)[2][4]) {
        float x[2][4];
        float cm = -INFINITY;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) s = M::mac(ka[sub][kc], qb[kc], s);
            const int t16 = 2 * t + sub, e = t16 / (BS / 16);
            const int nv = e < ne ? __builtin_amdgcn_readlane(my_nv, e) : 0;
            const int row = (t16 % (BS / 16)) * 16 + 4 * grp;  // this lane's four tokens of the block
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x[sub][v] = row + v < nv ? s[v] * scale_log2 : -INFINITY;
                cm = fmaxf(cm, x[sub][v]);
            }
        }
        const float m_new = fmaxf(sum.m, cm);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = exp2f(sum.m - m_use);
        sum.all *= alpha;
        sum.mid *= alpha;
        sum.m = m_new;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const int e = (2 * t + sub) / (BS / 16);
            float p = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) p += exp2f(x[sub][v] - m_use);
            sum.all += p;
            sum.mid += ((mid_mask >> (e & 63)) & 1u) ? p : 0.f;
        }
    };
    if (steps > 0) {
        vec ka[2][4], kb[2][4];
        load_k(0, ka);
        for (int t = 0; t < steps; t += 2) {  // past the last step: nothing is loaded, everything masked
            load_k(t + 1, kb);
            accumulate(t, ka);
            load_k(t + 2, ka);
            accumulate(t + 1, kb);
        }
    }
    sum.merge_lanes(16);
    sum.merge_lanes(32);
    if (lane < kMaxGroup) s_part[wave][lane] = make_float4(sum.m, sum.all, sum.mid, 0.f);
    __syncthreads();
    if (wave > 0) return;
    MamSum tot;
#pragma unroll
    for (int w = 0; w < kMamWaves; ++w) tot.merge(s_part[w][col].x, s_part[w][col].y, s_part[w][col].z);
    if (n_wg == 1) {
        const float mean = mean_mass(tot.mass(), G);
        if (lane == 0) mam[(size_t)r * Hkv + h] = has_middle(n, n_sink, n_local) ? mean : 0.f;
    } else if (lane < G) {
        part[(((size_t)r * Hkv + h) * n_wg + wg) * G + lane] = make_float4(tot.m, tot.all, tot.mid, 0.f);
    }
}

// Merge of the workgroup partials: grid = (Hkv, B); thread = (query head, one of
// kMamMergeThreads / 16 streams of partials), so a context split over hundreds of
// workgroups is a few dependent merges per thread (with one wave per head, 217 partials
// of a 55K-token request, 4 KV heads, took most of the call: 36 us, now 19).
constexpr int kMamMergeThreads = 512;

__global__ __launch_bounds__(kMamMergeThreads) void mam_merge_kernel(const float4* __restrict__ part, int32_t n_wg,
                                                                     const int32_t* __restrict__ ctx_len, int32_t bs,
                                                                     int32_t max_blocks, int32_t epw, int32_t G,
                                                                     int32_t n_sink, int32_t n_local,
                                                                     float* __restrict__ mam) {
    constexpr int kStreams = kMamMergeThreads / kMaxGroup;
    __shared__ float4 s_part[kMamMergeThreads / kWave][kMaxGroup];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane & 15;
    const int h = blockIdx.x, Hkv = gridDim.x, r = blockIdx.y;
    const int64_t ctx = ctx_len[r];
    int64_t n = ctx > 0 ? (ctx + bs - 1) / bs : 0;
    if (n > max_blocks) n = 0;
    const int per = kMamWaves * epw;
    const int nw = n > 0 ? (int)((n + per - 1) / per) : 1;  // workgroups that wrote a partial
    const float4* p = part + ((size_t)r * Hkv + h) * n_wg * G;
    MamSum sum;
    if (g < G) {
#pragma unroll 4
        for (int i = tid >> 4; i < nw; i += kStreams) {
            const float4 v = p[(size_t)i * G + g];
            sum.merge(v.x, v.y, v.z);
        }
    }
    sum.merge_lanes(16);
    sum.merge_lanes(32);
    if (lane < kMaxGroup) s_part[wave][lane] = make_float4(sum.m, sum.all, sum.mid, 0.f);
    __syncthreads();
    if (wave > 0) return;
    MamSum tot;
    for (int w = 0; w < kMamMergeThreads / kWave; ++w) tot.merge(s_part[w][g].x, s_part[w][g].y, s_part[w][g].z);
    const float mean = mean_mass(tot.mass(), G);
    if (lane == 0) mam[(size_t)r * Hkv + h] = has_middle((int)n, n_sink, n_local) ? mean : 0.f;
}

MamPlan mam_plan(int32_t B, int32_t Hkv, int32_t max_blocks, int32_t bs) {
    const int64_t units = (int64_t)B * Hkv;
    const int32_t step = bs >= kMamStep ? 1 : kMamStep / bs;
    const int32_t least = bs >= 2 * kMamStep ? 1 : 2 * kMamStep / bs;  // two steps: one in flight during the other
    int64_t want = units > 0 ? (kMamTargetWaves + units - 1) / units : 1;
    int64_t epw = (max_blocks + want - 1) / want;
    epw = (epw + step - 1) / step * step;
    if (epw < least) epw = least;
    if (epw > kWave) epw = kWave;
    MamPlan p;
    p.entries_per_wave = (int32_t)epw;
    p.n_wg = (int32_t)((max_blocks + epw * kMamWaves - 1) / (epw * kMamWaves));
    return p;
}

hipError_t launch_mam(const pulse_shape& s, const void* q, const void* pool, int32_t n_slots, const int32_t* table,
                      int32_t max_blocks, const int32_t* ctx_len, int32_t B, int32_t n_sink, int32_t n_local,
                      float sm_scale, float* mam, float4* part, int32_t* status, hipStream_t st) {
    const int32_t Hkv = s.num_kv_heads, Hq = s.num_q_heads, G = Hq / Hkv;
    const MamPlan p = mam_plan(B, Hkv, max_blocks, s.block_size);
    const dim3 grid((unsigned)p.n_wg, (unsigned)Hkv, (unsigned)B);
    const float scale_log2 = sm_scale * 1.4426950408889634f;
#define PULSE_MAM(DT, BS)                                                                                           \
    hipLaunchKernelGGL((mam_kernel<DT, BS>), grid, dim3(kMamWaves * kWave), 0, st, (const uint16_t*)q,              \
                       (const uint16_t*)pool, n_slots, table, max_blocks, ctx_len, Hq, G, n_sink, n_local,          \
                       p.entries_per_wave, scale_log2, part, mam, status)
    if (s.dtype == PULSE_BF16) {
        if (s.block_size == 16) PULSE_MAM(PULSE_BF16, 16);
        else if (s.block_size == 32) PULSE_MAM(PULSE_BF16, 32);
        else PULSE_MAM(PULSE_BF16, 64);
    } else {
        if (s.block_size == 16) PULSE_MAM(PULSE_F16, 16);
        else if (s.block_size == 32) PULSE_MAM(PULSE_F16, 32);
        else PULSE_MAM(PULSE_F16, 64);
    }
#undef PULSE_MAM
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.n_wg == 1) return e;
    hipLaunchKernelGGL(mam_merge_kernel, dim3((unsigned)Hkv, (unsigned)B), dim3(kMamMergeThreads), 0, st, (const float4*)part,
                       p.n_wg, ctx_len, s.block_size, max_blocks, p.entries_per_wave, G, n_sink, n_local, mam);
    return hipGetLastError();
}

}  // namespace pulse
