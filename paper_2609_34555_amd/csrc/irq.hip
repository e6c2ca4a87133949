// irq.hip -- interruptible layer-wise scheduling (IRQ, Sec. 4.2) of an offload
// batch (the sparse-KV path of this library) against a normal batch whose
// KV cache is resident in HBM, with semi-synchronous completion detection
// (Sec. 4.2.2).
//
// Offload layer m: score + select + recall plan on the compute stream; the
// recall copy on the I/O stream, followed by a one-thread signal kernel that
// writes m's sequence number into pinned, host-mapped memory (the "interrupt
// line": the host reads it without any driver call).  Alternatively the recall
// goes through the gather-scatter engine (CPU gather, one DMA per batch, GPU
// scatter), whose completion is host-visible the same way.  On MI355X, kernels
// on other streams make little progress through the XCDs on which a kernel
// streams from host memory (their memory requests wait behind the host reads),
// so here the gather kernel copies from one XCD only; the engine's DMA leaves
// every XCD to the normal batch.  While that recall is in
// flight the host keeps enqueuing normal-batch layers on the compute stream
// and, at each normal layer boundary, checks the flag.  Once it is set, the
// offload batch's attention for layer m is enqueued on the compute stream
// behind a stream wait on the recall's completion event (the host read orders
// nothing on the GPU), then layer m + 1's selection, which issues the next
// recall, and so on.
//
// Detection modes (Sec. 4.2.2):
//   SEMI_SYNC  after enqueuing a normal layer (attention, then FFN) the host
//              waits for its attention only, then checks the flag while the
//              FFN still runs;
//   SYNC       the host waits for the whole normal layer before checking;
//   ASYNC      the host never waits for normal layers (up to `async_ahead`
//              queued), checking the flag between enqueues;
//   BLOCKING   no interleaving: each offload layer waits for its recall with
//              no other work, then one normal layer runs (a single-batch
//              schedule, the baseline).  With the gather kernel everything is
//              in one stream, and the host does not look at the flag.
//
// A normal-batch layer is decode attention over its resident KV (every
// block selected; the attention kernel of this library) followed by a SwiGLU
// FFN on the attention output: x = bf16(out) (written by the attention), [g|u] = x W_gu^T, h = silu(g) *
// u, y = h W_down^T (bf16, fp32 accumulation; the two GEMMs are the MFMA
// kernel below).  Projections and norms are left out.
#include <chrono>
#include <vector>

#include "pulse_internal.h"

namespace pulse {

__global__ void irq_signal_kernel(int64_t* flag, int64_t value) {
    if (threadIdx.x == 0 && blockIdx.x == 0)
        __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ inline __bf16 swiglu(float g, float u) { return (__bf16)(g / (1.f + expf(-g)) * u); }

// x = bf16(out) and h = silu(g) * u in launches of their own: for layers whose x or h shares memory with what the
// attention or the gate and up product, which write them otherwise, still read.
__global__ __launch_bounds__(256) void to_bf16_kernel(const float* in, __bf16* out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        out[i] = (__bf16)in[i];
}

__global__ __launch_bounds__(256) void swiglu_kernel(const __bf16* gu, __bf16* h, int32_t F, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t b = i / F, c = i % F;
        h[i] = swiglu((float)gu[b * 2 * F + c], (float)gu[b * 2 * F + F + c]);
    }
}

static unsigned grid_for(int64_t n) { return (unsigned)((n < 4096 * 256 ? n + 255 : 4096 * 256) / 256); }

// ---- the FFN's GEMMs ------------------------------------------------------
// C[M][N] = A[M][K] . Wt[N][K]^T with bf16 inputs, fp32 accumulation and a bf16
// (round-to-nearest-even) result: the shape of a decode batch's projections,
// M (requests) small and N, K model widths, so the weights, read once, bound
// both products.  A workgroup of WV waves owns CT column tiles of 16 (PAIR: CT
// gate tiles and the CT up tiles they are multiplied with) and 16 * MT rows; its
// waves split K, each taking groups of U 32-element steps, and their partial
// tiles are summed in LDS.  Products are v_mfma_f32_16x16x32_bf16 (B operand:
// column = lane % 16, k = 8 * (lane / 16) ...; A operand likewise by rows; lane
// holds rows 4 * (lane / 16) + v, column lane % 16).
//
// In that operand layout neighbouring lanes hold different rows, and a load in
// it costs the cache one lookup per lane: about one 16-byte piece per clock and
// CU, which, not HBM, bound these products (32 x 14336 x 4096: activations
// alone 26 us, weights alone 23, both 45, whatever was in flight).  So each wave loads
// its rows with neighbouring lanes on neighbouring pieces, puts them into its
// own part of LDS and reads the operands there; piece p of row r lies at
// position p ^ r, which spreads the 16 rows of an operand over all banks.
// The next group is loaded before this one's products.  Workgroups start at
// different groups of K (rows are a multiple of 4 KiB apart, so in step they
// would all ask the same L2 channels; 1 us).  Weights are loaded non-temporally:
// the activations, read by every workgroup, then stay in L2.
// K must be a multiple of 8 and rows 16-byte aligned.
template <int MT, int CT, int U, int WV, bool PAIR>
__global__ __launch_bounds__(WV * kWave) void ffn_gemm_kernel(const __bf16* __restrict__ A,
                                                              const __bf16* __restrict__ Wt,
                                                              __bf16* __restrict__ C, __bf16* __restrict__ H,
                                                              int32_t M, int32_t N, int32_t K) {
    constexpr int NT = PAIR ? 2 * CT : CT;  // column tiles: CT of the output (PAIR: CT gate tiles, then CT up tiles)
    constexpr int PP = 4 * U;                   // 16-byte pieces of a row in one group of steps
    constexpr int RT = MT + NT;                 // row tiles staged per group: activations, then weights
    constexpr int NA = 16 * MT * PP / kWave, NB = 16 * NT * PP / kWave;  // pieces a lane stages per group
    constexpr int kStage = WV * 16 * RT * PP * 16, kRed = WV * NT * MT * 4 * kWave * 4;
    __shared__ __align__(16) uint8_t smem[kStage > kRed ? kStage : kRed];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int col = lane & 15, grp = lane >> 4;
    const int n0 = blockIdx.x * 16 * CT, m0 = blockIdx.y * 16 * MT;
    // columns past N and rows past M repeat the first one; their products are dropped
    const __bf16* wrow[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = n0 + nt % CT * 16 + col;
        wrow[nt] = Wt + ((size_t)(nt / CT) * N + (n < N ? n : 0)) * K + grp * 8;
    }
    const __bf16* arow[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = m0 + 16 * mt + col;
        arow[mt] = A + (size_t)(m < M ? m : 0) * K + grp * 8;
    }
    f32x4 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4* stage = reinterpret_cast<u32x4*>(smem) + wave * 16 * RT * PP;
    const __bf16* astage[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = (i * kWave + lane) / PP, p = lane % PP;
        astage[i] = A + (size_t)(m0 + row < M ? m0 + row : 0) * K + (p ^ (row % PP)) * 8;
    }
    const __bf16* wstage[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = (i * kWave + lane) / PP, p = lane % PP;
        const int n = n0 + row % (16 * CT);
        wstage[i] = Wt + ((size_t)(row / (16 * CT)) * N + (n < N ? n : 0)) * K + (p ^ (row % PP)) * 8;
    }
    auto load = [&](int j, u32x4 (&a)[NA], u32x4 (&b)[NB]) {
#pragma unroll
        for (int i = 0; i < NA; ++i) a[i] = *reinterpret_cast<const u32x4*>(astage[i] + j * U * 32);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            b[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wstage[i] + j * U * 32));
        __builtin_amdgcn_sched_barrier(0);  // ahead of the products that follow
    };
    auto products = [&](const u32x4 (&a)[NA], const u32x4 (&b)[NB]) {
#pragma unroll
        for (int i = 0; i < NA; ++i) stage[i * kWave + lane] = a[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) stage[(NA + i) * kWave + lane] = b[i];
        wave_lds_order();
        auto frag = [&](int tile, int u) {
            return stage[(16 * tile + col) * PP + ((u * 4 + grp) ^ (col % PP))];
        };
#pragma unroll
        for (int u = 0; u < U; ++u) {
            u32x4 bv[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bv[nt] = frag(MT + nt, u);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const u32x4 av = frag(mt, u);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                                          __builtin_bit_cast(bf16x8, bv[nt]),
                                                                          acc[nt][mt], 0, 0, 0);
            }
        }
        wave_lds_order();  // the next group overwrites the rows
    };
    // Groups that lie within K, every WV-th to each wave, loaded without a test (a test per load
    // makes the compiler wait for all loads in flight at every product).
    u32x4 a0[NA], a1[NA], b0[NB], b1[NB];
    const int groups = K / (32 * U);
    if (wave < groups) {
        const int mine = (groups - wave + WV - 1) / WV;
        const int rot = (int)(blockIdx.x / 8) % mine;
        auto at = [&](int i) { const int ii = i + rot; return wave + (ii < mine ? ii : ii - mine) * WV; };
        load(at(0), a0, b0);
        int i = 0;
        for (; i + 2 < mine; i += 2) {
            load(at(i + 1), a1, b1);
            products(a0, b0);
            load(at(i + 2), a0, b0);
            products(a1, b1);
        }
        if (i + 1 < mine) {
            load(at(i + 1), a1, b1);
            products(a0, b0);
            products(a1, b1);
        } else {
            products(a0, b0);
        }
    }
    if (wave == groups % WV) {  // the rest of K: whole steps and a last one of 8, 16 or 24 elements
        for (int k = groups * 32 * U; k < K; k += 32) {
            const bool ok = k + grp * 8 < K;
            const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const u32x4 bv = ok ? *reinterpret_cast<const u32x4*>(wrow[nt] + k) : zero;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const u32x4 av = ok ? *reinterpret_cast<const u32x4*>(arow[mt] + k) : zero;
                    acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                                          __builtin_bit_cast(bf16x8, bv),
                                                                          acc[nt][mt], 0, 0, 0);
                }
            }
        }
    }
    __syncthreads();  // the staged rows are read
    float(*red)[NT][MT][4][kWave] = reinterpret_cast<float(*)[NT][MT][4][kWave]>(smem);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][nt][mt][v][lane] = acc[nt][mt][v];
    __syncthreads();
    for (int o = tid; o < 16 * MT * 16 * CT; o += WV * kWave) {
        const int ml = o / (16 * CT), nl = o % (16 * CT);  // row of the workgroup's rows, column of its columns
        const int mt = ml / 16, i = ml % 16;
        const int v = i % 4, src = (i / 4) * 16 + nl % 16;
        float sum[NT / CT];
#pragma unroll
        for (int p = 0; p < NT / CT; ++p) {
            sum[p] = 0.f;
#pragma unroll
            for (int w = 0; w < WV; ++w) sum[p] += red[w][p * CT + nl / 16][mt][v][src];
        }
        const int m = m0 + ml, nn = n0 + nl;
        if (m >= M || nn >= N) continue;
        if constexpr (PAIR) {
            const __bf16 gb = (__bf16)sum[0], ub = (__bf16)sum[1];
            C[(size_t)m * 2 * N + nn] = gb;
            C[(size_t)m * 2 * N + N + nn] = ub;
            if (H) H[(size_t)m * N + nn] = swiglu((float)gb, (float)ub);
        } else {
            C[(size_t)m * N + nn] = (__bf16)sum[0];
        }
    }
}

// PAIR: gu [M][2N] = A . Wt^T for the N gate and N up rows of Wt, H [M][N] (optional) = silu(g) * u of the rounded
// values.
//
// Tiles, at 32 rows (M <= 32; larger M reads the weights once per 64 rows):
//   gate and up, 4096 -> 2 x 14336 (235 MB): two tiles of each per workgroup of 4 waves, so that the activations
//   are read half as often, 40.7 us (5.8 TB/s); one tile, 8 waves 47.2; two tiles, 8 waves 46.1; two tiles in steps
//   of 1 59.3.  Below 512 column tiles two per workgroup would leave CUs idle.
//   down, 14336 -> 4096 (117 MB): one tile, 8 waves, steps of 4: 27.8 us (4.2 TB/s); two tiles (half the CUs) 34.7;
//   steps of 2 29.9, 16 waves in steps of 2 30.8.
// The form before, operands loaded in their layout: 61.4 us + 4.8 of a SwiGLU kernel, and 49.7.
// Above 32 rows four row tiles and one column tile, 8 waves in steps of 2 (96 and 80 KiB of LDS, one workgroup per
// CU): at 64 rows gate and up 63.3 us (3.7 TB/s), down 42.2, before 148.3 + 5.1 and 78.0; at 256 rows, the weights
// read four times, 231 and 162, before 593 + 10 and 307.
template <bool PAIR>
static hipError_t launch_ffn_gemm(const void* A, const void* Wt, void* C, void* H, int32_t M, int32_t N, int32_t K,
                                  hipStream_t st) {
    const unsigned nx = (unsigned)((N + 15) / 16);
#define PULSE_GEMM(MT, CT, U, WV)                                                                                    \
    hipLaunchKernelGGL((ffn_gemm_kernel<MT, CT, U, WV, PAIR>),                                                       \
                       dim3((nx + CT - 1) / CT, (unsigned)((M + 16 * MT - 1) / (16 * MT))), dim3(WV * kWave), 0, st, \
                       (const __bf16*)A, (const __bf16*)Wt, (__bf16*)C, (__bf16*)H, M, N, K)
    if (M > 32) {
        PULSE_GEMM(4, 1, 2, 8);
    } else if constexpr (PAIR) {
        if (nx >= 512) {
            if (M <= 16) PULSE_GEMM(1, 2, 2, 4);
            else PULSE_GEMM(2, 2, 2, 4);
        } else {
            if (M <= 16) PULSE_GEMM(1, 1, 2, 8);
            else PULSE_GEMM(2, 1, 2, 8);
        }
    } else {
        if (M <= 16) PULSE_GEMM(1, 1, 4, 8);
        else PULSE_GEMM(2, 1, 4, 8);
    }
#undef PULSE_GEMM
    return hipGetLastError();
}

// The gather kernel copies from one XCD while normal-batch layers run: the link rate
// holds and the other XCDs keep serving HBM (from all XCDs, the concurrent layers
// would barely progress until the recall ends).
constexpr int32_t kIrqRecallXcds = 1;

}  // namespace pulse

namespace pulse {
// gather_engine.hip: whether an engine was created for shape `s` (its block size and
// staging are that shape's)
bool gs_engine_serves(const pulse_gs_engine* e, const pulse_shape& s);
}  // namespace pulse

using namespace pulse;

struct pulse_irq {
    hipStream_t cmp = nullptr, io = nullptr;
    int64_t* flag_host = nullptr;  // pinned, host-mapped
    int64_t* flag_dev = nullptr;
    int64_t seq = 0;
    std::vector<hipEvent_t> events;  // grown on demand, reused across steps
    size_t next_event = 0;

    hipEvent_t event() {
        if (next_event == events.size()) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) return nullptr;
            events.push_back(e);
        }
        return events[next_event++];
    }
    bool flag_reached(int64_t v) const { return __atomic_load_n(flag_host, __ATOMIC_ACQUIRE) >= v; }
};

static pulse_status check_normal(const pulse_normal_layer* n) {
    PULSE_REQUIRE(n && shape_supported(&n->shape), PULSE_ERR_INVALID_ARG);
    PULSE_REQUIRE(n->B >= 1 && n->k_max >= 1 && n->max_blocks >= 1 && n->n_slots >= 1 && n->d_ff >= 1,
                  PULSE_ERR_INVALID_ARG);
    PULSE_REQUIRE(n->q && n->slot_pool && n->block_table && n->sel_idx && n->sel_cnt && n->ctx_len && n->out &&
                      n->w_gate_up && n->w_down && n->x && n->gu && n->h && n->y && n->dev_status,
                  PULSE_ERR_INVALID_ARG);
    PULSE_REQUIRE(n->ws && n->ws_bytes >= ws_layout(n->shape, n->B, n->k_max, 0).total, PULSE_ERR_WORKSPACE);
    // the FFN GEMMs load 16-byte pieces of rows of length D and d_ff
    PULSE_REQUIRE(n->d_ff % 8 == 0, PULSE_ERR_UNSUPPORTED);
    for (const void* p : {n->w_gate_up, n->w_down, (const void*)n->x, (const void*)n->h})
        PULSE_REQUIRE(((uintptr_t)p & 15) == 0, PULSE_ERR_INVALID_ARG);
    return PULSE_OK;
}

static bool overlap(const void* a, size_t na, const void* b, size_t nb) {
    return a && b && (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

// Whether x shares memory with what the attention reads, or writes beside it.
static bool x_under_attention(const pulse_normal_layer& n, size_t x_bytes, size_t ws_used) {
    const size_t B = (size_t)n.B, i32 = sizeof(int32_t);
    auto at = [&](const void* p, size_t bytes) { return overlap(n.x, x_bytes, p, bytes); };
    return at(n.q, x_bytes) || at(n.slot_pool, (size_t)n.n_slots * pulse_block_bytes(&n.shape)) ||
           at(n.block_table, i32 * B * n.max_blocks) || at(n.sel_idx, i32 * B * n.k_max) || at(n.sel_cnt, i32 * B) ||
           at(n.ctx_len, i32 * B) || at(n.lse, sizeof(float) * B * n.shape.num_q_heads) || at(n.ws, ws_used);
}

// Enqueue one normal-batch layer on irq->cmp; ev_attn (optional) is recorded after its
// attention, ev_end (optional) after its FFN.
static pulse_status normal_layer(pulse_irq* irq, const pulse_normal_layer& n, hipEvent_t ev_attn, hipEvent_t ev_end) {
    const hipStream_t hs = irq->cmp;
    const WsLayout w = ws_layout(n.shape, n.B, n.k_max, 0);
    const int32_t D = n.shape.num_q_heads * n.shape.head_dim, F = n.d_ff, B = n.B;
    // x is written by the attention and h by the gate and up product, unless others still read that memory then
    const size_t x_bytes = (size_t)B * D * 2;
    const bool own_cast = x_under_attention(n, x_bytes, w.total);
    const bool own_swiglu = overlap(n.x, x_bytes, n.h, (size_t)B * F * 2);
    if (launch_attention(n.shape, n.q, n.slot_pool, n.n_slots, n.block_table, n.max_blocks, n.sel_idx, n.sel_cnt,
                         n.k_max, n.ctx_len, n.B, n.sm_scale, n.out, n.lse, ws_at<float>(n.ws, w.attn_o),
                         ws_at<float2>(n.ws, w.attn_ml), n.dev_status, hs, nullptr, nullptr,
                         own_cast ? nullptr : (__bf16*)n.x) != hipSuccess)
        return PULSE_ERR_HIP;
    if (ev_attn && hipEventRecord(ev_attn, hs) != hipSuccess) return PULSE_ERR_HIP;
    if (own_cast) {
        const int64_t nx = (int64_t)B * D;
        hipLaunchKernelGGL(to_bf16_kernel, dim3(grid_for(nx)), dim3(256), 0, hs, n.out, (__bf16*)n.x, nx);
        if (hipGetLastError() != hipSuccess) return PULSE_ERR_HIP;
    }
    // gu [B][2F] = x [B][D] . W_gu^T, h [B][F] = silu(g) * u
    if (launch_ffn_gemm<true>(n.x, n.w_gate_up, n.gu, own_swiglu ? nullptr : n.h, B, F, D, hs) != hipSuccess)
        return PULSE_ERR_HIP;
    if (own_swiglu) {
        const int64_t nh = (int64_t)B * F;
        hipLaunchKernelGGL(swiglu_kernel, dim3(grid_for(nh)), dim3(256), 0, hs, (const __bf16*)n.gu, (__bf16*)n.h, F,
                           nh);
        if (hipGetLastError() != hipSuccess) return PULSE_ERR_HIP;
    }
    // y [B][D] = h [B][F] . W_down^T
    if (launch_ffn_gemm<false>(n.h, n.w_down, n.y, nullptr, B, D, F, hs) != hipSuccess) return PULSE_ERR_HIP;
    if (ev_end && hipEventRecord(ev_end, hs) != hipSuccess) return PULSE_ERR_HIP;
    return PULSE_OK;
}

extern "C" {

pulse_status pulse_irq_create(pulse_stream_t compute_stream, pulse_stream_t io_stream, pulse_irq** out) {
    PULSE_REQUIRE(out, PULSE_ERR_INVALID_ARG);
    *out = nullptr;
    pulse_irq* irq = new pulse_irq();
    irq->cmp = (hipStream_t)compute_stream;
    irq->io = (hipStream_t)io_stream;
    bool fail = hipHostMalloc((void**)&irq->flag_host, sizeof(int64_t),
                              hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess;
    if (!fail) {
        *irq->flag_host = 0;
        fail = hipHostGetDevicePointer((void**)&irq->flag_dev, irq->flag_host, 0) != hipSuccess;
    }
    if (fail) {
        pulse_irq_destroy(irq);
        return PULSE_ERR_HIP;
    }
    *out = irq;
    return PULSE_OK;
}

pulse_status pulse_irq_destroy(pulse_irq* irq) {
    if (!irq) return PULSE_ERR_INVALID_ARG;
    if (irq->cmp) (void)hipStreamSynchronize(irq->cmp);
    if (irq->io) (void)hipStreamSynchronize(irq->io);
    for (hipEvent_t e : irq->events) (void)hipEventDestroy(e);
    if (irq->flag_host) (void)hipHostFree(irq->flag_host);
    delete irq;
    return PULSE_OK;
}

pulse_status pulse_irq_step(pulse_irq* irq, const pulse_layer_args* offload, int32_t n_offload_layers,
                            const pulse_normal_layer* normal, int32_t n_normal_layers, int32_t mode,
                            int32_t async_ahead, pulse_gs_engine* engine, int32_t* overlap_depth,
                            pulse_irq_stats* stats) {
    PULSE_REQUIRE(irq && stats && n_offload_layers >= 1 && offload, PULSE_ERR_INVALID_ARG);
    PULSE_REQUIRE(mode >= PULSE_IRQ_SEMI_SYNC && mode <= PULSE_IRQ_BLOCKING, PULSE_ERR_INVALID_ARG);
    PULSE_REQUIRE(n_normal_layers >= 0 && (normal || n_normal_layers == 0), PULSE_ERR_INVALID_ARG);
    PULSE_REQUIRE(mode != PULSE_IRQ_ASYNC || async_ahead >= 1, PULSE_ERR_INVALID_ARG);
    for (int32_t m = 0; m < n_offload_layers; ++m) {
        pulse_status st = check_layer_args(&offload[m]);
        if (st != PULSE_OK) return st;
        PULSE_REQUIRE(offload[m].B >= 1, PULSE_ERR_INVALID_ARG);
        // the engine moves blocks of the shape it was made for
        PULSE_REQUIRE(!engine || gs_engine_serves(engine, offload[m].shape), PULSE_ERR_INVALID_ARG);
    }
    for (int32_t l = 0; l < n_normal_layers; ++l) {
        pulse_status st = check_normal(&normal[l]);
        if (st != PULSE_OK) return st;
    }
    const auto t0 = std::chrono::steady_clock::now();
    const double wait_limit_s = 60.0;  // a recall that never signals means a broken device
    irq->next_event = 0;
    const size_t L = (size_t)n_offload_layers;
    std::vector<hipEvent_t> ev_sel(L), ev_rc0(L), ev_rc1(L), ev_att(L);
    std::vector<int32_t> depths(L, 0);
    int64_t nl = 0;  // normal layers enqueued
    std::vector<hipEvent_t> ring;  // layer-end events of queued normal layers (ASYNC throttle)
    size_t ring_head = 0;
    pulse_status result = PULSE_OK;
    int64_t engine_pending = 0;  // engine call submitted and not yet seen complete

    auto run_normal = [&](bool wait_attn, bool wait_all) -> pulse_status {
        hipEvent_t ea = nullptr, ee = nullptr;
        if (mode != PULSE_IRQ_BLOCKING) {  // the modes that wait for layers
            ea = irq->event();
            ee = irq->event();
            if (!ea || !ee) return PULSE_ERR_HIP;
        }
        if (mode == PULSE_IRQ_ASYNC) {
            if ((int64_t)(ring.size() - ring_head) >= async_ahead) {
                if (hipEventSynchronize(ring[ring_head]) != hipSuccess) return PULSE_ERR_HIP;
                ++ring_head;
            }
        }
        pulse_status st = normal_layer(irq, normal[nl % n_normal_layers], ea, ee);
        if (st != PULSE_OK) return st;
        ++nl;
        if (mode == PULSE_IRQ_ASYNC) ring.push_back(ee);
        if (wait_attn && hipEventSynchronize(ea) != hipSuccess) return PULSE_ERR_HIP;
        if (wait_all && hipEventSynchronize(ee) != hipSuccess) return PULSE_ERR_HIP;
        return PULSE_OK;
    };

    // BLOCKING with the gather kernel: nothing runs beside a recall, so it goes from every XCD and
    // on the compute stream, whose order is the wait.  (Through the I/O stream, the flag and the
    // host the chip idled about 30 us per layer: two cross-stream waits, and the launches that
    // followed the flag; 4 layers of a light offload batch beside 32 x 4K requests 1026 -> 901 us.)
    // Work the caller left on the I/O stream still comes first.
    const bool in_order = mode == PULSE_IRQ_BLOCKING && !engine;
    if (in_order) {
        const hipError_t q = hipStreamQuery(irq->io);
        if (q == hipErrorNotReady) {
            (void)hipGetLastError();  // an answer, not an error of a later call
            hipEvent_t e = irq->event();
            if (!e || hipEventRecord(e, irq->io) != hipSuccess || hipStreamWaitEvent(irq->cmp, e, 0) != hipSuccess)
                result = PULSE_ERR_HIP;
        } else if (q != hipSuccess) {
            result = PULSE_ERR_HIP;
        }
    }
    for (size_t m = 0; m < L && result == PULSE_OK; ++m) {
        const pulse_layer_args& a = offload[m];
        ev_sel[m] = irq->event();
        ev_rc0[m] = irq->event();
        ev_rc1[m] = irq->event();
        ev_att[m] = irq->event();
        if (!ev_sel[m] || !ev_rc0[m] || !ev_rc1[m] || !ev_att[m]) { result = PULSE_ERR_HIP; break; }
        // selection on the compute stream, then the recall: the GPU gather kernel + signal on
        // the I/O stream, or a submission to the gather-scatter engine
        if (layer_select(a, irq->cmp) != hipSuccess || hipEventRecord(ev_sel[m], irq->cmp) != hipSuccess) {
            result = PULSE_ERR_HIP;
            break;
        }
        int64_t seq = 0;
        if (in_order) {
            if (layer_recall(a, irq->cmp, 8, ev_rc0[m], ev_rc1[m]) != hipSuccess) {
                result = PULSE_ERR_HIP;
                break;
            }
        } else if (engine) {
            result = pulse_gs_recall_submit(engine, a.host_kv, a.blk_off, a.B, a.sel_idx, a.sel_cnt, a.k_max,
                                            a.block_table, a.max_blocks, a.free_slots, a.free_head, a.n_free,
                                            a.slot_pool, a.n_slots, a.stats, a.dev_status, a.ws, a.ws_bytes, &seq,
                                            irq->cmp);
            if (result != PULSE_OK) break;
            engine_pending = seq;
        } else {
            seq = ++irq->seq;
            if (hipStreamWaitEvent(irq->io, ev_sel[m], 0) != hipSuccess ||
                hipEventRecord(ev_rc0[m], irq->io) != hipSuccess ||
                layer_recall(a, irq->io, kIrqRecallXcds) != hipSuccess) {
                result = PULSE_ERR_HIP;
                break;
            }
            hipLaunchKernelGGL(irq_signal_kernel, dim3(1), dim3(64), 0, irq->io, irq->flag_dev, seq);
            if (hipGetLastError() != hipSuccess || hipEventRecord(ev_rc1[m], irq->io) != hipSuccess) {
                result = PULSE_ERR_HIP;
                break;
            }
        }
        auto recall_done = [&]() -> bool {
            if (!engine) return irq->flag_reached(seq);
            int32_t done = 0;
            const pulse_status ps = pulse_gs_recall_poll(engine, seq, &done);
            if (done) engine_pending = 0;
            if (done && ps != PULSE_OK && result == PULSE_OK) result = ps;
            return done != 0;
        };
        // wait for the recall: normal layers run meanwhile, checked at layer boundaries
        int32_t depth = 0;
        const auto w0 = std::chrono::steady_clock::now();
        while (!in_order && !recall_done()) {
            if (std::chrono::duration<double>(std::chrono::steady_clock::now() - w0).count() > wait_limit_s) {
                result = PULSE_ERR_TIMEOUT;
                break;
            }
            if (mode == PULSE_IRQ_BLOCKING || n_normal_layers == 0) continue;  // spin on the flag
            result = run_normal(mode == PULSE_IRQ_SEMI_SYNC, mode == PULSE_IRQ_SYNC);
            if (result != PULSE_OK) break;
            ++depth;
        }
        if (result != PULSE_OK) break;
        depths[m] = depth;
        // resume the offload batch: its attention for layer m
        // (the engine marks a call complete only after its streams have drained)
        if ((!engine && !in_order && hipStreamWaitEvent(irq->cmp, ev_rc1[m], 0) != hipSuccess) ||
            hipEventRecord(ev_att[m], irq->cmp) != hipSuccess || layer_attention(a, irq->cmp) != hipSuccess) {
            result = PULSE_ERR_HIP;
            break;
        }
        if (mode == PULSE_IRQ_BLOCKING && n_normal_layers > 0) {  // single-batch schedule: one normal layer per layer
            result = run_normal(false, false);
            if (result != PULSE_OK) break;
        }
    }
    // drain both streams (the GPU work enqueued is finite in every case) and, after an
    // early exit, the engine call still in flight, so the engine can take the next one
    const bool ok_sync = hipStreamSynchronize(irq->cmp) == hipSuccess && hipStreamSynchronize(irq->io) == hipSuccess;
    if (engine && engine_pending) (void)pulse_gs_recall_wait(engine, engine_pending, (int32_t)(wait_limit_s * 1e3));
    if (result == PULSE_OK && !ok_sync) result = PULSE_ERR_HIP;
    const auto t1 = std::chrono::steady_clock::now();
    *stats = pulse_irq_stats{};
    stats->normal_layers = nl;
    stats->wall_ms = std::chrono::duration<double, std::milli>(t1 - t0).count();
    if (result != PULSE_OK) return result;
    stats->offload_layers = n_offload_layers;
    double sum_resume = 0.0, sum_recall = 0.0, sum_stall = 0.0, sum_depth = 0.0;
    int32_t max_depth = 0;
    for (size_t m = 0; m < L; ++m) {
        float r = 0.f, c = 0.f, w = 0.f;
        if (hipEventElapsedTime(&w, ev_sel[m], ev_att[m]) != hipSuccess) return PULSE_ERR_HIP;
        if (!engine && (hipEventElapsedTime(&r, ev_rc1[m], ev_att[m]) != hipSuccess ||
                        hipEventElapsedTime(&c, ev_rc0[m], ev_rc1[m]) != hipSuccess))
            return PULSE_ERR_HIP;
        sum_resume += r;
        sum_recall += c;
        sum_stall += w;
        sum_depth += depths[m];
        max_depth = depths[m] > max_depth ? depths[m] : max_depth;
        if (overlap_depth) overlap_depth[m] = depths[m];
    }
    stats->mean_stall_us = sum_stall * 1e3 / (double)L;
    stats->mean_resume_us = engine ? -1.0 : sum_resume * 1e3 / (double)L;
    stats->mean_recall_us = engine ? -1.0 : sum_recall * 1e3 / (double)L;
    stats->mean_overlap_depth = sum_depth / (double)L;
    stats->max_overlap_depth = max_depth;
    return PULSE_OK;
}

}  // extern "C"
