// Capacity-bounded slot assignment.  The paper has no capacity (its batch is
// "dynamic", Section III-C); here every micro-batch of Section III-B is an
// independent MoE call with C_p rows per expert, which is what makes partition
// buffers exactly 1/n of the whole (Section III-D).  Inside a partition,
// positions are granted choice-major then in token order, by a stable ranking:
// per-block histograms, a prefix over the blocks that come earlier in that
// order, and a stable in-block rank.  No result depends on atomic ordering.
#include "common.h"

namespace moe {

constexpr int SLOT_BLOCK = 1024;   // assignments ranked by one workgroup
// The ranking kernel can count by itself what comes before a workgroup's assignments, in a read of all of the
// partition's, up to this many per thread.  One launch / two: 128 assignments, 8 experts 2.6 / 4.1 us; 3000, 6 experts 4.0
// / 4.3; 2048, 64 experts 4.1 / 4.4; 4096, 64 experts 5.3 / 4.7; 8192, 8 experts 4.9 / 4.9.
constexpr int COUNT_PASSES = 3;

// Lanes of the wavefront whose expert is this lane's (experts below 64; `bits` of them matter): one ballot per bit, not
// one per expert (4096 tokens, 64 experts: both kernels 8.8 us so, 4.7 now).
__device__ __forceinline__ unsigned long long same_expert(int e, int bits) {
    unsigned long long m = ~0ull;
    for (int i = 0; i < bits; ++i) {
        const bool one = (e >> i) & 1;
        const unsigned long long b = __ballot(one);
        m &= one ? b : ~b;
    }
    return m;
}

// hist[((p*k + j)*nb + b)*E + e] = number of tokens of block b (partition p) whose
// j-th choice is expert e
__global__ __launch_bounds__(SLOT_BLOCK) void slot_hist_kernel(
    const int* __restrict__ topk_idx, int* __restrict__ hist, int Tp, int k, int E, int nb) {
    __shared__ int h[64];
    const int b = blockIdx.x, j = blockIdx.y, p = blockIdx.z;
    if (threadIdx.x < 64) h[threadIdx.x] = 0;
    __syncthreads();
    const int tl = b * SLOT_BLOCK + threadIdx.x;
    if (tl < Tp) {
        int e = topk_idx[(size_t)(p * Tp + tl) * k + j];
        atomicAdd(&h[e], 1);             // integer counts: order does not matter
    }
    __syncthreads();
    if (threadIdx.x < E) hist[((size_t)(p * k + j) * nb + b) * E + threadIdx.x] = h[threadIdx.x];
}

// What the ranking kernel writes besides the slots (each may be NULL): the row weights of the kept assignments, the row
// map (see slot_rows_kernel) and, for one choice per token, zeros in the output rows of dropped tokens.
struct SlotExtras { const float* topk_w; float* slot_w; int* rows; char* y; int row_bytes; };

// COUNT: the workgroup counts the assignments that come before its own by itself, in a pass over all of its partition's
// (one launch instead of two; hist unused).
template <bool COUNT>
__global__ __launch_bounds__(SLOT_BLOCK) void slot_assign_kernel(
    const int* __restrict__ topk_idx, const int* __restrict__ hist, int* __restrict__ slot, int* __restrict__ counts,
    SlotExtras x, int Tp, int k, int E, int bits, int nb, int Cp) {
    __shared__ int before[64], total[64];
    __shared__ int wcount[SLOT_BLOCK / 64][64];
    const int b = blockIdx.x, j = blockIdx.y, p = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int tl = b * SLOT_BLOCK + tid;
    const bool valid = tl < Tp;
    const int t = p * Tp + tl;
    const int my_e = valid ? topk_idx[(size_t)t * k + j] : -1;
    const unsigned long long below = (1ull << lane) - 1ull;
    wcount[wid][lane] = 0;
    if (tid < 64) { before[tid] = 0; total[tid] = 0; }
    __syncthreads();
    if constexpr (COUNT) {
        const int* idx = topk_idx + (size_t)p * Tp * k;
        const int n = Tp * k;
        int q[COUNT_PASSES];                     // all on their way before the first is counted
#pragma unroll
        for (int r = 0; r < COUNT_PASSES; ++r) q[r] = r * SLOT_BLOCK + tid < n ? idx[r * SLOT_BLOCK + tid] : -1;
#pragma unroll
        for (int r = 0; r < COUNT_PASSES; ++r) {
            if (r * SLOT_BLOCK >= n) break;
            const int i = r * SLOT_BLOCK + tid, ti = i / k, ji = i - ti * k;
            const unsigned long long ahead = __ballot(ji < j || (ji == j && ti < b * SLOT_BLOCK));
            const unsigned long long peers = same_expert(q[r], bits) & __ballot(i < n);
            if (i < n && (peers & below) == 0) {          // the first of an expert's lanes speaks for all of them
                atomicAdd(&total[q[r]], __popcll(peers));
                atomicAdd(&before[q[r]], __popcll(peers & ahead));
            }
        }
    } else if (lane < E) {
        // lane e of a wavefront adds up every sixteenth block's count of expert e
        const int mine = j * nb + b;
        int sb = 0, st = 0;
#pragma unroll 4
        for (int q = wid; q < k * nb; q += SLOT_BLOCK / 64) {
            const int v = hist[((size_t)p * k * nb + q) * E + lane];
            st += v;
            if (q < mine) sb += v;
        }
        if (st) {
            atomicAdd(&total[lane], st);
            atomicAdd(&before[lane], sb);
        }
    }
    const unsigned long long peers = same_expert(my_e, bits) & __ballot(valid);
    if (valid && (peers & below) == 0) wcount[wid][my_e] = __popcll(peers);
    __syncthreads();
    if (b == 0 && j == 0 && tid < E) counts[p * E + tid] = total[tid] < Cp ? total[tid] : Cp;
    int s = -1;
    if (valid) {
        int pos = before[my_e] + __popcll(peers & below);
        for (int w = 0; w < wid; ++w) pos += wcount[w][my_e];
        s = pos < Cp ? my_e * Cp + pos : -1;
        slot[(size_t)t * k + j] = s;
        if (s >= 0 && x.slot_w) x.slot_w[(size_t)p * E * Cp + s] = x.topk_w[(size_t)t * k + j];
        if (s >= 0 && x.rows) x.rows[(size_t)p * E * Cp + s] = t;
    }
    if (x.y) {
        unsigned long long dropped = __ballot(valid && s < 0);
        while (dropped) {
            const int l = __builtin_ctzll(dropped);
            dropped &= dropped - 1;
            uint4* row = reinterpret_cast<uint4*>(x.y + (size_t)(p * Tp + b * SLOT_BLOCK + wid * 64 + l) * x.row_bytes);
            for (int c = lane; c < x.row_bytes / 16; c += 64) row[c] = make_uint4(0, 0, 0, 0);
        }
    }
}

// rows[p][slot[t,j]] = t for kept assignments: the map a gathering GEMM reads its rows through
__global__ __launch_bounds__(256) void slot_rows_kernel(const int* __restrict__ slot, int* __restrict__ rows,
                                                        int T, int Tp, int k, int Rp) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= T * k) return;
    const int t = i / k;
    const int s = slot[i];
    if (s >= 0) rows[(size_t)(t / Tp) * Rp + s] = t;
}

}  // namespace moe

extern "C" moe_status moe_slot_rows(const moe_config* cfg, const int32_t* slot, int32_t* rows, void* stream) {
    moe::Dims d;
    MOE_TRY(moe::make_dims(cfg, &d));
    if (!slot || !rows) return MOE_ERR_NULL;
    const int total = d.T * d.k;
    hipLaunchKernelGGL(moe::slot_rows_kernel, dim3((total + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       slot, rows, d.T, d.Tp, d.k, d.Rp);
    moe::count_launch(moe::LC_OTHER);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

extern "C" moe_status moe_slot_scratch_bytes(const moe_config* cfg, size_t* bytes) {
    moe::Dims d;
    MOE_TRY(moe::make_dims(cfg, &d));
    if (!bytes) return MOE_ERR_NULL;
    int nb = (d.Tp + moe::SLOT_BLOCK - 1) / moe::SLOT_BLOCK;
    *bytes = (size_t)d.n * d.k * nb * d.E * sizeof(int);
    return MOE_OK;
}

namespace moe {

moe_status assign_slots(const Dims& d, const int* topk_idx, const float* topk_w, int* slot, int* counts, float* slot_w,
                        int* rows, void* y, int* hist, hipStream_t s) {
    const int nb = (d.Tp + SLOT_BLOCK - 1) / SLOT_BLOCK;
    const dim3 grid(nb, d.k, d.n);
    const SlotExtras x = {topk_w, slot_w, rows, (char*)y, (int)(d.M * d.es)};
    ProfScope ps(PK_SLOTS, s);
    int bits = 1;
    while ((1 << bits) < d.E) ++bits;
    if ((long long)d.Tp * d.k <= COUNT_PASSES * SLOT_BLOCK) {
        hipLaunchKernelGGL((slot_assign_kernel<true>), grid, dim3(SLOT_BLOCK), 0, s, topk_idx, (const int*)hist, slot, counts, x,
                           d.Tp, d.k, d.E, bits, nb, d.Cp);
    } else {
        hipLaunchKernelGGL(slot_hist_kernel, grid, dim3(SLOT_BLOCK), 0, s, topk_idx, hist, d.Tp, d.k, d.E, nb);
        MOE_CHECK_LAUNCH();
        hipLaunchKernelGGL((slot_assign_kernel<false>), grid, dim3(SLOT_BLOCK), 0, s, topk_idx, (const int*)hist, slot, counts, x,
                           d.Tp, d.k, d.E, bits, nb, d.Cp);
    }
    count_launch(LC_OTHER, 2);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// Histogram memory of moe_assign_slots_static: one array per GPU, resident for the life of the
// process.  In host code this name is only a handle for hipGetSymbolAddress; the device address
// it yields (one per device) is what kernels are given.
constexpr size_t STATIC_SCRATCH_BYTES = 256 * 1024;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static void* g_static_scratch[MAX_DEVICES];

static moe_status static_scratch(void** out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return MOE_ERR_UNSUPPORTED;
    if (!g_static_scratch[dev]) {
        void* ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return MOE_ERR_HIP;
        g_static_scratch[dev] = ptr;
    }
    *out = g_static_scratch[dev];
    return MOE_OK;
}

}  // namespace moe

extern "C" moe_status moe_assign_slots(const moe_config* cfg, const int32_t* topk_idx, const float* topk_w,
                                       int32_t* slot, int32_t* counts, float* slot_w,
                                       void* scratch, void* stream) {
    moe::Dims d;
    MOE_TRY(moe::make_dims(cfg, &d));
    if (!topk_idx || !slot || !counts || !scratch) return MOE_ERR_NULL;
    if (slot_w && !topk_w) return MOE_ERR_NULL;
    return moe::assign_slots(d, topk_idx, topk_w, slot, counts, slot_w, nullptr, nullptr, (int*)scratch, (hipStream_t)stream);
}

extern "C" moe_status moe_assign_slots_static(const moe_config* cfg, const int32_t* topk_idx, const float* topk_w,
                                              int32_t* slot, int32_t* counts, float* slot_w, void* stream) {
    moe::Dims d;
    MOE_TRY(moe::make_dims(cfg, &d));
    if (!topk_idx || !slot || !counts) return MOE_ERR_NULL;
    if (slot_w && !topk_w) return MOE_ERR_NULL;
    size_t need = 0;
    MOE_TRY(moe_slot_scratch_bytes(cfg, &need));
    if (need > moe::STATIC_SCRATCH_BYTES) return MOE_ERR_WORKSPACE;
    void* hist = nullptr;
    MOE_TRY(moe::static_scratch(&hist));
    // every histogram entry the ranking kernel reads is written by the histogram kernel of the same
    // call, so nothing of an earlier call's contents has to be cleared
    return moe::assign_slots(d, topk_idx, topk_w, slot, counts, slot_w, nullptr, nullptr, (int*)hist, (hipStream_t)stream);
}
