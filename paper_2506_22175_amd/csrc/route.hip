// Gate of the MoE layer: float logits in a fixed summation order, softmax over
// all experts, top-k on the logits (Sections II-B2 and IV-A of the paper: a
// linear gate with E*M parameters and a top-k choice; the paper itself uses
// k = 1).  One wavefront handles TB tokens at a time; the gate weights sit in
// LDS as float, laid out so that every lane reads its own bank.
//
// Summation order (the same order is written out in the CPU oracle, which
// shares no code with this file): element d of a token row belongs to lane
// (d / 8) mod 64; a lane folds its elements in ascending d with one fused
// multiply-add each, starting from +0; the 64 lane sums are folded pairwise
// with offsets 32, 16, 8, 4, 2, 1; the bias is added last.
#include "common.h"
#include <climits>

namespace moe {

// Pairwise folding of NV values per lane across the 64 lanes.  While more than
// one value is left, the two lanes of a pair split the values between them
// (each keeps one half and adds the partner's copy of that half); the sums are
// the same ones a full butterfly would produce, since a + b == b + a exactly.
// On return v[0] of lane l is the total of value index l >> (6 - log2 NV0).
template <int NV, int OFF>
__device__ __forceinline__ void fold_lanes(float* v, int lane) {
    if constexpr (OFF >= 1) {
        if constexpr (NV > 1) {
            constexpr int HALF = NV / 2;
            const bool upper = (lane & OFF) != 0;
#pragma unroll
            for (int i = 0; i < HALF; ++i) {
                float send = upper ? v[i] : v[i + HALF];
                float keep = upper ? v[i + HALF] : v[i];
                float recv = __shfl_xor(send, OFF, 64);
                v[i] = keep + recv;
            }
            fold_lanes<HALF, OFF / 2>(v, lane);
        } else {
            v[0] = v[0] + __shfl_xor(v[0], OFF, 64);
            fold_lanes<1, OFF / 2>(v, lane);
        }
    }
}

constexpr int ROUTE_THREADS = 512;
constexpr int ROUTE_WAVES = ROUTE_THREADS / 64;

// softmax over E logits and the k largest of them; runs in one lane per token.  The row (EP floats in
// LDS, 16-byte aligned, E of them valid) is taken into registers first, so that nothing below waits on LDS;
// idx_out and w_out are the token's k places in global memory.
template <int EP>
__device__ __forceinline__ void softmax_topk(const float* lg, int E, int k, int renorm, int* idx_out, float* w_out) {
    float v[EP];
#pragma unroll
    for (int e4 = 0; e4 < EP / 4; ++e4) {
        const float4 q = *reinterpret_cast<const float4*>(lg + 4 * e4);
        v[4 * e4] = q.x; v[4 * e4 + 1] = q.y; v[4 * e4 + 2] = q.z; v[4 * e4 + 3] = q.w;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < EP; ++e)
        if (e < E) mx = fmaxf(mx, v[e]);
    float sum = 0.0f;
#pragma unroll
    for (int e = 0; e < EP; ++e)
        if (e < E) sum += expf(v[e] - mx);
    // the k largest logits in descending order, ties to the lower index; emit(j, expert, its logit)
    auto pick = [&](auto&& emit) __attribute__((always_inline)) {
        unsigned long long taken = 0ull;
        for (int j = 0; j < k; ++j) {
            int best = -1;
            float bv = 0.0f, braw = 0.0f;
#pragma unroll
            for (int e = 0; e < EP; ++e) {
                if (e < E && !((taken >> e) & 1ull)) {
                    const float o = (v[e] != v[e]) ? -INFINITY : v[e];       // NaN orders as -inf
                    if (best < 0 || o > bv) { best = e; bv = o; braw = v[e]; }
                }
            }
            taken |= 1ull << best;
            emit(j, best, braw);
        }
    };
    // weights: the chosen probabilities, or those divided by their sum over the k choices
    float den = sum;
    if (renorm) {
        den = 0.0f;
        pick([&](int, int, float raw) __attribute__((always_inline)) { den += expf(raw - mx); });
    }
    pick([&](int j, int best, float raw) __attribute__((always_inline)) {
        idx_out[j] = best;
        w_out[j] = expf(raw - mx) / den;
    });
}

// Eight consecutive elements of a token row through a buffer descriptor: a lane past the end of
// the descriptor gets zeros, so the loads sit in straight-line code and stay in flight while
// the previous elements are multiplied.
template <typename T> struct RowLoad;
template <> struct RowLoad<bf16_t> {
    static __device__ __forceinline__ void load(Raw8<bf16_t>& r, __amdgpu_buffer_rsrc_t rs, unsigned off) {
        r.u = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    }
};
template <> struct RowLoad<float> {
    static __device__ __forceinline__ void load(Raw8<float>& r, __amdgpu_buffer_rsrc_t rs, unsigned off) {
        r.a = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        r.b = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16u, 0, 0));
    }
};

// tokens whose logits a wavefront keeps in LDS before it ranks them (1 KB of LDS per padded expert
// for the workgroup; with 64 experts half as many, so that 512 gate-weight rows still fit beside them)
template <int EP> struct RouteHeld { static constexpr int N = EP >= 64 ? 16 : 32; };

// Where the gate weights of element i (of a lane's eight), experts 4*e4 .. 4*e4 + 3 and lane l lie in LDS, in 16-byte
// pieces from the span's first: a wavefront reads one (i, e4) at a time, any rotation of its 64 pieces without a
// conflict; the rotation here also spreads the writes of the staging threads, which have neighbouring (i, e4) of few
// lanes and would all meet in the same banks (a quarter to half of the kernel for 64 experts, 3 us for 8).
// (ROT: not where a workgroup stages once for many tokens: the rotated addresses cost 6 % of the inner loop)
template <int E4, bool ROT>
__device__ __forceinline__ int weight_piece(int i, int e4, int l) {
    return (i * E4 + e4) * 64 + (ROT ? (l + i * 8 + (e4 >> 1)) & 63 : l);
}

// All experts in a wavefront.  EP = E rounded up to a power of two (>= 4); TB tokens per wavefront, TB*EP <= 64.
// MC = gate-weight rows held in LDS at a time (multiple of 512, or >= M).
//
// A wavefront multiplies TB tokens at a time (a group) and parks their logits in LDS; once
// RouteHeld tokens are parked, or its groups are done, one lane per token does softmax and
// top-k, so that the serial part runs once for many tokens instead of once per group.
template <typename T, int EP, int TB>
__global__ __launch_bounds__(ROUTE_THREADS) void route_kernel(
    const T* __restrict__ x, const T* __restrict__ Wg, const float* __restrict__ bias,
    float* __restrict__ logits, int* __restrict__ topk_idx, float* __restrict__ topk_w,
    int Ttot, int M, int E, int k, int MC, int renorm) {
    extern __shared__ float smem[];
    float* wl = smem;                               // [MC/8 ... ] see index below
    float* lg = smem + (size_t)MC * EP;             // [ROUTE_WAVES][HELD][EP]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform, and visibly so
    const int ngroups = (Ttot + ROUTE_WAVES * TB - 1) / (ROUTE_WAVES * TB);
    const int nchunks = (M + MC - 1) / MC;
    constexpr int E4 = EP / 4;
    constexpr unsigned ES = sizeof(T);
    constexpr int HELD = RouteHeld<EP>::N;
    constexpr bool ROT = TB == 2 && EP <= 16;       // few tokens per workgroup
    float* mylg = lg + (size_t)wid * HELD * EP;
    int held = 0, held_g0 = 0;                      // parked tokens, and the group of the first of them

    // softmax and top-k of the parked tokens: token q of the wavefront belongs to group
    // held_g0 + (q / TB) * gridDim.x
    auto rank_held = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < held) {
            const int gq = held_g0 + (lane / TB) * (int)gridDim.x;
            const int t = (gq * ROUTE_WAVES + wid) * TB + lane % TB;
            if (t < Ttot) {
                const float* my = mylg + lane * EP;
                if (E == EP) {
#pragma unroll
                    for (int e4 = 0; e4 < EP / 4; ++e4)
                        *reinterpret_cast<float4*>(logits + (size_t)t * E + 4 * e4) = *reinterpret_cast<const float4*>(my + 4 * e4);
                } else {
                    for (int e = 0; e < E; ++e) logits[(size_t)t * E + e] = my[e];
                }
                softmax_topk<EP>(my, E, k, renorm, topk_idx + (size_t)t * k, topk_w + (size_t)t * k);
            }
        }
        __builtin_amdgcn_wave_barrier();
        held = 0;
    };

    // the TB token rows of group g as one descriptor; rows past the last token read as zeros
    auto rows_of = [&](int g) __attribute__((always_inline)) {
        const int t0 = (g * ROUTE_WAVES + wid) * TB;
        const int nt = min(TB, Ttot - t0);
        const T* base = x + (size_t)(nt > 0 ? t0 : 0) * M;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0,
                                                 nt > 0 ? (int)((size_t)nt * M * ES) : 0, 0x00020000);
    };
    // elements d0 .. d0+7 of the TB rows (a lane with d0 >= M reads something it never uses)
    auto fetch = [&](__amdgpu_buffer_rsrc_t rs, int d0, Raw8<T>* r) __attribute__((always_inline)) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
            RowLoad<T>::load(r[tb], rs, (unsigned)(((size_t)tb * M + d0) * ES));
    };

    // gate-weight rows c0 .. c0+MC-1 into LDS (whole workgroup; barriers before and after).
    // between() runs after the weights have been requested and before they are written to LDS:
    // an LDS write waits for every load issued before it, so the first token rows are requested there.
    auto stage_weights = [&](int c0, auto&& between) __attribute__((always_inline)) {
        __syncthreads();
        // LDS element of (row dl, expert e): span = dl/512, lane (dl/8)%64, i = dl%8
        if (EP % 8 == 0 && E == EP && (reinterpret_cast<unsigned long long>(Wg) & 15ull) == 0) {
            // eight experts of one row per load; a thread's loads (at most eight: MC*EP <= 32768) are all
            // in flight before the first is converted
            constexpr int G = EP / 8 > 0 ? EP / 8 : 1;
            constexpr int NP = 32768 / 8 / ROUTE_THREADS;
            Raw8<T> wr[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int q = tid + i * ROUTE_THREADS;
                const int d = c0 + q / G;
                if (q < MC * G && d < M) wr[i].load(Wg + (size_t)d * E + (q % G) * 8);
                else wr[i].zero();
            }
            between();
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int q = tid + i * ROUTE_THREADS;
                if (q < MC * G) {
                    const int dl = q / G, e0 = (q % G) * 8;
                    float v[8];
                    wr[i].to_float(v);
                    const int span = dl >> 9, l = (dl >> 3) & 63, i8 = dl & 7;
                    float* dst = wl + ((span * 8 * E4 * 64 + weight_piece<E4, ROT>(i8, e0 >> 2, l)) << 2);
                    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                    *reinterpret_cast<float4*>(dst + 256) = make_float4(v[4], v[5], v[6], v[7]);
                }
            }
        } else {
            between();
            for (int q = tid; q < MC * EP; q += ROUTE_THREADS) {
                int dl = q / EP, e = q % EP;
                int d = c0 + dl;
                float v = 0.0f;
                if (d < M && e < E) v = Elem<T>::ld(Wg + (size_t)d * E + e);
                int span = dl >> 9, l = (dl >> 3) & 63, i = dl & 7;
                wl[((span * 8 * E4 * 64 + weight_piece<E4, ROT>(i, e >> 2, l)) << 2) + (e & 3)] = v;
            }
        }
        __syncthreads();
    };

    // acc += the 8 elements of each of the TB rows times the gate weights of LDS span sp; the
    // weights of element i+1 are read from LDS while element i is multiplied
    auto multiply_span = [&](float* acc, const Raw8<T>* xr, int sp) __attribute__((always_inline)) {
        float xs[TB][8];
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) xr[tb].to_float(xs[tb]);
        float4 wv[2][E4];
        const float* wsp = wl + ((sp * 8 * E4 * 64) << 2);
#pragma unroll
        for (int e4 = 0; e4 < E4; ++e4) wv[0][e4] = *reinterpret_cast<const float4*>(wsp + (weight_piece<E4, ROT>(0, e4, lane) << 2));
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i + 1 < 8) {
#pragma unroll
                for (int e4 = 0; e4 < E4; ++e4)
                    wv[(i + 1) & 1][e4] = *reinterpret_cast<const float4*>(wsp + (weight_piece<E4, ROT>(i + 1, e4, lane) << 2));
            }
#pragma unroll
            for (int e4 = 0; e4 < E4; ++e4) {
                const float4 w4 = wv[i & 1][e4];
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) {
                    float* a = acc + tb * EP + e4 * 4;
                    a[0] = __builtin_fmaf(xs[tb][i], w4.x, a[0]);
                    a[1] = __builtin_fmaf(xs[tb][i], w4.y, a[1]);
                    a[2] = __builtin_fmaf(xs[tb][i], w4.z, a[2]);
                    a[3] = __builtin_fmaf(xs[tb][i], w4.w, a[3]);
                }
            }
        }
    };

    // fold the lane sums of group g, add the bias, park the logits; rank once enough are parked
    auto finish_group = [&](float* acc, int g) __attribute__((always_inline)) {
        fold_lanes<TB * EP, 32>(acc, lane);
        // lane l now holds value index vi = l >> SH in acc[0]; vi = tb*EP + e
        constexpr int NV = TB * EP;
        constexpr int SH = (NV == 64) ? 0 : (NV == 32) ? 1 : (NV == 16) ? 2 : (NV == 8) ? 3 : (NV == 4) ? 4 : 5;
        if (held == 0) held_g0 = g;
        const int vi = lane >> SH;
        const int e = vi % EP;
        if ((lane & ((1 << SH) - 1)) == 0 && e < E) {
            float v = acc[0];
            if (bias) v = v + bias[e];
            mylg[held * EP + vi] = v;
        }
        held += TB;
        if (held + TB > HELD) rank_held();
    };

    float acc[TB * EP];
#pragma unroll
    for (int i = 0; i < TB * EP; ++i) acc[i] = 0.0f;
    const int d_lane = lane * 8;

    if (nchunks == 1) {
        // The whole gate matrix stays in LDS.  Token elements are requested one span ahead of the
        // multiplications, across group boundaries, into two register sets in turn; past the last
        // group the descriptor is empty and the requests cost nothing.
        const int nspan = (M + 511) / 512;
        int rg = blockIdx.x, rsp = 0;               // the span to request next
        auto request = [&](Raw8<T>* r) __attribute__((always_inline)) {
            fetch(rows_of(rg), rsp * 512 + d_lane, r);
            if (++rsp == nspan) { rsp = 0; rg += gridDim.x; }
        };
        Raw8<T> xa[TB], xb[TB];
        stage_weights(0, [&]() __attribute__((always_inline)) { request(xa); });
        int g = blockIdx.x, sp = 0;                 // the span to multiply next
        auto multiply = [&](const Raw8<T>* cur) __attribute__((always_inline)) {
            if (sp * 512 + d_lane < M) multiply_span(acc, cur, sp);
            if (++sp == nspan) {
                finish_group(acc, g);
#pragma unroll
                for (int i = 0; i < TB * EP; ++i) acc[i] = 0.0f;
                sp = 0;
                g += gridDim.x;
            }
            return g < ngroups;
        };
        for (;;) {
            // (the barriers keep the instruction scheduler from sinking the requests to their uses)
            request(xb);
            __builtin_amdgcn_sched_barrier(0);
            if (!multiply(xa)) break;
            request(xa);
            __builtin_amdgcn_sched_barrier(0);
            if (!multiply(xb)) break;
        }
    } else {
        // The gate matrix passes through LDS in pieces of MC rows for every group of tokens.
        for (int g = blockIdx.x; g < ngroups; g += gridDim.x) {
            const __amdgpu_buffer_rsrc_t rs = rows_of(g);
            for (int ch = 0; ch < nchunks; ++ch) {
                const int c0 = ch * MC;
                stage_weights(c0, []() {});
                const int nspan = (min(MC, M - c0) + 511) / 512;
                for (int sp = 0; sp < nspan; ++sp) {
                    const int d0 = c0 + sp * 512 + d_lane;
                    Raw8<T> xr[TB];
                    fetch(rs, d0, xr);
                    if (d0 < M) multiply_span(acc, xr, sp);
                }
            }
            finish_group(acc, g);
#pragma unroll
            for (int i = 0; i < TB * EP; ++i) acc[i] = 0.0f;
        }
    }
    if (held > 0) rank_held();
}

// Many experts.  A workgroup takes ROUTE_WAVES * 16 / EP sets of TB tokens once; a wavefront has one set and
// sixteen of the experts, so that a gate weight read from LDS is used for TB tokens (with all experts in a wavefront there
// are registers for one or two, and the kernel reads LDS at twice the rate there is).  The gate weights pass through LDS
// once per workgroup, 64 KB at a time (ES of the eight elements of every lane of a span of 512), and two workgroups share
// a CU: one multiplies while the other waits for its weights, folds or ranks (eight lanes per token); four float32
// rows take too many registers for that.  us, bfloat16, launches back to back on the same inputs, against TB = 1 or 2
// tokens with all experts in a wavefront (in a step, x not in the caches: the first is 45):
// 8192 tokens x 768 x 64 experts 32 and 77, 1000 x 768 x 64 9.5 and 31, 4000 x 768 x 32 10.7 and 19, 3000 x 2048 x 48 60 and
// 138; the multiply-adds of the first take 11.  What is left is the way of the weights through LDS for every 8 tokens.
template <typename T, int EP, int TB>
__global__ __launch_bounds__(ROUTE_THREADS, sizeof(T) == 4 && TB == 4 ? 2 : 4) void route_wide_kernel(
    const T* __restrict__ x, const T* __restrict__ Wg, const float* __restrict__ bias,
    float* __restrict__ logits, int* __restrict__ topk_idx, float* __restrict__ topk_w,
    int Ttot, int M, int E, int k, int renorm) {
    constexpr int NB = EP / 16, SETS = ROUTE_WAVES / NB, TOK = SETS * TB;
    constexpr int E4 = EP / 4, NV = TB * 16, LGP = EP + 4;       // (logit rows 16 bytes further than whole banks)
    constexpr int ES = 256 / EP;                    // elements of a lane staged at a time
    constexpr unsigned EB = sizeof(T);
    extern __shared__ float smem[];
    float* wl = smem;                               // [ES][E4][64] float4: element, experts, lane (see weight_piece)
    float* lg = smem + 64 * ES * EP;                // [TOK][LGP]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int eb = wid % NB, set = wid / NB;
    const int tw = blockIdx.x * TOK, t0 = tw + set * TB;
    const int nt = max(0, min(TB, Ttot - t0));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(x + (size_t)(nt > 0 ? t0 : 0) * M), 0, nt > 0 ? (int)((size_t)nt * M * EB) : 0, 0x00020000);
    const int d_lane = lane * 8;
    float acc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.0f;
    const bool eights = (E & 7) == 0 && (reinterpret_cast<unsigned long long>(Wg) & 15ull) == 0;
    constexpr int G = EP / 8, NP = 64 * ES * G / ROUTE_THREADS;  // eight experts of a row per load, loads per thread
    constexpr int NPB = sizeof(T) == 2 ? NP : 2;                 // of which in flight together
    Raw8<T> xr[TB];
    for (int c0 = 0; c0 < M; c0 += 512) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) RowLoad<T>::load(xr[tb], rs, (unsigned)(((size_t)tb * M + c0 + d_lane) * EB));
#pragma unroll
        for (int i0 = 0; i0 < 8; i0 += ES) {
            if (c0 + i0 > 0) __syncthreads();       // the weights before these have been used
            // row r of a piece: lane r/ES, element i0 + r%ES
            if (eights) {
#pragma unroll
                for (int b = 0; b < NP; b += NPB) {
                    Raw8<T> wr[NPB];
#pragma unroll
                    for (int i = 0; i < NPB; ++i) {
                        const int q = tid + (b + i) * ROUTE_THREADS, r = q / G, d = c0 + (r / ES) * 8 + i0 + r % ES;
                        if (d < M && (q % G) * 8 < E) wr[i].load(Wg + (size_t)d * E + (q % G) * 8);
                        else wr[i].zero();
                    }
#pragma unroll
                    for (int i = 0; i < NPB; ++i) {
                        const int q = tid + (b + i) * ROUTE_THREADS, r = q / G, e0 = (q % G) * 8;
                        float v[8];
                        wr[i].to_float(v);
                        float* dst = wl + (weight_piece<E4, true>(r % ES, e0 >> 2, r / ES) << 2);
                        *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                        *reinterpret_cast<float4*>(dst + 256) = make_float4(v[4], v[5], v[6], v[7]);
                    }
                }
            } else {
                for (int q = tid; q < 64 * ES * EP; q += ROUTE_THREADS) {
                    const int r = q / EP, e = q % EP, d = c0 + (r / ES) * 8 + i0 + r % ES;
                    wl[(weight_piece<E4, true>(r % ES, e >> 2, r / ES) << 2) + (e & 3)] =
                        d < M && e < E ? Elem<T>::ld(Wg + (size_t)d * E + e) : 0.0f;
                }
            }
            __syncthreads();
            if (c0 + d_lane < M) {
                const float* wsp = wl + ((eb * 4 * 64) << 2);      // (the rotation of experts 16*eb on: 2*eb further)
                const int l = lane + 2 * eb;
#pragma unroll
                for (int i = 0; i < ES; ++i) {
                    float4 wv[4];
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4)
                        wv[e4] = *reinterpret_cast<const float4*>(wsp + (weight_piece<E4, true>(i, e4, l) << 2));
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) {
                        const float xs = xr[tb].at(i0 + i);
#pragma unroll
                        for (int e4 = 0; e4 < 4; ++e4) {
                            float* a = acc + tb * 16 + e4 * 4;
                            a[0] = __builtin_fmaf(xs, wv[e4].x, a[0]);
                            a[1] = __builtin_fmaf(xs, wv[e4].y, a[1]);
                            a[2] = __builtin_fmaf(xs, wv[e4].z, a[2]);
                            a[3] = __builtin_fmaf(xs, wv[e4].w, a[3]);
                        }
                    }
                }
            }
        }
    }
    fold_lanes<NV, 32>(acc, lane);
    // value index vi = tb*16 + expert: one in a lane of 64 values, one in two lanes of 32
    static_assert(NV == 64 || NV == 32, "two or four tokens of sixteen experts");
    constexpr int SHARE = 64 / NV;
    if (lane % SHARE == 0) {
        const int vi = lane / SHARE, e = eb * 16 + vi % 16;
        if (e < E) lg[(set * TB + vi / 16) * LGP + e] = bias ? acc[0] + bias[e] : acc[0];
    }
    __syncthreads();
    const int ntok = min(TOK, Ttot - tw);
    for (int q = tid; q < ntok * E; q += ROUTE_THREADS) logits[(size_t)tw * E + q] = lg[(q / E) * LGP + q % E];

    // softmax and top-k, eight lanes per token, lane `sub` of which has experts sub*EPL .. sub*EPL + EPL - 1
    constexpr int EPL = EP / 8;
    const int tk = tid >> 3, sub = tid & 7;
    if ((tid & ~63) / 8 >= ntok) return;            // (whole wavefronts leave)
    const bool live = tk < ntok;
    const float* row = lg + (live ? tk : 0) * LGP + sub * EPL;
    float v[EPL];
    float mx = -INFINITY, sum = 0.0f;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        v[i] = sub * EPL + i < E ? row[i] : -INFINITY;
        mx = fmaxf(mx, v[i]);
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if (!renorm) {
        // Expert by expert in ascending order, as softmax_topk adds them, so that a weight's bits do not depend on the kernel:
        // in step s lane `sub` = s continues from what lane s - 1 had in the step before (what the other lanes have is not used).
        float q[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) q[i] = sub * EPL + i < E ? expf(v[i] - mx) : 0.0f;      // (adding zero changes no bit of the sum)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s > 0) sum = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sum), 0x111 /* row_shr:1 */, 0xf, 0xf, false));
#pragma unroll
            for (int i = 0; i < EPL; ++i) sum += q[i];
        }
        sum = __shfl(sum, lane | 7, 64);
    }
    // the k largest logits in descending order, ties to the lower index, NaN as -inf
    int best_e[8];
    float raw[8];
    unsigned taken = 0;
    float den = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        best_e[j] = 0;
        raw[j] = 0.0f;
        if (j < k) {
            int e = 0x7fffffff;
            float o = -INFINITY, r = 0.0f;
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const float c = v[i] != v[i] ? -INFINITY : v[i];
                if (sub * EPL + i < E && !((taken >> i) & 1u) && (e == 0x7fffffff || c > o)) { e = sub * EPL + i; o = c; r = v[i]; }
            }
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) {
                const int e2 = __shfl_xor(e, off, 64);
                const float o2 = __shfl_xor(o, off, 64), r2 = __shfl_xor(r, off, 64);
                if (o2 > o || (o2 == o && e2 < e)) { e = e2; o = o2; r = r2; }
            }
            if (e / EPL == sub) taken |= 1u << (e % EPL);
            best_e[j] = e;
            raw[j] = r;
            den += expf(r - mx);
        }
    }
    if (!renorm) den = sum;
    if (live && sub == 0) {
        const size_t at = (size_t)(tw + tk) * k;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < k) { topk_idx[at + j] = best_e[j]; topk_w[at + j] = expf(raw[j] - mx) / den; }
    }
}

template <typename T, int EP, int TB>
static moe_status launch_route_wide(const Dims& d, const void* x, const void* Wg, const float* bias, float* logits, int* idx,
                                    float* w, hipStream_t s) {
    constexpr int TOK = ROUTE_WAVES * 16 / EP * TB;
    constexpr int lds = (64 * 256 + TOK * (EP + 4)) * (int)sizeof(float);
    auto kern = route_wide_kernel<T, EP, TB>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        attr_done = true;
    }
    ProfScope ps(PK_ROUTE, s);
    hipLaunchKernelGGL(kern, dim3((d.T + TOK - 1) / TOK), dim3(ROUTE_THREADS), lds, s,
                       (const T*)x, (const T*)Wg, bias, logits, idx, w, d.T, d.M, d.E, d.k, d.renorm);
    count_launch(LC_OTHER);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

static bool route_fits(int M, int EP) { return (M + 511) / 512 * 512 <= 32768 / EP; }

template <typename T, int EP, int TB>
static moe_status launch_route(const Dims& d, const void* x, const void* Wg, const float* bias,
                               float* logits, int* idx, float* w, hipStream_t s) {
    // Gate-weight rows held in LDS at a time.  If the whole matrix fits in 128 KB of
    // floats (route_fits) it is loaded once per workgroup, which then walks over many token groups;
    // otherwise it is streamed through LDS in 64 KB pieces for every token group.
    const int Mpad = ((d.M + 511) / 512) * 512;
    int MC = (32768 / EP) / 512 * 512;
    if (Mpad <= MC) MC = Mpad;
    else {
        MC = (16384 / EP) / 512 * 512;
        if (MC < 512) MC = 512;
    }
    size_t lds = ((size_t)MC * EP + (size_t)ROUTE_WAVES * RouteHeld<EP>::N * EP) * sizeof(float);
    auto kern = route_kernel<T, EP, TB>;
    static size_t attr_bytes = 0;                     // largest size asked for so far (per instantiation)
    if (lds > attr_bytes) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
        attr_bytes = lds;
    }
    int ngroups = (d.T + ROUTE_WAVES * TB - 1) / (ROUTE_WAVES * TB);
    const int cap = (lds > 80 * 1024 ? 1 : 2) * compute_units();      // one or two workgroups per CU fit
    int grid = ngroups < cap ? ngroups : cap;
    ProfScope ps(PK_ROUTE, s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(ROUTE_THREADS), lds, s,
                       (const T*)x, (const T*)Wg, bias, logits, idx, w, d.T, d.M, d.E, d.k, MC, d.renorm);
    count_launch(LC_OTHER);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

template <typename T>
static moe_status route_dispatch(const Dims& d, const void* x, const void* Wg, const float* bias,
                                 float* logits, int* idx, float* w, hipStream_t s) {
    // Tokens per wavefront: as many as the registers hold; two where that would leave half of the CUs without a workgroup
    // (64 tokens x 1024 x 8 experts 6.8 us against 9.7, 4096 x 512 x 8 5.9 / 8.4, 1024 x 1024 x 16 9.7 / 13.9) or, beyond
    // sixteen experts, fewer than two workgroups per CU.  Of five to eight experts in float32 only one such workgroup fits a CU,
    // so no more than one per CU (4300 x 64, 512, 1024 x 8 experts: two tokens 11.3, 11.3, 13.5 us, eight 10.0, 10.1, 11.5; 4096: 6.8, 7.2, 7.9 and
    // 9.9, 10.0, 11.4).
    const int cus = compute_units();
    constexpr bool f32 = sizeof(T) == 4;
    const bool few = d.T < (d.E > 4 && d.E <= 8 && f32 ? cus * ROUTE_WAVES * 2 + 1 : d.E <= 8 ? cus / 2 * ROUTE_WAVES * 8 : d.E <= 16 ? cus / 2 * ROUTE_WAVES * 4
                                                                    : 2 * cus * (ROUTE_WAVES * 16 / (d.E <= 32 ? 32 : 64)) * 2);
    if (d.E <= 4)
        return few ? launch_route<T, 4, 2>(d, x, Wg, bias, logits, idx, w, s) : launch_route<T, 4, 8>(d, x, Wg, bias, logits, idx, w, s);
    if (d.E <= 8)
        return few ? launch_route<T, 8, 2>(d, x, Wg, bias, logits, idx, w, s) : launch_route<T, 8, 8>(d, x, Wg, bias, logits, idx, w, s);
    if (d.E <= 16)
        return few ? launch_route<T, 16, 2>(d, x, Wg, bias, logits, idx, w, s) : launch_route<T, 16, 4>(d, x, Wg, bias, logits, idx, w, s);
    // Beyond sixteen experts: sixteen of them per wavefront, with the weights through LDS for every round of tokens (two
    // workgroups per CU), or all in a wavefront, with weights that stay in LDS where all fit.  The latter win from so many
    // rounds on; how many follows from the way of the weights to LDS, eight of a row per load or one by one.  us of the
    // former / the latter, columns 64 and 1024 (32 padded experts) or 512 (64):
    //   bfloat16, one by one   28 experts, 2 rounds: 24 / 28 and 46 / 53, 3: 34 / 34 and 67 / 62; 44, 2: 33 / 42 and 42 / 50, 3: 47 / 51 and 60 / 58
    //   bfloat16, by eights    32, 3: 29 / 32 and 47 / 47, 4: 37 / 39 and 60 / 57; 24 and 40 to 64: never (64, 12: 118 / 148)
    //   float32, one by one    28, 1: 18 / 21 and 36 / 40, 1.5: 25 / 24 and 66 / 47; 44, 1: 23 / 32 and 29 / 35, 1.5: 32 / 37 and 41 / 40
    //   float32, by eights     24, 3: 34 / 33 and 57 / 61, 4: 44 / 41 and 74 / 72; 32, 2: 24 / 27 and 41 / 39, 3: 34 / 33 and 58 / 48;
    //                          48, 6: 76 / 73 and 81 / 89, 8: 99 / 91 and 106 / 106; 64, 5: 64 / 63 and 69 / 68, 6: 76 / 72 and 81 / 78
    const int EP = d.E <= 32 ? 32 : 64, round = 2 * cus * (ROUTE_WAVES * 16 / EP) * 4;
    const bool eights = (d.E & 7) == 0 && ((uintptr_t)Wg & 15) == 0;
    const int rounds = !eights ? (f32 ? 1 : 2) : f32 ? (EP == 32 ? (d.E == 32 ? 2 : 3) : (d.E == 64 ? 5 : 6)) : d.E == 32 ? 3 : INT_MAX;
    long long most = (long long)rounds * round;      // tokens up to which sixteen experts per wavefront it is
    if (!eights && EP == 64 && d.M <= 384) most += most / 2;          // (60 experts, 1.5 rounds in float32: columns 64 32 / 37, 344 38 / 39, 504 42 / 41)
    const bool stay = route_fits(d.M, EP) && d.T > most;
    if (d.E <= 32) {
        if (stay) return launch_route<T, 32, 2>(d, x, Wg, bias, logits, idx, w, s);
        // (float32, one by one: two tokens per wavefront up to a whole round, 8192 x 1024 x 28 36 us against 42; but not for about
        // a thousand rows of a multiple of 16 KB: 1000 x 4096 x 20 51 us with four, 62 with two, 58 with all experts in a wavefront)
        const bool same_lines = !eights && d.T >= 700 && d.T < 2000 && (size_t)d.M * sizeof(T) % 16384 == 0;
        const bool two = same_lines ? false : f32 && !eights ? d.T <= round : few;
        return two ? launch_route_wide<T, 32, 2>(d, x, Wg, bias, logits, idx, w, s) : launch_route_wide<T, 32, 4>(d, x, Wg, bias, logits, idx, w, s);
    }
    if (stay) return launch_route<T, 64, 1>(d, x, Wg, bias, logits, idx, w, s);
    return few ? launch_route_wide<T, 64, 2>(d, x, Wg, bias, logits, idx, w, s) : launch_route_wide<T, 64, 4>(d, x, Wg, bias, logits, idx, w, s);
}

}  // namespace moe

extern "C" moe_status moe_route(const moe_config* cfg, const void* x, const void* Wg, const float* gate_bias,
                                float* logits, int32_t* topk_idx, float* topk_w, void* stream) {
    moe::Dims d;
    MOE_TRY(moe::make_dims(cfg, &d));
    if (!x || !Wg || !logits || !topk_idx || !topk_w) return MOE_ERR_NULL;
    hipStream_t s = (hipStream_t)stream;
    if (d.dtype == MOE_F32) return moe::route_dispatch<float>(d, x, Wg, gate_bias, logits, topk_idx, topk_w, s);
    return moe::route_dispatch<moe::bf16_t>(d, x, Wg, gate_bias, logits, topk_idx, topk_w, s);
}
