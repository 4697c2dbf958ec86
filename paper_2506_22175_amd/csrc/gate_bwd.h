// Gate backward up to dL, shared by the kernels that compute it: its own, and the launches of the GEMMs that follow
// GeLU-backward, beside which it runs.
#pragma once
#include "common.h"

namespace moe {

constexpr int GATE_THREADS = 256;

// dL[t,e] = p[t,e] * (dp[t,e] - sum_e' dp[t,e'] p[t,e']) with dp nonzero only at the chosen
// experts (the softmax Jacobian applied to the combine-weight gradients), then
// dWg += x^T dL.  A workgroup of 256 threads prepares dL for a block of DWG_TOK tokens, four
// lanes per token.
constexpr int DWG_TOK = 64;
constexpr int DWG_EMAX = 64;
constexpr int DWG_LD = DWG_EMAX + 4;     // floats per row of the block's LDS tile

// Combine-weight gradients of the block's (token, choice) pairs into sdw[ti*k + j]: either given,
// or the fixed-order sum of the GEMM epilogue's column-block partial sums (four lanes per pair).
// A thread has at most DWG_TOK*8*4/256 = 8 pairs; their slots are all requested before the first
// row of partial sums is read.
__device__ __forceinline__ void gate_block_dw(
    float* sdw, const int* __restrict__ slot, const float* __restrict__ dw, const float* __restrict__ dw_part,
    int parts, int t_first, int nt, int k) {
    constexpr int NI = DWG_TOK * 8 * 4 / GATE_THREADS;
    const int total = nt * k * 4;
    const int sub = threadIdx.x & 3;
    int sl[NI];
    float given[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int q = threadIdx.x + i * GATE_THREADS;
        const size_t at = (size_t)t_first * k + (q >> 2);          // pairs of the block are consecutive
        sl[i] = (q < total && dw_part) ? slot[at] : -1;
        given[i] = (q < total && !dw_part && sub == 0) ? dw[at] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int q = threadIdx.x + i * GATE_THREADS;
        if (q >= total) break;                                     // uniform over the four lanes of a pair
        float v = given[i];
        if (sl[i] >= 0) {
            const float* row = dw_part + (size_t)sl[i] * parts;
            if ((parts & 3) == 0) {
                // lane `sub` of the pair takes every fourth group of four partial sums, all
                // requested before the first is added (fixed order: groups ascending, then the lanes)
                const int ngrp = parts >> 2;
                for (int g0 = sub; g0 < ngrp; g0 += 32) {
                    float4 q4[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        q4[u] = (g0 + 4 * u < ngrp) ? *reinterpret_cast<const float4*>(row + 4 * (g0 + 4 * u))
                                                    : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
                    for (int u = 0; u < 8; ++u) v += (q4[u].x + q4[u].y) + (q4[u].z + q4[u].w);
                }
            } else {
                const int per = (parts + 3) >> 2;
                const int c1 = min(parts, (sub + 1) * per);
                for (int c = sub * per; c < c1; ++c) v += row[c];
            }
        }
        v += __shfl_xor(v, 1, 64);
        v += __shfl_xor(v, 2, 64);
        if (sub == 0) sdw[q >> 2] = v;
    }
}

// The block's logits (nt rows of E floats, contiguous in memory) into the LDS tile; a thread's
// loads (at most DWG_TOK*DWG_EMAX/256 = 16 floats) are all requested before the first is written.
__device__ __forceinline__ void gate_block_logits(float (*tile)[DWG_LD], const float* __restrict__ logits,
                                                  int t_first, int nt, int E) {
    const float* src = logits + (size_t)t_first * E;
    if ((E & 3) == 0 && (((size_t)t_first * E) & 3) == 0) {
        constexpr int NI = DWG_TOK * DWG_EMAX / 4 / GATE_THREADS;
        const int E4 = E >> 2, total = nt * E4;
        float4 v[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int q = threadIdx.x + i * GATE_THREADS;
            v[i] = q < total ? reinterpret_cast<const float4*>(src)[q] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int q = threadIdx.x + i * GATE_THREADS;
            if (q < total) *reinterpret_cast<float4*>(&tile[q / E4][4 * (q % E4)]) = v[i];
        }
    } else {
        for (int q = threadIdx.x; q < nt * E; q += GATE_THREADS) tile[q / E][q % E] = src[q];
    }
}

// The experts chosen by the token of this thread (thread / 4 within the block), -1 beyond k or past the
// last token; requested first so that the read is over by the time gate_block_dl needs it.
__device__ __forceinline__ void gate_block_ids(int (&ids)[8], const int* __restrict__ topk_idx, int t_first, int nt, int k) {
    const int ti = threadIdx.x >> 2;
#pragma unroll
    for (int j = 0; j < 8; ++j) ids[j] = (ti < nt && j < k) ? topk_idx[(size_t)(t_first + ti) * k + j] : -1;
}

// dL of the block's tokens, four lanes per token (lane `sub` takes experts sub, sub+4, ...; maxima and
// sums are folded over the four lanes).  The LDS tile holds the logits on entry and dL on return, with
// zeros in the rows of missing tokens and in columns E .. E16-1 (E16 = E rounded up to 16).  dL also
// goes to global memory, and, if dLt is given, as two bfloat16 terms (hi + lo, 16 bits of mantissa)
// to dLt[(e/16)*32 + e%16][token] and dLt[(e/16)*32 + 16 + e%16][token], rows of tp_pad tokens.
__device__ __forceinline__ void gate_block_dl(
    float (*tile)[DWG_LD], const float* sdw, const int (&ids)[8], float* __restrict__ dL,
    bf16_t* __restrict__ dLt, int tp_pad, int t_first, int tl0, int nt, int E, int k, int renorm) {
    const int ti = threadIdx.x >> 2, sub = threadIdx.x & 3;
    const int E16 = (E + 15) & ~15;
    const bool live = ti < nt;
    const int t = t_first + ti;
    float* row = tile[ti];
    float mx = -INFINITY;
    if (live)
        for (int e = sub; e < E; e += 4) mx = fmaxf(mx, row[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
    float g[8], pc[8];                  // gradient and exp(logit - max) of the chosen experts
    float den = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        g[j] = 0.0f; pc[j] = 0.0f;
        if (live && j < k) {
            g[j] = sdw[ti * k + j];
            pc[j] = expf(row[ids[j]] - mx);
            den += pc[j];
        }
    }
    if (!renorm) {
        float sum = 0.0f;
        if (live)
            for (int e = sub; e < E; e += 4) sum += expf(row[e] - mx);
        sum += __shfl_xor(sum, 1, 64);
        sum += __shfl_xor(sum, 2, 64);
        den = sum;
    }
    // (renormalised weights are a softmax over the chosen logits only: dL_e = w_j (dw_j - sum_j' dw_j' w_j')
    // for a chosen e, zero otherwise)
    const float inv = 1.0f / den;
    float inner = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) inner = fmaf(g[j], pc[j] * inv, inner);
    for (int e = sub; e < E16; e += 4) {
        float v = 0.0f;
        if (live && e < E) {
            float dp = 0.0f;
            bool chosen = false;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (ids[j] == e) { dp = g[j]; chosen = true; }
            if (!renorm) v = expf(row[e] - mx) * inv * (dp - inner);
            else if (chosen) v = expf(row[e] - mx) * inv * (dp - inner);
            dL[(size_t)t * E + e] = v;
        }
        row[e] = v;
        if (dLt) {
            const bf16_t hi = f32_to_bf16(v);
            const bf16_t lo = f32_to_bf16(v - bf16_to_f32(hi));
            bf16_t* col = dLt + ((size_t)((e >> 4) * 32 + (e & 15)) * tp_pad + tl0 + ti);
            col[0] = hi;
            col[(size_t)16 * tp_pad] = lo;
        }
    }
}

constexpr int GATE_DL_LDS = (DWG_TOK * DWG_LD + DWG_TOK * 8) * (int)sizeof(float);
// dL of one block of tokens (block / per_part is the partition), to global memory in float and, for bfloat16 storage,
// transposed as hi + lo bfloat16 terms (for the matrix-core kernel of the gate-weight gradient).
__device__ __forceinline__ void gate_dl(const GateDlArgs& a, int block, char* smem) {
    float (*sdl)[DWG_LD] = reinterpret_cast<float (*)[DWG_LD]>(smem);
    float* sdw = reinterpret_cast<float*>(smem) + DWG_TOK * DWG_LD;
    const int z = block / a.per_part;
    const int t_begin = (a.p0 + z) * a.Tp;
    const float* dw_part = a.dw_part ? a.dw_part + z * a.dw_part_stride : nullptr;
    bf16_t* dLt = a.dLt ? a.dLt + z * a.dLt_stride : nullptr;
    const int tl0 = (block - z * a.per_part) * DWG_TOK;
    const int nt = max(0, min(DWG_TOK, a.Tp - tl0));
    int ids[8];
    gate_block_ids(ids, a.topk_idx, t_begin + tl0, nt, a.k);
    gate_block_logits(sdl, a.logits, t_begin + tl0, nt, a.E);
    gate_block_dw(sdw, a.slot, a.dw, dw_part, a.parts, t_begin + tl0, nt, a.k);
    __syncthreads();
    gate_block_dl(sdl, sdw, ids, a.dL, dLt, a.tp_pad, t_begin + tl0, tl0, nt, a.E, a.k, a.renorm);
}

}  // namespace moe
