// Dispatch (S), combine (R) and their backward counterparts for one partition.
// In the paper S and R are the two All-to-All exchanges of expert parallelism
// (Fig. 1, Section II-A); on one GPU they are local row permutations between the
// token-ordered tensors T_I / T_O and the expert-contiguous T_DI / T_DO.  They
// are bound by HBM: every kernel moves whole rows with 16-byte accesses, one
// wavefront per token, and reads each token row once however many experts it
// goes to.  A launch does one partition, or the partition blockIdx.z of several
// (a launch takes 4.6 us of the GPU however little it does): partition buffers then
// lie a constant number of bytes apart.
#include "common.h"
#include "gate_bwd.h"

namespace moe {

constexpr int PERM_THREADS = 256;
constexpr int PERM_WAVES = PERM_THREADS / 64;

// 16-byte row accesses; NT = non-temporal (the row is read or written once per kernel)
typedef unsigned u32x4_hw __attribute__((ext_vector_type(4)));
template <bool NT> __device__ __forceinline__ uint4 ld_row(const uint4* p) {
    if (NT) {
        u32x4_hw v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_hw*>(p));
        return make_uint4(v[0], v[1], v[2], v[3]);
    }
    return *p;
}
template <bool NT> __device__ __forceinline__ void st_row(uint4* p, const uint4& u) {
    if (NT) {
        u32x4_hw v = {u.x, u.y, u.z, u.w};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4_hw*>(p));
    } else {
        *p = u;
    }
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// 16 bytes <-> floats (8 bf16 or 4 float)
template <typename T> struct Unit;
template <> struct Unit<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void to_float(const uint4& u, float* o) {
        const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[2 * i] = __uint_as_float(w[i] << 16);
            o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ uint4 from_float(const float* v) {
        return make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
};
template <> struct Unit<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void to_float(const uint4& u, float* o) {
        o[0] = __uint_as_float(u.x); o[1] = __uint_as_float(u.y); o[2] = __uint_as_float(u.z); o[3] = __uint_as_float(u.w);
    }
    static __device__ __forceinline__ uint4 from_float(const float* v) {
        return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
    }
};

// What the row permutations of one or several consecutive partitions work on.  Pointers are those of partition p0;
// strides are bytes from one partition's buffer to the next one's and may be negative (buffers used in turn).
struct RowArgs {
    const void* src[2];              // token-major rows that go to the experts; blockIdx.y chooses
    char* dst[2];                    // partition buffers they go to
    long long dst_stride[2];
    const char* rows;                // T_DO buffer: the combine's source; with `dw` also its gradient's
    long long rows_stride;
    const int* slot;
    const float* w;
    float* dw;
    void* y;
    int p0, Tp, M, k;
};

// dst[slot[t,j]] = src[t]; optionally on the way dw[t,j] = <src[t], rows[slot[t,j]]> (backward's dispatch of dy where
// T_DO was kept) and y[t] = sum_j w[t,j] rows[slot[t,j]] (forward's combine, which reads the same rows, in a step that
// has not run it yet).  dst may be the very buffer of these rows (dT_DO in T_DO's place): a row belongs to one token's
// wavefront, which has read a piece of it before it overwrites that piece.  One wavefront per token.  KM: choices per
// token at most.  All reads of a piece of the row - the token's and its experts' - are in flight before the first is
// used: 32768 tokens x 2048, two choices, with dw, 52 us a partition of 16384 under rocprofv3, 67 to 72 with the
// experts' rows read one after another (39 us is the time of a copy of as many bytes).
// (float accumulation, ascending j; a lane's part of a dot in ascending column order)
// STRAIGHT: rows through descriptors of their own, where lanes past the end and rows that are not there read zeros and write
// nothing.  Else under execution masks, where the compiler puts a wait for all that is in flight in front of every store: a
// wavefront has one store on its way.  See dispatch_straight.
template <typename T, int KM, bool DW, bool COMB, bool STRAIGHT>
__global__ __launch_bounds__(PERM_THREADS) void dispatch_kernel(RowArgs a) {
    const int lane = threadIdx.x & 63;
    const int tl = blockIdx.x * PERM_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tl >= a.Tp) return;
    const int z = blockIdx.z, which = blockIdx.y, k = a.k, M = a.M;
    const bool comb = COMB && which == 0;          // (the rows of the other source have nothing to do with T_DO)
    const size_t t = (size_t)(a.p0 + z) * a.Tp + tl;
    constexpr int N = Unit<T>::N;
    constexpr int UN = !DW && !COMB ? 4 : KM > 4 && !STRAIGHT ? 1 : KM > 2 ? 2 : 4;      // 16-byte units per row and lane in flight
    const int U = M / N;
    T* dst = reinterpret_cast<T*>(a.dst[which] + z * a.dst_stride[which]);
    const T* rows = DW || COMB ? reinterpret_cast<const T*>(a.rows + z * a.rows_stride) : nullptr;
    int s[KM];
    float ws[KM], dot[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        // (in straight-line code all on their way together; many wavefronts that write one store at a time are slower so, 8192 x 512
        // bfloat16, two choices 7.9 us instead of 6.7)
        if constexpr (STRAIGHT) s[j] = a.slot[t * k + min(j, k - 1)];
        else s[j] = j < k ? a.slot[t * k + j] : -1;
    }
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        if (STRAIGHT && j >= k) s[j] = -1;
        ws[j] = comb && s[j] >= 0 ? a.w[t * k + j] : 0.0f;
        dot[j] = 0.0f;
    }
    const int row_bytes = M * (int)sizeof(T);
    auto descriptor = [&](const void* row, bool there) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), 0, there ? row_bytes : 0, 0x00020000);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t row, int c) __attribute__((always_inline)) {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(row, c * 16, 0, 2 /* non-temporal */));
    };
    auto store = [&](__amdgpu_buffer_rsrc_t row, int c, const uint4& u) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_hw, u), row, c * 16, 0, 0);
    };
    const uint4* in = reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(a.src[which]) + t * M);
    const uint4 zero = make_uint4(0, 0, 0, 0);
    for (int c0 = 0; c0 < U; c0 += 64 * UN) {
        uint4 v[UN], r[KM][UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int c = c0 + u * 64 + lane;
            if constexpr (STRAIGHT) v[u] = load(descriptor(in, true), c);
            else if (c < U) v[u] = ld_row<true>(in + c);
        }
        if constexpr (DW || COMB) {
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                const uint4* row = reinterpret_cast<const uint4*>(rows + (size_t)max(s[j], 0) * M);
                const bool there = s[j] >= 0 && (DW || comb);
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int c = c0 + u * 64 + lane;
                    if constexpr (STRAIGHT) {
                        r[j][u] = load(descriptor(row, there), c);
                    } else {
                        r[j][u] = zero;
                        if (c < U && there) r[j][u] = ld_row<true>(row + c);
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            if (STRAIGHT && j >= k) break;
            if (!STRAIGHT && s[j] < 0) continue;
            uint4* out = reinterpret_cast<uint4*>(dst + (size_t)(STRAIGHT ? max(s[j], 0) : s[j]) * M);
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int c = c0 + u * 64 + lane;
                if constexpr (STRAIGHT) store(descriptor(out, s[j] >= 0), c, v[u]);
                else if (c < U) st_row<false>(out + c, v[u]);
            }
        }
        if constexpr (DW || COMB) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int c = c0 + u * 64 + lane;
                float x[N], acc[N];
                Unit<T>::to_float(STRAIGHT || c < U ? v[u] : zero, x);
#pragma unroll
                for (int i = 0; i < N; ++i) acc[i] = 0.0f;
#pragma unroll
                for (int j = 0; j < KM; ++j) {
                    float q[N];
                    Unit<T>::to_float(r[j][u], q);
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        if constexpr (DW) dot[j] = fmaf(x[i], q[i], dot[j]);
                        if constexpr (COMB) acc[i] = fmaf(ws[j], q[i], acc[i]);
                    }
                }
                if constexpr (COMB) {
                    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<T*>(a.y) + t * M);
                    if constexpr (STRAIGHT) store(descriptor(out, comb), c, Unit<T>::from_float(acc));
                    else if (c < U && comb) st_row<false>(out + c, Unit<T>::from_float(acc));
                }
            }
        }
    }
    if constexpr (DW) {
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            if (j < k) {
                const float d = wave_sum(dot[j]);
                if (lane == 0) a.dw[t * k + j] = s[j] >= 0 ? d : 0.0f;
            }
        }
    }
}

// y[t] = sum_j w[t,j] * rows[slot[t,j]]  (float accumulation, ascending j).  One wavefront per
// token; four 16-byte units per lane are in flight per source row.
template <typename T>
__global__ __launch_bounds__(PERM_THREADS) void combine_kernel(RowArgs a) {
    const int lane = threadIdx.x & 63;
    const int tl = blockIdx.x * PERM_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tl >= a.Tp) return;
    const int k = a.k;
    const size_t t = (size_t)(a.p0 + blockIdx.z) * a.Tp + tl;
    const T* DO = reinterpret_cast<const T*>(a.rows + blockIdx.z * a.rows_stride);
    constexpr int N = Unit<T>::N;
    const int U = a.M / N;
    int s[8];
    float ws[8];
    auto choices = [&](int j0, int j1) __attribute__((always_inline)) {      // (all on their way together)
#pragma unroll
        for (int j = j0; j < j1; ++j) {
            s[j] = a.slot[t * k + min(j, k - 1)];
            ws[j] = a.w[t * k + min(j, k - 1)];
        }
    };
    choices(0, 2);
    if (k > 2) choices(2, 8);
    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<T*>(a.y) + t * a.M);
    for (int c0 = 0; c0 < U; c0 += 256) {
        float acc[4][N];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int i = 0; i < N; ++i) acc[u][i] = 0.0f;
        for (int j = 0; j < k; ++j) {
            if (s[j] < 0) continue;
            const uint4* in = reinterpret_cast<const uint4*>(DO + (size_t)s[j] * a.M);
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * 64 + lane;
                v[u] = c < U ? ld_row<true>(in + c) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float r[N];
                Unit<T>::to_float(v[u], r);
#pragma unroll
                for (int i = 0; i < N; ++i) acc[u][i] = fmaf(ws[j], r[i], acc[u][i]);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * 64 + lane;
            if (c < U) st_row<false>(out + c, Unit<T>::from_float(acc[u]));
        }
    }
}

// dWg[i] += sum_b part[b][i], partition by partition: THREADS/8 consecutive outputs per workgroup, eight threads per
// output each taking every eighth partial block, then a fixed-order sum of the eight.
template <int THREADS>
__device__ __forceinline__ void gate_dwg_reduce(const GateSums& g, int block, float* red) {
    constexpr int COLS = THREADS / 8;
    const int col = threadIdx.x % COLS, sl = threadIdx.x / COLS;
    const int i = block * COLS + col;
    float total = 0.0f;
    if (sl == 0 && i < g.ME && !g.store) total = g.dWg[i];
    for (int q = 0; q < g.np; ++q) {
        const float* part = g.part + q * g.part_stride;
        float s = 0.0f;
        if (i < g.ME)
#pragma unroll 4
            for (int b = sl; b < g.nblk; b += 8) s += part[(size_t)b * g.ME + i];
        if (q) __syncthreads();
        red[sl * COLS + col] = s;
        __syncthreads();
        if (sl == 0) {
            float tot = 0.0f;
#pragma unroll
            for (int r = 0; r < 8; ++r) tot += red[r * COLS + col];
            total = q == 0 && g.store ? tot : total + tot;
        }
    }
    if (sl == 0 && i < g.ME) g.dWg[i] = total;
}

// Dispatch backward, both storage types: a workgroup owns the columns that one wavefront covers with 16
// bytes per lane and DXB_TG token groups, one wavefront each; they share the gate weights of those columns
// in LDS.  Tokens per group: sixteen (staging the weights then costs an eighth of the rows' traffic at 16
// experts), fewer where that would leave compute units without a workgroup, in steps of the four that make
// one round (2048 tokens x 512 columns, 8 experts, by HIP events: 16 workgroups of 16 tokens per wavefront
// 12.4 us, 64 of four 6.9; 4096 x 1024: 15.8 -> 10.0).
constexpr int DXB_CT = 64;           // column threads: one wavefront
constexpr int DXB_TG = 8;            // token groups per workgroup
constexpr int DXB_TOK = 16;          // most tokens per group
constexpr int DXB_THREADS = DXB_CT * DXB_TG;

// Partitions p0 .. p0 + gridDim.z - 1.  Blocks from token_rows on (in y) do not belong to dispatch backward: they add up
// the gate-weight gradient's partial sums, which saves that its own launch.  (The kernels' pointers are parameters of their own:
// what is read through a structure counts as something that the stores to dx may change, and is read by every lane instead
// of once per wavefront.  float32, 1001 tokens x 776 x 6 experts, five choices 9.8 us so, 6.6 now; 8192 x 2048 x 64, eight: 166 and 139.
// Nine to sixteen experts in bfloat16 take them from the structure all the same: 4096 x 2048 x 16 12.1 us so, 12.7 with parameters.)
struct DispatchBwdArgs {
    const void* dDI;
    long long dDI_stride;                // bytes
    const int* slot;
    const float* dL;
    const void* Wg;
    void* dx;
    int p0, Tp, tok, M, E, k, token_rows;
    GateSums sums;
};
template <int THREADS>
__device__ __forceinline__ bool dispatch_bwd_sums(const DispatchBwdArgs& a, char* smem) {
    if ((int)blockIdx.y < a.token_rows) return false;
    const int block = (((int)blockIdx.y - a.token_rows) * gridDim.x + blockIdx.x) * gridDim.z + blockIdx.z;
    gate_dwg_reduce<THREADS>(a.sums, block, reinterpret_cast<float*>(smem));
    return true;
}

// dx[t] = sum_j dDI[slot[t,j]] + dL[t,:] Wg^T for float32 storage.  A lane owns four columns; the gate
// weights of the workgroup's 256 columns sit in LDS expert by expert (row pitch DXF_PITCH floats: the
// transposing writes of four neighbouring experts fall into different banks), so that a lane's 16-byte read
// feeds the multiply-adds of four tokens; the gate gradients are wave-uniform scalar loads.  Bound by
// latency at small sizes (1024 tokens x 512 columns, 8 experts: 6.9 us, 10.8 with the whole gate matrix in
// LDS) and by the row traffic at large ones; a column slice fits LDS at every size, up to 64 experts.
constexpr int DXF_COLS = DXB_CT * 4;
constexpr int DXF_PITCH = DXF_COLS + 4;
__global__ __launch_bounds__(DXB_THREADS, 2) void dispatch_bwd_f32_kernel(
    const float* __restrict__ dDI, const int* __restrict__ slot, const float* __restrict__ dL,
    const float* __restrict__ Wg, float* __restrict__ dx, DispatchBwdArgs a) {
    extern __shared__ __attribute__((aligned(16))) char dxf_smem[];
    if (dispatch_bwd_sums<DXB_THREADS>(a, dxf_smem)) return;
    dDI = reinterpret_cast<const float*>(reinterpret_cast<const char*>(dDI) + blockIdx.z * a.dDI_stride);
    const int t_begin = (a.p0 + (int)blockIdx.z) * a.Tp, t_count = a.Tp, tok = a.tok, M = a.M, E = a.E, k = a.k;
    float* wgt = reinterpret_cast<float*>(dxf_smem);
    const int lane = threadIdx.x & 63;
    const int tg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c_base = blockIdx.x * DXF_COLS;
    const int ncols = min(DXF_COLS, M - c_base);
    const int c = c_base + lane * 4;
    const bool c_ok = c < M;                       // M is a multiple of eight: a lane's four columns exist or not
    const int cc = c_ok ? c : 0;
    const int tl0 = min((int)(blockIdx.y * DXB_TG + tg) * tok, t_count);
    const int tl1 = min(tl0 + tok, t_count);
    const float* wsrc = Wg + (size_t)c_base * E;
    if ((E & 3) == 0) {
        const int E4 = E >> 2;
        for (int q = threadIdx.x; q < ncols * E4; q += DXB_THREADS) {
            const int col = q / E4, e = (q - col * E4) * 4;
            const float4 v = reinterpret_cast<const float4*>(wsrc)[q];
            wgt[(e + 0) * DXF_PITCH + col] = v.x; wgt[(e + 1) * DXF_PITCH + col] = v.y;
            wgt[(e + 2) * DXF_PITCH + col] = v.z; wgt[(e + 3) * DXF_PITCH + col] = v.w;
        }
    } else {
        for (int q = threadIdx.x; q < ncols * E; q += DXB_THREADS) {
            const int col = q / E;
            wgt[(q - col * E) * DXF_PITCH + col] = wsrc[q];
        }
    }
    __syncthreads();
    for (int tb = tl0; tb < tl1; tb += 4) {
        float4 acc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const float* g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) g[u] = dL + (size_t)(t_begin + min(tb + u, tl1 - 1)) * E;
        for (int j = 0; j < k; ++j) {
            // the four tokens' rows of choice j in flight together (a missing row is read from row 0 and not added)
            float4 v[4];
            int sj[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                sj[u] = tb + u < tl1 ? slot[(size_t)(t_begin + tb + u) * k + j] : -1;
                v[u] = *reinterpret_cast<const float4*>(dDI + (size_t)max(sj[u], 0) * M + cc);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (sj[u] >= 0) { acc[u].x += v[u].x; acc[u].y += v[u].y; acc[u].z += v[u].z; acc[u].w += v[u].w; }
        }
        const float* wl = wgt + lane * 4;
#pragma unroll 4
        for (int e = 0; e < E; ++e) {
            const float4 w = *reinterpret_cast<const float4*>(wl + e * DXF_PITCH);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float ge = g[u][e];
                acc[u].x = fmaf(ge, w.x, acc[u].x); acc[u].y = fmaf(ge, w.y, acc[u].y);
                acc[u].z = fmaf(ge, w.z, acc[u].z); acc[u].w = fmaf(ge, w.w, acc[u].w);
            }
        }
        if (c_ok) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (tb + u < tl1) *reinterpret_cast<float4*>(dx + (size_t)(t_begin + tb + u) * M + c) = acc[u];
        }
    }
}

// dx[t] = sum_j dDI[slot[t,j]] + dL[t,:] Wg^T for bfloat16 storage, with the gate term on the
// matrix cores.  A lane owns eight consecutive columns (a wavefront 512, so every row access is
// a coalesced 1 KB), and its gate weights are the second operand of
// v_mfma_f32_4x4x4_16B_bf16: that instruction multiplies sixteen independent 4x4 blocks, block
// b = lane/4, D_b[i][j] += sum_k A_b[i][k] B_b[k][j], lane 4b+j holding column j of B_b and of
// D_b (rows i in its four result registers) and lane 4b+i holding row i of A_b.  With
// A_b[i][k] = dL[token i][expert 4g+k] (the same four tokens in every block) and
// B_b[k][j] = Wg[column of lane 4b+j][expert 4g+k], one instruction per column and expert
// group gives a lane the gate term of four tokens at one of its columns, at 1/8 of the issue
// slots of float FMAs.  dL is split into two bfloat16 terms (hi + lo), which keeps 16 bits of
// its mantissa; Wg is bfloat16 already.  With more than sixteen experts the products are float ones, all of
// dL's bits and its infinities included: v_mfma_f32_4x4x1_16B_f32, the same blocks with one expert per
// instruction and the weights widened when they are read.  There dL comes through LDS, in one request per round, and
// 128 registers leave room for a second workgroup on the CU (launches back to back: 8192 tokens x 768 columns x 64
// experts 23 us, 29 with dL in four requests one after the other and 156 registers; 8192 x 768 x 32: 15 and 20;
// 16384 x 2048 x 64: 82 and 101; in a step, its inputs not in the caches, the first is 34).  Up to 64 experts: a slice of the gate
// weights is at most 65 KB, so that two workgroups still fit a CU (the former: 1065 us with the weights read from
// memory again for every token; 776 columns x 6 experts x 1001 tokens: 22.4 -> 11.0
// by the number of tokens per group).  The kernel is bound by the latency of its row reads,
// so it is built for many wavefronts: the gate weights stay in LDS (read again every round)
// rather than in 64 registers, which lets four wavefronts per SIMD run.
typedef short bf16x4_hw __attribute__((ext_vector_type(4)));
typedef float f32x4_hw __attribute__((ext_vector_type(4)));
template <int EG>                    // expert groups of four: E <= 4*EG
__global__ __launch_bounds__(DXB_THREADS, EG > 4 ? 4 : 2) void dispatch_bwd_mfma_kernel(
    const bf16_t* __restrict__ dDI, const int* __restrict__ slot, const float* __restrict__ dL,
    const bf16_t* __restrict__ Wg, bf16_t* __restrict__ dx, DispatchBwdArgs a) {
    extern __shared__ __attribute__((aligned(16))) char dxm_smem[];
    if (dispatch_bwd_sums<DXB_THREADS>(a, dxm_smem)) return;
    if constexpr (EG == 4) {
        dDI = (const bf16_t*)a.dDI; slot = a.slot; dL = a.dL; Wg = (const bf16_t*)a.Wg; dx = (bf16_t*)a.dx;
    }
    dDI = reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(dDI) + blockIdx.z * a.dDI_stride);
    const int t_begin = (a.p0 + (int)blockIdx.z) * a.Tp, t_count = a.Tp, tok = a.tok, M = a.M, E = a.E, k = a.k;
    const int ct = threadIdx.x % DXB_CT;                       // column thread
    const int tg = __builtin_amdgcn_readfirstlane(threadIdx.x / DXB_CT);
    const int c = (blockIdx.x * DXB_CT + ct) * 8;
    const bool c_ok = c < M;                       // lanes beyond the row still feed the A operand
    const int lane = threadIdx.x & 63;
    const int tl0 = min((int)(blockIdx.y * DXB_TG + tg) * tok, t_count);
    const int tl1 = min(tl0 + tok, t_count);
    // The slots of the group's (token, choice) pairs, one per lane (two registers cover 16 tokens x 8
    // choices); a pair's slot is then broadcast from its lane, which costs no memory access per row.
    const int nsl = (tl1 - tl0) * k;
    const int* sl0 = slot + (size_t)(t_begin + tl0) * k;
    const int sv0 = lane < nsl ? sl0[lane] : -1;
    const int sv1 = lane + 64 < nsl ? sl0[lane + 64] : -1;
    const int cc = c_ok ? c : 0;
    // rows of four tokens, choices j0 and j0 + 1: eight 16-byte reads in flight per lane, no branch
    // around them (a missing row is read from row 0 and replaced by zeros)
    auto request = [&](int tb, int j0, uint4 (&raw)[4][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int i = (tb - tl0 + u) * k + j0 + jj;
                const int s0 = __builtin_amdgcn_readlane(sv0, i & 63), s1 = __builtin_amdgcn_readlane(sv1, i & 63);
                const int sj = (tb + u < tl1 && j0 + jj < k) ? (i < 64 ? s0 : s1) : -1;
                const uint4 v = ld_row<true>(reinterpret_cast<const uint4*>(dDI + (size_t)max(sj, 0) * M + cc));
                raw[u][jj] = sj >= 0 ? v : make_uint4(0, 0, 0, 0);
            }
    };
    constexpr bool SPLIT = EG <= 4;                // dL as two bfloat16 terms (else float products)
    // gate gradients of this lane's token (tb + lane%4) for the A operand
    auto request_dl = [&](int tb, float4 (&dl)[SPLIT ? EG : 1]) __attribute__((always_inline)) {
        const int ta = tb + (lane & 3);
#pragma unroll
        for (int g = 0; g < EG; ++g) {
            dl[g] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (ta < tl1) {
                const float* row = dL + (size_t)(t_begin + ta) * E + 4 * g;
                if (E == 4 * EG) {
                    dl[g] = *reinterpret_cast<const float4*>(row);
                } else {
                    if (4 * g + 0 < E) dl[g].x = row[0];
                    if (4 * g + 1 < E) dl[g].y = row[1];
                    if (4 * g + 2 < E) dl[g].z = row[2];
                    if (4 * g + 3 < E) dl[g].w = row[3];
                }
            }
        }
    };
    // With more than sixteen experts they would take too many registers, and piece by piece too many round trips to
    // memory: the four tokens' go through a row each of LDS, which the wavefront has to itself.  They are 4*E
    // consecutive floats, of which lane l requests l, l + 64, ...
    constexpr int DLN = EG > 4 ? EG / 4 : 1;
    constexpr int DLP = 4 * EG + 4;                // floats per row: the four tokens' reads fall into different banks
    float* dl_rows = reinterpret_cast<float*>(dxm_smem + DXB_CT * (64 * EG + 16)) + tg * 4 * DLP;
    auto request_dl_rows = [&](int tb, float (&v)[DLN]) __attribute__((always_inline)) {
        const int n = max(tl1 - tb, 0) * E;        // (fewer than 4*E at the end)
#pragma unroll
        for (int i = 0; i < DLN; ++i) {
            const int q = lane + 64 * i;
            v[i] = q < min(n, 4 * E) ? dL[(size_t)(t_begin + tb) * E + q] : 0.0f;
        }
    };
    auto put_dl_rows = [&](const float (&v)[DLN]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < DLN; ++i) {
            const int q = lane + 64 * i, u = q / E;
            if (u < 4) dl_rows[u * DLP + q - u * E] = v[i];
        }
        __builtin_amdgcn_wave_barrier();
    };
    // Gate weights of this workgroup's columns into LDS with coalesced 16-byte reads.  A lane's
    // piece (64*EG bytes: 8 columns x 4*EG experts) is padded by 16 bytes so that the reads of a
    // wavefront spread over all banks.  The weights are staged before the first rows are requested:
    // an LDS write waits for every load issued before it, and the rows take several times longer
    // to arrive than the weights.
    constexpr int CHUNK = 64 * EG;
    constexpr int PITCH = CHUNK + 16;
    const int c_base = blockIdx.x * DXB_CT * 8;
    const int ncols = min(DXB_CT * 8, M - c_base);
    const int pieces = ncols * EG / 2;             // 16-byte pieces of the slice
    constexpr int NPC = (DXB_CT * 8 * EG / 2 + DXB_THREADS - 1) / DXB_THREADS;     // at most so many per thread
    if (E == 4 * EG) {
        const uint4* src = reinterpret_cast<const uint4*>(Wg + (size_t)c_base * E);
        uint4 piece[NPC];
#pragma unroll
        for (int i = 0; i < NPC; ++i) piece[i] = src[min((int)threadIdx.x + i * DXB_THREADS, pieces - 1)];
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int q = threadIdx.x + i * DXB_THREADS;
            const int byte = q * 16;
            if (q < pieces) *reinterpret_cast<uint4*>(dxm_smem + (byte / CHUNK) * PITCH + byte % CHUNK) = piece[i];
        }
    } else {
        for (int q = threadIdx.x; q < ncols * 4 * EG; q += DXB_THREADS) {
            const int col = q / (4 * EG), e = q % (4 * EG);
            const bf16_t v = e < E ? Wg[(size_t)(c_base + col) * E + e] : (bf16_t)0;
            *reinterpret_cast<bf16_t*>(dxm_smem + (col / 8) * PITCH + (col % 8) * 8 * EG + e * 2) = v;
        }
    }
    uint4 raw[4][2];
    float4 dl[SPLIT ? EG : 1];
    float dlv[DLN];
    auto request_all = [&](int tb) __attribute__((always_inline)) {
        if constexpr (SPLIT) request_dl(tb, dl);
        else request_dl_rows(tb, dlv);
        request(tb, 0, raw);
    };
    if constexpr (!SPLIT)                          // experts that do not exist: zeros, as in the weights
        if (lane < 4)
            for (int e = E; e < 4 * EG; ++e) dl_rows[lane * DLP + e] = 0.0f;
    request_all(tl0);
    __syncthreads();
    for (int tb = tl0; tb < tl1; tb += 4) {
        if (tb > tl0) request_all(tb);
        f32x4_hw gate[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) gate[i] = f32x4_hw{0.0f, 0.0f, 0.0f, 0.0f};
        int my_off = ct * PITCH;                   // opaque: the compiler must not keep the weights in registers
        asm volatile("" : "+v"(my_off));
        auto weights = [&](int g, bf16x4_hw (&w)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = *reinterpret_cast<const bf16x4_hw*>(dxm_smem + my_off + (i * EG + g) * 8);
        };
        if constexpr (SPLIT) {
            bf16x4_hw hi[EG], lo[EG];
#pragma unroll
            for (int g = 0; g < EG; ++g) {
                const float v[4] = {dl[g].x, dl[g].y, dl[g].z, dl[g].w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bf16_t h = f32_to_bf16(v[r]);
                    hi[g][r] = (short)h;
                    lo[g][r] = (short)f32_to_bf16(v[r] - bf16_to_f32(h));
                }
            }
#pragma unroll
            for (int g = 0; g < EG; ++g) {
                bf16x4_hw w[8];
                weights(g, w);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    gate[i] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(hi[g], w[i], gate[i], 0, 0, 0);
                    gate[i] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(lo[g], w[i], gate[i], 0, 0, 0);
                }
            }
        } else {
            put_dl_rows(dlv);
#pragma unroll 2
            for (int g = 0; g < EG; ++g) {
                const float4 d4 = *reinterpret_cast<const float4*>(dl_rows + (lane & 3) * DLP + 4 * g);
                const float v[4] = {d4.x, d4.y, d4.z, d4.w};
                bf16x4_hw w[8];
                weights(g, w);
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        gate[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(v[r], bf16_to_f32((bf16_t)w[i][r]), gate[i], 0, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();
        }
        float acc[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float r0[8], r1[8];
            Unit<bf16_t>::to_float(raw[u][0], r0);
            Unit<bf16_t>::to_float(raw[u][1], r1);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[u][i] = gate[i][u] + (r0[i] + r1[i]);
        }
        for (int j0 = 2; j0 < k; j0 += 2) {            // further choices (k > 2)
            request(tb, j0, raw);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float r0[8], r1[8];
                Unit<bf16_t>::to_float(raw[u][0], r0);
                Unit<bf16_t>::to_float(raw[u][1], r1);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[u][i] += r0[i] + r1[i];
            }
        }
        if (c_ok) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (tb + u < tl1)
                    st_row<false>(reinterpret_cast<uint4*>(dx + (size_t)(t_begin + tb + u) * M + c), Unit<bf16_t>::from_float(acc[u]));
        }
    }
}

// ---- gate backward ------------------------------------------------------------
//
// part[s][d][e] = sum over the tokens of chunk s of x[t,d] * dL[t,e] for float32 storage, on
// v_mfma_f32_32x32x2_f32 (float operands, float accumulation): the tokens are the reduction dimension, lane l
// holds column l%32 of x (or expert l%32 of dL) at token l/32 of two, so both operands come straight from memory,
// 128 bytes of a token row per half-wavefront.  A wavefront owns 32 columns, all experts and a chunk of tokens;
// thirty-two tokens (sixteen beyond 32 experts) are requested while as many before are multiplied.  Bound by latency at small sizes, by HIP
// events with dL and reduction: 256 tokens x 64 columns x 4 experts 16.5 us, 30.6 as float FMAs with eight columns
// per thread (eight threads of 256 had columns); 1024 x 512 x 8: 25 against 28.
typedef float gate_f32x16 __attribute__((ext_vector_type(16)));
template <int EB>                    // expert blocks of 32: E <= 32*EB
__global__ __launch_bounds__(PERM_THREADS) void gate_dwg_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ dL, float* __restrict__ part,
    long long part_stride, int p0, int t_count, int M, int E, int S, int TC) {
    const int t_begin = (p0 + (int)blockIdx.z) * t_count;
    part += blockIdx.z * part_stride;
    constexpr int U = EB == 1 ? 16 : 8;           // matrix instructions of two tokens requested together
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int ncb = (M + 31) / 32;
    const int w = blockIdx.x * PERM_WAVES + (threadIdx.x >> 6);
    const int cb = w % ncb, s = w / ncb;
    if (s >= S) return;
    const int t0 = s * TC, t1 = min(t0 + TC, t_count);
    const int c = cb * 32 + r;
    const float* xcol = x + (size_t)t_begin * M + min(c, M - 1);
    const float* dcol = dL + (size_t)t_begin * E;
    struct Blk { float x[U], d[U][EB]; };
    // tokens past the chunk contribute zeros in both operands (the last token's row instead, times zero, would turn
    // its infinities into NaN); experts past the last have result rows of their own, which are not stored
    auto request = [&](Blk& q, int tb) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = tb + 2 * u + h, tc = min(t, t1 - 1);
            const float xv = xcol[(size_t)tc * M];
            q.x[u] = t < t1 ? xv : 0.0f;
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) {
                const int e = 32 * eb + r;
                const float v = dcol[(size_t)tc * E + min(e, E - 1)];
                q.d[u][eb] = (t < t1 && e < E) ? v : 0.0f;
            }
        }
    };
    gate_f32x16 acc[EB];
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[eb][q] = 0.0f;
    auto use = [&](const Blk& q) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
                acc[eb] = __builtin_amdgcn_mfma_f32_32x32x2f32(q.d[u][eb], q.x[u], acc[eb], 0, 0, 0);
    };
    Blk ka, kb;
    request(ka, t0);
    for (int tb = t0; tb < t1; tb += 4 * U) {
        // (the barriers keep the instruction scheduler from sinking the requests to their uses)
        request(kb, tb + 2 * U);
        __builtin_amdgcn_sched_barrier(0);
        use(ka);
        __builtin_amdgcn_sched_barrier(0);
        request(ka, tb + 4 * U);
        __builtin_amdgcn_sched_barrier(0);
        use(kb);                                  // (zeros where the chunk has ended)
        __builtin_amdgcn_sched_barrier(0);
    }
    // lane (r, h) holds column r and experts 8*(q/4) + 4*h + q%4 of every block
    if (c >= M) return;
    float* out = part + ((size_t)s * M + c) * E;
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e0 = 32 * eb + 8 * g + 4 * h;
            if ((E & 3) == 0) {
                if (e0 < E)
                    *reinterpret_cast<float4*>(out + e0) =
                        make_float4(acc[eb][4 * g], acc[eb][4 * g + 1], acc[eb][4 * g + 2], acc[eb][4 * g + 3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e0 + i < E) out[e0 + i] = acc[eb][4 * g + i];
            }
        }
}

__global__ __launch_bounds__(PERM_THREADS) void gate_dl_kernel(GateDlArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[GATE_DL_LDS];
    gate_dl(a, blockIdx.x, smem);
}

// part[s][d][e] = sum over the tokens of chunk s of x[t,d] * dL[t,e] on the matrix cores
// (bfloat16 storage).  The tokens are the reduction dimension of v_mfma_f32_32x32x16_bf16, and
// both operands want eight consecutive tokens in a lane: dL comes transposed from the kernel
// above; of x a lane reads one dword (two neighbouring columns) from each of eight token rows
// - every such read covers whole 128-byte lines of two rows - and splits them into the operand
// of the even and of the odd columns.  A wavefront owns 64 columns and a chunk of TC tokens;
// the first operand holds 32 columns of dL^T: sixteen experts' hi terms and their lo terms, so that
// hi and lo products land in accumulator registers q and q + 8 of the same lane.
// (The kernel is written for CPL = 2, 4 or 8 columns per lane; wider reads with fewer, fatter
// wavefronts measured no faster - 26-29 us for gate backward of 16384 x 2048 in every shape - and
// need more partial sums, so two it is.)
constexpr int DWG_CPL = 2;
typedef __bf16 gate_bf16x8 __attribute__((ext_vector_type(8)));
template <int W> struct GateWords;            // W dwords of a token row
template <> struct GateWords<1> { typedef unsigned type; static __device__ __forceinline__ unsigned word(const unsigned& v, int) { return v; } };
template <> struct GateWords<2> { typedef uint2 type; static __device__ __forceinline__ unsigned word(const uint2& v, int i) { return i == 0 ? v.x : v.y; } };
template <> struct GateWords<4> { typedef uint4 type; static __device__ __forceinline__ unsigned word(const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; } };
template <int EB, int CPL>           // expert blocks of sixteen: E <= 16*EB; columns per lane
__global__ __launch_bounds__(PERM_THREADS) void gate_dwg_mfma_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ dLt, long long dLt_stride, float* __restrict__ part,
    long long part_stride, int p0, int t_count, int tp_pad, int M, int E, int S, int TC) {
    const int t_begin = (p0 + (int)blockIdx.z) * t_count;
    dLt += blockIdx.z * dLt_stride;
    part += blockIdx.z * part_stride;
    constexpr int U = (EB * CPL <= 4) ? 4 : 2;      // MFMA steps of 16 tokens requested together
    constexpr int BT = 16 * U;
    constexpr int W = CPL / 2;
    typedef typename GateWords<W>::type row_t;
    const int lane = threadIdx.x & 63, r = lane & 31, g = lane >> 5;
    const int ncb = (M + 32 * CPL - 1) / (32 * CPL);
    const int w = blockIdx.x * PERM_WAVES + (threadIdx.x >> 6);
    const int cb = w % ncb, s = w / ncb;
    if (s >= S) return;
    const int t0 = s * TC, t1 = min(t0 + TC, tp_pad);
    const int c = cb * 32 * CPL + CPL * r;
    const row_t* xcol = reinterpret_cast<const row_t*>(x + (size_t)t_begin * M + min(c, M - CPL));
    const size_t row_units = (size_t)(M / CPL);
    struct Blk { row_t xa[U][8]; uint4 b[U][EB]; };
    // tokens past the partition are clamped to its last one (their dL is zero); a block past the
    // chunk is requested from the last block of the buffer and never used
    auto request = [&](Blk& q, int tb) {
        tb = min(tb, tp_pad - BT);
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                q.xa[u][j] = xcol[(size_t)min(tb + 16 * u + 8 * g + j, t_count - 1) * row_units];
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
                q.b[u][eb] = *reinterpret_cast<const uint4*>(dLt + ((size_t)(eb * 32 + r) * tp_pad + tb + 16 * u + 8 * g));
        }
    };
    gate_f32x16 acc[CPL][EB];
#pragma unroll
    for (int p = 0; p < CPL; ++p)
#pragma unroll
        for (int eb = 0; eb < EB; ++eb)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[p][eb][q] = 0.0f;
    auto use = [&](const Blk& q) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int p = 0; p < CPL; ++p) {
                // column p of the lane over its eight tokens: the low or the high halves of word p/2
                unsigned o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned a = GateWords<W>::word(q.xa[u][2 * i], p >> 1), b2 = GateWords<W>::word(q.xa[u][2 * i + 1], p >> 1);
                    o[i] = (p & 1) ? ((a >> 16) | (b2 & 0xffff0000u)) : ((a & 0xffffu) | (b2 << 16));
                }
                const gate_bf16x8 x8 = __builtin_bit_cast(gate_bf16x8, make_uint4(o[0], o[1], o[2], o[3]));
#pragma unroll
                for (int eb = 0; eb < EB; ++eb)
                    acc[p][eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(gate_bf16x8, q.b[u][eb]), x8,
                                                                         acc[p][eb], 0, 0, 0);
            }
    };
    Blk ka, kb;
    request(ka, t0);
    for (int tb = t0; tb < t1; tb += 2 * BT) {
        // (the barriers keep the instruction scheduler from sinking the requests to their uses)
        request(kb, tb + BT);
        __builtin_amdgcn_sched_barrier(0);
        use(ka);
        __builtin_amdgcn_sched_barrier(0);
        request(ka, tb + 2 * BT);
        __builtin_amdgcn_sched_barrier(0);
        if (tb + BT < t1) use(kb);
        __builtin_amdgcn_sched_barrier(0);
    }
    // Accumulator register q of lane (r, g) belongs to column r of the x operand and to row
    // 8*(q/4) + 4*g + q%4 of dL^T: rows 0-15 are the hi terms of sixteen experts, rows 16-31 their lo terms.
    if (c >= M) return;
#pragma unroll
    for (int p = 0; p < CPL; ++p) {
        float* out = part + ((size_t)s * M + c + p) * E;
#pragma unroll
        for (int eb = 0; eb < EB; ++eb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int e0 = 16 * eb + 8 * h + 4 * g;
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[p][eb][4 * h + i] + acc[p][eb][4 * h + i + 8];
                if ((E & 3) == 0) {
                    if (e0 < E) *reinterpret_cast<float4*>(out + e0) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (e0 + i < E) out[e0 + i] = v[i];
                }
            }
    }
}

__global__ __launch_bounds__(256) void gate_dwg_reduce_kernel(GateSums g) {
    __shared__ float red[256];
    gate_dwg_reduce<256>(g, blockIdx.x, red);
}

// Whether a plain dispatch runs in straight-line code.  One store on its way per wavefront is the faster one where many
// wavefronts write: their reads and writes come in longer runs.  It is slower where few wavefronts have to hide it, and
// for rows of several pieces (of 4 KB) with few choices.  us, masks / straight: 16 384 tokens x 512 bfloat16, two choices 11.2 / 12.4,
// 8192 x 2048 16.7 / 19.7, three 21.3 / 25.2, 2000 x 1024 4.3 / 4.2, 1000 x 776, eight 6.6 / 5.4; float32, 1000 x 776, six 8.3 / 6.5,
// 16 384 x 2048, two 88 / 81, 4096 x 2048, six 40 / 52.  (With more than four choices also rows of about 1 KB: 16 384 x 512 bfloat16,
// eight 35 / 30.)
static bool dispatch_straight(int row_bytes, int waves, int k) {
    const int units = row_bytes / 16;
    return (units > 64 && waves <= 2048) || (units > 256 && k <= 2) || (units >= 64 && units <= 96 && k > 4);
}
template <typename T, int KM, bool DW, bool COMB>
static void launch_dispatch_k(const RowArgs& a, dim3 grid, hipStream_t s) {
    // (with the rows of T_DO: straight-line code for more than two choices and rows of more than 1 KB; dots, masks / straight, 8192 x 2048
    // float32, eight 277 / 224, 1000 x 776, five 12.7 / 10.2, 16 384 x 256 bfloat16, five 21.6 / 27.5)
    constexpr bool plain = !DW && !COMB;
    const int row_bytes = a.M * (int)sizeof(T);
    if (plain ? dispatch_straight(row_bytes, a.Tp * (int)(grid.y * grid.z), a.k) : KM > 2 && row_bytes > 1024) {
        if constexpr (plain || KM > 2) hipLaunchKernelGGL((dispatch_kernel<T, KM, DW, COMB, true>), grid, dim3(PERM_THREADS), 0, s, a);
    } else {
        hipLaunchKernelGGL((dispatch_kernel<T, KM, DW, COMB, false>), grid, dim3(PERM_THREADS), 0, s, a);
    }
}
template <typename T, bool DW, bool COMB>
static moe_status launch_dispatch(const RowArgs& a, int sources, int np, hipStream_t s) {
    const dim3 grid((a.Tp + PERM_WAVES - 1) / PERM_WAVES, sources, np);
    if (a.k == 1) launch_dispatch_k<T, 1, DW, COMB>(a, grid, s);
    else if (a.k == 2) launch_dispatch_k<T, 2, DW, COMB>(a, grid, s);
    else if (a.k <= 4) launch_dispatch_k<T, 4, DW, COMB>(a, grid, s);
    else launch_dispatch_k<T, 8, DW, COMB>(a, grid, s);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}
template <typename T>
static moe_status dispatch_t(const RowArgs& a, int sources, int np, hipStream_t s) {
    if (a.y && a.dw) return launch_dispatch<T, true, true>(a, sources, np, s);
    if (a.y) return launch_dispatch<T, false, true>(a, sources, np, s);
    if (a.dw) return launch_dispatch<T, true, false>(a, sources, np, s);
    return launch_dispatch<T, false, false>(a, sources, np, s);
}

moe_status dispatch_rows(const Dims& d, int p0, int np, const RowMove* moves, int n_moves, const int* slot,
                         const void* DO, long long DO_stride, float* dw, const float* w, void* y, hipStream_t s) {
    RowArgs a = {};
    for (int i = 0; i < n_moves; ++i) { a.src[i] = moves[i].src; a.dst[i] = (char*)moves[i].dst; a.dst_stride[i] = moves[i].stride; }
    a.rows = (const char*)DO; a.rows_stride = DO_stride;
    a.slot = slot; a.w = w; a.dw = dw; a.y = y;
    a.p0 = p0; a.Tp = d.Tp; a.M = d.M; a.k = d.k;
    {
        ProfScope ps(PK_DISPATCH, s, n_moves * np, y ? PK_COMBINE : -1, np);
        MOE_TRY(d.dtype == MOE_F32 ? dispatch_t<float>(a, n_moves, np, s) : dispatch_t<bf16_t>(a, n_moves, np, s));
    }
    count_launch(LC_PERMUTE, (n_moves + (y ? 1 : 0)) * np);
    return MOE_OK;
}

moe_status combine_rows(const Dims& d, int p0, int np, const void* DO, long long DO_stride, const int* slot, const float* w,
                        void* y, hipStream_t s) {
    RowArgs a = {};
    a.rows = (const char*)DO; a.rows_stride = DO_stride;
    a.slot = slot; a.w = w; a.y = y;
    a.p0 = p0; a.Tp = d.Tp; a.M = d.M; a.k = d.k;
    const dim3 grid((d.Tp + PERM_WAVES - 1) / PERM_WAVES, 1, np);
    {
        ProfScope ps(PK_COMBINE, s, np);
        if (d.dtype == MOE_F32) hipLaunchKernelGGL((combine_kernel<float>), grid, dim3(PERM_THREADS), 0, s, a);
        else hipLaunchKernelGGL((combine_kernel<bf16_t>), grid, dim3(PERM_THREADS), 0, s, a);
    }
    count_launch(LC_PERMUTE, np);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

moe_status dispatch_bwd_rows(const Dims& d, int p0, int np, const void* dDI, long long dDI_stride, const int* slot,
                             const float* dL, const void* Wg, void* dx, const GateSums* sums, hipStream_t s) {
    const bool bf16 = d.dtype == MOE_BF16;
    const int cols = bf16 ? DXB_CT * 8 : DXF_COLS;
    const int slices = (d.M + cols - 1) / cols;
    // tokens per wavefront: as many as leave every compute unit a workgroup or two
    const int fit = (int)((long long)d.Tp * np * slices / (512 * DXB_TG)) / 4 * 4;
    const int tok = fit < 4 ? 4 : fit > DXB_TOK ? DXB_TOK : fit;
    DispatchBwdArgs a = {};
    a.dDI = dDI; a.dDI_stride = dDI_stride;
    a.slot = slot; a.dL = dL; a.Wg = Wg; a.dx = dx;
    a.p0 = p0; a.Tp = d.Tp; a.tok = tok; a.M = d.M; a.E = d.E; a.k = d.k;
    a.token_rows = (d.Tp + tok * DXB_TG - 1) / (tok * DXB_TG);
    int sum_rows = 0;
    if (sums) {
        a.sums = *sums;
        const int blocks = (sums->ME + DXB_THREADS / 8 - 1) / (DXB_THREADS / 8);
        sum_rows = (blocks + slices * np - 1) / (slices * np);
    }
    const dim3 grid(slices, a.token_rows + sum_rows, np);
    ProfScope ps(PK_DISPATCH_BWD, s, np);
#define LAUNCH_DXB(KERN, T_, LDS) do { \
        int lds = (LDS); \
        if (lds < DXB_THREADS * (int)sizeof(float)) lds = DXB_THREADS * (int)sizeof(float);     /* (the sums') */ \
        static int attr_bytes = 0;                  /* largest size asked for so far */ \
        if (lds > attr_bytes) { \
            HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, lds)); \
            attr_bytes = lds; \
        } \
        hipLaunchKernelGGL(KERN, grid, dim3(DXB_THREADS), lds, s, (const T_*)dDI, slot, dL, (const T_*)Wg, (T_*)dx, a); } while (0)
    if (!bf16) LAUNCH_DXB(dispatch_bwd_f32_kernel, float, DXF_PITCH * d.E * (int)sizeof(float));
    else if (d.E <= 4) LAUNCH_DXB((dispatch_bwd_mfma_kernel<1>), bf16_t, DXB_CT * (64 * 1 + 16));
    else if (d.E <= 8) LAUNCH_DXB((dispatch_bwd_mfma_kernel<2>), bf16_t, DXB_CT * (64 * 2 + 16));
    else if (d.E <= 16) LAUNCH_DXB((dispatch_bwd_mfma_kernel<4>), bf16_t, DXB_CT * (64 * 4 + 16));
    else if (d.E <= 32) LAUNCH_DXB((dispatch_bwd_mfma_kernel<8>), bf16_t, DXB_CT * (64 * 8 + 16) + DXB_TG * 64 * (8 + 1));
    else LAUNCH_DXB((dispatch_bwd_mfma_kernel<16>), bf16_t, DXB_CT * (64 * 16 + 16) + DXB_TG * 64 * (16 + 1));
#undef LAUNCH_DXB
    count_launch(LC_PERMUTE, np);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// Shape of the bfloat16 gate-backward: token chunks of the matrix-core kernel and the two regions of
// the scratch buffer (partial sums [S][M][E] float, then dL^T [EB*32][tp_pad] bfloat16).
struct GateMfmaPlan { int tp_pad, EB, ncb, S, TC; size_t dlt_off, bytes; };
static GateMfmaPlan gate_mfma_plan(const Dims& d) {
    GateMfmaPlan g;
    g.tp_pad = (d.Tp + DWG_TOK - 1) / DWG_TOK * DWG_TOK;
    g.EB = (d.E + 15) / 16;
    g.ncb = (d.M + 32 * DWG_CPL - 1) / (32 * DWG_CPL);
    const int blocks = g.tp_pad / 64;
    int S = 1024 / g.ncb;                     // about one wavefront per SIMD: more of them were slower
    S = S < 1 ? 1 : (S > blocks ? blocks : S);
    g.TC = (blocks + S - 1) / S * 64;
    g.S = (g.tp_pad + g.TC - 1) / g.TC;
    g.dlt_off = ((size_t)g.S * d.M * d.E * sizeof(float) + 255) / 256 * 256;
    g.bytes = g.dlt_off + (size_t)g.EB * 32 * g.tp_pad * sizeof(bf16_t);
    return g;
}

// Token chunks of the float32 gate-backward: about two wavefronts per SIMD (its loads are four bytes a lane), never
// more partial sums than the scratch buffer holds, one per DWG_TOK tokens.
struct GateF32Plan { int ncb, S, TC; };
static GateF32Plan gate_f32_plan(const Dims& d) {
    GateF32Plan g;
    g.ncb = (d.M + 31) / 32;
    const int blocks = (d.Tp + DWG_TOK - 1) / DWG_TOK;
    int S = 2048 / g.ncb;
    S = S < 1 ? 1 : (S > blocks ? blocks : S);
    g.TC = (blocks + S - 1) / S * DWG_TOK;
    g.S = (d.Tp + g.TC - 1) / g.TC;
    return g;
}

size_t gate_part_bytes(const Dims& d) {
    const int S = d.dtype == MOE_BF16 ? gate_mfma_plan(d).S : gate_f32_plan(d).S;
    return (size_t)S * d.M * d.E * sizeof(float);
}
size_t gate_dlt_bytes(const Dims& d) {
    if (d.dtype != MOE_BF16) return 0;
    const GateMfmaPlan g = gate_mfma_plan(d);
    return (size_t)g.EB * 32 * g.tp_pad * sizeof(bf16_t);
}
size_t gate_dlt_offset(const Dims& d) { return d.dtype == MOE_BF16 ? gate_mfma_plan(d).dlt_off : 0; }

GateDlArgs gate_dl_args(const Dims& d, int p0, int np, const float* logits, const int* idx, const int* slot, const float* dw,
                        const float* dw_part, long long dw_part_stride, int parts, float* dL, void* dLt) {
    GateDlArgs a = {};
    a.logits = logits; a.topk_idx = idx; a.slot = slot; a.dw = dw;
    a.dw_part = dw_part; a.dw_part_stride = dw_part_stride; a.parts = parts;
    a.dL = dL;
    if (d.dtype == MOE_BF16) {
        a.dLt = (bf16_t*)dLt;
        a.dLt_stride = (long long)(gate_dlt_bytes(d) / sizeof(bf16_t));
        a.tp_pad = gate_mfma_plan(d).tp_pad;
    }
    a.p0 = p0; a.Tp = d.Tp; a.E = d.E; a.k = d.k; a.renorm = d.renorm;
    a.per_part = (d.Tp + DWG_TOK - 1) / DWG_TOK;
    a.blocks = a.per_part * np;
    return a;
}

moe_status gate_bwd_rows(const Dims& d, int np, const void* x, const GateDlArgs& dl, bool dl_done, float* dWg,
                         float* part, long long part_stride, hipStream_t s, GateSums* sums) {
    const int p0 = dl.p0;
    ProfScope ps(PK_GATE_BWD, s, np);
    GateSums t = {};
    t.part = part; t.part_stride = part_stride; t.dWg = dWg;
    t.ME = d.M * d.E; t.np = np; t.store = d.overwrite && p0 == 0;
    if (!dl_done) {
        hipLaunchKernelGGL(gate_dl_kernel, dim3(dl.blocks), dim3(PERM_THREADS), 0, s, dl);
        MOE_CHECK_LAUNCH();
    }
    if (d.dtype == MOE_BF16) {
        const GateMfmaPlan g = gate_mfma_plan(d);
        const dim3 grid((g.ncb * g.S + PERM_WAVES - 1) / PERM_WAVES, 1, np);
#define LAUNCH_DWG(EB) hipLaunchKernelGGL((gate_dwg_mfma_kernel<EB, DWG_CPL>), grid, dim3(PERM_THREADS), 0, s, (const bf16_t*)x, \
                           (const bf16_t*)dl.dLt, dl.dLt_stride, part, part_stride, p0, d.Tp, g.tp_pad, d.M, d.E, g.S, g.TC)
        // (a kernel for every number of blocks: it reads all of its own of dL^T, which the plan has room for exactly so many of)
        switch (g.EB) {
            case 1: LAUNCH_DWG(1); break;
            case 2: LAUNCH_DWG(2); break;
            case 3: LAUNCH_DWG(3); break;
            case 4: LAUNCH_DWG(4); break;
            default: return MOE_ERR_UNSUPPORTED;
        }
#undef LAUNCH_DWG
        t.nblk = g.S;
    } else {
        const GateF32Plan g = gate_f32_plan(d);
        const dim3 grid((g.ncb * g.S + PERM_WAVES - 1) / PERM_WAVES, 1, np);
        if (d.E <= 32)
            hipLaunchKernelGGL((gate_dwg_f32_kernel<1>), grid, dim3(PERM_THREADS), 0, s, (const float*)x, (const float*)dl.dL, part,
                               part_stride, p0, d.Tp, d.M, d.E, g.S, g.TC);
        else
            hipLaunchKernelGGL((gate_dwg_f32_kernel<2>), grid, dim3(PERM_THREADS), 0, s, (const float*)x, (const float*)dl.dL, part,
                               part_stride, p0, d.Tp, d.M, d.E, g.S, g.TC);
        t.nblk = g.S;
    }
    MOE_CHECK_LAUNCH();
    count_launch(LC_OTHER, 3 * np);
    if (sums) { *sums = t; return MOE_OK; }
    hipLaunchKernelGGL(gate_dwg_reduce_kernel, dim3((t.ME + 31) / 32), dim3(256), 0, s, t);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

}  // namespace moe

using namespace moe;

extern "C" moe_status moe_dispatch(const moe_config* cfg, int32_t part, const void* src, const int32_t* slot,
                                   void* DI, const void* dO_saved, float* dw, void* stream) {
    Dims d;
    MOE_TRY(make_dims(cfg, &d));
    MOE_TRY(check_part(d, part));
    if (!src || !slot || !DI) return MOE_ERR_NULL;
    const RowMove m = {src, DI, 0};
    const bool with_dw = dO_saved && dw;
    return dispatch_rows(d, part, 1, &m, 1, slot, with_dw ? dO_saved : nullptr, 0, with_dw ? dw : nullptr, nullptr, nullptr,
                         (hipStream_t)stream);
}

extern "C" moe_status moe_combine(const moe_config* cfg, int32_t part, const void* DO, const int32_t* slot,
                                  const float* topk_w, void* y, void* stream) {
    Dims d;
    MOE_TRY(make_dims(cfg, &d));
    MOE_TRY(check_part(d, part));
    if (!DO || !slot || !topk_w || !y) return MOE_ERR_NULL;
    return combine_rows(d, part, 1, DO, 0, slot, topk_w, y, (hipStream_t)stream);
}

extern "C" moe_status moe_dispatch_bwd(const moe_config* cfg, int32_t part, const void* dDI, const int32_t* slot,
                                       const float* dL, const void* Wg, void* dx, void* stream) {
    Dims d;
    MOE_TRY(make_dims(cfg, &d));
    MOE_TRY(check_part(d, part));
    if (!dDI || !slot || !dL || !Wg || !dx) return MOE_ERR_NULL;
    return dispatch_bwd_rows(d, part, 1, dDI, 0, slot, dL, Wg, dx, nullptr, (hipStream_t)stream);
}

extern "C" moe_status moe_gate_scratch_bytes(const moe_config* cfg, size_t* bytes) {
    Dims d;
    MOE_TRY(make_dims(cfg, &d));
    if (!bytes) return MOE_ERR_NULL;
    *bytes = d.dtype == MOE_BF16 ? gate_mfma_plan(d).bytes
                                 : (size_t)((d.Tp + DWG_TOK - 1) / DWG_TOK) * d.M * d.E * sizeof(float);
    return MOE_OK;
}

extern "C" moe_status moe_gate_bwd(const moe_config* cfg, int32_t part, const void* x, const float* logits,
                                   const int32_t* topk_idx, const int32_t* slot, const float* dw,
                                   const float* dw_part, float* dL, float* dWg, void* scratch, void* stream) {
    Dims d;
    MOE_TRY(make_dims(cfg, &d));
    MOE_TRY(check_part(d, part));
    if (!x || !logits || !topk_idx || !slot || !dL || !dWg || !scratch) return MOE_ERR_NULL;
    if (!dw && !dw_part) return MOE_ERR_NULL;
    int parts = 0;
    MOE_TRY(moe_dw_parts(cfg, &parts));
    const GateDlArgs dl = gate_dl_args(d, part, 1, logits, topk_idx, slot, dw, dw_part, 0, parts, dL, (char*)scratch + gate_dlt_offset(d));
    return gate_bwd_rows(d, 1, x, dl, false, dWg, (float*)scratch, 0, (hipStream_t)stream, nullptr);
}
