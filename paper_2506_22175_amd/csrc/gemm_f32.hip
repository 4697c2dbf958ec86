// float32 grouped GEMM for the expert FFN (the two linear layers of an expert,
// Section II-B2, and their gradients) on the float32 matrix instructions
// (v_mfma_f32_32x32x2_f32: float operands, float accumulation; this path exists for
// the float32 workload, whose tolerance rules out reduced precision inputs).
//
// One workgroup computes a 64 x 64 tile of one expert with four wavefronts of 32 x 32.
// The matrix instruction takes 64 cycles for 32 x 32 x 2, so even this tile asks little
// of LDS (32 of its 128 bytes per cycle) and of L2 (38 bytes per ns and CU at the full
// rate); what counts is that small layers have enough tiles for the chip and that a
// tile's K loop never waits: operands travel global -> LDS by DMA through a ring of three
// 32-k stages, and three workgroups fit a CU (rings of two and of four stages measured the
// same).  2048 rows x 512 x 2048 over 8 experts (27 us at the rate of the instruction), by
// HIP events: first layer 57 us, second layer 79, GeLU-backward 61, input gradient 80,
// weight gradients 52 each (the 64 x 64 float-FMA tiles before: 107, 341, 106, 307, 113).
// The two with N = 512 have 288 tiles for 256 CUs.
#include "common.h"
#include "epilogue.h"
#include "gate_bwd.h"

namespace moe {

constexpr int F_BM = 64, F_BN = 64, F_BK = 32, F_NS = 3, F_THREADS = 256;
constexpr int F_TILE = F_BM * F_BK * 4;            // bytes of one operand's stage
typedef float f_acc_t __attribute__((ext_vector_type(16)));

// What a lane reads when its piece of a stage lies outside the operand.
static __device__ __align__(16) float f_zeros[4];

// 16 bytes per lane from the lane's own address to LDS at lds_off + 16*lane (lds_off wave-uniform).
// Assembly, so that the compiler does not wait for it at the next LDS read; the loop waits with
// s_waitcnt vmcnt(N) itself.
__device__ __forceinline__ void f_load_to_lds(const float* p, unsigned lds_off) {
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, off"
                 : : "s"(lds_off), "v"(p) : "memory");
}
template <int N> __device__ __forceinline__ void f_wait_loads() {
    // (lgkmcnt: this wave's own LDS reads are through too)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(N) : "memory");
}

// One operand of the tile: 64 rows (m or n) x 32 k per stage.
//   KC: k is contiguous in memory.  LDS [row][32 k], 16-byte chunk c of a row at c ^ (row/2 % 8): the sixteen
//       rows of a quarter of a 16-byte read cover all banks.
//   NC: the rows are contiguous in memory ([k][n]).  LDS [k][64 n]; k rows 4..7 of every eight have their
//       halves exchanged, so that the two half-wavefronts of a 4-byte read use different banks.
// A wavefront fills two of the eight 1 KB pieces of a stage.
template <bool KC> struct FOperand {
    const float* p[2];          // this lane's piece in the stage requested next
    int k[2];                   // its first k; at or beyond K it reads zeros
    long long step;             // elements from one stage to the next
    int K;
    __device__ __forceinline__ void init(const float* P, long long ld, int row0, int row_limit, int K_, int wid, int lane,
                                         const int* rows) {
        K = K_;
        step = KC ? F_BK : F_BK * ld;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int q = wid * 2 + j;
            bool ok;
            if (KC) {
                const int row = q * 8 + (lane >> 3);
                const int c = (lane & 7) ^ ((row >> 1) & 7);
                ok = row0 + row < row_limit;
                const long long src = !ok ? 0 : rows ? rows[row0 + row] : row0 + row;
                k[j] = c * 4;
                p[j] = P + src * ld + c * 4;
            } else {
                const int kr = q * 4 + (lane >> 4);
                const int u = (lane & 15) ^ (((kr >> 2) & 1) << 3);
                ok = row0 + u * 4 < row_limit;
                k[j] = kr;
                p[j] = P + (long long)kr * ld + row0 + u * 4;
            }
            if (!ok) k[j] = 0x40000000;            // never below K
        }
    }
    __device__ __forceinline__ void request(unsigned lds, int wid) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            f_load_to_lds(k[j] < K ? p[j] : f_zeros, lds + (wid * 2 + j) * 1024);
            p[j] += step;
            k[j] += F_BK;
        }
    }
    // operands of four matrix instructions: row rb + lane%32, k = 8*kk + 4*(lane/32) + 0..3
    static __device__ __forceinline__ void read(const char* tile, int rb, int kk, int lane, float* o) {
        const int row = rb + (lane & 31), h = lane >> 5;
        if (KC) {
            const float4 v = *reinterpret_cast<const float4*>(tile + row * 128 + (((2 * kk + h) ^ ((row >> 1) & 7)) << 4));
            o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
        } else {
            const char* at = tile + (8 * kk + 4 * h) * 256 + ((row * 4) ^ (h << 7));
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = *reinterpret_cast<const float*>(at + j * 256);
        }
    }
};

// Tile (tm, tn) of expert number v
template <int LAY, int EPI>
__device__ __forceinline__ void gemm_f32_one(const GemmArgs& g, int v, int tm, int tn, char* smem) {
    const ExpertOf x = LAY == GEMM_TN ? ExpertOf{v, 0} : expert_of(g, v);
    const int e = x.e, er = x.q * g.E + e;
    const int rows = g.counts[er];
    const int Mdim = LAY == GEMM_TN ? g.Mo : rows, Kdim = LAY == GEMM_TN ? rows : g.K;
    const int m0 = tm * F_BM, n0 = tn * F_BN;
    if (m0 >= Mdim) return;
    if (EPI == EPI_ACCUM_F32 && Kdim <= 0) return;            // nothing to add
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid >> 1, wn = wid & 1;
    const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) const char*)smem;

    FOperand<LAY != GEMM_TN> A;
    FOperand<LAY == GEMM_NT> B;
    const bool gathered = LAY != GEMM_TN && g.a_rows;         // gathered rows: one matrix for all experts
    A.init((const float*)g.A + (gathered ? 0 : (size_t)e * g.a_estride + (LAY == GEMM_TN ? 0 : x.q * g.a_pstride)), g.lda, m0, Mdim, Kdim, wid, lane,
           gathered ? g.a_rows + (size_t)er * g.Cp : nullptr);
    B.init((const float*)g.B + (size_t)e * g.b_estride, g.ldb, n0, g.N, Kdim, wid, lane, nullptr);
    const int KT = (Kdim + F_BK - 1) / F_BK;

    f_acc_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    // stages 0 .. NS-2 on their way; past the last k they are zeros that nobody reads
#pragma unroll
    for (int s = 0; s < F_NS - 1; ++s) {
        A.request(lds0 + s * 2 * F_TILE, wid);
        B.request(lds0 + s * 2 * F_TILE + F_TILE, wid);
    }
    for (int kt = 0; kt < KT; ++kt) {
        f_wait_loads<4 * (F_NS - 2)>();                       // this wave's part of stage kt is in
        __builtin_amdgcn_s_barrier();                         // everybody's is, and nobody reads stage kt-1 any more
        asm volatile("" ::: "memory");
        const unsigned ahead = lds0 + ((kt + F_NS - 1) % F_NS) * 2 * F_TILE;
        A.request(ahead, wid);
        B.request(ahead + F_TILE, wid);
        const char* as = smem + (kt % F_NS) * 2 * F_TILE;
        const char* bs = as + F_TILE;
        float a[F_BK / 8][4], b[F_BK / 8][4];
#pragma unroll
        for (int kk = 0; kk < F_BK / 8; ++kk) {
            A.read(as, wm * 32, kk, lane, a[kk]);
            B.read(bs, wn * 32, kk, lane, b[kk]);
        }
#pragma unroll
        for (int kk = 0; kk < F_BK / 8; ++kk)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[kk][j], a[kk][j], acc, 0, 0, 0);
    }
    f_wait_loads<0>();                                        // nothing is in flight into LDS any more

    // With B as the first operand a lane holds row lane%32 of its wave's block and four consecutive
    // columns 8*q + 4*(lane/32) per register group q.
    EpiCtx<float> c;
    c.ldc = g.ldc; c.ldz = g.ldz;
    c.C = EPI == EPI_SCATTER ? (float*)g.C : (float*)g.C + (size_t)e * g.c_estride + (LAY == GEMM_TN ? 0 : x.q * g.c_pstride);
    c.Cf = c.C;
    c.out_rows = g.c_rows ? g.c_rows + (size_t)er * g.Cp : nullptr;
    c.Z = g.Z ? (float*)g.Z + (size_t)e * g.Cp * g.ldz + x.q * g.z_pstride : nullptr;
    c.w = g.slot_w ? g.slot_w + (size_t)er * g.Cp : nullptr;
    const int r = m0 + wm * 32 + (lane & 31);
    float dot = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = n0 + wn * 32 + 8 * q + 4 * (lane >> 5);
        const float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        if (r < Mdim && n < g.N) dot += epilogue4<float, EPI>(c, r, n, v);
    }
    if (EPI == EPI_DGELU && g.dw_part) {
        // a row's 64 columns: two half-wavefronts of each of the two waves that share its rows
        dot += __shfl_xor(dot, 32, 64);
        float* sdot = reinterpret_cast<float*>(smem);
        __syncthreads();                                      // the ring is no longer read
        if (wn == 1 && lane < 32) sdot[wm * 32 + lane] = dot;
        __syncthreads();
        if (wn == 0 && lane < 32 && r < Mdim) g.dw_part[x.q * g.dw_pstride + ((size_t)e * g.Cp + r) * g.dw_parts + tn] = dot + sdot[wm * 32 + lane];
    }
}

template <int LAY, int EPI>
__global__ __launch_bounds__(F_THREADS, 2) void gemm_f32_kernel(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char smem[F_NS * 2 * F_TILE];
    gemm_f32_one<LAY, EPI>(g, blockIdx.z, blockIdx.y, blockIdx.x, smem);
}

// The input gradient (tiles_dm = 0: not there) and the two weight gradients, which do not depend on each other, in one
// launch: the tiles of the first, which take longest, fill up with those of the others instead of leaving the chip
// half idle in a last round.
struct F32BackwardArgs {
    GemmArgs d, w[2];
    int tiles_dm, tiles_dn, tiles_wm[2], tiles_wn[2];
    int d_from;                          // first block of the input gradient: 0, or behind the weight gradients'
    GateDlArgs gate;                     // in the last blocks (blocks = 0: not there)
};
template <int EPI>
__global__ __launch_bounds__(F_THREADS, 2) void gemm_f32_backward_kernel(F32BackwardArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[F_NS * 2 * F_TILE];
    int b = blockIdx.x;
    const int nd = launch_experts(a.d) * a.tiles_dm * a.tiles_dn;
    if (b >= a.d_from) {
        if (b < a.d_from + nd) {
            b -= a.d_from;
            const int per = a.tiles_dm * a.tiles_dn, e = b / per, r = b - e * per, tm = r / a.tiles_dn;
            gemm_f32_one<GEMM_NT, EPI_STORE>(a.d, e, tm, r - tm * a.tiles_dn, smem);
            return;
        }
        b -= nd;
    }
    const int n2 = a.w[0].E * a.tiles_wm[0] * a.tiles_wn[0], q = b >= n2 ? 1 : 0;
    b -= q * n2;
    if (q == 1 && b >= a.w[1].E * a.tiles_wm[1] * a.tiles_wn[1]) {
        gate_dl(a.gate, b - a.w[1].E * a.tiles_wm[1] * a.tiles_wn[1], smem);
        return;
    }
    const int tn = a.tiles_wn[q], per = a.tiles_wm[q] * tn, e = b / per, r = b - e * per, tm = r / tn;
    gemm_f32_one<GEMM_TN, EPI>(a.w[q], e, tm, r - tm * tn, smem);
}

void gemm_f32_tile(int* rows, int* cols) { *rows = F_BM; *cols = F_BN; }

int gemm_f32_dw_parts(int H) { return (H + F_BN - 1) / F_BN; }

template <int LAY, int EPI>
static moe_status launch_f32(const GemmArgs& a, hipStream_t s) {
    const int Mmax = (LAY == GEMM_TN) ? a.Mo : a.Cp;
    const int tiles_m = (Mmax + F_BM - 1) / F_BM, tiles_n = (a.N + F_BN - 1) / F_BN;
    {
        ProfScope ps(gemm_prof_kind(LAY, EPI), s, a.np > 1 ? a.np : 1);
        hipLaunchKernelGGL((gemm_f32_kernel<LAY, EPI>), dim3(tiles_n, tiles_m, launch_experts(a)), dim3(F_THREADS), 0, s, a);
    }
    count_launch(LC_GEMM, a.np > 1 ? a.np : 1);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

moe_status gemm_f32_backward(const GemmArgs* dgrad, const GemmArgs& w2, const GemmArgs& w1, GemmEpilogue epi,
                             const GateDlArgs* gate, hipStream_t s, bool* done) {
    static_assert(GATE_DL_LDS <= F_NS * 2 * F_TILE && GATE_THREADS == F_THREADS, "a block of the gate in a tile's workgroup");
    F32BackwardArgs b = {};
    b.w[0] = w2;
    b.w[1] = w1;
    auto tiles = [](int n, int t) { return (n + t - 1) / t; };
    if (dgrad) { b.d = *dgrad; b.tiles_dm = tiles(dgrad->Cp, F_BM); b.tiles_dn = tiles(dgrad->N, F_BN); }
    long long blocks = (long long)launch_experts(b.d) * b.tiles_dm * b.tiles_dn, wgrad_blocks = 0;
    for (int q = 0; q < 2; ++q) {
        b.tiles_wm[q] = tiles(b.w[q].Mo, F_BM);
        b.tiles_wn[q] = tiles(b.w[q].N, F_BN);
        wgrad_blocks += (long long)b.w[q].E * b.tiles_wm[q] * b.tiles_wn[q];
    }
    blocks += wgrad_blocks;
    // The tiles with the longer reduction first: a long one begun last is what the launch ends with (12 experts of 2454
    // rows, 152/224: 131 us with the weight gradients' tiles last, 99 with them first; 2048 rows x 5, 104/152: 52 and 47).
    const long long rows = (long long)w2.mean_rows * (w2.k_segs > 1 ? w2.k_segs : 1);
    b.d_from = dgrad && rows > dgrad->K ? (int)wgrad_blocks : 0;
    if (gate) { b.gate = *gate; blocks += gate->blocks; }
    // (one linear grid: beyond what one launch takes, the three are launched one by one)
    *done = blocks <= 0x7fffffff / F_THREADS;
    if (!*done) return MOE_OK;
    {
        ProfScope ps(PK_GEMM_WGRAD, s, 2, dgrad ? PK_GEMM_DGRAD : -1, dgrad && dgrad->np > 1 ? dgrad->np : 1);
        if (epi == EPI_STORE_F32)
            hipLaunchKernelGGL((gemm_f32_backward_kernel<EPI_STORE_F32>), dim3((unsigned)blocks), dim3(F_THREADS), 0, s, b);
        else
            hipLaunchKernelGGL((gemm_f32_backward_kernel<EPI_ACCUM_F32>), dim3((unsigned)blocks), dim3(F_THREADS), 0, s, b);
    }
    count_launch(LC_GEMM, 2 + (!dgrad ? 0 : dgrad->np > 1 ? dgrad->np : 1));
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

moe_status gemm_f32(GemmLayout lay, GemmEpilogue epi, const GemmArgs& a, hipStream_t s) {
    if (a.dw_part && a.dw_parts != gemm_f32_dw_parts(a.N)) return MOE_ERR_SHAPE;
    if (a.a_rows && (lay == GEMM_TN || a.a_row_limit <= 0)) return MOE_ERR_UNSUPPORTED;
    if (epi == EPI_SCATTER && (lay == GEMM_TN || !a.c_rows || !a.slot_w || a.c_row_limit <= 0)) return MOE_ERR_UNSUPPORTED;
    if (lay == GEMM_NN && epi == EPI_STORE) return launch_f32<GEMM_NN, EPI_STORE>(a, s);
    if (lay == GEMM_NN && epi == EPI_GELU) return launch_f32<GEMM_NN, EPI_GELU>(a, s);
    if (lay == GEMM_NN && epi == EPI_SCATTER) return launch_f32<GEMM_NN, EPI_SCATTER>(a, s);
    if (lay == GEMM_NT && epi == EPI_STORE) return launch_f32<GEMM_NT, EPI_STORE>(a, s);
    if (lay == GEMM_NT && epi == EPI_DGELU) return launch_f32<GEMM_NT, EPI_DGELU>(a, s);
    if (lay == GEMM_TN && epi == EPI_STORE_F32) return launch_f32<GEMM_TN, EPI_STORE_F32>(a, s);
    if (lay == GEMM_TN && epi == EPI_ACCUM_F32) return launch_f32<GEMM_TN, EPI_ACCUM_F32>(a, s);
    return MOE_ERR_UNSUPPORTED;
}

}  // namespace moe
