// bf16 grouped GEMM on the CDNA4 matrix cores for the expert FFN: the two linear
// layers of every local expert (Section II-B2) and their four backward GEMMs
// (Table II counts 2 forward and 4 backward GEMM units per partition, 5 with
// recomputation).  Float accumulation, in 256 x 256 tiles with v_mfma_f32_16x16x32_bf16:
// their main loops run at the chip's power limit, and of the two shapes of the instruction
// this one takes less power (all CUs, operands from registers, normally distributed: 1.95
// PFLOP/s at 1.95 GHz, 32x32x16 1.67 at 1.67 GHz).  Smaller tiles use v_mfma_f32_32x32x16_bf16
// (TileCfg::S32).
//
// One workgroup computes a BM x BN tile of one expert with WAVES_M x WAVES_N
// wavefronts, each owning (BM/WAVES_M) x (BN/WAVES_N) as 16x16 or 32x32 MFMA tiles.
//
// Operand tiles (32 or 64 K-elements deep) travel global -> LDS with
// buffer_load_dwordx4 ... lds: no staging registers, no LDS-write instructions,
// and rows beyond the valid range read as zeros in hardware (the buffer
// descriptor ends after the last valid row): no row needs a branch.
// Each lane of such a load lands at LDS base + 16*lane, so the LDS layout is
// chosen by choosing which 16 global bytes each lane fetches:
//   * an operand whose rows are K-contiguous in memory ("KC": A of NN/NT, B of
//     NT) is kept as [row][64 k] with a 16-byte-chunk XOR swizzle and read with
//     ds_read_b128 - conflict-free both ways;
//   * an operand stored [k][n] with n contiguous ("NC": B of NN, both of TN) is
//     kept as it is, with a 16-byte-unit XOR that depends on k, and read with
//     ds_read_b64_tr_b16, which hands each lane four consecutive k of one n.
// LDS is a ring of NS stages of BK K-elements each; the loads of the next NS-1
// tiles are in flight while one tile is multiplied (a CU draws about 64 KB per
// microsecond at speed and a miss in L2 takes longer than one tile's arithmetic,
// so the depth of the ring, not the hit rate, decides whether the matrix pipe
// waits).  One or two s_barriers per 64 k.
#include "common.h"
#include "epilogue.h"
#include "gate_bwd.h"
#include <type_traits>

namespace moe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;

constexpr unsigned OOB_OFFSET = 0x80000000u;
constexpr int DW_COLS = 128;         // columns per partial sum of GeLU-backward's row dots (an even number of blocks per row)

// Buffer descriptor (base, stride 0, size in bytes, raw 32-bit format) kept in SGPRs.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4i make_rsrc(const void* p, unsigned bytes) {
    // wave-uniform by construction; readfirstlane makes that visible to the compiler, which must
    // hand the descriptor to the assembly statements below in scalar registers
    const unsigned long long a = (unsigned long long)p;
    v4i d = {__builtin_amdgcn_readfirstlane((int)(unsigned)a), __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xffffu)),
             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
    return d;
}
// The descriptor of the same columns without the first rows, of `bytes` bytes together; none may be left.
__device__ __forceinline__ void drop_rows(v4i& rsrc, unsigned bytes) {
    const unsigned long long at = ((unsigned long long)(unsigned)rsrc[1] << 32 | (unsigned)rsrc[0]) + bytes;
    rsrc[0] = (int)(unsigned)at;
    rsrc[1] = (int)(unsigned)(at >> 32);
    rsrc[2] = max(rsrc[2] - (int)bytes, 0);
}
// 16 bytes per lane from the buffer straight into LDS at lds_off + 16*lane (lds_off is a
// wave-uniform LDS byte address).  Written as assembly so that the compiler's
// wait-count bookkeeping does not see an LDS store in flight: it would otherwise make
// every transposing LDS read wait for all of them (vmcnt(0)), which serialises the
// ring.  The kernel waits with explicit s_waitcnt vmcnt(N) before each barrier instead.
__device__ __forceinline__ void load_to_lds(v4i rsrc, unsigned lds_off, unsigned voff) {
    // m0 carries the LDS address of the load and nothing else in these kernels (no LDS-direct reads, no
    // relative register indexing, no message sends), so it is not saved and restored around the load
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, 0 offen lds"
                 : : "s"(lds_off), "v"(voff), "s"(rsrc) : "memory");
}
// The same in two parts for the main loops, with a matrix instruction between them (m0 has to be written one wait state
// before the load); the step along K is the load's scalar offset, which is no part of its bounds check, or in the descriptor.
// m0 is a reserved register, which a statement cannot name as written or read: that no instruction of the compiler's stands
// between the two parts is checked in the built code (tests/test_kernel_registers.py).
template <int ADD>
__device__ __forceinline__ void lds_destination(unsigned lds_off) {
    asm volatile("s_add_u32 m0, %0, %1" : : "s"(lds_off), "n"(ADD) : "memory", "scc");
}
__device__ __forceinline__ void lds_next_destination() { asm volatile("s_add_u32 m0, m0, 0x400" : : : "memory", "scc"); }
__device__ __forceinline__ void load_to_destination(v4i rsrc, unsigned voff, unsigned soff) {
    asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" : : "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ void load_to_destination(v4i rsrc, unsigned voff) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" : : "v"(voff), "s"(rsrc) : "memory");
}
// an address in a vector register moved by a wave-uniform step, here and now
__device__ __forceinline__ void move_address(unsigned& at, int by) { asm volatile("v_add_u32 %0, %1, %0" : "+v"(at) : "s"(by)); }
__device__ __forceinline__ void flip_address(unsigned& at, unsigned bits) { asm volatile("v_xor_b32 %0, %1, %0" : "+v"(at) : "s"(bits)); }
__device__ __forceinline__ unsigned lds_address(const char* p) {
    return (unsigned)(unsigned long long)(__attribute__((address_space(3))) const char*)p;
}

// ---- tile shape ------------------------------------------------------------------
// Four main loops, all hand-scheduled:
//   LOOP_PIPE32 ring of 32-k stages for both operands;
//   LOOP_W64    NN: 64-k steps with one ring per operand: the rows travel as whole 128-byte lines (units of
//               64 k), the weights in tiles of 32 k.
//   LOOP_R64    64-k steps with one ring for both operands (tiles small enough for three or more stages of 64 k);
//   LOOP_N64    256 x 256 of two K-contiguous operands: both travel as whole lines in units of 64 k, of which five fit;
//               the weights of a whole step are held in registers, so that their unit is free half a step early.
enum { LOOP_PIPE32 = 1, LOOP_W64 = 2, LOOP_R64 = 3, LOOP_N64 = 4 };
template <int BM_, int BN_, int BK_, int NS_, int WAVES_M_, int WAVES_N_, int OCC_, int LOOP_>
struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, NS = NS_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
    static constexpr int OCC = OCC_, LOOP = LOOP_;
    // Matrix instruction 32 x 32 x 16 (256 x 256: 16 x 16 x 32; two of the former add up the same products in the same order as
    // one of the latter, bit for bit in every case measured).  Smaller tiles keep it: their launches do not run at the power
    // limit, and half as many matrix instructions each hide twice as many others.  (With 16 x 16: 128 x 128 weight gradients
    // 1040 cycles a step of 32 k against 880, 64 x 128 with GeLU 1000 against 940; 9096 tokens, 160/480, n = 4: 168 us against 156.)
    static constexpr bool S32 = BM_ * BN_ < 256 * 256;
    static constexpr int WAVES = WAVES_M * WAVES_N;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    static constexpr int TM = WM / 32;                   // blocks of 32 rows of a wave: of epilogue passes, and of `active` rows
    static constexpr int RB = WM / 16, NB = WN / 16;     // its blocks of 16 rows and of 16 columns
    static constexpr int STAGE_BYTES = (BM + BN) * BK * 2;
    static constexpr int LDS_BYTES = LOOP == LOOP_W64 || LOOP == LOOP_N64 ? 160 * 1024 : NS * STAGE_BYTES;
    // columns of a wave's block that pass through the staging region at a time, and where that region starts
    static constexpr int CW = WN < 64 || (LOOP == LOOP_PIPE32 && OCC == 1) ? WN : LOOP == LOOP_R64 && OCC == 2 ? 32 : 64;
    static constexpr int SBR = (WAVES * 32 * CW * 4 + STAGE_BYTES - 1) / STAGE_BYTES;      // stages that region takes
    static constexpr int STAGING_OFF = LOOP == LOOP_W64 ? 64 * 1024 : LOOP == LOOP_N64 ? 128 * 1024 : LOOP == LOOP_R64 ? (NS - SBR) * STAGE_BYTES : 0;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS ring exceeds the CU's 160 KB");
    static_assert(BK == 32 || BK == 64, "tile depth");
    static_assert(LOOP != LOOP_PIPE32 || (BK == 32 && NS >= 3), "the hand-scheduled ring has stages of 32 k");
    static_assert((LOOP != LOOP_W64 && LOOP != LOOP_N64) || (BM == 256 && BN == 256 && BK == 64 && WAVES_M == 2 && WAVES_N == 2 && OCC == 1),
                  "the two-ring and the five-unit loop are written for four waves of 128 x 128");
    static_assert(LOOP != LOOP_R64 || (BK == 64 && NS >= 3 && SBR <= NS - 2),
                  "stages of 64 k; the epilogue stages through the last ones");
};

// ---- K-contiguous operand tile: R rows x BK k ---------------------------------------
// A row is CPR = BK/8 chunks of 16 bytes.  LDS byte of (row, chunk c) =
// row*ROWB + ((c ^ sw(row)) << 4), with sw by the rows that a ds_read_b128 serves together, so that they fall into 16
// different 16-byte bank groups (64 banks of 4 bytes).  A fragment of the 32 x 32 instruction (S32) is 32 rows of one chunk per half wave,
// and sixteen rows in succession are served together.  One of the 16 x 16 instruction is 16 rows, two chunks per half wave, of which the
// lanes 0-3, 12-15, 20-27 are served together, then the other sixteen: the rows 0-3 and 12-15 of one chunk and 4-11 of the next one.
// (With the former's swizzle 40 % of the LDS cycles of an NT launch in 256 x 256 were conflicts.)  One wave instruction fills 1024
// bytes = RPI rows: lane l -> row RPI*q + l/CPR, physical chunk l%CPR.
template <int R, int WAVES, int BK, bool S32>
struct KCRows {
    static constexpr int ROWB = BK * 2;
    static constexpr int CPR = BK / 8;
    static constexpr int RPI = 1024 / ROWB;
    static constexpr int NI = R / RPI / WAVES;         // load instructions per wave per tile
    static constexpr int BYTES = R * ROWB;
    static constexpr int READS = 1;                    // LDS reads per fragment
    static_assert(R % (RPI * WAVES) == 0 && NI >= 1, "rows must divide over the wavefronts");
    static_assert((NI & (NI - 1)) == 0, "wid*NI + j is wid*NI ^ j");
    static_assert(S32 || CPR == 8, "the 16 x 16 instruction's units are 64 k deep");
    static __device__ __forceinline__ int sw(int row) {
        if (S32) return CPR == 8 ? (row ^ (row >> 3)) & 7 : (row >> 2) & 3;
        return (row >> 1) & 7;
    }
    v4i rsrc;
    unsigned voff[NI];       // byte offset of this lane's chunk at k0 = 0
    int kc0;                 // first k of this lane's chunk in load 0
    int K;
    // ... in load j: loads of consecutive j lie eight rows of eight chunks apart, which the swizzle turns into the chunk number (S32) or
    // into one bit of it, or sixteen rows of four, which it does not see.
    __device__ __forceinline__ int first_k(int j) const { return CPR == 8 ? kc0 ^ (S32 ? 8 * j : 32 * (j & 1)) : kc0; }
    __device__ __forceinline__ void init_kc(int lane, int wid) {
        kc0 = ((lane % CPR) ^ sw(wid * NI * RPI + lane / CPR)) * 8;
    }
    // P: operand base of this expert; rows [row0, row_limit) x [0, K) are valid
    __device__ __forceinline__ void init(const bf16_t* P, int ld, int row0, int row_limit, int K_, int lane, int wid) {
        const int valid = min(R, row_limit - row0);
        K = K_;
        init_kc(lane, wid);
        rsrc = make_rsrc(P + (size_t)row0 * ld, K_ > 0 ? (unsigned)(((size_t)(valid - 1) * ld + K_) * 2) : 0u);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int q = wid * NI + j;
            const int row = q * RPI + lane / CPR;
            const int c = (lane % CPR) ^ sw(row);
            voff[j] = (unsigned)(row * ld + c * 8) * 2u;
        }
    }
    // The same tile with its rows gathered: row r of the tile is row rows[row0 + r] of the matrix P
    // (of n_rows rows); rows at or beyond row_limit read as zeros.  Only the lane offsets differ,
    // so the main loop is the same.
    __device__ __forceinline__ void init_gather(const bf16_t* P, int ld, const int* rows, int row0, int row_limit,
                                                int n_rows, int K_, int lane, int wid) {
        K = K_;
        init_kc(lane, wid);
        rsrc = make_rsrc(P, K_ > 0 ? (unsigned)(((size_t)(n_rows - 1) * ld + K_) * 2) : 0u);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int q = wid * NI + j;
            const int row = q * RPI + lane / CPR;
            const int c = (lane % CPR) ^ sw(row);
            const int src = row0 + row < row_limit ? rows[row0 + row] : -1;
            voff[j] = src >= 0 ? (unsigned)(src * ld + c * 8) * 2u : OOB_OFFSET;
        }
    }
};

// for the 32 x 32 instruction
template <int R, int WAVES, int BK>
struct KCTile : KCRows<R, WAVES, BK, true> {
    typedef KCRows<R, WAVES, BK, true> Rows;
    using Rows::ROWB;
    using Rows::NI;
    __device__ __forceinline__ void load_one(char* tile, int k0, int wid, int j) const {
        unsigned off = this->voff[j] + (unsigned)k0 * 2u;
        // only a tile that reaches beyond K (a wave-uniform condition) has lanes to switch off
        if (k0 + BK > this->K) off = (k0 + this->first_k(j) < this->K) ? off : OOB_OFFSET;
        load_to_lds(this->rsrc, lds_address(tile) + (wid * NI + j) * 1024, off);
    }
    // fragment of the 32 rows starting at rb: lane reads row rb + lane%32, k = 16*kk + 8*(lane/32) .. +7
    typedef bf16x8 Value;
    struct Frag {
        int addr;    // byte address inside the tile for kk = 0
        __device__ __forceinline__ void init(int rb, int lane) {
            const int row = rb + (lane & 31);
            addr = row * ROWB + (((lane >> 5) ^ Rows::sw(row)) << 4);
        }
        __device__ __forceinline__ bf16x8 read(const char* tile, int kk) const {
            return *reinterpret_cast<const bf16x8*>(tile + (addr ^ (kk << 5)));
        }
    };
    template <int BLOCKS16> using Frags = Frag[BLOCKS16 / 2];
};

// for the 16 x 16 instruction
template <int R, int WAVES, int BK>
struct KCTile16 : KCRows<R, WAVES, BK, false> {
    typedef KCRows<R, WAVES, BK, false> Rows;
    using Rows::ROWB;
    using Rows::CPR;
    using Rows::NI;
    // Loads of the tile at k0: voff[j] + koff(k0) to dst(tile) + 1024 * j.  Before the first of them end_at switches off the
    // lanes that lie beyond K, for this tile and all later ones (tiles are requested in ascending order).
    __device__ __forceinline__ unsigned koff(int k0) const { return (unsigned)k0 * 2u; }
    __device__ __forceinline__ void end_at(int k0) {
        if (k0 + BK > this->K) {                         // wave-uniform, and true of the last tiles only
            asm volatile("" ::: "memory");               // (a branch, not eight selections)
#pragma unroll
            for (int j = 0; j < NI; ++j) this->voff[j] = (k0 + this->first_k(j) < this->K) ? this->voff[j] : OOB_OFFSET;
        }
    }
    static __device__ __forceinline__ unsigned dst(const char* tile, int wid) { return lds_address(tile) + wid * NI * 1024; }
    // fragments of 16 rows x 32 k: of the rows rb + d .. rb + d + 15 a lane reads row lane%16, k = 32*kk + 8*(lane/16) .. +7.
    // rb and d are multiples of 16, which the swizzle does not see.
    // at: LDS addresses, one for each kk; fragments are constant offsets from them.
    struct Value {
        bf16x8 v;
        __device__ __forceinline__ bf16x8 all() const { return v; }
    };
    template <int BLOCKS> struct Frags {
        unsigned at[CPR / 4];
        template <typename D> __device__ __forceinline__ void init(unsigned tile, int rb, int lane, D&&) {
            const int row = rb + (lane & 15);
#pragma unroll
            for (int kk = 0; kk < CPR / 4; ++kk) at[kk] = tile + row * ROWB + (((4 * kk + (lane >> 4)) ^ Rows::sw(row)) << 4);
        }
        // fragment i, of the rows from rb + d on, in the tile `off` bytes behind the one that init was told
        __device__ __forceinline__ void read(Value& f, int, int d, int kk, int, unsigned off) const {
            f.v = *(lds_bf16x8*)(uintptr_t)(at[kk] + off + d * ROWB);
        }
    };
};

// ---- N-contiguous operand tile: BK k rows x R n --------------------------------------
// LDS byte of (k, 16-byte unit u) = k*PITCH + (place of u in row k << 4), so that the k rows that half a wave's transposing read
// touches fall into different banks (64 banks of 4 bytes).  32 x 32 instruction (S32): four k rows, four units each, rotated by
// four units: (u + 4*(k&3)) % UPR.  16 x 16: eight (k, k+1, k+2, k+3 and those eight further on), two units each: u ^ turn(k).
// One wave instruction fills 1024 bytes = RPI rows: lane l -> row RPI*q + l/UPR, place l%UPR.
template <int R, int WAVES, int BK, bool S32>
struct NCRows {
    static constexpr int PITCH = R * 2;                // bytes per k row
    static constexpr int UPR = R / 8;                  // 16-byte units per row
    static constexpr int RPI = 1024 / PITCH;           // rows per wave instruction
    static constexpr int NI = BK / RPI / WAVES;
    static constexpr int BYTES = BK * PITCH;
    static constexpr int READS = 2;                    // LDS reads per fragment
    static_assert(BK % (RPI * WAVES) == 0 && NI >= 1, "rows must divide over the wavefronts");
    static_assert(UPR >= 16 || (S32 && UPR == 8), "the turns of the k rows must fit a row of units (S32: or two)");
    static __device__ __forceinline__ int turn(int k) { return 4 * (k & 3) + 2 * ((k >> 3) & 1); }
    v4i rsrc;
    unsigned voff[NI];
    unsigned kstep;          // bytes per k row in memory
    // descriptor of rows [0, K) x columns [0, n_valid) of the matrix at P
    static __device__ __forceinline__ v4i rsrc_of(const bf16_t* P, int ld, int n_valid, int K) {
        return make_rsrc(P, K > 0 ? (unsigned)(((size_t)(K - 1) * ld + n_valid) * 2) : 0u);
    }
    // P: operand base of this expert ([k][n], n contiguous); rows [0, K) x columns [n0, n_limit) valid
    __device__ __forceinline__ void init(const bf16_t* P, int ld, int n0, int n_limit, int K, int lane, int wid) {
        const int n_valid = n_limit - n0;
        kstep = (unsigned)ld * 2u;
        rsrc = rsrc_of(P + n0, ld, n_valid, K);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int q = wid * NI + j;
            const int row = q * RPI + lane / UPR;
            const int u = S32 ? ((lane % UPR) - 4 * (row & 3) + 4 * UPR) % UPR : (lane % UPR) ^ turn(row);
            voff[j] = (u * 8 < n_valid) ? (unsigned)(row * ld + u * 8) * 2u : OOB_OFFSET;
        }
    }
};

// for the 32 x 32 instruction
template <int R, int WAVES, int BK>
struct NCTile : NCRows<R, WAVES, BK, true> {
    typedef NCRows<R, WAVES, BK, true> Rows;
    using Rows::PITCH;
    using Rows::UPR;
    using Rows::NI;
    // (the descriptor ends at the last row)
    __device__ __forceinline__ void load_one(char* tile, int k0, int wid, int j) const {
        load_to_lds(this->rsrc, lds_address(tile) + (wid * NI + j) * 1024, this->voff[j] + (unsigned)k0 * this->kstep);
    }
    // fragment of the 32 columns starting at nb: two transposing reads give the lane n = nb + lane%32, k = 16*kk +
    // 8*(lane/32) .. +7.  In a 16-lane group lane a points at row a/4, columns 4*(a%4)..+3; the hardware returns to lane i
    // four k of column i.
    typedef bf16x8 Value;
    struct Frag {
        int addr;
        __device__ __forceinline__ void init(int nb, int lane) {
            const int g = lane >> 4, a = lane & 15;
            const int k_in = 8 * (g >> 1) + (a >> 2);
            const int n = nb + 16 * (g & 1) + 4 * (a & 3);
            addr = k_in * PITCH + ((((n >> 3) + 4 * (k_in & 3)) % UPR) << 4) + ((n & 7) << 1);
        }
        __device__ __forceinline__ bf16x8 read(const char* tile, int kk) const {
            const char* p = tile + addr + kk * 16 * PITCH;
            v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p);
            v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(p + 4 * PITCH));
            typedef short v8s __attribute__((ext_vector_type(8)));
            v8s both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        }
    };
    template <int BLOCKS16> using Frags = Frag[BLOCKS16 / 2];
};

// for the 16 x 16 instruction
template <int R, int WAVES, int BK>
struct NCTile16 : NCRows<R, WAVES, BK, false> {
    typedef NCRows<R, WAVES, BK, false> Rows;
    using Rows::PITCH;
    using Rows::UPR;
    using Rows::RPI;
    using Rows::NI;
    int K, row0;             // k rows; this lane's row in load 0
    __device__ __forceinline__ void init(const bf16_t* P, int ld, int n0, int n_limit, int K, int lane, int wid) {
        Rows::init(P, ld, n0, n_limit, K, lane, wid);
        this->K = K;
        row0 = wid * NI * RPI + lane / UPR;
    }
    // as for K-contiguous operands
    __device__ __forceinline__ unsigned koff(int k0) const { return (unsigned)k0 * this->kstep; }
    __device__ __forceinline__ void end_at(int k0) {
        if (k0 + BK > K) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int j = 0; j < NI; ++j) this->voff[j] = (k0 + row0 + j * RPI < K) ? this->voff[j] : OOB_OFFSET;
        }
    }
    static __device__ __forceinline__ unsigned dst(const char* tile, int wid) { return lds_address(tile) + wid * NI * 1024; }
    // fragments of 16 columns x 32 k: two transposing reads give the lane column nb + d + lane%16, k = 32*kk +
    // 8*(lane/16) .. +7.  nb and d have no bits in common (and tiles begin at multiples of
    // PITCH), so that d turns into an exclusive or: an address each.
    struct Value {
        v4s lo, hi;
        __device__ __forceinline__ bf16x8 all() const {
            typedef short v8s __attribute__((ext_vector_type(8)));
            const v8s both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        }
    };
    template <int BLOCKS> struct Frags {
        unsigned at[BLOCKS];
        template <typename D> __device__ __forceinline__ void init(unsigned tile, int nb, int lane, D&& d) {
            const int g = lane >> 4, a = lane & 15;
            const int k_in = 8 * g + (a >> 2);
            const int n = nb + 4 * (a & 3);
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i) at[i] = (tile + k_in * PITCH + (((n >> 3) ^ Rows::turn(k_in)) << 4) + ((n & 7) << 1)) ^ (d(i) << 1);
        }
        // part (0 or 1) of fragment i
        __device__ __forceinline__ void read(Value& f, int i, int, int kk, int part, unsigned off) const {
            const unsigned p = at[i] + off + kk * 32 * PITCH;
            if (part == 0) f.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(uintptr_t)p);
            else f.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(uintptr_t)(p + 4 * PITCH));
        }
    };
};

// the operands' tiles of a layout, for either instruction
template <bool KC, bool S32, int R, int W, int BK>
using OperandTile = std::conditional_t<KC, std::conditional_t<S32, KCTile<R, W, BK>, KCTile16<R, W, BK>>,
                                       std::conditional_t<S32, NCTile<R, W, BK>, NCTile16<R, W, BK>>>;

struct Unit8 {
    static __device__ __forceinline__ void to_float(const uint4& u, float* o) {
        const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[2 * i] = __uint_as_float(w[i] << 16);
            o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};

// s_waitcnt vmcnt(N) only (N <= 63), with a compiler-level memory fence
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_lgkmcnt() { asm volatile("s_waitcnt lgkmcnt(%0)" : : "i"(N) : "memory"); }

// What goes behind which of the MB matrix instructions of a block.  A matrix instruction takes sixteen cycles; one other instruction
// of its wave behind it is free, or a vector and a scalar one, each further one costs eight cycles (one wave per SIMD; measured
// for independent vector, scalar and LDS instructions alike).  Hence: no address arithmetic in the loops but what moves from slot to
// slot, and everything in a gap of its own.  LDS reads, of which the four waves' together take 32 cycles (16 for the transposing
// ones), come behind the first eight, early enough for the next block, then two loads, in two parts, and moves of addresses between.
template <int MB>
struct Gaps {
    static constexpr int SPAN = MB >= 12 ? 8 : MB;
    template <typename F>
    static __device__ __forceinline__ void reads(int m, int n, F&& read) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (r < n && r * SPAN / n == m) read(r);
    }
    // two loads: prepare(l) is followed by go(l) one gap later, or in the same one where there are few
    template <typename P, typename G>
    static __device__ __forceinline__ void loads(int m, P&& prepare, G&& go) {
#pragma unroll
        for (int l = 0; l < 2; ++l) {
            const int at = MB >= 8 ? MB * (9 + 4 * l) / 16 : MB - 2 + l;
            if (m == at) prepare(l);
            if constexpr (MB < 8) { if (m == at) { asm volatile("s_nop 0" ::: "memory"); go(l); } }
            else if (m == at + 1) go(l);
        }
    }
    // four moves: between the reads where those leave room (`odd`), else around the loads
    template <typename F>
    static __device__ __forceinline__ void moves(int m, bool odd, F&& move) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int at = MB < 12 ? e * MB / 4 : odd ? 2 * e + 1 : (e == 0 ? 8 : e == 1 ? 11 : e == 2 ? 12 : 15) * MB / 16;
            if (m == at) move(e);
        }
    }
};

// The matrix instruction as volatile assembly with a memory clobber: the compiler keeps
// such statements, the LDS reads and the loads into LDS in the order they are written,
// which is what the hand-scheduled loop below relies on (it still allocates registers
// and inserts the s_waitcnt lgkmcnt for LDS reads it issued itself).
// Accumulators live in the AGPR half of the register file when a wave owns 512 registers, in ordinary VGPRs when two waves
// share a SIMD.
__device__ __forceinline__ void mfma_pinned(floatx4& acc, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b) : "memory");
}
template <bool ACC_IN_AGPR>
__device__ __forceinline__ void mfma32_pinned(floatx16& acc, const bf16x8& a, const bf16x8& b) {
    if constexpr (ACC_IN_AGPR)
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b) : "memory");
    else
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b) : "memory");
}

// TN only: the reduction dimension may run over the rows of several
// partitions (up to MAX_KSEGS row ranges, one per partition buffer); tiles never straddle two ranges.  KCursor says which range
// the tile that is being requested lies in and where.
constexpr int MAX_KSEGS = 8;
struct TileCoord { int e, q, er, tn, m0, n0, Mdim, Kdim, KT; };      // expert, partition of the launch, their place in row arrays
struct KCursor { int seg, jl, tiles; };

// Numbers of the tiles of a launch.  Only tiles that exist are numbered: an expert with fewer rows than the capacity
// has fewer tile rows (NN, NT), an expert without rows has no tiles at all (TN), so that the workgroups, which take
// the numbers b, b + grid, ..., all get the same amount of work whatever the spread of the counts.  The tile rows that
// an expert fills by more than half come first, expert by expert; a last tile row with fewer rows is numbered after
// all of those, since it takes less time (the 64-k loops multiply only the blocks of rows that hold something) and
// belongs at the end of a workgroup's list.  Lane l of every wavefront holds the tile rows of expert l (of expert
// l / np of partition l % np where the launch covers several; at most 64 in all);
// inclusive scans over the lanes give the numbers at which each expert ends.
struct TileNumbers {
    int lane_rows, lane_tm;              // rows, such tile rows of expert `lane`
    int lane_end, tail_end;              // numbers of whole tiles / of last tile rows up to and including this expert
    int nwhole, nblocks;                 // whole tiles; all tiles
};
template <int LAY, int EPI, typename C>
__device__ __forceinline__ TileNumbers number_tiles(const GemmArgs& g, int tiles_m, int tiles_n, int lane) {
    constexpr int BM = C::BM;
    TileNumbers t;
    t.lane_rows = t.lane_tm = 0;
    int lane_tail = 0;                   // whether a last tile row with fewer rows follows
    if (lane < (LAY == GEMM_TN ? g.E : launch_experts(g))) {
        int rows = 0;
        if constexpr (LAY == GEMM_TN) {
            const int segs = g.k_segs > 1 ? g.k_segs : 1;
            for (int sg = 0; sg < segs; ++sg) rows += g.counts[sg * g.E + lane];
        } else {
            const ExpertOf x = expert_of(g, lane);
            rows = g.counts[x.q * g.E + x.e];
        }
        t.lane_rows = rows;
        if (LAY == GEMM_TN) t.lane_tm = (rows > 0 || EPI == EPI_STORE_F32) ? tiles_m : 0;   // a plain store still writes zeros
        else {
            t.lane_tm = min(tiles_m, (rows + BM / 2 - 1) / BM);
            lane_tail = (t.lane_tm < tiles_m && rows > t.lane_tm * BM) ? 1 : 0;
        }
    }
    t.lane_end = t.lane_tm * tiles_n;
    t.tail_end = lane_tail;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(t.lane_end, off, 64), q = LAY == GEMM_TN ? 0 : __shfl_up(t.tail_end, off, 64);
        if (lane >= off) { t.lane_end += o; t.tail_end += q; }
    }
    t.nwhole = __builtin_amdgcn_readlane(t.lane_end, 63);
    t.nblocks = t.nwhole + __builtin_amdgcn_readlane(t.tail_end, 63) * tiles_n;
    return t;
}

// The tiles b0, b0 + step, b0 + 2 step, ... of one GEMM.  While a tile's epilogue runs (it needs only the
// staging part of LDS and no matrix instructions), the first operand tiles of the next
// tile are already on their way into the rest of the ring, so neither the launch of a new
// workgroup nor the first trip to memory stands between two main loops.
// ONE: tile b0 only.
template <int LAY, int EPI, typename C, bool ONE>
__device__ __forceinline__ void gemm_tiles(const GemmArgs& g, int tiles_m, int tiles_n, const TileNumbers& tiles, int b0, int step) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int BM = C::BM, BN = C::BN, WM = C::WM, WN = C::WN, TM = C::TM, RB = C::RB, NB = C::NB;
    constexpr int STAGE = C::STAGE_BYTES, BK = C::BK, NS = C::NS;
    constexpr bool S32 = C::S32;
    constexpr int TNN = WN / 32;
    constexpr bool W64 = C::LOOP == LOOP_W64, R64 = C::LOOP == LOOP_R64, N64 = C::LOOP == LOOP_N64;
    static_assert(!N64 || LAY == GEMM_NT, "units of 64 k of both operands");
    constexpr bool ALT = C::LOOP != LOOP_PIPE32;     // waves' row blocks alternate (see block_row)
    constexpr bool QUAD = C::LOOP == LOOP_PIPE32 && C::OCC == 1;
    // Depth of one load unit of each operand.  In the two-ring loop the rows travel 64 k at a time, so that every request
    // is a whole 128-byte line; the weights, whose rows are whole lines anyway, keep tiles of 32 k.
    constexpr int AK = BK, BKB = W64 ? 32 : BK;
    static_assert(!W64 || LAY == GEMM_NN, "one K-contiguous operand");
    constexpr int A_BYTES = BM * BK * 2;
    // The epilogue stages accumulators in the first SB stages of the ring; a tile's ring
    // starts at stage SB, so that its first operand tiles can arrive during the epilogue
    // of the tile before.  (Two-ring loop: in the third unit of the wide ring.)
    constexpr int SB = 2;
    constexpr int CW = C::CW;
    static_assert(ALT || C::WAVES * 32 * CW * 4 <= SB * STAGE, "staging does not fit below the ring's first stage");
    static_assert(!(W64 || N64) || C::WAVES * 32 * CW * 4 <= 32 * 1024, "staging does not fit one unit of the wide ring");
    // two-ring LDS map: three units of 64 k x 256 rows, then four tiles of 32 k x 256 rows
    constexpr int WIDE_UNIT = 32 * 1024, NARROW_TILE = 16 * 1024, NARROW_OFF = 3 * WIDE_UNIT;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / C::WAVES_N, wn = wid % C::WAVES_N;
    typedef OperandTile<LAY != GEMM_TN, S32, BM, C::WAVES, AK> AT;
    typedef OperandTile<LAY == GEMM_NT, S32, BN, C::WAVES, BKB> BT;
    constexpr int LPW = AT::NI + BT::NI;         // loads per wave per tile
    // Where two workgroups share a CU the operands' offsets and descriptors are formed again at the top of a
    // tile (the other workgroup covers that) instead of being carried from the one before: with 128 registers
    // for accumulators and fragments the compiler otherwise moves descriptors into vector registers, which the
    // load cannot take.
    constexpr bool REBIND = C::OCC == 2 && !ONE;
    // First row of the wave's block i of 32 rows.  In the 64-k loops the waves' blocks alternate, so that a tile
    // with few rows left needs only the first blocks of every wave (see `active` below).
    constexpr int ROW_STEP = ALT ? 32 * C::WAVES_M : 32;
    auto block_row = [&](int i) __attribute__((always_inline)) { return ALT ? i * ROW_STEP + wm * 32 : wm * WM + i * 32; };
    typename AT::template Frags<RB> fa;
    typename BT::template Frags<NB> fb;
    typedef typename AT::Value FA;
    typedef typename BT::Value FB;
    constexpr int AR = AT::READS, BR = BT::READS;
    auto dist_a = [](int i) __attribute__((always_inline)) { return (i >> 1) * ROW_STEP + (i & 1) * 16; };     // of a block of 16 rows from the first
    auto dist_b = [](int j) __attribute__((always_inline)) { return j * 16; };
    const unsigned lds0 = lds_address(smem);
    if constexpr (S32) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i].init(block_row(i), lane);
#pragma unroll
        for (int j = 0; j < TNN; ++j) fb[j].init(wn * WN + j * 32, lane);
    }
    // 256 x 256: addresses in the operands' tiles that begin at these LDS addresses (the loops move them along)
    auto frags_at = [&](unsigned a, unsigned b) __attribute__((always_inline)) {
        if constexpr (!S32) {
            int l = lane;                                // (formed for every tile: there are no registers to keep them in through an epilogue)
            asm volatile("" : "+v"(l));
            fa.init(a, block_row(0), l, dist_a);
            fb.init(b, wn * WN, l, dist_b);
            if constexpr (!N64) {
#pragma unroll
                for (unsigned& at : fa.at) asm volatile("" : "+v"(at));
#pragma unroll
                for (unsigned& at : fb.at) asm volatile("" : "+v"(at));
            }
        }
    };
    // fragment of the wave's block i of 16 rows / j of 16 columns, read in one part or two
    auto frag_a = [&](FA& f, unsigned off, int i, int kk, int part) __attribute__((always_inline)) { if constexpr (!S32) fa.read(f, i, dist_a(i), kk, part, off); };
    auto frag_b = [&](FB& f, unsigned off, int j, int kk, int part) __attribute__((always_inline)) { if constexpr (!S32) fb.read(f, j, dist_b(j), kk, part, off); };
    auto whole_a = [&](FA& f, unsigned off, int i, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < AR; ++q) frag_a(f, off, i, kk, q);
    };
    auto whole_b = [&](FB& f, unsigned off, int j, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < BR; ++q) frag_b(f, off, j, kk, q);
    };

    // ---- tile number -> (expert, tile) -----------------------------------------------
    const int lane_tm = tiles.lane_tm, lane_end = tiles.lane_end, tail_end = tiles.tail_end;
    const int nwhole = tiles.nwhole, nblocks = tiles.nblocks;
    // Tiles are numbered expert by expert, in groups of 4 tile-rows walked column by
    // column, so 32 consecutive numbers form a 4 x 8 block that shares 4 A panels and 8
    // B panels.  Hardware deals consecutive workgroup ids round-robin to the 8 XCDs (each
    // with its own L2), and the grid is a multiple of 8, so tile number b always runs on
    // XCD b mod 8; within every run of 256 numbers, XCD x is given the x-th block of 32
    // consecutive tiles, so each L2 serves a compact block while all eight XCDs stay on
    // the same expert(s) and share its weights through the memory-side cache.  (Against
    // plain order this halves what the L2s fetch; against giving each XCD its own experts
    // it is 3-5 % faster.)  A last partial run keeps plain order.
    auto decode = [&](int b, TileCoord& t) -> bool {
        const int lin = (b < (nwhole & ~255)) ? (b & ~255) + (b & 7) * 32 + ((b >> 3) & 31) : b;
        const int all = LAY == GEMM_TN ? g.E : launch_experts(g);
        int e, tm;
        if (LAY == GEMM_TN || lin < nwhole) {
            // the expert: as many experts end at or before lin as lanes say so (the ends never decrease)
            e = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane_end <= lin));
            if (e >= all) return false;
            const int tm_e = __builtin_amdgcn_readlane(lane_tm, e);      // tile rows of this expert
            const int rem = lin - (__builtin_amdgcn_readlane(lane_end, e) - tm_e * tiles_n);
            constexpr int GM = 4;
            const int grp = rem / (GM * tiles_n);
            const int first = grp * GM;
            const int gsz = min(GM, tm_e - first);
            const int in = rem - grp * GM * tiles_n;
            tm = first + in % gsz;
            t.tn = in / gsz;
        } else {
            const int q = (lin - nwhole) / tiles_n;                      // the q-th expert with such a last tile row
            t.tn = (lin - nwhole) - q * tiles_n;
            e = __builtin_popcountll(__builtin_amdgcn_ballot_w64(tail_end <= q));
            if (e >= all) return false;
            tm = __builtin_amdgcn_readlane(lane_tm, e);
        }
        const ExpertOf x = LAY == GEMM_TN ? ExpertOf{e, 0} : expert_of(g, e);
        t.er = x.q * g.E + x.e;
        const int rows = __builtin_amdgcn_readlane(tiles.lane_rows, e);
        if (LAY == GEMM_TN) { t.Mdim = g.Mo; t.Kdim = rows; } else { t.Mdim = rows; t.Kdim = g.K; }
        t.e = x.e;
        t.q = x.q;
        t.m0 = tm * BM;
        t.n0 = t.tn * BN;
        t.KT = (t.Kdim + BK - 1) / BK;
        if constexpr (LAY == GEMM_TN) {
            if (g.k_segs > 1) {
                t.KT = 0;
                for (int sg = 0; sg < g.k_segs; ++sg) t.KT += (g.counts[sg * g.E + t.e] + BK - 1) / BK;
            }
        }
        if (t.m0 >= t.Mdim) return false;
        if (t.Kdim <= 0 && EPI != EPI_STORE_F32) return false;   // nothing to add; a plain store still writes zeros
        return true;
    };
    auto next_tile = [&](int b, TileCoord& t) -> int {          // first tile of this workgroup at or after b, or -1
        for (; b < nblocks; b += step)
            if (decode(b, t)) return b;
        return -1;
    };
    auto bind = [&](const TileCoord& t, AT& ta_, BT& tb_, int lane) {
        const bf16_t* A = (const bf16_t*)g.A + (size_t)t.e * g.a_estride + (LAY == GEMM_TN ? 0 : t.q * g.a_pstride);
        const bf16_t* B = (const bf16_t*)g.B + (size_t)t.e * g.b_estride;
        bool gathered = false;
        if constexpr (LAY != GEMM_TN) {
            if (g.a_rows) {
                ta_.init_gather((const bf16_t*)g.A, g.lda, g.a_rows + (size_t)t.er * g.Cp, t.m0, t.Mdim, g.a_row_limit,
                                t.Kdim, lane, wid);
                gathered = true;
            }
        }
        if (!gathered) ta_.init(A, g.lda, t.m0, t.Mdim, t.Kdim, lane, wid);
        tb_.init(B, g.ldb, t.n0, g.N, t.Kdim, lane, wid);
    };
    // Tiles are requested in ascending order, over several row ranges (TN) with new descriptors where one is used up, and past
    // the last range everything reads as zeros.
    // operand descriptors of row range seg (TN), its rows
    auto bind_range = [&](const TileCoord& tc, int seg, AT& ta_, BT& tb_) -> int {
        int rows = 0;
        if constexpr (LAY == GEMM_TN) {
            int e = tc.e;
            if constexpr (!S32) asm volatile("" : "+s"(e));      // (what follows belongs here, not before the loop)
            rows = seg < g.k_segs ? g.counts[seg * g.E + e] : 0;
            const bf16_t* A = (const bf16_t*)g.A + (size_t)e * g.a_estride + seg * g.a_sstride + tc.m0;
            const bf16_t* B = (const bf16_t*)g.B + (size_t)e * g.b_estride + seg * g.b_sstride + tc.n0;
            ta_.rsrc = AT::rsrc_of(A, g.lda, tc.Mdim - tc.m0, rows);
            tb_.rsrc = BT::rsrc_of(B, g.ldb, g.N - tc.n0, rows);
        }
        return rows;
    };
    // into the next range with rows, if this one is used up
    auto next_range = [&](const TileCoord& tc, KCursor& kc_, AT& ta_, BT& tb_) __attribute__((always_inline)) {
        while (kc_.jl >= kc_.tiles) {
            ++kc_.seg;
            kc_.jl = 0;
            const int rows = bind_range(tc, kc_.seg, ta_, tb_);
            kc_.tiles = kc_.seg < g.k_segs ? (rows + BK - 1) / BK : 0x7fffffff;
        }
    };
    // 256 x 256 weight gradients: on to the next tile.  Its loads have no offset for K: the descriptors begin at the tile's first row
    // and end at the range's last one.  (Eight scalar instructions a tile.  With K in the loads' scalar offset, which is no part of the bounds
    // check, the lanes beyond the last row had to be switched off, and on again for the next range: half a microsecond more before
    // a tile's first product, which tiles of few steps show: 16 experts x 6 rows, 1920/5760: 568 us against 561; 64 experts x 64 rows,
    // 768/3072, two ranges: 1238 and 1231.)
    auto advance = [&](const TileCoord& tc, KCursor& kc_, AT& ta_, BT& tb_) __attribute__((always_inline)) {
        if constexpr (LAY == GEMM_TN && !S32) {
            drop_rows(ta_.rsrc, ta_.kstep * BK);
            drop_rows(tb_.rsrc, tb_.kstep * BK);
            ++kc_.jl;
            if (g.k_segs > 1) next_range(tc, kc_, ta_, tb_);
        }
    };
    // The descriptors into scalar registers, where the compiler does not keep them: a load may follow five wait states later.
    auto settle = [&](AT& ta_, BT& tb_) __attribute__((always_inline)) {
        for (v4i* r : {&ta_.rsrc, &tb_.rsrc}) {
            int w0 = __builtin_amdgcn_readfirstlane((*r)[0]), w1 = __builtin_amdgcn_readfirstlane((*r)[1]), w2 = __builtin_amdgcn_readfirstlane((*r)[2]);
            asm volatile("" : "+s"(w0), "+s"(w1), "+s"(w2) : : "memory");
            (*r)[0] = w0; (*r)[1] = w1; (*r)[2] = w2;
        }
    };
    // load l of the tile the descriptors begin with, to the LDS address in m0
    auto go = [&](const AT& ta_, const BT& tb_, int l) __attribute__((always_inline)) {
        if (l < AT::NI) load_to_destination(ta_.rsrc, ta_.voff[l]);
        else load_to_destination(tb_.rsrc, tb_.voff[l - AT::NI]);
    };
    // load l of the tile that starts at k0 (tiles in ascending order, each begun with load 0: that is where the cursor moves on)
    auto request = [&](const TileCoord& tc, KCursor& kc_, AT& ta_, BT& tb_, char* st, int k0, int l) {
        if constexpr (S32) {
            if constexpr (LAY == GEMM_TN) {
                if (g.k_segs > 1) {
                    if (l == 0) {
                        if (k0 == 0) { kc_.seg = -1; kc_.jl = 0; kc_.tiles = 0; } else ++kc_.jl;
                        next_range(tc, kc_, ta_, tb_);
                    }
                    k0 = kc_.jl * BK;
                }
            }
            if (l < AT::NI) ta_.load_one(st, k0, wid, l);
            else tb_.load_one(st + A_BYTES, k0, wid, l - AT::NI);
        } else {
            if (l == 0) {
                if (k0 > 0) advance(tc, kc_, ta_, tb_);
                else if (g.k_segs > 1) { kc_ = {-1, 0, 0}; next_range(tc, kc_, ta_, tb_); }
            }
            if (l < AT::NI) load_to_lds(ta_.rsrc, AT::dst(st, wid) + l * 1024, ta_.voff[l]);
            else load_to_lds(tb_.rsrc, BT::dst(st + A_BYTES, wid) + (l - AT::NI) * 1024, tb_.voff[l - AT::NI]);
        }
    };
    // unit of one operand (rings and units of their own): loads l0 to l1 - 1 of the unit that starts at k0
    auto load_unit = [&](auto& t_, const char* dst, int k0, int l0, int l1) __attribute__((always_inline)) {
        typedef std::remove_reference_t<decltype(t_)> OT;
        if (l0 == 0) t_.end_at(k0);
#pragma unroll
        for (int l = l0; l < l1; ++l) load_to_lds(t_.rsrc, OT::dst(dst, wid) + l * 1024, t_.voff[l] + t_.koff(k0));
    };
    auto wide_slot = [&](int slot3) __attribute__((always_inline)) { return smem + slot3 * WIDE_UNIT; };
    auto narrow_slot = [&](int slot4) __attribute__((always_inline)) { return smem + NARROW_OFF + slot4 * NARROW_TILE; };
    constexpr int WL = W64 ? AT::NI : 0;       // loads per wave: one wide unit (8)
    constexpr int NL = W64 ? BT::NI : 0;       //                 one narrow tile (4)
    static_assert(!W64 || (WL == 8 && NL == 4), "the two-ring schedule issues two wide and two narrow loads per block");
    // ring of 64-k stages: a wave's loads of a stage that go out in block 3 of a step, the rest follow in blocks 0 and 1
    constexpr int R64_G3 = (LPW + 2) / 3, R64_G0 = (LPW + 1) / 3, R64_G1 = LPW / 3;
    static_assert(!R64 || R64_G3 + R64_G0 + R64_G1 == LPW, "loads of a stage over the blocks");
    // ring of 32 k: loads of tile NS-1 that are on their way when the loop begins
    constexpr int PIPE_EARLY = LPW / 2;
    // five-unit loop: load l of the weights' / the rows' unit of step t into a unit slot
    constexpr int UL = N64 ? 8 : 0;
    static_assert(!N64 || (AT::NI == 8 && BT::NI == 8), "eight loads per wave and unit");
    // the part of a tile's first loads that does not touch the staging region, and the rest
    auto issue_early = [&](const TileCoord& tc, KCursor& kc_, AT& ta_, BT& tb_) {
        if constexpr (W64) {
            // what the loop expects to be on its way when it starts: wide units 0 and 1 and the first
            // quarter of unit 2 (late: its slot is the staging region), narrow tiles 0..2 and half of tile 3
            load_unit(ta_, wide_slot(0), 0, 0, WL);
            load_unit(tb_, narrow_slot(0), 0, 0, NL);
            load_unit(tb_, narrow_slot(1), 32, 0, NL);
            load_unit(ta_, wide_slot(1), 64, 0, WL);
            load_unit(tb_, narrow_slot(2), 64, 0, NL);
            load_unit(tb_, narrow_slot(3), 96, 0, NL / 2);
        } else if constexpr (N64) {
            // units 0 to 3: weights and rows of steps 0 and 1
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                load_unit(tb_, wide_slot(2 * t), t * 64, 0, UL);
                load_unit(ta_, wide_slot(2 * t + 1), t * 64, 0, UL);
            }
        } else {
            constexpr int FIRST = R64 ? 0 : SB, STAGES = R64 ? NS - C::SBR : NS - SB;
#pragma unroll
            for (int s = 0; s < STAGES; ++s)
#pragma unroll
                for (int l = 0; l < LPW; ++l) request(tc, kc_, ta_, tb_, smem + (FIRST + s) * STAGE, s * BK, l);
        }
    };
    auto issue_late = [&](const TileCoord& tc, KCursor& kc_, AT& ta_, BT& tb_) {
        if constexpr (W64) {
            load_unit(ta_, wide_slot(2), 128, 0, WL / 4);
        } else if constexpr (N64) {
            load_unit(tb_, wide_slot(4), 128, 0, UL / 4);
        } else if constexpr (R64) {
#pragma unroll
            for (int s = NS - C::SBR; s < NS - 1; ++s)
#pragma unroll
                for (int l = 0; l < LPW; ++l) request(tc, kc_, ta_, tb_, smem + s * STAGE, s * BK, l);
#pragma unroll
            for (int l = 0; l < R64_G3; ++l) request(tc, kc_, ta_, tb_, smem + (NS - 1) * STAGE, (NS - 1) * BK, l);
        } else {
#pragma unroll
            for (int s = NS - SB; s < NS - 1; ++s)
#pragma unroll
                for (int l = 0; l < LPW; ++l) request(tc, kc_, ta_, tb_, smem + (SB + s - NS) * STAGE, s * BK, l);
#pragma unroll
            for (int l = 0; l < PIPE_EARLY; ++l) request(tc, kc_, ta_, tb_, smem + (SB - 1) * STAGE, (NS - 1) * BK, l);
        }
    };

    TileCoord cur;
    int vb = next_tile(b0, cur);
    if (vb < 0) return;
    AT ta;
    BT tb;
    bind(cur, ta, tb, lane);
    KCursor kc = {};
    issue_early(cur, kc, ta, tb);
    issue_late(cur, kc, ta, tb);
    bool first = true;

    for (;;) {
        if constexpr (REBIND) {
            bind(cur, ta, tb, lane);
            if constexpr (LAY == GEMM_TN) { if (g.k_segs > 1) bind_range(cur, kc.seg, ta, tb); }
        }
        const int m0 = cur.m0, n0 = cur.n0, e = cur.e, q = cur.q, er = cur.er, tn = cur.tn, Mdim = cur.Mdim;
        // (256 x 256: an empty reduction is one tile of zeros, since a loop that may not run at all costs a copy of all accumulators behind it)
        const int KT = S32 ? cur.KT : max(cur.KT, 1);
        if constexpr (!S32) __builtin_assume(KT > 0);
        // blocks of 32 rows per wave that hold rows of this tile
        const int active = ALT && LAY != GEMM_TN ? min(TM, (Mdim - m0 + 32 * C::WAVES_M - 1) / (32 * C::WAVES_M)) : TM;
        floatx4 acc[S32 ? 1 : RB][S32 ? 1 : NB];
        floatx16 acc32[S32 ? TM : 1][S32 ? TNN : 1];
        if constexpr (S32) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TNN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc32[i][j][r] = 0.0f;
        } else {
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;
        }
        if constexpr (QUAD) {
            // (here, while the first loads are on their way: left to itself the compiler writes all 256 right before the loop.  With
            // a loop for each number of active blocks it would then have to move them between those, and spills.)
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
        // The compiler does not see the matrix instructions, which need two wait states behind a vector instruction that
        // writes an operand and up to eighteen before another one reads the result.  So every main loop begins with a pause, and
        // behind it the accumulators pass through a longer one before anything, a copy of the compiler's too, reads them.
        auto pause = [&]() __attribute__((always_inline)) { asm volatile("s_nop 1" ::: "memory"); };
        auto retire = [&]() __attribute__((always_inline)) {
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
            if constexpr (!S32) {
                static_assert(S32 || C::OCC == 1, "accumulators in the AGPR half");
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j) asm volatile("" : "+a"(acc[i][j]) : : "memory");
            }
        };
        // Product of the wave's 16 rows i and 16 columns j.
        auto mul = [&](int i, int j, const FA& rows, const FB& cols) __attribute__((always_inline)) {
            if constexpr (!S32) mfma_pinned(acc[i][j], cols.all(), rows.all());
        };
        // With 256 x 256 the accumulators leave registers for the fragments of one chunk of 32 k and no more.  A chunk is
        // therefore multiplied in four blocks - the lower half of the fragments X times the lower and the upper half of Y,
        // then the upper half of X times the upper and the lower half of Y - in each of which one half dies, whose registers
        // receive what the block after it needs: Y's upper half, X's upper half, X's lower half of the next chunk, and
        // Y's lower half of it in the place of the upper one (so the places of Y's halves change from chunk to chunk).  Of the
        // half that came last one fragment after the other is used, so that the last ones read have as long as the first.

        if constexpr (W64) {
            // Hand-scheduled loop over steps of 64 k = two chunks = eight blocks 0 to 7 (see above), with the rows as X and
            // the weights as Y.  While a block is multiplied the half it frees is filled and two loads are issued,
            // at most one LDS read or load per matrix instruction.  Step t reads wide unit t (slot t mod 3) and narrow
            // tiles 2t, 2t+1 (slots mod 4).  Two barriers per step:
            //   after block 1: every wave has read narrow tile 2t for the last time (its slot then receives
            //           tile 2t+4), and tile 2t+1 has landed;
            //   after block 5: every wave has read wide unit t and narrow tile 2t+1 for the last time (their
            //           slots receive unit t+3 and tile 2t+5), and unit t+1 and tile 2t+2 have landed.
            // Each wave issues, per step, in this order, two loads per block: 0 - wide unit t+2 loads 2,3, 1 - narrow tile
            // 2t+3 loads 2,3; 2 - unit t+2 loads 4,5, 3 - tile 2t+4 loads 0,1; 4 - unit t+2 loads 6,7, 5 - tile
            // 2t+4 loads 2,3; 6 - unit t+3 loads 0,1, 7 - tile 2t+5 loads 0,1.  At either barrier the sixteen
            // youngest loads of the wave may still be in flight; everything older is what the step needs next.
            frags_at(lds0, lds0 + NARROW_OFF);
            if (first) wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            // TMA: blocks of 32 rows per wave that hold something; loads, waits and barriers are the same for all
            auto loop = [&](auto tma) __attribute__((always_inline)) {
            constexpr int TMA = decltype(tma)::value;
            constexpr int HX = TMA, HY = NB / 2, MB = HX * HY;
            static_assert(AR == 1 && BR == 2, "rows read by ds_read_b128, weights by pairs of transposing reads");
            FA X[2][HX];
            FB Y[2][HY];
            // LDS read r of half h, of unit t or of the narrow tile `off` bytes behind tile 2t, by the addresses as they stand
            auto read_x = [&](FA (&to)[HX], int h, int r, int kk) __attribute__((always_inline)) { frag_a(to[r], 0, h * HX + r, kk, 0); };
            auto read_y = [&](FB (&to)[HY], int h, int r, unsigned off) __attribute__((always_inline)) { frag_b(to[r / 2], off, h * HY + r / 2, 0, r % 2); };
            // X's half xh times Y's half yh, which lies in Y[ys]; new_x: X's came last.  Beside it `reads` LDS reads, loads L0 and
            // L0 + 1 of a wide unit or narrow tile (byte offset k) to LDS address d, and moves of addresses.
            auto block = [&](int xh, int yh, int ys, bool new_x, int reads, auto&& read, bool wide, unsigned d, unsigned k, auto first_load, auto&& move)
                             __attribute__((always_inline)) {
                constexpr int L0 = decltype(first_load)::value;
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const int x = new_x ? m / HY : m % HX, y = new_x ? m % HY : m / HX;
                    mul(xh * HX + x, yh * HY + y, X[xh][x], Y[ys][y]);
                    Gaps<MB>::reads(m, reads, read);
                    Gaps<MB>::loads(m, [&](int l) __attribute__((always_inline)) { if (l == 0) lds_destination<L0 * 1024>(d); else lds_next_destination(); },
                                    [&](int l) __attribute__((always_inline)) {
                                        if (wide) load_to_destination(ta.rsrc, ta.voff[L0 + l], k); else load_to_destination(tb.rsrc, tb.voff[L0 + l], k);
                                    });
                    Gaps<MB>::moves(m, reads == HX, move);
                }
            };
#pragma unroll
            for (int r = 0; r < HX; ++r) read_x(X[0], 0, r, 0);
#pragma unroll
            for (int r = 0; r < 2 * HY; ++r) read_y(Y[0], 0, r, 0);
            constexpr unsigned TURN = NARROW_OFF ^ (NARROW_OFF + 2 * NARROW_TILE);       // between narrow slots 0, 1 and 2, 3
            static_assert(((NARROW_OFF | (2 * NARROW_TILE + NARROW_OFF)) & (NARROW_TILE - 1)) == 0, "slots differ in the bits above a tile's");
            const unsigned kn = tb.koff(32);            // bytes from one narrow tile to the next
            const unsigned w_end = AT::dst(wide_slot(3), wid);
            unsigned d_w = AT::dst(wide_slot(2), wid);       // where unit t+2 goes
            unsigned d_n = BT::dst(narrow_slot(0), wid), d_n3 = BT::dst(narrow_slot(2), wid);    // slots of tiles 2t and 2t+2
            unsigned kw = 256, k3 = 3 * kn;              // byte offsets of unit t+2 and of tile 2t+3
            int w3 = 0;                                  // slot of wide unit t
#define READ(what) [&](int r) __attribute__((always_inline)) { what; }
#define MOVE(what) [&](int e) __attribute__((always_inline)) { what; }
#define L(n) std::integral_constant<int, n>{}
#pragma unroll 1
            for (int t = 0; t < KT; ++t) {
                const int dx = w3 == 2 ? -2 * WIDE_UNIT : WIDE_UNIT;
                pause();
                block(0, 0, 0, false, 2 * HY, READ(read_y(Y[1], 1, r, 0)), true, d_w, kw, L(2), MOVE());
                block(0, 1, 1, false, HX, READ(read_x(X[1], 1, r, 0)), false, d_n3 + NARROW_TILE, k3, L(2), MOVE());
                wait_lgkmcnt<HX>();
                wait_vmcnt<16>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (t * 64 + 160 > g.K) tb.end_at(t * 64 + 128);
                k3 += kn;
                block(1, 1, 1, true, HX, READ(read_x(X[0], 0, r, 1)), true, d_w, kw, L(4), MOVE(if (e == 1) move_address(fa.at[0], dx)));
                block(1, 0, 0, true, 2 * HY, READ(read_y(Y[1], 0, r, NARROW_TILE)), false, d_n, k3, L(0), MOVE());
                block(0, 0, 1, false, 2 * HY, READ(read_y(Y[0], 1, r, NARROW_TILE)), true, d_w, kw, L(6), MOVE());
                // (the lower half's addresses of Y, which its reads in the last block need)
                block(0, 1, 0, false, HX, READ(read_x(X[1], 1, r, 1)), false, d_n, k3, L(2),
                      MOVE(flip_address(fb.at[e], TURN)));
                wait_lgkmcnt<0>();
                wait_vmcnt<16>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (t * 64 + 256 > g.K) {
                    ta.end_at(t * 64 + 192);
                    tb.end_at(t * 64 + 160);
                }
                kw += 128;
                k3 += kn;
                d_w += WIDE_UNIT;
                if (d_w == w_end) d_w -= 3 * WIDE_UNIT;
                block(1, 1, 0, true, HX, READ(read_x(X[0], 0, r, 0)), true, d_w, kw, L(0),
                      MOVE(flip_address(fb.at[4 + e], TURN)));
                block(1, 0, 1, true, 2 * HY, READ(read_y(Y[0], 0, r, 0)), false, d_n + NARROW_TILE, k3, L(0), MOVE(if (e == 1) move_address(fa.at[1], dx)));
                w3 = w3 == 2 ? 0 : w3 + 1;
                d_n ^= TURN;
                d_n3 ^= TURN;
            }
#undef L
#undef MOVE
#undef READ
            retire();
            };
            if (__builtin_expect(active == 4, 1)) loop(std::integral_constant<int, 4>{});
            else if (active == 3) loop(std::integral_constant<int, 3>{});
            else if (active == 2) loop(std::integral_constant<int, 2>{});
            else loop(std::integral_constant<int, 1>{});
        } else if constexpr (N64) {
            // Hand-scheduled loop over steps of 64 k = eight blocks: the lower half of the wave's rows over the two chunks of
            // 32 k (blocks 0, 1 and 2, 3), then the upper half (4, 5 and 6, 7), each time against the lower and the upper half
            // of the columns.  Unit 2t holds the weights of step t, unit 2t+1 its rows, unit u lies in slot u mod 5.  All
            // weights of a step are in registers when it begins; in blocks 4 to 7 those of the next step take their places,
            // each behind the last matrix instruction that needs the old ones.  Rows are read two blocks ahead.  Two barriers
            // per step:
            //   after block 3: every wave has read the weights of step t for the last time (block 7 of step t-1), their
            //           slot receives the rows of step t+2 (blocks 4 to 6); and the weights of step t+1 have landed;
            //   after block 5: every wave has read the rows of step t for the last time, their slot receives the weights
            //           of step t+3 (block 7 and blocks 0 to 2 of the next step); and the rows of step t+1 have landed.
            // So a unit is requested 1.3 (rows) or 1.6 steps (weights) before it has to be there, and at the barriers
            // the sixteen or fourteen youngest loads of a wave may still be in flight.  (LOOP_W64 has this layout's rows in tiles of
            // 32 k, that is in half lines.  Input gradient in launches by itself, 12 x 1400 rows x 640, K = 2560: 79.6 us with
            // LOOP_W64, 73.3 so; 16 x 2048 x 2048, K = 8192: 998 and 976; 8 x 4096 x 1024, K = 4096, with the weight gradients:
            // 242 and 235 per GEMM; all with the 32 x 32 instruction.)
            frags_at(lds0 + WIDE_UNIT, lds0);
            if (first) wait_vmcnt<16 + UL / 4>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            auto loop = [&](auto tma) __attribute__((always_inline)) {
            constexpr int TMA = decltype(tma)::value;
            FB W[2][NB];
            FA R[2][4];                              // weights per chunk; rows of this pair of blocks and of the next one
            constexpr int HN = NB / 2;
            static_assert(HN == 4, "blocks of up to 4 x 4");
            // rows of a pair of blocks: half g / 2 of the wave's rows, chunk g % 2
            const auto row_frag = [&](int g, int i) __attribute__((always_inline)) { whole_a(R[g & 1][i], 0, (g >> 1) * 4 + i, g & 1); };
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < NB; ++j) whole_b(W[kk][j], 0, j, kk);
#pragma unroll
            for (int i = 0; i < (TMA < 2 ? 2 : 4); ++i) row_frag(0, i);
            fb.at[0] += 2 * WIDE_UNIT;                  // the weights of step 1
            fb.at[1] += 2 * WIDE_UNIT;
            int s5 = 0;                              // slot of the weights of step t
            const auto slot = [&](int add) __attribute__((always_inline)) { const int v = s5 + add; return v >= 5 ? v - 5 : v; };
#pragma unroll 1
            for (int t = 0; t < KT; ++t) {
                // the rows' and the weights' addresses move two units on, of five
                const int da = s5 + 1 >= 3 && s5 + 1 < 5 ? -3 * WIDE_UNIT : 2 * WIDE_UNIT;
                const int db = s5 == 1 || s5 == 2 ? -3 * WIDE_UNIT : 2 * WIDE_UNIT;
                const unsigned to_a = AT::dst(wide_slot(s5), wid), to_b2 = BT::dst(wide_slot(slot(4)), wid), to_b3 = BT::dst(wide_slot(slot(1)), wid);
                const unsigned k2 = (t + 2) * 128, k3 = k2 + 128;
                pause();
                auto block = [&](auto number) __attribute__((always_inline)) {
                    constexpr int b = decltype(number)::value, g = b >> 1, gn = (g + 1) & 3, j0 = (b & 1) * HN;
                    // rows' blocks of this block and of the next pair
                    constexpr int LOW = TMA < 2 ? 2 : 4, HIGH = TMA < 3 ? 0 : 2 * TMA - 4;
                    constexpr int nr = g < 2 ? LOW : HIGH, nn = gn < 2 ? LOW : HIGH, MB = nr * HN;      // 16, 8 or none
                    auto rows_ahead = [&](int i) __attribute__((always_inline)) { const int f = 2 * (b & 1) + i; if (f < nn) row_frag(gn, f); };
                    auto weights_ahead = [&](int j) __attribute__((always_inline)) { if constexpr (b >= 4) whole_b(W[g & 1][j0 + j], 0, j0 + j, g & 1); };
                    // behind their last reads: rows of chunk 0 are read in blocks 2, 3 and 6, 7, of chunk 1 in 0, 1 and 4, 5,
                    // weights of chunk 0 in 4, 5, of chunk 1 in 6, 7
                    auto move = [&]() __attribute__((always_inline)) {
                        if constexpr (b == 4) move_address(fa.at[0], da);
                        if constexpr (b == 6) { move_address(fa.at[1], da); move_address(fb.at[0], db); }
                        if constexpr (b == 7) move_address(fb.at[1], db);
                    };
                    constexpr bool OF_B = b < 3 || b == 7;
                    constexpr int nl = b == 3 ? 0 : b == 4 || b == 5 ? 3 : 2, l0 = b < 3 ? 2 * (b + 1) : b == 7 ? 0 : 3 * (b - 4);
                    auto pre = [&](int l) __attribute__((always_inline)) {
                        if (l == 0) lds_destination<l0 * 1024>(b < 3 ? to_b2 : b == 7 ? to_b3 : to_a);
                        else lds_next_destination();
                    };
                    auto go = [&](int l) __attribute__((always_inline)) {
                        if constexpr (OF_B) load_to_destination(tb.rsrc, tb.voff[l0 + l], b == 7 ? k3 : k2);
                        else load_to_destination(ta.rsrc, ta.voff[l0 + l], k2);
                    };
                    if constexpr (b == 4) ta.end_at(t * 64 + 128);
                    if constexpr (b == 7) tb.end_at(t * 64 + 192);
                    if constexpr (MB > 0) {
#pragma unroll
                        for (int m = 0; m < MB; ++m) {
                            mul((g >> 1) * 4 + m / HN, j0 + m % HN, R[g & 1][m / HN], W[g & 1][j0 + m % HN]);
                            if (m == 0 || m == 2) rows_ahead(m / 2);
#pragma unroll
                            for (int l = 0; l < nl; ++l) {
                                const int at = MB == 16 ? 4 + 3 * l : 1 + 2 * l;
                                if (m == at) pre(l);
                                if (m == at + 1) go(l);
                            }
                            if (m / HN == nr - 1) weights_ahead(m % HN);
                        }
                        move();
                    } else {
#pragma unroll
                        for (int i = 0; i < 2; ++i) rows_ahead(i);
#pragma unroll
                        for (int j = 0; j < HN; ++j) weights_ahead(j);
                        move();
#pragma unroll
                        for (int l = 0; l < nl; ++l) { pre(l); asm volatile("s_nop 0" ::: "memory"); go(l); }
                    }
                    if constexpr (b == 3 || b == 5) {
                        // (of block 5 the reads of rows, which come before those of four fragments of weights)
                        if constexpr (b == 3) wait_vmcnt<16>(); else { wait_lgkmcnt<HN * BR>(); wait_vmcnt<14>(); }
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                    }
                };
                block(std::integral_constant<int, 0>{});
                block(std::integral_constant<int, 1>{});
                block(std::integral_constant<int, 2>{});
                block(std::integral_constant<int, 3>{});
                block(std::integral_constant<int, 4>{});
                block(std::integral_constant<int, 5>{});
                block(std::integral_constant<int, 6>{});
                block(std::integral_constant<int, 7>{});
                s5 = slot(2);
            }
            retire();
            };
            if (__builtin_expect(active == 4, 1)) loop(std::integral_constant<int, 4>{});
            else if (active == 3) loop(std::integral_constant<int, 3>{});
            else if (active == 2) loop(std::integral_constant<int, 2>{});
            else loop(std::integral_constant<int, 1>{});
        } else if constexpr (R64) {
            // Hand-scheduled loop over steps of 64 k = four blocks of TM x TN matrix instructions (16 k each).  A
            // ring of NS stages; while block b is multiplied the fragments of block b+1 are read.  One barrier per
            // step, after block 2: every wave has read stage t for the last time (its slot then receives stage
            // t+NS) and stage t+1 has landed.  A wave's loads of stage t+NS-1 go out in block 3 of step t-1 and the
            // first blocks of step t, as early as its slot is free; at the barrier those of NS-2 stages may still be
            // in flight.
            if (first) wait_vmcnt<(NS - 2) * LPW + R64_G3>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            auto loop = [&](auto tma) __attribute__((always_inline)) {
            constexpr int TMA = decltype(tma)::value;
            constexpr int MB = TMA * TNN, FR = TMA + TNN;
            // matrix instruction m of a block is followed by its share of the block's LDS reads, then loads
            auto follow = [&](int m, int nload, auto&& read, auto&& load) __attribute__((always_inline)) {
                const int items = FR + nload;
#pragma unroll
                for (int it = 0; it < FR + LPW; ++it)
                    if (it < items && it * MB / items == m) { if (it < FR) read(it); else load(it - FR); }
            };
            bf16x8 F0[FR], F1[FR];
            auto frag = [&](int f, int kk, const char* st) __attribute__((always_inline)) -> bf16x8 {
                return f < TMA ? fa[f].read(st, kk) : fb[f - TMA].read(st + A_BYTES, kk);
            };
#pragma unroll
            for (int f = 0; f < FR; ++f) F0[f] = frag(f, 0, smem);
            int s3 = 0;                               // slot of stage t
#pragma unroll 1
            for (int t = 0; t < KT; ++t) {
                const int s3a = s3 == NS - 1 ? 0 : s3 + 1;
                char* st = smem + s3 * STAGE;
                char* st1 = smem + s3a * STAGE;
                char* st2 = smem + (s3 == 0 ? NS - 1 : s3 - 1) * STAGE;      // of stage t + NS-1
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    mfma32_pinned<C::OCC == 1>(acc32[m / TNN][m % TNN], F0[TMA + m % TNN], F0[m / TNN]);
                    follow(m, R64_G0, [&](int f) __attribute__((always_inline)) { F1[f] = frag(f, 1, st); },
                           [&](int l) __attribute__((always_inline)) { request(cur, kc, ta, tb, st2, (t + NS - 1) * BK, R64_G3 + l); });
                }
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    mfma32_pinned<C::OCC == 1>(acc32[m / TNN][m % TNN], F1[TMA + m % TNN], F1[m / TNN]);
                    follow(m, R64_G1, [&](int f) __attribute__((always_inline)) { F0[f] = frag(f, 2, st); },
                           [&](int l) __attribute__((always_inline)) { request(cur, kc, ta, tb, st2, (t + NS - 1) * BK, R64_G3 + R64_G0 + l); });
                }
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    mfma32_pinned<C::OCC == 1>(acc32[m / TNN][m % TNN], F0[TMA + m % TNN], F0[m / TNN]);
                    follow(m, 0, [&](int f) __attribute__((always_inline)) { F1[f] = frag(f, 3, st); },
                           [&](int l) __attribute__((always_inline)) { request(cur, kc, ta, tb, st2, (t + NS - 1) * BK, 0); });
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wait_vmcnt<(NS - 2) * LPW>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    mfma32_pinned<C::OCC == 1>(acc32[m / TNN][m % TNN], F1[TMA + m % TNN], F1[m / TNN]);
                    follow(m, R64_G3, [&](int f) __attribute__((always_inline)) { F0[f] = frag(f, 0, st1); },
                           [&](int l) __attribute__((always_inline)) { request(cur, kc, ta, tb, st, (t + NS) * BK, l); });
                }
                s3 = s3a;
            }
            };
            if (TM == 1 || active == 1) loop(std::integral_constant<int, 1>{});
            else if (TM == 2 || active == 2) loop(std::integral_constant<int, TM < 2 ? 1 : 2>{});
            else if (active == 3) loop(std::integral_constant<int, TM < 3 ? 1 : 3>{});
            else loop(std::integral_constant<int, TM < 4 ? 1 : 4>{});
            retire();
        } else {
            // Hand-scheduled loop over tiles of 32 k = one chunk; the ring holds NS tiles, of which up to NS - 1 are in flight
            // towards a workgroup.  Every LDS read and every load into LDS sits between two matrix instructions (with one
            // wave per SIMD nothing else hides a stall).
            int st = SB;
            if constexpr (QUAD) {
                // 256 x 256: four blocks (see above), the rows as X, the columns as Y.  In iteration t blocks 0 and 1 read the
                // upper halves of tile t and request the second half of tile t+NS-1; then the wave waits for its part of
                // tile t+1 and meets the others (their parts have landed too, and nobody reads stage t any more); blocks 2
                // and 3 read the lower halves of tile t+1 and request the first half of tile t+NS into stage t.
                static_assert(RB == 8 && NB == 8 && LPW == 8, "four blocks of 4 x 4 with two loads each");
                frags_at(lds0 + SB * STAGE, lds0 + SB * STAGE + A_BYTES);
                if (first) wait_vmcnt<(NS - 2) * LPW + PIPE_EARLY>();         // tile 0 is in (later tiles: waited for at the handover)
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                FA X[2][4];
                FB Y[2][4];
                // (an odd number of tiles begins with the second half of an iteration; Y's lower half is read into both places rather
                // than into one of them, which would cost copies of it behind the branch)
                bool skip = KT & 1;
#pragma unroll
                for (int f = 0; f < 4; ++f) whole_a(X[0][f], 0, f, 0);
#pragma unroll
                for (int f = 0; f < 4; ++f) whole_b(Y[0][f], 0, f, 0);
#pragma unroll
                for (int f = 0; f < 4; ++f) whole_b(Y[1][f], 0, f, 0);
                int kt = 0;
                // y: the place of the lower half of Y
                auto tile = [&](auto y) __attribute__((always_inline)) {
                    constexpr int LO = decltype(y)::value, UP = LO ^ 1;
                    char* cs = smem + st * STAGE;
                    char* prv = smem + ((st == 0) ? NS - 1 : st - 1) * STAGE;
                    const int next = st == NS - 1 ? (1 - NS) * STAGE : STAGE;
                    auto block = [&](int xh, int yh, int ys, bool new_x, int reads, auto&& read, const char* to, auto first_load, auto&& move) __attribute__((always_inline)) {
                        constexpr int L0 = decltype(first_load)::value;
#pragma unroll
                        for (int m = 0; m < 16; ++m) {
                            const int x = new_x ? m / 4 : m % 4, y = new_x ? m % 4 : m / 4;
                            mul(xh * 4 + x, yh * 4 + y, X[xh][x], Y[ys][y]);
                            if (L0 == 0 && m == 7) { advance(cur, kc, ta, tb); settle(ta, tb); }
                            Gaps<16>::reads(m, reads, read);
                            Gaps<16>::loads(m, [&](int l) __attribute__((always_inline)) {
                                                if (l) lds_next_destination();
                                                else if constexpr (L0 < AT::NI) lds_destination<L0 * 1024>(AT::dst(to, wid));
                                                else lds_destination<A_BYTES + (L0 - AT::NI) * 1024>(BT::dst(to, wid));
                                            },
                                            [&](int l) __attribute__((always_inline)) { go(ta, tb, L0 + l); });
                            Gaps<16>::moves(m, false, move);
                        }
                    };
#define READ(what) [&](int r) __attribute__((always_inline)) { what; }
#define MOVE(what) [&](int e) __attribute__((always_inline)) { what; }
#define L(n) std::integral_constant<int, n>{}
                    pause();
                    block(0, 0, LO, false, 4 * BR, READ(frag_b(Y[UP][r / BR], 0, 4 + r / BR, 0, r % BR)), prv, L(4), MOVE(move_address(fa.at[e], next)));
                    block(0, 1, UP, false, 4 * AR, READ(frag_a(X[1][r / AR], 0, 4 + r / AR, 0, r % AR)), prv, L(6), MOVE(move_address(fb.at[4 + e], next)));
                    wait_lgkmcnt<0>();                                     // this wave no longer reads stage t
                    wait_vmcnt<(NS - 2) * LPW>();                          // its part of tile t+1 is in
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    block(1, 1, UP, true, 4 * AR, READ(frag_a(X[0][r / AR], 0, r / AR, 0, r % AR)), cs, L(0), MOVE(move_address(fb.at[e], next)));
                    block(1, 0, LO, true, 4 * BR, READ(frag_b(Y[UP][r / BR], 0, r / BR, 0, r % BR)), cs, L(2), MOVE(move_address(fa.at[4 + e], next)));
#undef L
#undef MOVE
#undef READ
                    st = (st + 1 == NS) ? 0 : st + 1;
                    ++kt;
                };
#pragma unroll 1
                while (kt < KT) {
                    if (!skip) tile(std::integral_constant<int, 0>{});
                    skip = false;
                    tile(std::integral_constant<int, 1>{});
                }
            } else {
            // Smaller tiles: two blocks of TM x TN matrix instructions.  In iteration t block 0 multiplies k 0..15 of tile t, reads
            // k 16..31 of it and requests the second half of tile t+NS-1; then the wave waits for its part of tile t+1 and meets
            // the others (their parts have landed too, and nobody reads stage t any more); block 1 multiplies k 16..31, reads
            // k 0..15 of tile t+1 and requests the first half of tile t+NS into stage t.
            constexpr int MB = TM * TNN;                 // matrix instructions per block
            constexpr int FR = TM + TNN;                 // fragments per block: A rows first, then B columns
            constexpr int LH = LPW / 2;                  // loads of a tile requested one block earlier than the rest
            // What follows matrix instruction m of a block, spread evenly: LDS reads first, then loads.
            constexpr int LMAX = LPW - LH;
            auto follow = [&](int m, int nload, auto&& read, auto&& load) __attribute__((always_inline)) {
                const int items = FR + nload;
#pragma unroll
                for (int it = 0; it < FR + LMAX; ++it) {
                    if (it < items && it * MB / items == m) {
                        if (it < FR) read(it);
                        else load(it - FR);
                    }
                }
            };
            if (first) wait_vmcnt<(NS - 2) * LPW + LH>();                 // tile 0 is in (later tiles: waited for at the handover)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            bf16x8 F0[FR], F1[FR];
#pragma unroll
            for (int f = 0; f < FR; ++f)
                F0[f] = f < TM ? fa[f].read(smem + SB * STAGE, 0) : fb[f - TM].read(smem + SB * STAGE + A_BYTES, 0);
#pragma unroll 1
            for (int kt = 0; kt < KT; ++kt) {
                char* cs = smem + st * STAGE;
                const int stn = (st + 1 == NS) ? 0 : st + 1;
                const int stp = (st == 0) ? NS - 1 : st - 1;
                char* nxt = smem + stn * STAGE;
                char* prv = smem + stp * STAGE;
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    mfma32_pinned<C::OCC == 1>(acc32[m / TNN][m % TNN], F0[TM + m % TNN], F0[m / TNN]);
                    follow(m, LPW - LH,
                           [&](int f) __attribute__((always_inline)) { F1[f] = f < TM ? fa[f].read(cs, 1) : fb[f - TM].read(cs + A_BYTES, 1); },
                           [&](int l) __attribute__((always_inline)) { request(cur, kc, ta, tb, prv, (kt + NS - 1) * BK, LH + l); });
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave no longer reads stage t
                wait_vmcnt<(NS - 2) * LPW>();                          // its part of tile t+1 is in
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    mfma32_pinned<C::OCC == 1>(acc32[m / TNN][m % TNN], F1[TM + m % TNN], F1[m / TNN]);
                    follow(m, LH,
                           [&](int f) __attribute__((always_inline)) { F0[f] = f < TM ? fa[f].read(nxt, 0) : fb[f - TM].read(nxt + A_BYTES, 0); },
                           [&](int l) __attribute__((always_inline)) { request(cur, kc, ta, tb, cs, (kt + NS) * BK, l); });
                }
                st = stn;
            }
            }
            retire();
        }
        wait_vmcnt<0>();                             // nothing of this workgroup is in flight into LDS any more
        __builtin_amdgcn_s_barrier();                // and every wave is done reading the ring
        asm volatile("" ::: "memory");

        // ---- the tile after this one ------------------------------------------------------
        TileCoord nx;
        // (beside the five-unit loop, and in GeLU-backward's passes, there are no registers to carry the next tile's offsets through
        // the epilogue: it forms them where they are used, from a lane number that the compiler cannot tell from another)
        constexpr bool LATE_BIND = N64 || (EPI == EPI_DGELU && C::OCC == 1);
        AT ta2;
        BT tb2;
        auto bind_again = [&]() __attribute__((always_inline)) {
            int l = lane;
            asm volatile("" : "+v"(l));
            bind(nx, ta2, tb2, l);
        };
        KCursor kc2 = {};
        int vn = -1;
        if constexpr (!ONE) {
            vn = next_tile(vb + step, nx);
            if (vn < 0) nx = cur;                    // (bound all the same, and never used)
            if constexpr (!LATE_BIND) bind(nx, ta2, tb2, lane);
        }

        // ---- epilogue -----------------------------------------------------------------------
        // An MFMA accumulator holds four consecutive columns of one row per lane (row = lane & 15,
        // columns 4 * (lane / 16) ..; S32: row = lane & 31, four such groups), which would make every global access a 8- or 16-byte
        // piece of 16 different rows.  Each wave therefore passes its 32 x WN blocks through a
        // private LDS region (float, 16-byte chunks XOR-swizzled by row) and picks them up
        // with eight consecutive columns per lane, so that eight lanes cover a whole line of
        // a row: all global reads and writes of the epilogue are 16 or 32 bytes per lane,
        // row-contiguous.  They go through buffer descriptors that end after the last valid
        // row, so there is no branch: out-of-range reads give zero, out-of-range writes are
        // dropped, and all reads of a 32-row pass are issued before the arithmetic starts.
        // A pass moves 32 rows x CW columns of the wave's block (CW = the block's width, or 64 where the
        // staging region is one ring unit).
        constexpr int CPRW = CW / 8;                 // 8-column pieces per row of a pass
        constexpr int SW = CW >= 64 ? 15 : CW / 4 - 1;       // the row bits that the 16-byte chunks of a staged row are swizzled by
        constexpr int NPIECE = 32 * CPRW / 64;       // pieces per lane
        constexpr int NCH = WN / CW, TJ = CW / 16;   // passes per 32 rows; 16-column accumulator blocks per pass
        constexpr int NPASS = TM * NCH;
        float* stage = reinterpret_cast<float*>(smem + C::STAGING_OFF + wid * (32 * CW * 4));
        constexpr int CES = (EPI == EPI_ACCUM_F32 || EPI == EPI_STORE_F32) ? 4 : 2;   // bytes per output element
        // The descriptors begin at the tile's first row: an expert's float gradients may exceed 2 GiB, and offset
        // OOB_OFFSET would then be an element of theirs.
        // (scattered rows: the whole output matrix, every row of which some tile may write)
        const int trows = min(BM, Mdim - m0);
        const char* Cbase = EPI == EPI_SCATTER ? (const char*)g.C
                                               : (const char*)g.C + ((size_t)e * g.c_estride + (size_t)m0 * g.ldc + (LAY == GEMM_TN ? 0 : q * g.c_pstride)) * CES;
        const __amdgpu_buffer_rsrc_t rC = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(Cbase), 0,
            (unsigned)(((size_t)((EPI == EPI_SCATTER ? g.c_row_limit : trows) - 1) * g.ldc + g.N) * CES), 0x00020000);
        const int* crows = g.c_rows ? g.c_rows + (size_t)er * g.Cp : nullptr;
        const bf16_t* Zbase = g.Z ? (const bf16_t*)g.Z + ((size_t)e * g.Cp + m0) * g.ldz + q * g.z_pstride : nullptr;
        const __amdgpu_buffer_rsrc_t rZ = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t*>(Zbase), 0, Zbase ? (unsigned)(((size_t)(trows - 1) * g.ldz + g.N) * 2) : 0u, 0x00020000);
        const float* wbase = g.slot_w ? g.slot_w + (size_t)er * g.Cp : nullptr;
        // What a pass reads from memory (the pre-activation and row weight for GeLU-backward, the old
        // sums for float accumulation) is requested one pass ahead.
        constexpr bool READS = (EPI == EPI_DGELU || EPI == EPI_ACCUM_F32 || EPI == EPI_SCATTER);
        struct PassIn { uint4 zin[NPIECE]; float4 cin0[NPIECE], cin1[NPIECE]; float wrow[NPIECE]; int crow[NPIECE]; };
        // Piece t of a lane: row RSTEP*t + prow of the pass, columns 8*c8 .. 8*c8 + 7.  Addresses are one vector
        // offset per column block (out of range: past the descriptor, and it stays there with any step added) and a
        // wave-uniform step per pass and piece, added to the vector offset.  (Not handed over as the scalar offset of
        // the access: that one is no part of the bounds check, and a step beyond the last valid row, as in every last
        // tile row, would reach whatever lies behind.)
        constexpr int RSTEP = 64 / CPRW;
        const int prow = lane / CPRW, c8 = lane % CPRW;
        unsigned baseC[NCH], baseZ[NCH];
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            const int n = n0 + wn * WN + ch * CW + c8 * 8;
            baseC[ch] = n < g.N ? (unsigned)(prow * g.ldc + n) * CES : OOB_OFFSET;
            baseZ[ch] = n < g.N ? (unsigned)(prow * g.ldz + n) * 2u : OOB_OFFSET;
        }
        auto row_of = [&](int ps, int t) __attribute__((always_inline)) { return block_row(ps / NCH) + RSTEP * t; };   // wave-uniform
        auto offC = [&](int ps, int t) __attribute__((always_inline)) { return baseC[ps % NCH] + (unsigned)(row_of(ps, t) * g.ldc) * CES; };
        auto offZ = [&](int ps, int t) __attribute__((always_inline)) { return baseZ[ps % NCH] + (unsigned)(row_of(ps, t) * g.ldz) * 2u; };
        // row weights, output rows and row dots through descriptors too: nothing below branches on the row
        const unsigned row4 = (unsigned)(m0 + prow) * 4u;
        const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wbase), 0, wbase ? Mdim * 4 : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rR = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(crows), 0, crows ? Mdim * 4 : 0, 0x00020000);
        float* dwbase = g.dw_part ? g.dw_part + (size_t)e * g.Cp * g.dw_parts + q * g.dw_pstride : nullptr;
        const __amdgpu_buffer_rsrc_t rD = __builtin_amdgcn_make_buffer_rsrc(dwbase, 0, dwbase ? Mdim * g.dw_parts * 4 : 0, 0x00020000);
        // Float outputs: a lane's two 16-byte halves of "piece" t are units 2t and 2t+1 of a numbering in which the
        // 64 lanes of one store (or load) cover whole rows of the pass - 4 columns per lane, CW/4 lanes per row - so
        // that every such instruction moves whole 128-byte lines (8 columns per lane would leave each instruction
        // with every other 16 bytes).  Unit u of a lane is UROWS*u rows below its unit 0, in the same columns: one
        // vector offset per pass and a constant step, in the vector offset as above.  (For the stores there is a
        // second reason: behind a 16-byte store with a scalar offset register the compiler may overwrite the store's
        // data registers in the very next instruction, and then the last lanes of the store have been seen to write
        // the new contents.)
        constexpr int ULANES = CW / 4, UROWS = 64 / ULANES;
        const int urow = lane / ULANES, uc4 = lane % ULANES;
        auto unit0 = [&](int ps) -> unsigned {
            const int n = n0 + wn * WN + (ps % NCH) * CW + uc4 * 4;
            return n < g.N ? (unsigned)((block_row(ps / NCH) + urow) * g.ldc + n) * 4u : OOB_OFFSET;
        };
        const unsigned ustep = (unsigned)(UROWS * g.ldc) * 4u;      // bytes from one unit of a lane to the next
        auto request_pass = [&](int ps, PassIn& in) {
#pragma unroll
            for (int t = 0; t < NPIECE; ++t) {
                if constexpr (EPI == EPI_DGELU)
                    in.zin[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rZ, offZ(ps, t), 0, 0));
                if constexpr (EPI == EPI_DGELU || EPI == EPI_SCATTER)
                    in.wrow[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rW, row4 + row_of(ps, t) * 4, 0, 0));
                if constexpr (EPI == EPI_SCATTER)
                    in.crow[t] = (int)__builtin_amdgcn_raw_buffer_load_b32(rR, row4 + row_of(ps, t) * 4, 0, 0);
                if constexpr (EPI == EPI_ACCUM_F32) {
                    const unsigned ob = unit0(ps);
                    in.cin0[t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rC, ob + (2 * t) * ustep, 0, 0));
                    in.cin1[t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rC, ob + (2 * t + 1) * ustep, 0, 0));
                }
            }
        };
        // (with two workgroups on the CU the other one covers the wait, and the registers are short)
        constexpr int PB = C::OCC == 1 ? 2 : 1;
        PassIn pin[PB];
        if constexpr (READS && PB == 2) request_pass(0, pin[0]);
        // the row of every 32 whose dot this lane ends up with, and where it goes
        const int dw_row = RSTEP * (((c8 >> 2) & 1) * 2 + ((c8 >> 1) & 1)) + prow;
        const unsigned dw_lane = (unsigned)((m0 + dw_row) * g.dw_parts + tn * C::WAVES_N + wn) * 4u;
        float dots[TM];                              // its finished rows, where a column block is two waves wide
        float dotacc[NPIECE];                        // GeLU-backward: <gelu(Z), G> of a row over the passes of its 32 rows
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) {
            const int i = ps / NCH, ch = ps % NCH;
            // no rows in the second half (wave-uniform; tested once, so that the scheduler sees long stretches)
            if (ALT && TM > 1 && ps == NPASS / 2 && active <= TM / 2) break;
            if constexpr (READS && PB == 1) request_pass(ps, pin[0]);
            if constexpr (S32) {
#pragma unroll
                for (int jj = 0; jj < CW / 32; ++jj)
#pragma unroll
                    for (int g4 = 0; g4 < 4; ++g4) {
                        const floatx16& a = acc32[i][ch * (CW / 32) + jj];
                        const int erow = lane & 31, cch = (jj * 32 + g4 * 8 + (lane >> 5) * 4) >> 2;
                        *reinterpret_cast<float4*>(stage + erow * CW + ((cch ^ (erow & SW)) << 2)) =
                            make_float4(a[g4 * 4], a[g4 * 4 + 1], a[g4 * 4 + 2], a[g4 * 4 + 3]);
                    }
            } else
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int jj = 0; jj < TJ; ++jj) {
                    const floatx4 a = acc[2 * i + h][ch * TJ + jj];
                    const int erow = h * 16 + (lane & 15), cch = jj * 4 + (lane >> 4);
                    *reinterpret_cast<float4*>(stage + erow * CW + ((cch ^ (erow & SW)) << 2)) = make_float4(a[0], a[1], a[2], a[3]);
                }
            if constexpr (READS && PB == 2) {
                if (ps + 1 < NPASS) request_pass(ps + 1, pin[(ps + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);   // (the scheduler would sink them to their uses)
            }
            const PassIn& in = pin[ps & (PB - 1)];
            // all LDS reads of the pass before its arithmetic: one round trip through LDS, not one per piece
            // (float accumulation keeps the old sums of two passes in registers and has none left for that)
            constexpr bool HOIST = EPI != EPI_ACCUM_F32;
            float4 lo[NPIECE], hi[NPIECE];
            auto read_piece = [&](int t) {
                if constexpr (CES == 4) {
                    const int r0 = urow + UROWS * (2 * t), r1 = r0 + UROWS;
                    lo[t] = *reinterpret_cast<const float4*>(stage + r0 * CW + ((uc4 ^ (r0 & SW)) << 2));
                    hi[t] = *reinterpret_cast<const float4*>(stage + r1 * CW + ((uc4 ^ (r1 & SW)) << 2));
                } else {
                    const int row = RSTEP * t + prow;
                    lo[t] = *reinterpret_cast<const float4*>(stage + row * CW + (((2 * c8) ^ (row & SW)) << 2));
                    hi[t] = *reinterpret_cast<const float4*>(stage + row * CW + (((2 * c8 + 1) ^ (row & SW)) << 2));
                }
            };
            if constexpr (HOIST) {
#pragma unroll
                for (int t = 0; t < NPIECE; ++t) read_piece(t);
            }
#pragma unroll
            for (int t = 0; t < NPIECE; ++t) {
                if constexpr (!HOIST) read_piece(t);
                float v[8] = {lo[t].x, lo[t].y, lo[t].z, lo[t].w, hi[t].x, hi[t].y, hi[t].z, hi[t].w};
                if constexpr (EPI == EPI_STORE) {
                    uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, o), rC, offC(ps, t), 0, 0);
                } else if constexpr (EPI == EPI_SCATTER) {
                    // the row's place in the output and its weight; rows and columns out of range are dropped
                    const float w = in.wrow[t];
                    const int n = n0 + wn * WN + (ps % NCH) * CW + c8 * 8;
                    const unsigned oS = (m0 + row_of(ps, t) + prow < Mdim && n < g.N) ? (unsigned)(in.crow[t] * g.ldc + n) * 2u : OOB_OFFSET;
                    uint4 o = make_uint4(pack_bf16x2(w * v[0], w * v[1]), pack_bf16x2(w * v[2], w * v[3]),
                                         pack_bf16x2(w * v[4], w * v[5]), pack_bf16x2(w * v[6], w * v[7]));
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, o), rC, oS, 0, 0);
                } else if constexpr (EPI == EPI_GELU) {
                    // (the activation is taken of the rounded pre-activation, unpacked from what is stored)
                    const uint4 oz = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                    float z[8], a[8];
                    Unit8::to_float(oz, z);
#pragma unroll
                    for (int q = 0; q < 8; ++q) a[q] = gelu_fast_f(z[q]);
                    uint4 oa = make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]), pack_bf16x2(a[6], a[7]));
                    if (Zbase) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, oz), rZ, offZ(ps, t), 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, oa), rC, offC(ps, t), 0, 0);
                } else if constexpr (EPI == EPI_DGELU) {
                    float z[8], dz[8], a[8];
                    Unit8::to_float(in.zin[t], z);
                    const float w = in.wrow[t];
                    float dot = ch == 0 ? 0.0f : dotacc[t];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        float gq, dg;
                        gelu_both_fast_f(z[q], &gq, &dg);
                        // columns out of range read z = 0 and an accumulator of 0: nothing to add; rows out of
                        // range are never written below
                        dot = fmaf(gq, v[q], dot);
                        a[q] = w * gq;
                        dz[q] = w * v[q] * dg;
                    }
                    dotacc[t] = dot;
                    uint4 od = make_uint4(pack_bf16x2(dz[0], dz[1]), pack_bf16x2(dz[2], dz[3]), pack_bf16x2(dz[4], dz[5]), pack_bf16x2(dz[6], dz[7]));
                    uint4 oa = make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]), pack_bf16x2(a[6], a[7]));
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, od), rC, offC(ps, t), 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, oa), rZ, offZ(ps, t), 0, 0);
                } else if constexpr (EPI == EPI_STORE_F32) {
                    const unsigned ob = unit0(ps);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, lo[t]), rC, ob + (2 * t) * ustep, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, hi[t]), rC, ob + (2 * t + 1) * ustep, 0, 0);
                } else {
                    const unsigned ob = unit0(ps);
                    float4 o0 = in.cin0[t], o1 = in.cin1[t];
                    o0.x += v[0]; o0.y += v[1]; o0.z += v[2]; o0.w += v[3];
                    o1.x += v[4]; o1.y += v[5]; o1.z += v[6]; o1.w += v[7];
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, o0), rC, ob + (2 * t) * ustep, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, o1), rC, ob + (2 * t + 1) * ustep, 0, 0);
                }
            }
            if constexpr (EPI == EPI_DGELU) {
                if (g.dw_part && ch == NCH - 1) {
                    // The row dots of the 32 rows are spread over the eight lanes of each row in four pieces.  Folding
                    // the lanes splits the pieces between them (lane c8 ends up with the total of piece dw_t), so that
                    // four shuffles and one store take the place of twelve and four (large layer: 30 us of a 1230 us
                    // launch).
                    static_assert(NPIECE == 4 && CPRW == 8, "four pieces over eight lanes");
                    const bool up4 = (c8 & 4) != 0, up2 = (c8 & 2) != 0;
                    const float k0 = (up4 ? dotacc[2] : dotacc[0]) + __shfl_xor(up4 ? dotacc[0] : dotacc[2], 4, 64);
                    const float k1 = (up4 ? dotacc[3] : dotacc[1]) + __shfl_xor(up4 ? dotacc[1] : dotacc[3], 4, 64);
                    const float k2 = (up2 ? k1 : k0) + __shfl_xor(up2 ? k0 : k1, 2, 64);
                    const float dot = k2 + __shfl_xor(k2, 1, 64);
                    if constexpr (WN == DW_COLS) {
                        if ((c8 & 1) == 0)
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, dot), rD,
                                                                  dw_lane + block_row(i) * g.dw_parts * 4, 0, 0);
                    } else {
                        dots[i] = dot;           // half a column block: added to the other wave's below
                    }
                }
            }
            // the next tile's first operand tiles start their trip once the first pass is through
            // (earlier, and this pass's own reads would have to wait behind them)
            if constexpr (!ONE) {
                if constexpr (LATE_BIND) { if (ps == 0) bind_again(); }
                if (ps == 0 && vn >= 0) issue_early(nx, kc2, ta2, tb2);
            }
        }
        if constexpr (EPI == EPI_DGELU && WN != DW_COLS) {
            if (g.dw_part) {
                // A column block of the row dots is the width of the two neighbouring waves: the right one hands its
                // rows' sums to the left one through its own staging region, which nobody else touches.
                static_assert(C::WAVES_N == 2 && 2 * WN == DW_COLS && BN == DW_COLS, "one column block per tile");
                if (wn == 1 && (c8 & 1) == 0) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) stage[i * 32 + dw_row] = dots[i];
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (wn == 0 && (c8 & 1) == 0) {
                    const float* right = stage + 32 * CW;
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int m = m0 + block_row(i) + dw_row;
                        if (m < Mdim) {
                            float* at = dwbase + (size_t)m * g.dw_parts + tn;
                            at[0] = dots[i] + right[i * 32 + dw_row];
                            if (tn == tiles_n - 1 && tn + 1 < g.dw_parts) at[1] = 0.0f;     // blocks come in pairs
                        }
                    }
                }
            }
        }
        if (ONE || vn < 0) break;
        // Everything this wave has in flight is through: the next tile's first operand tiles have
        // landed and the epilogue's stores are written.  (Counting on the stores being younger than
        // the loads would save waiting for the last of them, but the main loop's third wait would
        // wait for them anyway: vmcnt retires in order.)
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();                // every wave is done with the staging stages
        asm volatile("" ::: "memory");
        if constexpr (LATE_BIND) bind_again();
        issue_late(nx, kc2, ta2, tb2);
        kc = kc2;
        if constexpr (!REBIND) { ta = ta2; tb = tb2; }
        cur = nx;
        vb = vn;
        first = false;
    }
}

// Persistent workgroups: the grid has one workgroup per CU (two where two fit), and workgroup b works through
// the tiles b, b + grid, b + 2 grid, ...
template <int LAY, int EPI, typename C>
__global__ __launch_bounds__(C::THREADS) __attribute__((amdgpu_waves_per_eu(C::OCC, C::OCC)))
void gemm_bf16_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    gemm_tiles<LAY, EPI, C, false>(g, tiles_m, tiles_n, number_tiles<LAY, EPI, C>(g, tiles_m, tiles_n, threadIdx.x & 63),
                                   (int)blockIdx.x, (int)gridDim.x);
}

// What follows GeLU-backward - the input gradient dZ W1^T (NT) and the two weight gradients (TN), which do not depend
// on each other - in one launch, a tile per workgroup: whichever CU is free takes the next one.  Alone, each
// of the three ends in a round of tiles that leaves most of the chip idle (a launch of 128 or 144 tiles of 256 x 256 all
// the way through), and a tile's time varies with the rows of its expert.  The tiles that take longest,
// by the estimate that the tile shapes are chosen with, come first.  A workgroup's first operand loads are not covered by another tile's epilogue as in
// the persistent launches (2 to 3 us of a tile), so this is for launches of a few rounds.
struct BackwardArgs {
    GemmArgs d;                          // input gradient; not there if tiles_d == 0
    GemmArgs w[2];                       // weight gradients
    int tiles_dm, tiles_dn, tiles_wm[2], tiles_wn[2];
    int w_first;                         // the weight gradients' tiles come first
    GateDlArgs gate;                     // in the blocks after the last tile (blocks = 0: not there)
};
template <int EPI, typename CN, typename CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CT::OCC, CT::OCC)))
void gemm_bf16_backward_kernel(BackwardArgs a) {
    static_assert(CN::OCC == CT::OCC && CN::THREADS == 256 && CT::THREADS == 256 && GATE_THREADS == 256 && GATE_DL_LDS <= CT::LDS_BYTES,
                  "tiles of one launch share its shape");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63;
    auto space = [](const TileNumbers& t) { return (t.nblocks + 7) & ~7; };     // (a number keeps its place modulo the eight XCDs)
    int b = blockIdx.x, q = 0;                             // q: weight gradient, or 2: input gradient, 3: beyond both
    TileNumbers t = {};
    if (a.tiles_dm > 0 && !a.w_first) {
        t = number_tiles<GEMM_NT, EPI_STORE, CN>(a.d, a.tiles_dm, a.tiles_dn, lane);
        if (b < space(t)) q = 2;
        else b -= space(t);
    }
    if (q == 0) {
        t = number_tiles<GEMM_TN, EPI, CT>(a.w[0], a.tiles_wm[0], a.tiles_wn[0], lane);
        if (b >= space(t)) {
            b -= space(t);
            q = 1;
            t = number_tiles<GEMM_TN, EPI, CT>(a.w[1], a.tiles_wm[1], a.tiles_wn[1], lane);
            if (b >= space(t)) {
                b -= space(t);
                q = 3;
                if (a.w_first) {
                    t = number_tiles<GEMM_NT, EPI_STORE, CN>(a.d, a.tiles_dm, a.tiles_dn, lane);
                    if (b < space(t)) q = 2;
                    else b -= space(t);
                }
            }
        }
    }
    if (q == 2) {
        gemm_tiles<GEMM_NT, EPI_STORE, CN, true>(a.d, a.tiles_dm, a.tiles_dn, t, b, 1 << 30);
        return;
    }
    if (q == 3) {
        // the gate's dL, which only needs the row dots of the GeLU-backward GEMM: a launch of its own takes 4 to 6 us
        if (b < a.gate.blocks) gate_dl(a.gate, b, smem);
        return;
    }
    gemm_tiles<GEMM_TN, EPI, CT, true>(a.w[q], a.tiles_wm[q], a.tiles_wn[q], t, b, 1 << 30);
}

// Tile shapes in use.  The first three cover 256 x 256 per workgroup with four waves of 128 x 128, one per SIMD.
//   CfgW   two-ring loop: NN.  A request for half a 128-byte line costs the L1 as much as one for a whole line, and the
//          loops' speed follows the number of requests; here every request is a whole line.
//   CfgN   five-unit loop: NT, both epilogues; every request is a whole line.  (GeLU-backward in the two-ring loop, its rows
//          in half lines: 1.58 us a step against 1.39, 32 768 rows x 8192, K = 2048.)
//   Cfg4   ring of 5 x 32 k: the weight-gradient GEMMs (TN), whose two operands are N-contiguous
//          and come in whole lines anyway.
// (Shapes with two waves of 128 x 64 per SIMD - TileCfg<256, 256, 32, 5, 2, 4, 2, LOOP_PIPE32> - ran the GeLU
// epilogues faster and the main loops slower, reading half as much again from LDS; with the cheaper GeLU
// arithmetic the four-wave shapes won everywhere, measured with the 32 x 32 instruction.)
typedef TileCfg<256, 256, 32, 5, 2, 2, 1, LOOP_PIPE32> Cfg4;
typedef TileCfg<256, 256, 64, 3, 2, 2, 1, LOOP_W64> CfgW;
typedef TileCfg<256, 256, 64, 3, 2, 2, 1, LOOP_N64> CfgN;
template <int LAY, int EPI> struct CfgFor { typedef CfgW type; };
template <int EPI> struct CfgFor<GEMM_NT, EPI> { typedef CfgN type; };
template <int EPI> struct CfgFor<GEMM_TN, EPI> { typedef Cfg4 type; };
// Smaller tiles for launches that 256 x 256 leaves too few of, all layouts (the flat one: NN, NT):
//   CfgM   256 x 128, waves of 128 x 64, three 64-k stages of both operands, so that every request is a whole line.
//          A step takes 0.68 us alone against 1.0-1.4 for the large tile's, bound by the loads (48 KB per step, 96 KB
//          in flight) where the chip is full: 8 x 1024 rows, N = 1024, K = 4096: 72 us in 256 tiles, 107 in 128.
//   CfgS   128 x 128, waves of 64 x 64, five 32-k stages, two workgroups per CU: one's epilogue runs beside the
//          other's loop.  Its loop is bound by LDS (192 bytes per cycle wanted, 128 there).  8 x 512 rows, N = 2048,
//          K = 512, GeLU: 22 us against 25 in 256 x 256; N = 512, K = 2048: 22 against 38.
//   CfgT   64 x 128, waves of 32 x 64, six 64-k stages: few rows against long K, where a CU should have many bytes of
//          the weights in flight.  8 x 16 rows, N = 1024, K = 4096: 41 us against 60 (67 MB of weights: 13 us).
typedef TileCfg<256, 128, 64, 3, 2, 2, 1, LOOP_R64> CfgM;
typedef TileCfg<128, 128, 32, 5, 2, 2, 2, LOOP_PIPE32> CfgS;
typedef TileCfg<64, 128, 64, 6, 2, 2, 1, LOOP_R64> CfgT;
//   CfgT2  CfgT with three stages, two workgroups per CU: beside CfgS in one launch.
typedef TileCfg<64, 128, 64, 3, 2, 2, 2, LOOP_R64> CfgT2;
//   CfgU   64 x 64, waves of 32 x 32, ten 64-k stages, for plain stores over a long K of few tiles (few_tiles): their
//          steps in CfgT wait for loads that were requested five steps before.  8 rows of 16, N = 1024, K = 4096: 22 us in 64
//          tiles of CfgT, 13 in 128; 8 x 128 rows: 38.9 and 29.3.
typedef TileCfg<64, 64, 64, 10, 2, 2, 1, LOOP_R64> CfgU;

int gemm_bf16_dw_parts(int H) { return (H + 2 * DW_COLS - 1) / (2 * DW_COLS) * 2; }

template <int LAY, int EPI, typename C>
static moe_status launch_one(const GemmArgs& a, hipStream_t s) {
    const int Mmax = (LAY == GEMM_TN) ? a.Mo : a.Cp;
    const int tiles_m = (Mmax + C::BM - 1) / C::BM, tiles_n = (a.N + C::BN - 1) / C::BN;
    int nblocks = launch_experts(a) * tiles_m * tiles_n;
    nblocks = (nblocks + 7) / 8 * 8;
    // a full grid: one workgroup per CU (times TileCfg::OCC; together they fill a CU's LDS)
    int full = compute_units() - (a.free_cus + 7) / 8 * 8;
    if (full < 8) full = 8;
    full *= C::OCC;
    const int grid = nblocks < full ? nblocks : full;
    constexpr int lds = C::LDS_BYTES;
    auto kern = gemm_bf16_kernel<LAY, EPI, C>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        attr_done = true;
    }
    {
        ProfScope ps(gemm_prof_kind(LAY, EPI), s, a.np > 1 ? a.np : 1);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(C::THREADS), lds, s, a, tiles_m, tiles_n);
    }
    count_launch(LC_GEMM, a.np > 1 ? a.np : 1);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// Which tile a launch uses: the one whose estimated time is least.  Large tiles multiply fastest (per 256 x 256 x
// 64 on one CU: 1.1 to 1.5 us in one large tile, 1.7 in two half-size ones, 1.8 to 2.6 in four small ones two at a
// time, 3.5 in eight flat ones), but a launch with fewer tiles than the chip has CUs, or a few more than a multiple
// of that, leaves CUs idle, and a workgroup's epilogue is only covered where two workgroups share a CU.  The estimate
// counts the rounds of tiles over the workgroups; the times (us) of a 64-k step per layout (NN, NT, TN), of a step of
// a nearly empty tile, and of an epilogue (store, GeLU, GeLU-backward, float store, float accumulation) were fitted
// to 516 launches in all four shapes, measured when 256 x 256 tiles had the 32 x 32 instruction; their steps are 8 to 16 % shorter
// now where they fill the chip, the other shapes' are what they were.  They choose as well with the present loops: over 12 500 launches
// (the five GEMMs of 2500 layers, 1 to 64 experts of 8 to 8192 rows, dimensions 64 to 8192, even and uneven loads) the choice is
// on average 2.2 % slower than the best tile of each launch, in 12 % of them by more than 5 %; 256 x 256 throughout is 44 % slower.
// The host does not know the loads; it takes every expert to have the mean.  A launch for several
// partitions counts the tiles of all of them: a step of 3003 tokens x 3, 776/2600, 6 experts, three partitions takes
// 596 us, and 608 where it keeps the shape that suits one partition's tiles (of 35 layers, drawn and listed, seven gain
// 1.5 to 13 %, two lose 1.2 %).
struct TileCost { int bm, bn, per_cu; double step[3], tail_step, epi[5]; };
static constexpr TileCost TILE_COSTS[5] = {
    {256, 256, 1, {1.09, 1.52, 1.48}, 0.85, {3.3, 10.8, 27.0, 11.1, 20.9}},      // CfgW, CfgN, Cfg4
    {256, 128, 1, {0.87, 0.84, 0.93}, 0.72, {3.4, 8.6, 19.1, 6.7, 11.0}},        // CfgM
    {128, 128, 2, {0.90, 1.29, 0.94}, 0.0, {3.0, 5.0, 9.3, 6.5, 8.8}},           // CfgS (two tiles at a time)
    {64, 128, 1, {0.44, 0.42, 0.0}, 0.92, {1.5, 2.5, 5.0, 0.0, 0.0}},            // CfgT (not for TN)
    {64, 64, 1, {0.24, 0.0, 0.0}, 0.24, {1.2, 0.0, 0.0, 0.0, 0.0}},              // CfgU (NN stores)
};
// Tiles of a launch with rows of all experts alike; the last ones have fewer rows.
static void count_tiles(const TileCost& c, const GemmArgs& a, long long* whole, long long* tail) {
    const long long per_row = (long long)((a.N + c.bn - 1) / c.bn) * launch_experts(a);
    const int full = a.mean_rows / c.bm, rest = a.mean_rows - full * c.bm;
    *whole = full * per_row;
    // an even multiple on average: about half the experts have a few rows more, where the capacity allows it
    *tail = rest ? per_row : a.mean_rows < a.Cp ? per_row / 2 : 0;
}
// Whether a store over K has so few 64 x 64 tiles that CfgU may take it: not more than three quarters of the CUs, so that uneven loads find room
// beside them, and no second round of them with loads one deviation above the mean either.  More CUs read the weights at once, which is worth most
// where they come from memory; many tiles lose it to reading their operands twice as often.  us, of both expert GEMMs, the first the same,
// second in CfgT / CfgU, mean of 2021 launches, weights in the caches (and not): 0-63 tiles, K 1024-1999 0.6 less (0.9), 2000-3499 1.2 (2.4),
// 5000+ 3.8 (8.7); 128-191 tiles 0.3 (1.5), 1.0 (3.3), 3.8 (10.0); 192-255 0.3 more (1.5 less, up to 4.3 more), 0.2 less (3.0, up to 6.9 more);
// 256-319 2.9 more (1.8 more), 2.9 more (0.3 more); below K = 1024 0.2 (0.3).
static bool few_tiles(const GemmArgs& a, int cus) {
    const TileCost& c = TILE_COSTS[4];
    long long whole, tail;
    count_tiles(c, a, &whole, &tail);
    const double above = a.mean_rows + sqrt((double)a.mean_rows);
    const int rows = above < a.Cp ? (int)above : a.Cp;
    const long long most = (long long)((rows + c.bm - 1) / c.bm) * ((a.N + c.bn - 1) / c.bn) * launch_experts(a);
    return a.K >= 1024 && whole + tail <= cus * 3 / 4 && most <= cus;
}
// (one: a single tile's, not the launch's)
static double tile_time(const TileCost& c, int lay, int epi, const GemmArgs& a, int cus, bool one = false) {
    const int which = epi == EPI_GELU ? 1 : epi == EPI_DGELU ? 2 : epi == EPI_STORE_F32 ? 3 : epi == EPI_ACCUM_F32 ? 4 : 0;
    const int segs = a.k_segs > 1 ? a.k_segs : 1;
    const double kt = lay == GEMM_TN ? (double)((a.mean_rows + 63) / 64) * segs : (double)((a.K + 63) / 64);
    long long whole, tail = 0;                       // tiles; those of the experts' last, partly filled tile rows
    double share = 1.0;                              // how full a tail tile is, in quarters
    if (lay == GEMM_TN) {
        whole = (long long)((a.Mo + c.bm - 1) / c.bm) * ((a.N + c.bn - 1) / c.bn) * a.E;
    } else {
        const int rest = a.mean_rows % c.bm;
        count_tiles(c, a, &whole, &tail);
        share = rest ? (rest + c.bm / 4 - 1) / (c.bm / 4) * 0.25 : 0.25;
    }
    const double tile = kt * c.step[lay] + c.epi[which], launch = 1.7;
    if (one) return tile;
    if (c.per_cu == 2) {
        const long long n = whole + tail, rounds = n / (2 * cus), rest = n - rounds * 2 * cus;
        return launch + rounds * tile + (rest == 0 ? 0.0 : rest <= cus ? 0.53 * tile : tile);
    }
    if (c.bm <= 64) share = 1.0;
    const long long rounds = (whole + cus - 1) / cus, spare = rounds * cus - whole;
    const long long extra = tail > spare ? (tail - spare + cus - 1) / cus : 0;
    return launch + rounds * tile +
           extra * (kt * (c.tail_step + (c.step[lay] - c.tail_step) * share) + c.epi[which] * (0.4 + 0.6 * share));
}
static int tile_choice(int lay, int epi, const GemmArgs& a) {
    const int cus = compute_units();                  // (units left free change the time of a launch, not its results)
    int best = 0;
    double least = 0.0;
    const bool u = lay == GEMM_NN && (epi == EPI_STORE || epi == EPI_SCATTER) && few_tiles(a, cus);
    for (int c = 0; c < (lay == GEMM_TN ? 3 : u ? 5 : 4); ++c) {
        const double t = tile_time(TILE_COSTS[c], lay, epi, a, cus);
        // (a smaller tile has to be clearly better: skewed loads drop rows and make more cheap last tile rows)
        if (c == 0 || t < (best == 0 ? 0.93 : 1.0) * least) { best = c; least = t; }
    }
    return best;
}

// Only the combinations the expert FFN uses are instantiated: NN with plain, GeLU and scattered stores
// (both layers of forward, recomputation), NT with GeLU-backward and plain stores (the two input
// gradients), TN with float store and float accumulation (the weight gradients).
template <int LAY, int EPI>
static moe_status launch_cfg(const GemmArgs& a, hipStream_t s) {
    const int choice = tile_choice(LAY, EPI, a);
    if (choice == 2) return launch_one<LAY, EPI, CfgS>(a, s);
    if constexpr (LAY != GEMM_TN) { if (choice == 3) return launch_one<LAY, EPI, CfgT>(a, s); }
    if constexpr (LAY == GEMM_NN && EPI != EPI_GELU) { if (choice == 4) return launch_one<LAY, EPI, CfgU>(a, s); }
    if (choice == 1) return launch_one<LAY, EPI, CfgM>(a, s);
    return launch_one<LAY, EPI, typename CfgFor<LAY, EPI>::type>(a, s);
}

void gemm_bf16_tile(GemmLayout lay, GemmEpilogue epi, const GemmArgs& a, int* rows, int* cols) {
    const TileCost& c = TILE_COSTS[tile_choice(lay, epi, a)];
    *rows = c.bm;
    *cols = c.bn;
}

static moe_status check_args(GemmLayout lay, GemmEpilogue epi, const GemmArgs& a) {
    if (a.dw_part && a.dw_parts != gemm_bf16_dw_parts(a.N)) return MOE_ERR_SHAPE;
    // operand rows must be 16-byte aligned in memory
    if ((a.lda | a.ldb) & 7) return MOE_ERR_UNSUPPORTED;
    // buffer offsets are 32-bit: an expert's operands, and its rows of a bfloat16 output, must stay below 2 GiB
    // (rows of two to four million elements would also take the epilogue's row steps past 2^32)
    long long ldmax = a.lda > a.ldb ? a.lda : a.ldb;
    if (epi != EPI_ACCUM_F32 && epi != EPI_STORE_F32 && epi != EPI_SCATTER && a.ldc > ldmax) ldmax = a.ldc;
    const long long rmax = a.Cp > a.K ? a.Cp : a.K;
    if ((rmax + 8 * 64) * ldmax * 2 >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    if (a.k_segs > 1 && (lay != GEMM_TN || a.k_segs > MAX_KSEGS)) return MOE_ERR_UNSUPPORTED;
    if (a.np > 1 && (lay == GEMM_TN || launch_experts(a) > 64)) return MOE_ERR_UNSUPPORTED;
    if (epi == EPI_SCATTER) {
        if (lay == GEMM_TN || !a.c_rows || !a.slot_w || a.c_row_limit <= 0) return MOE_ERR_UNSUPPORTED;
        if (((long long)a.c_row_limit + 1) * a.ldc * 2 >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    }
    if (a.a_rows) {
        // gathered rows: only for the row operand of NN / NT, and the whole matrix must stay below 2 GiB
        if (lay == GEMM_TN || a.a_row_limit <= 0) return MOE_ERR_UNSUPPORTED;
        if (((long long)a.a_row_limit + 1) * a.lda * 2 >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    }
    return MOE_OK;
}

// Rounds of tiles from which on the persistent launches one by one are the faster ones: of 32 768 tokens, 2048/8192, 16
// experts, two partitions (2 x 16 rounds) the step takes 13.09 ms with them and 13.19 with all three
// together; 8192 tokens, 768/3072, 64 experts (18 rounds of weight gradients, 3 of the input gradient) 1.242 and 1.226 ms.
// Below: 16 384 tokens, 1024/4096, 8 experts, four partitions (0.6 + 4 rounds) 2.59 and 2.47
// ms, 16 unevenly loaded experts 2.59 and 2.46, 4096 tokens, 512/2048 345 and 311 us.
// (Tiles of full experts, since the host does not know the loads and a launch has to have room for them: what the capacity adds
// are workgroups without a tile at the launch's end.  Ten shapes at capacity factors of 1.25 to 8: what a launch below the line takes varies by 1 %.)
constexpr int BACKWARD_ROUNDS = 24;

// Whether they are the faster ones below that: apart, each ends in a round that leaves CUs idle and together only the last one does, but
// a workgroup of the launch for all has one tile and begins it with nothing requested yet, where a persistent one fetches its next
// tile under the last one's epilogue: 1.5 us a tile of 256 x 256 rows and columns (those of 128 x 128 have a second workgroup
// beside them).  Fitted to 1326 backwards, even and uneven loads, with the loops before the present ones; of 2500 with these, 81 are more than
// 2 % slower than the better of the two (20 more than 5 %, one 16 %).
// us of these kernels, apart / together: 64 experts x 64 rows, 768/3072 (9 + 9 rounds of weight gradients, 1.5) 312 / 318, 24 x 457, 2048/4096
// (12 + 12, 3) 775 / 798, 16 x 500, 2048/5120 632 / 634, 8 x 1024, 1024/4096 (2 + 2, 0.6) 221 / 217 and two launches less.
static bool together_pays(const GemmArgs* dgrad, const GemmArgs& w2, const GemmArgs& w1, const GateDlArgs* gate, int epi, int cw, int cd) {
    if (cw == 2) return true;
    const int cus = compute_units();
    const TileCost& c = TILE_COSTS[cw];
    // (apart, the gate's dL has a launch of its own: 8192 tokens, 64 experts 12 us and the gap before the next one, as a step measures it 18)
    double busy = 0.0, apart = gate ? 6.0 + 0.2 * w2.E : 0.0;
    for (const GemmArgs* w : {&w2, &w1}) {
        const long long n = (long long)((w->Mo + c.bm - 1) / c.bm) * ((w->N + c.bn - 1) / c.bn) * w->E;
        busy += n * (tile_time(c, GEMM_TN, epi, *w, cus, true) + 1.5);
        apart += tile_time(c, GEMM_TN, epi, *w, cus);
    }
    if (dgrad) {
        long long whole, tail;
        count_tiles(TILE_COSTS[cd], *dgrad, &whole, &tail);
        busy += (whole + tail) * (tile_time(TILE_COSTS[cd], GEMM_NT, EPI_STORE, *dgrad, cus, true) + 1.5);
        apart += tile_time(TILE_COSTS[cd], GEMM_NT, EPI_STORE, *dgrad, cus);
    }
    // (the two alone, without an input gradient to fill their rounds, have to promise more)
    return busy / cus < (dgrad ? 1.04 : 0.85) * apart;
}

template <int EPI, typename CN, typename CT>
static moe_status launch_backward(const GemmArgs* dgrad, const GemmArgs& w2, const GemmArgs& w1, bool w_first,
                                  const GateDlArgs* gate, hipStream_t s, bool* done) {
    BackwardArgs b = {};
    b.w_first = w_first;
    b.w[0] = w2;
    b.w[1] = w1;
    int blocks = 0;
    if (dgrad) {
        b.d = *dgrad;
        b.tiles_dm = (dgrad->Cp + CN::BM - 1) / CN::BM;
        b.tiles_dn = (dgrad->N + CN::BN - 1) / CN::BN;
        blocks += (launch_experts(*dgrad) * b.tiles_dm * b.tiles_dn + 7) / 8 * 8;
    }
    for (int q = 0; q < 2; ++q) {
        b.tiles_wm[q] = (b.w[q].Mo + CT::BM - 1) / CT::BM;
        b.tiles_wn[q] = (b.w[q].N + CT::BN - 1) / CT::BN;
        blocks += (b.w[q].E * b.tiles_wm[q] * b.tiles_wn[q] + 7) / 8 * 8;
    }
    *done = blocks <= BACKWARD_ROUNDS * CT::OCC * compute_units();
    if (!*done) return MOE_OK;
    if (gate) { b.gate = *gate; blocks += gate->blocks; }
    constexpr int lds = CN::LDS_BYTES > CT::LDS_BYTES ? CN::LDS_BYTES : CT::LDS_BYTES;
    auto kern = gemm_bf16_backward_kernel<EPI, CN, CT>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        attr_done = true;
    }
    {
        // (a weight gradient reduces the rows of all partitions of its group, an input gradient has those of one)
        ProfScope ps(PK_GEMM_WGRAD, s, 2, dgrad ? PK_GEMM_DGRAD : -1, dgrad && dgrad->np > 1 ? dgrad->np : 1,
                     w2.k_segs > 1 ? w2.k_segs : 1);
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, s, b);
    }
    count_launch(LC_GEMM, 2 + (!dgrad ? 0 : dgrad->np > 1 ? dgrad->np : 1));
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

template <int EPI>
static moe_status backward_cfg(const GemmArgs* dgrad, const GemmArgs& w2, const GemmArgs& w1, const GateDlArgs* gate,
                               hipStream_t s, bool* done) {
    // (the shapes are those of the launches by themselves; shapes with one workgroup per CU and with two do not mix)
    const int cw = tile_choice(GEMM_TN, EPI, w2), cd = dgrad ? tile_choice(GEMM_NT, EPI_STORE, *dgrad) : cw;
    if (cw == 1 || tile_choice(GEMM_TN, EPI, w1) != cw || w2.free_cus > 0) return MOE_OK;
    if (!together_pays(dgrad, w2, w1, gate, EPI, cw, cd)) return MOE_OK;
    const bool w_first = dgrad && tile_time(TILE_COSTS[cw], GEMM_TN, EPI, w2, compute_units(), true) >
                                      tile_time(TILE_COSTS[cd], GEMM_NT, EPI_STORE, *dgrad, compute_units(), true);
    if (cw == 2) {
        if (cd < 2) return MOE_OK;
        if (cd == 3) return launch_backward<EPI, CfgT2, CfgS>(dgrad, w2, w1, w_first, gate, s, done);
        return launch_backward<EPI, CfgS, CfgS>(dgrad, w2, w1, w_first, gate, s, done);
    }
    if (cd == 2) return MOE_OK;
    if (cd == 1) return launch_backward<EPI, CfgM, Cfg4>(dgrad, w2, w1, w_first, gate, s, done);
    if (cd == 3) return launch_backward<EPI, CfgT, Cfg4>(dgrad, w2, w1, w_first, gate, s, done);
    return launch_backward<EPI, CfgN, Cfg4>(dgrad, w2, w1, w_first, gate, s, done);
}

moe_status gemm_bf16_backward(const GemmArgs* dgrad, const GemmArgs& w2, const GemmArgs& w1, GemmEpilogue epi,
                              const GateDlArgs* gate, hipStream_t s, bool* done) {
    *done = false;
    if (dgrad) MOE_TRY(check_args(GEMM_NT, EPI_STORE, *dgrad));
    MOE_TRY(check_args(GEMM_TN, epi, w2));
    MOE_TRY(check_args(GEMM_TN, epi, w1));
    return epi == EPI_STORE_F32 ? backward_cfg<EPI_STORE_F32>(dgrad, w2, w1, gate, s, done)
                                : backward_cfg<EPI_ACCUM_F32>(dgrad, w2, w1, gate, s, done);
}

moe_status gemm_bf16(GemmLayout lay, GemmEpilogue epi, const GemmArgs& a, hipStream_t s) {
    MOE_TRY(check_args(lay, epi, a));
    if (lay == GEMM_NN && epi == EPI_STORE) return launch_cfg<GEMM_NN, EPI_STORE>(a, s);
    if (lay == GEMM_NN && epi == EPI_GELU) return launch_cfg<GEMM_NN, EPI_GELU>(a, s);
    if (lay == GEMM_NN && epi == EPI_SCATTER) return launch_cfg<GEMM_NN, EPI_SCATTER>(a, s);
    if (lay == GEMM_NT && epi == EPI_STORE) return launch_cfg<GEMM_NT, EPI_STORE>(a, s);
    if (lay == GEMM_NT && epi == EPI_DGELU) return launch_cfg<GEMM_NT, EPI_DGELU>(a, s);
    if (lay == GEMM_TN && epi == EPI_STORE_F32) return launch_cfg<GEMM_TN, EPI_STORE_F32>(a, s);
    if (lay == GEMM_TN && epi == EPI_ACCUM_F32) return launch_cfg<GEMM_TN, EPI_ACCUM_F32>(a, s);
    return MOE_ERR_UNSUPPORTED;
}

}  // namespace moe
