// (a) Remaining-length predictor head on gfx950.
//
// Section 4.2 (Eq. 1-2): the last-layer, last-token hidden state of every
// running request goes through a small MLP.  Here: a1 = act(W1 h + b1),
// logits = W2 a1 + b2 over length bins, p = softmax, E = sum p_j v_j, then
// the continuous-prediction smoothing of Section 4.3 and integerisation.
//
// Kernel 1 (gemm1_splitk): Z1 partials = H W1^T over a K-slice, on MFMA
//   (32x32 blocks), 128 bytes of K per row and step (64 bf16 / 32 fp32; half of
//   it with 256x256 tiles) through a ring of LDS slots filled by direct
//   global-to-LDS loads, split-K so that small batches still fill the CUs.  Tile shapes: 64x64 and 128x64
//   on 4 waves, 128x128 and 256x256 on 8 waves; a cost model picks one per
//   product.  Partials are fp32, reduced later in a fixed order
//   (deterministic results).
// Kernel 2 (head): 4 rows per workgroup (many workgroups, so the split-K
//   partial reads have plenty of loads in flight), 64 for large bf16 batches:
//   fixed-order split-K reduction, bias, activation, the bin GEMM (MFMA
//   16x16x32 on a bf16 hi/lo split of a1, or 16x16x4 in fp32), softmax,
//   expectation, EMA, round-half-even, clamp.
// Both in one (predict_fused): bf16 products of one K-slice, up to 128 bins.
#include <type_traits>

#include "star_common.hpp"
#include "star_internal.hpp"

namespace star {

// ---------------------------------------------------------------------------
// GEMM1
// ---------------------------------------------------------------------------
// K is staged through LDS in steps of 128 bytes of every row (64 bf16, 32
// fp32; 64 bytes in the 256 x 256 tile), by direct global-to-LDS loads into a
// ring of NS slots: NS - 1 steps of loads are in flight and none of them
// holds registers.  A slot's rows are packed, and chunk c (16 bytes) of row r
// lies at position c ^ (r / 2 % 8) (64-byte rows: c ^ (r / 4 % 4)), so that
// the 16 rows that a fragment read touches at a time cover all the banks.
// The permutation is made by the loads' addresses: a wave's load fills 1 KiB
// of LDS in lane order, 8 or 16 rows.  128 bytes are a whole cache line:
// loads alone, from a cold L2, ran at 37.6 bytes per cycle and CU with such
// rows and at 26.4 with half lines (1024 x 512 x 4096, 128 x 64 tiles).
// Map blockIdx to a logical tile index so that consecutive logical indices
// run on the same XCD (workgroups are dealt round-robin over the 8 XCDs):
// logical neighbours share operand rows and hence that XCD's L2.
__device__ inline int xcd_logical_block(int bid, int nblk) {
    const int q = nblk / 8, r = nblk % 8;
    const int x = bid % 8;
    return x * q + (x < r ? x : r) + bid / 8;
}

// Tile shape of the split-K product: BM x BN outputs per workgroup, WM x WN
// waves, each wave a (BM/WM) x (BN/WN) slab of 32 x 32 matrix-core blocks; a
// ring of NS slots of STEP bytes per row; kAlt: the two halves of the waves
// alternate (see g1_mainloop).
template <int kBM, int kBN, int kWM, int kWN, int kStep, int kNS, bool kAlternate>
struct G1Shape {
    static constexpr int BM = kBM, BN = kBN, WM = kWM, WN = kWN, STEP = kStep, NS = kNS;
    static constexpr bool kAlt = kAlternate;
    static constexpr int WAVES = WM * WN, THREADS = 64 * WAVES;
    static constexpr int MI = BM / WM / 32, NJ = BN / WN / 32;
    static constexpr int CPR = STEP / 16;           // 16-byte chunks per row
    static constexpr int RPL = 64 / CPR;            // rows of one wave's load
    static constexpr int KK = CPR / 2;              // products of a step, in K
    static constexpr int CA = BM * CPR / THREADS;   // 16-byte chunks per thread, A
    static constexpr int CB = BN * CPR / THREADS;   // ... and W
    static constexpr int SLOT = (BM + BN) * STEP, LDS = NS * SLOT;
    // position of chunk c of row r (see above)
    __device__ static constexpr int pos(int c, int r) {
        return STEP == 128 ? c ^ ((r >> 1) & 7) : c ^ ((r >> 2) & 3);
    }
    static_assert(STEP == 128 || STEP == 64, "whole or half cache lines");
    static_assert(MI >= 1 && NJ >= 1 && CA >= 1 && CB >= 1, "shape");
    static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
};
// Whole star_predict calls (us, captured graphs) with these rings, against
// the register-staged loop and padded LDS rows that they replace (before):
//   1024 x 512 x 4096  18.7 -> 15.8     4096 x 512 x 5120  44.0 -> 36.6
//   777 x 512 x 3584   17.2 -> 14.8     512 x 512 x 4096   15.0 -> 13.3
// Three slots: with four, the LDS of one workgroup less on a CU, 15.9, 36.6,
// 14.8 and 13.4, and 118 against 94.6 for 8 overlapped batches.  With six
// slots of half cache lines: 16.9, 39.9, 15.6 and 13.5.
using G1Small = G1Shape<64, 64, 2, 2, 128, 3, false>;     // 48 KiB of LDS: three per CU
using G1Mid = G1Shape<128, 64, 2, 2, 128, 3, false>;      // 72 KiB: two per CU
using G1Big = G1Shape<128, 128, 2, 4, 128, 3, false>;     // 96 KiB, 64 x 32 slabs
// 128 x 64 slabs, all 160 KiB of LDS: a third of G1Big's LDS reads per
// product.  Its two wave groups alternate (528 us without, 464-537 with; the
// register-staged loop took 550-609).
// What bounds it at 32768 x 1024 x 8192: the operand loads alone take 387 us
// and the MFMAs alone 340 us (at 1.77 GHz: the matrix cores run into the
// card's power limit; the whole kernel runs at 1.5-1.7 GHz).
using G1Huge = G1Shape<256, 256, 2, 4, 64, 5, true>;
constexpr int G1_HUGE_MIN_TILES = 256;    // 256 x 256 tiles (no split) from which G1Huge is used

// The work of one workgroup of the split-K product: tile (tm, tn), K-steps
// [kt0, kt0 + nk), and the last, partial step of a K that is no whole number
// of steps.  Workgroups are dealt to the XCDs round-robin; the logical
// order puts one K-slice of neighbouring tiles on each XCD.
struct G1Work {
    int split, tm, tn, kt0, nk;
    int tail;                 // bytes of K in the partial step (0: none)
};
template <class SH>
__device__ inline G1Work g1_work(int splits, int tiles_n, int64_t row_bytes, int bid,
                                 int nblocks) {
    G1Work w;
    const int logical = xcd_logical_block(bid, nblocks);
    const int tiles = nblocks / splits;
    w.split = logical / tiles;
    const int tile = logical % tiles;
    w.tm = tile / tiles_n;
    w.tn = tile % tiles_n;
    // at most 2^27 steps (K < 2^31) and 16 splits: 32-bit products, whose
    // divisions are short (64-bit ones took 400 instructions before the first load)
    const uint32_t steps = (uint32_t)(row_bytes / SH::STEP);
    w.kt0 = (int)((uint32_t)w.split * steps / (uint32_t)splits);
    w.nk = (int)((uint32_t)(w.split + 1) * steps / (uint32_t)splits) - w.kt0;
    w.tail = w.split == splits - 1 ? (int)(row_bytes % SH::STEP) : 0;
    return w;
}

// 16 bytes per lane from global memory to LDS (wave-uniform base + 16 lane)
__device__ __forceinline__ void g1_load_lds(const char* g, char* l) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
// at most kN of this wave's vector-memory operations outstanding
template <int kN>
__device__ __forceinline__ void g1_wait_vm() {
    static_assert(kN < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt((kN & 15) | (7 << 4) | (15 << 8) | ((kN >> 4) << 14));
}
__device__ __forceinline__ void g1_wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }
// A barrier that waits for no memory operation (the waits are explicit); the
// compiler moves nothing across it.
__device__ __forceinline__ void g1_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// A wave's fragments of one step: of each of its rows, the 16-byte chunks 2 kk
// + lane / 32 of K.  pos[kk]: where they lie in a row.
template <class SH>
struct G1Frag {
    u32x4 a[SH::KK][SH::MI], b[SH::KK][SH::NJ];
};
template <class SH>
__device__ __forceinline__ void g1_read_frag(const char* slot, int offa, int offb,
                                             const int (&pos)[SH::KK], G1Frag<SH>& f) {
#pragma unroll
    for (int kk = 0; kk < SH::KK; ++kk) {
#pragma unroll
        for (int i = 0; i < SH::MI; ++i)
            f.a[kk][i] = *(const u32x4*)(slot + offa + i * 32 * SH::STEP + pos[kk]);
#pragma unroll
        for (int j = 0; j < SH::NJ; ++j)
            f.b[kk][j] = *(const u32x4*)(slot + offb + j * 32 * SH::STEP + pos[kk]);
    }
}
// bf16: v_mfma_f32_32x32x16_bf16, lane feeds row lane % 32, the 8 k of its
// chunk.  fp32: v_mfma_f32_32x32x2_f32 takes one k of each half wave, so
// element e of the two chunks makes one product.
template <int kElemBytes, class SH>
__device__ __forceinline__ void g1_mfma(const G1Frag<SH>& f, f32x16 (&acc)[SH::MI][SH::NJ]) {
#pragma unroll
    for (int kk = 0; kk < SH::KK; ++kk) {
        if constexpr (kElemBytes == 2) {
#pragma unroll
            for (int i = 0; i < SH::MI; ++i)
#pragma unroll
                for (int j = 0; j < SH::NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8_t, f.a[kk][i]),
                        __builtin_bit_cast(bf16x8_t, f.b[kk][j]), acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < SH::MI; ++i)
#pragma unroll
                    for (int j = 0; j < SH::NJ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                            __uint_as_float(f.a[kk][i][e]), __uint_as_float(f.b[kk][j][e]),
                            acc[i][j], 0, 0, 0);
        }
    }
}

// Steps i + kJ, i + kJ + 1, .. of the last NS - 1, as far as nk: fewer and
// fewer loads stay outstanding.
template <int NS, int L, int kJ, class Step>
__device__ __forceinline__ void g1_drain(Step& step, int i, int nk) {
    if constexpr (kJ < NS - 1) {
        if (i + kJ >= nk) return;
        step(std::integral_constant<int, kJ < NS - 3 ? (NS - 3 - kJ) * L : 0>{}, -1);
        g1_drain<NS, L, kJ + 1>(step, i, nk);
    }
}

// Main loop of one workgroup's product; acc receives this wave's slab.  Rows
// past M or N repeat the last one (their outputs are never stored).
//
// Step i reads the wave's fragments of slot i % NS, requests step i + NS - 1
// into the slot of step i - 1, waits for its fragments and for its own loads
// of step i + 1, passes one barrier and multiplies.  The barrier publishes
// step i + 1 to all waves, and shows that all have read slot i % NS, which
// step i + 1 refills.
//
// kAlt: the upper half of the waves (one per SIMD, like the lower half) runs
// one barrier behind, and a second barrier follows the products, so that one
// half multiplies while the other reads.  The same two conditions hold half a
// step later: the upper half passes the barrier after its waits of step i
// before the lower half reads step i + 1, and the lower half requests a slot
// only after the upper half has read it.
template <int kElemBytes, class SH>
__device__ __forceinline__ void g1_mainloop(const char* __restrict__ A,
                                            const char* __restrict__ W, int M, int N,
                                            int64_t row_bytes, const G1Work& w, char* lds,
                                            f32x16 (&acc)[SH::MI][SH::NJ]) {
    constexpr int CA = SH::CA, CB = SH::CB, L = CA + CB, NS = SH::NS;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wid / SH::WN, wn = wid % SH::WN;
    const int r32 = lane & 31, khalf = lane >> 5;
#pragma unroll
    for (int i = 0; i < SH::MI; ++i)
#pragma unroll
        for (int j = 0; j < SH::NJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // this lane's 16 bytes of each of its wave's loads: load p fills the RPL
    // rows from (p WAVES + wid) RPL on.  The chunk is the one that belongs at
    // the lane's position; it is the same for every p, because RPL WAVES is a
    // multiple of the permutation's period.
    static_assert(SH::RPL * SH::WAVES % 16 == 0, "one permutation per lane");
    const int lrow = wid * SH::RPL + lane / SH::CPR;
    const int chunk = SH::pos(lane % SH::CPR, lrow) * 16;
    const char* pa[CA];
    const char* pb[CB];
#pragma unroll
    for (int p = 0; p < CA; ++p) {
        const int row = w.tm * SH::BM + p * SH::WAVES * SH::RPL + lrow;
        pa[p] = A + (int64_t)(row < M ? row : M - 1) * row_bytes + chunk;
    }
#pragma unroll
    for (int p = 0; p < CB; ++p) {
        const int row = w.tn * SH::BN + p * SH::WAVES * SH::RPL + lrow;
        pb[p] = W + (int64_t)(row < N ? row : N - 1) * row_bytes + chunk;
    }
    const int nk = w.nk;
    char* const mine = lds + wid * 1024;      // the wave's first KiB of a slot
    auto request = [&](int i, int slot) {
        const int64_t kb = (int64_t)(w.kt0 + (i < nk ? i : nk - 1)) * SH::STEP;
        char* l = mine + slot * SH::SLOT;
#pragma unroll
        for (int p = 0; p < CA; ++p) g1_load_lds(pa[p] + kb, l + p * SH::WAVES * 1024);
#pragma unroll
        for (int p = 0; p < CB; ++p)
            g1_load_lds(pb[p] + kb, l + SH::BM * SH::STEP + p * SH::WAVES * 1024);
    };
    // the partial step, if any, is requested first and held in registers until
    // the whole steps are done (its chunks past K read the row's start and are
    // zeroed when they are written to LDS)
    u32x4 ta[CA], tb[CB];
    if (w.tail) {
        const int64_t kb = chunk < w.tail ? (int64_t)(w.kt0 + nk) * SH::STEP : -(int64_t)chunk;
#pragma unroll
        for (int p = 0; p < CA; ++p) ta[p] = *(const u32x4*)(pa[p] + kb);
#pragma unroll
        for (int p = 0; p < CB; ++p) tb[p] = *(const u32x4*)(pb[p] + kb);
    }

    const int offa = (wm * 32 * SH::MI + r32) * SH::STEP;
    const int offb = SH::BM * SH::STEP + (wn * 32 * SH::NJ + r32) * SH::STEP;
    int pos[SH::KK];
#pragma unroll
    for (int kk = 0; kk < SH::KK; ++kk) pos[kk] = SH::pos(2 * kk + khalf, r32) * 16;
    G1Frag<SH> f;
    if (nk > 0) {
        // requests of the first NS - 1 steps; fewer steps repeat the last one
        // (a K-slice that short is all latency), so that the waits below hold
#pragma unroll
        for (int d = 0; d < NS - 1; ++d) request(d, d);
        g1_wait_vm<(NS - 2) * L>();
        g1_barrier();
        const bool late = SH::kAlt && wid >= SH::WAVES / 2;
        if (late) g1_barrier();
        int slot = 0;
        // one step; at most kOut of the wave's loads stay outstanding after it
        auto step = [&](auto kOut, int next) {
            __builtin_amdgcn_sched_barrier(0);
            g1_read_frag<SH>(lds + slot * SH::SLOT, offa, offb, pos, f);
            __builtin_amdgcn_sched_barrier(0);
            if (next >= 0) request(next, slot == 0 ? NS - 1 : slot - 1);
            __builtin_amdgcn_sched_barrier(0);
            g1_wait_lds();
            g1_wait_vm<decltype(kOut)::value>();
            g1_barrier();
            if (SH::kAlt) __builtin_amdgcn_s_setprio(1);
            g1_mfma<kElemBytes, SH>(f, acc);
            if (SH::kAlt) {
                __builtin_amdgcn_s_setprio(0);
                g1_barrier();
            }
            slot = slot + 1 == NS ? 0 : slot + 1;
        };
        int i = 0;
        for (; i + NS - 1 < nk; ++i)
            step(std::integral_constant<int, (NS - 2) * L>{}, i + NS - 1);
        // the last NS - 1 steps request nothing
        g1_drain<NS, L, 0>(step, i, nk);
        if (SH::kAlt && !late) g1_barrier();
        g1_wait_vm<0>();          // repeated requests
        g1_barrier();             // every wave has read its last fragments: the ring is free
    }
    if (w.tail) {
        const uint32_t in = chunk < w.tail ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int p = 0; p < CA; ++p)
            *(u32x4*)(mine + p * SH::WAVES * 1024 + lane * 16) = ta[p] & in;
#pragma unroll
        for (int p = 0; p < CB; ++p)
            *(u32x4*)(mine + SH::BM * SH::STEP + p * SH::WAVES * 1024 + lane * 16) = tb[p] & in;
        __syncthreads();
        g1_read_frag<SH>(lds, offa, offb, pos, f);
        g1_mfma<kElemBytes, SH>(f, acc);
    }
}

// Split-K product P[split] = A[:, Ks] W[:, Ks]^T over one BM x BN tile: the
// work of block `bid` of a grid of `nblocks` product blocks.
template <int kElemBytes, class SH>
__device__ __forceinline__ void gemm1_tile(const char* __restrict__ A, const char* __restrict__ W,
                                           float* __restrict__ P, int M, int N, int Kd,
                                           int splits, int tiles_n, int bid, int nblocks,
                                           char* lds) {
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
    const int wm = wid / SH::WN, wn = wid % SH::WN;
    const int64_t row_bytes = (int64_t)Kd * kElemBytes;
    const G1Work w = g1_work<SH>(splits, tiles_n, row_bytes, bid, nblocks);
    f32x16 acc[SH::MI][SH::NJ];
    g1_mainloop<kElemBytes, SH>(A, W, M, N, row_bytes, w, lds, acc);
    // Element v of lane l of a 32 x 32 block is row 8 (v / 4) + 4 (l / 32) +
    // v % 4, column l % 32: a store covers 128 contiguous bytes of two rows.
    // (Collecting rows in LDS first, for 16-byte stores, was slower: 9.9
    // against 9.6 us at 1024 x 512 x 4096.)  The partials are written once
    // and read once by the next kernel: non-temporal stores stream them out
    // instead of leaving them dirty in L2 for the end-of-kernel writeback.
    float* out = P + (int64_t)w.split * M * N;
    const int r32 = lane & 31, khalf = lane >> 5;
#pragma unroll
    for (int i = 0; i < SH::MI; ++i)
#pragma unroll
        for (int j = 0; j < SH::NJ; ++j) {
            const int gcol = w.tn * SH::BN + wn * 32 * SH::NJ + j * 32 + r32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int grow = w.tm * SH::BM + wm * 32 * SH::MI + i * 32 + 8 * (v >> 2) +
                                 4 * khalf + (v & 3);
                if (grow < M && gcol < N)
                    __builtin_nontemporal_store(acc[i][j][v], &out[(int64_t)grow * N + gcol]);
            }
        }
}

template <int kElemBytes, class SH>
__global__ __launch_bounds__(SH::THREADS) void gemm1_splitk_kernel(
    const char* __restrict__ A, const char* __restrict__ W, float* __restrict__ P,
    int M, int N, int Kd, int splits, int tiles_n) {
    __shared__ __attribute__((aligned(1024))) char lds[SH::LDS];
    gemm1_tile<kElemBytes, SH>(A, W, P, M, N, Kd, splits, tiles_n, blockIdx.x, gridDim.x, lds);
}

// Launch of the split-K product with the plan's tile shape.
template <class SH>
static void launch_gemm_shape(const GemmPlan& g, bool bf16, const void* A, const void* W,
                              float* P, int M, int N, int K, hipStream_t stream) {
    const dim3 grid(g.tiles_m * g.tiles_n * g.splits);
    if (bf16)
        hipLaunchKernelGGL((gemm1_splitk_kernel<2, SH>), grid, dim3(SH::THREADS), 0, stream,
                           (const char*)A, (const char*)W, P, M, N, K, g.splits, g.tiles_n);
    else
        hipLaunchKernelGGL((gemm1_splitk_kernel<4, SH>), grid, dim3(SH::THREADS), 0, stream,
                           (const char*)A, (const char*)W, P, M, N, K, g.splits, g.tiles_n);
}

static hipError_t launch_gemm(const GemmPlan& g, bool bf16, const void* A, const void* W,
                              float* P, int M, int N, int K, hipStream_t stream) {
    switch (g.shape) {
        case GemmPlan::kBig: launch_gemm_shape<G1Big>(g, bf16, A, W, P, M, N, K, stream); break;
        case GemmPlan::kHuge: launch_gemm_shape<G1Huge>(g, bf16, A, W, P, M, N, K, stream); break;
        case GemmPlan::kMid: launch_gemm_shape<G1Mid>(g, bf16, A, W, P, M, N, K, stream); break;
        default: launch_gemm_shape<G1Small>(g, bf16, A, W, P, M, N, K, stream);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// head
// ---------------------------------------------------------------------------
// Rows per workgroup: 4, so that the split-K partial reads of a batch have
// plenty of workgroups in flight (large bf16 batches take head_tiled_kernel).
constexpr int HD_RB = 4;
constexpr int HD_THREADS = 256;
// float4 items per thread whose partial loads are in flight together: more
// when there are few split-K planes (registers hold kS x batch float4)
template <int kS> constexpr int hd_batch() { return kS == 1 ? 8 : kS == 2 ? 4 : 2; }
// W2 fragments (a bin block x one K-step) a wave loads at a time, the first group
// at kernel entry so that its latency overlaps the split-K reads.  us per call
// with 2, 4, 8 and 16:
//   up to two workgroups per CU (512 of them) the deep group hides the reads of a
//   wide W2: 300 x 2048 x 4096 fp32, 256 bins 187, 142, 127, 118; 1500 x 1024 x
//   4096, 128 bins 37.7, 37.6, 37.4, 36.9; narrow ones would do with less: 1024 x
//   512 x 4096, 64 bins 16.4, 16.4, 16.5, 16.5; 64 rows of it 10.8, 10.7, 11.1, 11.0;
//   past them, other workgroups hide them and its registers (140 against 80 with
//   four planes) keep those out: 4096 x 512 x 5120, 64 bins 39.0, 39.6, 41.2, 41.7;
//   7000 x 256 x 8192 48.3, 48.5, 49.4, 52.5.
constexpr int HD_W2PF = 16;
constexpr int HD_W2PF_LOW = 2;
constexpr int HD_LOWREG_GROUPS = 512;

// GELU in its erf form, x Phi(x) with Phi the standard normal distribution
// function, without branches: h = Phi(-|x|) = erfc(|x| / sqrt 2) / 2 from the
// rational-times-Gaussian approximation of erfc in Abramowitz & Stegun 7.1.26
// (absolute error under 1.5e-7 in erf; in fp32 the result is within 1.5e-7
// max(1, |x|) of the exact GELU, twenty times below the rounding of the bf16
// hi/lo pair that carries activations into the next product), and
// x Phi(x) = x - x h for x >= 0, x h below.
__device__ inline float gelu_erf(float x) {
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, fabsf(x), 1.0f));
    // coefficients a5 .. a1 of 7.1.26, halved
    float q = fmaf(t, 0.5307027145f, -0.7265760135f);
    q = fmaf(t, q, 0.7107068705f);
    q = fmaf(t, q, -0.142248368f);
    q = fmaf(t, q, 0.127414796f);
    // exp(-x^2 / 2) = 2^(-x^2 / (2 ln 2))
    const float h = t * q * __builtin_amdgcn_exp2f(x * x * -0.72134752044448170f);
    const float xh = x * h;
    return x >= 0.0f ? x - xh : xh;
}

__device__ inline float apply_act(float x, int act) {
    if (act == STAR_ACT_RELU) return x > 0.0f ? x : 0.0f;
    return gelu_erf(x);
}

// K of one step of the second product: the 16-byte chunks of the four lane
// groups (32 bf16, or 16 fp32)
template <bool kBF16> constexpr int hd_step() { return kBF16 ? 32 : 16; }
// LDS of the head: a1 (rows padded by 16 bytes against bank conflicts, K to
// whole steps; the bf16 hi and lo parts, or fp32), then the four waves' shares
// of the logits
static constexpr size_t head_rows_lds(bool bf16, int m, int nb) {
    const size_t step = bf16 ? 32 : 16;
    const size_t mpad = (m + step - 1) / step * step;
    const size_t a1 = bf16 ? 2 * HD_RB * (mpad + 8) * 2 : HD_RB * (mpad + 4) * 4;
    return a1 + (HD_THREADS / 64) * HD_RB * (((size_t)nb + 15) / 16 * 16) * 4;
}

// kS = number of split-K partial planes (compile time, so that all of a
// thread's partial loads are issued before the first is consumed).
// kReg: the regression head's last two layers instead of the binned one
// (the nb "bin logits" are the third layer's outputs, `bins` holds w4 and
// phase 3 computes relu(z) . w4 + b4 in place of the softmax mean).
// The head over rows [blk HD_RB, (blk + 1) HD_RB), its buffers in `smem`
// (head_rows_lds bytes).
//
// A chain of latencies bounds it (1024 rows, 4 planes, 8 MiB read: 6.2-7.3
// us; the fp32 head of 64 rows went from 8.6 to 6.8).  The partials, which
// everything waits for, are requested before anything else.  In the second product each wave takes
// a quarter of the K-steps for every bin: it then reads a quarter of a1 from
// LDS, where a quarter of the bins per wave read all of it in every wave,
// and its products of four bin blocks are independent.  The four shares are
// summed in wave order.  The softmax reduces by DPP, not by LDS shuffles.
template <bool kBF16, int kS, bool kReg, int kPF>
__device__ __forceinline__ void head_rows(
    const float* __restrict__ P, int B, int m, int nb, const float* __restrict__ b1,
    const void* __restrict__ w2, const float* __restrict__ b2, const float* __restrict__ bins,
    int act, float ema_alpha, int ema_init, float* __restrict__ ema_state,
    float* __restrict__ expected, int32_t* __restrict__ rem_len, int len_max, float b4, int blk,
    char* smem) {
    constexpr int kBatch = hd_batch<kS>();
    constexpr int kWaves = HD_THREADS / 64;
    constexpr int kStep = hd_step<kBF16>();
    constexpr int kPB = kPF < 4 ? kPF : 4;        // bin blocks of 16 at a time
    constexpr int kPK = kPF / kPB;                // K-steps at a time
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int row0 = blk * HD_RB;
    const int mpad = (m + kStep - 1) / kStep * kStep;
    const int astride = mpad + (kBF16 ? 8 : 4);   // elements per LDS row
    const int nbpad = (nb + 15) & ~15;

    uint16_t* ahi = (uint16_t*)smem;
    uint16_t* alo = ahi + HD_RB * astride;
    float* a32 = (float*)smem;
    float* z = kBF16 ? (float*)(alo + HD_RB * astride) : a32 + HD_RB * astride;

    // 1) fixed-order split-K reduction, bias, activation (float4 items)
    const int m4 = m >> 2;
    const int items = HD_RB * m4;
    const int64_t plane4 = (int64_t)B * m4;
    const float4* P4 = (const float4*)P;
    f32x4 v[kBatch][kS], bv[kBatch];
    int row[kBatch], c4[kBatch];
    bool ok[kBatch];
    auto load_items = [&](int base) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const uint32_t e = base + i * HD_THREADS + tid;
            row[i] = (int)(e / (uint32_t)m4);
            c4[i] = (int)(e - (uint32_t)row[i] * (uint32_t)m4);
            ok[i] = (int)e < items && row0 + row[i] < B;
            const int64_t off = ok[i] ? (int64_t)(row0 + row[i]) * m4 + c4[i] : 0;
#pragma unroll
            for (int q = 0; q < kS; ++q)
                // read once: streamed past L2 (non-temporal), so they do not
                // evict the operands the next product reads
                v[i][q] = __builtin_nontemporal_load((const f32x4*)&P4[q * plane4 + off]);
            bv[i] = b1 ? *(const f32x4*)(b1 + 4 * c4[i]) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    load_items(0);
    __builtin_amdgcn_sched_barrier(0);

    // everything phases 2 and 3 read from global memory is requested next, so
    // that its latency overlaps the split-K reads.  A lane's fragment of bin
    // block j and K-step u: the 16 bytes at W2[16 j + lane % 16][u kStep + (lane
    // / 16) chunk].  Loads are unconditional (clamped indices) so none of them
    // is waited for before it is used; columns past nb are discarded, K past
    // m is zeroed (fp32) or meets a1's zero padding (bf16).
    const int r16 = lane & 15;
    const int kq = lane >> 4;
    const int ksteps = mpad / kStep;
    constexpr int kChunk = kBF16 ? 8 : 4;         // elements per fragment
    u32x4 wf[kPK][kPB];
    // K-steps s0 .. s0 + kPK - 1 of this wave (step s of it is s kWaves + wid)
    auto load_w2 = [&](int s0, int j0) {
#pragma unroll
        for (int u = 0; u < kPK; ++u)
#pragma unroll
            for (int j = 0; j < kPB; ++j) {
                const int bin = (j0 + j) * 16 + r16;
                const int k = ((s0 + u) * kWaves + wid) * kStep + kq * kChunk;
                const bool in = bin < nb && k < m;
                const int64_t off = in ? (int64_t)bin * m + k : 0;
                wf[u][j] = kBF16 ? *(const u32x4*)((const uint16_t*)w2 + off)
                                 : *(const u32x4*)((const float*)w2 + off);
                if (!kBF16) wf[u][j] &= in ? 0xFFFFFFFFu : 0u;
            }
    };
    load_w2(0, 0);
    float binv[4], b2v[4];                        // used only where lane + 64 i < nb
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = lane + 64 * i < nb ? lane + 64 * i : nb - 1;
        binv[i] = bins[j];
        b2v[i] = b2 ? b2[j] : 0.0f;
    }
    const int gr = row0 + wid;                    // the row this wave finishes in phase 3
    const float ema_prev =
        (ema_alpha > 0.0f && !ema_init) ? ema_state[gr < B ? gr : B - 1] : 0.0f;
    __builtin_amdgcn_sched_barrier(0);

    for (int base = 0; base < items; base += kBatch * HD_THREADS) {
        if (base > 0) load_items(base);
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int e = base + i * HD_THREADS + tid;
            if (e >= items) continue;
            f32x4 sum = v[i][0];
#pragma unroll
            for (int q = 1; q < kS; ++q) sum += v[i][q];
            float a[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] = ok[i] ? apply_act(sum[j] + bv[i][j], act) : 0.0f;
            if constexpr (kBF16) {
                uint32_t h0, l0, h1, l1;
                split_bf16x2(a[0], a[1], h0, l0);
                split_bf16x2(a[2], a[3], h1, l1);
                const int o = row[i] * astride + 4 * c4[i];
                *(uint2*)(ahi + o) = make_uint2(h0, h1);
                *(uint2*)(alo + o) = make_uint2(l0, l1);
            } else {
                *(float4*)(a32 + row[i] * astride + 4 * c4[i]) = make_float4(a[0], a[1], a[2], a[3]);
            }
        }
    }
    if (mpad > m) {             // zero K padding [m, mpad)
        for (int e = tid; e < HD_RB * (mpad - m); e += HD_THREADS) {
            const int r = e / (mpad - m), u = m + e % (mpad - m);
            if constexpr (kBF16) {
                ahi[r * astride + u] = 0;
                alo[r * astride + u] = 0;
            } else {
                a32[r * astride + u] = 0.0f;
            }
        }
    }
    __syncthreads();

    // 2) bin logits: lane feeds A row lane % 16 and B row (bin) lane % 16, the
    // chunk of K of group lane / 16; accumulator element v of lane l is row
    // 4 (l / 16) + v, column l % 16.  Only the first HD_RB rows are stored,
    // so the others repeat them (rows of a product do not mix).
    const int aoff = (r16 % HD_RB) * astride + kq * kChunk;
    const int nblocks = nbpad / 16;
    for (int j0 = 0; j0 < nblocks; j0 += kPB) {
        f32x4 acc[kPB];
#pragma unroll
        for (int j = 0; j < kPB; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int s0 = 0; s0 * kWaves + wid < ksteps; s0 += kPK) {
            if (j0 > 0 || s0 > 0) load_w2(s0, j0);
            u32x4 hv[kPK], lv[kPK];
#pragma unroll
            for (int u = 0; u < kPK; ++u) {
                const int st = (s0 + u) * kWaves + wid;
                const int o = aoff + (st < ksteps ? st : 0) * kStep;
                if constexpr (kBF16) {
                    hv[u] = *(const u32x4*)(ahi + o);
                    lv[u] = *(const u32x4*)(alo + o);
                } else {
                    hv[u] = *(const u32x4*)(a32 + o);
                }
            }
#pragma unroll
            for (int u = 0; u < kPK; ++u) {
                if ((s0 + u) * kWaves + wid >= ksteps) break;          // uniform
                if constexpr (kBF16) {
#pragma unroll
                    for (int j = 0; j < kPB; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8_t, hv[u]),
                            __builtin_bit_cast(bf16x8_t, wf[u][j]), acc[j], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < kPB; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8_t, lv[u]),
                            __builtin_bit_cast(bf16x8_t, wf[u][j]), acc[j], 0, 0, 0);
                } else {
                    // v_mfma_f32_16x16x4_f32 takes one k of each lane group
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int j = 0; j < kPB; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                __uint_as_float(hv[u][e]), __uint_as_float(wf[u][j][e]), acc[j],
                                0, 0, 0);
                }
            }
        }
        if (kq == 0) {
#pragma unroll
            for (int j = 0; j < kPB; ++j)
                if (j0 + j < nblocks)
#pragma unroll
                    for (int r = 0; r < HD_RB; ++r)
                        z[(wid * HD_RB + r) * nbpad + (j0 + j) * 16 + r16] = acc[j][r];
        }
    }
    static_assert(HD_RB == 4 && kWaves == HD_RB, "accumulator rows, one wave per row");
    __syncthreads();

    // 3) softmax, expectation, EMA, integerisation: one wave per row
    if (gr >= B) return;
    float zl[4];                                  // -inf (0 for the regression head) past nb
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = lane + 64 * i;
        const int jc = j < nb ? j : 0;
        float t = z[wid * nbpad + jc];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) t += z[(w * HD_RB + wid) * nbpad + jc];
        t += b2v[i];
        zl[i] = j < nb ? t : kReg ? 0.0f : -INFINITY;
    }
    float den = 1.0f, num = 0.0f;
    if constexpr (kReg) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (lane + 64 * i < nb) num += fmaxf(zl[i], 0.0f) * binv[i];
        num = wave_total_f32(num) + b4;
    } else {
        const float zmax = wave_top_f32(fmaxf(fmaxf(zl[0], zl[1]), fmaxf(zl[2], zl[3])));
        den = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (lane + 64 * i < nb) {
                const float e = expf(zl[i] - zmax);
                den += e;
                num += e * binv[i];
            }
        }
        den = wave_total_f32(den);
        num = wave_total_f32(num);
    }
    if (lane == 0) {
        const float E = kReg ? num : num / den;
        expected[gr] = E;
        float y = E;
        if (ema_alpha > 0.0f) {
            y = ema_init ? E : ema_alpha * E + (1.0f - ema_alpha) * ema_prev;
            ema_state[gr] = y;
        }
        if (rem_len) {
            float q = rintf(y);
            int32_t li;
            if (!(q >= 1.0f)) li = 1;
            else if (q >= (float)len_max) li = len_max;
            else li = (int32_t)q;
            rem_len[gr] = li;
        }
    }
}

template <bool kBF16, int kS, bool kReg = false, int kPF = HD_W2PF>
__global__ __launch_bounds__(HD_THREADS) void head_kernel(
    const float* __restrict__ P, int B, int m, int nb, const float* __restrict__ b1,
    const void* __restrict__ w2, const float* __restrict__ b2, const float* __restrict__ bins,
    int act, float ema_alpha, int ema_init, float* __restrict__ ema_state,
    float* __restrict__ expected, int32_t* __restrict__ rem_len, int len_max, float b4 = 0.0f) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    head_rows<kBF16, kS, kReg, kPF>(P, B, m, nb, b1, w2, b2, bins, act, ema_alpha, ema_init,
                                    ema_state, expected, rem_len, len_max, b4, blockIdx.x, smem);
}

// ---------------------------------------------------------------------------
// The head for large bf16 batches, K-chunked: 64 rows per workgroup of eight
// waves.  Wave w takes the 16 rows of group w % 4 and the 32-wide half w / 4
// of every chunk of 64 a1 columns.  Each lane loads from HBM exactly the 8
// partials that it feeds to the 16x16x32 MFMA as its A operand (row
// lane % 16 of the group, columns 8 (lane / 16) + 0..7 of the half), reduces
// the planes in a fixed order, adds b1 (staged in LDS once), applies the
// activation and splits the result into the bf16 hi/lo pair in registers:
// a1 never passes through LDS and every activation is computed once.  W2's
// chunk, the B operand the four row groups share, is staged in LDS in two
// stages with one barrier per chunk.  The two halves' logits are summed once
// at the end (lower half first), and the softmax runs on the logits in
// registers: a row's bins are spread over 16 lanes, plus registers.
// W2 is read once per 64 rows (the 4-row head reads it once per 4).
// ---------------------------------------------------------------------------
constexpr int HT_ROWS = 64;
constexpr int HT_KC = 64;                   // a1 columns per chunk
constexpr int HT_ASTR = HT_KC + 8;          // bf16 per LDS row of W2 (padding spreads banks)
constexpr int HT_THREADS = 512;             // 4 row groups x 2 halves of each chunk
constexpr int HT_MIN_REQ = 8192;            // batches from which the tiled head is used
constexpr int HT_MAX_SPLITS = 4;            // its partial registers: 2 float4 per plane

// bin blocks of 16 the tiled head computes: 4, 8 or 16 (compile time, so that
// every loop over them has a fixed trip count; blocks past nb carry zeros)
static int head_tiled_blocks(int nb) { return nb <= 64 ? 4 : nb <= 128 ? 8 : 16; }
// two W2 stages, then b1 (m fp32); the halves' logits meet in the stages
constexpr size_t head_tiled_stage_bytes(int nbb) { return (size_t)nbb * 16 * HT_ASTR * 2; }
static size_t head_tiled_lds(int nb, int m) {
    return 2 * head_tiled_stage_bytes(head_tiled_blocks(nb)) + (size_t)m * 4;
}

struct HtArgs {
    const float4* P4;
    const uint16_t* W2;
    int64_t plane4;
    int B, m, m4, nb;
};

// a lane's 8 partials of one chunk, per plane
template <int kS>
struct HtP {
    float4 v[kS][2];
};
// the thread's 16-byte pieces of a W2 chunk (kNBB x 16 bins x 8 pieces over
// the workgroup)
template <int kNBB>
struct HtW {
    static constexpr int kU = kNBB * 16 * 8 / HT_THREADS;
    static_assert(kU >= 1 && kU * HT_THREADS == kNBB * 128, "whole W2 pieces per thread");
    uint4 v[kU];
};

// partials of row `row`, columns k .. k + 7 (m % 8 == 0: all in range or
// none); rows past B and columns past m read offset 0 and are masked later
template <int kS>
__device__ __forceinline__ void ht_load_p(const HtArgs& a, int row, int k, HtP<kS>& g) {
    const bool ok = row < a.B && k < a.m;
    const int64_t off = ok ? (int64_t)row * a.m4 + (k >> 2) : 0;
#pragma unroll
    for (int q = 0; q < kS; ++q) {
        const f32x4 t0 = __builtin_nontemporal_load((const f32x4*)&a.P4[q * a.plane4 + off]);
        const f32x4 t1 = __builtin_nontemporal_load((const f32x4*)&a.P4[q * a.plane4 + off + 1]);
        g.v[q][0] = make_float4(t0[0], t0[1], t0[2], t0[3]);
        g.v[q][1] = make_float4(t1[0], t1[1], t1[2], t1[3]);
    }
}

template <int kNBB>
__device__ __forceinline__ void ht_load_w(const HtArgs& a, int c, HtW<kNBB>& g) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < HtW<kNBB>::kU; ++u) {
        const int it = u * HT_THREADS + tid;
        const int j = it >> 3, kk = c * HT_KC + (it & 7) * 8;
        const bool ok = j < a.nb && kk < a.m;
        g.v[u] = *(const uint4*)(a.W2 + (ok ? (int64_t)j * a.m + kk : 0));
    }
}

template <int kNBB>
__device__ __forceinline__ void ht_store_w(const HtArgs& a, int c, const HtW<kNBB>& g,
                                           uint16_t* wl) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < HtW<kNBB>::kU; ++u) {
        const int it = u * HT_THREADS + tid;       // row j < kNBB x 16 of the W2 chunk
        const int j = it >> 3, kk = c * HT_KC + (it & 7) * 8;
        const uint32_t z = (j < a.nb && kk < a.m) ? 0xFFFFFFFFu : 0u;
        *(uint4*)(wl + j * HT_ASTR + (it & 7) * 8) =
            make_uint4(g.v[u].x & z, g.v[u].y & z, g.v[u].z & z, g.v[u].w & z);
    }
}

// a1 = act(sum of the planes + b1) for the lane's 8 columns as the bf16
// hi/lo pair (zeros outside the batch and past m)
template <int kS, bool kGelu>
__device__ __forceinline__ void ht_act(const HtP<kS>& g, const float* b1s, int k, bool ok,
                                       bf16x8& hi, bf16x8& lo) {
    float4 s0 = g.v[0][0], s1 = g.v[0][1];
#pragma unroll
    for (int q = 1; q < kS; ++q) {
        s0.x += g.v[q][0].x; s0.y += g.v[q][0].y; s0.z += g.v[q][0].z; s0.w += g.v[q][0].w;
        s1.x += g.v[q][1].x; s1.y += g.v[q][1].y; s1.z += g.v[q][1].z; s1.w += g.v[q][1].w;
    }
    const float4 c0 = *(const float4*)(b1s + (ok ? k : 0));
    const float4 c1 = *(const float4*)(b1s + (ok ? k : 0) + 4);
    const float av[8] = {s0.x + c0.x, s0.y + c0.y, s0.z + c0.z, s0.w + c0.w,
                         s1.x + c1.x, s1.y + c1.y, s1.z + c1.z, s1.w + c1.w};
    uint32_t hw[4], lw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float y0 = av[2 * e], y1 = av[2 * e + 1];
        const float g0 = kGelu ? gelu_erf(y0) : fmaxf(y0, 0.0f);
        const float g1 = kGelu ? gelu_erf(y1) : fmaxf(y1, 0.0f);
        split_bf16x2(ok ? g0 : 0.0f, ok ? g1 : 0.0f, hw[e], lw[e]);
    }
    hi = __builtin_bit_cast(bf16x8, make_uint4(hw[0], hw[1], hw[2], hw[3]));
    lo = __builtin_bit_cast(bf16x8, make_uint4(lw[0], lw[1], lw[2], lw[3]));
}

// up to 128 bins and two planes, two workgroups per CU (four waves per
// SIMD, at most 128 VGPRs)
template <int kS, int kNBB, bool kGelu>
__global__ __launch_bounds__(HT_THREADS)
__attribute__((amdgpu_waves_per_eu(kNBB <= 8 && kS <= 2 ? 4 : 1))) void head_tiled_kernel(
    const float* __restrict__ P, int B, int m, int nb, const float* __restrict__ b1,
    const uint16_t* __restrict__ W2, const float* __restrict__ b2,
    const float* __restrict__ bins, float ema_alpha, int ema_init,
    float* __restrict__ ema_state, float* __restrict__ expected, int32_t* __restrict__ rem_len,
    int len_max) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int row0 = blockIdx.x * HT_ROWS;
    constexpr int kStage = (int)(head_tiled_stage_bytes(kNBB) / 2);   // bf16 per stage
    uint16_t* const st0 = (uint16_t*)smem;
    uint16_t* const st1 = st0 + kStage;
    float* const b1s = (float*)(st1 + kStage);
    HtArgs a;
    a.P4 = (const float4*)P;
    a.W2 = W2;
    a.m = m;
    a.m4 = m >> 2;
    a.B = B;
    a.plane4 = (int64_t)B * a.m4;
    a.nb = nb;
    const int nchunk = (m + HT_KC - 1) / HT_KC;
    // wave wid: rows of group rg, K half kh of every chunk
    const int rg = wid & 3;
    const int kh = wid >> 2;
    const int row = row0 + rg * 16 + (lane & 15);   // the lane's A row (MFMA row lane % 16)
    const int kofs = kh * 32 + (lane >> 4) * 8;     // its 8 columns within a chunk
    const bool row_ok = row < B;

    f32x4 acc[kNBB];
#pragma unroll
    for (int j = 0; j < kNBB; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // the products of one chunk: the lane's A pair x kNBB bin blocks of W2
    auto products = [&](const uint16_t* wl, const bf16x8& h, const bf16x8& l) {
        // per group of 4 blocks, the hi products, then the lo ones:
        // consecutive MFMAs are independent
        constexpr int kG = kNBB < 4 ? kNBB : 4;
#pragma unroll
        for (int j0 = 0; j0 < kNBB; j0 += kG) {
            bf16x8_t wb[kG];
#pragma unroll
            for (int j = 0; j < kG; ++j)
                wb[j] = __builtin_bit_cast(bf16x8_t, *(const bf16x8*)(wl + ((j0 + j) * 16 + (lane & 15)) * HT_ASTR + kofs));
#pragma unroll
            for (int j = 0; j < kG; ++j)
                acc[j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, h), wb[j], acc[j0 + j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < kG; ++j)
                acc[j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, l), wb[j], acc[j0 + j], 0, 0, 0);
        }
    };

    // The partials and W2's chunks are loaded one chunk ahead (chunk c + 1's
    // partials are requested once chunk c is activated).  Loads complete in
    // issue order for the wait counter, so in each step W2, needed sooner,
    // is requested before the partials.
    // workgroups start at different chunks (block index mod chunks), so that
    // at any time the chip reads every column range of the partial rows, not
    // one 256-byte range of all of them (measured at 32768 x 1024 x 128: 48.9
    // against 51.9 us); the chunks' order in each row's sums changes with it
    const int rot = (int)(blockIdx.x % (unsigned)nchunk);
    auto chunk = [&](int c) { return c + rot < nchunk ? c + rot : c + rot - nchunk; };
    HtP<kS> p0;
    HtW<kNBB> w;
    ht_load_w(a, chunk(0), w);
    ht_load_p(a, row, chunk(0) * HT_KC + kofs, p0);
    for (int i = tid; i < m; i += HT_THREADS) b1s[i] = b1 ? b1[i] : 0.0f;
    ht_store_w(a, chunk(0), w, st0);
    if (nchunk > 1) ht_load_w(a, chunk(1), w);
    __syncthreads();

    // step c: activate chunk c and request chunk c + 1's partials, chunk c's
    // products on stage c % 2, W2 of chunk c + 1 into the other stage (last
    // read before the previous barrier)
    int c = 0;
    for (;; ++c) {
        const int k = chunk(c) * HT_KC + kofs;
        bf16x8 h, l;
        ht_act<kS, kGelu>(p0, b1s, k, row_ok && k < m, h, l);
        if (c + 1 < nchunk) ht_load_p(a, row, chunk(c + 1) * HT_KC + kofs, p0);
        products((c & 1) ? st1 : st0, h, l);
        if (c + 1 == nchunk) break;
        ht_store_w(a, chunk(c + 1), w, (c & 1) ? st0 : st1);
        if (c + 2 < nchunk) ht_load_w(a, chunk(c + 2), w);
        __syncthreads();
    }

    // the upper K half's logits join the lower half's, in that order, through
    // the stages (kNBB x 4 KiB; two stages hold kNBB x 4.5 KiB)
    {
        static_assert(4 * kNBB * 64 * 16 <= 2 * kStage * 2, "exchange fits the stages");
        f32x4* const xs = (f32x4*)smem;
        __syncthreads();                        // every wave's last products are done
        if (kh == 1) {
#pragma unroll
            for (int j = 0; j < kNBB; ++j) xs[(rg * kNBB + j) * 64 + lane] = acc[j];
        }
        __syncthreads();
        if (kh == 1) return;                    // no barrier follows
#pragma unroll
        for (int j = 0; j < kNBB; ++j) {
            const f32x4 o = xs[(rg * kNBB + j) * 64 + lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[j][v] += o[v];
        }
    }

    // softmax over the bins: element v of acc[j] is row 4 (lane / 16) + v of
    // the wave's 16, bin 16 j + lane % 16
    // logits with b2; absent bins (past nb) become -inf
    // and their bin values 0, so that the loops below need no conditions
    float bvl[kNBB];
#pragma unroll
    for (int j = 0; j < kNBB; ++j) {
        const int col = j * 16 + (lane & 15);
        const bool ok = col < nb;
        const int cc = ok ? col : 0;
        bvl[j] = ok ? bins[cc] : 0.0f;
        const float bias = b2 ? b2[cc] : 0.0f;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[j][v] = ok ? acc[j][v] + bias : -INFINITY;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < kNBB; ++j) mx = fmaxf(mx, acc[j][v]);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 16));
        float den = 0.0f, num = 0.0f;
#pragma unroll
        for (int j = 0; j < kNBB; ++j) {
            const float e = expf(acc[j][v] - mx);      // exp(-inf) = 0 for absent bins
            den += e;
            num += e * bvl[j];
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            den += __shfl_xor(den, o, 16);
            num += __shfl_xor(num, o, 16);
        }
        const int gr = row0 + rg * 16 + 4 * (lane >> 4) + v;
        if ((lane & 15) == 0 && gr < B) {
            const float E = num / den;
            expected[gr] = E;
            float y = E;
            if (ema_alpha > 0.0f) {
                y = ema_init ? E : ema_alpha * E + (1.0f - ema_alpha) * ema_state[gr];
                ema_state[gr] = y;
            }
            if (rem_len) {
                const float q = rintf(y);
                int32_t li;
                if (!(q >= 1.0f)) li = 1;
                else if (q >= (float)len_max) li = len_max;
                else li = (int32_t)q;
                rem_len[gr] = li;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The whole binned head in one kernel (bf16), for products that take one
// K-slice (no split-K): first product, bias, activation, second product,
// softmax, expectation, EMA and integerisation.
//
// Every workgroup computes one BM x BN tile of z1 = H W1^T over all of K,
// adds b1 and applies the activation.  The second product is linear in a1's
// columns, so the workgroup then multiplies its BN columns of a1 with the
// same BN columns of W2: the tile's share of every bin logit of its BM rows.
// The column tiles of a row block meet through a counter; the last to
// arrive sums the shares in column order (the same fixed order whatever the
// arrival order) and finishes its rows: b2, softmax over the bins, mean over
// the bin values, EMA, round half to even, clamp.  z1 never leaves the chip.
//
// The shares meet through the cache-maintenance-free exchange of the common
// header (device-coherent stores and loads, a counter per row block).
//
// Products that need a K-split take the two-kernel path instead (split-K
// product, then the head kernel): meeting the K-slices in this kernel as
// well put two exchanges and the whole head of the last tile on one
// workgroup's critical path, which measured slower than the kernel boundary.
// ---------------------------------------------------------------------------
constexpr int FU_NB_MAX = 128;            // bins of the fused head (its logits fit the LDS)
constexpr int FU_NBP = FU_NB_MAX + 4;     // fp32 per LDS row of logits (banks spread by rows)
constexpr int FU_MAX_TICKETS = kMaxTickets;

__device__ inline void fu_store(f32x4 v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    xch_store(__builtin_bit_cast(u32x4, v), r, off);
}
__device__ inline f32x4 fu_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(f32x4, xch_load(r, off));
}

__device__ inline f32x4 fu_chunk(const f32x16& a, int q) {
    return f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
}

struct FusedArgs {
    const char* A;            // hidden [M, Kd] bf16
    const char* W;            // w1 [N, Kd] bf16
    const float* b1;          // [N] or null
    const uint16_t* W2;       // [nb, N] bf16
    const float* b2;          // [nb] or null
    const float* bins;        // [nb]
    float* lpart;             // logit shares: [tiles_m][tiles_n][blocks][1024] (tiles_n > 1)
    uint32_t* tix_row;        // [tiles_m]
    float* ema_state;
    float* expected;
    int32_t* rem_len;
    int M, N, Kd, nb, tiles_n, act, ema_init, len_max;
    float ema_alpha;
};

template <class SH>
__global__ __launch_bounds__(SH::THREADS) void predict_fused_kernel(FusedArgs a) {
    constexpr int MI = SH::MI, NJ = SH::NJ, T = SH::THREADS, NW = T / 64;
    constexpr int BM = SH::BM, BN = SH::BN;
    constexpr int ZST = BN * 4 + 16;             // bytes per LDS row of the z1 / a1 tile
    constexpr int C8 = BN / 8;                   // 8-column chunks per row
    static_assert(T % C8 == 0, "a thread keeps its chunk column");
    constexpr int NBI = BM / 32;                 // row blocks of the logit product
    constexpr int MAXB = (NBI * (FU_NB_MAX / 32) + NW - 1) / NW;   // logit blocks per wave
    constexpr int LPR = T / BM;                  // lanes per row in the softmax
    static_assert(LPR >= 1 && (LPR & (LPR - 1)) == 0 && LPR <= 64, "lanes per row");
    // the main loop's ring, reused for the z1 / a1 tile and then the logits
    constexpr int kMainBytes = SH::LDS;
    constexpr int kLogitBytes = (BM * FU_NBP + 2 * FU_NB_MAX) * 4;   // logits, bin values, b2
    constexpr int kTileBytes = BM * ZST;
    constexpr int kEpiBytes = kLogitBytes > kTileBytes ? kLogitBytes : kTileBytes;
    __shared__ __attribute__((aligned(1024))) char lds_raw[kMainBytes > kEpiBytes ? kMainBytes : kEpiBytes];
    __shared__ uint32_t s_ticket;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int wm = wid / SH::WN, wn = wid % SH::WN;
    const int r32 = lane & 31;
    const int khalf = lane >> 5;
    const int64_t row_bytes = (int64_t)a.Kd * 2;
    const G1Work w = g1_work<SH>(1, a.tiles_n, row_bytes, blockIdx.x, gridDim.x);
    f32x16 acc[MI][NJ];
    g1_mainloop<2, SH>(a.A, a.W, a.M, a.N, row_bytes, w, lds_raw, acc);

    // The head's global reads (W2 fragments, b1, b2, bin values, EMA state)
    // are all requested at once: one memory latency instead of one per use.
    const int nbj = (a.nb + 31) >> 5;
    const int nblk = NBI * nbj;
    bf16x8 wf[MAXB][BN / 16];
    f32x4 b1v[2];                                 // b1 of this thread's 8-column chunk
    float binv, b2v, ema_prev;
    const int c8 = tid % C8;
    const int r = tid / LPR, sub = tid % LPR;     // the row this thread finishes in 5)
    const int gr = w.tm * BM + r;
    auto prefetch = [&]() {
#pragma unroll
        for (int u = 0; u < MAXB; ++u) {
            const int blk = wid + u * NW;
            const int jrow = (blk / NBI) * 32 + r32;
#pragma unroll
            for (int ks = 0; ks < BN / 16; ++ks) {
                // clamped, unconditional; m % 8 == 0, so a chunk is wholly in or out
                const int c = w.tn * BN + ks * 16 + 8 * khalf;
                const bool ok = blk < nblk && jrow < a.nb && c < a.N;
                const bf16x8 t = *(const bf16x8*)(a.W2 + (ok ? (int64_t)jrow * a.N + c : 0));
                wf[u][ks] = t & (ok ? (short)-1 : (short)0);
            }
        }
        {
            // m % 8 == 0: the chunk is wholly in or out; b1 is 16-byte aligned
            const int gcol = w.tn * BN + c8 * 8;
            b1v[0] = b1v[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (a.b1 && gcol < a.N) {
                b1v[0] = *(const f32x4*)(a.b1 + gcol);
                b1v[1] = *(const f32x4*)(a.b1 + gcol + 4);
            }
        }
        const int jb = tid < a.nb ? tid : 0;
        binv = tid < a.nb ? a.bins[jb] : 0.0f;
        b2v = (a.b2 && tid < a.nb) ? a.b2[jb] : 0.0f;
        ema_prev = (a.ema_alpha > 0.0f && !a.ema_init) ? a.ema_state[gr < a.M ? gr : a.M - 1] : 0.0f;
    };

    prefetch();
    __syncthreads();                         // the last products have read the LDS

    // 1) z1 into LDS rows [BM][ZST bytes] (fp32); then, a chunk of 8 columns
    //    at a time, bias and activation, written back in place as the bf16
    //    pair [hi x 8 | lo x 8].  Element v of lane l of a 32 x 32 block is
    //    row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.
    char* zt = lds_raw;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int col = wn * 32 * NJ + j * 32 + r32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = wm * 32 * MI + i * 32 + 8 * (v >> 2) + 4 * khalf + (v & 3);
                *(float*)(zt + row * ZST + col * 4) = acc[i][j][v];
            }
        }
    __syncthreads();
    {
        const bool cok = w.tn * BN + c8 * 8 < a.N;
#pragma unroll 1
        for (int e = tid; e < BM * C8; e += T) {
            char* pz = zt + (e / C8) * ZST + c8 * 32;
            const f32x4 z0 = *(const f32x4*)pz, z1 = *(const f32x4*)(pz + 16);
            float x[8];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k] = cok ? apply_act(z0[k] + b1v[0][k], a.act) : 0.0f;
                x[k + 4] = cok ? apply_act(z1[k] + b1v[1][k], a.act) : 0.0f;
            }
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) split_bf16x2(x[2 * k], x[2 * k + 1], hi[k], lo[k]);
            *(uint4*)pz = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *(uint4*)(pz + 16) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
    }
    __syncthreads();

    // 2) this tile's share of the bin logits, [BM rows] x [bins] over its BN
    //    columns: v_mfma_f32_32x32x16_bf16 with A = a1 rows (hi, then lo) and
    //    B = W2 rows.  Wave wid takes the blocks wid, wid + NW, ...
    f32x16 lg[MAXB];
#pragma unroll
    for (int u = 0; u < MAXB; ++u) {
#pragma unroll
        for (int e = 0; e < 16; ++e) lg[u][e] = 0.0f;
        const int blk = wid + u * NW;
        if (blk < nblk) {
            const int ib = blk % NBI;
#pragma unroll
            for (int ks = 0; ks < BN / 16; ++ks) {
                const char* pa = zt + (ib * 32 + r32) * ZST + (2 * ks + khalf) * 32;
                const bf16x8_t h = __builtin_bit_cast(bf16x8_t, *(const bf16x8*)pa);
                const bf16x8_t l = __builtin_bit_cast(bf16x8_t, *(const bf16x8*)(pa + 16));
                const bf16x8_t b = __builtin_bit_cast(bf16x8_t, wf[u][ks]);
                lg[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h, b, lg[u], 0, 0, 0);
                lg[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l, b, lg[u], 0, 0, 0);
            }
        }
    }

    // 3) the column tiles of the row block meet; the last to arrive sums the
    //    shares in column order (share layout: float4 q of lane l of block
    //    blk at (blk 4 + q) 64 + l).  It reads its own share back too (its
    //    stores have completed), so every load is unconditional; tiles past
    //    the last read 0 (an offset past the buffer); the sum starts at -0,
    //    which adds exactly.
    if (a.tiles_n > 1) {
        const uint32_t share = (uint32_t)nblk * 1024u;            // floats per share
        const __amdgpu_buffer_rsrc_t rl =
            xch_rsrc(a.lpart + (size_t)w.tm * a.tiles_n * share, (uint32_t)a.tiles_n * share * 4u);
#pragma unroll
        for (int u = 0; u < MAXB; ++u) {
            const int blk = wid + u * NW;
            if (blk < nblk)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    fu_store(fu_chunk(lg[u], q), rl,
                             (uint32_t)w.tn * share * 4u + (uint32_t)((blk * 4 + q) * 64 + lane) * 16u);
        }
        xch_wait_stores();
        if (!xch_last_arrival(&a.tix_row[w.tm], (uint32_t)a.tiles_n, &s_ticket)) return;
        constexpr int G = 8;                  // shares loaded together
#pragma unroll
        for (int u = 0; u < MAXB; ++u) {
            const int blk = wid + u * NW;
            if (blk >= nblk) continue;
            f32x4 sum[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[q] = f32x4{-0.0f, -0.0f, -0.0f, -0.0f};
#pragma unroll 1
            for (int t0 = 0; t0 < a.tiles_n; t0 += G) {
                f32x4 v[G][4];
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int t = t0 + g;
                        const uint32_t off = (uint32_t)t * share * 4u +
                                             (uint32_t)((blk * 4 + q) * 64 + lane) * 16u;
                        v[g][q] = fu_load(rl, t < a.tiles_n ? off : kXchOob);
                    }
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int q = 0; q < 4; ++q) sum[q] += v[g][q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) lg[u][4 * q + e] = sum[q][e];
        }
    }

    // 4) logits into LDS rows [BM][FU_NBP], the bin values and b2 beside
    //    them; then LPR lanes per row: + b2, softmax, mean over the bin
    //    values, EMA, integerisation
    __syncthreads();                          // every wave has read a1 from LDS
    float* zl = (float*)lds_raw;
    float* sbin = zl + BM * FU_NBP;           // [FU_NB_MAX] bin values, then [FU_NB_MAX] b2
    if (tid < FU_NB_MAX) {
        sbin[tid] = binv;
        sbin[FU_NB_MAX + tid] = b2v;
    }
#pragma unroll
    for (int u = 0; u < MAXB; ++u) {
        const int blk = wid + u * NW;
        if (blk >= nblk) continue;
        const int ib = blk % NBI, jb = blk / NBI;
        const int j = jb * 32 + r32;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = ib * 32 + 8 * (v >> 2) + 4 * khalf + (v & 3);
            zl[row * FU_NBP + j] = lg[u][v];
        }
    }
    __syncthreads();
    const float* zr = zl + r * FU_NBP;
    float zmax = -INFINITY;
#pragma unroll 4
    for (int j = sub; j < a.nb; j += LPR) zmax = fmaxf(zmax, zr[j] + sbin[FU_NB_MAX + j]);
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, LPR));
    float den = 0.0f, num = 0.0f;
#pragma unroll 4
    for (int j = sub; j < a.nb; j += LPR) {
        const float e = expf(zr[j] + sbin[FU_NB_MAX + j] - zmax);
        den += e;
        num += e * sbin[j];
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) {
        den += __shfl_xor(den, o, LPR);
        num += __shfl_xor(num, o, LPR);
    }
    if (sub == 0 && gr < a.M) {
        const float E = num / den;
        a.expected[gr] = E;
        float y = E;
        if (a.ema_alpha > 0.0f) {
            y = a.ema_init ? E : a.ema_alpha * E + (1.0f - a.ema_alpha) * ema_prev;
            a.ema_state[gr] = y;
        }
        if (a.rem_len) {
            const float q = rintf(y);
            int32_t li;
            if (!(q >= 1.0f)) li = 1;
            else if (q >= (float)a.len_max) li = a.len_max;
            else li = (int32_t)q;
            a.rem_len[gr] = li;
        }
    }
}

// ---------------------------------------------------------------------------
// (f3) between the regression head's first two layers: fixed-order split-K
// reduction, bias, ReLU, and the operand of the next product (bf16, round
// to nearest even, or fp32)
// ---------------------------------------------------------------------------
constexpr int ACT_THREADS = 256;
constexpr int ACT_BATCH = 4;      // float4 items per thread in flight

template <int kS, bool kBF16>
__global__ __launch_bounds__(ACT_THREADS) void act_kernel(const float* __restrict__ P,
                                                          int64_t items, int m4,
                                                          const float* __restrict__ bias,
                                                          void* __restrict__ out) {
    const float4* P4 = (const float4*)P;
    for (int64_t base = (int64_t)blockIdx.x * ACT_THREADS * ACT_BATCH; base < items;
         base += (int64_t)gridDim.x * ACT_THREADS * ACT_BATCH) {
        float4 v[ACT_BATCH][kS];
#pragma unroll
        for (int i = 0; i < ACT_BATCH; ++i) {
            const int64_t e = base + i * ACT_THREADS + threadIdx.x;
            const int64_t o = e < items ? e : 0;
#pragma unroll
            for (int q = 0; q < kS; ++q) {
                const f32x4 t = __builtin_nontemporal_load((const f32x4*)&P4[q * items + o]);
                v[i][q] = make_float4(t[0], t[1], t[2], t[3]);
            }
        }
#pragma unroll
        for (int i = 0; i < ACT_BATCH; ++i) {
            const int64_t e = base + i * ACT_THREADS + threadIdx.x;
            if (e >= items) break;
            float4 sum = v[i][0];
#pragma unroll
            for (int q = 1; q < kS; ++q) {
                sum.x += v[i][q].x; sum.y += v[i][q].y; sum.z += v[i][q].z; sum.w += v[i][q].w;
            }
            const int c = (int)(e % m4) * 4;
            const float4 bv = bias ? *(const float4*)(bias + c) : make_float4(0.f, 0.f, 0.f, 0.f);
            const float a0 = fmaxf(sum.x + bv.x, 0.0f), a1 = fmaxf(sum.y + bv.y, 0.0f);
            const float a2 = fmaxf(sum.z + bv.z, 0.0f), a3 = fmaxf(sum.w + bv.w, 0.0f);
            if constexpr (kBF16) {
                ((uint2*)out)[e] = make_uint2(pack_bf16x2_rne(a0, a1), pack_bf16x2_rne(a2, a3));
            } else {
                ((float4*)out)[e] = make_float4(a0, a1, a2, a3);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Tiles and split-K factor of one product [M, K] x [N, K]^T: the smallest
// cost over the 64 x 64, 128 x 64 and 128 x 128 tiles and 1 to 16 K-slices (a
// power of two; at least two K-steps each).  The cost, in ns:
//  * the K-steps of the busiest CU.  A step (128 bytes of every row) of the w
//    workgroups that a CU holds at once takes at least 270, 350 or 430 ns
//    (the ring's latency at 64 x 64, 128 x 64, 128 x 128), and its bytes at
//    107 B/ns; in fp32, its products at 256 FLOP per cycle and 2.4 GHz.  The
//    rings' LDS admits three, two and one workgroups;
//  * the partials of a split product, written and read back by the next
//    kernel, at 4.5 B/ps, and 120 ns of that kernel per plane.
// Fitted to whole star_predict calls in captured graphs (bf16, us), which it
// puts in the order measured:
//   1024 x 512 x 4096: 64 x 64 with 4 slices 15.8, 128 x 64 with 4 16.9,
//     128 x 128 with 8 17.0, 128 x 128 with 4 17.8, 64 x 64 with 2 19.3;
//   2048 x 512 x 4096: 128 x 128 with 4 22.8, 128 x 64 with 4 23.0, 64 x 64
//     with 2 24.0, 128 x 64 with 2 25.2, 128 x 128 with 2 26.5;
//   512 x 512 x 4096: 64 x 64 with 8 13.3, 128 x 64 with 8 14.3, 64 x 64
//     with 4 14.5;  64 rows: 64 x 64 with 8 11.3, with 16 12.1.
constexpr int64_t G1_MAX_SPLIT_BYTES = STAR_NOALLOC_SCRATCH_BYTES - STAR_WS_HEADER_BYTES;
GemmPlan plan_gemm(int M, int N, int K, int elem) {
    GemmPlan best;
    double best_cost = 0.0;
    struct Cand { int shape, bm, bn, at_once; double floor_ns; };
    const Cand cands[3] = {{GemmPlan::kBig, G1Big::BM, G1Big::BN, 1, 430.0},
                           {GemmPlan::kMid, G1Mid::BM, G1Mid::BN, 2, 350.0},
                           {GemmPlan::kSmall, G1Small::BM, G1Small::BN, 3, 270.0}};
    const int64_t steps = ceil_div((int64_t)K * elem, 128);
    for (const Cand& c : cands) {
        const int64_t tm = ceil_div(M, c.bm), tn = ceil_div(N, c.bn);
        const double load_ns = (c.bm + c.bn) * 128 / 107.0;
        const double mfma_ns = elem == 4 ? c.bm * c.bn * 64 / 256 / 2.4 : 0.0;
        for (int s = 1; s <= 16; s *= 2) {
            // a split product's partials stay within the allocation-free
            // entry point's scratch, which one K-slice may need less of
            const int64_t partials = (int64_t)s * M * N * 4;
            if (s > 1 && (steps < 2 * s || partials > G1_MAX_SPLIT_BYTES)) break;
            // nor do narrow tiles take more of it than 128 x 128 ones would,
            // by the logit shares of the fused kernel (up to 128 bins)
            if (s == 1 && c.shape != GemmPlan::kBig && tn > 1 &&
                tm * c.bm * tn * FU_NB_MAX * 4 > G1_MAX_SPLIT_BYTES)
                continue;
            const int64_t w = ceil_div(tm * tn * s, 256);          // on the busiest CU
            const double held = (double)(w < c.at_once ? w : c.at_once);
            double step_ns = held * (load_ns > mfma_ns ? load_ns : mfma_ns);
            if (step_ns < c.floor_ns) step_ns = c.floor_ns;
            const double cost = (double)ceil_div(steps, s) * step_ns * (w / held) +
                                (s > 1 ? partials / 4.5e3 + 120.0 * s : 0.0);
            if ((c.shape == GemmPlan::kBig && s == 1) || cost < best_cost) {
                best.shape = c.shape;
                best.tiles_m = (int)tm;
                best.tiles_n = (int)tn;
                best.splits = s;
                best_cost = cost;
            }
        }
    }
    if (best.shape == GemmPlan::kBig && best.splits == 1) {
        const int hm = (int)ceil_div(M, G1Huge::BM), hn = (int)ceil_div(N, G1Huge::BN);
        if ((int64_t)hm * hn >= G1_HUGE_MIN_TILES) {       // 256 x 256 tiles
            best.shape = GemmPlan::kHuge;
            best.tiles_m = hm;
            best.tiles_n = hn;
        }
    }
    return best;
}

// Products the fused kernel takes: one K-slice (no split-K), a tile shape
// with an LDS epilogue, at most FU_NB_MAX bins, and a counter per row block
// in the workspace header.  Measured against the two-kernel path with one
// slice (64 bins): 49.5 against 52.7 us at 8192 x 512 x 4096, 48.6 against 60.4
// at 4096 x 1024 x 4096, 55.0 against 63.5 at 6622 x 576 x 2928, 30.9 against
// 30.6 at 16384 x 256 x 2048.
static bool fused_fits(const GemmPlan& g, int nb) {
    if (g.shape != GemmPlan::kSmall && g.shape != GemmPlan::kBig && g.shape != GemmPlan::kMid)
        return false;
    if (nb > FU_NB_MAX || g.splits != 1) return false;
    return g.tiles_n == 1 || g.tiles_m <= FU_MAX_TICKETS;
}

static int gemm_bm(int shape) {
    return shape == GemmPlan::kSmall ? G1Small::BM : shape == GemmPlan::kHuge ? G1Huge::BM : G1Big::BM;
}

PredictPlan plan_predict(const star_predict_params& p, bool tiled_ok, bool fused_ok) {
    PredictPlan pl;
    const GemmPlan g = plan_gemm(p.n_req, p.d_hidden, p.d_model, p.dtype == STAR_BF16 ? 2 : 4);
    pl.gemm = g;
    const int s = g.splits;
    pl.splits = s;
    if (fused_ok && p.dtype == STAR_BF16 && fused_fits(g, p.n_bins)) {
        pl.fused = true;
        const size_t bm = (size_t)gemm_bm(g.shape);
        const size_t tiles = (size_t)g.tiles_m * g.tiles_n;
        const size_t nb32 = (size_t)((p.n_bins + 31) / 32) * 32;
        pl.lpart_bytes = g.tiles_n > 1 ? align_up(tiles * bm * nb32 * sizeof(float), 256) : 0;
        pl.partial_bytes = pl.lpart_bytes;
        pl.head_rows = (int)bm;
        return pl;
    }
    pl.partial_bytes = (size_t)s * (size_t)p.n_req * (size_t)p.d_hidden * sizeof(float);
    pl.head_tiled = tiled_ok && p.dtype == STAR_BF16 && p.n_req >= HT_MIN_REQ &&
                    s <= HT_MAX_SPLITS;
    pl.head_rows = pl.head_tiled ? HT_ROWS : HD_RB;
    pl.head_lds = pl.head_tiled ? head_tiled_lds(p.n_bins, p.d_hidden)
                                : head_rows_lds(p.dtype == STAR_BF16, p.d_hidden, p.n_bins);
    return pl;
}

template <class SH>
static hipError_t launch_fused_shape(const PredictPlan& pl, const FusedArgs& a, hipStream_t stream) {
    const dim3 grid(pl.gemm.tiles_m * pl.gemm.tiles_n);
    hipLaunchKernelGGL((predict_fused_kernel<SH>), grid, dim3(SH::THREADS), 0, stream, a);
    return hipGetLastError();
}

static hipError_t launch_fused(const star_predict_params& p, const PredictPlan& pl,
                               const void* hidden, const void* w1, const float* b1,
                               const void* w2, const float* b2, const float* bins,
                               float* ema_state, float* expected, int32_t* rem_len, char* scratch,
                               uint32_t* tickets, hipStream_t stream) {
    FusedArgs a;
    a.A = (const char*)hidden;
    a.W = (const char*)w1;
    a.b1 = b1;
    a.W2 = (const uint16_t*)w2;
    a.b2 = b2;
    a.bins = bins;
    a.lpart = (float*)scratch;
    a.tix_row = tickets;
    a.ema_state = ema_state;
    a.expected = expected;
    a.rem_len = rem_len;
    a.M = p.n_req;
    a.N = p.d_hidden;
    a.Kd = p.d_model;
    a.nb = p.n_bins;
    a.tiles_n = pl.gemm.tiles_n;
    a.act = p.act;
    a.ema_init = p.ema_init;
    a.len_max = p.len_max;
    a.ema_alpha = p.ema_alpha;
    switch (pl.gemm.shape) {
        case GemmPlan::kSmall: return launch_fused_shape<G1Small>(pl, a, stream);
        case GemmPlan::kBig: return launch_fused_shape<G1Big>(pl, a, stream);
        case GemmPlan::kMid: return launch_fused_shape<G1Mid>(pl, a, stream);
    }
    return hipErrorInvalidValue;
}

template <bool kBF16, int kS, bool kReg, int kPF>
static hipError_t launch_head_rows(const star_predict_params& p, const PredictPlan& pl,
                                   const float* partials, const float* b1, const void* w2,
                                   const float* b2, const float* bins, float* ema_state,
                                   float* expected, int32_t* rem_len, float b4,
                                   hipStream_t stream) {
    if (pl.head_lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)head_kernel<kBF16, kS, kReg, kPF>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)pl.head_lds);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)ceil_div(p.n_req, HD_RB));
    hipLaunchKernelGGL((head_kernel<kBF16, kS, kReg, kPF>), grid, dim3(HD_THREADS), pl.head_lds,
                       stream, partials, p.n_req, p.d_hidden, p.n_bins, b1, w2, b2, bins, p.act,
                       p.ema_alpha, p.ema_init, ema_state, expected, rem_len, p.len_max, b4);
    return hipGetLastError();
}

template <int kS, int kNBB, bool kGelu>
static hipError_t launch_head_tiled_act(const star_predict_params& p, const PredictPlan& pl,
                                    const float* partials, const float* b1, const void* w2,
                                    const float* b2, const float* bins, float* ema_state,
                                    float* expected, int32_t* rem_len, hipStream_t stream) {
    if (pl.head_lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)head_tiled_kernel<kS, kNBB, kGelu>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)pl.head_lds);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)ceil_div(p.n_req, HT_ROWS));
    hipLaunchKernelGGL((head_tiled_kernel<kS, kNBB, kGelu>), grid, dim3(HT_THREADS), pl.head_lds, stream,
                       partials, p.n_req, p.d_hidden, p.n_bins, b1, (const uint16_t*)w2, b2, bins,
                       p.ema_alpha, p.ema_init, ema_state, expected, rem_len, p.len_max);
    return hipGetLastError();
}

template <int kS, int kNBB>
static hipError_t launch_head_tiled(const star_predict_params& p, const PredictPlan& pl,
                                    const float* partials, const float* b1, const void* w2,
                                    const float* b2, const float* bins, float* ema_state,
                                    float* expected, int32_t* rem_len, hipStream_t stream) {
    return p.act == STAR_ACT_GELU_ERF
        ? launch_head_tiled_act<kS, kNBB, true>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, stream)
        : launch_head_tiled_act<kS, kNBB, false>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, stream);
}

// The tiled head only for the bf16 binned head with at most HT_MAX_SPLITS
// planes (the plan never picks it elsewhere).
template <bool kBF16, int kS, bool kReg>
static hipError_t launch_head_s(const star_predict_params& p, const PredictPlan& pl,
                                const float* partials, const float* b1, const void* w2,
                                const float* b2, const float* bins, float* ema_state,
                                float* expected, int32_t* rem_len, float b4, hipStream_t stream) {
    if constexpr (kBF16 && !kReg && kS <= HT_MAX_SPLITS) {
        if (pl.head_tiled) {
            const int nbb = head_tiled_blocks(p.n_bins);
            return nbb == 4 ? launch_head_tiled<kS, 4>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, stream)
                 : nbb == 8 ? launch_head_tiled<kS, 8>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, stream)
                            : launch_head_tiled<kS, 16>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, stream);
        }
    }
    if (pl.head_tiled || pl.head_rows != HD_RB) return hipErrorInvalidValue;
    if constexpr (kBF16) {
        if (ceil_div(p.n_req, HD_RB) > HD_LOWREG_GROUPS)
            return launch_head_rows<kBF16, kS, kReg, HD_W2PF_LOW>(p, pl, partials, b1, w2, b2, bins,
                                                                 ema_state, expected, rem_len, b4,
                                                                 stream);
    }
    return launch_head_rows<kBF16, kS, kReg, HD_W2PF>(p, pl, partials, b1, w2, b2, bins, ema_state,
                                                      expected, rem_len, b4, stream);
}

template <bool kBF16, bool kReg = false>
static hipError_t launch_head(const star_predict_params& p, const PredictPlan& pl,
                              const float* partials, const float* b1, const void* w2,
                              const float* b2, const float* bins, float* ema_state,
                              float* expected, int32_t* rem_len, hipStream_t stream,
                              float b4 = 0.0f) {
    switch (pl.splits) {
        case 1: return launch_head_s<kBF16, 1, kReg>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, b4, stream);
        case 2: return launch_head_s<kBF16, 2, kReg>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, b4, stream);
        case 4: return launch_head_s<kBF16, 4, kReg>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, b4, stream);
        case 8: return launch_head_s<kBF16, 8, kReg>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, b4, stream);
        case 16: return launch_head_s<kBF16, 16, kReg>(p, pl, partials, b1, w2, b2, bins, ema_state, expected, rem_len, b4, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_predict(const star_predict_params& p, const PredictPlan& pl, const void* hidden,
                          const void* w1, const float* b1, const void* w2, const float* b2,
                          const float* bins, float* ema_state, float* expected, int32_t* rem_len,
                          char* scratch, uint32_t* tickets, hipStream_t stream) {
    if (p.n_req == 0) return hipSuccess;
    if (pl.fused)
        return launch_fused(p, pl, hidden, w1, b1, w2, b2, bins, ema_state, expected, rem_len,
                            scratch, tickets, stream);
    float* partials = (float*)scratch;
    hipError_t e = launch_gemm(pl.gemm, p.dtype == STAR_BF16, hidden, w1, partials, p.n_req,
                               p.d_hidden, p.d_model, stream);
    if (e != hipSuccess) return e;
    return p.dtype == STAR_BF16 ? launch_head<true>(p, pl, partials, b1, w2, b2, bins,
                                                    ema_state, expected, rem_len, stream)
                                : launch_head<false>(p, pl, partials, b1, w2, b2, bins,
                                                     ema_state, expected, rem_len, stream);
}

// ---------------------------------------------------------------------------
// Two batches in one launch.  Blocks [0, gemm_blocks) compute the next
// batch's first-layer split-K partials (64 x 64 or 128 x 64 tiles); the blocks
// after them run the previous batch's head from its partials.  The roles share no
// data, and each block takes one role for its whole life, so they need no
// synchronisation.  One launch removes the kernel boundary between the
// previous batch's head and the next batch's product, and the head's
// workgroups take the CUs as the product's workgroups leave them.
// ---------------------------------------------------------------------------
struct OverlapArgs {
    // the next batch's product
    const char* A;
    const char* W1;
    float* Pn;
    int M, N, Kd, splits, tiles_n, gemm_blocks;
    // the previous batch's head
    const float* Pp;
    const float* b1;
    const void* w2;
    const float* b2;
    const float* bins;
    float* ema_state;
    float* expected;
    int32_t* rem_len;
    int B, m, nb, act, ema_init, len_max;
    float ema_alpha;
};
// W2 fragments the head role loads at a time.  LDS alone sets the workgroups
// per compute unit (two of 128 x 64, three of 64 x 64), so more fragments would
// cost no occupancy, but they take longer to request: 8 and 16 were 2.2 and 3.8%
// slower than 4 over 171 shapes of 128 to 4096 rows with 128 x 64 tiles, 2.8 and
// 5.7% with 64 x 64 (1024 x 512 x 4096, 128 bins: 14.7, 14.9, 14.9 us per batch).
constexpr int OV_W2PF = 4;

template <int kS, class SH>
__global__ __launch_bounds__(HD_THREADS) void predict_overlap_kernel(OverlapArgs a) {
    static_assert(SH::THREADS == HD_THREADS, "one block size for both roles");
    __shared__ __attribute__((aligned(1024))) char lds[SH::LDS];
    if ((int)blockIdx.x < a.gemm_blocks)
        gemm1_tile<2, SH>(a.A, a.W1, a.Pn, a.M, a.N, a.Kd, a.splits, a.tiles_n, blockIdx.x,
                          a.gemm_blocks, lds);
    else
        head_rows<true, kS, false, OV_W2PF>(a.Pp, a.B, a.m, a.nb, a.b1, a.w2, a.b2, a.bins,
                                            a.act, a.ema_alpha, a.ema_init, a.ema_state,
                                            a.expected, a.rem_len, a.len_max, 0.0f,
                                            (int)blockIdx.x - a.gemm_blocks, lds);
}

template <class SH>
static hipError_t launch_overlap_shape(int head_blocks, const OverlapArgs& a,
                                       hipStream_t stream) {
    const dim3 g((unsigned)(a.gemm_blocks + head_blocks)), t(HD_THREADS);
    switch (a.splits) {
        case 1: hipLaunchKernelGGL((predict_overlap_kernel<1, SH>), g, t, 0, stream, a); break;
        case 2: hipLaunchKernelGGL((predict_overlap_kernel<2, SH>), g, t, 0, stream, a); break;
        case 4: hipLaunchKernelGGL((predict_overlap_kernel<4, SH>), g, t, 0, stream, a); break;
        case 8: hipLaunchKernelGGL((predict_overlap_kernel<8, SH>), g, t, 0, stream, a); break;
        case 16: hipLaunchKernelGGL((predict_overlap_kernel<16, SH>), g, t, 0, stream, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_predict_overlap(const star_predict_params& p, const PredictPlan& pl,
                                  const void* hidden_next, float* partials_next,
                                  const float* partials_prev, const void* w1, const float* b1,
                                  const void* w2, const float* b2, const float* bins,
                                  float* ema_state, float* expected, int32_t* rem_len,
                                  hipStream_t stream) {
    if (pl.fused) return hipErrorInvalidValue;
    if (p.n_req == 0 || (!hidden_next && !partials_prev)) return hipSuccess;
    const bool bf16 = p.dtype == STAR_BF16;
    const int head_blocks = (int)ceil_div(p.n_req, HD_RB);
    // One launch, and its tiles: the product's K-slices are star_predict's, so
    // the sums are the same over the same slices in the same order whatever the
    // tile.  128 x 64 tiles, but 64 x 64 ones where those would leave almost half
    // of the compute units without a product workgroup; 128 x 128 tiles, whose
    // workgroups are not the head's size, give way only where the product is
    // short or leaves places for the head (two workgroups of 128 x 64 per compute
    // unit).  Both lines from 570 shapes of 128 to 4096 rows, us per batch (64 x 64,
    // 128 x 64, two launches):
    //   895 x 280 x 3032, 4 slices, 140 wide workgroups: 10.7, 12.9, 15.4
    //   174 x 808 x 7104, 8 slices, 208: 15.8, 14.1
    //   1884 x 272 x 1720, 4 slices of 7 steps, 300: 14.6, 15.3, 17.8
    //   1654 x 256 x 5472, 8 slices of 11 steps, 416: 21.2, 19.4, 21.2
    //   1789 x 928 x 7416, 2 slices of 58 steps, 420: 75.5, 60.2, 53.7
    //   3778 x 496 x 2856, 2 slices of 23 steps, 480: 38.6, 36.4, 33.8
    //   3824 x 424 x 1544, 1 slice of 25 steps, 210: 25.5, 25.3, 31.1
    constexpr int OV_MIN_WIDE = 140;       // fewer wide workgroups take 64 x 64 tiles
    constexpr int OV_MAX_WIDE = 384;       // wide workgroups that leave the head its places
    constexpr int OV_SHORT_STEPS = 19;     // K-steps per slice of a short product
    GemmPlan g = pl.gemm;
    GemmPlan wide = g;
    wide.shape = GemmPlan::kMid;
    wide.tiles_m = (int)ceil_div(p.n_req, G1Mid::BM);
    wide.tiles_n = (int)ceil_div(p.d_hidden, G1Mid::BN);
    const int64_t wide_blocks = (int64_t)wide.tiles_m * wide.tiles_n * wide.splits;
    const int64_t steps = ceil_div((int64_t)p.d_model * 2, (int64_t)G1Mid::STEP * g.splits);
    const bool small = g.shape == GemmPlan::kSmall && wide_blocks <= OV_MIN_WIDE &&
                       pl.head_lds <= (size_t)G1Small::LDS;
    const bool narrow = g.shape == GemmPlan::kSmall || g.shape == GemmPlan::kMid ||
                        (g.shape == GemmPlan::kBig &&
                         (steps <= OV_SHORT_STEPS || wide_blocks <= OV_MAX_WIDE));
    const bool one = hidden_next && partials_prev && bf16 && narrow && !pl.head_tiled &&
                     pl.head_rows == HD_RB && pl.head_lds <= (size_t)G1Mid::LDS;
    const bool mid = one && !small;
    if (mid) g = wide;
    if (!one) {          // the two kernels one after the other, same results
        if (partials_prev) {
            const hipError_t e =
                bf16 ? launch_head<true>(p, pl, partials_prev, b1, w2, b2, bins, ema_state,
                                         expected, rem_len, stream)
                     : launch_head<false>(p, pl, partials_prev, b1, w2, b2, bins, ema_state,
                                          expected, rem_len, stream);
            if (e != hipSuccess) return e;
        }
        if (hidden_next)
            return launch_gemm(g, bf16, hidden_next, w1, partials_next, p.n_req, p.d_hidden,
                               p.d_model, stream);
        return hipSuccess;
    }
    OverlapArgs a;
    a.A = (const char*)hidden_next;
    a.W1 = (const char*)w1;
    a.Pn = partials_next;
    a.M = p.n_req;
    a.N = p.d_hidden;
    a.Kd = p.d_model;
    a.splits = g.splits;
    a.tiles_n = g.tiles_n;
    a.gemm_blocks = g.tiles_m * g.tiles_n * g.splits;
    a.Pp = partials_prev;
    a.b1 = b1;
    a.w2 = w2;
    a.b2 = b2;
    a.bins = bins;
    a.ema_state = ema_state;
    a.expected = expected;
    a.rem_len = rem_len;
    a.B = p.n_req;
    a.m = p.d_hidden;
    a.nb = p.n_bins;
    a.act = p.act;
    a.ema_init = p.ema_init;
    a.len_max = p.len_max;
    a.ema_alpha = p.ema_alpha;
    return mid ? launch_overlap_shape<G1Mid>(head_blocks, a, stream)
               : launch_overlap_shape<G1Small>(head_blocks, a, stream);
}

// ---------------------------------------------------------------------------
// (f3) the regression head: GEMM (layer 1) -> act -> GEMM (layer 2) -> head
// (layers 3 and 4, EMA, integerisation)
// ---------------------------------------------------------------------------
// The head kernel's view of the last two layers: a "binned head" whose
// input width is m2, whose nb = m3 outputs get ReLU and are dotted with w4.
static star_predict_params head_view(const star_mlp4_params& p) {
    star_predict_params h;
    h.n_req = p.n_req;
    h.d_model = p.m1;
    h.d_hidden = p.m2;
    h.n_bins = p.m3;
    h.dtype = p.dtype;
    h.act = STAR_ACT_RELU;
    h.ema_alpha = p.ema_alpha;
    h.ema_init = p.ema_init;
    h.len_max = p.len_max;
    return h;
}

Mlp4Plan plan_mlp4(const star_mlp4_params& p) {
    Mlp4Plan pl;
    const int elem = p.dtype == STAR_BF16 ? 2 : 4;
    pl.g1 = plan_gemm(p.n_req, p.m1, p.d_model, elem);
    pl.head = plan_predict(head_view(p), false, false);   // layer 2 and the head
    size_t off = 0;
    pl.p1_off = off;
    off += align_up((size_t)pl.g1.splits * p.n_req * p.m1 * sizeof(float), 256);
    pl.a1_off = off;
    off += align_up((size_t)p.n_req * p.m1 * elem, 256);
    pl.p2_off = off;
    off += align_up(pl.head.partial_bytes, 256);
    pl.total = off;
    return pl;
}

template <bool kBF16>
static hipError_t launch_act(int splits, dim3 grid, const float* P, int64_t items, int m4,
                             const float* bias, void* out, hipStream_t stream) {
    switch (splits) {
        case 1: hipLaunchKernelGGL((act_kernel<1, kBF16>), grid, dim3(ACT_THREADS), 0, stream, P, items, m4, bias, out); break;
        case 2: hipLaunchKernelGGL((act_kernel<2, kBF16>), grid, dim3(ACT_THREADS), 0, stream, P, items, m4, bias, out); break;
        case 4: hipLaunchKernelGGL((act_kernel<4, kBF16>), grid, dim3(ACT_THREADS), 0, stream, P, items, m4, bias, out); break;
        case 8: hipLaunchKernelGGL((act_kernel<8, kBF16>), grid, dim3(ACT_THREADS), 0, stream, P, items, m4, bias, out); break;
        case 16: hipLaunchKernelGGL((act_kernel<16, kBF16>), grid, dim3(ACT_THREADS), 0, stream, P, items, m4, bias, out); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_mlp4(const star_mlp4_params& p, const Mlp4Plan& pl, const void* hidden,
                       const void* w1, const float* b1, const void* w2, const float* b2,
                       const void* w3, const float* b3, const float* w4, float* ema_state,
                       float* expected, int32_t* rem_len, char* ws, hipStream_t stream) {
    if (p.n_req == 0) return hipSuccess;
    const bool bf = p.dtype == STAR_BF16;
    float* P1 = (float*)(ws + pl.p1_off);
    void* A1 = ws + pl.a1_off;
    float* P2 = (float*)(ws + pl.p2_off);
    hipError_t e;
    if ((e = launch_gemm(pl.g1, bf, hidden, w1, P1, p.n_req, p.m1, p.d_model, stream)) !=
        hipSuccess)
        return e;
    const int64_t items = (int64_t)p.n_req * p.m1 / 4;
    int64_t ab = ceil_div(items, (int64_t)ACT_THREADS * ACT_BATCH);
    const dim3 ga((unsigned)(ab > 2048 ? 2048 : ab));
    e = bf ? launch_act<true>(pl.g1.splits, ga, P1, items, p.m1 / 4, b1, A1, stream)
           : launch_act<false>(pl.g1.splits, ga, P1, items, p.m1 / 4, b1, A1, stream);
    if (e != hipSuccess) return e;
    const star_predict_params h = head_view(p);
    if ((e = launch_gemm(pl.head.gemm, bf, A1, w2, P2, p.n_req, p.m2, p.m1, stream)) !=
        hipSuccess)
        return e;
    return bf ? launch_head<true, true>(h, pl.head, P2, b2, w3, b3, w4, ema_state, expected,
                                        rem_len, stream, p.b4)
              : launch_head<false, true>(h, pl.head, P2, b2, w3, b3, w4, ema_state, expected,
                                         rem_len, stream, p.b4);
}

}  // namespace star

