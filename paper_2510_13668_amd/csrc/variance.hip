// (f1) Time-weighted variance change of every migration, on gfx950.
//
// Section 5.2 takes as the migration objective the variance of the
// instances' token loads now plus a beta-weighted sum of the variances of
// their predicted loads at later steps (Eq. 3-4).  Over bucketed curves that
// is Phi = sum_k beta_k Var_i(L_i[k]).  Moving request r (own curve R) from s
// to t keeps every bucket's mean, and changes bucket k's population variance
// by (2/n) R_k (R_k + L_t[k] - L_s[k]).  The library reports
//     G(r, t) = sum_k beta_k R_k (R_k + L_t[k] - L_s[k])   (= (n/2) dPhi),
// exactly, in 128-bit two's complement.  Sums, differences and products are
// taken modulo 2^128, which gives the exact value whenever |G| < 2^127; the
// host rejects sizes for which that could fail.
//
// With R_k = alpha + b^2 k below the request's end bucket k_e, p at k_e
// (the load model of Section 5.2), and the prefix sums
//     B0[k] = sum_{j<k} beta_j,   B1[k] = sum_{j<k} beta_j j,
//     B2[k] = sum_{j<k} beta_j j^2,
//     QA_i[k] = sum_{j<k} beta_j L_i[j],   QB_i[k] = sum_{j<k} beta_j j L_i[j],
// all read at k = k_e,
//     G = alpha^2 B0 + 2 alpha b^2 B1 + b^4 B2 + alpha (QA_t - QA_s)
//         + b^2 (QB_t - QB_s) + beta_{k_e} p (p + L_t[k_e] - L_s[k_e]),
// where the last term is present only when k_e < K.  The target enters
// through three gathers, so a candidate costs O(1) instead of the O(H)
// incremental update of the complexity analysis.
//
// Algorithm 1's best-feasible selection keeps the migration with the largest
// reduction, and only if it reduces the objective at all.  That is the
// smallest key (G, r n + t) with G < 0.
//
// Kernels:
//  * var_prep_kernel: one workgroup per instance (QA, QB) plus one for the
//    weight sums (B0, B1, B2); a scan by DPP, LDS only across the waves.  The
//    per-instance tables are stored bucket-major, [k][t] (and a bucket-major
//    copy of the curves), so that the lanes scoring one request's targets
//    read one contiguous run.
//  * var_score_kernel: up to 16 lanes per request; a lane walks every 16th
//    target (reads and writes stay contiguous across the request's lanes)
//    and keeps its best key in registers, and a short DPP scan combines the
//    lanes.  Negative best keys are reduced per workgroup.  In small grids the last workgroup to finish
//    (atomic ticket) reduces the workgroups' partials and writes the best
//    feasible move; larger grids leave that to var_final_kernel.
#include "star_common.hpp"
#include "star_internal.hpp"

namespace star {

typedef unsigned __int128 u128;
typedef __int128 s128;

constexpr int VP_THREADS = 256;
constexpr int VS_THREADS = 256;
constexpr int VS_WAVES = VS_THREADS / kWave;

// Grids up to this many workgroups find the best move in the scoring kernel
// (the last workgroup to finish reduces the partials); larger ones hand the
// partials to a one-workgroup kernel, because every workgroup's release
// fence would write back its XCD's L2, full of freshly written gains.
constexpr int VS_TICKET_BLOCKS = 64;
constexpr int VS_MAX_LG = 4;             // at most 16 lanes per request
constexpr int PLAN_MAX_INST = 1024;      // instances a plan classifies in LDS

__device__ inline u128 wide(int64_t v) { return (u128)(s128)v; }

// a * x modulo 2^128 for a 128-bit a and a non-negative 64-bit x: one full
// 64 x 64 product and one low half
__device__ inline u128 mul_u64(u128 a, uint64_t x) {
    return (u128)(uint64_t)a * x + ((u128)((uint64_t)(a >> 64) * x) << 64);
}
// a * x modulo 2^128 for a signed 64-bit x (x sign-extended to 128 bits)
__device__ inline u128 mul_s64(u128 a, int64_t x) {
    u128 r = mul_u64(a, (uint64_t)x);
    if (x < 0) r -= a << 64;
    return r;
}

// a * x modulo 2^128 for a 32-bit x: four chained 32 x 32 + 64 multiply-adds,
// about half of mul_u64's
__device__ inline u128 mul_u32(u128 a, uint32_t x) {
    const uint64_t p0 = (uint64_t)(uint32_t)a * x;
    const uint64_t p1 = (uint64_t)(uint32_t)(a >> 32) * x + (p0 >> 32);
    const uint64_t p2 = (uint64_t)(uint32_t)(a >> 64) * x + (p1 >> 32);
    const uint32_t p3 = (uint32_t)(a >> 96) * x + (uint32_t)(p2 >> 32);
    return ((u128)(((uint64_t)p3 << 32) | (uint32_t)p2) << 64) |
           (((uint64_t)(uint32_t)p1 << 32) | (uint32_t)p0);
}

// one bucket-major table entry: QA_t[k], b^2 QB_t[k].  The factor b^2 is the
// same for every request, so it is taken into the tables once (also into the
// weight sums: B0, b^2 B1, b^4 B2) instead of into every candidate: with the
// short products of inst_value, var_score_kernel<4> went from 20.1 to 17.4 us
// at 2 M candidates.
struct QEntry {
    u128 qa, qb;
};

// al QA + b^2 QB + bp L: the part of a gain that depends on one instance
// (taken at the target, less the source's).  small: al and bp's factor fit
// the short products in every lane of the wave (al < 2^32, bp < 2^64).
__device__ inline u128 inst_value(const QEntry& q, int64_t l, uint64_t al, u128 bp, bool small) {
    if (small) {
        u128 v = mul_u32(q.qa, (uint32_t)al) + q.qb;
        // bp < 2^64 and a signed l: one 64 x 64 product, the sign taken off
        v += (u128)(uint64_t)bp * (u128)(uint64_t)l;
        if (l < 0) v -= bp << 64;
        return v;
    }
    return mul_u64(q.qa, al) + q.qb + mul_s64(bp, l);
}
// whether the short products hold for every lane of the wave
__device__ inline bool wave_small(uint64_t al, u128 bp) {
    return __ballot((al >> 32) != 0 || (uint64_t)(bp >> 64) != 0) == 0;
}

// ---------------------------------------------------------------------------
// prefix tables
// ---------------------------------------------------------------------------
// Row i < n: QA_i[k], b^2 QB_i[k] for k = 0..K.  Row n: B0[k], b^2 B1[k],
// b^4 B2[k].
// Thread j of the workgroup owns the buckets [j*per, (j+1)*per); its sums
// are scanned across its wave by DPP and across the waves through LDS (a
// scan of all 256 sums in LDS, two barriers a step, took 10.4 us per call at
// 64 instances x 1024 buckets against 7.8 now), the exclusive prefix is
// the inclusive one minus the thread's own sum, which modular arithmetic
// allows, and each thread writes its run.  Up to
// VP_REG buckets per thread stay in registers between the two passes, so
// that no load waits behind the table stores (loads and stores share one
// counter on gfx9).
constexpr int VP_REG = 8;
constexpr int VP_WAVES = VP_THREADS / kWave;

template <int kCtrl, int kRowMask>
__device__ inline u128 dpp_add_u128(u128 v) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)dpp_i32<kCtrl, kRowMask>((int)(uint32_t)(v >> (32 * i)), 0);
    return v + (((u128)(((uint64_t)w[3] << 32) | w[2]) << 64) | (((uint64_t)w[1] << 32) | w[0]));
}
// Inclusive prefix sum over the 64 lanes (lane order), modulo 2^128.
__device__ inline u128 wave_incl_add_u128(u128 v) {
    v = dpp_add_u128<kDppRowShr1, 0xF>(v);
    v = dpp_add_u128<kDppRowShr2, 0xF>(v);
    v = dpp_add_u128<kDppRowShr4, 0xF>(v);
    v = dpp_add_u128<kDppRowShr8, 0xF>(v);
    v = dpp_add_u128<kDppRowBcast15, 0xA>(v);
    v = dpp_add_u128<kDppRowBcast31, 0xC>(v);
    return v;
}

__device__ inline void prep_load(const uint16_t* beta, const int64_t* L, bool wrow, int c0,
                                 int last, uint32_t* wv, int64_t* lv) {
#pragma unroll
    for (int i = 0; i < VP_REG; ++i) {
        const int j = c0 + i < last ? c0 + i : last;   // clamped: no branch per slot
        wv[i] = beta[j];
        lv[i] = wrow ? 0 : L[j];
    }
}

// The tables of one row, computed by the whole workgroup (sx: the waves'
// sums in LDS, used by nothing else); bb = b^2, and k b^2 < 2^60 (b K <=
// 2^30).  qt1 and lt1: a second copy of the instance tables, or null.  L is the
// instance's curve (row < n) or unused (the weights' row, wrow).
__device__ void prep_row(const int64_t* __restrict__ L, const uint16_t* __restrict__ beta, int n,
                         int K, int row, bool wrow, QEntry* __restrict__ qt,
                         int64_t* __restrict__ lt, u128* __restrict__ bs, uint64_t bb,
                         u128 (*sx)[VP_WAVES], QEntry* __restrict__ qt1 = nullptr,
                         int64_t* __restrict__ lt1 = nullptr) {
    const int tid = threadIdx.x;
    const int K1 = K + 1;
    const int per = (K + VP_THREADS - 1) / VP_THREADS;
    const int j0 = min(tid * per, K), j1 = min(j0 + per, K);

    uint32_t wv[VP_REG];
    int64_t lv[VP_REG];
    u128 x0 = 0, x1 = 0, x2 = 0;
    for (int c0 = j0; c0 < j1; c0 += VP_REG) {
        prep_load(beta, L, wrow, c0, j1 - 1, wv, lv);
#pragma unroll
        for (int i = 0; i < VP_REG; ++i) {
            const bool in = c0 + i < j1;
            const u128 w = in ? (u128)wv[i] : (u128)0;
            const uint64_t uj = bb * (uint64_t)(c0 + i);
            if (wrow) {
                x0 += w;
                x1 += mul_u64(w, uj);
                x2 += mul_u64(mul_u64(w, uj), uj);
            } else {
                const u128 wl = mul_s64(w, lv[i]);
                x0 += wl;
                x1 += mul_u64(wl, uj);
            }
        }
    }
    const int lane = tid & (kWave - 1), wid = tid / kWave;
    u128 t0 = wave_incl_add_u128(x0), t1 = wave_incl_add_u128(x1), t2 = 0;
    if (wrow) t2 = wave_incl_add_u128(x2);
    if (lane == kWave - 1) {
        sx[0][wid] = t0;
        sx[1][wid] = t1;
        sx[2][wid] = t2;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < VP_WAVES - 1; ++w) {
        if (w >= wid) break;
        t0 += sx[0][w];
        t1 += sx[1][w];
        t2 += sx[2][w];
    }
    // t0..t2: the sums through this thread's run; p0..p2: before it
    u128 p0 = t0 - x0, p1 = t1 - x1, p2 = t2 - x2;
    for (int c0 = j0; c0 < j1; c0 += VP_REG) {
        if (per > VP_REG) prep_load(beta, L, wrow, c0, j1 - 1, wv, lv);
#pragma unroll
        for (int i = 0; i < VP_REG; ++i) {
            const int j = c0 + i;
            if (j >= j1) break;
            const u128 w = wv[i];
            const uint64_t uj = bb * (uint64_t)j;
            if (wrow) {
                bs[j] = p0;
                bs[K1 + j] = p1;
                bs[2 * (size_t)K1 + j] = p2;
                p0 += w;
                p1 += mul_u64(w, uj);
                p2 += mul_u64(mul_u64(w, uj), uj);
            } else {
                qt[(size_t)j * n + row] = QEntry{p0, p1};
                lt[(size_t)j * n + row] = lv[i];
                if (qt1) {
                    qt1[(size_t)j * n + row] = QEntry{p0, p1};
                    lt1[(size_t)j * n + row] = lv[i];
                }
                const u128 wl = mul_s64(w, lv[i]);
                p0 += wl;
                p1 += mul_u64(wl, uj);
            }
        }
    }
    if (tid == VP_THREADS - 1) {
        if (wrow) {
            bs[K] = t0;
            bs[K1 + K] = t1;
            bs[2 * (size_t)K1 + K] = t2;
        } else {
            qt[(size_t)K * n + row] = QEntry{t0, t1};
            if (qt1) qt1[(size_t)K * n + row] = QEntry{t0, t1};
        }
    }
}

__global__ __launch_bounds__(VP_THREADS) void var_prep_kernel(const int64_t* __restrict__ load,
                                                              const uint16_t* __restrict__ beta,
                                                              int n, int K, uint64_t bb,
                                                              QEntry* __restrict__ qt,
                                                              int64_t* __restrict__ lt,
                                                              u128* __restrict__ bs,
                                                              uint32_t* __restrict__ ticket) {
    __shared__ u128 sx[3][VP_WAVES];
    const int row = blockIdx.x;
    if (row == 0 && threadIdx.x == 0) *ticket = 0u;   // the scoring kernel runs after this one
    prep_row(load + (size_t)(row == n ? 0 : row) * K, beta, n, K, row, row == n, qt, lt, bs, bb,
             sx);
}

// ---------------------------------------------------------------------------
// keys (gain, r n + t), ascending
// ---------------------------------------------------------------------------
struct VKey {
    s128 g;
    uint32_t idx;
};
constexpr uint32_t kNoIdx = 0xFFFFFFFFu;
__device__ inline VKey no_key() { return VKey{(s128)(~(u128)0 >> 1), kNoIdx}; }
__device__ inline bool vless(const VKey& a, const VKey& b) {
    return a.g < b.g || (a.g == b.g && a.idx < b.idx);
}
__device__ inline VKey vmin(const VKey& a, const VKey& b) { return vless(b, a) ? b : a; }

// DPP move of a whole key; a lane whose source lies outside its row, or in
// a row that kRowMask leaves out, receives the no-key sentinel
template <int kCtrl, int kRowMask>
__device__ inline VKey dpp_key(const VKey& k) {
    const u128 u = (u128)k.g;
    const u128 inf = ~(u128)0 >> 1;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(inf >> (32 * i)),
                                                    (int)(uint32_t)(u >> (32 * i)), kCtrl,
                                                    kRowMask, 0xF, false);
    VKey o;
    o.g = (s128)(((u128)w[3] << 96) | ((u128)w[2] << 64) | ((u128)w[1] << 32) | (u128)w[0]);
    o.idx = (uint32_t)__builtin_amdgcn_update_dpp((int)kNoIdx, (int)k.idx, kCtrl, kRowMask, 0xF,
                                                  false);
    return o;
}

// Minimum over each aligned group of 2^lg lanes (lg <= 6), valid in the
// group's last lane: an inclusive min-scan by DPP row shifts, where a lane
// ignores a source in the previous group (tl = lane index in its group),
// then the row broadcasts for groups of 32 and 64 lanes.  Every lane of the
// wave must be active.
__device__ inline VKey group_min(VKey k, int lg, int tl) {
    VKey o;
    if (lg >= 1) {
        o = dpp_key<kDppRowShr1, 0xF>(k);
        if (tl >= 1 && vless(o, k)) k = o;
    }
    if (lg >= 2) {
        o = dpp_key<kDppRowShr2, 0xF>(k);
        if (tl >= 2 && vless(o, k)) k = o;
    }
    if (lg >= 3) {
        o = dpp_key<kDppRowShr4, 0xF>(k);
        if (tl >= 4 && vless(o, k)) k = o;
    }
    if (lg >= 4) {
        o = dpp_key<kDppRowShr8, 0xF>(k);
        if (tl >= 8 && vless(o, k)) k = o;
    }
    if (lg >= 5) {
        o = dpp_key<kDppRowBcast15, 0xA>(k);
        if (vless(o, k)) k = o;
    }
    if (lg >= 6) {
        o = dpp_key<kDppRowBcast31, 0xC>(k);
        if (vless(o, k)) k = o;
    }
    return k;
}

__device__ inline u128 readlane_u128(u128 v, int lane) {
    const uint64_t lo = (uint64_t)readlane_i64((int64_t)(uint64_t)v, lane);
    const uint64_t hi = (uint64_t)readlane_i64((int64_t)(uint64_t)(v >> 64), lane);
    return ((u128)hi << 64) | (u128)lo;
}
// The smallest of the wave's keys, all of them negative gains or no-key, in
// every lane (scalar registers).  The high words decide nearly always: only
// they are reduced (a third of the steps of group_min), and whole keys are
// compared where the smallest high word is not unique.
__device__ inline VKey wave_min_key(const VKey& k) {
    const int64_t hi = (int64_t)(k.g >> 64);
    const int64_t top = ~readlane_i64(wave_incl_max_i64(~hi), kWave - 1);   // min hi
    if (top >= 0) return no_key();
    const uint64_t who = __ballot(hi == top);
    VKey m = k;
    int lane = __ffsll((unsigned long long)who) - 1;
    if (who & (who - 1)) {
        m = group_min(k, 6, (int)threadIdx.x & (kWave - 1));
        lane = kWave - 1;
    }
    VKey o;
    o.g = (s128)readlane_u128((u128)m.g, lane);
    o.idx = (uint32_t)__builtin_amdgcn_readlane((int)m.idx, lane);
    return o;
}
// The smallest of `count` <= 64 keys in LDS, in every lane of each wave.
__device__ inline VKey lds_min_key(const VKey* keys, int count) {
    const int lane = threadIdx.x & (kWave - 1);
    VKey k = keys[lane < count ? lane : 0];
    if (lane >= count) k = no_key();
    return wave_min_key(k);
}

// A workgroup's partial, written and read with device-scope atomics so the
// last workgroup sees every other XCD's value.
struct VPart {
    uint64_t w[3];   // gain low, gain high, index
    uint64_t pad;
};
__device__ inline void store_part(VPart* p, const VKey& k) {
    const u128 u = (u128)k.g;
    __hip_atomic_store(&p->w[0], (uint64_t)u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p->w[1], (uint64_t)(u >> 64), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p->w[2], (uint64_t)k.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline VKey load_part(VPart* p) {
    const uint64_t lo = __hip_atomic_load(&p->w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t hi = __hip_atomic_load(&p->w[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t ix = __hip_atomic_load(&p->w[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return VKey{(s128)(((u128)hi << 64) | (u128)lo), (uint32_t)ix};
}

// One workgroup: the smallest of `parts` partial keys, returned to every
// thread.
template <bool kAtomic>
__device__ VKey reduce_keys(VPart* part, int parts, VKey* wbest) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    constexpr int kBatch = 8;   // partials in flight per thread
    VKey k = no_key();
    for (int g0 = tid; g0 < parts; g0 += VS_THREADS * kBatch) {
        VKey p[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int g = g0 + i * VS_THREADS;
            VPart* src = &part[g < parts ? g : parts - 1];
            if (kAtomic) {
                p[i] = load_part(src);
            } else {
                const VPart v = *src;
                p[i] = VKey{(s128)(((u128)v.w[1] << 64) | (u128)v.w[0]), (uint32_t)v.w[2]};
            }
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) k = vmin(k, p[i]);   // repeats are harmless
    }
    k = group_min(k, 6, lane);
    if (lane == kWave - 1) wbest[wid] = k;
    __syncthreads();
    VKey m = wbest[0];
    for (int w = 1; w < VS_THREADS / kWave; ++w) m = vmin(m, wbest[w]);
    __syncthreads();
    return m;
}

// The move record of key m (or the no-move record).
__device__ inline star_move move_of(const VKey& m, const int32_t* inst, int n) {
    star_move mv;
    if (m.idx != kNoIdx) {
        const int r = (int)(m.idx / (uint32_t)n);
        mv.req = r;
        mv.src = inst[r];
        mv.tgt = (int)(m.idx - (uint32_t)r * (uint32_t)n);
        mv.gain.lo = (uint64_t)(u128)m.g;
        mv.gain.hi = (int64_t)(m.g >> 64);
    } else {
        mv.req = mv.src = mv.tgt = -1;
        mv.gain.lo = 0;
        mv.gain.hi = 0;
    }
    mv.reserved = 0;
    return mv;
}

// The same, written as the move (or the no-move record when none is negative).
template <bool kAtomic>
__device__ void reduce_parts(VPart* part, int parts, const int32_t* inst, int n, star_move* move,
                             VKey* wbest) {
    const VKey m = reduce_keys<kAtomic>(part, parts, wbest);
    if (threadIdx.x == 0) *move = move_of(m, inst, n);
}

// A request's target-independent part of G, staged in LDS.
struct ReqStash {
    u128 base, bp;
    uint64_t al;
    int32_t ke;
    int32_t s;        // source instance; -2: invalid request; -1: past the end
};

struct VarArgs {
    const int32_t* cur;
    const int32_t* rem;
    const int32_t* inst;
    const uint16_t* beta;
    const QEntry* qt;        // [K + 1][n]
    const int64_t* lt;       // [K][n]
    const u128* bs;          // [3][K + 1]
    u128* gain;              // [N, n] or null
    int32_t* best_target;    // [N] or null
    u128* best_gain;         // [N] or null
    star_move* move;         // one, or null
    VPart* part;             // [gridDim.x] when move != null
    uint32_t* ticket;
    int32_t* err;
    int N, n, b, K;
    int ticketed;            // 1: the last workgroup reduces the partials
    int64_t H;
};

constexpr int VS_M = 4;      // targets per lane per chunk

// (g, t) keys of one request: smaller gain, then smaller target
__device__ inline bool gt_less(s128 ga, int ta, s128 gb, int tb) {
    return ga < gb || (ga == gb && (uint32_t)ta < (uint32_t)tb);
}

// One DPP step of the per-request reduction: the key of lane - S (row
// shift) replaces this lane's if smaller; lanes whose source lies in the
// previous request's group (or row) keep theirs.
template <int kCtrl, int S>
__device__ inline void dpp_step(s128& g, int& t, int tl) {
    const u128 u = (u128)g;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int x = (int)(uint32_t)(u >> (32 * i));
        w[i] = (uint32_t)__builtin_amdgcn_update_dpp(x, x, kCtrl, 0xF, 0xF, false);
    }
    const int to = __builtin_amdgcn_update_dpp(t, t, kCtrl, 0xF, 0xF, false);
    const s128 go =
        (s128)(((u128)w[3] << 96) | ((u128)w[2] << 64) | ((u128)w[1] << 32) | (u128)w[0]);
    if (tl >= S && gt_less(go, to, g, t)) {
        g = go;
        t = to;
    }
}

// A workgroup takes VS_WAVES * 64 / P requests (P = 2^LG <= 16 lanes per
// request).  Phase A: thread j stages request j's target-independent terms
// in LDS (coalesced reads, one gather of the weight sums and of its
// source's entry).  Phase B: each wave takes 64 / P requests at once; lane
// l of a request's group walks the targets l, l + P, ... in chunks of
// VS_M, loading a chunk's table entries (contiguous across the group)
// before storing its gains and keeping its best key in registers; then an
// LG-step DPP row-shift scan leaves the request's best key in the group's
// last lane.  One pass per wave: on gfx9 loads and stores share one
// counter, so a second pass's loads would wait for the first pass's stores.
template <int LG>
__global__ __launch_bounds__(VS_THREADS) void var_score_kernel(VarArgs a) {
    constexpr int P = 1 << LG, RPW = kWave / P, TILE = VS_WAVES * RPW;
    __shared__ ReqStash st[TILE];
    __shared__ VKey wbest[VS_WAVES];
    __shared__ bool last;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int sub = lane >> LG, tl = lane & (P - 1);
    const int n = a.n, K = a.K, K1 = K + 1;
    const QEntry* __restrict__ qt = a.qt;
    const int64_t* __restrict__ lt = a.lt;
    u128* __restrict__ gain = a.gain;

    VKey feas = no_key();   // best key of this lane's request that lowers the objective
    const int r0 = blockIdx.x * TILE;
    if (tid < TILE) {
        const int r = r0 + tid;
        ReqStash e;
        e.base = 0;
        e.bp = 0;
        e.al = 0;
        e.ke = 0;
        e.s = -1;
        if (r < a.N) {
            const ReqTerms q = request_terms(a.inst[r], a.cur[r], a.rem[r], n, a.b, a.H);
            report_error(a.err, q.bad);
            e.s = q.bad ? -2 : q.s;
            if (!q.bad) {
                // alpha, b^2 and p are non-negative and below 2^62
                const uint64_t al = (uint64_t)q.alpha;
                const int ke = q.ke;
                const u128 b0 = a.bs[ke], b1 = a.bs[K1 + ke], b2 = a.bs[2 * (size_t)K1 + ke];
                const QEntry qs = qt[(size_t)ke * n + q.s];
                u128 base = mul_u64(mul_u64(b0, al), al) + mul_u64(b1, 2 * al) + b2 -
                            mul_u64(qs.qa, al) - qs.qb;
                u128 bp = 0;
                if (ke < K) {
                    bp = (u128)a.beta[ke] * (u128)(uint64_t)q.p;
                    base += mul_s64(bp, q.p - lt[(size_t)ke * n + q.s]);
                }
                e.base = base;
                e.bp = bp;
                e.al = al;
                e.ke = ke;
            }
        }
        st[tid] = e;
    }
    __syncthreads();

    const int j = wid * RPW + sub;
    const int r = r0 + j;
    const u128 base = st[j].base, bp = st[j].bp;
    const uint64_t al = st[j].al;
    const int ke = st[j].ke, src = st[j].s;
    const bool live = src != -1, valid = src >= 0;
    const bool small = wave_small(al, bp);
    const size_t row = valid ? (size_t)ke * n : 0;   // others read entry 0, unused
    s128 bg = ~(u128)0 >> 1;
    int bt = -1;
    for (int c0 = 0; c0 < n; c0 += P * VS_M) {
        QEntry qe[VS_M];
        int64_t le[VS_M];
#pragma unroll
        for (int i = 0; i < VS_M; ++i) {
            const int t = c0 + tl + P * i;
            const size_t o = row + (t < n ? t : 0);
            qe[i] = qt[o];
            le[i] = lt[o];     // past the curves where ke == K: there bp is 0
        }
#pragma unroll
        for (int i = 0; i < VS_M; ++i) {
            const int t = c0 + tl + P * i;
            u128 g = 0;
            if (valid) g = base + inst_value(qe[i], le[i], al, bp, small);
            const bool mig = valid && t < n && t != src;
            if (!mig) g = 0;
            if (mig && (s128)g < bg) {   // targets ascend within a lane
                bg = (s128)g;
                bt = t;
            }
            if (gain && live && t < n) gain[(size_t)r * n + t] = g;
        }
    }
    if (LG >= 1) dpp_step<kDppRowShr1, 1>(bg, bt, tl);
    if (LG >= 2) dpp_step<kDppRowShr2, 2>(bg, bt, tl);
    if (LG >= 3) dpp_step<kDppRowShr4, 4>(bg, bt, tl);
    if (LG >= 4) dpp_step<kDppRowShr8, 8>(bg, bt, tl);

    if (live && tl == P - 1) {
        if (a.best_target) a.best_target[r] = bt;
        if (a.best_gain) a.best_gain[r] = bt >= 0 ? (u128)bg : (u128)0;
        if (bt >= 0 && bg < 0) feas = VKey{bg, (uint32_t)r * (uint32_t)n + (uint32_t)bt};
    }
    if (!a.move) return;

    // best negative key of the workgroup, then (small grids) of the grid
    feas = group_min(feas, 6, lane);
    if (lane == kWave - 1) wbest[wid] = feas;
    __syncthreads();
    if (tid == 0) {
        VKey k = wbest[0];
        for (int w = 1; w < VS_WAVES; ++w) k = vmin(k, wbest[w]);
        store_part(&a.part[blockIdx.x], k);
        if (a.ticketed) {
            // small grids only: this release fence writes back the XCD's L2
            __threadfence();
            last = atomicAdd(a.ticket, 1u) == gridDim.x - 1;
        }
    }
    if (!a.ticketed) return;
    __syncthreads();
    if (!last) return;
    __threadfence();
    reduce_parts<true>(a.part, gridDim.x, a.inst, n, a.move, wbest);
    if (tid == 0) *a.ticket = 0u;
}

// The best feasible move from the scoring workgroups' partials (large grids,
// after the scoring kernel has finished).
__global__ __launch_bounds__(VS_THREADS) void var_final_kernel(VPart* part, int parts,
                                                               const int32_t* inst, int n,
                                                               star_move* move) {
    __shared__ VKey wbest[VS_WAVES];
    reduce_parts<false>(part, parts, inst, n, move, wbest);
}

// ---------------------------------------------------------------------------
// (f2) Algorithm 1 end to end: one migration per pass, repeated
//
// One launch per pass, plus one after the last.  Launch q settles the move
// that pass q - 1 found (every workgroup reduces that pass's partial keys
// itself, so no workgroup waits for another), then scores pass q.  The
// tables come in two copies, so that no workgroup writes what another reads:
// launch q reads copy (q - 1) & 1, which holds the state before move q - 1,
// and adds that move's effect to the few entries it touches as it reads
// them; its update workgroups bring copy q & 1, two moves behind, up to date
// for launch q + 1.  Moving R from s to t changes the tables by closed
// forms: with F_A(k) = sum_{j<k} beta_j R_j, F_B(k) = b^2 sum_{j<k} beta_j j R_j,
//     F_A(k) = alpha B0[k] + b^2 B1[k],  F_B(k) = alpha b^2 B1[k] + b^4 B2[k]
// for k <= k_e, and for k > k_e the value at k_e plus beta_{k_e} p (times
// b^2 k_e for F_B); QA and b^2 QB of row s fall by F, those of row t rise.
//
// What bounds a pass is a chain of dependent reads (partials, request record,
// table entries), not bytes or arithmetic.  So it is one launch, not a
// scoring and an update launch in turn.  A request's terms are computed once,
// by launch 0, and kept in a record, which also follows what the moves do to
// its source's share.  A thread reads its request's record while the partials
// are on their way; a partial carries all that its move does to the tables.
// The requests that may move (those on an instance of O) are then packed in
// LDS, so that the lanes of the waves all score.  Requests are dealt to the
// workgroups in blocks of 16, because those on one crowded instance are often
// neighbours.  Measured at 32768 requests on 64 instances, K = 1024: 12.5 us
// per move, against 18.0 + 10.6 us for the two launches (of 13.2 us, before the
// last request's spare reads went: 2.9 until the move is known, 0.9
// classification, 1.1 packing, 3.3, 5.2 in the slowest workgroup, the targets,
// 1.7 the workgroup's best key).
// ---------------------------------------------------------------------------
constexpr int PL_THREADS = 512;           // 160 registers a thread: 1024 would spill
constexpr int PL_WAVES = PL_THREADS / kWave;
// A compute unit holds one of these workgroups (over 128 registers a thread),
// so scoring and update workgroups together are at most the 256 units: nine
// more of them had to wait for a free unit, and a launch took 16 us, not 13.
constexpr int PL_MAX_BLOCKS = 240;       // scoring workgroups
constexpr int PL_UPDATERS = 16;          // update workgroups
constexpr int PL_OWN = 256;              // requests per workgroup and iteration
constexpr int PL_U = 2;                  // requests per lane group
constexpr int PL_RUN = 16;               // neighbouring requests dealt together
constexpr int PLAN_REQ_CHUNK = 4096;     // requests per current-load workgroup, at least
constexpr int PLAN_MAX_CHUNKS = 64;
static_assert(PL_MAX_BLOCKS <= PL_THREADS && PL_OWN <= PL_THREADS, "one per thread");

// What a pass needs of a request.  base and place follow the moves; only the
// thread that takes the request in every launch writes them.  Stored as
// PL_WORDS arrays of 16-byte words (word w of request r at w N + r), so that
// neighbouring threads read and write neighbouring words: as one 128-byte
// record per request, launch 0 took 26 us, not 15.
struct PlanReq {
    u128 base;        // gain less the target's share, in the state before the last move
    u128 bp;          // beta_{k_e} p (0 where k_e = K)
    u128 b0, b1, b2;  // B0, b^2 B1, b^4 B2 at k_e
    uint64_t al;      // alpha
    int64_t need;     // memory the request takes on a target
    int64_t p;        // the request's load in its last bucket
    int32_t ke, c;    // k_e, cur_len
    int32_t place;    // its instance; -1: Algorithm 1 never moves it
    int32_t pad[3];
};
constexpr int PL_WORDS = 8;
static_assert(sizeof(PlanReq) == 16 * PL_WORDS, "whole words");
__device__ inline PlanReq req_load(const u32x4* req, size_t N, size_t r) {
    struct Words { u32x4 w[PL_WORDS]; } x;
#pragma unroll
    for (int i = 0; i < PL_WORDS; ++i) x.w[i] = req[i * N + r];
    return __builtin_bit_cast(PlanReq, x);
}
// words [w0, w1) of a record
template <int w0, int w1>
__device__ inline void req_store(u32x4* req, size_t N, size_t r, const PlanReq& e) {
    struct Words { u32x4 w[PL_WORDS]; };
    const Words x = __builtin_bit_cast(Words, e);
#pragma unroll
    for (int i = w0; i < w1; ++i) req[i * N + r] = x.w[i];
}

// A request that may move, packed in LDS.
struct PlanCand {
    u128 base, dv;    // gain less the target's share; the last move's effect on that share
    u128 bp, b0, b1, b2;
    uint64_t al;
    int64_t need, p;
    int32_t ke, c, r, src;
};

// A workgroup's best migration and what it does to the tables; idx kNoIdx:
// none lowers the objective.
struct PlanPart {
    u128 g;
    uint32_t idx;     // r n + t
    int32_t src, ke, c;
    uint64_t al;
    int64_t p;
    u128 bp, fa, fb, pad[2];
};
static_assert(sizeof(PlanPart) == 128, "one partial per cache line");

struct PlanArgs {
    const int32_t* cur;
    const int32_t* rem;
    int32_t* inst;           // updated in place
    int64_t* load;           // [n, K], updated in place
    const uint16_t* beta;
    QEntry* qt[2];           // [K + 1][n], two copies (see above)
    int64_t* lt[2];          // [K + 1][n] (row K unused), two copies
    int64_t* now[2];         // [n] current loads N_i, two copies
    PlanPart* part[2];       // [parts], of the even and the odd passes
    u128* bs;                // [3][K + 1]
    u128* wsum;              // sum of w_i: moves leave it as it is
    int64_t* now_part;       // [chunks][n] current loads of each request chunk
    u32x4* req;              // [PL_WORDS][N], see PlanReq
    int32_t* done;
    int32_t* n_moves;        // caller's move count
    star_move* moves;        // caller's [max_moves]
    int32_t* err;
    int N, n, b, K;
    int chunks, chunk_len;
    int blocks;              // scoring workgroups (0: the last launch)
    int parts;               // partials of a pass
    int pass;                // q
    int theta_num, theta_den, u_rule, mem_rule, min_rem;
    int64_t mem_cap;
    int64_t H;
};

// Workgroups 0..n: the tables of every row (as var_prep_kernel), both copies.
// The others: each sums cur_len per instance over a chunk of valid requests
// in LDS, and reports invalid requests.
__global__ __launch_bounds__(VP_THREADS) void plan_prep_kernel(PlanArgs a) {
    __shared__ u128 sx[3][VP_WAVES];
    __shared__ unsigned long long hist[PLAN_MAX_INST];
    const int row = blockIdx.x, tid = threadIdx.x, n = a.n;
    if (row == 0 && tid == 0) {
        *a.done = 0;
        *a.n_moves = 0;
    }
    if (row <= n) {
        prep_row(a.load + (size_t)(row == n ? 0 : row) * a.K, a.beta, n, a.K, row, row == n,
                 a.qt[0], a.lt[0], a.bs, (uint64_t)a.b * (uint64_t)a.b, sx, a.qt[1], a.lt[1]);
        return;
    }
    for (int i = tid; i < n; i += VP_THREADS) hist[i] = 0;
    __syncthreads();
    const int chunk = row - n - 1;
    const int64_t r0 = (int64_t)chunk * a.chunk_len;
    const int64_t r1 = r0 + a.chunk_len < a.N ? r0 + a.chunk_len : a.N;
    int32_t bad = 0;
    for (int64_t r = r0 + tid; r < r1; r += VP_THREADS) {
        const int s = a.inst[r], c = a.cur[r], l = a.rem[r];
        int32_t f = 0;
        if (s < 0 || s >= n) f |= STAR_DEV_BAD_INST;
        if (c < 1) f |= STAR_DEV_BAD_CUR;
        if (l < 1) f |= STAR_DEV_BAD_REM;
        if (!f) atomicAdd(&hist[s], (unsigned long long)c);
        bad |= f;
    }
    report_error(a.err, bad);
    __syncthreads();
    for (int i = tid; i < n; i += VP_THREADS)
        a.now_part[(size_t)chunk * n + i] = (int64_t)hist[i];
}

// A settled move: the request's terms, F_A and F_B at its k_e.
struct PlanMove {
    u128 g, bp, fa, fb;
    uint64_t al;
    int64_t p;
    int ke, src, tgt, r, c;
};
// F_A(k) and F_B(k) from the weight sums at min(k, k_e)
__device__ inline void move_f(const PlanArgs& a, uint64_t al, u128 bp, int ke, uint64_t bb, int k,
                              u128& fa, u128& fb) {
    const size_t kk = k <= ke ? k : ke, K1 = (size_t)a.K + 1;
    const u128 b0 = a.bs[kk], b1 = a.bs[K1 + kk], b2 = a.bs[2 * K1 + kk];
    fa = mul_u64(b0, al) + b1;
    fb = mul_u64(b1, al) + b2;
    if (k > ke) {
        fa += bp;
        fb += mul_u64(bp, bb * (uint64_t)ke);
    }
}
// the moved request's own curve at bucket k < K
__device__ inline int64_t move_r(uint64_t al, int64_t p, int ke, uint64_t bb, int k) {
    return k < ke ? (int64_t)al + (int64_t)bb * k : k == ke ? p : 0;
}
// +1 where the move adds its curve to instance i, -1 where it takes it away
__device__ inline int move_sign(int src, int tgt, int i) { return (i == tgt) - (i == src); }
__device__ inline u128 signed_part(u128 f, int sign) {
    return sign > 0 ? f : sign < 0 ? (u128)0 - f : (u128)0;
}

// The update workgroups of launch q (block u of `nb`): with the settled
// move `m`, copy q & 1 of the tables and of the current loads (two moves
// behind, one where q = 1), the curves, inst_of and the move record.
__device__ void plan_update(const PlanArgs& a, const PlanMove& m, int u, int nb) {
    const int tid = threadIdx.x, n = a.n, K = a.K, q = a.pass;
    const uint64_t bb = (uint64_t)a.b * (uint64_t)a.b;
    QEntry* qt = a.qt[q & 1];
    int64_t* lt = a.lt[q & 1];
    PlanReq o{};                             // the move before it
    int osrc = -1, otgt = -1;
    if (q >= 2) {
        const star_move mv = a.moves[q - 2];
        o = req_load(a.req, a.N, mv.req);
        osrc = mv.src;
        otgt = mv.tgt;
    }
    // one table entry of one of the (up to four) changed columns per thread
    for (int64_t e = (int64_t)u * PL_THREADS + tid; e < 4 * (int64_t)(K + 1);
         e += (int64_t)nb * PL_THREADS) {
        const int k = (int)(e >> 2), w = (int)(e & 3);
        const int col = w == 0 ? m.src : w == 1 ? m.tgt : w == 2 ? osrc : otgt;
        // a column named twice is changed once, by its first name
        if (col < 0 || (w >= 2 && (col == m.src || col == m.tgt))) continue;
        const int sm = move_sign(m.src, m.tgt, col), so = move_sign(osrc, otgt, col);
        QEntry* p = &qt[(size_t)k * n + col];
        const QEntry v = *p;
        u128 fa, fb;
        move_f(a, m.al, m.bp, m.ke, bb, k, fa, fb);
        u128 da = signed_part(fa, sm), db = signed_part(fb, sm);
        int64_t dl = k < K ? sm * move_r(m.al, m.p, m.ke, bb, k) : 0;
        if (so) {
            move_f(a, o.al, o.bp, o.ke, bb, k, fa, fb);
            da += signed_part(fa, so);
            db += signed_part(fb, so);
            if (k < K) dl += so * move_r(o.al, o.p, o.ke, bb, k);
        }
        *p = QEntry{v.qa + da, v.qb + db};
        if (k < K) {
            lt[(size_t)k * n + col] += dl;
            if (w < 2 && k <= m.ke)
                a.load[(size_t)col * K + k] += sm * move_r(m.al, m.p, m.ke, bb, k);
        }
    }
    if (u == 0) {
        if (tid < 4) {
            const int col = tid == 0 ? m.src : tid == 1 ? m.tgt : tid == 2 ? osrc : otgt;
            if (col >= 0 && !(tid >= 2 && (col == m.src || col == m.tgt)))
                a.now[q & 1][col] += (int64_t)move_sign(m.src, m.tgt, col) * m.c +
                                     (int64_t)move_sign(osrc, otgt, col) * o.c;
        }
        if (tid == 0) {
            star_move mv;
            mv.req = m.r;
            mv.src = m.src;
            mv.tgt = m.tgt;
            mv.reserved = 0;
            mv.gain.lo = (uint64_t)m.g;
            mv.gain.hi = (int64_t)(m.g >> 64);
            a.moves[q - 1] = mv;
            *a.n_moves = q;
            a.inst[m.r] = m.tgt;
        }
    }
}

// The request of thread `tid` in iteration `it` (-1: none).  Launch 0
// computes its record, the others read it (reads are clamped, not branched
// around, so that nothing waits for them here).
template <bool kFirst>
__device__ __forceinline__ int64_t plan_own(const PlanArgs& a, int64_t it, PlanReq& e) {
    const int tid = threadIdx.x, n = a.n;
    const int64_t run = (it * (PL_OWN / PL_RUN) + tid / PL_RUN) * a.blocks + blockIdx.x;
    const int64_t r = run * PL_RUN + tid % PL_RUN;
    const bool in = tid < PL_OWN && r < a.N;
    const int64_t rc = in ? r : a.N - 1;
    if (kFirst) {
        const int c = a.cur[rc], l = a.rem[rc];
        const ReqTerms t = request_terms(a.inst[rc], c, l, n, a.b, a.H);
        e.place = !t.bad && l > a.min_rem ? t.s : -1;
        e.al = (uint64_t)t.alpha;            // alpha, b^2 and p: non-negative, below 2^62
        e.ke = t.ke;
        e.p = t.p;
        e.c = c;
        e.need = l + (a.mem_rule ? (int64_t)c : 0);
        e.bp = t.ke < a.K ? (u128)a.beta[t.ke] * (u128)(uint64_t)t.p : (u128)0;
        const size_t ke = t.ke, K1 = (size_t)a.K + 1;
        e.b0 = a.bs[ke];
        e.b1 = a.bs[K1 + ke];
        e.b2 = a.bs[2 * K1 + ke];
        e.pad[0] = e.pad[1] = e.pad[2] = 0;
    } else {
        e = req_load(a.req, a.N, rc);
    }
    if (!in) e.place = -1;
    return in ? r : -1;
}

// alpha^2 B0 + 2 alpha b^2 B1 + b^4 B2 + beta p^2: the part of a request's
// gains that depends on no instance
__device__ inline u128 own_value(const PlanReq& e) {
    return mul_u64(mul_u64(e.b0, e.al) + 2 * e.b1, e.al) + e.b2 + mul_u64(e.bp, (uint64_t)e.p);
}

template <int LG, bool kFirst>
__global__ __launch_bounds__(PL_THREADS) void plan_pass_kernel(PlanArgs a) {
    constexpr int P = 1 << LG, RPW = kWave / P;
    __shared__ PlanCand cand[PL_OWN];
    __shared__ PlanMove s_mv;
    __shared__ PlanPart s_best;
    __shared__ VKey wbest[PL_WAVES];
    __shared__ int64_t room_m[PLAN_MAX_INST];
    __shared__ uint8_t over_m[PLAN_MAX_INST];
    __shared__ u128 wred[kFirst ? PL_WAVES : 1];
    __shared__ int listed;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int n = a.n, K = a.K, q = a.pass;
    const uint64_t bb = (uint64_t)a.b * (uint64_t)a.b;
    const bool scorer = (int)blockIdx.x < a.blocks;
    const int u = (int)blockIdx.x - a.blocks, nu = (int)gridDim.x - a.blocks;
    const QEntry* __restrict__ qt = a.qt[kFirst ? 0 : (q - 1) & 1];
    const int64_t* __restrict__ lt = a.lt[kFirst ? 0 : (q - 1) & 1];

    // everything that does not depend on the last move is requested first:
    // the partials, this thread's instance, and its request
    PlanPart pk;
    int ended = 0;
    if (!kFirst) {
        // a launch that ends the plan stores q + 1: its own workgroups go on
        // whichever value they read, and all come to the same end
        ended = *a.done;
        const PlanPart* part = a.part[(q - 1) & 1];
        pk = part[tid < a.parts ? tid : 0];
        if (tid >= a.parts) pk.idx = kNoIdx;
    }
    // weighted and current load of instance i before the last move
    auto inst_w = [&](int i) { return qt[(size_t)K * n + i].qa; };
    auto inst_now = [&](int i) {
        if (!kFirst) return a.now[(q - 1) & 1][i];
        int64_t x = 0;
        for (int c = 0; c < a.chunks; ++c) x += a.now_part[(size_t)c * n + i];
        return x;
    };
    u128 w = 0, wsum = 0;
    int64_t now = 0;
    PlanReq own;
    int64_t own_r = -1;
    if (scorer && a.N > 0) {
        w = inst_w(tid < n ? tid : 0);
        now = inst_now(tid < n ? tid : 0);
        if (!kFirst) wsum = *a.wsum;
        own_r = plan_own<kFirst>(a, 0, own);
    }

    // the move that the last pass found
    if (!kFirst) {
        if (ended != 0 && ended <= q) return;
        const int pw = (a.parts + kWave - 1) / kWave;     // waves that hold partials
        const VKey k = pk.idx != kNoIdx ? VKey{(s128)pk.g, pk.idx} : no_key();
        if (wid < pw) {
            const VKey wk = wave_min_key(k);
            if (lane == 0) wbest[wid] = wk;
        }
        __syncthreads();
        const VKey m = lds_min_key(wbest, pw);
        if (m.idx == kNoIdx) {               // nothing lowers the objective: the plan ends
            if (!scorer && u == 0 && tid == 0) *a.done = q + 1;
            return;
        }
        if (pk.idx == m.idx) {               // keys are distinct: one thread holds it
            const int r = (int)(m.idx / (uint32_t)n);
            PlanMove mv;
            mv.g = pk.g;
            mv.bp = pk.bp;
            mv.fa = pk.fa;
            mv.fb = pk.fb;
            mv.al = pk.al;
            mv.p = pk.p;
            mv.ke = pk.ke;
            mv.src = pk.src;
            mv.tgt = (int)(m.idx - (uint32_t)r * (uint32_t)n);
            mv.r = r;
            mv.c = pk.c;
            s_mv = mv;
        }
        __syncthreads();
        if (!scorer) {
            plan_update(a, s_mv, u, nu);
            return;
        }
    }

    // classification: O, and the targets' room (or -1 outside U)
    if (kFirst) {
        wsum = tid < n ? w : (u128)0;
        for (int i = tid + PL_THREADS; i < n; i += PL_THREADS) wsum += inst_w(i);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint64_t lo = __shfl_xor((unsigned long long)(uint64_t)wsum, o, kWave);
            const uint64_t hi = __shfl_xor((unsigned long long)(uint64_t)(wsum >> 64), o, kWave);
            wsum += ((u128)hi << 64) | (u128)lo;
        }
        if (lane == 0) wred[wid] = wsum;
        __syncthreads();
        wsum = 0;
        for (int i = 0; i < PL_WAVES; ++i) wsum += wred[i];
        if (blockIdx.x == 0 && tid == 0) *a.wsum = wsum;
    }
    // uniform over the workgroup (and so kept in scalar registers)
    const int m_src = kFirst ? -1 : __builtin_amdgcn_readfirstlane(s_mv.src);
    const int m_tgt = kFirst ? -1 : __builtin_amdgcn_readfirstlane(s_mv.tgt);
    const int m_r = kFirst ? -1 : __builtin_amdgcn_readfirstlane(s_mv.r);
    // n den (1 +- theta) mean w against n den w_i: factors of at most 2^21 and 2^30
    const uint32_t nd = (uint32_t)n * (uint32_t)a.theta_den;
    const s128 hi = (s128)mul_u32(wsum, (uint32_t)(a.theta_den + a.theta_num));
    const int dl = a.theta_den - a.theta_num;
    const u128 lo_abs = mul_u32(wsum, (uint32_t)(dl < 0 ? -dl : dl));
    const s128 lo = (s128)(dl < 0 ? (u128)0 - lo_abs : lo_abs);
    for (int i = tid; i < n; i += PL_THREADS) {
        if (i >= PL_THREADS) {
            w = inst_w(i);
            now = inst_now(i);
        }
        if (kFirst) {
            if (blockIdx.x == 0) a.now[0][i] = a.now[1][i] = now;
        } else {
            // F_A(K): its value at k_e, and past k_e the last bucket's share
            // (bp is 0 where k_e = K)
            const int sg = move_sign(m_src, m_tgt, i);
            w += signed_part(s_mv.fa + s_mv.bp, sg);
            now += (int64_t)sg * s_mv.c;
        }
        const s128 nw = (s128)mul_u32(w, nd);
        over_m[i] = nw > hi;
        const bool under = a.u_rule == 0 ? (s128)mul_u32(wide(now), nd) < hi : nw < lo;
        room_m[i] = under ? a.mem_cap - now : -1;
    }
    if (tid == 0) {
        listed = 0;
        s_best.idx = kNoIdx;
        s_best.g = ~(u128)0 >> 1;
    }

    const int64_t runs = ceil_div(a.N, PL_RUN);
    const int sub = lane >> LG, tl = lane & (P - 1);
    constexpr int RPI = PL_OWN / PL_RUN;     // runs per workgroup and iteration
    for (int64_t it = 0; it * RPI * a.blocks < runs; ++it) {
        if (it > 0) own_r = plan_own<kFirst>(a, it, own);
        __syncthreads();             // classified, or the last iteration done
        // the requests on instances of O, packed
        if (wid < PL_OWN / kWave) {
            int s = own.place;
            const bool small = wave_small(own.al, own.bp);
            u128 dv = 0;
            if (kFirst) {
                const size_t at = (size_t)own.ke * n + (s >= 0 ? s : 0);
                own.base = own_value(own) - inst_value(qt[at], lt[at], own.al, own.bp, small);
                if (own_r >= 0) req_store<0, PL_WORDS>(a.req, a.N, own_r, own);
            } else {
                const int ke = own.ke, m_ke = s_mv.ke;
                QEntry f;
                const uint64_t m_al = s_mv.al;
                if (ke <= m_ke) {
                    const bool short_al = (m_al >> 32) == 0;          // uniform
                    f.qa = (short_al ? mul_u32(own.b0, (uint32_t)m_al) : mul_u64(own.b0, m_al)) +
                           own.b1;
                    f.qb = (short_al ? mul_u32(own.b1, (uint32_t)m_al) : mul_u64(own.b1, m_al)) +
                           own.b2;
                } else {
                    f.qa = s_mv.fa + s_mv.bp;
                    f.qb = s_mv.fb + mul_u64(s_mv.bp, bb * (uint64_t)m_ke);
                }
                dv = inst_value(f, move_r(m_al, s_mv.p, m_ke, bb, ke), own.al, own.bp, small);
                if (own_r == m_r) {
                    // it has moved: its gain was base + its target's share,
                    // which now also holds its own curve
                    s = m_tgt;
                    own.base = own_value(own) - (s_mv.g - own.base) - dv;
                    own.place = s;
                    req_store<0, 1>(a.req, a.N, own_r, own);
                    req_store<PL_WORDS - 1, PL_WORDS>(a.req, a.N, own_r, own);
                } else if (s >= 0 && (s == m_src || s == m_tgt)) {
                    own.base -= signed_part(dv, move_sign(m_src, m_tgt, s));
                    req_store<0, 1>(a.req, a.N, own_r, own);
                }
            }
            if (s >= 0 && !over_m[s]) s = -1;
            const uint64_t act = __ballot(s >= 0);
            int at = 0;
            if (lane == 0 && act) at = atomicAdd(&listed, (int)__popcll(act));
            at = __builtin_amdgcn_readfirstlane(at);
            if (s >= 0) {
                PlanCand* c = &cand[at + (int)__popcll(act & ((1ull << lane) - 1))];
                c->base = own.base;
                c->dv = dv;
                c->bp = own.bp;
                c->b0 = own.b0;
                c->b1 = own.b1;
                c->b2 = own.b2;
                c->al = own.al;
                c->need = own.need;
                c->p = own.p;
                c->ke = own.ke;
                c->c = own.c;
                c->r = (int)own_r;
                c->src = s;
            }
        }
        __syncthreads();
        const int cnt = listed;
        VKey feas = no_key();
        int fj = -1;
        constexpr int SLOTS = PL_WAVES * RPW;
        for (int j0 = wid * RPW; j0 < cnt; j0 += PL_U * SLOTS) {
            // PL_U requests per lane group, their reads issued together (those
            // past the last one are not read: with them, plans over many
            // instances were slower than two launches per move: 8 moves, 20000
            // requests on one of 900, prep and projection included: 646 us in two
            // launches each, 709 with, 648 without; on one of 64: 196, 178, 151)
            u128 base[PL_U], dv[PL_U], bp[PL_U];
            uint64_t al[PL_U];
            int64_t need[PL_U];
            int src[PL_U], r[PL_U], bt[PL_U];
            size_t row[PL_U];
            bool valid[PL_U], small[PL_U];
            s128 bg[PL_U];
#pragma unroll
            for (int x = 0; x < PL_U; ++x) {
                const int j = j0 + x * SLOTS + sub;
                valid[x] = j < cnt;
                const PlanCand* e = &cand[valid[x] ? j : 0];
                base[x] = e->base;
                dv[x] = e->dv;
                bp[x] = e->bp;
                al[x] = e->al;
                need[x] = e->need;
                src[x] = e->src;
                r[x] = e->r;
                row[x] = (size_t)e->ke * n;
                small[x] = wave_small(al[x], bp[x]);
                bg[x] = ~(u128)0 >> 1;
                bt[x] = -1;
            }
            for (int c0 = 0; c0 < n; c0 += P * VS_M) {
                QEntry qe[PL_U][VS_M];
                int64_t le[PL_U][VS_M];
#pragma unroll
                for (int x = 0; x < PL_U; ++x) {
                    if (x > 0 && j0 + x * SLOTS >= cnt) break;      // uniform
#pragma unroll
                    for (int i = 0; i < VS_M; ++i) {
                        const int t = c0 + tl + P * i;
                        const size_t o = row[x] + (t < n ? t : 0);
                        qe[x][i] = qt[o];
                        le[x][i] = lt[o];   // row K: unused, there bp is 0
                    }
                }
#pragma unroll
                for (int x = 0; x < PL_U; ++x) {
                    if (j0 + x * SLOTS >= cnt) break;       // uniform
#pragma unroll
                    for (int i = 0; i < VS_M; ++i) {
                        const int t = c0 + tl + P * i;
                        const u128 g = base[x] +
                                       inst_value(qe[x][i], le[x][i], al[x], bp[x], small[x]) +
                                       signed_part(dv[x], move_sign(m_src, m_tgt, t));
                        const bool mig = valid[x] && t < n && t != src[x] &&
                                         need[x] <= room_m[t < n ? t : 0];
                        if (mig && (s128)g < bg[x]) {   // targets ascend within a lane
                            bg[x] = (s128)g;
                            bt[x] = t;
                        }
                    }
                }
            }
            // the lane's best; the lanes of one request are not compared
            // apart, their keys are distinct
#pragma unroll
            for (int x = 0; x < PL_U; ++x) {
                if (bt[x] >= 0 && bg[x] < 0) {
                    const VKey k{bg[x], (uint32_t)r[x] * (uint32_t)n + (uint32_t)bt[x]};
                    if (vless(k, feas)) {
                        feas = k;
                        fj = j0 + x * SLOTS + sub;
                    }
                }
            }
        }
        // the workgroup's best key that lowers the objective
        const int aw = min((cnt + RPW - 1) / RPW, PL_WAVES);   // waves that scored
        if (wid < aw) {
            const VKey wk = wave_min_key(feas);
            if (lane == 0) wbest[wid] = wk;
        }
        __syncthreads();
        VKey k{(s128)s_best.g, s_best.idx};
        if (aw > 0) k = vmin(k, lds_min_key(wbest, aw));
        const uint32_t before = s_best.idx;
        __syncthreads();             // every thread has read s_best and the keys
        if (k.idx != before && feas.idx == k.idx) {   // one lane holds it
            const PlanCand* e = &cand[fj];
            PlanPart v;
            v.g = (u128)k.g;
            v.idx = k.idx;
            v.src = e->src;
            v.ke = e->ke;
            v.c = e->c;
            v.al = e->al;
            v.p = e->p;
            v.bp = e->bp;
            v.fa = mul_u64(e->b0, e->al) + e->b1;
            v.fb = mul_u64(e->b1, e->al) + e->b2;
            v.pad[0] = v.pad[1] = 0;
            s_best = v;
        }
        if (tid == 0) listed = 0;
    }
    __syncthreads();
    if (tid < (int)(sizeof(PlanPart) / 16))
        ((u32x4*)&a.part[q & 1][blockIdx.x])[tid] = ((const u32x4*)&s_best)[tid];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static void launch_score_lg(int lg, int blocks, const VarArgs& a, hipStream_t stream) {
    const dim3 g(blocks), t(VS_THREADS);
    switch (lg) {
        case 0: hipLaunchKernelGGL(var_score_kernel<0>, g, t, 0, stream, a); break;
        case 1: hipLaunchKernelGGL(var_score_kernel<1>, g, t, 0, stream, a); break;
        case 2: hipLaunchKernelGGL(var_score_kernel<2>, g, t, 0, stream, a); break;
        case 3: hipLaunchKernelGGL(var_score_kernel<3>, g, t, 0, stream, a); break;
        default: hipLaunchKernelGGL(var_score_kernel<4>, g, t, 0, stream, a); break;
    }
}

VarPlan plan_variance(const star_load_params& p) {
    VarPlan pl;
    const int n = p.n_inst, N = p.n_req;
    const size_t K1 = (size_t)p.n_buckets + 1;
    int lg = 0;
    while ((1 << lg) < n && lg < VS_MAX_LG) ++lg;
    pl.lg = lg;
    const int64_t blocks = ceil_div(N, (int64_t)VS_WAVES * (kWave >> lg));
    pl.blocks = (int)(blocks < 1 ? 1 : blocks);
    pl.ticketed = pl.blocks <= VS_TICKET_BLOCKS;
    size_t off = STAR_WS_HEADER_BYTES;
    pl.qt_off = off;
    off += align_up((size_t)n * K1 * sizeof(QEntry), 256);
    pl.lt_off = off;
    off += align_up((size_t)n * K1 * sizeof(int64_t), 256);
    pl.bs_off = off;
    off += align_up(3 * K1 * sizeof(u128), 256);
    pl.part_off = off;
    off += align_up((size_t)pl.blocks * sizeof(VPart), 256);
    pl.total = off;
    return pl;
}

hipError_t launch_variance(const star_load_params& p, const VarPlan& pl, const int32_t* cur,
                           const int32_t* rem, const int32_t* inst, const int64_t* load,
                           const uint16_t* beta, star_i128* gain, int32_t* best_target,
                           star_i128* best_gain, star_move* move, char* ws, int32_t* err,
                           hipStream_t stream) {
    static_assert(sizeof(star_i128) == sizeof(u128), "star_i128 is one 128-bit integer");
    const int n = p.n_inst, K = p.n_buckets;
    QEntry* qt = (QEntry*)(ws + pl.qt_off);
    int64_t* lt = (int64_t*)(ws + pl.lt_off);
    u128* bs = (u128*)(ws + pl.bs_off);
    uint32_t* ticket = (uint32_t*)(ws + kHdrVarTicket);
    hipLaunchKernelGGL(var_prep_kernel, dim3(n + 1), dim3(VP_THREADS), 0, stream, load, beta, n,
                       K, (uint64_t)p.bucket * (uint64_t)p.bucket, qt, lt, bs, ticket);
    VarArgs a;
    a.cur = cur;
    a.rem = rem;
    a.inst = inst;
    a.beta = beta;
    a.qt = qt;
    a.lt = lt;
    a.bs = bs;
    a.gain = (u128*)gain;
    a.best_target = best_target;
    a.best_gain = (u128*)best_gain;
    a.move = move;
    a.part = (VPart*)(ws + pl.part_off);
    a.ticket = ticket;
    a.err = err;
    a.N = p.n_req;
    a.n = n;
    a.b = p.bucket;
    a.K = K;
    a.ticketed = pl.ticketed;
    a.H = (int64_t)p.bucket * K;
    launch_score_lg(pl.lg, pl.blocks, a, stream);
    if (move && !pl.ticketed)
        hipLaunchKernelGGL(var_final_kernel, dim3(1), dim3(VS_THREADS), 0, stream, a.part,
                           pl.blocks, inst, n, move);
    return hipGetLastError();
}

PlanPlan plan_plan(const star_plan_params& p) {
    PlanPlan pl;
    pl.v = plan_variance(p.load);
    const size_t n = (size_t)p.load.n_inst, K1 = (size_t)p.load.n_buckets + 1;
    const size_t N = (size_t)p.load.n_req;
    // one request per 2^lg lanes; past one workgroup per compute unit the
    // workgroups take several rounds
    const int64_t blocks = ceil_div((int64_t)N << pl.v.lg, PL_THREADS);
    pl.blocks = (int)(blocks < 1 ? 1 : blocks > PL_MAX_BLOCKS ? PL_MAX_BLOCKS : blocks);
    const int64_t even = align_up((size_t)ceil_div((int64_t)N, PLAN_MAX_CHUNKS), 256);
    pl.chunk_len = (int)(even > PLAN_REQ_CHUNK ? even : PLAN_REQ_CHUNK);
    pl.chunks = (int)ceil_div((int64_t)N, pl.chunk_len);
    size_t off = pl.v.total;
    auto take = [&off](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes, 256);
        return at;
    };
    pl.qt1_off = take(n * K1 * sizeof(QEntry));
    pl.lt1_off = take(n * K1 * sizeof(int64_t));
    for (int i = 0; i < 2; ++i) {
        pl.now_off[i] = take(n * sizeof(int64_t));
        pl.part_off[i] = take((size_t)pl.blocks * sizeof(PlanPart));
    }
    pl.wsum_off = take(sizeof(u128));
    pl.nowp_off = take((size_t)pl.chunks * n * sizeof(int64_t));
    pl.req_off = take(N * sizeof(PlanReq));
    pl.total = off;
    return pl;
}

template <bool kFirst>
static void launch_pass(int lg, int blocks, const PlanArgs& a, hipStream_t stream) {
    const dim3 g(blocks), t(PL_THREADS);
    switch (lg) {
        case 0: hipLaunchKernelGGL((plan_pass_kernel<0, kFirst>), g, t, 0, stream, a); break;
        case 1: hipLaunchKernelGGL((plan_pass_kernel<1, kFirst>), g, t, 0, stream, a); break;
        case 2: hipLaunchKernelGGL((plan_pass_kernel<2, kFirst>), g, t, 0, stream, a); break;
        case 3: hipLaunchKernelGGL((plan_pass_kernel<3, kFirst>), g, t, 0, stream, a); break;
        default: hipLaunchKernelGGL((plan_pass_kernel<4, kFirst>), g, t, 0, stream, a); break;
    }
}

hipError_t launch_plan(const star_plan_params& p, const PlanPlan& pl, const int32_t* cur,
                       const int32_t* rem, int32_t* inst, int64_t* load, const uint16_t* beta,
                       star_move* moves, int32_t* n_moves, char* ws, int32_t* err,
                       hipStream_t stream) {
    const int n = p.load.n_inst, K = p.load.n_buckets;
    PlanArgs a;
    a.cur = cur;
    a.rem = rem;
    a.inst = inst;
    a.load = load;
    a.beta = beta;
    a.qt[0] = (QEntry*)(ws + pl.v.qt_off);
    a.qt[1] = (QEntry*)(ws + pl.qt1_off);
    a.lt[0] = (int64_t*)(ws + pl.v.lt_off);
    a.lt[1] = (int64_t*)(ws + pl.lt1_off);
    for (int i = 0; i < 2; ++i) {
        a.now[i] = (int64_t*)(ws + pl.now_off[i]);
        a.part[i] = (PlanPart*)(ws + pl.part_off[i]);
    }
    a.bs = (u128*)(ws + pl.v.bs_off);
    a.wsum = (u128*)(ws + pl.wsum_off);
    a.now_part = (int64_t*)(ws + pl.nowp_off);
    a.req = (u32x4*)(ws + pl.req_off);
    a.done = (int32_t*)(ws + kHdrPlanDone);
    a.n_moves = n_moves;
    a.moves = moves;
    a.err = err;
    a.N = p.load.n_req;
    a.n = n;
    a.b = p.load.bucket;
    a.K = K;
    a.chunks = pl.chunks;
    a.chunk_len = pl.chunk_len;
    a.blocks = a.parts = pl.blocks;
    a.pass = 0;
    a.theta_num = p.theta_num;
    a.theta_den = p.theta_den;
    a.u_rule = p.u_rule;
    a.mem_rule = p.mem_rule;
    a.min_rem = p.min_rem;
    a.mem_cap = p.mem_cap;
    a.H = (int64_t)p.load.bucket * K;
    hipLaunchKernelGGL(plan_prep_kernel, dim3(n + 1 + pl.chunks), dim3(VP_THREADS), 0, stream, a);
    if (p.max_moves == 0) return hipGetLastError();
    int64_t updaters = ceil_div(4 * (int64_t)(K + 1), PL_THREADS);
    if (updaters > PL_UPDATERS) updaters = PL_UPDATERS;
    launch_pass<true>(pl.v.lg, a.blocks, a, stream);
    for (a.pass = 1; a.pass <= p.max_moves; ++a.pass) {
        if (a.pass == p.max_moves) a.blocks = 0;   // the last move is settled, nothing scored
        launch_pass<false>(pl.v.lg, a.blocks + (int)updaters, a, stream);
    }
    return hipGetLastError();
}

}  // namespace star
