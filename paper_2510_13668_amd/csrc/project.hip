// (b) Per-instance predicted load curves on gfx950.
//
// Section 5.2 (problem formulation, Eq. 4): request r with N(r) = c current
// tokens and N^(r) = l remaining steps holds c + t tokens at future step
// t < l.  Over a horizon of H = b K steps in buckets of b steps, with
// l' = min(l, H), k_e = l' div b and mu = l' mod b, r contributes
//     b c + b(b-1)/2 + b^2 k          to every full bucket k < k_e,
//     mu c + mu k_e b + mu(mu-1)/2    to the partial bucket k_e (mu > 0),
// i.e. sum_{t in bucket}(c + t).  So an instance's curve is
//     L[k] = S_A(k) + b^2 k S_n(k) + D_P[k],
// with S_A(k) / S_n(k) the sum of alpha_r = b c + b(b-1)/2 / the count over
// its requests with k_e > k (suffix sums of histograms indexed by k_e), and
// D_P the partial-bucket histogram.
//
// Request streams of 8192 to 32768 (16-byte aligned arrays, K <= 1024): one
// workgroup per instance reads every request's instance, packs the places of
// its own requests and scatters those into LDS histograms by k_e, runs the
// suffix scan and writes load[i, :].  A crowded instance is taken by slices
// that meet instead, as below.
//
// Longer streams, or many requests per instance: one workgroup per (instance,
// slice of the requests) scatters its instance's requests of its slice into
// LDS histograms by k_e and stores them; the last workgroup of an instance to
// finish sums the slices' histograms and goes on as above.
//
// Shorter streams whose curve planes the scoring wants (K <= 1024) take the
// same kernel with one slice.
//
// Otherwise one workgroup per (instance, bucket chunk): it streams every
// request (coalesced 16-byte reads of four requests for long streams from
// 16-byte aligned arrays, else int32 reads), scatters its own instance's
// requests into LDS histograms with int64 LDS atomics, runs a block-wide
// suffix scan and writes its chunk of load[i, :].  Requests whose k_e lies
// beyond the chunk are folded into one overflow slot, so chunks are
// independent.
#include "star_common.hpp"
#include "star_internal.hpp"

namespace star {

constexpr int PL_THREADS = 512;
constexpr int PL_CHUNK = 1024;
constexpr int PL_RBATCH = 4;      // loads per thread and array in flight together
// 16-byte reads from this many requests on (the longer kernel costs more
// than it saves on short streams: measured 4.4 -> 5.3 us at 64 requests and
// 4.7 -> 5.2 us at 4096; 15.6 -> 11.5 us at 32768)
constexpr int PL_VEC_MIN_REQ = 8192;

// kVec: requests read four at a time (16-byte loads; the arrays are 16-byte
// aligned), which issues a quarter of the load instructions -- the stream
// of every request through each workgroup is bound by instruction issue to
// the address units, not by bytes (measured at 32768 requests on 64
// instances: loads alone cost as much as the whole kernel).
template <bool kVec>
__global__ __launch_bounds__(PL_THREADS) void project_load_kernel(
    const int32_t* __restrict__ cur, const int32_t* __restrict__ rem,
    const int32_t* __restrict__ inst, int N, int n, int b, int K, int chunk,
    int64_t* __restrict__ load, int32_t* __restrict__ err_word) {
    __shared__ int64_t hA[PL_CHUNK + 1];   // alpha_r by k_e (slot len: k_e >= chunk end)
    __shared__ int64_t hN[PL_CHUNK + 1];   // request count by k_e
    __shared__ int64_t hP[PL_CHUNK];       // partial-bucket contributions
    __shared__ int64_t tmp[PL_THREADS / 64 + 1];

    const int tid = threadIdx.x;
    const int i = blockIdx.x;
    const int c = blockIdx.y;
    const int64_t k0 = (int64_t)c * chunk;
    const int64_t k1 = k0 + chunk < K ? k0 + chunk : K;
    const int len = (int)(k1 - k0);
    const int64_t H = (int64_t)b * K;
    const int64_t alpha0 = (int64_t)b * (b - 1) / 2;

    auto clear_lds = [&]() {
        for (int j = tid; j <= len; j += PL_THREADS) {
            hA[j] = 0;
            hN[j] = 0;
            if (j < len) hP[j] = 0;
        }
        __syncthreads();
    };
    int32_t bad = 0;
    // one request: error flags, then its own instance's histogram entries
    auto take = [&](int s, int cr, int lr) {
        int32_t f = 0;
        if (s < 0 || s >= n) f |= STAR_DEV_BAD_INST;
        if (cr < 1) f |= STAR_DEV_BAD_CUR;
        if (lr < 1) f |= STAR_DEV_BAD_REM;
        bad |= f;
        if (f || s != i) return;
        // l' < 2^31, 1 <= b < 2^31: 32-bit division is exact and cheap
        const uint32_t lp = (uint32_t)((int64_t)lr < H ? (int64_t)lr : H);
        const int64_t ke = (int64_t)(lp / (uint32_t)b);
        const int64_t mu = (int64_t)lp - ke * b;
        if (ke > k0) {
            const int jj = (int)((ke < k1 ? ke : k1) - k0);          // 1..len
            atomicAdd((unsigned long long*)&hA[jj], (unsigned long long)((int64_t)b * cr + alpha0));
            atomicAdd((unsigned long long*)&hN[jj], 1ull);
        }
        if (mu > 0 && ke >= k0 && ke < k1) {
            const int64_t pr = mu * cr + mu * ke * b + mu * (mu - 1) / 2;
            atomicAdd((unsigned long long*)&hP[ke - k0], (unsigned long long)pr);
        }
    };
    // Requests are read PL_RBATCH loads per thread at a time, all issued
    // before the first is used (indices clamped, so the loads are
    // unconditional); the first batch is in flight while LDS is cleared.
    if constexpr (kVec) {
        const int N4 = N >> 2;
        const int4* s4 = (const int4*)inst;
        const int4* c4 = (const int4*)cur;
        const int4* l4 = (const int4*)rem;
        if (N4 == 0) clear_lds();
        for (int base = 0; base < N4; base += PL_THREADS * PL_RBATCH) {
            int4 sv[PL_RBATCH], cv[PL_RBATCH], lv[PL_RBATCH];
#pragma unroll
            for (int j = 0; j < PL_RBATCH; ++j) {
                const int q = base + j * PL_THREADS + tid;
                const int qc = q < N4 ? q : N4 - 1;
                sv[j] = s4[qc];
                cv[j] = c4[qc];
                lv[j] = l4[qc];
            }
            if (base == 0) clear_lds();
#pragma unroll
            for (int j = 0; j < PL_RBATCH; ++j) {
                if (base + j * PL_THREADS + tid >= N4) continue;
                take(sv[j].x, cv[j].x, lv[j].x);
                take(sv[j].y, cv[j].y, lv[j].y);
                take(sv[j].z, cv[j].z, lv[j].z);
                take(sv[j].w, cv[j].w, lv[j].w);
            }
        }
        for (int r = 4 * N4 + tid; r < N; r += PL_THREADS) take(inst[r], cur[r], rem[r]);
    } else {
        if (N == 0) clear_lds();
        for (int base = 0; base < N; base += PL_THREADS * PL_RBATCH) {
            int sv[PL_RBATCH], cv[PL_RBATCH], lv[PL_RBATCH];
#pragma unroll
            for (int j = 0; j < PL_RBATCH; ++j) {
                const int r = base + j * PL_THREADS + tid;
                const int rc = r < N ? r : N - 1;
                sv[j] = inst[rc];
                cv[j] = cur[rc];
                lv[j] = rem[rc];
            }
            if (base == 0) clear_lds();
#pragma unroll
            for (int j = 0; j < PL_RBATCH; ++j) {
                if (base + j * PL_THREADS + tid >= N) continue;
                take(sv[j], cv[j], lv[j]);
            }
        }
    }
    if (i == 0 && c == 0) {
        bad = wave_or_i32(bad);
        if ((tid & 63) == 0) report_error(err_word, bad);
    }
    __syncthreads();

    // Suffix sums over x[q] = h[q + 1], q in [0, len): thread t owns the
    // reversed positions p in [t*seg, (t+1)*seg), q = len - 1 - p.
    const int seg = (len + PL_THREADS - 1) / PL_THREADS;
    const int p0 = tid * seg;
    const int p1 = p0 + seg < len ? p0 + seg : len;
    int64_t la = 0, ln = 0;
    for (int p = p0; p < p1; ++p) {
        const int q = len - 1 - p;
        la += hA[q + 1];
        ln += hN[q + 1];
    }
    int64_t ra = block_exclusive_scan_i64<PL_THREADS>(la, OpAdd(), 0, tmp, (int64_t*)nullptr);
    int64_t rn = block_exclusive_scan_i64<PL_THREADS>(ln, OpAdd(), 0, tmp, (int64_t*)nullptr);
    const int64_t bb = (int64_t)b * b;
    int64_t* out = load + (int64_t)i * K;
    for (int p = p0; p < p1; ++p) {
        const int q = len - 1 - p;
        ra += hA[q + 1];
        rn += hN[q + 1];
        const int64_t k = k0 + q;
        out[k] = ra + bb * k * rn + hP[q];
    }
}

// ---------------------------------------------------------------------------
// split projection
// ---------------------------------------------------------------------------
constexpr int PS_THREADS = 1024;     // one bucket per thread when the slices are summed
constexpr int PS_MAX_K = PS_THREADS;
constexpr int PS_MAX_SLICES = 8;
constexpr int PS_TARGET_GROUPS = 256;  // workgroups the slices aim for (one per CU)
constexpr int PS_MIN_SLICE = 1024;     // requests per slice at least
constexpr int PS_RV = 2;               // 16-byte reads per thread and array in flight
// request streams from which the split is used (at 4096 requests on 16
// instances it took 11.4 us against 4.6 + 4 us for the chunked kernel and
// the separate plane preparation: the meeting's latency dominates)
constexpr int PS_MIN_REQ = 8192;
// One workgroup per instance instead of slices that meet, for streams that one
// round of its reads covers.  us per call at K = 1024, remaining lengths of a
// Pareto law (slices that meet for every instance, this kernel); blocks: an
// instance's requests are neighbours; 1/4, all: that share of all requests on
// one instance, in front of the others:
//                blocks     shuffled   1/4         all
//   32768 x 64:  10.1, 6.5  11.2, 7.1  20.5, 17.0  20.8, 20.2
//   32768 x 16:  11.2, 8.4  10.3, 8.9  13.9, 12.1  14.0, 12.2
//   16384 x 8:   10.9, 8.0   8.9, 8.4  10.7, 9.4   10.6, 9.4
//   8192 x 64:    9.3, 5.9   9.7, 6.1  10.5, 7.7   10.8, 10.4
//   32768 x 80:  13.3, 6.6  13.7, 7.9  24.5, 17.2  22.2, 25.4
//   32768 x 128: 10.7, 6.4  12.2, 6.8  21.5, 16.9  34.0, 41.5
// (80 instances leave compute units for two slices each, 86 and more for none;
// half of all requests on one of 128: 33.6, 25.0).
// More per instance on average (32768 x 8) goes to slices at once: most
// instances would.
constexpr int PW_RV = 8;               // 16-byte reads of instances per thread
constexpr int PW_U = 2;                // list entries per thread in flight
constexpr int PW_MAX_REQ = PS_THREADS * PW_RV * 4;
static_assert(PW_MAX_REQ <= 65536 && PW_RV <= 8, "16-bit places, 32 marks");
constexpr int PW_MAX_PER_INST = 2048;  // requests per instance, on average
// requests of an instance that its one workgroup takes: 8.9 us for 2816 of them
// in a stream of 8192 against 9.4 for slices, 7.9 against 9.2 for 2304
constexpr int PW_ALONE = 3072;

struct SplitArgs {
    const int32_t* cur;
    const int32_t* rem;
    const int32_t* inst;
    int64_t* load;
    int32_t* err_word;
    int64_t* part;          // [n][slices][arrays][KP]: the slices' histograms
    uint32_t* tickets;      // [n] arrival counters (zero between calls)
    CurvePlanes planes;     // written too when planes.tpm is set
    int N, n, b, K, KP, slices, slice_len;
};

// Histograms by k_e, in LDS: [0] alpha_r and [1] the request count (k_e 1..K),
// [2] partial-bucket contributions (k_e 0..K-1).  Packed, for streams of at
// most PW_MAX_REQ requests: [0] the sum of cur_len with the count above it
// (alpha_r = b cur_len + alpha0), [1] the partial-bucket contributions; two
// 64-bit LDS atomics per request instead of three, whose serial turns on a
// popular bucket are what a crowded instance costs.
constexpr int PS_H = PS_MAX_K + 2;
constexpr int PW_COUNT_SHIFT = 47;     // 2^15 requests of cur_len < 2^31 below it
static_assert((int64_t)PW_MAX_REQ << 31 <= (int64_t)1 << PW_COUNT_SHIFT, "sums stay below the count");
template <bool kPacked> constexpr int ps_arrays() { return kPacked ? 2 : 3; }

template <bool kPacked>
__device__ __forceinline__ void clear_hists(int64_t (*h)[PS_H], int KP) {
    for (int j = threadIdx.x; j < KP; j += PS_THREADS) {
#pragma unroll
        for (int x = 0; x < ps_arrays<kPacked>(); ++x) h[x][j] = 0;
    }
}

// one request into the histograms
template <bool kPacked>
__device__ __forceinline__ void scatter_request(int cr, int lr, int b, int64_t H, int64_t alpha0,
                                                int64_t (*h)[PS_H]) {
    // l' < 2^31, 1 <= b < 2^31: 32-bit division is exact
    const uint32_t lp = (uint32_t)((int64_t)lr < H ? (int64_t)lr : H);
    const uint32_t ke = lp / (uint32_t)b;
    const int64_t mu = (int64_t)(lp - ke * (uint32_t)b);
    if (ke > 0) {
        if constexpr (kPacked) {
            atomicAdd((unsigned long long*)&h[0][ke], (1ull << PW_COUNT_SHIFT) + (uint32_t)cr);
        } else {
            atomicAdd((unsigned long long*)&h[0][ke],
                      (unsigned long long)((int64_t)b * cr + alpha0));
            atomicAdd((unsigned long long*)&h[1][ke], 1ull);
        }
    }
    if (mu > 0) {                                     // then k_e < K
        const int64_t pr = mu * cr + mu * (int64_t)ke * b + mu * (mu - 1) / 2;
        atomicAdd((unsigned long long*)&h[ps_arrays<kPacked>() - 1][ke], (unsigned long long)pr);
    }
}

// Slice sl's requests of instance i into the histograms, every request of the
// slice checked; the histograms are cleared first, while the first reads are in
// flight (kClear).  Returns the STAR_DEV_* bits that this thread saw.
template <bool kPacked, bool kClear>
__device__ __forceinline__ int32_t scatter_slice(const SplitArgs& a, int i, int sl,
                                                 int64_t (*h)[PS_H]) {
    const int tid = threadIdx.x, b = a.b;
    const int64_t H = (int64_t)b * a.K;
    const int64_t alpha0 = (int64_t)b * (b - 1) / 2;
    const int64_t r0 = (int64_t)sl * a.slice_len;     // slice_len % 4 == 0
    const int64_t rend = r0 + a.slice_len;
    const int r1 = (int)(rend < a.N ? rend : a.N);
    int32_t bad = 0;
    auto take = [&](int s, int cr, int lr) {
        int32_t f = 0;
        if (s < 0 || s >= a.n) f |= STAR_DEV_BAD_INST;
        if (cr < 1) f |= STAR_DEV_BAD_CUR;
        if (lr < 1) f |= STAR_DEV_BAD_REM;
        bad |= f;
        if (f || s != i) return;
        scatter_request<kPacked>(cr, lr, b, H, alpha0, h);
    };
    const int4* s4 = (const int4*)a.inst;
    const int4* c4 = (const int4*)a.cur;
    const int4* l4 = (const int4*)a.rem;
    const int q0 = (int)(r0 >> 2), q1 = r1 >> 2;    // whole groups of four requests
    bool cleared = !kClear;
    for (int base = q0; base < q1 || !cleared; base += PS_THREADS * PS_RV) {
        int4 sv[PS_RV], cv[PS_RV], lv[PS_RV];
#pragma unroll
        for (int j = 0; j < PS_RV; ++j) {
            const int q = base + j * PS_THREADS + tid;
            const int qc = q < q1 ? q : (q1 > q0 ? q1 - 1 : q0);
            if (q1 > q0) {
                sv[j] = s4[qc];
                cv[j] = c4[qc];
                lv[j] = l4[qc];
            }
        }
        if (!cleared) {
            clear_hists<kPacked>(h, a.KP);
            __syncthreads();
            cleared = true;
        }
#pragma unroll
        for (int j = 0; j < PS_RV; ++j) {
            if (base + j * PS_THREADS + tid >= q1) continue;
            take(sv[j].x, cv[j].x, lv[j].x);
            take(sv[j].y, cv[j].y, lv[j].y);
            take(sv[j].z, cv[j].z, lv[j].z);
            take(sv[j].w, cv[j].w, lv[j].w);
        }
    }
    for (int r = 4 * q1 + tid; r < r1; r += PS_THREADS) take(a.inst[r], a.cur[r], a.rem[r]);
    return bad;
}

// The curve of instance i, and its scoring planes where they are wanted, from
// the histograms' sums: thread t holds bucket q = K-1-t, with xa and xn the sums
// of h_A and h_N at q+1 and xp that of h_P at q (zeros past K).  hA and hN are
// overwritten after the first scan's barriers.
__device__ __forceinline__ void finish_curve(const SplitArgs& a, int64_t xa, int64_t xn, int64_t xp,
                                             int64_t* hA, int64_t* hN, int64_t* tmp) {
    const int tid = threadIdx.x, i = blockIdx.x, K = a.K, b = a.b;
    const int q = K - 1 - tid;
    const bool live = tid < K;
    // inclusive prefix in thread order = suffix sums over k_e > q
    block_incl_add2_i64<PS_THREADS>(xa, xn, tmp);
    const int64_t bb = (int64_t)b * b;
    const int64_t Lq = xa + bb * q * xn + xp;
    if (live) a.load[(int64_t)i * K + q] = Lq;
    if (!a.planes.tpm) return;

    // The scoring's planes of this instance (see CurvePlanes):
    // SM (suffix max of L) is the inclusive prefix max in this thread order;
    // PM (max of L[j] + b^2 j over j < k) takes the forward order j = t,
    // with L passed through LDS.
    const CurvePlanes& pl = a.planes;
    if (live) hA[q] = Lq;
    __syncthreads();
    const int j = tid;
    int64_t sm = live ? Lq : INT64_MIN;
    int64_t pm = j < K ? hA[j] + bb * j : INT64_MIN;
    block_incl_max2_i64<PS_THREADS>(sm, pm, tmp);
    hN[j] = pm;                                   // inclusive; PM[j] is thread j-1's
    __syncthreads();
    if (live) {
        pl.tl[q * pl.sk + i * pl.st] = Lq;
        if (q > 0) pl.tsm[(q - 1) * pl.sk + i * pl.st] = sm;
        else pl.peak[i] = sm;
    }
    if (j < K) pl.tpm[j * pl.sk + i * pl.st] = j > 0 ? hN[j - 1] : INT64_MIN;
    if (tid == 0) {
        pl.tpm[K * pl.sk + i * pl.st] = hN[K - 1];
        pl.tl[K * pl.sk + i * pl.st] = INT64_MIN;
        pl.tsm[(K - 1) * pl.sk + i * pl.st] = INT64_MIN;
        pl.tsm[K * pl.sk + i * pl.st] = INT64_MIN;
    }
}

// What thread t of instance i's curve needs of the histograms: bucket q = K-1-t
// takes the sums of alpha_r and of the counts at q+1 and of the partial-bucket
// contributions at q (zeros past K).
template <bool kPacked>
__device__ __forceinline__ void curve_terms(const SplitArgs& a, const int64_t* x, int64_t& xa,
                                            int64_t& xn, int64_t& xp) {
    if constexpr (kPacked) {
        xn = x[0] >> PW_COUNT_SHIFT;
        xa = (int64_t)a.b * (x[0] & (((int64_t)1 << PW_COUNT_SHIFT) - 1)) +
             (int64_t)a.b * (a.b - 1) / 2 * xn;
        xp = x[1];
    } else {
        xa = x[0];
        xn = x[1];
        xp = x[2];
    }
}

// This workgroup's histograms as they are: nothing to meet.
template <bool kPacked>
__device__ __forceinline__ void own_terms(const SplitArgs& a, const int64_t (*h)[PS_H],
                                          int64_t& xa, int64_t& xn, int64_t& xp) {
    constexpr int A = ps_arrays<kPacked>();
    const int q = a.K - 1 - (int)threadIdx.x;
    int64_t x[A] = {};
    if (q >= 0)
#pragma unroll
        for (int i = 0; i < A; ++i) x[i] = h[i][i < A - 1 ? q + 1 : q];
    curve_terms<kPacked>(a, x, xa, xn, xp);
}

// The slices of instance i meet: slice sl's histograms go to the instance's
// shares by coherent 16-byte stores, and the last workgroup to arrive (true)
// sums the slices', every read issued first.
template <bool kPacked>
__device__ __forceinline__ bool meet_slices(const SplitArgs& a, int i, int sl,
                                            const int64_t (*h)[PS_H], uint32_t* s_ticket,
                                            int64_t& xa, int64_t& xn, int64_t& xp) {
    constexpr int A = ps_arrays<kPacked>();
    const int tid = threadIdx.x, KP = a.KP;
    const uint32_t share = (uint32_t)(A * KP) * 8u;           // bytes per slice
    const __amdgpu_buffer_rsrc_t rs =
        xch_rsrc(a.part + (size_t)i * a.slices * A * KP, (uint32_t)a.slices * share);
    for (int p = tid; p < A * KP / 2; p += PS_THREADS) {
        const int arr = p / (KP / 2), j = 2 * (p - arr * (KP / 2));
        const int64_t v0 = h[arr][j], v1 = h[arr][j + 1];
        const u32x4 v = {(uint32_t)v0, (uint32_t)(v0 >> 32), (uint32_t)v1, (uint32_t)(v1 >> 32)};
        xch_store(v, rs, (uint32_t)sl * share + (uint32_t)(arr * KP + j) * 8u);
    }
    xch_wait_stores();
    if (!xch_last_arrival(&a.tickets[i], (uint32_t)a.slices, s_ticket)) return false;
    const int q = a.K - 1 - tid;
    u32x2 v[A][PS_MAX_SLICES];
#pragma unroll
    for (int u = 0; u < PS_MAX_SLICES; ++u)
#pragma unroll
        for (int x = 0; x < A; ++x) {
            const uint32_t o = (uint32_t)u * share + (uint32_t)(x * KP + (x < A - 1 ? q + 1 : q)) * 8u;
            v[x][u] = xch_load_b64(rs, q >= 0 && u < a.slices ? o : kXchOob);
        }
    int64_t x[A];
#pragma unroll
    for (int k = 0; k < A; ++k) {
        x[k] = 0;
#pragma unroll
        for (int u = 0; u < PS_MAX_SLICES; ++u)
            x[k] += (int64_t)(((uint64_t)v[k][u].y << 32) | v[k][u].x);
    }
    curve_terms<kPacked>(a, x, xa, xn, xp);
    return true;
}

// kMeet: the slices of an instance meet at a counter.  Otherwise one workgroup
// takes an instance's whole stream and its histograms never leave LDS: for
// streams below the split's whose curve planes are wanted too.  One launch then
// does what project_load_kernel and score_prep_kernel do in two: whole calls at
// 4096 requests x 16 instances x 512 buckets 26.1 -> 24.0 us, 7000 x 40 x 200
// without a top-k 17.1 -> 12.7, 100 x 20 x 300 21.3 -> 19.3.
template <bool kMeet>
__global__ __launch_bounds__(PS_THREADS) void project_split_kernel(SplitArgs a) {
    __shared__ int64_t h[ps_arrays<false>()][PS_H];
    __shared__ int64_t tmp[2 * PS_THREADS / 64];
    __shared__ uint32_t s_ticket;
    const int tid = threadIdx.x;
    const int i = blockIdx.x, sl = blockIdx.y;
    int32_t bad = scatter_slice<false, true>(a, i, sl, h);
    if (i == 0) {
        bad = wave_or_i32(bad);
        if ((tid & 63) == 0) report_error(a.err_word, bad);
    }
    __syncthreads();
    int64_t xa, xn, xp;
    if constexpr (kMeet) {
        if (!meet_slices<false>(a, i, sl, h, &s_ticket, xa, xn, xp)) return;
    } else {
        own_terms<false>(a, h, xa, xn, xp);
    }
    finish_curve(a, xa, xn, xp, h[0], h[1], tmp);
}

// One workgroup takes an instance's whole stream where the instance is not
// crowded, and slices that meet take it where it is: the time of one workgroup
// grows with its own requests, and their spread over the instances is known on
// the device alone.  Every workgroup of an instance reads all instances and
// counts its requests, so all of them come to the same choice.
//
// blockIdx.y 0 goes on alone up to PW_ALONE requests: it reads lengths only of
// its own: each thread marks those among its 32, a prefix sum over the wave
// packs their places into a list, and the threads then take one list entry
// each, so that every lane has a request whatever their order in the stream.
// It checks the validity of a share of N / n of all requests besides.
// blockIdx.y - 1 = 0..slices-1: the slices, which meet past PW_ALONE requests;
// they scatter before they know, on compute units that would be idle.  Without
// any (slices 0), the first workgroup takes a crowded instance as one slice.
//
// A chain of latencies bounds the first workgroup: 6.5 us at 32768 x 64, K =
// 1024, of which a launch on its own is about 2.5, where slices that meet took
// 10.1; on a crowded instance, the serial atomics on its popular buckets do.
// Below 8192 requests it is 0.8-1.9 us slower than one slice of the split
// kernel (100 to 8191 requests, 3 to 64 instances).
__global__ __launch_bounds__(PS_THREADS) void project_whole_kernel(SplitArgs a) {
    __shared__ int64_t h[ps_arrays<true>()][PS_H];
    __shared__ int64_t tmp[2 * PS_THREADS / 64];
    __shared__ uint16_t list[PW_ALONE];             // this instance's requests
    __shared__ int count;
    __shared__ uint32_t s_ticket;
    const int tid = threadIdx.x, i = blockIdx.x, n = a.n;
    const int q1 = a.N >> 2;                        // whole groups of four requests
    const int4* s4 = (const int4*)a.inst;
    int4 sv[PW_RV];
#pragma unroll
    for (int j = 0; j < PW_RV; ++j) {
        const int q = j * PS_THREADS + tid;
        sv[j] = make_int4(-1, -1, -1, -1);
        if (q < q1) sv[j] = s4[q];
    }
    if (tid == 0) count = 0;
    int64_t xa, xn, xp;
    if (blockIdx.y > 0) {
        const int sl = blockIdx.y - 1;
        scatter_slice<true, true>(a, i, sl, h);
        int own = 0;
#pragma unroll
        for (int j = 0; j < PW_RV; ++j)
            own += (int)(__popcll(__ballot(sv[j].x == i)) + __popcll(__ballot(sv[j].y == i)) +
                         __popcll(__ballot(sv[j].z == i)) + __popcll(__ballot(sv[j].w == i)));
        if ((tid & (kWave - 1)) == 0 && own) atomicAdd(&count, own);
        __syncthreads();
        if (count <= PW_ALONE) return;
        if (!meet_slices<true>(a, i, sl, h, &s_ticket, xa, xn, xp)) return;
    } else {
        const int b = a.b;
        const int64_t H = (int64_t)b * a.K;
        const int64_t alpha0 = (int64_t)b * (b - 1) / 2;
        const int4* c4 = (const int4*)a.cur;
        const int4* l4 = (const int4*)a.rem;
        int32_t bad = 0;
        auto check = [&](int s, int cr, int lr) {
            if (s < 0 || s >= n) bad |= STAR_DEV_BAD_INST;
            if (cr < 1) bad |= STAR_DEV_BAD_CUR;
            if (lr < 1) bad |= STAR_DEV_BAD_REM;
        };
        // the groups whose validity this workgroup checks; the first are requested now
        const int v0 = (int)((int64_t)q1 * i / n), v1 = (int)((int64_t)q1 * (i + 1) / n);
        int4 vs, vc, vl;
        if (v0 + tid < v1) {
            vs = s4[v0 + tid];
            vc = c4[v0 + tid];
            vl = l4[v0 + tid];
        }
        clear_hists<true>(h, a.KP);
        __syncthreads();
        uint32_t own = 0;
#pragma unroll
        for (int j = 0; j < PW_RV; ++j) {
            own |= (sv[j].x == i ? 1u : 0u) << (4 * j);
            own |= (sv[j].y == i ? 2u : 0u) << (4 * j);
            own |= (sv[j].z == i ? 4u : 0u) << (4 * j);
            own |= (sv[j].w == i ? 8u : 0u) << (4 * j);
        }
        const int mine = __builtin_popcount(own);
        const int incl = wave_incl_add_i32(mine);
        const int sum = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (sum > 0) {
            int at = 0;
            if ((tid & (kWave - 1)) == 0) at = atomicAdd(&count, sum);
            at = __builtin_amdgcn_readfirstlane(at) + incl - mine;
            for (; own && at < PW_ALONE; own &= own - 1) {
                const int bit = __ffs((int)own) - 1;
                list[at++] = (uint16_t)(((bit >> 2) * PS_THREADS + tid) * 4 + (bit & 3));
            }
        }
        __syncthreads();
        const int cnt = count;
        const bool alone = cnt <= PW_ALONE;
        for (int e0 = tid; alone && e0 < cnt; e0 += PS_THREADS * PW_U) {
            int cr[PW_U], lr[PW_U];
#pragma unroll
            for (int u = 0; u < PW_U; ++u) {
                const int e = e0 + u * PS_THREADS;
                const int r = list[e < cnt ? e : e0];
                cr[u] = a.cur[r];
                lr[u] = a.rem[r];
            }
#pragma unroll
            for (int u = 0; u < PW_U; ++u) {
                if (e0 + u * PS_THREADS < cnt && cr[u] >= 1 && lr[u] >= 1)
                    scatter_request<true>(cr[u], lr[u], b, H, alpha0, h);
            }
        }
        for (int r = 4 * q1 + tid; r < a.N; r += PS_THREADS) {
            const int s = a.inst[r], cr = a.cur[r], lr = a.rem[r];
            check(s, cr, lr);
            if (alone && s == i && cr >= 1 && lr >= 1)
                scatter_request<true>(cr, lr, b, H, alpha0, h);
        }
        for (int q = v0 + tid; q < v1; q += PS_THREADS) {
            if (q != v0 + tid) {
                vs = s4[q];
                vc = c4[q];
                vl = l4[q];
            }
            check(vs.x, vc.x, vl.x);
            check(vs.y, vc.y, vl.y);
            check(vs.z, vc.z, vl.z);
            check(vs.w, vc.w, vl.w);
        }
        bad = wave_or_i32(bad);
        if ((tid & 63) == 0) report_error(a.err_word, bad);
        if (!alone) {
            if (a.slices > 0) return;
            scatter_slice<true, false>(a, i, 0, h);
        }
        __syncthreads();
        own_terms<true>(a, h, xa, xn, xp);
    }
    finish_curve(a, xa, xn, xp, h[0], h[1], tmp);
}

LoadPlan plan_load(const star_load_params& p) {
    LoadPlan pl;
    pl.chunk = p.n_buckets < PL_CHUNK ? p.n_buckets : PL_CHUNK;
    pl.n_chunks = (int)ceil_div(p.n_buckets, pl.chunk);
    pl.split = p.n_req >= PS_MIN_REQ && p.n_buckets <= PS_MAX_K && p.n_inst <= kMaxTickets;
    pl.whole = pl.split && p.n_req <= PW_MAX_REQ &&
               p.n_req <= (int64_t)PW_MAX_PER_INST * p.n_inst;
    if (pl.split) {
        int s = (int)ceil_div(PS_TARGET_GROUPS, p.n_inst);
        s = s < PS_MAX_SLICES ? s : PS_MAX_SLICES;
        const int smax = (int)(p.n_req / PS_MIN_SLICE);
        s = s < smax ? s : smax;
        s = s > 1 ? s : 1;
        pl.kp = (int)align_up((size_t)p.n_buckets + 1, 2);
        pl.slice_len = (int)align_up((size_t)ceil_div(p.n_req, s), 4);
        pl.slices = (int)ceil_div(p.n_req, pl.slice_len);
        // (the crowded instances' fewer slices of two arrays fit in it too)
        pl.part_bytes = align_up((size_t)p.n_inst * pl.slices * ps_arrays<false>() * pl.kp * 8, 256);
        if (pl.whole) {
            // the slices that a crowded instance would need, on the compute
            // units that the instances' first workgroups leave: one more
            // workgroup than units, and the spread streams wait for it (four
            // slices of 64 instances: 8.1 us, not 6.5, at 32768 requests)
            const int left = PS_TARGET_GROUPS / p.n_inst - 1;
            s = s < left ? s : left;
            pl.slice_len = s < 2 ? p.n_req : (int)align_up((size_t)ceil_div(p.n_req, s), 4);
            pl.slices = s < 2 ? 0 : (int)ceil_div(p.n_req, pl.slice_len);
        }
    }
    return pl;
}

hipError_t launch_project_load(const star_load_params& p, const LoadPlan& pl, const int32_t* cur,
                               const int32_t* rem, const int32_t* inst, int64_t* load,
                               char* ws, char* part, const CurvePlanes* planes,
                               bool* planes_written, hipStream_t stream) {
    int32_t* err_word = (int32_t*)(ws + kHdrErrorWord);
    const bool aligned16 = (((uintptr_t)cur | (uintptr_t)rem | (uintptr_t)inst) & 15) == 0;
    if (planes_written) *planes_written = false;
    // shorter streams: one slice, where the curve planes are wanted
    const bool shorter = !pl.split && planes && p.n_buckets <= PS_MAX_K;
    if ((pl.split || shorter) && aligned16) {
        SplitArgs a;
        a.cur = cur; a.rem = rem; a.inst = inst; a.load = load; a.err_word = err_word;
        a.part = (int64_t*)part;
        a.tickets = (uint32_t*)(ws + kHdrTickets);
        a.planes = planes ? *planes : CurvePlanes{};
        if (planes_written) *planes_written = planes != nullptr;
        a.N = p.n_req; a.n = p.n_inst; a.b = p.bucket; a.K = p.n_buckets;
        a.KP = (int)align_up((size_t)p.n_buckets + 1, 2);
        a.slices = shorter ? 1 : pl.slices;
        a.slice_len = shorter ? p.n_req : pl.slice_len;
        if (pl.whole)
            hipLaunchKernelGGL(project_whole_kernel, dim3(p.n_inst, pl.slices + 1),
                               dim3(PS_THREADS), 0, stream, a);
        else if (shorter)
            hipLaunchKernelGGL(project_split_kernel<false>, dim3(p.n_inst), dim3(PS_THREADS), 0,
                               stream, a);
        else
            hipLaunchKernelGGL(project_split_kernel<true>, dim3(p.n_inst, pl.slices),
                               dim3(PS_THREADS), 0, stream, a);
        return hipGetLastError();
    }
    const bool vec = p.n_req >= PL_VEC_MIN_REQ && aligned16;
    if (vec)
        hipLaunchKernelGGL(project_load_kernel<true>, dim3(p.n_inst, pl.n_chunks), dim3(PL_THREADS),
                           0, stream, cur, rem, inst, p.n_req, p.n_inst, p.bucket, p.n_buckets,
                           pl.chunk, load, err_word);
    else
        hipLaunchKernelGGL(project_load_kernel<false>, dim3(p.n_inst, pl.n_chunks), dim3(PL_THREADS),
                           0, stream, cur, rem, inst, p.n_req, p.n_inst, p.bucket, p.n_buckets,
                           pl.chunk, load, err_word);
    return hipGetLastError();
}

}  // namespace star
