// Verification of the replayed tree on gfx950 (Section 2.3, eq. (1);
// Appendix A: recursive rejection sampling without replacement; Section 3.3:
// the probabilities are those of the replayed candidates).
//
//   target_partials  a workgroup per chunk of the flat target: one streaming
//                    read of every target row of the tree; online max and sum
//                    of exp per piece of a row (binary32 terms, binary64 per
//                    lane). More workgroups write the walk's node records.
//   verify_walk      G workgroups per request, by tickets. All G
//                    workgroups of a request replay the same scalar walk;
//                    every vocabulary-wide reduction of the walk (residual
//                    mass after a rejection, the bonus draw) is split over
//                    them and exchanged through the request's tagged slots
//                    (each workgroup polls the others' slots).
//
// Closed form of WoR-RRS used by the walk (equal to the literal recursion
// of residuals; derived from eq. (1) and the without-replacement update):
// with C_0 = 0, S_0 = 1, Z_0 = 1 at a node, child i with token y is accepted
// iff U < max(p(y) - C_i q(y), 0) / (W_i q(y)), W_i = Z_i / S_i; on
// rejection C_{i+1} = C_i + W_i, S_{i+1} = S_i - q(y),
// Z_{i+1} = sum_v max(p_v - C_{i+1} q_v, 0). The bonus token is
// argmax_v ln max(p_v - C q_v, 0) + G_v (Gumbel-max of the residual; C = 0
// at an accepted leaf).
#include <math.h>

#include <algorithm>
#include <atomic>

#include "tsb_device.hpp"
#include "tsb_exchange.hpp"
#include "tsb_kernels.hpp"
#include "tsb_target.hpp"

namespace tsb {

// ------------------------------------------------------------------ K4
// The target stream on a grid of its own (tsb_verify and the other
// verification entry points; a round runs it inside the replay scan's grid).
template <int DT, bool VEC>
__global__ __launch_bounds__(kBlock) void target_partials(const void* __restrict__ target, int V, int B, int nrows,
                                                          long long chunk, int P, float invT,
                                                          const int32_t* __restrict__ n_nodes,
                                                          float* __restrict__ tm, double* __restrict__ ts,
                                                          int* __restrict__ tf, XRegion X, int R, int ngroups,
                                                          RecordJob rec) {
    if ((int)blockIdx.x >= ngroups) {
        record_block<DT>(rec, (int)blockIdx.x - ngroups, invT);
        return;
    }
    target_chunk<DT, VEC, kTargetPrefetch>(blockIdx.x, ngroups, target, V, B, nrows, chunk, P, invT, n_nodes, tm, ts, tf, X, R);
}

// ------------------------------------------------------------------ K5
struct WalkArgs {
    const void* draft;
    const double* draft_lse;
    const void* target;
    tsb_tree tree;
    const int32_t* node_tok;
    tsb_verdict out;
    const float* tm;
    const double* ts;
    const int* tf;
    XRegion X;  // exchange slots of the requests
    int V, D, B, S4;
    int R, G;   // requests and workgroups per request of the launch (tickets)
    unsigned long long* stats;  // work counters (null: none)
    float invT;
    uint32_t k0, k1, step;
    // pool walk only: pools [R, D, P] and transition scores [R, D-1, P, P]
    const int32_t* pool_tok;
    const float* trans;
    int P;
    // node records (kRecWords per node), written by the round's merge or by the
    // kernel before a walk launched on its own (not for the pool walk)
    const uint32_t* nrec;
    // the RRS walk reads each target row as it enters the node (else the row
    // normalisers come from a stream of every row, through the records or the
    // partials), except rows 0 and 1, streamed before it into their own
    // partials [R][kChainRows][kChainPieces]
    int reads_rows;
    const float* cm;
    const double* cs;
    const int* cf;
};

// binary64 log-sum-exp of target row (r, node) from its segment partials
__device__ double target_lse(const WalkArgs& A, int r, int node, int* bad) {
    return target_row_lse(A.tm, A.ts, A.tf, A.S4, (size_t)r * (A.B + 1) + node, bad);
}

__device__ __forceinline__ double rec_f64(uint32_t lo, uint32_t hi) {
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

struct SplitF {  // binary64 value as binary32 hi + lo
    float hi, lo;
};
__device__ __forceinline__ SplitF split(double v) {
    SplitF s;
    s.hi = (float)v;
    s.lo = (float)(v - (double)s.hi);
    return s;
}

// ---------------------------------------------------------------- walk
// A walk workgroup owns the slice [v0, v1) of the vocabulary; thread t owns
// the slice's groups of four tokens at v0 + 4 (k kWalkThreads + t). The raw
// logits of the node the walk is at are loaded into registers when it enters
// the node; once the node needs them, every thread evaluates, in binary64,
// p~_v = exp(a^t_{u,v} - L0) (L0 the streamed estimate of the target
// normaliser) and q_v = exp(a^d_{depth(u),v} - lse_d) of its tokens into LDS,
// where the residual passes after rejections and the residual bonus read them
// (only the owner does: no barrier). Slices of up to kWalkSliceTokens leave
// room for two workgroups on a compute unit; slices above kWalkHeldTokens are
// recomputed in every pass.
//
// Bound by latency: a node is a chain of its record's load, its rows' load
// (after the record: the topology checks come first) and an exchange. Slices
// were 9728 tokens, one workgroup of 512 threads on a compute unit with 19
// tokens a thread to evaluate and to read in every pass.
//
// Registers: the three walks are held to 128, so that two workgroups of eight
// waves share a compute unit; what does not fit goes to scratch (verify_walk 56
// bytes a lane for bf16, 40 to 44 for binary32; verify_pool_walk 12 to 20;
// verify_traversal none for bf16, 60 to 64 for binary32). Left to the compiler
// they take 160 to 168, 140, and 127 and 154, mostly one workgroup a compute
// unit: verify_walk over 16 requests of 151936 tokens 78 -> 90 to 102 us (three
// inputs), over 64 254 to 290 -> 344 to 395, the pool walk over 16 58 -> 88; one
// request alone, whose workgroups all run at once either way, 29.1 -> 27.5.
constexpr int kWalkThreads = kWalkThreadsPerGroup;
constexpr int kWalkWaves = kWalkThreads / kWave;
constexpr int kWalkPass = 4 * kWalkThreads;  // tokens of one group per thread

template <int DT>
__device__ __forceinline__ void load4_scaled(const void* base, size_t off, int valid, bool vec, float invT,
                                             float a[4]) {
    float x[4];
    load4<DT>(base, off, valid, vec, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = e < valid ? x[e] * invT : -INFINITY;
}

struct WalkSlice {
    int v0, v1;
    int groups;  // groups of four tokens in a whole slice
    bool held;   // (p~, q) fit the LDS
};
__device__ __forceinline__ WalkSlice walk_slice(int V, int g, int G) {
    // start a multiple of 4; an empty slice is [0, 0)
    const int span = walk_span(V, G);
    const bool has = (long long)g * span < V;
    WalkSlice S;
    S.v0 = has ? g * span : 0;
    S.v1 = has ? min(V, S.v0 + span) : 0;
    S.groups = span / 4;
    S.held = span <= kWalkHeldTokens;  // the same for every workgroup of the request
    return S;
}

// The thread's index as a value the compiler takes for new each time: what a
// pass derives from it (addresses, bounds, first random rounds) is recomputed
// there instead of being kept in registers, or spilled, over the whole walk.
__device__ __forceinline__ int pass_tid() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
// The thread's first kWalkRaw groups of one row as loaded; the logits of later
// groups (slices above 4096 tokens have them) are read where they are used.
constexpr int kWalkRaw = 2;
template <int DT>
struct RawRow {
    Raw4<DT> g[kWalkRaw];
    __device__ __forceinline__ void load(const void* base, bool vec, const WalkSlice& S, size_t row) {
        const int n = S.v1 - S.v0, tid = pass_tid();
#pragma unroll
        for (int k = 0; k < kWalkRaw; ++k) {
            const int i = k * kWalkPass + tid * 4;
            const int valid = max(0, min(4, n - i));
            raw_load4<DT>(base, row + S.v0 + (valid ? i : 0), valid, vec, g[k]);
        }
    }
};
// Tokens of a thread's k-th group inside the slice (0 to 4).
__device__ __forceinline__ int group_valid(const WalkSlice& S, int k, int tid) {
    return max(0, min(4, S.v1 - S.v0 - k * kWalkPass - tid * 4));
}
// f(k, logits x scale of one row) for every group of the thread in the slice,
// and f(k, target logits, draft logits). Compile-time k where the logits are
// held (an index at run time would put them into scratch memory).
template <int DT, typename F>
__device__ __forceinline__ void row_groups(const void* base, bool vec, const WalkSlice& S, size_t row,
                                           const RawRow<DT>& t, float scale, F f) {
    const int tid = pass_tid();
#pragma unroll
    for (int k = 0; k < kWalkRaw; ++k) {
        const int valid = group_valid(S, k, tid);
        if (valid > 0) {
            float a[4];
            raw_scaled4<DT>(t.g[k], valid, scale, a);
            f(k, tid, a);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll 1
    for (int k = kWalkRaw; group_valid(S, k, tid) > 0; ++k) {
        float a[4];
        load4_scaled<DT>(base, row + S.v0 + k * kWalkPass + tid * 4, group_valid(S, k, tid), vec, scale, a);
        f(k, tid, a);
    }
}
template <int DT, typename F>
__device__ __forceinline__ void row_pair_groups(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow,
                                                size_t drow, const RawRow<DT>& t, const RawRow<DT>& d, F f) {
    const int tid = pass_tid();
#pragma unroll
    for (int k = 0; k < kWalkRaw; ++k) {
        const int valid = group_valid(S, k, tid);
        if (valid > 0) {
            float at[4], ad[4];
            raw_scaled4<DT>(t.g[k], valid, A.invT, at);
            raw_scaled4<DT>(d.g[k], valid, A.invT, ad);
            f(k, tid, at, ad);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll 1
    for (int k = kWalkRaw; group_valid(S, k, tid) > 0; ++k) {
        float at[4], ad[4];
        const size_t o = S.v0 + (size_t)k * kWalkPass + tid * 4;
        load4_scaled<DT>(A.target, trow + o, group_valid(S, k, tid), vec, A.invT, at);
        load4_scaled<DT>(A.draft, drow + o, group_valid(S, k, tid), vec, A.invT, ad);
        f(k, tid, at, ad);
    }
}
// Groups of this thread in the slice.
__device__ __forceinline__ int slice_groups(const WalkSlice& S, int tid) {
    return max(0, (S.v1 - S.v0 - tid * 4 + kWalkPass - 1) / kWalkPass);
}

__device__ __forceinline__ double exp_or_0(float a, double L, const double* et) {
    return a > -INFINITY ? exp64((double)a - L, et) : 0.0;
}

// (p~, q) of the thread's tokens in LDS (0 past the slice): token e of group
// i at e * groups + i, so that a wave's accesses are to consecutive words.
struct HeldPQ {
    double* lds;
    int groups;
    __device__ __forceinline__ double& p(int k, int e, int tid) const { return lds[e * groups + k * kWalkThreads + tid]; }
    __device__ __forceinline__ double& q(int k, int e, int tid) const {
        return lds[(4 + e) * groups + k * kWalkThreads + tid];
    }
    // Evaluates them, calling f(p~, q) for each token.
    template <int DT, typename F>
    __device__ __forceinline__ void fill(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow, size_t drow,
                                         const RawRow<DT>& t, const RawRow<DT>& d, double L0, double Ld,
                                         const double* et, F f) const {
        row_pair_groups<DT>(A, vec, S, trow, drow, t, d, [&](int k, int tid, const float(&at)[4], const float(&ad)[4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double pt = exp_or_0(at[e], L0, et), qd = exp_or_0(ad[e], Ld, et);
                p(k, e, tid) = pt;
                q(k, e, tid) = qd;
                if (e & 1) __builtin_amdgcn_sched_barrier(0);  // four exponentials in flight
                f(pt, qd);
            }
        });
    }
    // sum over the thread's tokens of max(a p~ - c q, 0)
    __device__ __forceinline__ double residual(const WalkSlice& S, double a, double c) const {
        const int tid = pass_tid(), ng = slice_groups(S, tid);
        double z = 0.0;
#pragma unroll 1
        for (int k = 0; k < ng; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double rr = p(k, e, tid) * a - c * q(k, e, tid);
                z += rr > 0.0 ? rr : 0.0;
            }
        return z;
    }
};

// Token-wise visit of (p~, q) over a slice that is not held, recomputed:
// f(token, p~, q).
template <int DT, typename F>
__device__ __forceinline__ void visit_pq(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow, size_t drow,
                                         double L0, double Ld, const double* et, F f) {
    const int n = S.v1 - S.v0;
    for (int i = pass_tid() * 4; i < n; i += kWalkPass) {
        const int valid = min(4, n - i);
        float at[4], ad[4];
        load4_scaled<DT>(A.target, trow + S.v0 + i, valid, vec, A.invT, at);
        load4_scaled<DT>(A.draft, drow + S.v0 + i, valid, vec, A.invT, ad);
        for (int e = 0; e < valid; ++e) f(S.v0 + i + e, exp_or_0(at[e], L0, et), exp_or_0(ad[e], Ld, et));
    }
}

// A Gumbel-max candidate of the thread: largest key, its smallest token.
struct BestKey {
    float k = -INFINITY;
    int v = 0x7FFFFFFF;
    __device__ __forceinline__ void offer(float key, int tok) {
        if (key > k || (key == k && tok < v)) {
            k = key;
            v = tok;
        }
    }
    // as one ordered word: key descending, then token ascending
    __device__ __forceinline__ uint64_t packed() const {
        return ((uint64_t)ordered_bits(k) << 32) | (uint32_t)~v;
    }
};

// Bonus sample from p_u alone (leaf, or empty residual): argmax ln p_v + G_v
// over the slice.
template <int DT>
__device__ __forceinline__ BestKey bonus_from_p(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow,
                                                const RawRow<DT>& t, double Lt, const RngKey& key, uint32_t node) {
    BestKey b;
    const SplitF Ls = split(Lt);
    row_groups<DT>(A.target, vec, S, trow, t, A.invT, [&](int k, int tid, const float(&at)[4]) {
        const int v = S.v0 + k * kWalkPass + tid * 4;
        const uint4 w = rng_block(key, node, kStreamBonus, (uint32_t)(v >> 2));
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (at[e] > -INFINITY) b.offer(((at[e] - Ls.hi) - Ls.lo) + gumbel_f32(ws[e]), v + e);
    });
    return b;
}

// Gumbel-max of ln max(a p~ - c q, 0) over the slice, and the thread's part of
// the residual's mass.
template <int DT>
__device__ __forceinline__ BestKey bonus_residual(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow,
                                                  size_t drow, const HeldPQ& pq, double L0, double Ld, double a,
                                                  double c, const double* et, const RngKey& key, uint32_t node,
                                                  double& mass) {
    BestKey b;
    mass = 0.0;
    if (S.held) {
        const int tid = pass_tid(), ng = slice_groups(S, tid);
#pragma unroll 1
        for (int k = 0; k < ng; ++k) {
            const int v = S.v0 + k * kWalkPass + tid * 4;
            const uint4 w = rng_block(key, node, kStreamBonus, (uint32_t)(v >> 2));
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double rr = pq.p(k, e, tid) * a - c * pq.q(k, e, tid);
                if (rr > 0.0) {
                    mass += rr;
                    b.offer(logf((float)rr) + gumbel_f32(ws[e]), v + e);
                }
            }
        }
    } else {
        visit_pq<DT>(A, vec, S, trow, drow, L0, Ld, et, [&](int v, double p, double q) {
            const double rr = p * a - c * q;
            if (rr > 0.0) {
                mass += rr;
                b.offer(logf((float)rr) + gumbel_f32(rng_word(key, node, kStreamBonus, (uint32_t)v)), v);
            }
        });
    }
    return b;
}

// Block reductions and exchanges among the G workgroups of a request in one:
// the waves' parts meet in LDS, wave 0 adds them, publishes up to four words
// into the workgroup's slot (one lane a word, one store instruction), polls
// the slots of all G workgroups (lane l: word l % 4 of slot l / 4 and of every
// 16th slot after it, the loads of four such sets in flight together) and
// hands the result back through LDS: two barriers a round, the LDS buffers
// double-buffered by the round's parity. Everyone gets the same bits: sums are
// added in a fixed order. Partials travel with 2^-44 relative resolution.
// Among 16 workgroups a round takes 1.3 us (1.9 with a thread storing all
// words and a lane loading each slot's words in turn), among 38 about 1.7.
// One workgroup alone exchanges nothing.
constexpr int kExVals = 4;
constexpr int kExSets = 4;                       // slot sets in flight
constexpr int kExPer = kWave / kExVals;          // slots a set covers

// Wave sum through DPP row shifts and broadcasts; the total is in lane 63.
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_add_step(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWMASK, 0xf, true);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWMASK, 0xf, true);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum_last(double v) {
    v = dpp_add_step<0x111, 0xF>(v);  // row_shr:1
    v = dpp_add_step<0x112, 0xF>(v);  // row_shr:2
    v = dpp_add_step<0x114, 0xF>(v);  // row_shr:4
    v = dpp_add_step<0x118, 0xF>(v);  // row_shr:8
    v = dpp_add_step<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add_step<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ double xor_f64(double v, int j) {
    return __longlong_as_double((long long)shfl_xor_u64((uint64_t)__double_as_longlong(v), j));
}
// the value of lane Q of the lane's quad
template <int Q>
__device__ __forceinline__ uint64_t quad_u64(uint64_t v) {
    constexpr int c = Q * 0x55;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), c, 0xF, 0xF, true);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, c, 0xF, 0xF, true);
    return ((uint64_t)hi << 32) | lo;
}

struct Exchange {
    const WalkArgs* A;
    int r, g, G;
    uint32_t nb;  // rounds run
    int timeout;

    // Wave 0: lanes 0 to 3 publish their word, then f(set base, q) gets the
    // words of 64 slots at a time: q[c] holds word lane % 4 of slot
    // base + 16 c + lane / 4 (0 past G). Returns whether a wait was abandoned.
    template <typename F>
    __device__ __forceinline__ int round(uint64_t mine, F f) {
        const int lane = threadIdx.x;
        if (G == 1) {
            uint64_t q[kExSets] = {lane < kExVals ? mine & ~kTagMask : 0ull, 0ull, 0ull, 0ull};
            f(0, q);
            return 0;
        }
        const uint64_t t = xtag(nb);
        uint64_t* const s = xslot(A->X, r, nb, 0);
        if (lane < kExVals)
            __hip_atomic_store(&s[(size_t)g * kSlotWords + lane], (mine & ~kTagMask) | t, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        int to = 0;
        for (int b = 0; b < G; b += kExSets * kExPer) {
            uint64_t q[kExSets];
            for (uint32_t spins = 0;; ++spins) {
                bool ok = true;
#pragma unroll
                for (int c = 0; c < kExSets; ++c) {
                    const int h = b + c * kExPer + lane / kExVals;
                    q[c] = t;
                    if (h < G)
                        q[c] = __hip_atomic_load(&s[(size_t)h * kSlotWords + lane % kExVals], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int c = 0; c < kExSets; ++c) ok = ok && (q[c] & kTagMask) == t;
                if (__ballot(!ok) == 0ull) break;
                if (spins >= kPollLimit) {
                    to = 1;
                    break;
                }
            }
#pragma unroll
            for (int c = 0; c < kExSets; ++c) q[c] = b + c * kExPer + lane / kExVals < G ? q[c] & ~kTagMask : 0ull;
            f(b, q);
        }
        return to;
    }

    // v[k]: the thread's parts in, the request's sums out.
    template <int NV>
    __device__ __forceinline__ void sum(double (&v)[NV]) {
        static_assert(NV <= kExVals && kWalkWaves * kExVals <= kWave, "exchange width");
        __shared__ double s_red[2][kExVals][kWalkWaves];
        __shared__ double s_tot[2][kExVals];
        __shared__ int s_to[2];
        const int par = (int)(nb & 1u), lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = wave_sum_last(v[k]);
        if (lane == kWave - 1)
#pragma unroll
            for (int k = 0; k < NV; ++k) s_red[par][k][wave] = v[k];
        __syncthreads();
        if (wave == 0) {
            double x = lane < NV * kWalkWaves ? s_red[par][lane / kWalkWaves][lane % kWalkWaves] : 0.0;
#pragma unroll
            for (int j = 1; j < kWalkWaves; j <<= 1) x += xor_f64(x, j);
            const double mine = __shfl(x, (lane % kExVals) * kWalkWaves, kWave);
            double tot = 0.0;
            const int to = round((uint64_t)__double_as_longlong(mine), [&](int, const uint64_t(&q)[kExSets]) {
#pragma unroll
                for (int c = 0; c < kExSets; ++c) tot += __longlong_as_double((long long)q[c]);
            });
#pragma unroll
            for (int j = kExVals; j < kWave; j <<= 1) tot += xor_f64(tot, j);
            if (lane < kExVals) s_tot[par][lane] = tot;
            if (lane == 0) s_to[par] = to;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = s_tot[par][k];
        if (s_to[par]) timeout = 1;
        ++nb;
    }

    // The request's best key's token (-1: none), and the sum of `part`.
    __device__ __forceinline__ int best(const BestKey& b, double part, double* total) {
        __shared__ uint64_t s_key[2][kWalkWaves];
        __shared__ double s_red[2][kWalkWaves];
        __shared__ double s_tot[2];
        __shared__ uint64_t s_best[2];
        __shared__ int s_to[2];
        const int par = (int)(nb & 1u), lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
        const uint64_t wk = wave_max_u64(b.packed());
        const double ws = wave_sum_last(part);
        if (lane == kWave - 1) {
            s_key[par][wave] = wk;
            s_red[par][wave] = ws;
        }
        __syncthreads();
        if (wave == 0) {
            uint64_t k = lane < kWalkWaves ? s_key[par][lane] : 0ull;
            double x = lane < kWalkWaves ? s_red[par][lane] : 0.0;
#pragma unroll
            for (int j = 1; j < kWalkWaves; j <<= 1) {
                const uint64_t o = shfl_xor_u64(k, j);
                k = o > k ? o : k;
                x += xor_f64(x, j);
            }
            k = lane_u64(k, 0);
            x = lane_f64(x, 0);
            // words: mass, key, token
            const uint64_t mine = lane == 0 ? (uint64_t)__double_as_longlong(x)
                                            : (lane == 1 ? (k >> 32) << 32 : (lane == 2 ? k << 32 : 0ull));
            uint64_t top = 0ull;
            double tot = 0.0;
            const int to = round(mine, [&](int, const uint64_t(&q)[kExSets]) {
#pragma unroll
                for (int c = 0; c < kExSets; ++c) {
                    const uint64_t kk = quad_u64<1>(q[c]) | (quad_u64<2>(q[c]) >> 32);
                    top = kk > top ? kk : top;
                    tot += __longlong_as_double((long long)quad_u64<0>(q[c]));
                }
            });
#pragma unroll
            for (int j = kExVals; j < kWave; j <<= 1) {
                const uint64_t o = shfl_xor_u64(top, j);
                top = o > top ? o : top;
                tot += xor_f64(tot, j);
            }
            if (lane == 0) {
                s_tot[par] = tot;
                s_best[par] = top;
                s_to[par] = to;
            }
        }
        __syncthreads();
        *total = s_tot[par];
        const uint64_t top = s_best[par];
        if (s_to[par]) timeout = 1;
        ++nb;
        // a key of -inf is no candidate
        return (uint32_t)(top >> 32) > ordered_bits(-INFINITY) ? (int)~(uint32_t)top : -1;
    }

    // Log-sum-exp of the request's row from the threads' parts (m the largest
    // raw logit, s = sum 2^((x - m) c), c = invT log2(e); nf: a NaN or +inf):
    // the largest maximum, then every sum rescaled to it and added in a fixed
    // order. *bad if a part is unusable, or if none holds a finite logit.
    __device__ __forceinline__ double lse(float m, double s, bool nf, float c, float invT, const double* s_exp,
                                          bool* bad) {
        __shared__ float s_m[2][kWalkWaves];
        __shared__ double s_s[2][kWalkWaves];
        __shared__ int s_nf[2][kWalkWaves];
        __shared__ double s_l[2];
        __shared__ int s_b[2], s_to[2];
        const int par = (int)(nb & 1u), lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
        const float wm = wave_max(m);
        const double ws = wave_sum_last(m == -INFINITY ? 0.0 : (m == wm ? s : s * (double)exp2f((m - wm) * c)));
        const bool wnf = __ballot(nf) != 0ull;
        if (lane == kWave - 1) {
            s_m[par][wave] = wm;
            s_s[par][wave] = ws;
            s_nf[par][wave] = wnf ? 1 : 0;
        }
        __syncthreads();
        if (wave == 0) {
            float M = -INFINITY;
            bool pb = false;
            for (int w = 0; w < kWalkWaves; ++w) {
                M = fmaxf(M, s_m[par][w]);
                pb = pb || s_nf[par][w] != 0;
            }
            double x = 0.0;
            if (lane < kWalkWaves && M > -INFINITY && M < INFINITY && s_m[par][lane] > -INFINITY)
                x = s_s[par][lane] * (double)exp2f((s_m[par][lane] - M) * c);
#pragma unroll
            for (int j = 1; j < kWalkWaves; j <<= 1) x += xor_f64(x, j);
            x = lane_f64(x, 0);
            pb = pb || M == INFINITY || !isfinite(x);
            const double mx = M > -INFINITY && !pb ? (double)(M * invT) : -INFINITY;
            const double sx = pb ? 0.0 : x;
            // words: maximum, sum, flag
            const uint64_t mine = lane == 0 ? (uint64_t)__double_as_longlong(mx)
                                            : (lane == 1 ? (uint64_t)__double_as_longlong(sx)
                                                         : (lane == 2 ? xpack_u32(pb ? 1u : 0u) : 0ull));
            double T = 0.0, top = -INFINITY;  // running sum and its reference
            int b = 0;
            const int to = round(mine, [&](int base, const uint64_t(&q)[kExSets]) {
                double hm[kExSets], M2 = top;
#pragma unroll
                for (int c4 = 0; c4 < kExSets; ++c4) {
                    hm[c4] = base + c4 * kExPer + lane / kExVals < G
                                 ? __longlong_as_double((long long)quad_u64<0>(q[c4]))
                                 : -INFINITY;
                    b |= quad_u64<2>(q[c4]) != 0ull ? 1 : 0;
                    M2 = fmax(M2, hm[c4]);
                }
#pragma unroll
                for (int j = kExVals; j < kWave; j <<= 1) M2 = fmax(M2, xor_f64(M2, j));
                double t = 0.0;
#pragma unroll
                for (int c4 = 0; c4 < kExSets; ++c4)
                    if (hm[c4] > -INFINITY)
                        t += __longlong_as_double((long long)quad_u64<1>(q[c4])) * exp64x(hm[c4] - M2, s_exp);
#pragma unroll
                for (int j = kExVals; j < kWave; j <<= 1) t += xor_f64(t, j);
                T = (top > -INFINITY ? T * exp64x(top - M2, s_exp) : 0.0) + t;
                top = M2;
            });
            const bool anyb = __ballot(b) != 0ull;
            if (lane == 0) {
                const bool none = !(top > -INFINITY) || !(T > 0.0);
                s_l[par] = none ? 0.0 : top + log64(T, s_exp);
                s_b[par] = anyb || none || !isfinite(top) || !isfinite(T);
                s_to[par] = to;
            }
        }
        __syncthreads();
        const double L = s_l[par];
        *bad = s_b[par] != 0;
        if (s_to[par]) timeout = 1;
        ++nb;
        return L;
    }
};

// Streamed normaliser of the target row of the node the walk enters (the
// walk reads a target row only when it enters its node): every thread's
// running maximum of the raw logits and binary32 terms 2^(x c - m c) added in
// binary64, as the target stream does, then one exchange. Within ~1e-6 of ln
// sum_v exp(a_v); *bad if the row holds a NaN or +inf logit, or no finite one.
struct RowPart {
    float m = -INFINITY;
    double sum = 0.0;
    bool nf = false;
    __device__ __forceinline__ void add(const float (&x)[4], float c) {
        float cm = m;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            nf |= __builtin_amdgcn_classf(x[e], 0x203);  // signalling NaN, quiet NaN, +inf
            cm = fmaxf(cm, x[e]);                        // NaN is ignored
        }
        if (cm > m) {
            if (m > -INFINITY) sum *= (double)exp2f((m - cm) * c);
            m = cm;
        }
        if (m > -INFINITY && m < INFINITY) {
            const float mc = m * c;
            float cs = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) cs += __builtin_amdgcn_exp2f(fmaf(x[e], c, -mc));
            sum += (double)cs;
        }
    }
};

template <int DT>
__device__ __forceinline__ double entered_row_lse(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow,
                                                  const RawRow<DT>& t, Exchange& X, const double* et,
                                                  bool* bad) {
    const float c = A.invT * 1.4426950408889634f;
    RowPart p;
    row_groups<DT>(A.target, vec, S, trow, t, 1.0f, [&](int, int, const float(&x)[4]) { p.add(x, c); });
    return X.lse(p.m, p.sum, p.nf, c, A.invT, et, bad);
}

// Relative half-width of the band in which an acceptance test taken with the
// streamed normaliser is recomputed with the exact one (the streamed
// normaliser is within ~1e-6 of it: binary32 terms, binary64 accumulation).
constexpr double kDecisionBand = 1e-4;

// First exact pass at a node: the thread's parts of sum p~, and, for the
// first residual (C = 1), of sum p~ and sum q over tokens with p~ > q (beyond
// the band where the normaliser could flip the sign) and the number of tokens
// inside that band.
struct FirstPass {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    __device__ __forceinline__ void add(double pt, double qd) {
        v[0] += pt;
        if (pt > qd * (1.0 + 1e-5)) {
            v[1] += pt;
            v[2] += qd;
        } else if (pt >= qd * (1.0 - 1e-5) && pt > 0.0) {
            v[3] += 1.0;
        }
    }
};

// End of a walk: the request's outputs, and the optional normaliser output
// (from the target stream's partials, which the caller streamed when it asked
// for it), both by the request's first workgroup: another one may start only
// after this one has ended a walk without an exchange (an unusable root row),
// and would take the status written here for the planner's. rows_bad < 0:
// every target row of the tree must be usable (from the partials); otherwise
// rows_bad is the walk's own verdict on the rows it entered.
__device__ __forceinline__ void walk_tail(const WalkArgs& A, int r, int g, int n, bool draft_bad, bool invalid, int nacc,
                          int bonus_out, int add_status, int tcount, int rows_bad = -1) {
    if (g != 0 && !A.out.target_lse) return;  // uniform over the workgroup
    __shared__ int s_bad;
    const int tid = threadIdx.x;
    const int B1 = A.B + 1;
    const size_t tb = (size_t)r * B1;
    int* status_p = A.out.req_status + r;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    if (!draft_bad && rows_bad < 0)
        for (int i = tid; i < n; i += kWalkThreads)
            if (target_row_bad(A.tm, A.tf, A.S4, tb + i)) atomicOr(&s_bad, 1);
    __syncthreads();
    const bool bad = draft_bad || (rows_bad < 0 ? s_bad != 0 : rows_bad != 0);
    if (A.out.target_lse) {
        // a request rejected by a verifier that reads every row reports no normaliser
        const bool none = draft_bad || (bad && rows_bad < 0);
        // (g past 0 starts beyond the last row; a branch on g, here or above, costs
        // verify_walk scratch and 0.3 to 0.8% of its time)
        for (int i = g * (TSB_MAX_B + 1) + tid; i < B1; i += kWalkThreads) {
            double l = (double)NAN;
            if (!none && i < n) {
                int b;
                l = target_lse(A, r, i, &b);
                if (b) l = (double)NAN;
            }
            A.out.target_lse[tb + i] = l;
        }
    }
    if (g == 0 && tid == 0) {
        if (bad) {
            nacc = 0;
            bonus_out = -1;
            add_status = (add_status & ~(TSB_REQ_DEGENERATE_RESIDUAL | TSB_REQ_WALK_TIMEOUT)) | TSB_REQ_NONFINITE;
        } else if (invalid) {  // a malformed tree or token: outputs defined, without meaning
            nacc = 0;
            bonus_out = -1;
        }
        for (int i = nacc; i < A.D; ++i) {
            A.out.acc_node[(size_t)r * A.D + i] = -1;
            A.out.acc_tok[(size_t)r * A.D + i] = -1;
        }
        A.out.n_acc[r] = (bad || invalid) ? -1 : nacc;
        A.out.bonus[r] = bonus_out;
        *status_p |= add_status;
        if (A.out.trace)
            for (int i = tcount; i < TSB_TRACE_MAX; ++i)
                for (int f = 0; f < 4; ++f) A.out.trace[((size_t)r * TSB_TRACE_MAX + i) * 4 + f] = -1.0;
    }
}

// What a walk knows of a node it enters: its topology checks, normalisers and
// children, one child per lane (every wave loads them for itself).
struct Entered {
    TreeNode t;
    double L0, Ld;     // streamed target normaliser (where known), draft normaliser of the children's row
    bool l0, row_bad;  // L0 and row_bad are known
    int tok;           // child lane's token, and its draft and target logits x invT
    float xd, xt;
    int kids;          // child lane's own child count (traversal)
};

// Values that are the same in every lane, moved to scalar registers (the walks
// keep about thirty of them, which would take half of a thread's vector
// registers).
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ double uni(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ Entered enter_record(const uint32_t* nrec, size_t node, int lane) {
    const uint32_t* rp = nrec + node * kRecWords;
    const uint4 h0 = *(const uint4*)rp;
    const uint4 h1 = *(const uint4*)(rp + 4);
    const uint4 c = lane < TSB_MAX_K ? *(const uint4*)(rp + 8 + 4 * lane) : make_uint4(0u, 0u, 0u, 0u);
    Entered e;
    const int flags = uni((int)h0.w);
    e.t.m = uni((int)h0.x);
    e.t.fc = uni((int)h0.y);
    e.t.d = uni((int)h0.z);
    e.t.ok = (flags & (int)kRecOk) != 0;
    e.row_bad = (flags & (int)kRecTargetBad) != 0;
    e.l0 = (flags & (int)kRecNoL0) == 0;
    e.L0 = uni(rec_f64(h1.x, h1.y));
    e.Ld = uni(rec_f64(h1.z, h1.w));
    e.tok = (int)c.x;
    e.xd = __uint_as_float(c.y);
    e.xt = __uint_as_float(c.z);
    e.kids = (int)c.w;
    return e;
}

template <int DT, bool VEC>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(4))) void verify_walk(WalkArgs A) {
    extern __shared__ double s_pq[];  // (p~, q) of the slice
    __shared__ double s_exp[kExpTable];
    const int G = A.G;
    const int ticket = xticket(A.X, A.R);
    const int g = ticket % G;
    const int r = ticket / G;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int B1 = A.B + 1;
    const size_t tb = (size_t)r * B1;
    const bool vec = VEC;
    int* status_p = A.out.req_status + r;
    const int n_raw = A.tree.n_nodes[r];
    const bool count_ok = tree_count_ok(n_raw, A.B);
    const int n = count_ok ? n_raw : 0;
    const bool lead = (g == 0 && tid == 0);
    exp64_table_init(s_exp);

    const WalkSlice S = walk_slice(A.V, g, G);
    const HeldPQ pq{s_pq, S.groups};
    const bool draft_bad = (*status_p & TSB_REQ_NONFINITE) != 0;

    int tcount = 0;
    int n_entered = 0;  // nodes entered (work counter)
    double* const trace = (lead && A.out.trace) ? A.out.trace + (size_t)r * TSB_TRACE_MAX * 4 : nullptr;

    int bonus_out = -1, add_status = count_ok ? 0 : TSB_REQ_BAD_TREE, nacc = 0;
    bool invalid = !count_ok;
    int rows_bad = 0;  // an entered node's target row is unusable
    if (!draft_bad && count_ok) {
        RngKey key;
        key.k0 = A.k0;
        key.k1 = A.k1;
        key.request = (uint32_t)r;
        key.step = A.step;
        Exchange X{&A, r, g, G, 0u, 0};
        int u = 0;
        bool from_p = false;  // the round ends with a bonus from p_u, normaliser from_L
        double from_L = 0.0;
        RawRow<DT> rt, rd;    // u's rows
        while (true) {
            ++n_entered;
            const size_t trow = ((size_t)r * B1 + u) * (size_t)A.V;
            // every workgroup reads the same entries, so all take the same exit
            Entered N = enter_record(A.nrec, tb + u, lane);
            if (!N.t.ok || (N.t.m > 0 && nacc >= A.D)) {
                add_status |= TSB_REQ_BAD_TREE;
                invalid = true;
                break;
            }
            const int m = N.t.m, fc = N.t.fc;
            const size_t drow = ((size_t)r * A.D + (m > 0 ? N.t.d : 0)) * (size_t)A.V;
            // the rows' slices are in flight while the children's probabilities
            // and, where it is known, the normaliser are worked out
            rt.load(A.target, vec, S, trow);
            if (m > 0) rd.load(A.draft, vec, S, drow);
            // the streamed normaliser of u's row, and whether the row is usable
            if (A.reads_rows) {
                if (u < kChainRows) {  // the root or node 1: streamed before the walk
                    int tbad;
                    N.L0 = target_row_lse(A.cm, A.cs, A.cf, kChainPieces, (size_t)r * kChainRows + u, &tbad);
                    N.row_bad = tbad != 0;
                } else {
                    N.L0 = entered_row_lse<DT>(A, vec, S, trow, rt, X, s_exp, &N.row_bad);
                }
            } else if (!N.l0) {
                int tbad;
                N.L0 = target_lse(A, r, u, &tbad);
                N.row_bad = tbad != 0;
            }
            if (N.row_bad) {
                rows_bad = 1;
                break;
            }
            const double L0 = uni(N.L0), Ld = N.Ld;
            if (m == 0) {  // accepted leaf: bonus from p_u
                from_p = true;
                from_L = L0;
                break;
            }
            // lane j: child j's uniform and probabilities; a token outside
            // [0, V) is never used as an address
            if (__ballot(lane < m && !(N.tok >= 0 && N.tok < A.V))) {
                add_status |= TSB_REQ_BAD_TOKEN;
                invalid = true;
                break;
            }
            const double ul = u24d(rng_word(key, (uint32_t)(fc + lane), kStreamAccept, 0u));
            const double ql = exp64x((double)N.xd - Ld, s_exp);
            double pl = exp64x((double)N.xt - L0, s_exp);

            bool exact = false;
            double Lt = L0, inv = 1.0;
            double C = 0.0, Sq = 1.0, Z = 1.0, Z1 = -1.0;
            bool accepted = false, degenerate = false;
            for (int j = 0; j < m; ++j) {
                const int c = fc + j;
                const double qy = lane_f64(ql, j);
                const double U = lane_f64(ul, j);
                const double W = uni(Z / Sq);
                double num = lane_f64(pl, j) - C * qy;
                double ratio = (num > 0.0 ? num : 0.0) / (W * qy);
                if (trace && tcount < TSB_TRACE_MAX) {
                    trace[tcount * 4 + 0] = c;
                    trace[tcount * 4 + 1] = U;
                    trace[tcount * 4 + 3] = -1.0;
                }
                ++tcount;
                // Before the exact pass only the first test of a node is taken, with
                // the streamed normaliser; it stands if U is clear of the ratio by
                // the band. A rejection needs the exact residual anyway.
                if (!exact && (fabs(U - ratio) <= kDecisionBand * ratio || !(U < ratio))) {
                    FirstPass f;
                    if (S.held)
                        pq.fill<DT>(A, vec, S, trow, drow, rt, rd, L0, Ld, s_exp, [&](double p, double q) { f.add(p, q); });
                    else
                        visit_pq<DT>(A, vec, S, trow, drow, L0, Ld, s_exp, [&](int, double p, double q) { f.add(p, q); });
                    X.sum<4>(f.v);
                    Lt = uni(L0 + log64(f.v[0], s_exp));
                    inv = uni(1.0 / f.v[0]);
                    // first residual (C = 1): sum over {p > q} of p - q, exact when no
                    // token lies in the band where the normaliser decides the sign
                    Z1 = uni(f.v[3] == 0.0 ? f.v[1] * inv - f.v[2] : -1.0);
                    exact = true;
                    pl = exp64x((double)N.xt - Lt, s_exp);
                    num = lane_f64(pl, j) - C * qy;
                    ratio = (num > 0.0 ? num : 0.0) / (W * qy);
                }
                if (trace && tcount <= TSB_TRACE_MAX) trace[(tcount - 1) * 4 + 2] = ratio;
                if (U < ratio) {
                    if (lead) {
                        A.out.acc_node[(size_t)r * A.D + nacc] = c;
                        A.out.acc_tok[(size_t)r * A.D + nacc] = (int)lane_u32((uint32_t)N.tok, j);
                    }
                    ++nacc;
                    u = c;
                    accepted = true;
                    break;
                }
                C = uni(C + W);
                Sq = uni(Sq - qy);
                if (j + 1 == m) break;
                // residual mass at the new C
                if (j == 0 && Z1 >= 0.0) {
                    Z = Z1;
                } else {
                    double zp[1] = {0.0};
                    if (S.held)
                        zp[0] = pq.residual(S, inv, C);
                    else
                        visit_pq<DT>(A, vec, S, trow, drow, L0, Ld, s_exp, [&](int, double p, double q) {
                            const double rr = p * inv - C * q;
                            zp[0] += rr > 0.0 ? rr : 0.0;
                        });
                    X.sum<1>(zp);
                    Z = uni(zp[0]);
                }
                if (trace && tcount <= TSB_TRACE_MAX) trace[(tcount - 1) * 4 + 3] = Z;
                if (Z <= 0.0 || Sq <= 0.0) {
                    degenerate = true;
                    break;
                }
            }
            if (accepted) continue;
            // every child rejected: bonus from the residual max(p - C q, 0)
            if (!degenerate) {
                double zp, mass;
                const BestKey b = bonus_residual<DT>(A, vec, S, trow, drow, pq, L0, Ld, inv, C, s_exp, key,
                                                     (uint32_t)u, zp);
                const int fi = X.best(b, zp, &mass);
                if (trace && tcount >= 1 && tcount <= TSB_TRACE_MAX) trace[(tcount - 1) * 4 + 3] = mass;
                if (mass > 0.0 && fi >= 0) {
                    bonus_out = fi;
                } else {
                    degenerate = true;
                }
            }
            if (degenerate) {  // empty residual: bonus from p_u
                from_p = true;
                from_L = Lt;
                add_status |= TSB_REQ_DEGENERATE_RESIDUAL;
            }
            break;
        }
        if (from_p) {
            const size_t trow = ((size_t)r * B1 + u) * (size_t)A.V;
            double unused;
            bonus_out = X.best(bonus_from_p<DT>(A, vec, S, trow, rt, from_L, key, (uint32_t)u), 0.0, &unused);
        }
        if (X.timeout) add_status |= TSB_REQ_WALK_TIMEOUT;
        if (A.stats && lead) {
            atomicAdd(&A.stats[kStWalkRequests], 1ull);
            atomicAdd(&A.stats[kStWalkNodes], (unsigned long long)n_entered);
            atomicAdd(&A.stats[kStWalkTests], (unsigned long long)tcount);
            atomicAdd(&A.stats[kStWalkExchanges], (unsigned long long)X.nb);
        }
    }

    walk_tail(A, r, g, n, draft_bad, invalid, nacc, bonus_out, add_status, tcount, rows_bad);
}


// ---------------------------------------------------------------- pool walk
// Verification with pool-restricted, context-dependent q_u (Section 3.1;
// Section 3.3: the probabilities of the replayed candidates, normalised in
// the pool). At node u (depth d, token in slot s_u of pool d - 1) wave 0
// rebuilds q_u over pool d from the draft logits and the transition scores,
// z_j = fl32(a_j + fl32(c[d-1][s_u][j] invT)), q_j = exp(z_j - L_u), and
// reads the target logits at the pool tokens. q vanishes off the pool, so
// after a rejection the residual mass needs no vocabulary pass:
//   Z = sum_{v off pool} p_v + sum_{v in pool} max(p_v - C q_v, 0)
//     = (S~ - sum_{pool} p~_v) / S~ + sum_{pool} max(p~_v / S~ - C q_v, 0)
// with p~_v = exp(a^t_v - L0) and S~ = sum_v p~_v from the one exact pass
// over the target row (L0 the streamed normaliser). The residual bonus is a
// Gumbel-max over the slice with the pool tokens left out (a bitmap of the
// slice in LDS), merged with the pool tokens' residual keys.

// Exact pass over the target row of the slice: the thread's part of the sum
// of exp(a^t_v - L0).
template <int DT>
__device__ __forceinline__ double target_pass(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow, double L0,
                                              const double* et) {
    double sp = 0.0;
    const int n = S.v1 - S.v0;
    int i = (int)threadIdx.x * 4;
    float at[4];
    {
        const int valid = max(0, min(4, n - i));
        load4_scaled<DT>(A.target, trow + S.v0 + (valid ? i : 0), valid, vec, A.invT, at);
    }
    for (; i < n; i += kWalkPass) {
        const int inext = i + kWalkPass;
        float nt[4];
        const int vn = max(0, min(4, n - inext));
        load4_scaled<DT>(A.target, trow + S.v0 + (vn ? inext : 0), vn, vec, A.invT, nt);
#pragma unroll
        for (int e = 0; e < 4; ++e) sp += exp_or_0(at[e], L0, et);
#pragma unroll
        for (int e = 0; e < 4; ++e) at[e] = nt[e];
    }
    return sp;
}

// Gumbel-max of ln p_v over the slice's tokens outside the pool.
template <int DT>
__device__ __forceinline__ BestKey bonus_off_pool(const WalkArgs& A, bool vec, const WalkSlice& S, size_t trow,
                                                  double Lt, const RngKey& key, uint32_t node, const uint32_t* bits) {
    BestKey b;
    const SplitF Ls = split(Lt);
    const int n = S.v1 - S.v0;
    for (int i = (int)threadIdx.x * 4; i < n; i += kWalkPass) {
        const int valid = min(4, n - i);
        float at[4];
        load4_scaled<DT>(A.target, trow + S.v0 + i, valid, vec, A.invT, at);
        const uint4 w = rng_block(key, node, kStreamBonus, (uint32_t)((S.v0 + i) >> 2));
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (e >= valid || at[e] == -INFINITY) continue;
            if ((bits[(i + e) >> 5] >> ((i + e) & 31)) & 1u) continue;  // a pool token
            b.offer(((at[e] - Ls.hi) - Ls.lo) + gumbel_f32(ws[e]), S.v0 + i + e);
        }
    }
    return b;
}

template <int DT, bool VEC>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(4))) void verify_pool_walk(WalkArgs A) {
    extern __shared__ uint32_t s_bits[];  // pool membership over the slice
    __shared__ double s_exp[kExpTable];
    __shared__ int s_ptok[kPoolMax];
    __shared__ double s_q[kPoolMax], s_pp[kPoolMax];
    __shared__ float s_pat[kPoolMax];
    __shared__ int s_tok[TSB_MAX_K], s_cslot[TSB_MAX_K];
    __shared__ float s_xt[TSB_MAX_K];
    __shared__ double s_u[TSB_MAX_K];
    __shared__ double s_z;
    __shared__ int s_badtok;
    const int G = A.G;
    const int ticket = xticket(A.X, A.R);
    const int g = ticket % G;
    const int r = ticket / G;
    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int B1 = A.B + 1;
    const int P = A.P;
    const size_t tb = (size_t)r * B1;
    const bool vec = VEC;
    const int n_raw = A.tree.n_nodes[r];
    const bool count_ok = tree_count_ok(n_raw, A.B);
    const int n = count_ok ? n_raw : 0;
    const bool lead = (g == 0 && tid == 0);
    exp64_table_init(s_exp);
    if (tid == 0) s_badtok = 0;

    const WalkSlice S = walk_slice(A.V, g, G);
    const int nwords = (S.v1 - S.v0 + 31) / 32;
    const bool draft_bad = (A.out.req_status[r] & TSB_REQ_NONFINITE) != 0;

    int tcount = 0;
    double* const trace = (lead && A.out.trace) ? A.out.trace + (size_t)r * TSB_TRACE_MAX * 4 : nullptr;

    int bonus_out = -1, add_status = count_ok ? 0 : TSB_REQ_BAD_TREE, nacc = 0;
    bool invalid = !count_ok;
    if (!draft_bad && count_ok) {
        RngKey key;
        key.k0 = A.k0;
        key.k1 = A.k1;
        key.request = (uint32_t)r;
        key.step = A.step;
        Exchange X{&A, r, g, G, 0u, 0};
        int u = 0, su = 0;
        while (true) {
            // every workgroup reads the same entries, so all take the same exit
            const TreeNode nd = tree_node(A.tree, tb, u, n, A.D);
            if (!nd.ok || (nd.m > 0 && nacc >= A.D)) {
                add_status |= TSB_REQ_BAD_TREE;
                invalid = true;
                break;
            }
            const int m = nd.m, d = nd.d;
            const size_t trow = ((size_t)r * B1 + u) * (size_t)A.V;
            int tbad;
            const double L0 = target_lse(A, r, u, &tbad);
            if (m == 0) {  // accepted leaf: bonus from p_u
                double unused;
                RawRow<DT> rt;
                rt.load(A.target, vec, S, trow);
                bonus_out = X.best(bonus_from_p<DT>(A, vec, S, trow, rt, L0, key, (uint32_t)u), 0.0, &unused);
                break;
            }
            // q_u over pool d, target logits at the pool tokens
            if (tid < kWave) {
                float z = -INFINITY, at = -INFINITY;
                int tok = -1;
                if (lane < P) {
                    tok = A.pool_tok[((size_t)r * A.D + d) * P + lane];
                    if (tok >= 0 && tok < A.V) {
                        z = load_logit<DT>(A.draft, ((size_t)r * A.D + d) * A.V + tok) * A.invT;
                        if (d > 0) {
                            const float c = A.trans[(((size_t)r * (A.D - 1) + (d - 1)) * P + su) * (size_t)P + lane];
                            const float cs = c * A.invT;
                            z = z + cs;
                        }
                        at = load_logit<DT>(A.target, trow + tok) * A.invT;
                    }
                }
                const float zm = wave_max(z);
                double q = 0.0;
                if (zm > -INFINITY) {
                    const double e = z > -INFINITY ? exp64((double)z - (double)zm, s_exp) : 0.0;
                    const double Lz = (double)zm + log64(wave_sum(e), s_exp);
                    q = z > -INFINITY ? exp64((double)z - Lz, s_exp) : 0.0;
                }
                if (lane < P) {
                    s_ptok[lane] = tok;
                    s_q[lane] = q;
                    s_pat[lane] = at;
                }
            }
            const int fc = nd.fc;
            if (tid < m) {
                const int y = A.node_tok[tb + fc + tid];
                s_tok[tid] = y;
                s_xt[tid] = (y >= 0 && y < A.V) ? load_logit<DT>(A.target, trow + y) * A.invT : -INFINITY;
                s_u[tid] = u24d(rng_word(key, (uint32_t)(fc + tid), kStreamAccept, 0u));
            }
            __syncthreads();
            if (tid < m) {  // pool slot of each child's token
                const int y = s_tok[tid];
                int sl = -1;
                for (int j = 0; j < P; ++j)
                    if (s_ptok[j] == y) {
                        sl = j;
                        break;
                    }
                s_cslot[tid] = sl;
                if (sl < 0) s_badtok = 1;
            }
            __syncthreads();

            bool exact = false;
            double Lt = L0, inv = 1.0, Stot = 1.0;
            double C = 0.0, Sq = 1.0, Z = 1.0;
            bool accepted = false, degenerate = false;
            for (int j = 0; j < m; ++j) {
                const int c = fc + j;
                const int y = s_tok[j];
                const int sl = s_cslot[j];
                const double qy = sl >= 0 ? s_q[sl] : 0.0;
                const double U = s_u[j];
                const double W = Z / Sq;
                double py = s_xt[j] > -INFINITY ? exp64x((double)s_xt[j] - Lt, s_exp) : 0.0;
                double num = py - C * qy;
                double ratio = qy > 0.0 ? (num > 0.0 ? num : 0.0) / (W * qy) : (py > 0.0 ? INFINITY : 0.0);
                if (trace && tcount < TSB_TRACE_MAX) {
                    trace[tcount * 4 + 0] = c;
                    trace[tcount * 4 + 1] = U;
                    trace[tcount * 4 + 3] = -1.0;
                }
                ++tcount;
                if (!exact && (fabs(U - ratio) <= kDecisionBand * ratio || !(U < ratio))) {
                    double sp[1] = {target_pass<DT>(A, vec, S, trow, L0, s_exp)};
                    X.sum<1>(sp);
                    Stot = sp[0];
                    Lt = L0 + log64(Stot, s_exp);
                    inv = 1.0 / Stot;
                    exact = true;
                    // pool probabilities p~_v with the same exponential as the pass
                    if (tid < kWave) {
                        const double pp = lane < P && s_pat[lane] > -INFINITY ? exp64((double)s_pat[lane] - L0, s_exp)
                                                                              : 0.0;
                        if (lane < P) s_pp[lane] = pp;
                    }
                    __syncthreads();
                    py = s_xt[j] > -INFINITY ? exp64x((double)s_xt[j] - Lt, s_exp) : 0.0;
                    num = py - C * qy;
                    ratio = qy > 0.0 ? (num > 0.0 ? num : 0.0) / (W * qy) : (py > 0.0 ? INFINITY : 0.0);
                }
                if (trace && tcount <= TSB_TRACE_MAX) trace[(tcount - 1) * 4 + 2] = ratio;
                if (U < ratio) {
                    if (lead) {
                        A.out.acc_node[(size_t)r * A.D + nacc] = c;
                        A.out.acc_tok[(size_t)r * A.D + nacc] = y;
                    }
                    ++nacc;
                    u = c;
                    su = sl >= 0 ? sl : 0;
                    accepted = true;
                    break;
                }
                C = C + W;
                Sq = Sq - qy;
                // residual mass at the new C, from the pool alone
                if (tid < kWave) {
                    double pin = 0.0, res = 0.0;
                    if (lane < P) {
                        pin = s_pp[lane];
                        const double rr = s_pp[lane] * inv - C * s_q[lane];
                        res = rr > 0.0 ? rr : 0.0;
                    }
                    pin = wave_sum(pin);
                    res = wave_sum(res);
                    if (lane == 0) s_z = (Stot - pin) * inv + res;
                }
                __syncthreads();
                Z = s_z;
                __syncthreads();
                if (trace && tcount <= TSB_TRACE_MAX) trace[(tcount - 1) * 4 + 3] = Z;
                if (Z <= 0.0 || (j + 1 < m && Sq <= 0.0)) {
                    degenerate = true;
                    break;
                }
            }
            __syncthreads();  // s_tok & co. are rewritten at the next node
            if (accepted) continue;
            // every child rejected: bonus from the residual max(p - C q, 0)
            if (!degenerate) {
                for (int w = tid; w < nwords; w += kWalkThreads) s_bits[w] = 0u;
                __syncthreads();
                if (tid < P) {
                    const int t = s_ptok[tid];
                    if (t >= S.v0 && t < S.v1) atomicOr(&s_bits[(t - S.v0) >> 5], 1u << ((t - S.v0) & 31));
                }
                __syncthreads();
                BestKey b = bonus_off_pool<DT>(A, vec, S, trow, Lt, key, (uint32_t)u, s_bits);
                if (tid < P) {
                    const int t = s_ptok[tid];
                    if (t >= S.v0 && t < S.v1) {
                        const double rr = s_pp[tid] * inv - C * s_q[tid];
                        if (rr > 0.0) {
                            b.offer(logf((float)rr) + gumbel_f32(rng_word(key, (uint32_t)u, kStreamBonus, (uint32_t)t)), t);
                        }
                    }
                }
                double unused;
                const int fi = X.best(b, 0.0, &unused);
                if (fi >= 0) {
                    bonus_out = fi;
                } else {
                    degenerate = true;
                }
            }
            if (degenerate) {  // empty residual: bonus from p_u
                double unused;
                RawRow<DT> rt;
                rt.load(A.target, vec, S, trow);
                bonus_out = X.best(bonus_from_p<DT>(A, vec, S, trow, rt, Lt, key, (uint32_t)u), 0.0, &unused);
                add_status |= TSB_REQ_DEGENERATE_RESIDUAL;
            }
            break;
        }
        if (X.timeout) add_status |= TSB_REQ_WALK_TIMEOUT;
        __syncthreads();
        if (s_badtok) add_status |= TSB_REQ_BAD_TOKEN;
    }
    walk_tail(A, r, g, n, draft_bad, invalid, nacc, bonus_out, add_status, tcount);
}

// ---------------------------------------------------------- traversal walk
// Traversal verification (Appendix A; Table 2): sequence-level recursive
// rejection sampling over the replayed tree. All G workgroups of a request
// replay the same scalar traversal over a stack of the current path (in
// LDS); every vocabulary-wide quantity is split over their slices and
// exchanged:
//   * the binary64 target normaliser of an internal node when the traversal
//     first descends from it (its children's acceptance probabilities need
//     p_u);
//   * the residual mass T = sum_v max(A' p_v - C' q_v, 0) at a node after one
//     of its children was rejected;
//   * the bonus draw at the node that ends the round.
// Closed form of a node's state (equal to the literal updates): Mb_u =
// max(A p - C q, 0) / Z is the bonus distribution at u, Ms_u = q / S over
// the tokens not yet removed the draft distribution of its remaining
// children; a node enters with alpha from its parent and (A, C, Z, S) =
// (1, 0, 1, 1). The child of u with token y has
//   alpha_c = min(1, alpha_u max(A p(y) - C q(y), 0) / Z * S / q(y));
// rejecting it maps u's state to A' = alpha A / Z, C' = alpha C / Z + 1 / S,
// Z' = T, alpha' = T / (T + 1 - alpha), S' = S - q(y).
// The traversal is post-order (the first remaining child first, down to a
// node with none left, which is tested with U < alpha); the root has
// alpha = 1 and is accepted once its children are all rejected. The (p~, q)
// slice held is that of the node the last pass was over, so consecutive
// rejections among the children of one node reuse it.
//
// Bound by latency: a request's tests follow one another (up to one per node,
// 128 in the slowest of 16 requests of 128 nodes, where the others take one),
// each with a pass over the slice and an exchange. Everything else a test
// needs is in registers when it is reached: a node's children (tokens, logits,
// uniforms, probabilities, whether they are leaves) come with its record, one
// child a lane, and a leaf is tested without entering it.
// The node the traversal is at, the same in every thread. The states of its
// ancestors wait on a stack in LDS; the node's children (Entered) and its
// slice's (p~, q) are held in registers and read again when the traversal
// comes back to it.
struct TravState {
    int node, left;       // left: children rejected so far
    double alpha, A, C, Z, S;
    double L;             // binary64 log normaliser of the node's target row, NaN until computed
    double qself, uself;  // the node's own token's draft probability and uniform (as a child)
};

template <int DT, bool VEC>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(4))) void verify_traversal(WalkArgs A) {
    extern __shared__ double s_dyn[];  // the stack, root .. depth D, then (p~, q) of the slice
    __shared__ double s_exp[kExpTable];
    TravState* const s_stk = (TravState*)s_dyn;
    const int G = A.G;
    const int ticket = xticket(A.X, A.R);
    const int g = ticket % G;
    const int r = ticket / G;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int B1 = A.B + 1;
    const size_t tb = (size_t)r * B1;
    const bool vec = VEC;
    int* status_p = A.out.req_status + r;
    const int n_raw = A.tree.n_nodes[r];
    const bool count_ok = tree_count_ok(n_raw, A.B);
    const int n = count_ok ? n_raw : 0;
    const bool lead = (g == 0 && tid == 0);
    exp64_table_init(s_exp);

    const WalkSlice S = walk_slice(A.V, g, G);
    const HeldPQ pq{s_dyn + (A.D + 1) * (sizeof(TravState) / sizeof(double)), S.groups};
    const bool draft_bad = (*status_p & TSB_REQ_NONFINITE) != 0;

    int tcount = 0;
    double* const trace = (lead && A.out.trace) ? A.out.trace + (size_t)r * TSB_TRACE_MAX * 4 : nullptr;
    int bonus_out = -1, add_status = count_ok ? 0 : TSB_REQ_BAD_TREE, nacc = 0;
    bool invalid = !count_ok;
    if (!draft_bad && count_ok) {
        RngKey key;
        key.k0 = A.k0;
        key.k1 = A.k1;
        key.request = (uint32_t)r;
        key.step = A.step;
        Exchange X{&A, r, g, G, 0u, 0};
        int top = 0;
        TravState E;
        Entered N;
        double ul = 0.0, pl = 0.0, ql = 0.0;  // lane j: child j's uniform and probabilities
        RawRow<DT> rt, rd;
        bool raw = false, filled = false;  // the slice's logits, its (p~, q) are E.node's
        const auto rows = [&](int u, int d, size_t& trow, size_t& drow) {
            trow = ((size_t)r * B1 + u) * (size_t)A.V;
            drow = ((size_t)r * A.D + d) * (size_t)A.V;
        };
        // children of E.node, from its record
        const auto children = [&]() {
            N = enter_record(A.nrec, tb + E.node, lane);
            if (!N.l0) {
                int tbad;
                N.L0 = uni(target_lse(A, r, E.node, &tbad));
            }
            ul = u24d(rng_word(key, (uint32_t)(N.t.fc + lane), kStreamAccept, 0u));
            raw = filled = false;
        };
        const auto load_rows = [&]() {
            if (raw) return;
            size_t trow, drow;
            rows(E.node, N.t.d, trow, drow);
            rt.load(A.target, vec, S, trow);
            rd.load(A.draft, vec, S, drow);
            raw = true;
        };
        const auto probabilities = [&]() {
            ql = exp64x((double)N.xd - N.Ld, s_exp);
            pl = exp64x((double)N.xt - E.L, s_exp);
        };
        // the slice's (p~, q) of E.node (nothing if they are held already);
        // returns the thread's sum of p~ then evaluated
        const auto fill = [&]() -> double {
            if (!S.held || filled) return 0.0;
            load_rows();
            size_t trow, drow;
            rows(E.node, N.t.d, trow, drow);
            double sp = 0.0;
            pq.fill<DT>(A, vec, S, trow, drow, rt, rd, N.L0, N.Ld, s_exp, [&](double p, double) { sp += p; });
            filled = true;
            return sp;
        };
        E = TravState{0, 0, 1.0, 1.0, 0.0, 1.0, 1.0, (double)NAN, 1.0, 0.0};
        children();
        // end of the round: 1: bonus from Mb of E.node (or of the accepted leaf), 2: degenerate (bonus from p)
        int end_kind = 0;
        int leaf = -1;  // an accepted leaf child of E.node
        while (true) {
            // every workgroup reads the same entries, so all take the same exits;
            // a tree's nodes are tested once each, nodes that share children would
            // be once per path, of which there can be m^depth
            if (!N.t.ok || tcount >= n) {
                add_status |= TSB_REQ_BAD_TREE;
                invalid = true;
                break;
            }
            double qy;           // the rejected child's draft probability
            if (E.left < N.t.m) {  // descend to the next remaining child
                if (top + 1 > A.D) {
                    add_status |= TSB_REQ_BAD_TREE;
                    invalid = true;
                    break;
                }
                if (isnan(E.L)) {  // first descent: binary64 normaliser of the node's target row
                    double s[1] = {0.0};
                    if (S.held) {
                        s[0] = fill();
                    } else {
                        size_t trow, drow;
                        rows(E.node, N.t.d, trow, drow);
                        visit_pq<DT>(A, vec, S, trow, drow, N.L0, N.Ld, s_exp, [&](int, double p, double) { s[0] += p; });
                    }
                    X.sum<1>(s);
                    E.L = uni(N.L0 + log64(s[0], s_exp));
                    probabilities();
                }
                const int c = N.t.fc + E.left;
                const int y = (int)lane_u32((uint32_t)N.tok, E.left);
                if (y < 0 || y >= A.V) {
                    add_status |= TSB_REQ_BAD_TOKEN;
                    invalid = true;
                    break;
                }
                qy = lane_f64(ql, E.left);
                const double num = E.A * lane_f64(pl, E.left) - E.C * qy;  // Z Mb_u(y) before the max
                const double ms = qy / E.S;                                // Ms_u(y)
                double ac;
                if (!(ms > 0.0))
                    ac = (num > 0.0 && E.alpha > 0.0) ? 1.0 : 0.0;
                else
                    ac = num > 0.0 ? fmin(1.0, E.alpha * (num / E.Z) / ms) : 0.0;
                ac = uni(ac);
                const double U = lane_f64(ul, E.left);
                if ((int)lane_u32((uint32_t)N.kids, E.left) != 0) {
                    // a child with children of its own: its state waits for theirs
                    __syncthreads();  // the stack's entry may still be read
                    if (tid == 0) s_stk[top] = E;
                    __syncthreads();
                    ++top;
                    E = TravState{c, 0, ac, 1.0, 0.0, 1.0, 1.0, (double)NAN, qy, U};
                    children();
                    if (N.t.ok && N.t.m > 0) load_rows();
                    continue;
                }
                // a leaf: tested on the spot
                if (trace && tcount < TSB_TRACE_MAX) {
                    trace[tcount * 4 + 0] = c;
                    trace[tcount * 4 + 1] = U;
                    trace[tcount * 4 + 2] = ac;
                    trace[tcount * 4 + 3] = -1.0;
                }
                ++tcount;
                if (U < ac) {
                    leaf = c;
                    end_kind = 1;
                    break;
                }
            } else {
                if (top == 0) {  // every child of the root rejected: the root is accepted
                    end_kind = 1;
                    break;
                }
                // test the node: accept the path root .. node with probability alpha
                if (trace && tcount < TSB_TRACE_MAX) {
                    trace[tcount * 4 + 0] = E.node;
                    trace[tcount * 4 + 1] = E.uself;
                    trace[tcount * 4 + 2] = E.alpha;
                    trace[tcount * 4 + 3] = -1.0;
                }
                ++tcount;
                if (E.uself < E.alpha) {
                    end_kind = 1;
                    break;
                }
                qy = E.qself;
                --top;
                {
                    const TravState w = s_stk[top];
                    E = TravState{uni(w.node), uni(w.left), uni(w.alpha), uni(w.A), uni(w.C), uni(w.Z),
                                  uni(w.S), uni(w.L), uni(w.qself), uni(w.uself)};
                }
                children();
                load_rows();
                probabilities();
            }
            // the child was rejected: update E with the quantities it was drawn from
            const double A2 = uni(E.alpha * E.A / E.Z);
            const double C2 = uni(E.alpha * E.C / E.Z + 1.0 / E.S);
            const double inv = uni(exp64x(N.L0 - E.L, s_exp));
            double z[1] = {0.0};
            if (S.held) {
                fill();
                z[0] = pq.residual(S, A2 * inv, C2);
            } else {
                size_t trow, drow;
                rows(E.node, N.t.d, trow, drow);
                visit_pq<DT>(A, vec, S, trow, drow, N.L0, N.Ld, s_exp, [&](int, double p, double q) {
                    const double rr = p * (A2 * inv) - C2 * q;
                    z[0] += rr > 0.0 ? rr : 0.0;
                });
            }
            X.sum<1>(z);
            const double T = uni(z[0]);
            if (trace && tcount <= TSB_TRACE_MAX) trace[(tcount - 1) * 4 + 3] = T;
            const int left = E.left + 1;
            const double S2 = uni(E.S - qy);
            if ((T <= 0.0 && E.alpha >= 1.0) || (S2 <= 0.0 && left < N.t.m)) {
                end_kind = 2;
                break;
            }
            E.left = left;
            E.S = S2;
            if (T > 0.0) {
                E.alpha = uni(T / (T + (1.0 - E.alpha)));
                E.A = A2;
                E.C = C2;
                E.Z = T;
            } else {
                E.alpha = 0.0;
                E.A = 0.0;
                E.C = 0.0;
                E.Z = 1.0;
            }
        }
        if (end_kind != 0) {
            const int u = leaf >= 0 ? leaf : E.node;
            const size_t trow = ((size_t)r * B1 + u) * (size_t)A.V;
            // a node whose residual was never formed: Mb = p
            bool from_p = end_kind == 2 || leaf >= 0 || E.left == 0;
            if (!from_p) {
                // Gumbel-max of ln max(p - (C / A) q, 0) (the positive factor A and the normaliser Z shift
                // every key alike)
                size_t tr, dr;
                rows(E.node, N.t.d, tr, dr);
                const double lam = E.C / E.A;
                const double inv = exp64x(N.L0 - E.L, s_exp);
                fill();
                double unused_mass, unused;
                const BestKey b = bonus_residual<DT>(A, vec, S, tr, dr, pq, N.L0, N.Ld, inv, lam, s_exp, key,
                                                         (uint32_t)u, unused_mass);
                const int fi = X.best(b, 0.0, &unused);
                if (fi >= 0) {
                    bonus_out = fi;
                } else {
                    from_p = true;
                    end_kind = 2;
                }
            }
            if (from_p) {
                double L = E.L;
                if (leaf >= 0 || isnan(L)) {
                    int tbad;
                    L = target_lse(A, r, u, &tbad);
                }
                RawRow<DT> t;
                t.load(A.target, vec, S, trow);
                double unused;
                bonus_out = X.best(bonus_from_p<DT>(A, vec, S, trow, t, L, key, (uint32_t)u), 0.0, &unused);
            }
            if (end_kind == 2) add_status |= TSB_REQ_DEGENERATE_RESIDUAL;
            nacc = top + (leaf >= 0 ? 1 : 0);
            if (lead)
                for (int i = 1; i <= nacc; ++i) {
                    const int c = i == top + 1 ? leaf : (i == top ? E.node : s_stk[i].node);
                    A.out.acc_node[(size_t)r * A.D + i - 1] = c;
                    A.out.acc_tok[(size_t)r * A.D + i - 1] = A.node_tok[tb + c];
                }
        }
        if (X.timeout) add_status |= TSB_REQ_WALK_TIMEOUT;
    }
    walk_tail(A, r, g, n, draft_bad, invalid, nacc, bonus_out, add_status, tcount);
}

// ------------------------------------------------------------------ launch
// Workgroups of the walk that fit on the current device at once (the tickets
// need the G of one request to). Queried once per (device, kernel instance).
static hipError_t walk_capacity(const void* fn, int kind, int dt, int vec, size_t lds, int* cap) {
    constexpr int kDevs = 64;
    static std::atomic<int> cached[kDevs][3][2][2];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kDevs) {
        const int v = cached[dev][kind][dt][vec].load(std::memory_order_relaxed);
        if (v > 0) {
            *cap = v;
            return hipSuccess;
        }
    }
    int cus = 0, per_cu = 0;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kWalkThreads, lds)) != hipSuccess) return e;
    *cap = per_cu * cus;
    if (dev >= 0 && dev < kDevs && *cap > 0) cached[dev][kind][dt][vec].store(*cap, std::memory_order_relaxed);
    return hipSuccess;
}

TargetJob target_job(const tsb_config& c, const void* target, const tsb_tree& tree, const double* draft_lse,
                     char* ws, bool rows) {
    const Geometry g = geometry(c);
    const VerifyWs w = verify_ws(c);
    TargetJob j;
    j.target = target;
    j.n_nodes = tree.n_nodes;
    j.tm = (float*)(ws + w.tm);
    j.ts = (double*)(ws + w.ts);
    j.tf = (int*)(ws + w.tf);
    j.slots = (uint64_t*)(ws + xchg_ws(c).slots);
    j.chunk = g.chunk4;
    j.nrows = c.R * (c.B + 1);
    j.P = g.S4;
    j.ngroups = g.G4;
    j.R = c.R;
    j.vec = (c.dtype == TSB_BF16) ? (c.V % 8 == 0 && ((uintptr_t)target & 15) == 0)
                                  : (c.V % 4 == 0 && ((uintptr_t)target & 15) == 0);
    j.nrec = draft_lse ? (uint32_t*)(ws + w.nrec) : nullptr;
    j.draft_lse = draft_lse;
    if (!rows) {
        // no row: the job's workgroups only clear the exchange slots
        j.nrows = 0;
        j.ngroups = kClearWorkgroups;
    }
    return j;
}

// With a record job, workgroups after the chunks' write the walk's node
// records (without the normalisers, which only the chunks hold).
static hipError_t launch_target_partials(const tsb_config& c, float invT, const void* target, const tsb_tree& tree,
                                         const VerifyWs& w, char* ws, hipStream_t st, const RecordJob& rec) {
    TargetJob j = target_job(c, target, tree, nullptr, ws);
    j.tm = (float*)(ws + w.tm);
    j.ts = (double*)(ws + w.ts);
    j.tf = (int*)(ws + w.tf);
    XRegion X;
    X.slots = j.slots;
    hipError_t e = hook_before(TSB_KERNEL_TARGET_PARTIALS, st);
    if (e != hipSuccess) return e;
    auto fn = c.dtype == TSB_BF16 ? (j.vec ? target_partials<TSB_BF16, true> : target_partials<TSB_BF16, false>)
                                  : (j.vec ? target_partials<TSB_F32, true> : target_partials<TSB_F32, false>);
    fn<<<j.ngroups + record_blocks(rec, kBlock), kBlock, 0, st>>>(target, c.V, c.B, j.nrows, j.chunk, j.P, invT,
                                                                  j.n_nodes, j.tm, j.ts, j.tf, X, c.R, j.ngroups, rec);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return hook_after(TSB_KERNEL_TARGET_PARTIALS, st);
}

// Rows 0 and 1 of every request for a walk that reads the other rows itself
// (tsb_verify; a round streams them beside the planner), the clearing of the
// walk's exchange slots and, on the workgroups after those, its node records.
// No profiling id: tsb_profile_kernel's target stream is target_partials alone.
template <int DT, bool VEC>
__global__ __launch_bounds__(kChainThreads) void chain_rows(ChainJob cj, XRegion X, int R, float invT, int nchain,
                                                            RecordJob rec) {
    if ((int)blockIdx.x >= nchain) {
        record_block<DT>(rec, (int)blockIdx.x - nchain, invT);
        return;
    }
    xclear(X, R, (size_t)blockIdx.x * kChainThreads + threadIdx.x, (size_t)nchain * kChainThreads);
    for (int g = blockIdx.x; g < cj.items; g += nchain)
        chain_piece<DT, VEC>(g, cj.target, cj.V, cj.B, invT, cj.cm, cj.cs, cj.cf);
}

static hipError_t launch_chain_rows(const tsb_config& c, float invT, const void* target, char* ws, hipStream_t st,
                                    const RecordJob& rec) {
    const ChainJob j = chain_job(c, target, ws);
    XRegion X;
    X.slots = (uint64_t*)(ws + xchg_ws(c).slots);
    const int grid = std::max(kClearWorkgroups, std::min(j.items, 1024));
    auto fn = c.dtype == TSB_BF16 ? (j.vec ? chain_rows<TSB_BF16, true> : chain_rows<TSB_BF16, false>)
                                  : (j.vec ? chain_rows<TSB_F32, true> : chain_rows<TSB_F32, false>);
    fn<<<grid + record_blocks(rec, kChainThreads), kChainThreads, 0, st>>>(j, X, c.R, invT, grid, rec);
    return hipGetLastError();
}

// Workgroups per request of a walk, at most the resident ones of its kernel
// (the tickets need those of one request to fit on the device at once), and
// the LDS of the slices that this many leave: the kernel works its slice out
// from the same G (a slice recomputed in every pass needs no LDS).
struct WalkShape {
    int G;
    size_t lds;
};
static WalkShape walk_shape(const tsb_config& c, int resident) {
    WalkShape w;
    w.G = std::min(geometry(c).G, resident);
    const int span = walk_span(c.V, w.G);
    w.lds = span <= kWalkHeldTokens ? (size_t)span * 2 * sizeof(double) : 0;
    return w;
}
// What residency is asked with: the largest LDS a launch may need.
constexpr size_t kWalkLdsMax = (size_t)kWalkHeldTokens * 2 * sizeof(double);
constexpr size_t trav_stack_bytes(int D) { return (size_t)(D + 1) * sizeof(TravState); }

// Walk arguments shared by both walks.
static WalkArgs walk_args(const tsb_config& c, float invT, const void* draft, const double* draft_lse,
                          const void* target, const tsb_tree& tree, const int32_t* node_tok, uint32_t step,
                          const tsb_verdict& out, const VerifyWs& w, char* ws) {
    const Geometry g = geometry(c);
    WalkArgs A;
    A.draft = draft;
    A.draft_lse = draft_lse;
    A.target = target;
    A.tree = tree;
    A.node_tok = node_tok;
    A.out = out;
    A.tm = (const float*)(ws + w.tm);
    A.ts = (const double*)(ws + w.ts);
    A.tf = (const int*)(ws + w.tf);
    A.X.slots = (uint64_t*)(ws + xchg_ws(c).slots);
    A.V = c.V;
    A.D = c.D;
    A.B = c.B;
    A.S4 = g.S4;
    A.R = c.R;
    A.G = 1;
    A.stats = stats_ptr();
    A.invT = invT;
    A.k0 = (uint32_t)c.seed;
    A.k1 = (uint32_t)(c.seed >> 32);
    A.step = step;
    A.pool_tok = nullptr;
    A.trans = nullptr;
    A.P = 0;
    A.nrec = (const uint32_t*)(ws + w.nrec);
    A.reads_rows = 0;
    const XchgWs x = xchg_ws(c);
    A.cm = (const float*)(ws + x.cm);
    A.cs = (const double*)(ws + x.cs);
    A.cf = (const int*)(ws + x.cf);
    return A;
}

// One launch of a walk grid: G workgroups per request, each taking its
// (request, slice) from a ticket (xticket), so only G workgroups need to fit
// on the device at once.
static hipError_t launch_walk_grid(const void* fn, WalkArgs& A, int R, int G, size_t lds, hipStream_t st) {
    A.R = R;
    A.G = G;
    void* args[] = {&A};
    return hipLaunchKernel(fn, dim3((unsigned)(A.G * R)), dim3(kWalkThreads), args, lds, st);
}

hipError_t launch_verify(const tsb_config& c, float invT, const void* draft, const double* draft_lse,
                         const void* target, const tsb_tree& tree, const int32_t* node_tok, uint32_t step,
                         const tsb_verdict& out, char* ws, hipStream_t st, int stages) {
    const VerifyWs w = verify_ws(c);
    hipError_t e = hipSuccess;
    // a walk that reads the rows of the nodes it enters needs every row
    // streamed only for the optional normaliser output
    const bool reads = walk_reads_rows(c);
    if (stages & kStageTarget) {
        const RecordJob rec{draft, target, tree, node_tok, draft_lse, (uint32_t*)(ws + w.nrec), c.R, c.B, c.D, c.V};
        const RecordJob none{};
        if ((out.target_lse || !reads) &&
            (e = launch_target_partials(c, invT, target, tree, w, ws, st, reads ? none : rec)) != hipSuccess)
            return e;
        if (reads && (e = launch_chain_rows(c, invT, target, ws, st, rec)) != hipSuccess) return e;
    }
    if (!(stages & kStageWalk)) return hipSuccess;
    WalkArgs A = walk_args(c, invT, draft, draft_lse, target, tree, node_tok, step, out, w, ws);
    A.reads_rows = reads ? 1 : 0;
    const bool vec4 = c.V % 4 == 0 && ((uintptr_t)target & 15) == 0 && ((uintptr_t)draft & 15) == 0;
    const bool bf16 = c.dtype == TSB_BF16;
    const void* fn = bf16 ? (vec4 ? (const void*)verify_walk<TSB_BF16, true> : (const void*)verify_walk<TSB_BF16, false>)
                          : (vec4 ? (const void*)verify_walk<TSB_F32, true> : (const void*)verify_walk<TSB_F32, false>);
    int cap = 0;
    if ((e = walk_capacity(fn, 0, bf16 ? 1 : 0, vec4 ? 1 : 0, kWalkLdsMax, &cap)) != hipSuccess) return e;
    if (cap < 1) return hipErrorLaunchOutOfResources;
    const WalkShape shape = walk_shape(c, cap);
    if ((e = hook_before(TSB_KERNEL_VERIFY_WALK, st)) != hipSuccess) return e;
    if ((e = launch_walk_grid(fn, A, c.R, shape.G, shape.lds, st)) != hipSuccess) return e;
    return hook_after(TSB_KERNEL_VERIFY_WALK, st);
}

hipError_t launch_verify_traversal(const tsb_config& c, float invT, const void* draft, const double* draft_lse,
                                   const void* target, const tsb_tree& tree, const int32_t* node_tok, uint32_t step,
                                   const tsb_verdict& out, char* ws, hipStream_t st, int stages) {
    const VerifyWs w = verify_ws(c);
    hipError_t e = hipSuccess;
    const RecordJob rec{draft, target, tree, node_tok, draft_lse, (uint32_t*)(ws + w.nrec), c.R, c.B, c.D, c.V};
    if ((stages & kStageTarget) && (e = launch_target_partials(c, invT, target, tree, w, ws, st, rec)) != hipSuccess)
        return e;
    if (!(stages & kStageWalk)) return hipSuccess;
    WalkArgs A = walk_args(c, invT, draft, draft_lse, target, tree, node_tok, step, out, w, ws);
    const bool vec4 = c.V % 4 == 0 && ((uintptr_t)target & 15) == 0 && ((uintptr_t)draft & 15) == 0;
    const bool bf16 = c.dtype == TSB_BF16;
    const void* fn = bf16 ? (vec4 ? (const void*)verify_traversal<TSB_BF16, true> : (const void*)verify_traversal<TSB_BF16, false>)
                          : (vec4 ? (const void*)verify_traversal<TSB_F32, true> : (const void*)verify_traversal<TSB_F32, false>);
    int cap = 0;
    if ((e = walk_capacity(fn, 2, bf16 ? 1 : 0, vec4 ? 1 : 0, kWalkLdsMax + trav_stack_bytes(TSB_MAX_D), &cap)) != hipSuccess) return e;
    if (cap < 1) return hipErrorLaunchOutOfResources;
    const WalkShape shape = walk_shape(c, cap);
    if ((e = hook_before(TSB_KERNEL_TRAVERSAL_WALK, st)) != hipSuccess) return e;
    if ((e = launch_walk_grid(fn, A, c.R, shape.G, shape.lds + trav_stack_bytes(c.D), st)) != hipSuccess) return e;
    return hook_after(TSB_KERNEL_TRAVERSAL_WALK, st);
}

hipError_t launch_pool_verify(const tsb_config& c, int P, float invT, const void* draft, const float* trans,
                              const int32_t* pool_tok, const void* target, const tsb_tree& tree,
                              const int32_t* node_tok, uint32_t step, const tsb_verdict& out, char* ws,
                              hipStream_t st, int stages) {
    const VerifyWs w = pool_verify_ws(c);
    hipError_t e = hipSuccess;
    if ((stages & kStageTarget) &&
        (e = launch_target_partials(c, invT, target, tree, w, ws, st, RecordJob{})) != hipSuccess)
        return e;
    if (!(stages & kStageWalk)) return hipSuccess;
    WalkArgs A = walk_args(c, invT, draft, nullptr, target, tree, node_tok, step, out, w, ws);
    A.pool_tok = pool_tok;
    A.trans = trans;
    A.P = P;
    const bool vec4 = c.V % 4 == 0 && ((uintptr_t)target & 15) == 0;
    const void* fn = nullptr;
    if (c.dtype == TSB_BF16)
        fn = vec4 ? (const void*)verify_pool_walk<TSB_BF16, true> : (const void*)verify_pool_walk<TSB_BF16, false>;
    else
        fn = vec4 ? (const void*)verify_pool_walk<TSB_F32, true> : (const void*)verify_pool_walk<TSB_F32, false>;
    // the slice bitmap: one bit per token of the widest slice at the fewest
    // workgroups per request the capacity allows
    const size_t lds_max = kPoolBitmapBytes;
    int cap = 0;
    if ((e = walk_capacity(fn, 1, c.dtype == TSB_BF16 ? 1 : 0, vec4 ? 1 : 0, lds_max, &cap)) != hipSuccess) return e;
    if (cap < 1) return hipErrorLaunchOutOfResources;
    int G = geometry(c).G;
    if (G > cap) G = cap;
    const long long span = (((long long)c.V + G - 1) / G + 3) & ~3ll;
    const size_t lds = (size_t)((span + 31) / 32) * sizeof(uint32_t);
    if (lds > lds_max) return hipErrorInvalidConfiguration;  // vocabulary too wide for the slice bitmap
    if ((e = hook_before(TSB_KERNEL_POOL_WALK, st)) != hipSuccess) return e;
    if ((e = launch_walk_grid(fn, A, c.R, G, lds, st)) != hipSuccess) return e;
    return hook_after(TSB_KERNEL_POOL_WALK, st);
}

}  // namespace tsb
