// Second pass of a tree-replay round on gfx950 (Section 3.2, eq. (2);
// Appendix A): every parent u at depth d refills its m_u child slots with the
// m_u largest Gumbel keys a_{d,v} + G(u, v) over the whole vocabulary
// (Gumbel-top-k = ordered sampling without replacement).
//
//   replay_threshold  one wave per parent: a lower bound of its m-th key
//                 from its planning candidates and a sample of the row; the
//                 first workgroups write the flat list of the parents of the
//                 batch (request-major, BFS order, so a depth's parents are
//                 contiguous).
//   replay_scan   one wave per (parent, vocabulary tile) item, dealt
//                 grid-stride over a persistent grid (parents of one (request,
//                 depth) are adjacent, so their tiles of draft row d meet in
//                 cache). Per item, tokens whose key cannot reach the
//                 parent's threshold are skipped before any random
//                 number is drawn; the survivors are compacted within the
//                 wave and pay for Philox; the few whose words can reach the
//                 threshold are compacted again and pay for two logarithms.
//   replay_scan_target
//                 the scan of a whole round (tsb_step and its variants): one
//                 grid whose first workgroups stream the target's row
//                 normalisers for verification (target_chunk) while the
//                 others scan, so the HBM-bound stream and the VALU-bound
//                 scan share the compute units.
//   replay_merge  one wave per parent: the m best (key desc, token asc) of the
//                 tiles' keys, in slot order.
//
// Keys are binary32 and relative to the row's largest logit c_d:
// key = fl32(a_v - c_d) + G_v (the offset is common to all tokens of the
// row, so the order is that of a_v + G_v).
#include <math.h>

#include <algorithm>

#include "tsb_device.hpp"
#include "tsb_kernels.hpp"
#include "tsb_target.hpp"

namespace tsb {

constexpr int kTileGroups = kReplayTile / 4;  // groups of four tokens per tile
constexpr int kPassGroups = kTileGroups / 4;  // groups per compaction pass
constexpr int kScanWaves = kBlock / kWave;
constexpr int kHitCap = 128;                  // list of hits per wave: a batch of 64 more fits at up to 64
// Target workgroups of replay_scan_target (about 2.7 waves per SIMD, three
// chunks each of the 2048 of a large target; the scan's workgroups fill the
// rest as they fit, and start as workgroups finish). Measured with inputs
// rotated over four sets: 683 beat 1024 (two chunks each) by 7% and 512 (four
// each) by 2% at the batched workload, where the scan ends last.
constexpr int kFusedTargetWorkgroups = 683;
constexpr bool kFusedTargetPrefetch = false;  // see kTargetPrefetch
constexpr int kScanWorkgroupsMin = 1024, kScanWorkgroupsMax = 16384;

// A parent that replay fills: a well-formed node of the caller's topology
// (entries in range, see tree_node) with 1 <= m <= K children. Malformed
// parents, and every node of a request whose n_nodes lies outside
// [1, B + 1], are skipped: their child slots are not written.
__device__ __forceinline__ bool replay_parent(const tsb_tree& tree, int r, int u, int B, int D, int K, TreeNode* nd) {
    const int nn = tree.n_nodes[r];
    const int n = tree_count_ok(nn, B) ? nn : 0;
    if (u >= n) return false;
    *nd = tree_node(tree, (size_t)r * (B + 1), u, n, D);
    return nd->ok && nd->m > 0 && nd->m <= K;
}

// The parent list is written in chunks of kListNodes nodes, one to a workgroup
// for up to kListGroups chunks (65536 nodes), equal runs of chunks beyond. A
// workgroup counts the parents before its own chunks itself instead of waiting
// for the others: a chunk counted is a chunk of loads (all in flight together),
// a chunk written by the same workgroup before was a serial step of 4 us (16448
// nodes: the launch 39.1 us with one workgroup, 20.4 with nine; 2064 nodes:
// 10.3 either way, the thresholds' own time). With a workgroup for every chunk
// the counting grows with the square of the nodes: a replay of 4.2 M nodes took
// 9.5 ms, 8.4 M 32.3 (with runs of chunks 5.4 and 11.0, whether in 32, 64 or 128
// workgroups).
constexpr int kListPer = 8;
constexpr int kListNodes = kBlock * kListPer;
constexpr int kListGroups = 32;
struct ListSplit {
    int chunks, per, groups;  // chunks in all, of a workgroup, and workgroups
};
static ListSplit list_split(int nodes) {
    ListSplit l;
    l.chunks = (nodes + kListNodes - 1) / kListNodes;
    l.per = (l.chunks + kListGroups - 1) / kListGroups;
    l.groups = (l.chunks + l.per - 1) / l.per;
    return l;
}

// Which of nodes i0 + k * 64 + lane (k < kListPer) are parents: bit `lane` of
// par[k]. Every entry is loaded before any is tested (replay_parent's
// conditions, without its dependent loads).
__device__ __forceinline__ void list_parents(int i0, int total_nodes, int B, int D, int K, const tsb_tree& tree,
                                             uint64_t (&par)[kListPer]) {
    const int lane = lane_id();
    int nn[kListPer], nm[kListPer], nfc[kListPer], nd[kListPer];
#pragma unroll
    for (int k = 0; k < kListPer; ++k) {
        const int i = i0 + k * kWave + lane;
        const size_t e = i < total_nodes ? (size_t)i : 0;
        nn[k] = tree.n_nodes[e / (size_t)(B + 1)];
        nm[k] = tree.n_children[e];
        nfc[k] = tree.first_child[e];
        nd[k] = tree.depth[e];
    }
#pragma unroll
    for (int k = 0; k < kListPer; ++k) {
        const int i = i0 + k * kWave + lane;
        const int u = i % (B + 1);
        const int n = tree_count_ok(nn[k], B) ? nn[k] : 0;
        const int m = nm[k], fc = nfc[k], d = nd[k];
        const bool ok = m > 0 && m <= TSB_MAX_K && fc > u && fc <= n - m && d >= 0 && d < D;
        par[k] = __ballot(i < total_nodes && u < n && ok && m <= K);
    }
}

// Flat list of every parent, request-major, BFS order within a request (so
// parents of one (request, depth) are contiguous): plist[i] =
// r * (B + 1) + u; ptotal[0] = list length. Workgroup `group` writes the
// parents of its chunks (a wave kListPer * 64 nodes of each).
__device__ void prep_list(int group, const ListSplit& L, int R, int B, int D, int K, const tsb_tree& tree,
                          int* __restrict__ plist, int* __restrict__ ptotal) {
    __shared__ int s_before[kBlock / kWave], s_own[2][kBlock / kWave];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int total_nodes = R * (B + 1);
    const int c0 = group * L.per, c1 = min(L.chunks, c0 + L.per);
    uint64_t par[kListPer];
    int before = 0;
    for (int c = 0; c < c0; ++c) {
        list_parents(c * kListNodes + wave * kListPer * kWave, total_nodes, B, D, K, tree, par);
#pragma unroll
        for (int k = 0; k < kListPer; ++k) before += __popcll(par[k]);
    }
    int base = 0;
    for (int c = c0; c < c1; ++c) {
        const int i0 = c * kListNodes + wave * kListPer * kWave;
        list_parents(i0, total_nodes, B, D, K, tree, par);
        int own = 0;
#pragma unroll
        for (int k = 0; k < kListPer; ++k) own += __popcll(par[k]);
        int* const s = s_own[(c - c0) & 1];  // one barrier a chunk: the next one writes the other
        if (lane == 0) {
            s[wave] = own;
            s_before[wave] = before;
        }
        __syncthreads();
        if (c == c0)
            for (int w = 0; w < kBlock / kWave; ++w) base += s_before[w];
        int o = base;
        for (int w = 0; w < kBlock / kWave; ++w) {
            o += w < wave ? s[w] : 0;
            base += s[w];
        }
#pragma unroll
        for (int k = 0; k < kListPer; ++k) {
            if ((par[k] >> lane) & 1) plist[o + lanes_below_u64(par[k])] = i0 + k * kWave + lane;
            o += __popcll(par[k]);
        }
    }
    if (group == L.groups - 1 && threadIdx.x == 0) ptotal[0] = base;
}

__device__ __forceinline__ bool key_better(float ka, int ia, float kb, int ib) {
    return ka > kb || (ka == kb && ia < ib);
}

// Four consecutive logits of a tile as loaded (two words of bf16 pairs, or
// four binary32); positions at or past `tn` read as -inf. FULL: the whole tile
// exists and rows are vector-aligned, so the four are one unconditional load.
template <int DT>
struct Group4 {
    uint32_t w[DT == TSB_BF16 ? 2 : 4];
};
template <int DT, bool VEC, bool FULL>
__device__ __forceinline__ void load_group4(const void* __restrict__ draft, size_t base, int e0, int tn,
                                            Group4<DT>& g) {
    if (FULL || (VEC && e0 + 4 <= tn)) {
        if constexpr (DT == TSB_BF16) {
            const uint2 raw = *(const uint2*)((const uint16_t*)draft + base + e0);
            g.w[0] = raw.x;
            g.w[1] = raw.y;
        } else {
            const uint4 raw = *(const uint4*)((const float*)draft + base + e0);
            g.w[0] = raw.x;
            g.w[1] = raw.y;
            g.w[2] = raw.z;
            g.w[3] = raw.w;
        }
    } else if constexpr (DT == TSB_BF16) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = e0 + 2 * h;
            const uint32_t lo = e < tn ? (uint32_t)((const uint16_t*)draft)[base + e] : 0xFF80u;
            const uint32_t hi = e + 1 < tn ? (uint32_t)((const uint16_t*)draft)[base + e + 1] : 0xFF80u;
            g.w[h] = lo | (hi << 16);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            g.w[e] = e0 + e < tn ? __float_as_uint(((const float*)draft)[base + e0 + e]) : 0xFF800000u;
    }
}

// Groups of four tokens per lane whose keys a parent's threshold is sampled
// from (the first 1024 or 2048 tokens of the row; twice as many cost the
// threshold what they save the scan). Sampled are rows of at least
// kSampleMinV tokens (a row of a few tiles has few keys above any threshold)
// in calls of at least kSampleMinNodes nodes.
//
// What decides is the rows' spread, more than the nodes. A replay without and
// with the sample, 151936 logits, at 65, 256 and 520 nodes (us): standard
// deviation 0.05 37.6 / 25.7, 40.0 / 28.4, 48.4 / 32.0; 1: 33 / 29, 36 / 31,
// 42 / 34; rows of 1 to 6: 29.5 / 27.6, 31.2 / 30.5, 38.3 / 35.2; of 2 to 5:
// 25.2 / 25.8, 27.4 / 29.3, 31.6 / 34.2; 6: 17.9 / 20.7, 20.3 / 23.3, 32.3 /
// 35.4 (32000 logits: the same to 2 us). So it costs steep rows 1 to 3 us at
// any size and saves flat ones 4 to 16. The rule does not know the spread:
// below the line, calls of few requests, whose rows are mostly steep, go
// without it; above, batches mix rows and the flattest end the scan.
constexpr int kSampleGroups = 4;
constexpr int kSampleFewChildren = 4;  // up to this many children one round of groups, else two
constexpr int kSampleMinV = 4 * kReplayTile;
constexpr int kSampleMinNodes = 256;

template <int DT>
struct SampleGroups {
    Group4<DT> g[kSampleGroups];
    __device__ __forceinline__ void load(const void* __restrict__ draft, size_t rowbase, bool vec, int h, int lane) {
#pragma unroll
        for (int k = 0; k < kSampleGroups; ++k) {
            const int e0 = ((h * kSampleGroups + k) * kWave + lane) * 4;
            if (vec)
                load_group4<DT, true, true>(draft, rowbase, e0, kSampleMinV, g[k]);
            else
                load_group4<DT, false, false>(draft, rowbase, e0, kSampleMinV, g[k]);
        }
    }
    // largest key of the lane's groups (round h), and of `best`
    __device__ __forceinline__ float keys(float best, float invT, float cd, const RngKey& key, int u, int h,
                                          int lane) const {
#pragma unroll
        for (int k = 0; k < kSampleGroups; ++k) {
            const uint4 w = rng_block(key, (uint32_t)u, kStreamReplay, (uint32_t)((h * kSampleGroups + k) * kWave + lane));
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t x = DT == TSB_BF16 ? (e & 1 ? g[k].w[e >> 1] & 0xFFFF0000u : g[k].w[e >> 1] << 16)
                                                  : g[k].w[DT == TSB_BF16 ? 0 : e];
                const float b = __uint_as_float(x) * invT - cd;
                best = fmaxf(best, b + gumbel_f32(ws[e]));  // NaN is ignored
            }
        }
        return best;
    }
};

// Per parent u (one wave each): a lower bound of its m_u-th largest key over
// the vocabulary (the same key arithmetic as the scan; -inf without pruning),
// the larger of two: the m_u-th largest among the keys of its planning
// candidates, which is near on peaked rows, and a sample's, which is near on
// flat ones (there the candidates alone let 75 to 240 tokens of a tile pass
// for 6 to 10 children, each inserted one by one, and such items ended the
// scan). It is stored with what the scan needs of the parent in one record
// (c_d, thr, depth, m_u). The grid's first workgroups build the parent list
// instead.
template <int DT>
__global__ __launch_bounds__(kBlock) void replay_threshold(const void* __restrict__ draft, int R, int V, int D, int B,
                                                           int K, float invT, const int32_t* __restrict__ topk_tok,
                                                           tsb_tree tree, uint32_t k0, uint32_t k1, uint32_t step,
                                                           int prune, int vec, float4* __restrict__ rec,
                                                           int* __restrict__ plist, int* __restrict__ ptotal,
                                                           ListSplit list) {
    if ((int)blockIdx.x < list.groups) {
        prep_list(blockIdx.x, list, R, B, D, K, tree, plist, ptotal);
        return;
    }
    const int lane = threadIdx.x % kWave;
    const int node = ((int)blockIdx.x - list.groups) * (kBlock / kWave) + threadIdx.x / kWave;
    if (node >= R * (B + 1)) return;
    const int r = node / (B + 1), u = node % (B + 1);
    TreeNode nd;
    if (!replay_parent(tree, r, u, B, D, K, &nd)) return;
    const int m = nd.m, d = nd.d;
    const size_t rowbase = ((size_t)r * D + d) * (size_t)V;
    const int32_t* tk = topk_tok + ((size_t)r * D + d) * K;
    // the sampled groups are in flight beside the candidates
    const bool sample = prune && V >= kSampleMinV && R * (B + 1) >= kSampleMinNodes;
    SampleGroups<DT> sg;
    if (sample) sg.load(draft, rowbase, vec != 0, 0, lane);
    // candidate tokens are checked before they become addresses; the
    // threshold is a lower bound of the m-th key only over K distinct tokens
    // of the row, so an out-of-range or repeated candidate turns pruning off
    const int t0 = tk[0];
    const float cd = (t0 >= 0 && t0 < V) ? load_logit<DT>(draft, rowbase + t0) * invT : 0.f;
    RngKey key;
    key.k0 = k0;
    key.k1 = k1;
    key.request = (uint32_t)r;
    key.step = step;
    float kj = -INFINITY;
    int tj = 0x7FFFFFFF;
    bool tok_ok = true;
    if (lane < K) {
        tj = tk[lane];
        tok_ok = tj >= 0 && tj < V;
        const float a = tok_ok ? load_logit<DT>(draft, rowbase + tj) * invT : -INFINITY;
        const float bj = a - cd;
        kj = bj + gumbel_f32(rng_word(key, (uint32_t)u, kStreamReplay, (uint32_t)tj));
    }
    int above = 0;
    for (int j = 0; j < K; ++j) {
        const float kk = __shfl(kj, j, kWave);
        const int tt = __shfl(tj, j, kWave);
        above += key_better(kk, tt, kj, tj) ? 1 : 0;
        tok_ok = tok_ok && !(lane < K && j < lane && tt == tj);
    }
    const bool cands_ok = __ballot(!tok_ok) == 0ull && t0 >= 0 && t0 < V;
    const uint64_t at = __ballot(lane < K && above == m - 1);  // one lane for distinct finite keys
    float thr = (prune && cands_ok && at != 0ull) ? lane_f32(kj, (int)__ffsll((unsigned long long)at) - 1) : -INFINITY;
    if (sample && cands_ok) {
        // the m-th largest (m <= 32) of the lane maxima over the keys of the
        // row's first tokens is at most the m-th largest key: lanes hold
        // distinct tokens
        float best = sg.keys(-INFINITY, invT, cd, key, u, 0, lane);
        if (m > kSampleFewChildren) {
            sg.load(draft, rowbase, vec != 0, 1, lane);
            best = sg.keys(best, invT, cd, key, u, 1, lane);
        }
        thr = fmaxf(thr, wave_kth_largest(best, m));
    }
    if (lane == 0) rec[node] = make_float4(cd, thr, __int_as_float(d), __int_as_float(m));
}

// Four logits of the draft row as b = fl32(a - c_d); positions at or past
// `tn` (relative to the tile) read as -inf.
template <int DT, bool VEC>
__device__ __forceinline__ void load_b4(const void* __restrict__ draft, size_t base, int e0, int tn, float invT,
                                        float cd, float b[4]) {
    float x[4];
    if (VEC && e0 + 4 <= tn) {
        if (DT == TSB_BF16) {
            const uint2 raw = *(const uint2*)((const uint16_t*)draft + base + e0);
            x[0] = __uint_as_float(raw.x << 16);
            x[1] = __uint_as_float(raw.x & 0xFFFF0000u);
            x[2] = __uint_as_float(raw.y << 16);
            x[3] = __uint_as_float(raw.y & 0xFFFF0000u);
        } else {
            const float4 a = *(const float4*)((const float*)draft + base + e0);
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (e0 + e < tn) ? load_logit<DT>(draft, base + e0 + e) : -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = (e0 + e < tn) ? x[e] * invT - cd : -INFINITY;
}

// Largest of a group's four bf16 logits (NaN is ignored).
__device__ __forceinline__ float group_max_bf16(uint32_t w0, uint32_t w1) {
    return fmaxf(fmaxf(__uint_as_float(w0 << 16), __uint_as_float(w0 & 0xFFFF0000u)),
                 fmaxf(__uint_as_float(w1 << 16), __uint_as_float(w1 & 0xFFFF0000u)));
}

// Test of four bf16 logits against a bound on x, on packed patterns without
// an order-preserving map: x >= xt > 0 means a pattern of at least xt's as
// signed 16-bit numbers, and x >= xt with xt <= 0 a pattern of at most xt's as
// unsigned ones. Flipping the sign bit (positive xt) or every bit (otherwise)
// makes both "some flipped pattern is above `below` as an unsigned number".
//
// xt is the smallest x with fl32(fl32(x invT) - c_d) >= bound, lowered by far
// more than the roundings on both sides (2^-20 of the magnitudes, against
// three roundings of 2^-24): a necessary condition only. -inf never passes (no
// draw keeps it); an overflow or a NaN lets every other pattern pass.
struct LiveTest {
    uint32_t flip, below;  // both halves alike
    __device__ __forceinline__ void init(float bound, float cd, float invT) {
        const float y = (bound + cd) - (fabsf(bound) + fabsf(cd)) * 0x1p-20f;
        const float q = y / invT;
        const float x = q - fabsf(q) * 0x1p-20f;
        uint32_t f = 0xFFFFu, t = 0xFF80u ^ 0xFFFFu;  // above -inf
        if (x > -INFINITY && x < INFINITY) {
            const uint32_t b = __float_as_uint(x);
            if (x > 0.0f) {
                f = 0x8000u;
                t = (((b + 0xFFFFu) >> 16) ^ f) - 1u;  // rounded up: the smallest bf16 at least x
            } else {
                const uint32_t p = 0x8000u | ((b & 0x7FFFFFFFu) >> 16);  // toward zero; -0 for +0
                if (p < 0xFF80u) t = (p ^ f) - 1u;
            }
        }
        flip = f | (f << 16);
        below = t | (t << 16);
    }
    __device__ __forceinline__ bool live(uint32_t w0, uint32_t w1) const {
        const tsb_u16x2 a = __builtin_bit_cast(tsb_u16x2, w0 ^ flip), b = __builtin_bit_cast(tsb_u16x2, w1 ^ flip);
        const tsb_u16x2 t = __builtin_bit_cast(tsb_u16x2, below);
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_elementwise_max(a, b), t)) != below;
    }
};

// Which raw Philox words a token may hold for its key to reach thr when its
// logit is at most x: a necessary condition only (other words are certain
// misses, these are evaluated exactly). With y = thr - b, the key can reach
// thr only if G(u) >= y - s' for a slack s' that covers the rounding of the
// binary32 Gumbel map and of the key sum (both near 1e-6 of thr); G(u) >= y
// means -ln u <= e^-y, and -ln u >= 1 - u, so it needs 1 - u <= e^(s' - y) with
// 1 - u = (2^23 - (w >> 9) - 1/2) 2^-23 >= (~w - 2^8) 2^-32. So
//   ~w <= 2^32 e^(x invT - c_d - thr + s) + 2^10,
// evaluated as 2^(x scale + shift) by one FMA and the hardware exponential.
// The slack s = 1/4 plus 2^-20 of the magnitudes involved is far above s' and
// the roundings here (|x invT| <= |c_d| + |thr| + 17 for a live group). An
// overflowing or NaN shift admits every word.
struct WordTest {
    float scale, shift;
    __device__ __forceinline__ void init(float thr, float cd, float invT) {
        const float s = 0.25f + (fabsf(thr) + fabsf(cd) + 17.0f) * 0x1p-20f;
        scale = invT * 1.44269504088896341f;
        shift = ((s - thr) - cd) * 1.44269504088896341f + 32.0f;
        if (!(scale < INFINITY)) {  // temperatures below 5e-39
            scale = 0.0f;
            shift = INFINITY;
        }
    }
    __device__ __forceinline__ bool admits(uint32_t wmax, float x) const {
        const float lim = __builtin_amdgcn_exp2f(fmaf(x, scale, shift)) + 1024.0f;
        return !((float)(~wmax) > lim);
    }
};

struct ScanArgs {
    const void* draft;
    int V, D, B, T;
    float invT;
    const int* plist;
    const float4* rec;
    uint32_t k0, k1, step;
    uint64_t* out_cand;
    int* out_cnt;
};
// Work counters of one wave in LDS (items, tokens, live groups, keyed
// groups), kept only while counting is on; lane 0 updates them.
struct ScanCounters {
    unsigned long long* c;  // null: not counting
    __device__ void add(int k, unsigned long long v, int lane) const {
        if (c && lane == 0) c[k] += v;
    }
    __device__ void flush(unsigned long long* stats, int lane) const {
        if (c && lane == 0 && c[0]) {
            atomicAdd(&stats[kStReplayItems], c[0]);
            atomicAdd(&stats[kStReplayTokens], c[1]);
            atomicAdd(&stats[kStReplayLive], c[2]);
            atomicAdd(&stats[kStReplayKeyed], c[3]);
        }
    }
};
__device__ __forceinline__ ScanCounters scan_counters(unsigned long long (*s)[4], int wave, int lane,
                                                      const unsigned long long* stats) {
    ScanCounters C;
    C.c = stats ? s[wave] : nullptr;
    if (C.c && lane < 4) C.c[lane] = 0;
    return C;
}

// A wave's LDS: the live groups of the current pass and the list of hits.
// bf16: a group's two words and its index in the tile (pass-relative in gl);
// binary32: (index, bits of the largest b), the logits are read again.
struct ScanQueue {
    uint2 w[kPassGroups];
    uint2 hw[kHitCap];
    uint16_t hg[kHitCap];
    uint8_t gl[kPassGroups];
};
static_assert(kPassGroups <= 256, "the pass-relative index is 8 bits");

// What an item's passes share.
struct ScanItem {
    RngKey key;
    uint32_t u;
    size_t tbase;
    int t0, tn;
    float cd, thr, bound;
};

// Exact keys of the 64 hits from `base` on, one group per lane: kv[e] is -inf
// where the key stays below thr, g the group's index in the tile. The random
// words are drawn again: a hit is one group in about fifty, so its second
// Philox costs less than carrying its words through LDS.
template <int DT, bool VEC>
__device__ __forceinline__ void hit_keys(const ScanArgs& A, const ScanItem& I, int lane, const ScanQueue& Q, int base,
                                         int hn, float (&kv)[4], int& g) {
    const bool valid = base + lane < hn;
    const int q = valid ? base + lane : 0;
    g = Q.hg[q];
    const uint4 w = rng_block(I.key, I.u, kStreamReplay, (uint32_t)(I.t0 >> 2) + (uint32_t)g);
    float bv[4];
    if constexpr (DT == TSB_BF16) {
        // the group's logits come from the list (no second read)
        const uint2 x = Q.hw[q];
        const float xq[4] = {__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xFFFF0000u),
                             __uint_as_float(x.y << 16), __uint_as_float(x.y & 0xFFFF0000u)};
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[e] = (valid && g * 4 + e < I.tn) ? xq[e] * A.invT - I.cd : -INFINITY;
    } else {
        load_b4<DT, VEC>(A.draft, I.tbase, g * 4, valid ? I.tn : 0, A.invT, I.cd, bv);
    }
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool in = bv[e] >= I.bound && bv[e] > -INFINITY;
        const float k = in ? bv[e] + gumbel_f32(ws[e]) : -INFINITY;
        kv[e] = k >= I.thr ? k : -INFINITY;
    }
}

// The hits' keys into the sorted list of the item's m best (an item whose hits
// overflow the list of hits, or hold more keys than a tile's slots: rare with
// the sampled threshold).
template <int DT, bool VEC>
__device__ __forceinline__ void list_hits(const ScanArgs& A, const ScanItem& I, int lane, const ScanQueue& Q, int hn,
                                          WaveTopList& top) {
    for (int base = 0; base < hn; base += kWave) {
        float kv[4];
        int g;
        hit_keys<DT, VEC>(A, I, lane, Q, base, hn, kv, g);
#pragma unroll 1
        for (int e = 0; e < 4; ++e) {
            const float k = e < 2 ? (e == 0 ? kv[0] : kv[1]) : (e == 2 ? kv[2] : kv[3]);
            top.offer(cand_key(k, (uint32_t)(I.t0 + g * 4 + e)), k > -INFINITY);
        }
    }
}

// One (parent, tile) item, by one wave (`it` in a scalar register: the
// parent's record, the bounds and the first rounds of its random numbers are
// scalar work). Its slots receive the tile's keys that reach thr, in no
// order, or, where they are more than m, at least the m best of them.
//
// Bound by VALU issue (about 4.6 cycles an instruction here, v_mad_u64_u32
// like the rest): per 64 groups about 15 instructions to load, test and queue
// them, and about 60 per 64 live ones, 36 of them Philox. 16 x 129 nodes x
// 151936 bf16 logits: 60.7 -> 46.0 us; 64 x 257: 295 -> 234 us.
template <int DT, bool VEC>
__device__ __forceinline__ void scan_item(const ScanArgs& A, long long it, int lane, ScanQueue& Q,
                                          const ScanCounters& C) {
    const void* __restrict__ draft = A.draft;
    const int V = A.V, D = A.D, B = A.B, T = A.T;
    const float invT = A.invT;
    const int pi = (int)(it / T);
    const int t = (int)(it - (long long)pi * T);
    const int node = A.plist[pi];
    const float4 pr = A.rec[node];  // (c_d, thr, depth, m) of the parent
    const int r = node / (B + 1);
    const int m = __float_as_int(pr.w);
    ScanItem I;
    I.u = (uint32_t)(node - r * (B + 1));
    I.cd = pr.x;
    I.thr = pr.y;
    I.bound = I.thr - kGumbelMaxBound;
    I.t0 = t * kReplayTile;
    I.tn = min(kReplayTile, V - I.t0);
    I.tbase = ((size_t)r * D + __float_as_int(pr.z)) * (size_t)V + I.t0;
    I.key.k0 = A.k0;
    I.key.k1 = A.k1;
    I.key.request = (uint32_t)r;
    I.key.step = A.step;
    const bool full = VEC && I.tn == kReplayTile;
    const uint32_t blk0 = (uint32_t)(I.t0 >> 2);
    constexpr int kPer = kPassGroups / kWave;  // groups per lane and pass
    Group4<DT> nx[kPer];
    auto issue = [&](int g0) {
        if (full) {
#pragma unroll
            for (int k = 0; k < kPer; ++k)
                load_group4<DT, VEC, true>(draft, I.tbase, (g0 + k * kWave + lane) * 4, I.tn, nx[k]);
        } else {
#pragma unroll
            for (int k = 0; k < kPer; ++k)
                load_group4<DT, VEC, false>(draft, I.tbase, (g0 + k * kWave + lane) * 4, I.tn, nx[k]);
        }
    };
    issue(0);
    WordTest wt;
    wt.init(I.thr, I.cd, invT);
    LiveTest lt;
    if (DT == TSB_BF16) lt.init(I.bound, I.cd, invT);
    WaveTopList top;      // the item's m best keys, once it keeps a sorted list
    top.init(m);
    bool listed = false;
    int hn = 0;           // groups in the list of hits
    const int ng = (I.tn + 3) / 4;
#pragma unroll 1
    for (int g0 = 0; g0 < ng; g0 += kPassGroups) {
        // the next pass's loads are in flight while this one is processed
        Group4<DT> x[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) x[k] = nx[k];
        if (g0 + kPassGroups < ng) issue(g0 + kPassGroups);
        // 1. groups whose largest b = fl32(x invT - c_d) cannot reach thr are
        // dropped, the rest are compacted within the wave
        int qn = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            bool live;
            float gx = 0.f;
            if constexpr (DT == TSB_BF16) {
                live = lt.live(x[k].w[0], x[k].w[1]);
            } else {
                // b is non-decreasing in x, so the largest is that of the largest logit
                gx = fmaxf(fmaxf(__uint_as_float(x[k].w[0]), __uint_as_float(x[k].w[1])),
                           fmaxf(__uint_as_float(x[k].w[2]), __uint_as_float(x[k].w[3])));
                const float bmax = gx * invT - I.cd;
                live = bmax >= I.bound && bmax > -INFINITY;
            }
            const uint64_t bal = __builtin_amdgcn_ballot_w64(live);
            if (live) {
                const int at = qn + lanes_below_u64(bal);
                if constexpr (DT == TSB_BF16) {
                    Q.w[at] = make_uint2(x[k].w[0], x[k].w[1]);
                    Q.gl[at] = (uint8_t)(k * kWave + lane);
                } else {
                    Q.w[at] = make_uint2((uint32_t)(g0 + k * kWave + lane), __float_as_uint(gx));
                }
            }
            qn += __popcll(bal);
        }
        wave_lds_fence();
        C.add(2, (unsigned)qn, lane);

        // 2. Philox for the survivors; groups whose largest word is a certain
        // miss are dropped, the others (about 2 of 64) are kept in the list of
        // hits, whose keys are evaluated once for the item: with the batch
        // that holds them, 86% of the batches ran the logarithms and a sorted
        // insert for about two lanes of 64
        for (int base = 0; base < qn; base += kWave) {
            const uint64_t valid = qn - base >= kWave ? ~0ull : (1ull << (qn - base)) - 1ull;
            const int q = base + lane;  // past qn: an old entry, masked below
            const uint2 ent = Q.w[q];
            int gl;
            float gx;
            if constexpr (DT == TSB_BF16) {
                gl = g0 + (int)Q.gl[q];
                gx = group_max_bf16(ent.x, ent.y);
            } else {
                gl = (int)ent.x;
                gx = __uint_as_float(ent.y);
            }
            const uint4 w = rng_block(I.key, I.u, kStreamReplay, blk0 + (uint32_t)gl);
            const uint64_t pb = __builtin_amdgcn_ballot_w64(wt.admits(max(max(w.x, w.y), max(w.z, w.w)), gx)) & valid;
            C.add(3, (unsigned)__popcll(pb), lane);
            if (pb == 0) continue;
            if (__builtin_amdgcn_inverse_ballot_w64(pb)) {
                const int at = hn + lanes_below_u64(pb);
                Q.hg[at] = (uint16_t)gl;
                if constexpr (DT == TSB_BF16) Q.hw[at] = ent;
            }
            hn += __popcll(pb);
            if (hn > kHitCap - kWave) {
                wave_lds_fence();
                list_hits<DT, VEC>(A, I, lane, Q, hn, top);
                listed = true;
                hn = 0;
                // with m keys kept, the tile's m-th best is a bound too: fewer
                // of the groups after these pass (a parent that is not pruned
                // keeps its -inf: every token of its row is scored)
                if (I.thr > -INFINITY && top.thr != 0ull && cand_value(top.thr) > I.thr) {
                    I.thr = cand_value(top.thr);
                    I.bound = I.thr - kGumbelMaxBound;
                    wt.init(I.thr, I.cd, invT);
                    if (DT == TSB_BF16) lt.init(I.bound, I.cd, invT);
                }
                wave_lds_fence();  // the list of hits is rewritten
            }
        }
        wave_lds_fence();  // the queue is rewritten by the next pass
    }
    const size_t o = (size_t)node * (size_t)T + t;
    int cnt = 0;
    if (!listed && hn > 0) {
        // the usual end: at most 64 hits, whose keys that reach thr go
        // straight to the slots
        float kv[4];
        int g;
        uint64_t kb[4];
        hit_keys<DT, VEC>(A, I, lane, Q, 0, hn, kv, g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kb[e] = __builtin_amdgcn_ballot_w64(kv[e] > -INFINITY);
            cnt += __popcll(kb[e]);
        }
        if (cnt > m) {
            // more than the merge can use: keep what reaches the m-th largest
            // of the lane maxima (lanes hold distinct tokens), m keys or a few more
            const float lo = wave_kth_largest(fmaxf(fmaxf(kv[0], kv[1]), fmaxf(kv[2], kv[3])), m);
            cnt = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!(kv[e] >= lo)) kv[e] = -INFINITY;
                kb[e] = __builtin_amdgcn_ballot_w64(kv[e] > -INFINITY);
                cnt += __popcll(kb[e]);
            }
        }
        listed = cnt > TSB_MAX_K;
        if (!listed) {
            int at = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (kv[e] > -INFINITY)
                    A.out_cand[o * TSB_MAX_K + at + lanes_below_u64(kb[e])] =
                        cand_key(kv[e], (uint32_t)(I.t0 + g * 4 + e));
                at += __popcll(kb[e]);
            }
        }
    }
    if (listed) {
        if (hn > 0) list_hits<DT, VEC>(A, I, lane, Q, hn, top);
        cnt = __popcll(__ballot(lane < m && top.v != 0ull));
        if (lane < cnt) A.out_cand[o * TSB_MAX_K + lane] = top.v;
    }
    if (lane == 0) A.out_cnt[o] = cnt;
    C.add(0, 1, lane);
    C.add(1, (unsigned)I.tn, lane);
}

template <int DT, bool VEC>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(VEC ? 7 : 6))) void replay_scan(ScanArgs A, const int* __restrict__ ptotal,
                                                      unsigned long long* __restrict__ stats) {
    __shared__ ScanQueue s_queue[kScanWaves];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const long long items = (long long)ptotal[0] * A.T;
    const long long nw = (long long)gridDim.x * kScanWaves;
    __shared__ unsigned long long s_cnt[kScanWaves][4];
    const ScanCounters C = scan_counters(s_cnt, wave, lane, stats);
    for (long long it = (long long)blockIdx.x * kScanWaves + wave; it < items; it += nw)
        scan_item<DT, VEC>(A, it, lane, s_queue[wave], C);
    C.flush(stats, lane);
}

// The scan and the target stream of verification in one grid: the first nt
// workgroups stream the target (the job's chunks dealt over them) and the
// others scan (items dealt grid-stride over the scan's workgroups, as in
// replay_scan). The target's workgroups come first, so they are dispatched
// first and every compute unit mixes the target's HBM stream with the
// scan's VALU work; the scan's workgroups beyond what fits start as others
// finish.
template <int DT, bool VEC, bool TVEC>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(VEC ? 7 : 6))) void replay_scan_target(ScanArgs A, const int* __restrict__ ptotal,
                                                             unsigned long long* __restrict__ stats, TargetJob job,
                                                             int nt) {
    if ((int)blockIdx.x < nt) {
        // chunks blockIdx.x, blockIdx.x + nt, ... of the job
        XRegion X;
        X.slots = job.slots;
        for (int g = blockIdx.x; g < job.ngroups; g += nt)
            target_chunk<DT, TVEC, kFusedTargetPrefetch>(g, job.ngroups, job.target, A.V, A.B, job.nrows, job.chunk, job.P, A.invT,
                                   job.n_nodes, job.tm, job.ts, job.tf, X, job.R);
        return;
    }
    __shared__ ScanQueue s_queue[kScanWaves];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const long long items = (long long)ptotal[0] * A.T;
    const int sb = (int)blockIdx.x - nt;
    const long long nw = (long long)((int)gridDim.x - nt) * kScanWaves;
    __shared__ unsigned long long s_cnt[kScanWaves][4];
    const ScanCounters C = scan_counters(s_cnt, wave, lane, stats);
    for (long long it = (long long)sb * kScanWaves + wave; it < items; it += nw)
        scan_item<DT, VEC>(A, it, lane, s_queue[wave], C);
    C.flush(stats, lane);
}

template <int DT>
__global__ __launch_bounds__(kWave) void replay_merge(int B, int D, int K, int T, tsb_tree tree,
                                                      const uint64_t* __restrict__ cand, const int* __restrict__ cc,
                                                      int32_t* __restrict__ node_tok, const void* __restrict__ draft,
                                                      int V, float invT, TargetJob job) {
    const int r = blockIdx.y;
    const int u = blockIdx.x;
    const int lane = threadIdx.x;
    const size_t tb = (size_t)r * (B + 1);
    const int nn = tree.n_nodes[r];
    const int n = tree_count_ok(nn, B) ? nn : 0;
    if (u == 0 || u >= n) {
        if (lane == 0) node_tok[tb + u] = -1;
    }
    NodeHead head;
    if (job.nrec && u < n) {
        head = node_head(tree, job.draft_lse, r, u, n, tb, D, lane);
        if (job.nrows > 0) {
            head.L0 = target_row_lse(job.tm, job.ts, job.tf, job.P, tb + u, &head.bad);
            head.l0 = true;
        }
    }
    TreeNode nd;
    if (!replay_parent(tree, r, u, B, D, K, &nd)) {
        if (job.nrec && u < n) {
            // a leaf, or a node replay leaves alone: its children (if any) keep
            // the tokens the caller's topology gave them
            const TreeNode& t = head.t;
            const int tok = (t.ok && lane < t.m) ? node_tok[tb + t.fc + lane] : -1;
            write_record<DT>(job.nrec, head, draft, job.target, V, D, invT, r, tb + u, tok, lane);
        }
        return;
    }
    const int m = nd.m;
    const int fc = nd.fc;
    // the children's tokens (lane j < m: child j), then the node record
    auto finish = [&](int tok) {
        if (lane < m) node_tok[tb + fc + lane] = tok;
        if (job.nrec) write_record<DT>(job.nrec, head, draft, job.target, V, D, invT, r, tb + u, tok, lane);
    };
    const size_t o = (tb + u) * (size_t)T;
    // 64 tiles at a time, lane t holds tile t's count; the keys of their slots
    // (in no order) are gathered contiguously, their indices placed through LDS
    // (reading every slot of 65 tiles took 21.5 us for one request of 65 nodes
    // and 29.3 for 16 of 129, gathering them 11.6 and 17.9)
    __shared__ uint16_t s_idx[kWave * TSB_MAX_K];
    __shared__ uint64_t s_key[kWave];
    auto gather = [&](int t0) -> int {
        const int ct = t0 + lane < T ? cc[o + t0 + lane] : 0;
        int nv = 0;
        for (int j = 0;; ++j) {
            const uint64_t bj = __ballot(j < ct);
            if (!bj) break;
            if (j < ct) s_idx[nv + lanes_below_u64(bj)] = (uint16_t)(lane * TSB_MAX_K + j);
            nv += __popcll(bj);
        }
        wave_lds_fence();
        return nv;
    };
    int nv = gather(0);
    const uint64_t* cb = cand + o * TSB_MAX_K;
    // the keys are loaded together, up to kMergeKeys a lane. The m-th
    // largest of the lane maxima is a lower bound of the m-th key (lanes hold
    // distinct keys): the few keys that reach it are compacted, one per lane,
    // and a key's rank is the number of larger ones. (A sort of 64 keys takes
    // about 1.3 us here, an insert 0.15 us.)
    constexpr int kMergeKeys = 12;
    if (T <= kWave && nv <= kMergeKeys * kWave) {
        uint64_t kb[kMergeKeys], mx = 0ull;
#pragma unroll
        for (int q = 0; q < kMergeKeys; ++q) {
            const int e = q * kWave + lane;
            kb[q] = e < nv ? cb[s_idx[e]] : 0ull;
        }
        int c = nv;
        uint64_t mine = kb[0];
        if (nv > kWave) {
#pragma unroll
            for (int q = 0; q < kMergeKeys; ++q) mx = kb[q] > mx ? kb[q] : mx;
            const uint32_t hi = (uint32_t)(mx >> 32);
            int above = 0;
            for (int l = 0; l < kWave; ++l) above += lane_u32(hi, l) > hi ? 1 : 0;
            // the smallest of the maxima with fewer than m above them
            uint32_t lo = above < m ? hi : 0xFFFFFFFFu;
#pragma unroll
            for (int f = 32; f > 0; f >>= 1) lo = min(lo, xor_lane_red_u32(lo, f));
            c = 0;
#pragma unroll
            for (int q = 0; q < kMergeKeys; ++q) {
                const bool keep = (uint32_t)(kb[q] >> 32) >= lo;
                const uint64_t b = __ballot(keep);
                const int at = c + lanes_below_u64(b);
                if (keep && at < kWave) s_key[at] = kb[q];
                c += __popcll(b);
            }
            wave_lds_fence();
            mine = lane < c ? s_key[lane] : 0ull;
            wave_lds_fence();
        }
        if (c <= kWave) {
            int rank = 0;
            for (int l = 0; l < c; ++l) rank += lane_u64(mine, l) > mine ? 1 : 0;
            if (lane < c) s_key[rank] = mine;
            wave_lds_fence();
            finish((int32_t)cand_id(lane < c ? s_key[lane] : 0ull));
            return;
        }
    }
    // more keys than that, ties of their upper halves, or more tiles: inserted
    // in batches of 64, the loads of several in flight together
    WaveTopList top;
    top.init(m);
    constexpr int kMergeBatches = 8;
    for (int t0 = 0;;) {
        for (int b0 = 0; b0 < nv; b0 += kMergeBatches * kWave) {
            uint64_t kb[kMergeBatches];
#pragma unroll
            for (int q = 0; q < kMergeBatches; ++q) {
                const int e = b0 + q * kWave + lane;
                kb[q] = e < nv ? cb[s_idx[e]] : 0ull;
            }
#pragma unroll
            for (int q = 0; q < kMergeBatches; ++q) top.offer(kb[q], kb[q] != 0);
        }
        t0 += kWave;
        if (t0 >= T) break;
        wave_lds_fence();  // the next tiles' indices take their place
        nv = gather(t0);
        cb += kWave * TSB_MAX_K;
    }
    finish((int32_t)cand_id(top.v));
}

// Workgroups of the scan. The item count (parents x tiles) is only known on
// the device; about a quarter of the nodes have children, so this is about
// one item per wave: the hardware then deals the items as workgroups finish
// (their costs differ fivefold with the row's spread). At 64 x 257 nodes
// 16384 workgroups take 5% less than 4096, at 16 x 129 4128 as long as 2048.
static int scan_workgroups(const tsb_config& c, const Geometry& g) {
    const long long n = (long long)c.R * (c.B + 1) * g.T / (4 * kScanWaves);
    return (int)std::min<long long>(kScanWorkgroupsMax, std::max<long long>(kScanWorkgroupsMin, n));
}

hipError_t launch_replay(const tsb_config& c, float invT, const void* draft, const int32_t* topk_tok,
                         const tsb_tree& tree, uint32_t step, int32_t* node_tok, char* ws, hipStream_t st,
                         const TargetJob* tj) {
    const Geometry g = geometry(c);
    const ReplayWs w = replay_ws(c);
    uint64_t* cand = (uint64_t*)(ws + w.cand);
    int* cc = (int*)(ws + w.cnt);
    int* plist = (int*)(ws + w.plist);
    int* ptotal = (int*)(ws + w.ptotal);
    const uint32_t k0 = (uint32_t)c.seed, k1 = (uint32_t)(c.seed >> 32);
    const int prune = (c.flags & TSB_FLAG_NO_PRUNE) ? 0 : 1;
    const bool vec = c.V % 4 == 0 && ((uintptr_t)draft & 15) == 0;
    float4* rec = (float4*)(ws + w.thr);
    // the parent list's workgroups, and one per four nodes
    const int nodes = c.R * (c.B + 1);
    const ListSplit list = list_split(nodes);
    const int nthr = list.groups + (nodes + kBlock / kWave - 1) / (kBlock / kWave);
    if (c.dtype == TSB_BF16)
        replay_threshold<TSB_BF16><<<nthr, kBlock, 0, st>>>(draft, c.R, c.V, c.D, c.B, c.K, invT, topk_tok, tree, k0,
                                                            k1, step, prune, vec ? 1 : 0, rec, plist, ptotal, list);
    else
        replay_threshold<TSB_F32><<<nthr, kBlock, 0, st>>>(draft, c.R, c.V, c.D, c.B, c.K, invT, topk_tok, tree, k0,
                                                           k1, step, prune, vec ? 1 : 0, rec, plist, ptotal, list);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int scan_id = tj ? TSB_KERNEL_SCAN_TARGET : TSB_KERNEL_REPLAY_SCAN;
    if ((e = hook_before(scan_id, st)) != hipSuccess) return e;
    unsigned long long* const stats = stats_ptr();
    ScanArgs A{draft, c.V, c.D, c.B, g.T, invT, plist, rec, k0, k1, step, cand, cc};
    if (tj) {
        const int nt = std::min(tj->ngroups, kFusedTargetWorkgroups);
        const int nscan = scan_workgroups(c, g);
        const int grid = nt + nscan;
        const bool tv = tj->vec;
        if (c.dtype == TSB_BF16) {
            auto fn = vec ? (tv ? replay_scan_target<TSB_BF16, true, true> : replay_scan_target<TSB_BF16, true, false>)
                          : (tv ? replay_scan_target<TSB_BF16, false, true> : replay_scan_target<TSB_BF16, false, false>);
            fn<<<grid, kBlock, 0, st>>>(A, ptotal, stats, *tj, nt);
        } else {
            auto fn = vec ? (tv ? replay_scan_target<TSB_F32, true, true> : replay_scan_target<TSB_F32, true, false>)
                          : (tv ? replay_scan_target<TSB_F32, false, true> : replay_scan_target<TSB_F32, false, false>);
            fn<<<grid, kBlock, 0, st>>>(A, ptotal, stats, *tj, nt);
        }
    } else {
        const int grid = scan_workgroups(c, g);
        auto fn = c.dtype == TSB_BF16 ? (vec ? replay_scan<TSB_BF16, true> : replay_scan<TSB_BF16, false>)
                                      : (vec ? replay_scan<TSB_F32, true> : replay_scan<TSB_F32, false>);
        fn<<<grid, kBlock, 0, st>>>(A, ptotal, stats);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = hook_after(scan_id, st)) != hipSuccess) return e;
    if ((e = hook_before(TSB_KERNEL_REPLAY_MERGE, st)) != hipSuccess) return e;
    TargetJob none{};
    const TargetJob& rj = tj ? *tj : none;  // node records only in a whole round
    if (c.dtype == TSB_BF16)
        replay_merge<TSB_BF16><<<dim3(c.B + 1, c.R), kWave, 0, st>>>(c.B, c.D, c.K, g.T, tree, cand, cc, node_tok,
                                                                     draft, c.V, invT, rj);
    else
        replay_merge<TSB_F32><<<dim3(c.B + 1, c.R), kWave, 0, st>>>(c.B, c.D, c.K, g.T, tree, cand, cc, node_tok,
                                                                    draft, c.V, invT, rj);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return hook_after(TSB_KERNEL_REPLAY_MERGE, st);
}

}  // namespace tsb
