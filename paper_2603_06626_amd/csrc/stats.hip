// Routing statistics computed from cached top-k expert ids (integer work, one pass over the ids each):
//   * per-sample routing affinity counts, their entropy, expert loads and the maximal violation
//     (Sec. 3.3.2 first equation; App. "Efficiency Experiment Detail", expert grouping; App. "Maximal Violation")
//   * sample placement: per (sample, node) the number of tokens that find an expert on the node, and the
//     best node (App. "Efficiency Experiment Detail", algorithm "Optimize Sample-to-Node Assignment")
//   * expert folding: co-activation matrix, greedy affinity grouping, folded score weights (Sec. 3.2.1)
//
// The per-sample statistics (affinity counts, entropy, loads, placement) come from one kernel that reads every id
// once: a lane takes one token, loads its k ids with one coalesced access (8 bytes for the cached format of
// k = 8 one-byte ids), counts membership with LDS atomics and votes per node with wave ballots.  (The co-activation
// matrix has a file of its own.)  Membership is an indicator per token: an id repeated inside a token counts once, ids outside
// [0,E) are ignored.  Integer arithmetic throughout, so every result is bit-reproducible.
#include <type_traits>

#include "stats_ids.hpp"

namespace grouter {

namespace {

constexpr int kStatThreads = 256;
constexpr int kMaxStatK = 64;           // a token's validity mask is one 64-bit word

// Bit j of the result is set when slot j of the token holds an id in [0,E) that no earlier slot holds.
template <class IdxT>
__device__ __forceinline__ uint64_t unique_slots(const IdxT* ids, int k, int E) {
    uint64_t m = 0;
    for (int j = 0; j < k; ++j) {
        const int64_t e = (int64_t)ids[j];
        bool ok = e >= 0 && e < E;
#pragma unroll 4
        for (int i = 0; i < j; ++i) ok &= (int64_t)ids[i] != e;   // no early exit: the loads of a round are independent
        if (ok) m |= 1ull << j;
    }
    return m;
}

// ---------------------------------------------------------------------------------------------------
// Fast path for k <= 8 (the paper's models route to 8 or fewer experts): the ids of token t live in registers,
// e[j] = id of slot j, or -1 when the slot does not exist, is out of range, or repeats an earlier slot.
// One 8-byte access for the cached format (uint8, k = 8), two 16-byte ones for int32 ids with k = 8.
// (Fetched and decoded in two functions: written as one, it compiles to longer code that takes 2 to 5 % more on short samples.)
struct RawIds8 {   // the k <= 8 ids of one token as fetched, before range check and de-duplication
    int e[8];
};
template <class IdxT>
__device__ __forceinline__ RawIds8 fetch_token8(const IdxT* __restrict__ base, int64_t t, int k) {
    RawIds8 r;
    const IdxT* ids = base + t * k;
    if (sizeof(IdxT) == 1 && k == 8 && (reinterpret_cast<uintptr_t>(base) & 7u) == 0) {
        const uint2 w = *reinterpret_cast<const uint2*>(ids);
        r.e[0] = (int)w.x;      // unpacked by decode_token8
        r.e[1] = (int)w.y;
    } else if (sizeof(IdxT) == 4 && k == 8 && (reinterpret_cast<uintptr_t>(base) & 15u) == 0) {
        const int4 a = reinterpret_cast<const int4*>(ids)[0], b = reinterpret_cast<const int4*>(ids)[1];
        r.e[0] = a.x; r.e[1] = a.y; r.e[2] = a.z; r.e[3] = a.w;
        r.e[4] = b.x; r.e[5] = b.y; r.e[6] = b.z; r.e[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) r.e[j] = j < k ? (int)ids[j] : -1;
    }
    return r;
}
template <class IdxT>
__device__ __forceinline__ void decode_token8(const IdxT* __restrict__ base, const RawIds8& r, int k, int E, int (&e)[8]) {
    if (sizeof(IdxT) == 1 && k == 8 && (reinterpret_cast<uintptr_t>(base) & 7u) == 0) {
        const uint32_t x = (uint32_t)r.e[0], y = (uint32_t)r.e[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            e[j] = (int)((x >> (8 * j)) & 0xffu);
            e[4 + j] = (int)((y >> (8 * j)) & 0xffu);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = r.e[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (e[j] < 0 || e[j] >= E) e[j] = -1;
#pragma unroll
    for (int j = 1; j < 8; ++j) {
        bool dup = false;
#pragma unroll
        for (int i = 0; i < j; ++i) dup = dup || (e[i] == e[j]);
        if (dup) e[j] = -1;
    }
}
template <class IdxT>
__device__ __forceinline__ void load_token8(const IdxT* __restrict__ base, int64_t t, int k, int E, int (&e)[8]) {
    decode_token8(base, fetch_token8(base, t, k), k, E, e);
}

// Entropy of a sample's counts in bits: H = -sum p log2 p with p = c / n, i.e. log2(n) - (sum c log2 c) / n, from every
// thread's part of n and of the sum; in thread 0.  The order of the additions is fixed.
__device__ __forceinline__ double block_entropy(long long tot, double clogc, double* s_red, long long* s_tot, int tid) {
    for (int o = 32; o > 0; o >>= 1) {
        clogc += __shfl_xor(clogc, o);
        tot += __shfl_xor(tot, o);
    }
    if ((tid & 63) == 0) {
        s_red[tid >> 6] = clogc;
        s_tot[tid >> 6] = tot;
    }
    __syncthreads();
    double sum = 0.0;
    long long n = 0;
    for (int w = 0; w < kStatThreads / 64; ++w) {
        sum += s_red[w];
        n += s_tot[w];
    }
    return n > 0 ? log2((double)n) - sum / (double)n : 0.0;
}

// One workgroup per sample, one pass over its ids for both statistics:
//   AFF    histogram of token membership, entropy of the normalised histogram (fp64, fixed summation order)
//   PLACE  expert_nodes[e] has bit n set when expert e lives on node n, so the nodes a token reaches are the OR
//          over its experts; per node the wave counts its lanes with one ballot
// WIDE: k > 8.  Apart, because what one of the two forms needs in registers costs the other occupancy.  2048 samples of 4096
// tokens (512 for k = 16), E = 128, placement alone: k = 8 45 us as one
// kernel, 40 apart; k = 16 285 -> 190 with the independent loads (affinity 287, then 298 for a while -> 201).
template <class IdxT, bool AFF, bool PLACE, bool WIDE>
__global__ __launch_bounds__(kStatThreads) void k_sample_stats(const IdxT* __restrict__ idx, int L, int k, int E,
                                                               int32_t* __restrict__ counts, double* __restrict__ entropy,
                                                               const uint64_t* __restrict__ expert_nodes, int n_nodes,
                                                               int32_t* __restrict__ comm, int32_t* __restrict__ best_node) {
    __shared__ int32_t s_hist[AFF ? kMaxExperts : 1];
    __shared__ uint64_t s_nodes[PLACE ? kMaxExperts : 1];
    __shared__ int32_t s_comm[64];
    __shared__ double s_red[kStatThreads / 64];
    __shared__ long long s_tot[kStatThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t s = blockIdx.x;
    if (AFF)
        for (int e = tid; e < E; e += kStatThreads) s_hist[e] = 0;
    if (PLACE) {
        for (int e = tid; e < E; e += kStatThreads) s_nodes[e] = expert_nodes[e];
        if (tid < 64) s_comm[tid] = 0;
    }
    __syncthreads();
    const IdxT* base = idx + (size_t)s * L * k;
    int acc = 0;  // PLACE: lane n of every wave counts node n
    // whole waves take part in every ballot: the loop bound is rounded up to the workgroup size
    for (int tb = 0; tb < L; tb += kStatThreads) {
        const int t = tb + tid;
        uint64_t reach = 0;
        if (t < L) {
            if constexpr (!WIDE) {
                int e[8];
                load_token8(base, t, k, E, e);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (e[j] >= 0) {
                        if (AFF) atomicAdd(&s_hist[e[j]], 1);
                        if (PLACE) reach |= s_nodes[e[j]];
                    }
            } else {
                const IdxT* ids = base + (size_t)t * k;
                const uint64_t m = unique_slots(ids, k, E);
                for (int j = 0; j < k; ++j)
                    if ((m >> j) & 1) {
                        if (AFF) atomicAdd(&s_hist[(int)ids[j]], 1);
                        if (PLACE) reach |= s_nodes[(int)ids[j]];
                    }
            }
        }
        if (PLACE)
            for (int n = 0; n < n_nodes; ++n) {
                const uint64_t b = __ballot((reach >> n) & 1);
                if (lane == n) acc += __popcll(b);
            }
    }
    if (PLACE && lane < n_nodes && acc) atomicAdd(&s_comm[lane], acc);
    __syncthreads();
    if (PLACE) {
        if (tid < n_nodes) comm[s * n_nodes + tid] = s_comm[tid];
        if (tid == 0) {
            int best = 0, mx = -1;
            for (int n = 0; n < n_nodes; ++n)
                if (s_comm[n] > mx) {
                    mx = s_comm[n];
                    best = n;
                }
            best_node[s] = best;
        }
    }
    if (!AFF) return;
    long long tot = 0;
    double clogc = 0.0;
    for (int e = tid; e < E; e += kStatThreads) {
        const int c = s_hist[e];
        counts[s * E + e] = c;
        if (c > 0) {
            tot += c;
            clogc += (double)c * log2((double)c);
        }
    }
    const double h = block_entropy(tot, clogc, s_red, s_tot, tid);
    if (tid == 0) entropy[s] = h;
}

// The same for k <= 8, E <= 247, at most 16 nodes and samples of at most 255 * 256 tokens that are long enough (packed_pays).
// The general kernel above is bound by LDS bank conflicts (64 lanes add to and look up random experts: about five rounds per
// access) and by 28 compares per token.  Here
//   * a word of the table is (node set << 16 | count) and there are R columns of them: per id one read that tells the nodes and one
//     add that returns nothing (together cheaper than one that returns the word).  R = 64 up to 128 experts: every lane of a wave
//     has a column of its own and no access conflicts.  R = 32 beyond, where 64 would not leave room for four workgroups on a
//     CU: lanes l and l + 32 share a column, two rounds per access at most;
//   * the ids of the next two tokens are on their way while one is counted, and all its reads are issued before the first is used;
//   * ids that do not count (out of range, repeated, tokens past the end) go to a spare row;
//   * repeats are detected four bytes at a time on the packed ids; only a wave that has one compares slot by slot;
//   * a lane keeps its votes per node as bytes and adds them up at the end.
// Measured, both statistics (a call of three launches; general kernel / this one with returning adds and one token ahead / now):
// 2048 x 4096 tokens, k = 8, uint8, 4 nodes, E = 128 86 / 45.6 / 40 us; 700 x 3000, k = 5, uint8, E = 200 - / 22.5 / 19; 512 x 2048,
// k = 8, int32, E = 128 - / 16.2 / 14.7.
constexpr int kFastStatE = 247, kFastStatNodes = 16, kFastStatL = 255 * kStatThreads;

// nonzero if two of the eight bytes of (x, y) are equal
__device__ __forceinline__ uint32_t equal_bytes8(uint32_t x, uint32_t y) {
    auto rot = [](uint32_t v, int n) { return __builtin_amdgcn_alignbyte(v, v, n); };
    auto zero_bytes = [](uint32_t v) { return (v - 0x01010101u) & ~v; };   // bit 7 of the lowest zero byte is set
    const uint32_t y1 = rot(y, 1), y2 = rot(y, 2);
    const uint32_t z = zero_bytes(x ^ y) | zero_bytes(x ^ y1) | zero_bytes(x ^ y2) | zero_bytes(x ^ rot(y, 3)) |
                       zero_bytes(x ^ rot(x, 1)) | zero_bytes(x ^ rot(x, 2)) | zero_bytes(y ^ y1) | zero_bytes(y ^ y2);
    return z & 0x80808080u;
}

template <class IdxT, bool AFF, bool PLACE, int R>
__global__ __launch_bounds__(kStatThreads) void k_sample_stats8(const IdxT* __restrict__ idx, int64_t S, int L, int k, int E,
                                                                int32_t* __restrict__ counts, double* __restrict__ entropy,
                                                                const uint64_t* __restrict__ expert_nodes, int n_nodes,
                                                                int32_t* __restrict__ comm, int32_t* __restrict__ best_node) {
    constexpr int kRows = (R == 64 ? 128 : kFastStatE) + 1;
    __shared__ __attribute__((aligned(16))) uint32_t s_tab[kRows * R];
    __shared__ int32_t s_cnt[kRows];
    __shared__ int32_t s_comm[kFastStatNodes];
    __shared__ double s_red[kStatThreads / 64];
    __shared__ long long s_tot[kStatThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t s = blockIdx.x;
    const IdxT* const base = idx + (size_t)s * L * k;
    using Ids = IdWindow<IdxT, 8>;
    const int last = (int)min((S - s) * L * k - Ids::kWindow, (int64_t)0x7fffffff);
    Ids ids[2];   // the next two tokens of this lane
    // past the sample's end its last token is fetched again, not the next sample's, which then came from memory twice (k = 8, int32,
    // E = 128, both statistics: 2048 samples of 2048 tokens 37.2 -> 34.4 us, of 1100 tokens 32.8 -> 28.0; 1024 of 1024 17.8 -> 15.9)
    auto fetch = [&](Ids& window, int t) { window.fetch(base, min(t, L - 1) * k, last); };
    fetch(ids[0], tid);
    fetch(ids[1], tid + kStatThreads);
    if (!PLACE) {
        for (int i = tid; i < (E + 1) * (R / 4); i += kStatThreads) reinterpret_cast<uint4*>(s_tab)[i] = uint4{0u, 0u, 0u, 0u};
    } else if (tid <= E) {   // a thread fills a row, so that it loads one node set; each begins at another bank
        const uint32_t w = tid < E ? (uint32_t)expert_nodes[tid] << 16 : 0u;
#pragma unroll
        for (int q = 0; q < R / 4; ++q) reinterpret_cast<uint4*>(s_tab)[tid * (R / 4) + ((q + tid) & (R / 4 - 1))] = uint4{w, w, w, w};
    }
    if (tid <= E) s_cnt[tid] = 0;
    if (tid < kFastStatNodes) s_comm[tid] = 0;
    __syncthreads();
    uint32_t* const column = s_tab + (lane & (R - 1));
    uint32_t votes[4] = {0u, 0u, 0u, 0u};
    // bytes of slots past k: values that no expert has
    const uint32_t keep_x = k >= 4 ? ~0u : (1u << (8 * k)) - 1u, keep_y = k >= 8 ? ~0u : k <= 4 ? 0u : (1u << (8 * (k - 4))) - 1u;
    auto turn = [&](Ids& window, int t) {
        window.settle();
        uint32_t e[8], x, y;
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = t < L && j < k ? min(window.id(j), (uint32_t)E) : (uint32_t)E;
        if constexpr (sizeof(IdxT) == 1) {
            x = window.w[0];
            y = window.w[1];
        } else {
            x = e[0] | (e[1] << 8) | (e[2] << 16) | (e[3] << 24);
            y = e[4] | (e[5] << 8) | (e[6] << 16) | (e[7] << 24);
        }
        x = (x & keep_x) | (0xfbfaf9f8u & ~keep_x);
        y = (y & keep_y) | (0xfffefdfcu & ~keep_y);
        fetch(window, t + 2 * kStatThreads);
        if (__any(t < L && equal_bytes8(x, y))) {
#pragma unroll
            for (int j = 1; j < 8; ++j) {
                bool dup = false;
#pragma unroll
                for (int i = 0; i < j; ++i) dup = dup || (e[i] == e[j]);
                if (dup) e[j] = E;
            }
        }
        // all reads, then all adds; slots past k go to the spare row too (with a branch per slot every read was waited for)
        uint32_t seen = 0;
        auto slots = [&](auto n) {
            constexpr int N = decltype(n)::value;
            uint32_t word[N];
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (PLACE) word[j] = column[e[j] * R];
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (AFF) atomicAdd(&column[e[j] * R], 1u);   // (the returned word would cost twice a read and an add without)
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (PLACE) seen |= word[j];
        };
        if (k > 4) slots(std::integral_constant<int, 8>{});
        else slots(std::integral_constant<int, 4>{});
        if (PLACE) {
            const uint32_t reach = seen >> 16;
#pragma unroll
            for (int q = 0; q < 4; ++q)   // four bits to four bytes
                if (4 * q < n_nodes) votes[q] += (((reach >> (4 * q)) & 15u) * 0x00204081u) & 0x01010101u;
        }
    };
    int t0 = 0;
    for (; t0 + kStatThreads < L; t0 += 2 * kStatThreads) {
        turn(ids[0], t0 + tid);
        turn(ids[1], t0 + kStatThreads + tid);
    }
    if (t0 < L) turn(ids[0], t0 + tid);
    if (PLACE) {
        // four byte counts become two words of two 16-bit sums (at most 64 * 255 each), which are added over the wave: chains that
        // run side by side instead of one after the other per node (32 samples of 256 tokens, 16 nodes: 13.1 -> 9.8 us)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (4 * q < n_nodes) {
                uint32_t even = votes[q] & 0x00ff00ffu, odd = (votes[q] >> 8) & 0x00ff00ffu;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) {
                    even += __shfl_xor(even, o);
                    odd += __shfl_xor(odd, o);
                }
                if (lane < 4 && 4 * q + lane < n_nodes) atomicAdd(&s_comm[4 * q + lane], (int)(((lane & 1 ? odd : even) >> (lane & 2 ? 16 : 0)) & 0xffffu));
            }
    }
    __syncthreads();
    if (PLACE) {
        if (tid < n_nodes) comm[s * n_nodes + tid] = s_comm[tid];
        if (tid == 64) {
            int best = 0, mx = -1;
            for (int n = 0; n < n_nodes; ++n)
                if (s_comm[n] > mx) {
                    mx = s_comm[n];
                    best = n;
                }
            best_node[s] = best;
        }
    }
    if (!AFF) return;
    // columns -> counts: a thread adds 16 words of a row (starting points rotated, so that the lanes use all banks)
    constexpr int kParts = R / 16;
    for (int i = tid; i < E * kParts; i += kStatThreads) {
        uint32_t v = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 w = reinterpret_cast<const uint4*>(s_tab)[i * 4 + ((q + (i >> 2)) & 3)];
            v += w.x + w.y + w.z + w.w;
        }
        const int e = i / kParts;
        if (PLACE) v -= ((uint32_t)expert_nodes[e] << 16) * 16u;   // modulo 2^32; the count itself is below 2^16
        atomicAdd(&s_cnt[e], (int)v);
    }
    __syncthreads();
    long long tot = 0;
    double clogc = 0.0;
    if (tid < E) {
        const int c = s_cnt[tid];
        counts[s * E + tid] = c;
        if (c > 0) {
            tot = c;
            clogc = (double)c * log2((double)c);
        }
    }
    const double h = block_entropy(tot, clogc, s_red, s_tot, tid);
    if (tid == 0) entropy[s] = h;
}

// loads[e] = sum over the samples of counts[s][e].  A workgroup owns 16 experts (one 64-byte segment of every row).
constexpr int kLoadsCols = 16, kLoadsThreads = 1024;
__global__ __launch_bounds__(kLoadsThreads) void k_loads(const int32_t* __restrict__ counts, int64_t S, int E,
                                                         unsigned long long* __restrict__ loads) {
    __shared__ unsigned long long s_sum[kLoadsThreads];
    const int tid = threadIdx.x, e = (int)blockIdx.x * kLoadsCols + tid % kLoadsCols;
    unsigned long long v = 0;
    if (e < E)
#pragma unroll 8
        for (int64_t s = tid / kLoadsCols; s < S; s += kLoadsThreads / kLoadsCols) v += (unsigned long long)counts[s * E + e];
    s_sum[tid] = v;
    __syncthreads();
    for (int w = kLoadsThreads / 2; w >= kLoadsCols; w >>= 1) {
        if (tid < w) s_sum[tid] += s_sum[tid + w];
        __syncthreads();
    }
    if (tid < kLoadsCols && e < E) loads[e] = s_sum[tid];
}

// loads and maxvio of few samples in one workgroup (one launch instead of two, 4 us): thread t adds up column t % E.
__global__ __launch_bounds__(kLoadsThreads) void k_loads_maxvio(const int32_t* __restrict__ counts, int S, int E,
                                                                unsigned long long* __restrict__ loads, double* __restrict__ out) {
    __shared__ unsigned long long s_sum[kLoadsThreads], s_max[kLoadsThreads];
    const int tid = threadIdx.x, per = kLoadsThreads / E;   // rows side by side
    unsigned long long v = 0;
    if (tid < per * E)
#pragma unroll 8
        for (int i = tid; i < S * E; i += per * E) v += (unsigned long long)counts[i];
    s_sum[tid] = v;
    __syncthreads();
    v = 0;
    if (tid < E) {
        for (int r = 0; r < per; ++r) v += s_sum[r * E + tid];
        loads[tid] = v;
    }
    __syncthreads();
    s_sum[tid] = v;
    s_max[tid] = v;
    __syncthreads();
    for (int w = kLoadsThreads / 2; w > 0; w >>= 1) {
        if (tid < w) {
            s_max[tid] = s_max[tid + w] > s_max[tid] ? s_max[tid + w] : s_max[tid];
            s_sum[tid] += s_sum[tid + w];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double mean = (double)s_sum[0] / (double)E;
        out[0] = s_sum[0] > 0 ? ((double)s_max[0] - mean) / mean : 0.0;
    }
}

// (max L - mean L) / mean L over the E loads; one workgroup.
__global__ __launch_bounds__(kStatThreads) void k_maxvio(const unsigned long long* __restrict__ loads, int E,
                                                         double* __restrict__ out) {
    __shared__ unsigned long long s_max[kStatThreads], s_sum[kStatThreads];
    const int tid = threadIdx.x;
    unsigned long long mx = 0, sum = 0;
    for (int e = tid; e < E; e += kStatThreads) {
        const unsigned long long v = loads[e];
        mx = v > mx ? v : mx;
        sum += v;
    }
    s_max[tid] = mx;
    s_sum[tid] = sum;
    __syncthreads();
    for (int w = kStatThreads / 2; w > 0; w >>= 1) {
        if (tid < w) {
            s_max[tid] = s_max[tid + w] > s_max[tid] ? s_max[tid + w] : s_max[tid];
            s_sum[tid] += s_sum[tid + w];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double mean = (double)s_sum[0] / (double)E;
        out[0] = s_sum[0] > 0 ? ((double)s_max[0] - mean) / mean : 0.0;
    }
}

// ---------------------------------------------------------------------------------------------------
// Greedy affinity grouping.  Groups are filled one after the other; a group starts with the lowest unassigned expert, then
// takes the unassigned expert with the largest summed co-activation with its members (lowest number on ties): a serial
// chain of E_S rounds, so what counts is the length of one round.
//
// Up to 256 experts one wave runs it, lane l holding the experts l, l + 64, ...: a round is a maximum over the wave in six
// DPP steps, and one row of the matrix from LDS, staged by the whole workgroup first, or L2.  No barrier is involved.  Score and
// expert make one key, of 32 bits where scores stay below 2^24, of 64 below 2^54; larger ones are compared as they are, and
// ballots find who holds the maximum.
// Measured, a workgroup with three barriers per round / doubles and ballots, staged where they fit, or int64 from L2 / now.  Scores below
// 2^24: 128 -> 32 groups 131 / 28.7 / 22.1 us, 64 -> 10 - / 12.8 / 10.4, 200 -> 50 - / 80.8 / 44.2; below 2^54: 128 -> 32 28.7 / 27.1, 64 ->
// 10 12.8 / 12.5, 200 -> 50 81 / 64, 256 -> 32 114 / 90; beyond: 128 -> 32 37.1 / 31.6, 64 -> 10 16.4 / 14.6, 200 -> 50 77.0 / 77.7.  (A maximum of
// 64-bit keys as such, five instructions a step, took 31.2 and 71 where two of 32 bits, six instructions each, take 27.1 and 64.)
template <int ctrl>
__device__ __forceinline__ long long dpp_max(long long v) {
    const int low = __builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, 0xf, 0xf, false);
    const int high = __builtin_amdgcn_update_dpp((int)(v >> 32), (int)(v >> 32), ctrl, 0xf, 0xf, false);
    const long long other = (long long)((uint64_t)(uint32_t)high << 32 | (uint32_t)low);
    return other > v ? other : v;
}
// the maximum over the wave, in every lane
__device__ __forceinline__ long long wave_max(long long v) {
    v = dpp_max<0x111>(v);   // row_shr:1, 2, 4, 8: lane 15 of each row of 16
    v = dpp_max<0x112>(v);
    v = dpp_max<0x114>(v);
    v = dpp_max<0x118>(v);
    v = dpp_max<0x142>(v);   // row_bcast:15, row_bcast:31: lane 63 of the wave
    v = dpp_max<0x143>(v);
    const uint32_t low = (uint32_t)__builtin_amdgcn_readlane((int)v, 63), high = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), 63);
    return (long long)((uint64_t)high << 32 | low);
}

// unsigned: a lane without a source takes 0, and every step is one instruction
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define GROUTER_STEP(ctrl) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true))
    GROUTER_STEP(0x111);
    GROUTER_STEP(0x112);
    GROUTER_STEP(0x114);
    GROUTER_STEP(0x118);
    GROUTER_STEP(0x142);
    GROUTER_STEP(0x143);
#undef GROUTER_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// row(e, i): entry (e, lane + 64 i) of the matrix
template <int PER, class Row>
__device__ __forceinline__ void fold_loop(int E_S, int E_T, int lane, int32_t* __restrict__ group_of, Row row) {
    constexpr long long lowest = -0x7fffffffffffffffLL - 1;
    uint64_t open[PER];   // unassigned experts, by lane
#pragma unroll
    for (int i = 0; i < PER; ++i) open[i] = __ballot(lane + 64 * i < E_S);
    const int g_avg = E_S / E_T, n_extra = E_S % E_T;
    int group[PER] = {};
    for (int g = 0; g < E_T; ++g) {
        const int size = g_avg + (g < n_extra ? 1 : 0);
        long long score[PER];
        for (int m = 0; m < size; ++m) {
            uint64_t best[PER];
            if (m == 0) {   // every unassigned expert ties
#pragma unroll
                for (int i = 0; i < PER; ++i) best[i] = open[i];
            } else {
                long long cand[PER], mx = lowest;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    cand[i] = ((open[i] >> lane) & 1) ? score[i] : lowest;
                    mx = cand[i] > mx ? cand[i] : mx;
                }
                mx = wave_max(mx);
#pragma unroll
                for (int i = 0; i < PER; ++i) best[i] = __ballot(cand[i] == mx) & open[i];
            }
            int pick = -1;
#pragma unroll
            for (int i = PER - 1; i >= 0; --i)
                if (best[i]) pick = 64 * i + (int)__builtin_ctzll(best[i]);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (pick >> 6 == i) open[i] &= ~(1ull << (pick & 63));
                if (pick == lane + 64 * i) group[i] = g;
            }
            if (m + 1 < size) {
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const long long p = row(pick, i);
                    score[i] = m == 0 ? p : score[i] + p;
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (lane + 64 * i < E_S) group_of[lane + 64 * i] = group[i];
}

// The same loop on keys, score * 256 + 255 - expert: their maximum over the wave names the expert, the lowest of those that tie.
// Key: uint32_t for scores below 2^24 and up to 255 experts, where a step of the maximum is one instruction; long long for scores
// below 2^54 in size.  row(at): entry at + mine of the matrix, mine the lane's first expert or the last one there is.
template <class Key, int PER, class Row>
__device__ __forceinline__ void fold_keys(int E_S, int E_T, int lane, int mine, int32_t* __restrict__ group_of, Row row) {
    using U = std::make_unsigned_t<Key>;   // (the keys of experts that are taken may wrap)
    uint64_t open[PER];   // unassigned experts, by lane
    uint32_t alive[PER];  // the same, as a mask of each lane's own
    int group[PER] = {};
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        open[i] = __ballot(lane + 64 * i < E_S);
        alive[i] = lane + 64 * i < E_S ? ~0u : 0u;
    }
    const int g_avg = E_S / E_T, n_extra = E_S % E_T;
    const int last = E_S * E_S - 1 - mine;
    for (int g = 0; g < E_T; ++g) {
        const int size = g_avg + (g < n_extra ? 1 : 0);
        U key[PER];
        int pick = 0;   // the group's first member: the lowest unassigned expert
#pragma unroll
        for (int i = PER - 1; i >= 0; --i)
            if (open[i]) pick = 64 * i + (int)__builtin_ctzll(open[i]);
        for (int m = 0;; ++m) {
            const bool done = m + 1 >= size;
            U p[PER];
            if (!done) {   // requested first: the rest of the bookkeeping runs meanwhile (what a lane without an expert reads is masked)
#pragma unroll
                for (int i = 0; i < PER; ++i) p[i] = (U)row(min(pick * E_S + 64 * i, last));
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (pick >> 6 == i) open[i] &= ~(1ull << (pick & 63));
                if (pick == lane + 64 * i) {
                    alive[i] = 0u;
                    group[i] = g;
                }
            }
            if (done) break;
            if constexpr (sizeof(Key) == 4) {
                uint32_t mx = 0;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    key[i] = (p[i] << 8) + (m == 0 ? 255u - (uint32_t)(lane + 64 * i) : key[i]);
                    mx = max(mx, key[i] & alive[i]);
                }
                pick = 255 - (int)(wave_max_u32(mx) & 255u);
            } else {
                // the upper words first, offset so that none is 0, then the lower ones of those that hold the maximum
                uint32_t high[PER], mx = 0, mn = 0;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    key[i] = (p[i] << 8) + (m == 0 ? (U)(255 - (lane + 64 * i)) : key[i]);
                    high[i] = ((uint32_t)(key[i] >> 32) ^ 0x80000000u) & alive[i];
                    mx = max(mx, high[i]);
                }
                mx = wave_max_u32(mx);
#pragma unroll
                for (int i = 0; i < PER; ++i) mn = max(mn, high[i] == mx ? (uint32_t)key[i] : 0u);
                pick = 255 - (int)(wave_max_u32(mn) & 255u);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (lane + 64 * i < E_S) group_of[lane + 64 * i] = group[i];
}

// Up to 128 experts the matrix is staged in LDS as it is, and keys of either width are made of its entries.  Up to 200 experts its low
// words are staged, for the narrow keys; what does not fit is read from L2.  Scores of 2^54 and more, in size, are compared as they
// are.  The checks are a few instructions per entry in short loops: one workgroup runs this code once, and what it waits for then
// is the code itself (entries kept in registers, the same instructions 16 times: 128 -> 32 22 -> 25 us).  A division per entry, to leave
// out the diagonal, which decides nothing, took 1 us at 64 experts and 3 at 150.
constexpr int kFoldStaged = 200;
template <int PER>   // E_S <= 64 PER
__global__ __launch_bounds__(1024) void k_fold_groups_wave(const long long* __restrict__ P, int E_S, int E_T, int32_t* __restrict__ group_of) {
    constexpr bool WHOLE = PER <= 2;
    constexpr int kWords = WHOLE ? 2 * 64 * PER * 64 * PER : kFoldStaged * kFoldStaged;
    constexpr int kLarge = 1 << 14;   // upper words of entries below 2^46 in size: sums of up to 256 of them are below 2^54
    __shared__ __attribute__((aligned(16))) uint32_t s_words[kWords];
    __shared__ int s_large, s_wide;
    long long* const s_P = reinterpret_cast<long long*>(s_words);
    const int tid = threadIdx.x, n = E_S * E_S;
    if (E_S == E_T) {
        if (tid < E_S) group_of[tid] = tid;
        return;
    }
    if (tid == 0) s_large = s_wide = 0;
    __syncthreads();
    const uint32_t limit = 0xffffffu / (unsigned)((E_S + E_T - 1) / E_T);
    int high = 0, low = 0;       // largest and smallest upper word
    uint32_t most = 0;           // largest lower word
    bool wide = !WHOLE && E_S > kFoldStaged;
    int i = tid;
    if (!wide) {
        uint32_t at = (uint32_t)tid % (uint32_t)(E_S + 1);   // 0 on the diagonal
        const uint32_t step = 1024u % (uint32_t)(E_S + 1);
        auto look = [&](int i, long long v) {
            if constexpr (WHOLE) s_P[i] = v;
            else s_words[i] = (uint32_t)v;
            v = at == 0 ? 0 : v;
            high = max(high, (int)(v >> 32));
            low = min(low, (int)(v >> 32));
            most = max(most, (uint32_t)v);
            at += step;
            at = min(at, at - (uint32_t)(E_S + 1));
        };
        if constexpr (WHOLE) {
#pragma unroll 8
            for (; i < n; i += 1024) look(i, P[i]);
        } else {   // (large entries are seen early, and no more is staged then)
            for (; i + 7 * 1024 < n && !wide; i += 8 * 1024) {
                long long v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = P[i + 1024 * q];
#pragma unroll
                for (int q = 0; q < 8; ++q) look(i + 1024 * q, v[q]);
                wide = __any(high | low | (int)(most > limit)) != 0;
            }
            if (!wide)
                for (; i < n; i += 1024) look(i, P[i]);
        }
        wide = (high | low) != 0 || most > limit;
    }
    if constexpr (!WHOLE) {
#pragma unroll 8
        for (; i < n; i += 1024) {
            const int v = (int)(P[i] >> 32);
            high = max(high, v);
            low = min(low, v);
        }
    }
    if (high >= kLarge || low < -kLarge) s_large = 1;
    if (wide) s_wide = 1;
    __syncthreads();
    if (tid >= 64) return;
    const int mine = min(tid, E_S - 1);
    const uint32_t* const words = s_words + (WHOLE ? 2 * mine : mine);
    const long long* whole = P + mine;
    if constexpr (WHOLE) whole = s_P + mine;
    if (!s_wide) fold_keys<uint32_t, PER>(E_S, E_T, tid, mine, group_of, [&](int at) { return words[WHOLE ? 2 * at : at]; });
    else if (!s_large) fold_keys<long long, PER>(E_S, E_T, tid, mine, group_of, [&](int at) { return whole[at]; });
    else fold_loop<PER>(E_S, E_T, tid, group_of, [&](int e, int i) { return whole[e * E_S + min(64 * i, E_S - 1 - mine)]; });
}

// More than 256 experts: one workgroup, thread j <-> source expert j.
constexpr long long kNoCandidate = -0x7fffffffffffffffLL - 1;  // below every real score

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_fold_groups(const long long* __restrict__ P, int E_S, int E_T,
                                                         int32_t* __restrict__ group_of) {
    constexpr int kWaves = THREADS / 64;
    __shared__ long long s_key[kWaves];
    __shared__ int s_idx[kWaves];
    __shared__ int s_pick;
    const int j = threadIdx.x;
    const int lane = j & 63, wave = j >> 6;
    const bool real = j < E_S;
    bool assigned = !real;
    long long score = 0;
    const int g_avg = E_S / E_T, n_extra = E_S % E_T;
    for (int g = 0; g < E_T; ++g) {
        const int size = g_avg + (g < n_extra ? 1 : 0);
        for (int m = 0; m < size; ++m) {
            // key: for the first member every unassigned expert ties (lowest number wins); later the score
            long long key = assigned ? kNoCandidate : (m == 0 ? 0 : score);
            int who = j;
            for (int off = 32; off > 0; off >>= 1) {
                const long long ok = __shfl_down(key, off);
                const int ow = __shfl_down(who, off);
                if (ok > key || (ok == key && ow < who)) {
                    key = ok;
                    who = ow;
                }
            }
            if (lane == 0) {
                s_key[wave] = key;
                s_idx[wave] = who;
            }
            __syncthreads();
            if (j == 0) {
                long long bk = s_key[0];
                int bw = s_idx[0];
                for (int w = 1; w < kWaves; ++w)
                    if (s_key[w] > bk || (s_key[w] == bk && s_idx[w] < bw)) {
                        bk = s_key[w];
                        bw = s_idx[w];
                    }
                s_pick = bw;
            }
            __syncthreads();
            const int pick = s_pick;
            if (j == pick) {
                assigned = true;
                group_of[j] = g;
            }
            if (real) score = (m == 0 ? 0 : score) + P[(size_t)pick * E_S + j];
            __syncthreads();  // s_pick, s_key are rewritten by the next round
        }
    }
}

// out[r][g] = sum over source experts e with group_of[e] == g of W[r][e], e ascending, fp32.
// A workgroup takes 8 rows.  It first lists the members of every group in ascending order, so an output adds its own members
// only instead of looking at all E_S, eight loads at a time.  2048 rows, a search through all experts / lists with one
// dependent load after the other / now: 128 -> 32 12.4 / 7.1 / 6.2 us; 128 -> 1 14.4 / 22.4 / 7.2; 1024 -> 1 95 / 230 / 26.
//   E_S <= 64   the place of an expert is counted by comparing it with all others: no further barriers (64 -> 32: 4.6 us)
//   more        counting sort as in the routing plan: by comparing / sorting 128 -> 32 6.8 / 6.2, 200 -> 25 (4096 rows)
//               10.0 / 7.1, 256 -> 1 14.3 / 10.0, 1024 -> 256 111 / 13
constexpr int kFoldRows = 8, kFoldCompare = 64;
template <bool SORT>
__global__ __launch_bounds__(kStatThreads) void k_fold_weights(const float* __restrict__ W, const int32_t* __restrict__ group_of,
                                                               int d, int E_S, int E_T, float* __restrict__ out) {
    constexpr int kMax = SORT ? kMaxExperts : kFoldCompare, kWaves = kStatThreads / 64;
    __shared__ float s_w[kFoldRows * kMax];
    __shared__ __attribute__((aligned(16))) int32_t s_g[kMax];
    __shared__ int32_t s_member[kMax], s_start[kMax], s_end[kMax];
    __shared__ int32_t s_cursor[SORT ? kWaves * kMax : 1], s_wave[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = (int)blockIdx.x * kFoldRows, rows = min(kFoldRows, d - r0);
    for (int i = tid; i < rows * E_S; i += kStatThreads) s_w[i] = W[(size_t)r0 * E_S + i];
    for (int e = tid; e < kMax; e += kStatThreads) {
        s_g[e] = e < E_S ? group_of[e] : 0x7fffffff;
        s_start[e] = s_end[e] = 0;   // a group without members
    }
    if constexpr (SORT)
        for (int i = tid; i < kWaves * kMax; i += kStatThreads) s_cursor[i] = 0;
    __syncthreads();
    if constexpr (!SORT) {
        // place of expert e: the experts of lower groups, and those of its own group that come before it
        if (tid < E_S) {
            const int g = s_g[tid];
            int at = 0, before = 0, size = 0;
#pragma unroll 4
            for (int o = 0; o < E_S; o += 4) {
                const int4 v = *(const int4*)(s_g + o);
                at += (v.x < g) + (v.y < g) + (v.z < g) + (v.w < g);
                before += ((v.x == g) & (o < tid)) + ((v.y == g) & (o + 1 < tid)) + ((v.z == g) & (o + 2 < tid)) + ((v.w == g) & (o + 3 < tid));
                size += (v.x == g) + (v.y == g) + (v.z == g) + (v.w == g);
            }
            if ((uint32_t)g < (uint32_t)E_T) {
                s_member[at + before] = tid;
                if (before == 0) {
                    s_start[g] = at;
                    s_end[g] = at + size;
                }
            }
        }
    } else {
        // every wave counts its quarter of the experts, a scan over groups and waves gives the cursors, and the waves place
        // their experts 64 at a time; groups outside [0, E_T) are left out
        constexpr int kRun = kMax / kWaves;
        int32_t* const mine = s_cursor + wave * kMax;
        for (int i = lane; i < kRun; i += 64) {
            const int g = s_g[wave * kRun + i];
            if ((uint32_t)g < (uint32_t)E_T) atomicAdd(&mine[g], 1);
        }
        __syncthreads();
        constexpr int kPer = kMax / kStatThreads;   // a thread's groups
        int sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            for (int w = 0; w < kWaves; ++w) sum += s_cursor[w * kMax + tid * kPer + i];
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int run = incl - sum;
        for (int w = 0; w < wave; ++w) run += s_wave[w];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int g = tid * kPer + i;
            s_start[g] = run;
            for (int w = 0; w < kWaves; ++w) {
                const int n = s_cursor[w * kMax + g];
                s_cursor[w * kMax + g] = run;
                run += n;
            }
            s_end[g] = run;
        }
        __syncthreads();
        volatile int32_t* const cursor = mine;   // a wave's own: its rounds need no barrier
        const uint64_t below = (1ull << lane) - 1;
        for (int i0 = 0; i0 < kRun; i0 += 64) {
            const int e = wave * kRun + i0 + lane, g = s_g[e];
            const bool counts = (uint32_t)g < (uint32_t)E_T;
            uint64_t peers = __ballot(counts);
            for (int b = 0; (1 << b) < E_T; ++b) {
                const bool bit = (g >> b) & 1;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            if (counts) {
                const int p = cursor[g] + __popcll(peers & below);
                s_member[p] = e;
                if ((peers >> lane) == 1ull) cursor[g] = p + 1;   // the group's highest lane
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < rows * E_T; i += kStatThreads) {
        const int r = i / E_T, g = i - r * E_T, end = s_end[g];
        const float* const w = s_w + r * E_S;
        float acc = 0.f;
        int m = s_start[g];
        for (; m + 8 <= end; m += 8) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = w[s_member[m + j]];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc += v[j];
        }
        for (; m < end; ++m) acc += w[s_member[m]];
        out[(size_t)r0 * E_T + i] = acc;
    }
}

}  // namespace

// Whether k_sample_stats8 pays for its table, which it fills and adds up once per sample.  With a workgroup per CU that is
// one table in a row, and a second round of tokens (L > 256) pays for it; up to 1024 samples the CUs hold all tables at once and a
// fourth round does; beyond, tables follow each other.  A placement alone only reads its table, so it pays earlier, unless k is small.
// The general kernel's adds wait for each other where tokens agree, the packed one's do not, so the lines lie where the two are about
// even on evenly spread ids: there the one loses up to 1.08 on these, the other up to 5 on ids that all tokens share (not with one id).
// Measured, general kernel / k_sample_stats8, uint8, 4 nodes; E = 128 evenly spread, E = 8, E = 128 with all tokens alike:
//   256 samples of 257 tokens, both statistics: k = 8 11.0 / 10.4 us, 11.3 / 10.4, 12.4 / 10.4; k = 1 9.8 / 9.7; placement alone: k = 1 4.2 / 3.9
//   1024 samples, affinity alone: k = 8 512 tokens 12.3 / 12.6, 13.1 / 11.0, 24.3 / 12.6; 600 13.0 / 13.7, 14.1 / 11.8, 26.8 / 13.4
//   both: 769 tokens, k = 8 16.7 / 16.1, 16.7 / 13.8, 34.0 / 15.8; k = 1 15.0 / 15.2, 13.9 / 13.4, 15.1 / 15.2
//   placement alone, E = 128: k = 4 300 tokens (600 samples) 4.8 / 4.6, 400 5.2 / 5.0; k = 1 600 5.9 / 6.1, 900 7.0 / 6.3
//   2048 samples, affinity alone: k = 8 1024 tokens 20.1 / 20.6, 24.3 / 16.7, 67.9 / 20.6; both: k = 8 700 tokens 21.1 / 23.7, 22.6 / 19.9,
//   52.7 / 24.4; 1100 25.5 / 26.2, 28.9 / 22.2, 75.0 / 26.0; k = 4, E = 128 2048 tokens 29.4 / 26.7; k = 1 27.9 / 26.9 (int32, 8192 samples 83 / 86)
//   placement alone: 1024 tokens, k = 3 11.3 / 10.6, 11.3 / 10.2, 11.3 / 10.5; k = 1, E = 128 11.4 / 11.3 at 1100 (8192 samples 32.9 / 34.8)
// The lines take no account of id type, E and nodes.  Over uint8 and int32, E = 8, 64, 128, 200 and 247, 4 and 16 nodes, the packed kernel's
// largest losses on evenly spread ids are: int32, k = 8, both, 2048 samples of 1100 tokens 27.5 / 29.7; 8192 of 1024, 16 nodes 84.5 / 90.5 (E = 8,
// 4 nodes 79.7 / 63.9); affinity alone, k = 3, 1024 of 600 12.8 / 13.6; one id, which stays with the general kernel there, 12.4 / 13.3.
static bool packed_pays(int64_t S, int L, int k, bool affinity, bool placement) {
    const int64_t ids = (int64_t)L * k;
    if (S <= 256) return L > 256;
    if (!affinity) return S <= 1024 ? L > 768 || (L > 256 && k >= 4) : L >= 2048 || (L >= 1024 && k >= 4);
    if (S <= 1024) return (k > 1 && L >= (placement ? 1024 : 512)) || (L > 768 && ids >= 1024);
    return ids >= 8192 || (L >= 2048 && ids >= 4096);
}

// counts == nullptr skips the affinity half, comm == nullptr the placement half.
hipError_t launch_sample_stats(const void* idx, int idx_dtype, int64_t S, int L, int k, int E, int32_t* counts,
                               double* entropy, int64_t* loads, double* maxvio, const uint64_t* expert_nodes, int n_nodes,
                               int32_t* comm, int32_t* best_node, hipStream_t s) {
    auto* l = reinterpret_cast<unsigned long long*>(loads);
    const dim3 grid((unsigned)S), block(kStatThreads);
#define GROUTER_STATS(T_, A_, P_)                                                                                  \
    do {                                                                                                           \
        if (k <= 8) hipLaunchKernelGGL((k_sample_stats<T_, A_, P_, false>), grid, block, 0, s, (const T_*)idx, L, k, E, counts, entropy, \
                                       expert_nodes, n_nodes, comm, best_node);                                    \
        else hipLaunchKernelGGL((k_sample_stats<T_, A_, P_, true>), grid, block, 0, s, (const T_*)idx, L, k, E, counts, entropy, \
                                expert_nodes, n_nodes, comm, best_node);                                           \
    } while (0)
#define GROUTER_STATS8(T_, A_, P_, R_)                                                                             \
    hipLaunchKernelGGL((k_sample_stats8<T_, A_, P_, R_>), grid, block, 0, s, (const T_*)idx, S, L, k, E, counts, entropy, \
                       expert_nodes, n_nodes, comm, best_node)
    const bool fast = k <= 8 && E <= kFastStatE && n_nodes <= kFastStatNodes && L <= kFastStatL && packed_pays(S, L, k, counts != nullptr, comm != nullptr);
    // a column per lane where the table then fits 33 KB
#define GROUTER_STATS_T(A_, P_)                                                      \
    do {                                                                             \
        if (idx_dtype == 1) {                                                        \
            if (fast && E <= 128) GROUTER_STATS8(uint8_t, A_, P_, 64);               \
            else if (fast) GROUTER_STATS8(uint8_t, A_, P_, 32);                      \
            else GROUTER_STATS(uint8_t, A_, P_);                                     \
        } else {                                                                     \
            if (fast && E <= 128) GROUTER_STATS8(int32_t, A_, P_, 64);               \
            else if (fast) GROUTER_STATS8(int32_t, A_, P_, 32);                      \
            else GROUTER_STATS(int32_t, A_, P_);                                     \
        }                                                                            \
    } while (0)
    if (counts && comm) GROUTER_STATS_T(true, true);
    else if (counts) GROUTER_STATS_T(true, false);
    else GROUTER_STATS_T(false, true);
#undef GROUTER_STATS_T
#undef GROUTER_STATS8
#undef GROUTER_STATS
    // one workgroup reads 32 numbers per thread in 3 us; at 2048 x 128 it would take 17 against the 9 us of two launches
    if (counts && S * E <= 32 * kLoadsThreads) {
        hipLaunchKernelGGL(k_loads_maxvio, dim3(1), dim3(kLoadsThreads), 0, s, counts, (int)S, E, l, maxvio);
    } else if (counts) {
        hipLaunchKernelGGL(k_loads, dim3((unsigned)((E + kLoadsCols - 1) / kLoadsCols)), dim3(kLoadsThreads), 0, s, counts, S, E, l);
        hipLaunchKernelGGL(k_maxvio, dim3(1), dim3(kStatThreads), 0, s, l, E, maxvio);
    }
    return hipGetLastError();
}

hipError_t launch_affinity(const void* idx, int idx_dtype, int64_t S, int L, int k, int E, int32_t* counts,
                           double* entropy, int64_t* loads, double* maxvio, hipStream_t s) {
    return launch_sample_stats(idx, idx_dtype, S, L, k, E, counts, entropy, loads, maxvio, nullptr, 0, nullptr, nullptr, s);
}

hipError_t launch_placement(const void* idx, int idx_dtype, int64_t S, int L, int k, int E, const uint64_t* expert_nodes,
                            int n_nodes, int32_t* comm, int32_t* best_node, hipStream_t s) {
    return launch_sample_stats(idx, idx_dtype, S, L, k, E, nullptr, nullptr, nullptr, nullptr, expert_nodes, n_nodes, comm,
                               best_node, s);
}

hipError_t launch_fold_groups(const int64_t* P, int E_S, int E_T, int32_t* group_of, hipStream_t s) {
    const long long* p = (const long long*)P;
    if (E_S <= 64) hipLaunchKernelGGL(k_fold_groups_wave<1>, dim3(1), dim3(1024), 0, s, p, E_S, E_T, group_of);
    else if (E_S <= 128) hipLaunchKernelGGL(k_fold_groups_wave<2>, dim3(1), dim3(1024), 0, s, p, E_S, E_T, group_of);
    else if (E_S <= 256) hipLaunchKernelGGL(k_fold_groups_wave<4>, dim3(1), dim3(1024), 0, s, p, E_S, E_T, group_of);
    else hipLaunchKernelGGL(k_fold_groups<1024>, dim3(1), dim3(1024), 0, s, p, E_S, E_T, group_of);
    return hipGetLastError();
}

hipError_t launch_fold_weights(const float* W, const int32_t* group_of, int d, int E_S, int E_T, float* out, hipStream_t s) {
    const dim3 grid((unsigned)((d + kFoldRows - 1) / kFoldRows)), block(kStatThreads);
    if (E_S <= kFoldCompare) hipLaunchKernelGGL(k_fold_weights<false>, grid, block, 0, s, W, group_of, d, E_S, E_T, out);
    else hipLaunchKernelGGL(k_fold_weights<true>, grid, block, 0, s, W, group_of, d, E_S, E_T, out);
    return hipGetLastError();
}

}  // namespace grouter
