// Routing-plan kernels: per-expert histogram, exclusive scan and stable scatter of the N = T*k routed
// slots (the cached top-k expert ids of Sec. 3.3.1), plus the row-tile list the grouped GEMMs walk.
//
// The scatter must reproduce the stable counting sort exactly (ties in ascending slot order), so ranks
// come from prefix counts, never from the arrival order of atomics.
//
// What bounds a plan is latency: launches, dependent memory round trips, and the serial walk over a wave's slots.
//   N <= kPlanCounting  one launch: the workgroup of every chunk counts all slots, in LDS, and places its own
//   larger N            two launches: k_plan_hist counts the chunks; then every chunk's workgroup adds up the counts of the
//                       chunks before it (at most 256 x E numbers out of L2, cheaper than a launch of its own for a scan)
//                       and places its slots
// In both, one further workgroup writes counts, offsets, load order and tile list meanwhile.
// In the placing pass a wave walks its slots 64 at a time in order; a lane's rank among the lanes of the same expert
// comes from wave ballots, the running per-expert cursor from the wave's own LDS column.
// Back-to-back builds in a graph, one workgroup that does everything (up to 4096 slots) or two launches / one launch of chunks that
// count / and with the load ranks shared by all threads: N = 6, E = 64 6.5 / 5.9 / 4.6 us; 1600, E = 64 7.8 / 6.2 / 5.5; 2400, E = 128
// 10.5 / 8.1 / 5.8; 4096, E = 64 9.8 / 6.6 / 6.4; 4995, E = 60, skewed 8.3 / 6.6 / 6.5; two launches, 20000, E = 128 10.8 / - / 8.9; 49152,
// E = 64 9.2 / - / 8.5.
// One launch against two where the line is drawn: 8192 slots, E = 64, uniform 7.0 against 8.2 us, all on one expert 7.8 / 10.0.
// The most counts to add up in two launches, 256 x 1024 in each of 257 workgroups: N = 131072, E = 1024 70 us.
// Nothing is accumulated into memory that an earlier launch must have cleared, so a plan can be rebuilt in
// place and the build can be captured into a HIP graph as it is.
#include "common.hpp"

namespace grouter {

// An id outside [0,E) is reported through *bad and handled as expert 0, so no access leaves the workspace.
template <typename IdxT>
__device__ __forceinline__ int load_expert(const IdxT* idx, int64_t i, int E, bool* bad) {
    int e = (int)idx[i];
    if (e < 0 || e >= E) {
        *bad = true;
        e = 0;
    }
    return e;
}

constexpr int kPlanThreads = kPlanWaves * 64;  // thread e <-> expert e (E <= 1024)

// Exclusive prefix sum over the workgroup's threads; *total receives the sum.  s_w: kPlanWaves + 1 words.
__device__ __forceinline__ int block_exclusive_scan(int v, int32_t* s_w, int tid, int* total) {
    const int lane = tid & 63, wave = tid >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        const int w = lane < kPlanWaves ? s_w[lane] : 0;
        int wi = w;
        for (int o = 1; o < kPlanWaves; o <<= 1) {
            const int up = __shfl_up(wi, o, 64);
            if (lane >= o) wi += up;
        }
        if (lane < kPlanWaves) s_w[lane] = wi - w;
        if (lane == kPlanWaves - 1) s_w[kPlanWaves] = wi;
    }
    __syncthreads();
    const int res = s_w[wave] + incl - v;
    *total = s_w[kPlanWaves];
    __syncthreads();  // s_w may be reused right away
    return res;
}

// chunk_hist[chunk][e], chunk_bad[chunk]
template <typename IdxT>
__global__ __launch_bounds__(kPlanThreads) void k_plan_hist(const IdxT* __restrict__ idx, int64_t N, int E, int chunk,
                                                            int32_t* __restrict__ chunk_hist, int32_t* __restrict__ chunk_bad) {
    __shared__ int32_t cnt[kMaxExperts];
    __shared__ int32_t s_bad;
    const int tid = threadIdx.x;
    if (tid < E) cnt[tid] = 0;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * chunk, end = min(N, begin + chunk);
    bool bad = false;
    for (int64_t i = begin + tid; i < end; i += kPlanThreads) atomicAdd(&cnt[load_expert(idx, i, E, &bad)], 1);
    if (bad) atomicOr(&s_bad, 1);
    __syncthreads();
    if (tid < E) chunk_hist[(size_t)blockIdx.x * E + tid] = cnt[tid];
    if (tid == 0) chunk_bad[blockIdx.x] = s_bad;
}

struct PlanOut {
    int32_t* header; int32_t* counts; int32_t* offsets; int32_t* by_load;
    int32_t* row_to_src; int32_t* src_to_row; int32_t* row_token;
    int32_t* tiles; int max_tiles;
};

// Workgroup c < n_chunks places chunk c, workgroup n_chunks writes what concerns the plan as a whole.  COUNTING: every workgroup
// counts all slots itself; otherwise the counts of the chunks come from k_plan_hist.
// It does so in eight columns per expert, which lanes take in turn: where many slots pick the same expert, adds to one word wait for
// each other, a wave's 64 in a row (one word each for the slots of an expert and for those in earlier chunks / eight columns, one
// word for both, E = 64: N = 8192 on one expert 18.4 / 7.8 us, Zipf 10.3 / 7.0, uniform 7.4 / 7.0; N = 4096 11.5 / 7.2, 7.6 / 6.4, 6.5 / 6.4;
// N = 2000 8.0 / 6.8, 6.2 / 6.0, 6.1 / 6.1; four columns 8.5 at N = 8192 on one expert, sixteen as eight).
constexpr int kPlanColumns = 8;
static_assert(kPlanCounting < 1 << 16 && kPlanColumns % 4 == 0, "a column's word holds two counts");
template <typename IdxT, bool COUNTING>
__global__ __launch_bounds__(kPlanThreads) void k_plan_place(const IdxT* __restrict__ idx, int N, int E, int k, int bits, int chunk,
                                                             int n_chunks, const int32_t* __restrict__ chunk_hist,
                                                             const int32_t* __restrict__ chunk_bad, const PlanOut out) {
    __shared__ int32_t s_hist[kPlanWaves * kMaxExperts];   // [wave][expert]: counts, then cursors
    __shared__ __attribute__((aligned(16))) int32_t s_cnt[kMaxExperts];
    __shared__ int32_t s_off[kMaxExperts];
    __shared__ int32_t s_before[kMaxExperts];     // slots of the expert in earlier chunks; later the load order
    __shared__ int32_t s_first[kMaxExperts + 1];  // first tile of each load rank
    __shared__ int32_t s_w[kPlanWaves + 1];
    __shared__ int32_t s_bad;
    __shared__ uint4 s_col[COUNTING ? kMaxExperts * kPlanColumns / 4 : 1];   // [expert][column]: slots, and above them those in earlier chunks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool place = (int)blockIdx.x < n_chunks;
    const int64_t begin = (int64_t)blockIdx.x * chunk;
    const int64_t end = min((int64_t)N, begin + chunk);
    const int per_wave = chunk / kPlanThreads * 64;
    const int64_t w_begin = begin + (int64_t)wave * per_wave, w_end = min(end, w_begin + per_wave);
    int32_t* const my_hist = s_hist + wave * E;

    if (tid == 0) s_bad = 0;
    s_cnt[tid] = tid < E ? 0 : -1;   // (no expert: ranks behind every expert)
    s_before[tid] = 0;
    s_first[tid] = 0;
    if (place)
        for (int e = lane; e < E; e += 64) my_hist[e] = 0;
    if (COUNTING)
        for (int i = tid; i < E * (kPlanColumns / 4); i += kPlanThreads) s_col[i] = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
    bool bad = false;
    if (place)
        for (int64_t i = w_begin + lane; i < w_end; i += 64) atomicAdd(&my_hist[load_expert(idx, i, E, &bad)], 1);
    if constexpr (!COUNTING) {
        const int n = n_chunks * E, mine = (int)blockIdx.x * E;
        for (int i = tid; i < n; i += kPlanThreads) {
            const int v = chunk_hist[i], e = (int)((uint32_t)i % (uint32_t)E);
            if (v) {
                atomicAdd(&s_cnt[e], v);
                if (i < mine) atomicAdd(&s_before[e], v);
            }
        }
        if (!place)
            for (int c = tid; c < n_chunks; c += kPlanThreads) bad |= chunk_bad[c] != 0;
    } else {
        uint32_t* const column = reinterpret_cast<uint32_t*>(s_col) + tid % kPlanColumns;
#pragma unroll 8
        for (int i = tid; i < N; i += kPlanThreads)
            atomicAdd(&column[load_expert(idx, i, E, &bad) * kPlanColumns], place && i < begin ? 0x10001u : 1u);
    }
    if (bad) atomicOr(&s_bad, 1);
    __syncthreads();
    int cnt = 0;
    if (tid < E) {
        if constexpr (COUNTING) {
            uint32_t both = 0;
#pragma unroll
            for (int q = 0; q < kPlanColumns / 4; ++q) {
                const uint4 c = s_col[tid * (kPlanColumns / 4) + q];
                both += c.x + c.y + c.z + c.w;
            }
            s_cnt[tid] = (int)(both & 0xffffu);
            s_before[tid] = (int)(both >> 16);
        }
        cnt = s_cnt[tid];
    }
    int total;
    const int off = block_exclusive_scan(cnt, s_w, tid, &total);
    if (tid < E) {
        s_off[tid] = off;
        if (place) {
            int run = off + s_before[tid];
#pragma unroll
            for (int w = 0; w < kPlanWaves; ++w) {
                const int t = s_hist[w * E + tid];
                s_hist[w * E + tid] = run;
                run += t;
            }
        }
    }
    __syncthreads();
    if (place) {
        // the cursors of a wave are its own: no barrier between its rounds, LDS accesses of one wave stay in order
        volatile int32_t* const cursor = my_hist;
        const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        for (int64_t i0 = w_begin; i0 < w_end; i0 += 64) {
            const int64_t i = i0 + lane;
            const bool valid = i < w_end;
            bool bad_unused = false;  // already reported by the counting pass
            const int e = valid ? load_expert(idx, i, E, &bad_unused) : 0;
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < bits; ++b) {
                const bool bit = (e >> b) & 1;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            if (valid) {
                const int p = cursor[e] + __popcll(peers & below);
                out.row_to_src[p] = (int32_t)i;
                out.src_to_row[i] = p;
                out.row_token[p] = (int32_t)((uint32_t)i / (uint32_t)k);
                if ((peers >> lane) == 1ull) cursor[e] = p + 1;  // highest lane of the group advances the cursor
            }
        }
    }
    if (place) return;

    // offsets, load order, tile list, header
    int32_t* const s_order = s_before;  // expert id at each load rank
    if (tid < E) {
        out.counts[tid] = cnt;
        out.offsets[tid] = off;
    }
    // load ranks, heaviest first, ties by lower id: an expert's comparisons are shared by kPlanThreads / 2^bits threads, which add
    // up what they find in s_first
    {
        const int e = tid & ((1 << bits) - 1), parts = kPlanThreads >> bits;
        const int per = ((E + parts - 1) / parts + 3) & ~3;
        const int mine = s_cnt[e];
        auto rank_among = [&](int part) {
            const int from = part * per;
            int rank = 0;
#pragma unroll 4
            for (int o = from; o < min(E, from + per); o += 4) {   // (entries from E on are -1)
                const int4 co = *(const int4*)(s_cnt + o);
                rank += ((co.x > mine) | ((co.x == mine) & (o < e))) + ((co.y > mine) | ((co.y == mine) & (o + 1 < e))) +
                        ((co.z > mine) | ((co.z == mine) & (o + 2 < e))) + ((co.w > mine) | ((co.w == mine) & (o + 3 < e)));
            }
            return rank;
        };
        // from 33 experts on the lanes of a wave have the same part: known to be so, the loop counts in scalars (E = 1024: 51.0 -> 49.1 us at
        // 8200 slots)
        const int rank = bits >= 6 ? rank_among(__builtin_amdgcn_readfirstlane(tid >> bits)) : rank_among(tid >> bits);
        if (e < E && rank) atomicAdd(&s_first[e], rank);
    }
    __syncthreads();
    if (tid < E) {
        s_order[s_first[tid]] = tid;
        out.by_load[s_first[tid]] = tid;
    }
    if (tid == 0) out.offsets[E] = total;
    __syncthreads();
    // row tiles in load-rank order: thread r owns the expert of rank r
    const int rows = tid < E ? s_cnt[s_order[tid]] : 0;
    const int n_tiles = (rows + kTileRowsSmall - 1) / kTileRowsSmall;
    int total_tiles;
    const int t = block_exclusive_scan(n_tiles, s_w, tid, &total_tiles);
    if (tid == 0) {
        out.header[0] = s_bad;
        out.header[1] = total_tiles;
        out.header[2] = N;
        out.header[3] = k;
        out.header[4] = E;
    }
    if (tid < E) s_first[tid] = t;
    if (tid == 0) s_first[E] = total_tiles;
    __syncthreads();
    // every tile is written by its own thread: find the load rank whose tile range holds tile ti
    for (int ti = tid; ti < min(total_tiles, out.max_tiles); ti += kPlanThreads) {
        int lo = 0, hi = E - 1;  // largest rank r with s_first[r] <= ti (ranks without tiles share their successor's start)
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_first[mid] <= ti) lo = mid;
            else hi = mid - 1;
        }
        // one 32-byte record per tile, the same for every tile of an expert: a kernel that is handed tile ti learns
        // from it where any other tile of that expert lies, with one load
        const int ex = s_order[lo];
        int4* const rec = (int4*)(out.tiles + 8 * (size_t)ti);
        rec[0] = int4{ex, s_off[ex], s_cnt[ex], s_first[lo]};
        rec[1] = int4{s_first[lo + 1] - s_first[lo], 0, 0, 0};
    }
}

template <typename IdxT>
static void launch_plan_t(const IdxT* idx, const PlanLayout& L, char* b, hipStream_t s) {
    int32_t* const hist = (int32_t*)(b + L.off_chunk_hist);
    int32_t* const bad = (int32_t*)(b + L.off_chunk_bad);
    const PlanOut out{(int32_t*)(b + L.off_header), (int32_t*)(b + L.off_counts), (int32_t*)(b + L.off_offsets),
                      (int32_t*)(b + L.off_by_load), (int32_t*)(b + L.off_row_to_src), (int32_t*)(b + L.off_src_to_row),
                      (int32_t*)(b + L.off_row_token), (int32_t*)(b + L.off_tiles_small), L.max_tiles_small};
    int bits = 0;
    while ((1 << bits) < L.E) ++bits;
    const dim3 grid((unsigned)L.n_chunks + 1);
    if (L.N <= kPlanCounting) {
        hipLaunchKernelGGL((k_plan_place<IdxT, true>), grid, dim3(kPlanThreads), 0, s, idx, (int)L.N, L.E, L.k, bits, L.chunk, L.n_chunks,
                           (const int32_t*)nullptr, (const int32_t*)nullptr, out);
        return;
    }
    hipLaunchKernelGGL(k_plan_hist<IdxT>, dim3((unsigned)L.n_chunks), dim3(kPlanThreads), 0, s, idx, L.N, L.E, L.chunk, hist, bad);
    hipLaunchKernelGGL((k_plan_place<IdxT, false>), grid, dim3(kPlanThreads), 0, s, idx, (int)L.N, L.E, L.k, bits, L.chunk, L.n_chunks,
                       (const int32_t*)hist, (const int32_t*)bad, out);
}

hipError_t launch_plan_build(const void* idx, int idx_dtype, const PlanLayout& L, void* plan_ws, hipStream_t s) {
    if (idx_dtype == 0) launch_plan_t((const int32_t*)idx, L, (char*)plan_ws, s);
    else launch_plan_t((const uint8_t*)idx, L, (char*)plan_ws, s);
    return hipGetLastError();
}

}  // namespace grouter
