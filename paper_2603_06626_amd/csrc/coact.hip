// Co-activation counts P[i][j] = number of tokens whose top-k set holds both i and j: the Gram matrix of the
// token x expert indicator matrix.  A workgroup owns a contiguous run of tokens.  A lane sets the (at most k) 4-bit cells of
// its token in an expert-major matrix ind[e][t] in LDS, and 64-token slabs of it are multiplied by their transpose with
// v_mfma_scale_f32_32x32x64_f8f6f4 on 4-bit floats (a cell is 0 or 1.0, scales are 1).  Both operands are 32 consecutive
// token cells of one expert, i.e. one 16-byte LDS read, and the same read serves as row operand and as column operand.  P is
// symmetric, so only the 32 x 32 blocks on and above the diagonal are computed.
//
// What bounds the main loop is the LDS: per 64 tokens 8 ORs at random banks (about 8 cycles each), the clearing and the
// fragment reads.  Hence
//   * 4-bit cells: half the reads, half the clearing and half the matrix-core time of bytes.  Eight tokens share a word, so a
//     cell is set with ds_or_b32, which without a returned value costs no more than a byte store; a repeated id, or one that
//     another lane sets in the same word, needs no care;
//   * up to 128 experts a wave holds all blocks (10 x 16 accumulator registers) and works alone: it sets slabs of its own 64
//     tokens, reads a slab's fragments once (4 reads per 10 MFMAs) and multiplies, with three slab buffers per wave and no
//     barrier at all, since the LDS accesses of one wave stay in order: while slab i is multiplied, the fragments of i + 1 are
//     read and i + 2 is set;
//   * 256 experts are 36 blocks, which four wave groups share: group g owns block rows g and NBLK-1-g, NBLK+1 blocks whatever
//     g is.  The workgroup then sets 256 tokens at a time for all waves, in three buffers with one barrier per pass: while
//     pass p is multiplied, pass p + 1 is set and the buffer of pass p - 1 is cleared for p + 2.
// fp32 accumulators count exactly to 2^24; kCoactMaxRun keeps a wave's counts at 2^21 and below.
//
// At the end the waves' parts are summed as integers through LDS and added into P with 64-bit integer atomics, every
// workgroup beginning elsewhere.  These atomics cost about 0.03 us per workgroup at E = 128, all workgroups queueing for the
// same cells (0.06 with one cell per atomic), so two cells, (r, c) and (r + 1, c), travel in one word while they are summed (T
// below 2^32, so that the lower one never carries).  The words of block (i, j) lie in the storage of block (j, i) below the
// diagonal, or of the diagonal block itself, and k_coact_finish spreads them out and fills the blocks below the diagonal.
//
// Few tokens are bound by what a workgroup does once: clearing its buffers, and writing and adding up the waves' blocks, which is
// why those meet in 16-bit halves, why nothing is set or cleared past a run's end and why places are found without a division.
//
// Measured (three launches; kernel on byte cells, with two barriers per pass and one cell per atomic / this one): 2048 x 4096 tokens, E = 128,
// k = 8, uint8 113 / 56 us; 512 x 2048, E = 128, k = 8, int32 48 / 24; 700 x 3000, E = 200, k = 5, uint8 107 / 67 (one cell per atomic 92);
// 300 x 1500, E = 60, k = 3, int32 22.3 / 13.5; 4000 tokens, k = 8, uint8, E = 128 15.0 / 12.5, E = 256 21.0 / 19.3; 500, E = 256 17.8 / 17.6.
// More than 8 ids, which are loaded one by one when they are set: 2^20 tokens, k = 16, uint8, E = 128 56 / 28, E = 200, int32 144 / 57; k = 64,
// uint8, E = 200 152 / 76; 48000, k = 16, E = 128 19.1 / 13.2; 2^23, k = 12, E = 64 125 / 81.
// Slower than on byte cells where all tokens pick the same experts, since then eight lanes OR each word and few cells queue, which would
// allow more workgroups: k = 8, uint8, E = 64, 2^23 tokens 60 / 71, 450000 16 / 19, E = 128 18 / 24; with a dozen experts in use 18 / 19.
// Cells of one bit (32 tokens a word) or two need fewer reads, but more lanes then OR the same word: 113 -> 89 and 80 instead of 73 at E = 200.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "stats_ids.hpp"

namespace grouter {
namespace {

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kCoactThreads = 512, kCoactWaves = kCoactThreads / 64;
constexpr int64_t kCoactMaxRun = 1 << 22;   // tokens of a workgroup

template <int EP>
struct CoactShape {
    static constexpr int NBLK = EP / 32;                                   // 32-expert blocks per side
    static constexpr int GROUPS = EP <= 128 ? 1 : NBLK / 2;                // wave groups that share the blocks
    static constexpr int SPLIT = kCoactWaves / GROUPS;                     // waves per group, which share the slabs
    static constexpr int NSLOT = GROUPS == 1 ? NBLK * (NBLK + 1) / 2 : NBLK + 1;   // blocks of a wave
    static constexpr int SLABS = GROUPS == 1 ? 1 : 4;                      // of 64 tokens in a buffer
    // a row of a slab is one expert: 32 bytes, and 16 more so that 16-byte reads of neighbouring experts miss each other's banks;
    // one more row than experts: ids beyond EP are pointed at it.  (Rows from E on hold what ids in [E, EP) set; no cell of
    // theirs is ever written out.)
    static constexpr int PITCH = 48, SLAB = (EP + 1) * PITCH, BUFFER = SLABS * SLAB;
    static constexpr int WAVE_BUFFERS = 3, BUFFERS = GROUPS == 1 ? WAVE_BUFFERS * kCoactWaves : 3;
    // at the end the LDS takes blocks of 2 KB from every wave, ROUND at a time
    static constexpr int ROUND = NSLOT < 10 ? NSLOT : 5;
    static constexpr int LDS = BUFFERS * BUFFER > kCoactWaves * ROUND * 2048 ? BUFFERS * BUFFER : kCoactWaves * ROUND * 2048;
    // tokens of a workgroup up to which no wave has more than 2^16 - 1: it has 64 of every 64 * SPLIT, at the end 64 for any rest
    static constexpr int SHORT = (1 << 16) * SPLIT - 64 * SPLIT;
    static_assert(SLAB % 16 == 0, "cleared in 16-byte pieces");
    // block (row, col) of slot s in wave group g
    static constexpr __device__ __host__ int row_of(int g, int s) {
        if (GROUPS > 1) return s < NBLK - g ? g : NBLK - 1 - g;
        int r = 0;
        while (s >= NBLK - r) s -= NBLK - r++;
        return r;
    }
    static constexpr __device__ __host__ int col_of(int g, int s) {
        if (GROUPS > 1) return s < NBLK - g ? g + s : NBLK - 1 - g + (s - (NBLK - g));
        int r = 0;
        while (s >= NBLK - r) s -= NBLK - r++;
        return r + s;
    }
};

// Where the word of rows (2 rp, 2 rp + 1) and column c of block (bi, bj) is summed.  The storage used is that of block (bj, bi):
// `cols` rows of 32 cells (of `cols` on the diagonal), taken in order; 16 row pairs (or half of an odd last block) x cols words
// always fit.  Every second row of blocks uses the lower half of its rows instead of the upper: at E = 128 the 256-byte segments
// of the upper halves alone fall on half of the memory channels, up to four on one, and the atomics of all workgroups queue
// there (2048 x 4096 tokens: 71 us, so 63).
__device__ __forceinline__ size_t coact_word(int E, int bi, int bj, int rp, int c) {
    const int cols = min(32, E - 32 * bj), half = cols == 32 ? 16 * (bj & 1) : 0;
    const int at = rp * cols + c;
    const int row = bi == bj ? rp : at >> 5, col = bi == bj ? c : at & 31;   // (dividing `at` by the width took 3 us of a call at E = 256)
    return (size_t)(32 * bj + half + row) * E + 32 * bi + col;
}

__device__ __forceinline__ i32x8_t coact_frag(const unsigned char* at) {
    const i32x4_t v = *reinterpret_cast<const i32x4_t*>(at);
    return __builtin_shufflevector(v, v, 0, 1, 2, 3, -1, -1, -1, -1);   // (a 4-bit operand is four registers)
}
__device__ __forceinline__ void coact_mfma(const i32x8_t& a, const i32x8_t& b, f32x16_t& c) {
    constexpr int kOne = 0x7f7f7f7f, kFp4 = 4;
    c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, kFp4, kFp4, 0, kOne, 0, kOne);
}

// N: most ids of a token that are kept in registers (4 or 8, k <= N), or 0 for k > 8
template <class IdxT, int EP, int N>
__global__ __launch_bounds__(kCoactThreads, 2) void k_coactivation(const IdxT* __restrict__ idx, int64_t T, int k, int E, int64_t tokens_per_group,
                                                                   bool packed, unsigned long long* __restrict__ P) {
    using S = CoactShape<EP>;
    constexpr int NSLOT = S::NSLOT, TOK = 64 * S::SLABS;
    __shared__ __attribute__((aligned(16))) unsigned char s_ind[S::LDS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave % S::GROUPS, part = wave / S::GROUPS;
    const int64_t begin = (int64_t)blockIdx.x * tokens_per_group;
    const int64_t end = min(T, begin + tokens_per_group);
    f32x16_t acc[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0.f;
    const int frag_at = (lane & 31) * S::PITCH + 16 * (lane >> 5);   // this lane's 32 tokens of expert (block * 32 + lane % 32)
    const int col = tid & (TOK - 1);
    const uint32_t bit = 2u << (4 * (col & 7));   // 1.0 in the cell of this lane's token
    // a lane has every 512th token; of the shared buffers the lower half of the workgroup sets the even ones, the upper half the odd
    constexpr bool FEW = N > 0;
    using Ids = IdWindow<IdxT, FEW ? N : 4>;
    const IdxT* const base = idx + begin * k;
    const int n = (int)(end - begin), last = (int)min((T - begin) * k - Ids::kWindow, (int64_t)0x7fffffff);
    int mine = tid;   // the token it sets next
    // sets its cells, with between(j) after the j-th of N, and fetches the ids of token `later`
    auto set = [&](unsigned char* ind, Ids& ids, int later, auto between) {
        const uint32_t v = mine < n ? bit : 0u;
        unsigned char* const at = ind + (col >> 6) * S::SLAB + ((col >> 3) & 7) * 4;
        auto one = [&](uint32_t e) { atomicOr(reinterpret_cast<uint32_t*>(at + min(e, (uint32_t)EP) * S::PITCH), v); };
        if constexpr (FEW) {
            ids.settle();
#pragma unroll
            for (int j = 0; j < N; ++j) {
                one(ids.id(j) | (j < k ? 0u : 0x10000u));   // (without a branch: see IdWindow)
                between(j);
            }
            ids.fetch(base, later * k, last);
        } else {
            if (mine < n)
                for (int j = 0; j < k; ++j) one((uint32_t)base[(size_t)mine * k + j]);
            between(0);
        }
        mine += kCoactThreads;
    };
    auto nothing = [](int) {};
    auto clear = [&](unsigned char* ind, int who, auto threads) {
        constexpr int kThreads = decltype(threads)::value, kPieces = S::SLABS * EP * 2;   // (padding stays zero, the spare row may keep its cells)
        static_assert(kPieces % kThreads == 0, "no remainder");
#pragma unroll
        for (int i = 0; i < kPieces / kThreads; ++i) {
            const int piece = i * kThreads + who, row = piece / 2;
            *reinterpret_cast<uint4*>(ind + row / EP * S::SLAB + row % EP * S::PITCH + piece % 2 * 16) = uint4{0u, 0u, 0u, 0u};
        }
    };
    using Wave = std::integral_constant<int, 64>;
    using Group = std::integral_constant<int, kCoactThreads>;
    if constexpr (S::GROUPS == 1) {
        unsigned char* const own = s_ind + wave * S::WAVE_BUFFERS * S::BUFFER;
        auto in_order = []() {   // for the compiler: the wave's LDS accesses stay in order by themselves
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        Ids ids[2] = {};   // of the next two slabs: a turn is shorter than a trip to memory
        if constexpr (FEW) {
            ids[0].fetch(base, mine * k, last);
            ids[1].fetch(base, (mine + kCoactThreads) * k, last);
        }
        clear(own, lane, Wave{});
        clear(own + S::BUFFER, lane, Wave{});
        in_order();
        set(own, ids[0], mine + 2 * kCoactThreads, nothing);
        set(own + S::BUFFER, ids[1], mine + 2 * kCoactThreads, nothing);   // (under a condition, the loop's first wait would be for both fetches)
        i32x8_t f[2][S::NBLK];
        auto read = [&](i32x8_t (&to)[S::NBLK], int from) {
            in_order();
#pragma unroll
            for (int c = 0; c < S::NBLK; ++c) to[c] = coact_frag(own + from + c * 32 * S::PITCH + frag_at);
            in_order();
        };
        read(f[0], 0);
        int here = 0, next = S::BUFFER, after = 2 * S::BUFFER, t0 = wave * 64;
        if (t0 + 2 * kCoactThreads < n) clear(own + after, lane, Wave{});
        // slot s is block (r, r + s - start of row r)
        auto multiply = [&](const i32x8_t (&x)[S::NBLK], int from, int to) {
#pragma unroll
            for (int s = from; s < to; ++s)
#pragma unroll
                for (int r = 0; r < S::NBLK; ++r) {
                    const int start = r * S::NBLK - r * (r - 1) / 2;
                    if (s >= start && s < start + S::NBLK - r) coact_mfma(x[r], x[r + s - start], acc[s]);
                }
        };
        // slab i is multiplied, the fragments of i + 1 are read, i + 2 is set between the MFMAs, and i's buffer is cleared
        auto turn = [&](auto which) {
            constexpr int b = decltype(which)::value;
            read(f[b ^ 1], next);
            constexpr int M = FEW ? N : 1;
            set(own + after, ids[b], mine + 2 * kCoactThreads, [&](int j) { multiply(f[b], j * S::NSLOT / M, (j + 1) * S::NSLOT / M); });
            in_order();
            clear(own + here, lane, Wave{});
            const int free = here;
            here = next;
            next = after;
            after = free;
        };
        for (; t0 + 2 * kCoactThreads < n; t0 += 2 * kCoactThreads) {
            turn(std::integral_constant<int, 0>{});
            turn(std::integral_constant<int, 1>{});   // it may set an empty slab (a way out between the two made the accumulators spill)
        }
        // the last two slabs are set already; nothing is set, fetched or cleared for turns that do not come
        read(f[1], next);
        if (t0 < n) multiply(f[0], 0, S::NSLOT);
        if (t0 + kCoactThreads < n) multiply(f[1], 0, S::NSLOT);
    } else {
        clear(s_ind, tid, Group{});
        if (n > TOK) clear(s_ind + S::BUFFER, tid, Group{});
        __syncthreads();
        const bool upper = wave >= kCoactWaves / 2;
        Ids ids{};
        if constexpr (FEW) ids.fetch(base, mine * k, last);
        if (!upper) set(s_ind, ids, mine + kCoactThreads, nothing);
        __syncthreads();
        // The four groups walk through loops of their own (with the branch on the group inside of one loop, accumulators spilled) and so meet at
        // four places of the code, where __syncthreads() is not meant for.  The barrier instruction counts arrivals, wherever they come
        // from: what must hold is that every walk makes the same number of rounds, which depends on n alone, and leaves none early.
        auto meet = []() {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        };
        auto walk = [&](auto group) {
            int here = 0, next = S::BUFFER, after = 2 * S::BUFFER;
            bool odd = false;
            auto multiply = [&]() {
                // (cells past the last token of a short pass are zero, so the slabs need no bound of their own)
#pragma unroll
                for (int i = 0; i < S::SLABS / S::SPLIT; ++i) {
                    // the two row fragments and two column fragments at a time: all of them do not fit beside the accumulators
                    constexpr int G = decltype(group)::value, ROW_B = S::NBLK - 1 - G;
                    auto frag = [&](int block) { return coact_frag(s_ind + here + (part + i * S::SPLIT) * S::SLAB + block * 32 * S::PITCH + frag_at); };
                    const i32x8_t a = frag(G), b = frag(ROW_B);
                    i32x8_t x = a;
#pragma unroll
                    for (int c = G; c < S::NBLK; ++c) {
                        const i32x8_t now = x;
                        if (c + 1 < S::NBLK) x = c + 1 == ROW_B ? b : frag(c + 1);
                        coact_mfma(a, now, acc[c - G]);
                        if (c >= ROW_B) coact_mfma(b, now, acc[S::NBLK - G + c - ROW_B]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            for (int t0 = 0; t0 + TOK < n; t0 += TOK) {
                if (upper != odd) set(s_ind + next, ids, mine + kCoactThreads, nothing);
                multiply();
                clear(s_ind + after, tid, Group{});
                meet();
                const int free = here;
                here = next;
                next = after;
                after = free;
                odd = !odd;
            }
            multiply();   // the last pass: nothing is left to set
        };
        if (grp == 0) walk(std::integral_constant<int, 0>{});
        else if (grp == 1) walk(std::integral_constant<int, 1>{});
        else if (grp == 2) walk(std::integral_constant<int, 2>{});
        else walk(std::integral_constant<int, 3>{});
        static_assert(S::GROUPS == 4, "one walk per group");
    }
    // ---- the waves' parts meet in LDS, 16 bits of a count at a time and two rows to a word, which halves what is written and read (all of a
    // wave's blocks are 40 KB of counts at E = 128); thread -> quad of rows (slot, v / 4, lane)
    // accumulator element v of a lane is row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32 of the block
    uint2* const xchg = reinterpret_cast<uint2*>(s_ind);
    auto add_up = [&](auto bits_below) {
        constexpr int kBelow = decltype(bits_below)::value, ROUND = S::ROUND, kQuads = ROUND * 256;   // quads per wave
#pragma unroll
        for (int s0 = 0; s0 < NSLOT; s0 += ROUND) {
            const int n_here = min(ROUND, NSLOT - s0);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ROUND; ++i)
                if (s0 + i < NSLOT)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        auto pair = [&](int v) { return (uint32_t)acc[s0 + i][v] >> kBelow | (uint32_t)acc[s0 + i][v + 1] >> kBelow << 16; };
                        xchg[wave * kQuads + (i * 4 + q) * 64 + lane] = uint2{pair(4 * q), pair(4 * q + 2)};
                    }
            __syncthreads();
            const int n_work = S::GROUPS * n_here * 256;
#pragma unroll 3
            for (int w0 = tid; w0 < n_work; w0 += kCoactThreads) {
                // every workgroup begins at another place, so that they do not queue for the same cells
                int w = w0 + (int)(blockIdx.x % (unsigned)(n_work / 64)) * 64;
                if (w >= n_work) w -= n_work;
                const int g = w / (n_here * 256), at = w % (n_here * 256);
                uint32_t sum[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int p = 0; p < S::SPLIT; ++p) {
                    const uint2 part = xchg[(p * S::GROUPS + g) * kQuads + at];
                    sum[0] += part.x & 0xffffu;
                    sum[1] += part.x >> 16;
                    sum[2] += part.y & 0xffffu;
                    sum[3] += part.y >> 16;
                }
                const int slot = s0 + at / 256, q = (at / 64) & 3, l = at & 63;
                const int bi = S::row_of(g, slot), bj = S::col_of(g, slot), row = 8 * q + 4 * (l >> 5), column = l & 31;
                if (32 * bj + column >= E) continue;
#pragma unroll
                for (int v = 0; v < 4; v += 2) {
                    const int at_row = 32 * bi + row + v, at_col = 32 * bj + column;
                    if (at_row >= E) break;
                    const unsigned long long low = (unsigned long long)sum[v] << kBelow;
                    const unsigned long long high = at_row + 1 < E ? (unsigned long long)sum[v + 1] << kBelow : 0ull;   // (a row past E is not written)
                    if (packed) {
                        if (low | high) atomicAdd(&P[coact_word(E, bi, bj, (row + v) / 2, column)], high << 32 | low);
                    } else {
                        if (low) atomicAdd(&P[(size_t)at_row * E + at_col], low);
                        if (high) atomicAdd(&P[(size_t)(at_row + 1) * E + at_col], high);
                    }
                }
            }
        }
    };
    if (n > S::SHORT) {   // the upper halves first
        add_up(std::integral_constant<int, 16>{});
#pragma unroll
        for (int s = 0; s < NSLOT; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][v] = (float)((uint32_t)acc[s][v] & 0xffffu);
    }
    add_up(std::integral_constant<int, 0>{});
}

// One workgroup per block (bi, bj) on or above the diagonal: spreads out its words if they are packed, and writes block (bj, bi).
// (A mirrored atomic per cell in the kernel above would touch one cache line per lane.)
__global__ __launch_bounds__(512) void k_coact_finish(int E, bool packed, unsigned long long* __restrict__ P) {
    int bi = 0, bj = (int)blockIdx.x;
    for (const int n = (E + 31) / 32; bj >= n - bi; ++bi) bj -= n - bi;
    bj += bi;
    const int rp = threadIdx.x >> 5, c = threadIdx.x & 31;
    const int row = 32 * bi + 2 * rp, column = 32 * bj + c;
    const bool first = row < E && column < E, second = row + 1 < E && column < E;
    unsigned long long v0 = 0, v1 = 0;
    if (packed) {
        if (first) v0 = P[coact_word(E, bi, bj, rp, c)];
        v1 = v0 >> 32;
        v0 &= 0xffffffffull;
    } else {
        if (first) v0 = P[(size_t)row * E + column];
        if (second) v1 = P[(size_t)(row + 1) * E + column];
    }
    __syncthreads();   // every word of this block has been read before the cells that held them are written
    if (first) P[(size_t)row * E + column] = v0;
    if (second) P[(size_t)(row + 1) * E + column] = v1;
    if (bi != bj) {
        if (first) P[(size_t)column * E + row] = v0;
        if (second) P[(size_t)column * E + row + 1] = v1;
    }
}

__global__ void k_fill_u64(unsigned long long* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

}  // namespace

template <class IdxT>
static void launch_coact_t(const IdxT* idx, int64_t T, int k, int E, bool packed, unsigned long long* P, hipStream_t s) {
    // A workgroup has a CU for itself, so there are no more than CUs.  Fewer groups have longer runs but fewer sums queue at the end.
    // Up to about a hundred groups the queueing does not show, so short lists are cut into the shortest useful runs, and beyond the two
    // are even at the root of T.  With one id per token only the diagonal is summed, with two on more than 128 experts few cells.
    // Measured (groups: us), uint8: T = 48000, E = 128, k = 8 8: 22.5, 24: 18.1, 48: 18.1, 94: 18.7; 100000 49: 20.3, 98: 18.9, 196: 23.7;
    // 450000 48: 27.5, 96: 22.9, 128: 23.1, 256: 26.3; 2^21 128: 36.9, 192: 34.3, 256: 36.4; E = 64, k = 8, 450000 48: 18.1, 96: 15.5, 256: 15.6;
    // 2^20 128: 18.5, 256: 18.2, on another box 147: 20.8, 256: 23.4; E = 200, k = 4, 150000 48: 31.8, 96: 27.8, 256: 31.6; 2^20 96: 59.9, 192: 49.7, 256:
    // 51.7; two ids, 100000 48: 29.0, 98: 25.4, 196: 21.8; one id, 450000 64: 44.6, 128: 31.3, 256: 25.9.
    constexpr int64_t kMaxGroups = 256;
    // tokens that a workgroup takes in one turn: two slabs per wave, or two passes (more than 8 ids make a turn long, and few tokens on many
    // experts are worth a workgroup per pass)
    const int64_t unit = E <= 128 && k <= 8 ? 1024 : T <= 1024 ? 256 : 512;
    int64_t groups = (int64_t)std::sqrt((double)T / (E <= 128 ? 48.0 : 28.0));
    groups = std::min(kMaxGroups, std::max(groups, (int64_t)(k == 1 ? 256 : k == 2 && E > 128 ? 192 : 96)));
    groups = std::max(groups, (T + kCoactMaxRun - 1) / kCoactMaxRun);
    const int64_t per = ((T + groups - 1) / groups + unit - 1) / unit * unit;
    const dim3 grid((unsigned)((T + per - 1) / per)), block(kCoactThreads);
#define GROUTER_COACT(EP_)                                                                                         \
    do {                                                                                                           \
        if (k <= 4 && T * k >= 8) hipLaunchKernelGGL((k_coactivation<IdxT, EP_, 4>), grid, block, 0, s, idx, T, k, E, per, packed, P);      \
        else if (k <= 8 && T * k >= 8) hipLaunchKernelGGL((k_coactivation<IdxT, EP_, 8>), grid, block, 0, s, idx, T, k, E, per, packed, P); \
        else hipLaunchKernelGGL((k_coactivation<IdxT, EP_, 0>), grid, block, 0, s, idx, T, k, E, per, packed, P);  \
    } while (0)
    if (E <= 64) GROUTER_COACT(64);
    else if (E <= 128) GROUTER_COACT(128);
    else GROUTER_COACT(256);
#undef GROUTER_COACT
}

hipError_t launch_coactivation(const void* idx, int idx_dtype, int64_t T, int k, int E, int64_t* P, hipStream_t s) {
    auto* p = reinterpret_cast<unsigned long long*>(P);
    const int64_t n = (int64_t)E * E;
    const int blocks = (E + 31) / 32;
    // one block needs no finishing launch if its cells are added where they belong; a count of 2^32 does not fit half a word
    const bool packed = blocks > 1 && T < (1ll << 32);
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    if (idx_dtype == 1) launch_coact_t((const uint8_t*)idx, T, k, E, packed, p, s);
    else launch_coact_t((const int32_t*)idx, T, k, E, packed, p, s);
    if (blocks > 1) hipLaunchKernelGGL(k_coact_finish, dim3((unsigned)(blocks * (blocks + 1) / 2)), dim3(512), 0, s, E, packed, p);
    return hipGetLastError();
}

}  // namespace grouter
