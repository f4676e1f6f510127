// Forward GEMMs for few tokens (decoding).
//
// With so few rows per expert the layer reads every weight of the experts in use once and does next to no arithmetic per
// byte: HBM bandwidth is the bound, and what matters is that all CUs have loads in flight from the first microsecond on.
// The 128-row tiles do not manage that: for one token they are 66 workgroups that walk the whole of K in steps of 32
// rows, each step waiting for LDS copies and a barrier.
//
// Here a workgroup owns 64 columns of one expert and its waves share out K: wave w takes every W-th block of 32 K-rows
// and has STAGES of them in flight.  Weights go straight from memory to registers, with no LDS and no barrier in the
// loop.  A lane loads 4 columns of 8 K-rows and turns them into MFMA operands with one v_perm per two elements: the K-rows
// 8 (l / 16) .. + 7 of column 4 (l % 16) + j are the 8 consecutive K values per lane that the 16x16x32 operand of block
// j wants, if block j is taken to be the columns 4 c + j.  A lane of the accumulators then holds 16 consecutive columns
// of one row.  The activations' operand (RB blocks of 16 rows, 8 consecutive K per lane) is loaded directly, too.  At the end the waves'
// partial sums meet in LDS and are added in wave order, so results do not depend on timing.
//
// Measured, 128-row tiles -> here (d = 2048, f = 1408, E = 64, k = 6, between events): one token gate/up 31.5 -> 16 us, down
// 23.7 -> 11, that is 4.3 and 3.2 TB/s; a layer with its combine 61 -> 26; T = 4 79 -> 72; T = 16 181 -> 164 (5.4 TB/s); d = 4096 and
// E = 128 at T = 16 unchanged (5.6 TB/s, what this memory gives).  4 columns per lane (whole 128-byte lines per K-row) beat 2 (27 us) and 8 (30 us, too
// few workgroups); 8 waves beat 4 and 16; 1 to 8 stages are within 1 % once every wave has a block for each.
#pragma once
#include "gemm_kernels.hpp"
#include "stream_map.hpp"

namespace grouter {

enum StreamMode { kStreamGateUp = 0, kStreamGateUpOnly = 1, kStreamDown = 2 };

struct StreamArgs : RowsArgs {
    StreamOrder order;   // of the workgroups; the column blocks of n_ntiles are 64 wide
};

// RB: row blocks of 16 that share one pass over the weights
template <int MODE, int W, int STAGES, int RB>
__global__ __launch_bounds__(W * 64, RB == 1 && STAGES == 1 ? 4 : 2) void k_stream_gemm(const StreamArgs a) {
    constexpr bool GATEUP = MODE != kStreamDown;
    constexpr int NB = GATEUP ? 2 : 1;
    constexpr int CPL = kStreamCols / 16, kCols = kStreamCols;
    using Sums = StreamSums<NB, kCols>;
    static_assert(CPL == 4, "8 bytes of every K-row per lane");
    __shared__ __attribute__((aligned(16))) char smem[W * Sums::kWaveBytes];

    typedef int32_t i32x8 __attribute__((ext_vector_type(8)));
    i32x8 rec;
    StreamTile tile;
    if (!tile.pick((int)blockIdx.x, a.n_ntiles, a.order, [&]() { return a.plan.row_tiles(); },
                   [&](int mt) { rec = *(const i32x8*)(a.tiles + 8 * (size_t)mt); }))
        return;
    const int col0 = tile.cb * kCols;
    const int e = rec[0], m_in = tile.mt - rec[3];
    const int tile_row0 = rec[1] + m_in * kTileM;
    const int tile_rows = min(kTileM, rec[2] - m_in * kTileM);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g16 = lane >> 4;
    const int K = a.K, Ncols = a.Ncols;
    const int n_blocks = (K + 31) / 32;

    const uint32_t slab_bytes = (uint32_t)K * (uint32_t)Ncols * 2u;
    const size_t slab = (size_t)e * K * Ncols;
    __amdgpu_buffer_rsrc_t bufB[NB];
    bufB[0] = __builtin_amdgcn_make_buffer_rsrc((void*)(a.B0 + slab), 0, (int)slab_bytes, 0x00020000);
    if constexpr (NB == 2) bufB[1] = __builtin_amdgcn_make_buffer_rsrc((void*)(a.B1 + slab), 0, (int)slab_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t bufA = __builtin_amdgcn_make_buffer_rsrc((void*)a.A0, 0, (int)a.a_total_bytes, 0x00020000);
    const uint32_t row_b = (uint32_t)Ncols * 2u;
    const int b_col = col0 + l16 * CPL;
    const uint32_t b_voff = b_col < Ncols ? (uint32_t)(8 * g16) * row_b + b_col * 2u : kOutOfRange;

    // an expert of more than 16 RB rows (only possible when a token names it more than once) takes several turns
    for (int r0 = 0; r0 < tile_rows; r0 += kStreamRows * RB) {
        const int rows = min(kStreamRows * RB, tile_rows - r0);
        struct Block {
            uint32_t b[NB][8][2];   // not register pairs: those spill with one stage
            u32x4 a[RB];
        };
        Block st[STAGES];
        auto load_b = [&](int kb, Block& s) {
            // K is a multiple of 8, so a lane's 8 K-rows exist or do not together; what does not exist reads as zero
            const uint32_t soff = kb < n_blocks ? (uint32_t)kb * 32u * row_b : 0u;
            const uint32_t voff = kb * 32 + 8 * g16 < K ? b_voff : kOutOfRange;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(bufB[nb], (int)voff, (int)(soff + i * row_b), 0);
                    s.b[nb][i][0] = v.x;
                    s.b[nb][i][1] = v.y;
                }
        };
#pragma unroll
        for (int s = 0; s < STAGES; ++s) load_b(wave + s * W, st[s]);
        uint32_t a_voff[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int my_row = tile_row0 + r0 + min(rb * kStreamRows + l16, rows - 1);
            a_voff[rb] = ((GATEUP ? (uint32_t)a.row_token[my_row] : (uint32_t)my_row) * (uint32_t)K + 8u * g16) * 2u;
        }
        auto load_a = [&](int kb, Block& s) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                s.a[rb] = __builtin_amdgcn_raw_buffer_load_b128(bufA, (int)(kb * 32 + 8 * g16 < K ? a_voff[rb] : kOutOfRange), kb * 64, 0);
        };
#pragma unroll
        for (int s = 0; s < STAGES; ++s) load_a(wave + s * W, st[s]);
        f32x4 acc[RB][NB][CPL];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < CPL; ++j) acc[rb][nb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto multiply = [&](const Block& s) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < CPL; ++j) {
                    u32x4 w;
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        w[p] = __builtin_amdgcn_perm(s.b[nb][2 * p + 1][j >> 1], s.b[nb][2 * p][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[rb][nb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, s.a[rb]), acc[rb][nb][j], 0, 0, 0);
                }
        };
        int kb = wave;
        for (; kb + STAGES * W < n_blocks; kb += STAGES * W) {
#pragma unroll
            for (int s = 0; s < STAGES; ++s) {
                multiply(st[s]);
                load_b(kb + (s + STAGES) * W, st[s]);
                load_a(kb + (s + STAGES) * W, st[s]);
            }
        }
#pragma unroll
        for (int s = 0; s < STAGES; ++s) multiply(st[s]);   // blocks past the end are all zero

        // ---- the waves' partial sums meet in LDS
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb * kStreamRows >= rows) break;
            if (r0 + rb) __syncthreads();
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int h = 0; h < CPL; ++h) {   // columns 4 h .. + 3 of this lane's 16
                    f32x4 v;
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = acc[rb][nb][(4 * h + c) % CPL][(4 * h + c) / CPL];
                    *(f32x4*)(smem + wave * Sums::kWaveBytes + l16 * Sums::kPitch + (nb * kCols + g16 * 4 * CPL + h * 4) * 4) = v;
                }
            __syncthreads();
            static_assert(Sums::kThreads <= W * 64, "one quad per thread");
            const Sums mine(tid);
            if (mine.finishes(rows - rb * kStreamRows, Ncols - col0)) {
                f32x4 sum[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    sum[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int w = 0; w < W; ++w) sum[nb] += *(const f32x4*)(smem + mine.at(w, nb));
                }
                const int row = tile_row0 + r0 + rb * kStreamRows + mine.row;
                const size_t at = (size_t)row * Ncols + col0 + mine.col;
                if constexpr (GATEUP) {
                    const float gate = a.row_gate[row];
                    float P[4], Q[4], H[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float g = sum[0][c], u = sum[NB - 1][c];
                        const float s = sigmoid_fast(g);
                        Q[c] = g * s;
                        P[c] = u * (s + Q[c] * (1.f - s));
                        H[c] = gate * (Q[c] * u);
                    }
                    if constexpr (MODE == kStreamGateUp) {
                        *(u32x2*)(a.C0 + at) = u32x2{pack_bf16_rne(P[0], P[1]), pack_bf16_rne(P[2], P[3])};
                        *(u32x2*)(a.C1 + at) = u32x2{pack_bf16_rne(Q[0], Q[1]), pack_bf16_rne(Q[2], Q[3])};
                    }
                    *(u32x2*)(a.C2 + at) = u32x2{pack_bf16_rne(H[0], H[1]), pack_bf16_rne(H[2], H[3])};
                } else {
                    *(u32x2*)(a.C0 + at) = u32x2{pack_bf16_rne(sum[0][0], sum[0][1]), pack_bf16_rne(sum[0][2], sum[0][3])};
                }
            }
        }
    }
}

}  // namespace grouter
