// Forward grouped GEMMs: G,U = x_rows W1_e, x_rows W3_e with the fused gate-weighted SiLU*up epilogue (the rows of
// x read through the plan's row map), and O = H W2_e.
#include "gemm_kernels.hpp"
#include "gemm_stream.hpp"

namespace grouter {

static RowsArgs base_args(const PlanView& P) {
    RowsArgs a{};
    a.tiles = P.tiles_small;
    a.plan = P.dims();
    a.col_group = 3;  // measured best of 0 (plain order), 1, 2, 3 on the forward GEMMs
    return a;
}

static unsigned rows_grid(const PlanView& P, int n_ntiles) { return (unsigned)P.max_tiles_small * (unsigned)n_ntiles; }

// When the streaming kernels take over.  Up to 16 tokens no expert holds more than 16 rows (unless a token names it twice)
// and they read the weights once at full width.  From 17 to 64 tokens they still read them once, with 2 or 4 row
// blocks, which pays where the 128-row tiles are too few to occupy the chip.  Measured, time of the 128-row tiles over the
// streaming kernels' by number of tiles (128 columns for gate/up, 256 for down):
//   17 to 32 tokens   gate/up 64 to 126 tiles 1.35-1.64, 135 to 200 0.84-1.08, 230 to 310 0.95-1.11; down to 126 1.2-1.9, 140 to 200
//                     1.0-1.2, 220 to 450 0.85-1.0
//   33 to 64 tokens   gate/up 64 to 128 1.27-1.50, 130 to 190 0.88-1.0; down to 128 1.05-1.8 (but 0.94 with K = 256), 130 to 140
//                     0.82-0.97, 180 to 510 0.65-0.92
// and a second pass over the weights loses (d = 568, f = 1088, E = 8, k = 2, T = 100: 33 -> 35 us).
// Stages: with K of at most one block per wave a second stage would only load zeros (d = 256, f = 576, E = 128, k = 7,
// T = 16: 28.5 -> 25.1 us).  With more workgroups than CUs one stage lets two share a CU, which pays as long as a wave has few
// blocks (two stages / one: K = 768 gate/up 45 / 39 us and down 39 / 36.5, K = 1024 gate/up 27.5 / 26.5; but K = 1000 down 27.9 / 28.3,
// K = 3072 gate/up 67 / 67); where every CU has a workgroup at most, two stages are 3 to 10 % faster.
// Order: runs of ceil(blocks / 8) column blocks per XCD are even where the blocks come in eights, and then 3 to 6 % faster than
// the plain order (d = 4096, f = 1536, E = 128, k = 8, T = 12: gate/up 314 / 331 us, down 149 / 159).  Otherwise some XCDs get less
// or nothing (runs / plain): 12 blocks, d = 2048, f = 768, E = 128, k = 8, T = 6 gate/up 60.6 / 47.7 us; 22 blocks, d = 2048,
// f = 1408, E = 64, k = 6, T = 12 101 / 91; 4 blocks, d = f = 256, E = 48, k = 2, T = 32 12.1 / 8.6; 2 and 4 blocks, d = 128, f = 256,
// E = 128, k = 1, T = 48 the layer 20.2 / 14.7 (19 with the 128-row tiles).
// By expert: with rows of 592 bytes (d = 704, f = 296, E = 64, k = 5, T = 10), where neighbouring column blocks share lines,
// three layers take 121 us with an expert's blocks spread over the XCDs and 87 us on one.
constexpr int64_t kStreamTiles = 128;

// Up to 16 tokens the streaming kernels lose where the 128-row tiles number 160 to 256, that is one workgroup on nearly every
// CU and no second round, while the streaming ones take two rounds: gate/up with K = 3072 or 4096 0.91-0.96 of the
// tiles' speed, and with rows that do not begin on a line (d = 1928, f = 1000) 0.88-0.92; otherwise 0.94-1.2.  Down
// with K > 768 (two stages) and 192 tiles or more 0.87-0.97.  Beyond 256 tiles they are as fast or faster again (T = 12,
// d = 1928, f = 1000, E = 60, k = 5: 113 -> 105 us a layer).  The host does not know how many experts the tokens pick; this is the
// number expected of evenly spread picks.  Skewed picks touch fewer: the same layer with Zipf loads has 216 tiles where 311 are
// expected and takes 80 us instead of 73.
static bool tiles_fill_one_round(const PlanView& P, const RowsArgs& a, bool down) {
    double missed = 1.0;
    for (int64_t t = 0; t < P.T; ++t) missed *= 1.0 - (double)P.k / P.E;
    const double tiles = P.E * (1.0 - missed) * a.n_ntiles;
    if (tiles > 256.0) return false;
    return down ? a.K > 768 && tiles >= 192.0 : (a.K >= 3072 || a.Ncols % 64 != 0) && tiles > 160.0;
}

template <int MODE>
static bool launch_stream(const PlanView& P, const RowsArgs& rows, hipStream_t s) {
    constexpr int kWaves = 8;
    const int64_t tiles = P.max_tiles_small < P.N ? P.max_tiles_small : P.N;   // no tile is empty
    const bool few_rows = P.T <= kStreamRows;
    if (few_rows ? tiles_fill_one_round(P, rows, MODE == kStreamDown) : P.T > 4 * kStreamRows || tiles * rows.n_ntiles > kStreamTiles) return false;
    StreamArgs a{rows, kStreamPlain};
    a.n_ntiles = (a.Ncols + kStreamCols - 1) / kStreamCols;
    if (a.Ncols % kStreamCols != 0) a.order = tiles >= 32 ? kStreamByExpert : kStreamRuns;   // a block is as wide as a line; with fewer experts some XCDs would idle
    else if (a.n_ntiles % 8 == 0) a.order = kStreamRuns;
    const bool one_stage = a.K <= 32 * kWaves || (tiles * a.n_ntiles > 256 && a.K <= (MODE == kStreamDown ? 768 : 1024));
    const dim3 grid((unsigned)stream_grid(a.order, (int)tiles, a.n_ntiles)), block(kWaves * 64);
    if (few_rows && one_stage) hipLaunchKernelGGL((k_stream_gemm<MODE, kWaves, 1, 1>), grid, block, 0, s, a);
    else if (few_rows) hipLaunchKernelGGL((k_stream_gemm<MODE, kWaves, 2, 1>), grid, block, 0, s, a);
    else if (P.T <= 2 * kStreamRows) hipLaunchKernelGGL((k_stream_gemm<MODE, kWaves, 2, 2>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_stream_gemm<MODE, kWaves, MODE == kStreamDown ? 2 : 1, 4>), grid, block, 0, s, a);
    return true;
}

hipError_t launch_gateup(const PlanView& P, int d, int f, const bf16_t* x, const float* row_gate, const bf16_t* W1,
                         const bf16_t* W3, bf16_t* dSdG, bf16_t* dSdU, bf16_t* H, hipStream_t s) {
    RowsArgs a = base_args(P);
    a.A0 = x; a.B0 = W1; a.B1 = W3; a.C0 = dSdG; a.C1 = dSdU; a.C2 = H;
    a.K = d; a.Ncols = f; a.n_ntiles = (f + 127) / 128;
    a.row_token = P.row_token; a.a_total_bytes = (uint32_t)((uint64_t)P.T * (uint64_t)d * 2u);
    a.row_gate = row_gate;
    if (dSdG && dSdU ? launch_stream<kStreamGateUp>(P, a, s) : launch_stream<kStreamGateUpOnly>(P, a, s)) return hipGetLastError();
    if (dSdG && dSdU)
        hipLaunchKernelGGL((k_fwd_gemm<kGateUp, true, false>), dim3(rows_grid(P, a.n_ntiles)), dim3(kThreads), 0, s, a);
    else  // forward only: nothing is kept for backward
        hipLaunchKernelGGL((k_fwd_gemm<kGateUp, true, true>), dim3(rows_grid(P, a.n_ntiles)), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_down(const PlanView& P, int d, int f, const bf16_t* H, const bf16_t* W2, bf16_t* O, hipStream_t s) {
    RowsArgs a = base_args(P);
    a.A0 = H; a.B0 = W2; a.C0 = O;
    a.K = f; a.Ncols = d; a.n_ntiles = (d + 255) / 256;
    a.a_total_bytes = (uint32_t)((uint64_t)P.N * (uint64_t)f * 2u);
    if (launch_stream<kStreamDown>(P, a, s)) return hipGetLastError();
    hipLaunchKernelGGL(k_fwd_gemm<kDown>, dim3(rows_grid(P, a.n_ntiles)), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace grouter
