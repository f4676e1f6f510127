// Forward grouped GEMMs: G,U = x_rows W1_e, x_rows W3_e with the fused gate-weighted SiLU*up epilogue (the rows of
// x read through the plan's row map), and O = H W2_e.
#include "gemm_kernels.hpp"
#include "gemm_stream.hpp"

namespace grouter {

static RowsArgs base_args(const PlanView& P) {
    RowsArgs a{};
    a.tiles = P.tiles_small;
    a.max_tiles = P.max_tiles_small;
    a.plan = P.dims();
    a.col_group = 3;  // measured best of 0 (plain order), 1, 2, 3 on the forward GEMMs
    return a;
}

static unsigned rows_grid(const PlanView& P, int n_ntiles) { return (unsigned)P.max_tiles_small * (unsigned)n_ntiles; }

// Up to 16 tokens no expert holds more than 16 rows (unless a token names it twice): the streaming kernels then read the
// weights once at full width.  From 17 on the 128-row tiles fill the chip and are as fast (T = 16: 350 us against 375 us
// for two layers of d = 2048, f = 1408, E = 64, k = 6; 1090 us both for d = 4096, f = 1536, E = 128, k = 8), while here an
// expert's second 16 rows would read its weights again (T = 200: 366 us against 211 us).
template <int MODE>
static bool launch_stream(const PlanView& P, RowsArgs a, hipStream_t s) {
    constexpr int kCpl = 4, kWaves = 8, kStages = 2;
    if (P.T > kStreamRows) return false;
    a.n_ntiles = (a.Ncols + 16 * kCpl - 1) / (16 * kCpl);
    const int64_t tiles = P.max_tiles_small < P.N ? P.max_tiles_small : P.N;   // no tile is empty
    const dim3 grid((unsigned)(tiles * ((a.n_ntiles + 7) / 8 * 8)));
    hipLaunchKernelGGL((k_stream_gemm<MODE, kCpl, kWaves, kStages>), grid, dim3(kWaves * 64), 0, s, a);
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
