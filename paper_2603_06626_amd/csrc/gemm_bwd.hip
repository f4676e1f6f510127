// Backward grouped GEMMs, in two launches of two products each: dW2_e = (gate * H)_e^T dY_e together with
// dH = gate * (dY rows) W2_e^T and its dSwiGLU epilogue; then dW1_e = x_e^T dG_e, dW3_e = x_e^T dU_e together with
// dXp = dG W1_e^T + dU W3_e^T.  x_e and dY_e are the expert's rows of the token-ordered x and dY, read through the
// plan's row map.
#include "gemm_kernels.hpp"

namespace grouter {

static RowsArgs rows_args(const PlanView& P) {
    RowsArgs a{};
    a.tiles = P.tiles_small;
    a.plan = P.dims();
    return a;
}

static DwArgs dw_args(const PlanView& P) {
    DwArgs a{};
    a.plan = P.dims();
    a.by_load = P.by_load;
    a.offsets = P.offsets;
    a.counts = P.counts;
    a.row_token = P.row_token;
    a.n_experts = P.E;
    return a;
}

static unsigned rows_grid(const PlanView& P, int n_ntiles) { return (unsigned)P.max_tiles_small * (unsigned)n_ntiles; }

// Workgroups of the weight-gradient tiles of four experts of neighbouring load ranks: 8 XCDs x (largest per-XCD share); the
// share pattern repeats every 4 experts.
static unsigned dw_grid_of_four(int n_mt, int n_nt) {
    int worst = 0;
    for (int x = 0; x < 8; ++x) {
        int per_quad = 0;
        for (int tq = 0; tq < 4; ++tq) per_quad += DwShare(x, tq, n_mt, n_nt).tiles();
        worst = per_quad > worst ? per_quad : worst;
    }
    return 8u * (unsigned)worst;
}

// Whether the weight gradients take the step loop with fragments in two register sets (step_pipeline_ahead).  Measured over
// uniform and skewed loads, 8 to 64 experts, d from 256 to 4096 (time without / with it):
//   dW2       mean rows per expert 128: 0.99-1.04, 192: 0.99-1.06, 256: 0.96-1.05, 384: 1.02-1.09, 768: 0.98-1.08, 2048: 0.99-1.08
//   dW1/dW3   below 512 rows: 0.96-1.03; from 512 on with at least 8192 tiles (16 times what is resident) 0.99-1.02,
//             T = 16384, d = 4096, f = 1536, E = 128, k = 8 1.045; with fewer tiles 0.94-1.03
// Short reductions lose most: 8 rows per expert (T = 128, d = 4096, f = 1536, E = 128, k = 8) dW2 298 us without, 338 with it;
// 64 rows (T = 2048, d = f = 1024, E = 64, k = 2) dW1/dW3 73 and 80 us.
static bool two_register_sets(BwdMode mode, const PlanView& P, const DwArgs& w) {
    const int64_t mean_rows = P.N / P.E;
    return mode == kDh ? mean_rows >= 256 : mean_rows >= 512 && (int64_t)P.E * w.n_mt * w.n_nt >= 8192;
}

// Whether the row tiles open the grid.  A row tile has 2 K / 64 steps (for each of dXp's two phases), a weight-gradient tile one
// per 32 rows of its expert, and the hottest experts hold several times the mean (2 to 10 times with Zipf exponents around
// 1.2).  Where 4 times the mean reaches the row tiles' length, the heaviest eighth of the experts goes first.  Measured, rows
// first / heaviest eighth first: T = 500, d = 256, f = 1536, E = 128, k = 8, skewed (mean 0 and row tiles 8 and 96 steps):
// 167 / 193 us; T = 1334, d = 1600, f = 768, E = 16, k = 3 (7; 50, 48): 95 / 106; T = 4000, d = 512, f = 1536, E = 96, k = 4 (5; 16, 96):
// 349 / 331, each product by this rule 320; T = 9000, d = 704, f = 1088, E = 64, k = 5 (21; 22, 68): 604 / 558, by this
// rule 560; T = 16384, the same widths (40; 22, 68): 1076 / 972, 963.
static bool rows_first(BwdMode mode, const PlanView& P, const RowsArgs& a) {
    const int64_t row_steps = (mode == kDxp ? 4 : 2) * (int64_t)((a.K + 63) / 64);
    return 4 * (P.N / P.E / 32) < row_steps;
}

template <BwdMode MODE>
static hipError_t launch_pair(BwdPart part, const PlanView& P, const DwArgs& w, const RowsArgs& a, hipStream_t s) {
    const unsigned fours = (unsigned)((P.E + 3) / 4), per_four = dw_grid_of_four(w.n_mt, w.n_nt);
    const unsigned n_dw = part == kBwdRows ? 0u : fours * per_four;
    const unsigned n_rows = part == kBwdWeights ? 0u : (rows_grid(P, a.n_ntiles) + 7u) / 8u * 8u;
    const unsigned head = part == kBwdBoth && !rows_first(MODE, P, a) ? (fours + 7u) / 8u * per_four : 0u;
    const dim3 grid(n_dw + n_rows), block(kThreads);
    if (two_register_sets(MODE, P, w)) hipLaunchKernelGGL((k_bwd_pair<MODE, true>), grid, block, 0, s, w, a, (int)n_dw, (int)head, (int)n_rows);
    else hipLaunchKernelGGL((k_bwd_pair<MODE, false>), grid, block, 0, s, w, a, (int)n_dw, (int)head, (int)n_rows);
    return hipGetLastError();
}

hipError_t launch_dw2_dh(BwdPart part, const PlanView& P, int d, int f, const bf16_t* dY, const float* row_gate, const bf16_t* H, const bf16_t* W2,
                         const bf16_t* dSdG, const bf16_t* dSdU, bf16_t* dW2, bf16_t* dG, bf16_t* dU, hipStream_t s) {
    DwArgs w = dw_args(P);
    // H is the saved gate-weighted H, so the upstream gradient enters unscaled, straight from dY [T][d]
    w.A = H; w.B0 = dY; w.C0 = dW2;
    w.Mdim = f; w.Ndim = d; w.n_mt = (f + kTileM - 1) / kTileM; w.n_nt = (d + 255) / 256;
    w.gathered_bytes = (uint32_t)((uint64_t)P.T * (uint64_t)d * 2u);
    RowsArgs a = rows_args(P);
    a.A0 = dY; a.B0 = W2; a.E0 = dSdG; a.E1 = dSdU; a.C0 = dG; a.C1 = dU;
    a.K = d; a.Ncols = f; a.n_ntiles = (f + 255) / 256;
    a.row_token = P.row_token; a.a_total_bytes = w.gathered_bytes;
    a.row_gate = row_gate;
    a.col_group = 3;   // column tiles walked in groups, row tiles fastest (as in the forward GEMMs): measured -2 % against the plain order
    return launch_pair<kDh>(part, P, w, a, s);
}

hipError_t launch_dw13_dxp(BwdPart part, const PlanView& P, int d, int f, const bf16_t* x, const bf16_t* dG, const bf16_t* dU, const bf16_t* W1,
                           const bf16_t* W3, bf16_t* dW1, bf16_t* dW3, bf16_t* dXp, hipStream_t s) {
    DwArgs w = dw_args(P);
    w.A = x; w.B0 = dG; w.B1 = dU; w.C0 = dW1; w.C1 = dW3;
    w.Mdim = d; w.Ndim = f; w.n_mt = (d + kTileM - 1) / kTileM; w.n_nt = (f + 127) / 128;
    w.gathered_bytes = (uint32_t)((uint64_t)P.T * (uint64_t)d * 2u);
    RowsArgs a = rows_args(P);
    a.A0 = dG; a.A1 = dU; a.B0 = W1; a.B1 = W3; a.C0 = dXp;
    a.K = f; a.Ncols = d; a.n_ntiles = (d + 255) / 256;
    a.col_group = 4;   // measured best of 0 (plain order), 2, 3, 4: -2 %
    return launch_pair<kDxp>(part, P, w, a, s);
}

}  // namespace grouter
