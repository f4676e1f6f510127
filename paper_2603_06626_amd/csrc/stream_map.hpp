// Which tile a workgroup of k_stream_gemm takes, where its waves put their partial sums and who adds them up.  Apart from
// the kernel and free of device types, so that a host program can enumerate every access.
#pragma once

#if defined(__HIPCC__)
#define GROUTER_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define GROUTER_HOST_DEVICE inline
#endif

namespace grouter {

// Workgroup -> (row tile mt, column block cb).
// Workgroups of one expert: the 8 XCDs take one contiguous run of column blocks each, so a line that two blocks share is
// fetched by one L2.  Where rows do not begin on a line, every block shares its first and last line with its neighbours:
// given enough experts, one XCD then takes all blocks of an expert (by_expert).
// n_tiles() loads the plan header and gives the number of row tiles, negative for a plan of other dimensions; record(mt) loads
// the record of tile mt.  The record is loaded only after the header has vouched for it: a plan of other
// dimensions may be a smaller allocation that ends before the place where the caller's dimensions put the record.
struct StreamTile {
    int mt, cb;
    template <class NTiles, class Record>
    GROUTER_HOST_DEVICE bool pick(int block, int n_col_blocks, bool by_expert, NTiles n_tiles, Record record) {
        if (by_expert) {
            const int q = block >> 3;
            mt = q / n_col_blocks * 8 + (block & 7);
            cb = q % n_col_blocks;
        } else {
            const int per_xcd = (n_col_blocks + 7) >> 3;
            mt = block / (per_xcd * 8);
            const int b = block - mt * per_xcd * 8;
            cb = (b & 7) * per_xcd + (b >> 3);
        }
        if (mt >= n_tiles() || cb >= n_col_blocks) return false;
        record(mt);
        return true;
    }
};

constexpr int kStreamRows = 16;   // rows of one MFMA, and of one round of partial sums

// Partial sums of 16 rows x NB * COLS columns, fp32, one area per wave.
template <int NB, int COLS>
struct StreamSums {
    static constexpr int kPitch = NB * COLS * 4 + 16;            // bytes of a row
    static constexpr int kWaveBytes = kStreamRows * kPitch;
    static constexpr int kPerRow = COLS / 4;                     // a thread finishes 4 columns of one row
    static constexpr int kThreads = kStreamRows * kPerRow;       // threads that have something to finish
    int row, col;   // inside the 16 rows and the COLS columns
    GROUTER_HOST_DEVICE explicit StreamSums(int tid) : row(tid / kPerRow), col(tid % kPerRow * 4) {}
    // rows_left, cols_left: what exists from the round's first row and the workgroup's first column on.  A workgroup has
    // more threads than a round has quads: without the first condition they would take rows of the next round.
    GROUTER_HOST_DEVICE bool finishes(int rows_left, int cols_left) const { return row < kStreamRows && row < rows_left && col < cols_left; }
    GROUTER_HOST_DEVICE int at(int wave, int nb) const { return wave * kWaveBytes + row * kPitch + (nb * COLS + col) * 4; }
};

}  // namespace grouter
