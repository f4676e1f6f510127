// Which tile a workgroup of k_stream_gemm takes, where its waves put their partial sums and who adds them up.  Apart from
// the kernel and free of device types, so that a host program can enumerate every access.
#pragma once

#if defined(__HIPCC__)
#define GROUTER_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define GROUTER_HOST_DEVICE inline
#endif

namespace grouter {

// Workgroup -> (row tile mt, column block cb).  Consecutive workgroups go to the 8 XCDs in turn, each with its own L2.
//   kStreamPlain     block after block: the XCDs share the work evenly.  For rows that begin on a 128-byte line, where no two
//                    blocks share a line.
//   kStreamRuns      the XCDs take one contiguous run of an expert's column blocks each, so a line that two blocks share is
//                    mostly fetched by one L2
//   kStreamByExpert  one XCD takes all blocks of an expert
enum StreamOrder { kStreamPlain = 0, kStreamRuns = 1, kStreamByExpert = 2 };

// Workgroups that cover max_tiles row tiles.
GROUTER_HOST_DEVICE int stream_grid(StreamOrder order, int max_tiles, int n_col_blocks) {
    if (order == kStreamPlain) return max_tiles * n_col_blocks;
    if (order == kStreamRuns) return max_tiles * ((n_col_blocks + 7) / 8 * 8);
    return (max_tiles + 7) / 8 * 8 * n_col_blocks;
}

// n_tiles() loads the plan header and gives the number of row tiles, negative for a plan of other dimensions; record(mt) loads
// the record of tile mt.  The record is loaded only after the header has vouched for it: a plan of other
// dimensions may be a smaller allocation that ends before the place where the caller's dimensions put the record.
struct StreamTile {
    int mt, cb;
    template <class NTiles, class Record>
    GROUTER_HOST_DEVICE bool pick(int block, int n_col_blocks, StreamOrder order, NTiles n_tiles, Record record) {
        if (order == kStreamPlain) {
            mt = block / n_col_blocks;
            cb = block - mt * n_col_blocks;
        } else if (order == kStreamRuns) {
            const int per_xcd = (n_col_blocks + 7) >> 3;
            mt = block / (per_xcd * 8);
            const int b = block - mt * per_xcd * 8;
            cb = (b & 7) * per_xcd + (b >> 3);
        } else {
            const int q = block >> 3;
            mt = q / n_col_blocks * 8 + (block & 7);
            cb = q % n_col_blocks;
        }
        if (mt >= n_tiles() || cb >= n_col_blocks) return false;
        record(mt);
        return true;
    }
};

constexpr int kStreamRows = 16;   // rows of one MFMA, and of one round of partial sums
constexpr int kStreamCols = 64;   // columns of a workgroup

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
