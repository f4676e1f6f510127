// Where k_stream_gemm puts its waves' partial sums and who adds them up.  Apart from the kernel and free of device types, so
// that a host program can enumerate every access.
#pragma once

#if defined(__HIPCC__)
#define GROUTER_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define GROUTER_HOST_DEVICE inline
#endif

namespace grouter {

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
