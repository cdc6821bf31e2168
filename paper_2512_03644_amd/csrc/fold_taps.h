// Generated by gen_fold_taps.py -- do not edit.  Sparse multiples of the CRC32C generator;
// see the generator's docstring for the algebra.  TAP_E/TAP_F[f][k]: the dword that
// leaves the top of column f is XORed into state position (row TAP_E, column TAP_F).
#pragma once

namespace ffsnap {

struct Fold16x16 {
    static constexpr int ROW_BYTES = 1024;  // bytes one wavefront reads per step
    static constexpr int STRIDE = 256;     // dword distance between a lane's rows
    static constexpr int NF = 4;         // dwords per lane per row
    static constexpr int NE = 16;         // rows of state
    static constexpr int NTAP = 9;       // slots per column (255 = unused)
    static constexpr unsigned char TAP_E[NF][NTAP] = {{0, 0, 7, 8, 9, 9, 13, 15, 15}, {0, 2, 3, 4, 5, 6, 7, 9, 13}, {0, 0, 0, 2, 4, 5, 5, 9, 12}, {0, 2, 3, 4, 6, 10, 14, 14, 14}};
    static constexpr unsigned char TAP_F[NF][NTAP] = {{0, 1, 2, 1, 0, 3, 3, 2, 3}, {0, 1, 3, 0, 3, 0, 1, 0, 2}, {0, 1, 2, 1, 2, 1, 3, 0, 1}, {1, 3, 0, 0, 3, 3, 0, 1, 3}};
};

}  // namespace ffsnap
