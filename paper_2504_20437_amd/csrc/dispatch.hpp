// Rules that choose between the forms of a kernel by the sizes of a call. Plain
// host code, so that tests can ask for the choice a launch makes. Times of single
// kernels here and beside them in the sources are device times on one MI355X, the
// forms taken in turn in one process: event pairs around many back-to-back calls
// of the entry point, or around the stage of a traced update.
#pragma once
#include <cstdint>

namespace galore {

// The column scans of a projector (sign convention, switch): workgroups of 16
// columns and 512 threads instead of 64 columns and 256, while the latter would
// leave CUs idle. A 16-column workgroup reads 64-byte pieces of rows and moves
// half the bytes per second once the chip is full.
//   sign (whole stage): 4096x1024 projectors, 1: 100 -> 45 us; 8 (128 workgroups of
//   64 columns): 160 -> 117; 10: 171 against 180 narrow; 25: 313 against 417; 64:
//   663 against 988. 2048x256: 40: 87 -> 82, 64: 114 against 147. Below 1024 rows
//   combining 128 row groups costs more than the scan saves (512x128, 1: 27.5
//   against 29.4, 64: 29.9 against 38.4).
inline bool narrow_sign_columns(int rows, int r, int64_t batch) {
    return rows >= 1024 && static_cast<int64_t>((r + 63) / 64) * batch < 144;
}
//   switch: 4096x1024, 1: 39 -> 19 us; 6 (96 workgroups): 66 -> 65; 7: 66 against 69
//   narrow, 8: 67 against 80, 64: 364 against 682; 1024x256, 32: 18 against 22.
inline bool narrow_align_columns(int r, int64_t batch) {
    return static_cast<int64_t>((r + 63) / 64) * batch < 112;
}

}  // namespace galore
