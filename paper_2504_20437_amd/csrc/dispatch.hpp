// Rules that choose between the forms of a kernel by the sizes of a call. Plain
// host code, so that tests can ask for the choice a launch makes. Times of single
// kernels here and beside them in the sources are device times on one MI355X, the
// forms taken in turn in one process: event pairs around many back-to-back calls
// of the entry point, or around the stage of a traced update.
#pragma once
#include <cstdint>

namespace galore {

inline int64_t tile_count(int M, int N, int tile_m, int tile_n, int64_t batch) {
    return static_cast<int64_t>((N + tile_n - 1) / tile_n) * ((M + tile_m - 1) / tile_m) * batch;
}

// The column scans of a projector (sign convention, switch): workgroups of 16
// columns and 512 threads instead of 64 columns and 256, while the latter would
// leave CUs idle. A 16-column workgroup reads 64-byte pieces of rows and moves
// half the bytes per second once the chip is full.
//   sign (whole stage, n = workgroups of 64 columns; wide / narrow us): combining the
//   128 row groups costs more than the scan of few rows saves. Rows on 16 bytes:
//   512x128, n = 2: 27 / 29; 640x200, 4: 31 / 30, 32: 32 / 32, 64: 33 / 36; 768x200,
//   32: 35 / 34, 64: 36 / 38; 1000x200, 64: 46 / 43, 128: 53 / 54; 2048x256, 128: 86 /
//   72, 160: 87 / 82, 256: 114 / 147; 4096x1024, 16: 100 / 45, 128: 160 / 117, 160: 171
//   / 180, 1024: 663 / 988. Others (single loads): 128x65, 2: 26 / 28; 256x65, 32: 34 /
//   31, 128: 36 / 37; 512x127, 128: 59 / 53, 200: 63 / 71; 1000x201, 200: 106 / 96, 256:
//   110 / 113; 4096x1023, 160: 359 / 311, 256: 398 / 477.
inline bool narrow_sign_columns(int rows, int r, bool vec, int64_t batch) {
    const int64_t blocks = static_cast<int64_t>((r + 63) / 64) * batch;
    return vec ? blocks < (rows < 1088 ? (rows - 512) / 4 : 144) : blocks < (rows < 528 ? (rows - 160) / 2 : 184);
}
//   switch: 4096x1024, 1: 39 -> 19 us; 6 (96 workgroups): 66 -> 65; 7: 66 against 69
//   narrow, 8: 67 against 80, 64: 364 against 682; 1024x256, 32: 18 against 22.
inline bool narrow_align_columns(int r, int64_t batch) {
    return static_cast<int64_t>((r + 63) / 64) * batch < 112;
}

// Tiles of the fp32 products (gemm.hip): 128 x 128 x 32, two workgroups to a CU;
// 64 x 64 x 64, two to a CU; 64 x 64 x 32, four to a CU. With T wide and t narrow
// tiles (T counts padding, t much less of it):
//  * t <= 512, one round of two to a CU: the deep narrow tile, half the stages,
//    each of which waits a memory latency (A Omega of 8 x 1024x1024, k = 136:
//    deep 115, shallow 123, wide 187 us; at t = 576: 172, 153, 202);
//  * else the shallow narrow tile: its rounds are finer (7 x 1024x1024, k = 272,
//    T = 168, t = 560: deep 178, shallow 153, wide 202; T = 528: 399, 360, 448);
//  * but the wide one where its rounds of 512 are full but for an eighth by t (a
//    fifth where rows of A run along K: their narrow tiles cost more, N = k being
//    seldom a multiple of 64): the narrow tiles stage every operand twice as often
//    (projection, K = 2048, T = t / 4 = 420: 277 narrow, 281 wide; 480: 311, 282;
//    508: 315, 283; 516: 362, 454; 860: 548, 557; 900: 587, 557; 1016: 630, 566;
//    A X, K = 2736, t / 4 = 400: 859, 833; 420: 895, 833; 800: 1581, 1597; 840:
//    1645, 1629), unless the product adds to C, whose reads four workgroups a CU
//    hide better (K = 128, T = 512: 37 narrow, 44 wide; 1016: 68, 83; K = 512,
//    1016: 175, 181);
//  * past 1280 wide tiles, two and a half rounds, always the wide one (2 x
//    4096x11008, r = 1024, T = 1376: 1840 narrow, 1779 wide; K = 512, T = 1500:
//    249, 228).
enum F32Tile { kTile128, kTile64, kTile64x4 };
inline F32Tile f32_tile(int M, int N, bool a_kcontig, bool adds, int64_t batch) {
    const int64_t wide = tile_count(M, N, 128, 128, batch), narrow = tile_count(M, N, 64, 64, batch);
    if (wide > 1280) return kTile128;
    if (narrow <= 512) return kTile64;
    const int64_t rounds = (wide + 511) / 512;
    const int64_t full = 4 * 512 * rounds;
    if (!adds && (a_kcontig ? 5 * narrow > 4 * full : 8 * narrow > 7 * full)) return kTile128;
    return kTile64x4;
}
// The triangular product Y R^-1 (fp32 output): the wide tile's 4 x 1 waves or the
// deep narrow tile, which wins its first round of 512 at every k. Past it the
// launch waits for its longest column tile, K deep, and further narrow rounds fit
// into that time the better the larger K is (k: t: narrow / wide us): 24: 512: 20 /
// 20, 576: 27 / 21; 72: 512: 25 / 33, 640: 33 / 33, 800: 37 / 34; 112: 704: 40 / 46,
// 800: 45 / 46; 136: 576: 32 / 37, 624: 41 / 37; 200: 768: 49 / 56, 896: 59 / 57; 272:
// 960: 125 / 133, 1040: 144 / 136, 1680: 199 / 148; 368: 1536: 98 / 120, 1728: 119 /
// 119; 528: 1728: 274 / 279, 2016: 334 / 295; 640: 1920: 150 / 172; 1056: 1596: 448 /
// 474.
inline F32Tile f32_tril_tile(int M, int N, int K, int64_t batch) {
    const int64_t wide = tile_count(M, N, 128, 128, batch), narrow = tile_count(M, N, 64, 64, batch);
    const int64_t most = K <= 40 ? 512 : (K > 96 && K <= 128) ? 800 : K < 176 ? 608 : static_cast<int64_t>(K) * 21 / 5;
    return wide <= 512 && narrow <= most ? kTile64 : kTile128;
}

// The products of one or three bf16 planes (bf16x3.hip), two workgroups to a CU:
// 128 x 128 tiles instead of 256 x 128 up to 256 of the latter, which as half tiles
// are one round of 512. Past it the half tiles begin a second round and stage B
// twice as often (projection, three planes, r = 1024, s = 4096, wide / half: 176
// tiles: 177 / 175 us, 248: 197 / 194, 264: 252 / 299, 512: 315 / 372; r = 128, s =
// 512: 100: 32 / 26, 250: 38 / 36, 262: 46 / 51; the sketch product of one
// 4096x11008, 144: 246 / 191; low-bit back-projection, r = 1024, 248: 70 / 68,
// 264: 91 / 99).
inline bool three_plane_half(int M, int N, int64_t batch) { return tile_count(M, N, 256, 128, batch) <= 256; }

// The projection of a bf16 gradient off the 16-byte grid: planes against a padded
// copy (three launches), or the fp32 matrix cores on the gradient as it is (one).
// The latter is done first while the contraction is three of its 32-deep stages at
// most and the launch has the narrow tiles to fill the chip (f32_tile: at most 1280
// wide ones). One s x l gradient unless a batch is named, times copy / fp32 cores:
// 24x30000, r = 4: 11 / 7 us; 8 of them, 1880 wide tiles: 25 / 35; 40x4001: 11 / 7;
// 8 x 33x20001: 29 / 26; 8 x 64x10001, r = 64: 38 / 19; 32 of them, 2528 tiles: 92 /
// 98; 8 x 96x10001, r = 32: 30 / 24; 8 x 80x20001, r = 8: 33 / 36; 8 x 130x10001, r =
// 4: 28 / 31; 200x5001 r = 4: 15 / 15; 1000x4000: 33 / 40.
inline bool padded_projection(int s, int l, int r, int64_t batch) {
    return s > 96 || tile_count(r, l, 128, 128, batch) > 1280;
}

// The six-plane product: 128 x 128 tiles, two workgroups to a CU (rounds of 512),
// instead of 256 x 256, one to a CU (rounds of 256). For the same work the small
// tiles cost 1.3 times as much up to K = 320 and, half round by half round, 1.4
// times beyond; they win where the wide ones leave their last round nearly empty
// (back-projection, small / wide tiles, us; T wide ones): K = 1024, T = 64: 80 /
// 145, 128: 137 / 154, 152: 178 / 154, 260: 303 / 333, 320: 339 / 352, 352: 386 /
// 357, 384: 409 / 367, 520: 572 / 559; K = 512, 320: 179 / 191, 352: 206 / 194; K =
// 256, 320: 103 / 118, 352: 113 / 117, 420: 129 / 121, 688: 229 / 208; K = 288, 375: 2% less; K = 64, 384:
// 59 / 63, 508: 75 / 73).
inline bool six_plane_small(int M, int N, int K, int64_t batch) {
    const int64_t wide = tile_count(M, N, 256, 256, batch), small = tile_count(M, N, 128, 128, batch);
    const int64_t cost = K < 320 ? 13 * ((small + 511) / 512) : 7 * ((small + 255) / 256);
    return cost < 20 * ((wide + 255) / 256);
}

// A step of the small SVD (jacobi.hip): four groups of waves a workgroup, one
// workgroup to a CU, or one group, four to a CU. `batch` matrices in this launch,
// `in_flight` with those of the launch that runs beside it on the second stream.
// On one stream the wide form wins as long as its workgroups have a CU each (k =
// 1056, whole stage, 16 matrices, 256 workgroups: 18.9 against 24.5 ms; k = 528,
// 256: 7.2, 8.3; k = 136, 240: 1.40, 1.44). Two halves on two streams are seldom in
// the same phase, so a few more than 256 in all still gain, the more the longer
// the chunk loops are (k = 1056, 272: 21.6, 25.6 ms; 352: 24.9, 26.6; 384: 24.9,
// 25.9; 448: 29.2, 27.9; 512: 31.1, 28.1; k = 528, 320: 8.5, 8.7; 384: 9.5, 8.9; k
// = 136, 260: 2.7, 2.8; 300: 1.71, 1.64; k = 40, 300: 0.48, 0.43; k = 2048, 480:
// 84.0, 88.4; 512: 94.5, 88.7; whole update, k = 2560, 480: 193, 219; k = 4096, 512:
// 508, 616).
// (pairs of a step of k columns in blocks: an odd number of blocks, at least three,
// has a padding block, whose pair is not launched)
inline int step_pairs(int k, int block) {
    const int real = (k + block - 1) / block;
    return real % 2 != 0 && real >= 3 ? real / 2 : (real + 1) / 2;
}
inline bool wide_pairs(int k, int pairs, int64_t batch, int64_t in_flight) {
    return pairs * batch <= 256 && pairs * in_flight < 256 + k / 8;
}

}  // namespace galore
