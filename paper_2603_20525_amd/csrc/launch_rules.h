// Rules by which launches are chosen from sizes alone: plain host code without
// the HIP runtime, so that they can be tested without a device.
#pragma once

namespace plan {

constexpr int EST_SHARE_MAX_ROUNDS = 6;

// Waves per SIMD among which a rollout of the extended single-track model shares
// its steps equally, or 0: it gives each wave a group of 64 candidates. Sharing
// saves the last, partial round of waves but runs the rest with one wave per
// SIMD fewer, which pays up to a remainder that depends on how well that many
// waves hide each other's latency. 16 intervals of 50 substeps, shared / not, in
// us: 66 000 candidates (1.01 waves per SIMD) 262 / 342, 80 000 (1.22) 307 / 340,
// 90 000 (1.37) 370 / 343; 137 000 (2.09) 339 / 468, 170 000 (2.59) 416 / 473,
// 185 000 (2.82) 501 / 499; 204 288 (3.12) 472 / 597, 240 000 (3.66) 552 / 598;
// 270 000 (4.12) 592 / 725, 300 000 (4.58) 826 / 820; 350 000 (5.34) 739 / 851;
// 400 000 (6.10) 827 / 981.
// A single substep an interval streams its controls besides, which fewer waves
// hide worse, so that only smaller remainders pay: 100 intervals, 66 000 46.7 /
// 50.9, 80 000 55.4 / 51.0; 150 000 (2.29) 62.1 / 70.1, 170 000 78.0 / 73.4;
// 204 288 87.4 / 91.4, 240 000 102.8 / 97.8; 270 000 117.9 / 123.7.
// And the hand-off of a group takes some microseconds, so a few steps are not
// shared: 66 000 x 10 11.6 / 9.4, x 20 15.1 / 13.3, x 30 18.5 / 18.3, x 50 26.1 /
// 27.3; 400 000 x 5 16.6 / 11.5, x 20 34.8 / 33.1, x 30 46.7 / 46.1.
inline int est_share_rounds(int groups, int simds, int N, int S) {
    const int rounds = groups / simds, rest = groups - rounds * simds;
    if (rounds < 1 || rounds > EST_SHARE_MAX_ROUNDS || rest == 0) return 0;
    if ((long long)N * S < 25) return 0;
    int eighths;  // of a round that may remain
    if (S == 1)
        eighths = rounds == 1 ? 1 : 2;
    else
        eighths = rounds == 1 ? 2 : rounds <= 3 ? 6 : 4;
    return 8ll * rest <= (long long)eighths * simds ? rounds : 0;
}

// Whether the distance costmap of a W x H grid takes tiles of 16 x 16 nodes
// instead of 32 x 32: where the larger ones number fewer than 7/4 per compute
// unit, so that units would idle or wait for one that has two. Larger / smaller
// tiles, in us: 256 x 256 nodes, 20 obstacles and a boundary 27.1 / 14.8, a
// boundary of 1 300 edges 424 / 238; 600 x 600 (1.4 a unit) 23.7 / 16.0, 606 / 475;
// 700 x 700 (1.9) 24.1 / 19.9, 612 / 620, with every perimeter in reach of every
// node 118 / 131; 1 400 x 1 400 37.5 / 42.4, 1 306 / 1 485.
inline bool costmap_small_tiles(int W, int H, int units) {
    const long long tiles = (long long)((W + 31) / 32) * ((H + 31) / 32);
    return 4 * tiles < 7ll * units;
}

// Plan entries (of the 2 N) that a workgroup of the softmin takes: the fewest
// that leave no unit of the chip's 256 two workgroups, times with launch and
// wait: K = 10 007, N = 73 18.5 -> 15.6 us (one; two 16.5), 65 536 x 50 45.9 ->
// 24.6, 65 536 x 200 51.9 -> 31.6 (two; one 37.7), 4 096 x 100 15.3 -> 13.6;
// beyond, every workgroup's own pass over the costs weighs more: 4 096 x 1 000
// 14.5 with four, 19.1 with two. Where one pass of 8 192 candidates is about
// full, or a second one short, four take as long as two on half the workgroups:
// four / two, 8 192 x 256 15.7 / 16.4, 12 363 x 228 15.6 / 17.7, 16 384 x 176 16.9
// / 18.3; but 4 096 x 256 15.7 / 14.0, 12 363 x 150 18.5 / 17.1, 20 000 x 256 18.5 /
// 17.3.
inline int softmin_entries(int K, int N) {
    const long long rows = 2ll * N;
    if (rows <= 256) return 1;
    const bool full_pass = K > 6144 && K < 20000 && !(rows <= 340 && K < 14336);
    return rows <= 512 && !full_pass ? 2 : 4;
}

}  // namespace plan
