// Tile shapes of the multi-step kernels (K = 2, 3 steps per launch through
// LDS) per storage form, shared by the kernels and host builds of the
// per-node arithmetic (the CPU replay of the step kernels in the tests).
#pragma once

#include "lbm_node.h"

namespace lbm {

constexpr int round64(int n) { return (n + 63) / 64 * 64; }

// Storage forms with a K-step kernel: every form, K = 2, 3.
constexpr bool stepk_available(int, int k) { return k == 2 || k == 3; }
// Those a caller may ask for, in every tile shape and with a persistent grid.
// FP64 has two steps per launch at most there; its three-step launches, in one
// shape, are the library's own choice (three_steps below).
constexpr bool stepk_offered(int st, int k) {
    return stepk_available(st, k) && (k == 2 || (st != ST_F64 && st != ST5_F64));
}

template <int ST>
struct Step2Tile;
// Tile shapes are build options (LBM_S2_*) for tuning; the defaults below.
#ifndef LBM_S2_F32_TW
#define LBM_S2_F32_TW 32
#define LBM_S2_F32_TH 12
#endif
#ifndef LBM_S2_F32Q5_TW
#define LBM_S2_F32Q5_TW 64
#define LBM_S2_F32Q5_TH 5
#endif
template <>
struct Step2Tile<ST_F32> {  // 27 x 4 + 4 = 112 B per slot (default 34 x 14 slots: 3 per CU)
    static constexpr int TW = LBM_S2_F32_TW, TH = LBM_S2_F32_TH, NT = round64((TW + 2) * (TH + 2));
};
template <>
struct Step2Tile<ST5_F32> {  // 19 x 4 + 4 = 80 B per slot (default 66 x 7 slots: 4 per CU)
    static constexpr int TW = LBM_S2_F32Q5_TW, TH = LBM_S2_F32Q5_TH, NT = round64((TW + 2) * (TH + 2));
};
template <>
struct Step2Tile<ST_F32H> {  // 26 x 4 + 8 + 4 = 116 B per slot, 34 x 13 slots: 3 per CU
    static constexpr int TW = 32, TH = 11, NT = 448;
};
template <>
struct Step2Tile<ST5_F32H> {  // 18 x 4 + 8 + 4 = 84 B per slot, 66 x 7 slots: 4 per CU
    static constexpr int TW = 64, TH = 5, NT = 512;
};
template <>
struct Step2Tile<ST_F16> {  // 27 x 2 + 4 = 58 B per slot, 34 x 15 slots (29 KiB)
    static constexpr int TW = 32, TH = 13, NT = 512;
};
template <>
struct Step2Tile<ST_BF16> {
    static constexpr int TW = 32, TH = 13, NT = 512;
};
template <>
struct Step2Tile<ST_F16S> {  // 6 x 4 + 24 x 2 + 4 = 76 B per slot, 34 x 15 slots (38 KiB: 4 per CU)
    static constexpr int TW = 32, TH = 13, NT = 512;
};
template <>
struct Step2Tile<ST_BF16S> : Step2Tile<ST_F16S> {};
#ifndef LBM_S2_F64_TW
#define LBM_S2_F64_TW 32
#define LBM_S2_F64_TH 5
#endif
template <>
struct Step2Tile<ST_F64> {  // 27 x 8 + 8 = 224 B per slot (default 32 x 5 with push placement: 160 slots, 37 KiB)
    static constexpr int TW = LBM_S2_F64_TW, TH = LBM_S2_F64_TH, NT = round64((TW + 2) * (TH + 2));
};
#ifndef LBM_S2_F64Q5_TW
#define LBM_S2_F64Q5_TW 32
#define LBM_S2_F64Q5_TH 8
#endif
template <>
struct Step2Tile<ST5_F64> {  // 19 x 8 + 8 = 160 B per slot (default 34 x 10 slots, 56 KiB)
    static constexpr int TW = LBM_S2_F64Q5_TW, TH = LBM_S2_F64Q5_TH, NT = round64((TW + 2) * (TH + 2));
};

// Tile shapes of the three-steps-per-launch kernel (a two-node ring; build
// options LBM_S3_* for tuning).  Measured on the 8192^2 cavity: the shape
// must leave three (D2Q9) or four (D2Q5) workgroups per CU; with two, the
// three updates and their barriers leave too little to overlap (32 x 11:
// 28.6 GLUPS against 43.7 for 32 x 9).
template <int ST>
struct Step3Tile;
#ifndef LBM_S3_F32_TW
#define LBM_S3_F32_TW 32
#define LBM_S3_F32_TH (LBM_PUSH_F32_K3 ? 10 : 9)
#endif
#ifndef LBM_S3_F32Q5_TW
#define LBM_S3_F32Q5_TW 32
#define LBM_S3_F32Q5_TH 10
#endif
template <>
struct Step3Tile<ST_F32> {  // 112 B per slot (push 32 x 10: 34 x 12 slots, 46 KiB, 3 per CU with all the
                             // registers they can have: 53.1 GLUPS on the 8192^2 cavity and 23.0 us a step at
                             // 1024^2, against 52.1 and 25.1 for 32 x 8 held to the registers of 4 per CU)
    static constexpr int TW = LBM_S3_F32_TW, TH = LBM_S3_F32_TH, NT = round64((TW + 4) * (TH + 4));
};
template <>
struct Step3Tile<ST5_F32> {  // 80 B per slot (default 36 x 14 slots, 39 KiB: 4 per CU)
    static constexpr int TW = LBM_S3_F32Q5_TW, TH = LBM_S3_F32Q5_TH, NT = round64((TW + 4) * (TH + 4));
};
#ifndef LBM_S3_F16_TW
#define LBM_S3_F16_TW 32
#define LBM_S3_F16_TH 10
#endif
#ifndef LBM_S3_F16S_TW
#define LBM_S3_F16S_TW 32
#define LBM_S3_F16S_TH 10
#endif
template <>
struct Step3Tile<ST_F16> {  // 58 B per slot (default 36 x 14 slots, 29 KiB)
    static constexpr int TW = LBM_S3_F16_TW, TH = LBM_S3_F16_TH, NT = round64((TW + 4) * (TH + 4));
};
template <>
struct Step3Tile<ST_BF16> {
    static constexpr int TW = LBM_S3_F16_TW, TH = LBM_S3_F16_TH, NT = round64((TW + 4) * (TH + 4));
};
template <>
struct Step3Tile<ST_F16S> {  // 76 B per slot (default 36 x 14 slots, 38 KiB)
    static constexpr int TW = LBM_S3_F16S_TW, TH = LBM_S3_F16S_TH, NT = round64((TW + 4) * (TH + 4));
};
template <>
struct Step3Tile<ST_BF16S> : Step3Tile<ST_F16S> {};
#ifndef LBM_S3_F32H_TW
#define LBM_S3_F32H_TW 32
#define LBM_S3_F32H_TH (LBM_PUSH_F32H_K3 ? 10 : 9)
#endif
template <>
struct Step3Tile<ST_F32H> {  // 116 B per slot (push 32 x 10: 34 x 12 slots, 46 KiB, 3 per CU: chosen at
                             // 45.7 GLUPS on the 8192^2 cavity, 51.3 since, against 45.1 for 32 x 8 with 4 per CU;
                             // pull 32 x 9: 53 KiB, 3)
    static constexpr int TW = LBM_S3_F32H_TW, TH = LBM_S3_F32H_TH, NT = round64((TW + 4) * (TH + 4));
};
template <>
struct Step3Tile<ST5_F32H> {  // 84 B per slot, 36 x 14 slots (41 KiB: 3 per CU)
    static constexpr int TW = 32, TH = 10, NT = 512;
};

// FP64: two workgroups per CU (77 and 65 KiB of LDS).  The two-step kernels
// move 2 x 224 B (D2Q5: 2 x 160 B) a node and launch and are bound by HBM; three
// steps per launch move two thirds of that a step, for tiles whose first update
// covers 1.7 times their nodes.  us a step, two steps -> three: D2Q9 1024^2
// 51.8 -> 45.7, 4096^2 767 -> 644; D2Q5 51.5 -> 31.7 and 758 -> 436.  Other shapes
// lose: D2Q9 32x6 67.4 (1024^2), 16x16 46.9, 24x11 48.8, one workgroup per CU
// (32x10 55.7, 32x16 55.3, 48x12 53.5); D2Q5 32x8 35.0, 24x14 33.1, 28x12 32.9, 16x16
// (three per CU) 37.7, 32x12 40.6.
template <>
struct Step3Tile<ST_F64> {  // 224 B per slot, 34 x 10 slots
    static constexpr int TW = 32, TH = 8, NT = round64((TW + 4) * (TH + 4));
};
template <>
struct Step3Tile<ST5_F64> {  // 160 B per slot, 34 x 12 slots
    static constexpr int TW = 32, TH = 10, NT = round64((TW + 4) * (TH + 4));
};
// The tiles of an FP64 handle: three-step ones, those of them next to a wall,
// and two-step ones.
struct ThreeStepTiles {
    int64_t three, wall, two;
};
// Whether a handle with those tiles runs three steps per launch.  D2Q5: always.
// D2Q9: from three quarters of the workgroups the chip holds (two per CU); with
// fewer, the three-step kernel's tiles take their time with CUs to spare and
// the smaller two-step tiles are faster (us a step, two -> three steps: 270^2, 306
// tiles, 6.56 -> 7.81; 300^2, 380 tiles, 7.64 -> 7.91; 350^2, 484 tiles, 9.82 -> 8.63;
// 450^2 14.3 -> 13.8; 640^2 24.2 -> 21.2.  D2Q5 270^2, 243 tiles, 8.05 -> 5.69).
// Beyond one round of tiles (two per CU) a launch takes as long as the fullest CU,
// so three steps need that CU's tiles to be less than three quarters of the
// two-step kernel's, unless few tiles are at walls, which cost the three-step
// kernel about twice the others (two steps -> three: 16 cavities of 101x41 to
// 240x203, 3 tiles on the fullest CU against 4, two thirds at walls, 10.2 -> 14.6;
// 30 of 65^2, 4 against 5, all at walls, 13.3 -> 15.1; 20000x4 6.8 -> 8.3; 500x300, 3
// against 4, a sixth at walls, 10.7 -> 10.5; 957x204, 4 against 5, a seventh, 13.1 ->
// 11.7).  Of 1756 handles of mixed sizes 32 are then slower than with two steps
// per launch of the kernels before, the worst by 9%, instead of 150, the worst by
// 35%.
// The plan, which knows no device, reserves for the CUs of an MI355X; a handle
// on a device with other ones asks again with its own number.
constexpr int kCus = 256;
constexpr bool three_steps(int st, const ThreeStepTiles &t, int n_cu = kCus) {
    if (st != ST_F64) return st == ST5_F64;
    const int64_t fullest3 = (t.three + n_cu - 1) / n_cu, fullest2 = (t.two + n_cu - 1) / n_cu;
    return 2 * t.three >= 3 * (int64_t)n_cu &&
           (t.three <= 2 * (int64_t)n_cu || 4 * fullest3 < 3 * fullest2 || 10 * t.wall < 3 * t.three);
}

template <int ST, int K>
struct StepKTile;
template <int ST>
struct StepKTile<ST, 2> : Step2Tile<ST> {};
template <int ST>
struct StepKTile<ST, 3> : Step3Tile<ST> {};

// Tile shapes chosen at run time (lbm_launch_config.tile_shape): 0 is the
// default above; 1 is about twice as wide and half as tall, 2 about half as
// wide and twice as tall, each within 64 KiB of LDS, 1024 threads and the
// band rule (TH + 2K <= LBM_MIN_BAND_ROWS).  The autotuner times them: a
// cavity whose width leaves a narrow last tile in one shape fits another.
constexpr int kTileShapes = 3;
struct TileDims {
    int tw, th;
};
constexpr TileDims alt_dims(int st, int k, int i) {
    if (k == 3) {
        if (st == ST_F32 || st == ST_F32H) return i == 1 ? TileDims{64, 4} : TileDims{16, 16};
        return i == 1 ? TileDims{64, 5} : TileDims{16, 20};  // D2Q5 FP32 forms, 16-bit forms
    }
    switch (st) {
        case ST_F32: return i == 1 ? TileDims{64, 6} : TileDims{16, 24};
        case ST_F32H: return i == 1 ? TileDims{64, 5} : TileDims{16, 22};
        case ST5_F32:
        case ST5_F32H: return i == 1 ? TileDims{32, 10} : TileDims{128, 3};
        case ST_F64: return i == 1 ? TileDims{64, 3} : TileDims{16, 10};
        case ST5_F64: return i == 1 ? TileDims{64, 4} : TileDims{16, 16};
        default: return i == 1 ? TileDims{64, 6} : TileDims{16, 26};  // 16-bit forms
    }
}
template <int ST, int K, int I>
struct StepKTileI {
    static constexpr TileDims d = alt_dims(ST, K, I);
    static constexpr int TW = d.tw, TH = d.th, NT = round64((TW + 2 * (K - 1)) * (TH + 2 * (K - 1)));
};
template <int ST, int K>
struct StepKTileI<ST, K, 0> : StepKTile<ST, K> {};

// Width and height of tile shape i of the K-step kernel of storage st.
template <int ST, int K>
constexpr TileDims dims_of(int i) {
    return i == 0 ? TileDims{StepKTile<ST, K>::TW, StepKTile<ST, K>::TH} : alt_dims(ST, K, i);
}

// Deep launches: tiles of a handle that fits one per CU, and the most steps
// of a launch.  Of the shapes that leave at most kDeepTiles tiles the first
// (smallest) is taken: a launch's fixed part (2.4 us between launches, 0.5 for
// its constants, 1.4 for the cold first loads, 0.5 for the stores) is shared
// by its steps, and an update costs what its waves per SIMD make it, so
// shapes trade steps for waves.  us a step against the K-step kernels, one
// MI355X: FP32_H64 64^2 8x8x6 4.46 -> 2.73 (8x8x7 2.92, 12x12x6 3.14), 151^2
// 12x12x6 4.46 -> 3.26, 200^2 16x12x6 4.5 -> 3.69, 256^2 16x16x5 4.45 -> 3.77
// (x6 3.87, x4 4.21); FP64 64^2 8x8x5 5.86 -> 3.44 (x6 3.87, x4 3.83), 151^2
// 16x8x4 5.41 -> 4.26 (x5 4.60), 200^2 16x12x4 6.18 -> 5.37, 256^2 16x16x4 7.17
// -> 5.70; D2Q5 FP32 64^2 3.93 -> 2.13, 256^2 3.80 -> 2.82.  Batches and thin
// cavities of up to 256 tiles gain alike (156 handles of all six forms, 1.06 to
// 2.85 times: FP64 16 of 64^2 6.81 -> 5.93, 256 of 8^2 7.62 -> 3.18, 4x2048 10.1 ->
// 3.54; D2Q5 16 of 64^2 5.18 -> 4.87).  With two tiles on a CU they lose (FP32_H64
// 300^2 16x16: 6.0 -> 7.7).
constexpr int kDeepShapes = 4;
constexpr int kDeepTiles = kCus;  // reserved for by the plan
constexpr bool deep_fits(int64_t tiles, int n_cu) { return tiles <= n_cu; }  // what a handle then runs
struct DeepDims {
    int tw, th, k;
};
constexpr bool deep_available(int st) {
    return st == ST_F64 || st == ST_F32 || st == ST_F32H || st == ST5_F64 || st == ST5_F32 || st == ST5_F32H;
}
constexpr DeepDims deep_dims(int st, int i) {
    const bool f64 = st == ST_F64 || st == ST5_F64;
    const DeepDims wide[kDeepShapes] = {{8, 8, 5}, {16, 8, 4}, {16, 12, 4}, {16, 16, 4}};
    const DeepDims narrow[kDeepShapes] = {{8, 8, 6}, {12, 12, 6}, {16, 12, 6}, {16, 16, 5}};
    return f64 ? wide[i] : narrow[i];
}

}  // namespace lbm
