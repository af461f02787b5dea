// Eligibility test and tile-configuration choice for the MFMA path.
#include <cstdlib>
#include "gemm_mfma_launch.h"
#include "gemm_mfma_tile64.h"

namespace pbk {

static bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// The MFMA path moves operands in whole 16-byte pieces (8 elements): bases,
// leading dimensions, batch strides and K must keep every piece aligned and
// entirely inside or outside the matrix; likewise N for row-major B and Cin
// for the convolution (a piece must not straddle two filter taps).
bool mfma_supported(const Problem& p) {
    // 8-bit operand types (FP8, int8): 16 values per 16-byte piece
    const bool e8 = p.in_dtype == DT_FP8_E4M3 || p.in_dtype == DT_FP8_E5M2 || p.in_dtype == DT_INT8;
    const bool f32 = p.in_dtype == DT_F32;
    if (p.in_dtype != DT_BF16 && p.in_dtype != DT_F16 && !e8 && !f32) return false;
    const int per16 = e8 ? 16 : f32 ? 4 : 8;         // elements per 16-byte piece
    const int esz = e8 ? 1 : f32 ? 4 : 2;
    if (f32 && p.K >= (1 << 29)) return false;        // k sizes are doubled for the kernel
    if (p.K < per16 || p.K % per16) return false;
    if (!al16(p.A) || !al16(p.B)) return false;
    if (p.stride_a % per16 || p.stride_b % per16) return false;
    // per-lane buffer offsets are 32-bit and must stay below 2^31
    const int64_t lim = (int64_t)1 << 31;
    if (p.is_conv) {
        if ((e8 || f32) && p.conv.transposed) return false;   // the transposed form is built for 16-bit types
        if (p.conv.Cin % per16 || p.N % per16) return false;
        int64_t img = (int64_t)(p.M / (p.conv.OH * p.conv.OW)) * p.conv.H * p.conv.W * p.conv.Cin * esz;
        int64_t halo = ((int64_t)p.conv.pad_h * p.conv.W + p.conv.pad_w + p.conv.W) * p.conv.Cin * esz;
        if (img + halo >= lim) return false;
    } else {
        if (p.lda % per16 || p.ldb % per16) return false;
        if (!p.trans_b && p.N % per16) return false;
        if (256 * p.lda * esz + 256 >= lim) return false;
    }
    if (256 * p.ldb * esz + 1024 >= lim) return false;
    return true;
}

// A launch holds fewer than 2^32 threads: from so many tiles on the forms with 512 threads a tile cannot be launched (2^23 small entries of a batched
// product, or 2^30 rows).
static constexpr long long kTilesOf512 = 1LL << 23;
static long long square_tiles(const Problem& p) { return (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch; }

// fp32 operands take the staged kernel only when there is enough work to fill the chip with 128-row tiles.  (Plain products of up to
// 4096 tiles of 16 x 16 take the kernel without staging before this is asked: small_f32_preferred.)
bool mfma_preferred(const Problem& p) {
    if (p.in_dtype != DT_F32) return p.in_dtype == DT_BF16 || p.in_dtype == DT_F16 || square_tiles(p) < kTilesOf512;      // (8-bit types: 512 threads in every form)
    long long t = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
    return p.M >= 128 && p.N >= 128 && t >= 64;
}

// 128 x 128 tiles: with at most one per compute unit (256), the four-stage ring (three k-tiles in flight) covers the memory latency
// that two workgroups per unit hide from each other otherwise: bf16 2048 x 2048 x 4096 34.4 against 49.4 us, 577 x 4096 x 1024
// 11.1 against 15.0, FP8 512 x 4096 x 4096 15.3 against 26.1.  Beyond one round two workgroups share a unit (4 x 32 x 28 x 28
// rows of a transposed convolution, 784 tiles: 42.4 against 56.1 us).
// Filling the deeper ring costs more than it gives (figures of four waves per tile)
// - in a convolution whose k-tiles span taps, so that every address is divided out, up to some eight k-tiles (3 x 3, bf16 32 -> 64, five:
//   12.5 against 12.1 us; int8 64 -> 128, five: 25.0 against 24.4; bf16 96 -> 128, fourteen: 4 % ahead);
// - in a 16-bit product of three or four k-tiles up to some 160 tiles (577 x 4096 x 256: 7.4 against 7.2 us; 1536 x 2048 x 256,
//   192 tiles: 7.7 against 7.6, 2048 x 2048 x 256: 8.1 against 8.3; with two k-tiles or five it is even or ahead).
// Two tiles per unit, one k-tile or one and a half, and an epilogue that loads nothing: the time is starting the waves and storing, of which four
// waves per tile are the lesser part, with rows of 128 bytes in a store instead of 64 (3, 16-bit plain products, eight waves first: 12 x 704 x 704 x 32
// 6.88 and 6.55 us, 33 x 320 x 320 x 64 5.95 and 5.74, 32 x 384 x 384 x 96 7.18 and 6.90; 192 8.08 and 8.43 for 12 x 704 x 704; with a bias
// 6.83 and 7.23, with fp32 results 8.12 and 8.43; 468 tiles even, 512: 7.68 and 7.84; 60000 x 128 x 64: 7.35 and 7.85).  Where few units have two tiles,
// up to two and a half (k-major B: 17 x 512 x 512 x 128, 272 tiles, 7.15 and 6.76, x 160 8.11 and 7.94, x 192 7.70 and 7.82; 9 x 768 x 768 x 128, 324 tiles, 7.35 and
// 7.25; 40 x 384 x 384 x 128, 360 tiles, 7.58 and 7.73).
static int square_config(const Problem& p) {
    const long long t = square_tiles(p);
    const bool b8 = p.in_dtype != DT_BF16 && p.in_dtype != DT_F16;
    if (t >= kTilesOf512 && !b8) return p.is_conv ? 6 : 3;        // 256 threads a tile
    if (t > 256) return !b8 && !p.is_conv && p.K <= (t <= 330 ? 160 : 96) && t <= 448 && p.N >= 256 && p.out_dtype != DT_F32 && !epi_has_bias(p.epi) && !p.R ? 3 : 1;
    const int bk = b8 ? 128 : 64, kt = (p.K + bk - 1) / bk;        // values per k-tile, k-tiles
    if (p.is_conv) return p.conv.Cin % bk != 0 && kt <= 8 ? 1 : 2;
    return !b8 && kt >= 3 && kt <= 4 && t <= 160 ? 1 : 2;
}

// Cost of 128 x 128 tiles, two of which share a unit, in the units of pair_choice, for every tile that a unit has (one round of 512, 2048 x 4096: K = 512
// 13.5 us with these, 13.7 with 128 x 256 in the pair pipeline, 1024 20.4 and 19.2, 2048 34.8 and 31.2; conv 25088 x 256 x 4608 71.5 and 58.5; e4m3
// 2048 x 4096 x 4096 34.4 and 28.4).
static long long square_cost(long long t128, int k) { return (t128 + 255) / 256 * (160 + k / 86); }

// Rows of the pair pipeline's tiles (configurations 9 to 13: 256, 224, 192, 160, 128 rows, 256 columns, one workgroup per compute unit): the
// height whose rounds of 256 tiles cost least, a round being h + 200 units (its loads and its multiplications grow with h, what it fetches of B
// does not).  With 256 rows only, a second round a third full cost as much as a full one.  Times in us, 256 rows first, then the height taken:
// 4608 x 4864 x 4480, k-major B, 342 tiles: 177 and 152 (192 rows, 456 tiles); 5303 x 4608 x 3328: 142 and 126 (192); 5376 x 7168 x 1792: 126
// and 118 (224); 21 x 56 x 56 x 512 -> 512, 3 x 3: 295 and 258 (192); e4m3 7590 x 2176 x 3712: 74.6
// and 54.0 (160); 8192^3 stays on 256: 744, 830, 847, 879, 853.  Over 151 shapes the height that the rule takes was the fastest of the five but for
// three (2 to 4 % behind), with any constant from 100 to 300.
// Several rounds of a long contraction leave 256 rows only where that saves a tenth.  Under load the board's power bounds them, lower tiles fetch B more often for the same
// product, and which is ahead changes with the card: 32 x 56 x 56 x 256 -> 256, 3 x 3, two rounds of either, 256 and 224 rows: 106.7 and 104.4, 112.0 and
// 112.2, 111.8 and 113.2, 115.6 and 117.7 on four of them; 6400 x 4096 x 8192 326 and 328, 30 x 56 x 56 x 512 -> 256 194 and 199, elsewhere 210 and 204.
struct PairChoice { int cfg, height; long long rounds, cost; };
static PairChoice pair_choice(const Problem& p) {
    static const struct { int cfg, height; } forms[] = {{9, 256}, {10, 224}, {11, 192}, {12, 160}, {13, 128}};
    PairChoice best{}, tallest{};
    for (const auto& f : forms) {
        const long long tiles = (long long)((p.M + f.height - 1) / f.height) * ((p.N + 255) / 256) * p.batch, rounds = (tiles + 255) / 256;
        const long long cost = rounds * (f.height + 200);
        if (f.height == 256) tallest = PairChoice{f.cfg, f.height, rounds, cost};
        if (!best.cfg || cost < best.cost) best = PairChoice{f.cfg, f.height, rounds, cost};
    }
    const long long t128 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
    return p.K >= 2048 && tallest.rounds > 1 && 10 * best.cost > 9 * tallest.cost && tallest.cost <= square_cost(t128, p.K) ? tallest : best;
}

// 8-bit operands, both k-major: its configuration from the second 128 x 128 tile per compute unit on, up to two of them from `least` k on; 0: not taken.
static int pair_config8(const Problem& p, long long t128, int least) {
    if (!p.trans_b || p.is_conv || p.M < 128 || p.N <= 128 || t128 <= 256 || (p.K < least && t128 <= 512)) return 0;
    const PairChoice c = pair_choice(p);
    return c.cost <= square_cost(t128, p.K) ? c.cfg : 0;
}

// 16-bit operands: the pair pipeline from the second 128 x 128 tile per compute unit on, unless that form costs less (narrow matrices: 20000 x 384 x
// 1024, k-major B: 20.1 against 21.0), and for long enough contractions.  Times in us, the form taken before first:
// - row-major B from K = 640 on (1168 x 4608 x 640: 13.7 and 12.8; K = 576: 1606 x 4288 15.2 and 15.7, 2165 x 3072 13.6 and 12.8); from 320 on where
//   there are more than 256 tiles of 128 x 256 and fewer rows than 256 fit better (1771 x 5184 x 320: 18.2 and 16.7, 4666 x 1600 x 512: 20.4 and 16.9; with
//   256 rows 6638 x 2304 x 576 23.8 and 25.2; 4066 x 3328 x 264: 14.2 and 15.4);
// - k-major B from 512 on (2.5 to 20 %), and beyond 256 wherever there are more than 256 tiles of 128 x 256, whose k-major form is slow (2163 x 4608 x 320:
//   16.1 and 13.3, 7133 x 3520 x 264 30.3 and 27.5; 1335 x 3904 x 448, 256 of them: 11.0 both);
// - convolutions whose channels 64 divides (a 64-deep piece of the image lies inside one tap) from K = 512 on (16464 x 256 x 576: 13.4 and 13.0; 23520 x
//   256 x 128: 8.5 and 8.9), up to 768 for at most two rounds of fewer rows than 256 (3 x 3, 56 x 56 x 64, images -> channels, from memory and from the caches: 23 ->
//   256, 160 rows, 37.7/32.7 and 33.4/29.8, 35 -> 256, 224 rows, 43.2/38.0 and 41.5/38.0; 256 rows, 20 -> 512 56.7/47.3 and 58.0/50.5, 38 -> 256 57.0/46.3 and
//   57.0/49.4; three rounds, 50 -> 256 72.8/60.2 and 76.9/68.4, 47 -> 256, all full, 57.1/48.8 and 53.3/48.6).
static bool pair_preferred(const Problem& p, const PairChoice& c, long long t, long long t128) {
    if (p.M < 128 || p.N <= 128 || c.cost > square_cost(t128, p.K)) return false;
    if (p.is_conv) return p.conv.Cin % 64 == 0 && p.K >= 512 && (p.K >= 768 || (c.rounds <= 2 && c.height < 256));
    if (p.trans_b) return p.K >= 512 || (p.K > 256 && t > 256);
    return p.K >= 640 || (p.K >= 320 && t > 256 && c.height < 256);
}

// Convolutions of up to 128 columns, and transposed ones by residue classes: the same pipeline on tiles of 256, 320, 384 or 448 rows and 128 columns
// (configurations 14 to 17), whose compute units load 128 columns of the weights for more rows than with two 128 x 128 tiles.  Rule as above, a round
// being h + 107 units (up to 64 columns the 128 x 128 tiles, whose waves without columns only fetch, take a tenth less).  Times in us, 128 x 128 tiles first:
// transposed 32 x 28 x 28 x 256 -> 128, 4 x 4, stride 2: 43.1 and 34.7 (448 rows, one round; 256 to 384 rows, two: 45.4 to 57.5), 23 x 32 x 27 x 256 ->
// 128 38.4 and 28.9 (320), 29 x 12 x 58 x 128 -> 128 24.6 and 20.1; 28 x 56 x 56 x 128 -> 128, 3 x 3: 38.2 and 30.1 (384), 64 x 56 x 56: 79.6 and
// 67.4 (448, two rounds), 57 x 28 x 28 x 512 -> 128 75.5 and 61.5 (256); 10 x 46 x 27 x 128 -> 128, transposed, two tiles per unit: 16.7 and 19.3 (not taken).
// Below K = 512: 6 x 57 x 58 x 64 -> 64, transposed, K = 256 15.1 and 14.9.
// k: values that the longest contraction of the call runs over.  0: not this form.
static int tall_config(const Problem& p, int k) {
    if (p.conv.Cin % 64 != 0 || k < 512) return 0;
    static const struct { int cfg, height; } forms[] = {{14, 256}, {15, 320}, {16, 384}, {17, 448}};
    const long long cols = (p.N + 127) / 128;
    auto row_tiles = [&](int h) { return p.conv.transposed ? convt_row_tiles(p, h) : (long long)((p.M + h - 1) / h); };
    const long long t128 = row_tiles(128) * cols, square = square_cost(t128, k);
    long long best = p.N <= 64 ? square * 9 / 10 : square;
    int cfg = 0;
    if (t128 <= 256) return 0;
    for (const auto& f : forms) {
        const long long cost = (row_tiles(f.height) * cols + 255) / 256 * (f.height + 107);
        if (cost < best) { best = cost; cfg = f.cfg; }
    }
    return cfg;
}

// 16-bit operands.  Configurations 5-7 and 9 on use the 16x16x32 MFMA blocks (measured against their
// 32x32x16 twins 3, 0: 8192^3 786 against 816 us, 3x3 convolution 144 against 151 us, the
// store-bound attention-score product equal); 7 also stages A 64 deep (762 us), 9 to 13 have one barrier per two k-tiles (739 us).
static int choose_config(const Problem& p) {
    const long long t = (long long)((p.M + 127) / 128) * ((p.N + 255) / 256) * p.batch;
    const long long t128 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
    if (t128 > 256) {
        const PairChoice pair = pair_choice(p);
        if (pair_preferred(p, pair, t, t128)) return pair.cfg;
    }
    if (p.is_conv && p.N <= 128)
        if (const int cfg = tall_config(p, p.K)) return cfg;
    // The 128x256 tiles, two workgroups per unit, whose two barrier domains fill each other's bubbles: short contractions (store-dominated), and
    // convolutions that the pair pipeline cannot take.  Long contractions with a k-major B are slow there (8192^3: 1044 us against 874 for 256x256x32).
    if (!p.is_conv && p.K >= (p.trans_b ? 512 : 640)) return square_config(p);
    if (p.M >= 128 && p.N >= 256 && t > 256) return 6;
    return square_config(p);
}

// Transposed convolution by residue classes (tile configurations 1, 2 and 14 to 17): what the form can address and launch.
static bool convt_classes_fit(const Problem& p) {
    // where k-tiles (up to 64 deep) span taps, any weight row is reached from the first one with a 32-bit offset
    if (p.conv.Cin % 64 != 0 && (int64_t)p.K * p.ldb * 2 >= ((int64_t)1 << 31)) return false;
    // A launch holds fewer than 2^32 threads: fewer than 2^23 tiles of 512.  (A stride beyond the image makes nearly every output pixel a
    // class, and a tile, of its own.)
    return convt_row_tiles(p, 128) * ((p.N + 127) / 128) < kTilesOf512;
}

// Classes, or all taps for every output pixel?  By how much the longest class shortens the k loop.  Its rows of C are apart, its tiles
// are 128 x 128 (with 128 x 256 the row mapping of the epilogue does not fit the registers), and with too little to save that costs more
// than it gives.  Times in us, all taps first, 2700 sizes of stride 1 to 4; with this rule none is more than 2.5 % behind all taps:
// - nothing saved (stride 1, one tap, a dilation that is a multiple of the stride): 4 x 28 x 28 x 64 -> 128, 1 x 1, stride 2: 8.1
//   against 10.1; 16 x 56 x 56 x 96 -> 256, 5 x 5, stride 1: 79 against 140;
// - up to 128 columns, saved 24 (Cin = 8, 2 x 2, stride 2): 1.3 times as long by classes; 96: 0.9 to 1.15 times, 160 to 200: 0.7 to 0.9
//   on average, from 384 at most 0.7;
// - where the 128 x 256 tiles would be taken: saved 96: 1.3 to 1.5 times, 160 to 200: 1.0 on average and up to 1.27, from 320 on at most
//   0.9, with k-tiles that span taps from 1152 on (480: 32 x 56 x 56 x 96 -> 512, 3 x 3: 261 against 271; 512: 32 x 28 x 28 x 32 -> 256,
//   5 x 5: 52.5 against 55.5; 1536: 0.8).
// (values of k that the longest class keeps)
static int convt_class_k(const Problem& p) {
    const ConvTAxis h = convt_axis_of(p.conv.OH, p.conv.stride_h, p.conv.dil_h, p.conv.KH);
    const ConvTAxis w = convt_axis_of(p.conv.OW, p.conv.stride_w, p.conv.dil_w, p.conv.KW);
    return ((p.conv.KH + h.step.d - 1) / h.step.d) * ((p.conv.KW + w.step.d - 1) / w.step.d) * p.conv.Cin;     // (at most K)
}

// Residue classes on 32 x 64 tiles (gemm_mfma_tile64.hip), as long as the 256 compute units hold all of them, two each, or, of a single round of k and up to 64 columns, one each.  Times in
// us, 128 x 128 tiles first: 140 tiles, Cin x taps of a class = 1024 12.8 and 9.9, 24 tiles, 512 9.4 and 7.8, 92 tiles, 256 7.8 and 6.9, 112 tiles, 128 7.7 and 6.4,
// 408 tiles, 1024 12.9 and 11.5, 332 tiles, 512 9.6 and 9.2, but 140 tiles, 64 5.9 and 6.4; 516 tiles, 256 7.8 and 11.1; 128, up to 256 tiles 0.92 of the time
// over 230 sizes, 257 to 512 tiles up to 64 columns 1.02 to 1.08 (8 x 53 x 9 x 128 -> 32, 2 x 2, stride 2, 6.7 and 7.2; 9 x 22 x 14 x 32 -> 32, 3 x 3, 6.8 and
// 7.1), 128 columns 0.90 to 0.92 (10 x 13 x 12 x 32 -> 128, 4 x 4, 392 tiles, 8.0 and 7.2).
// (Any weight row is reached from the first one with a 32-bit offset.)
static bool convt_tile64(const Problem& p) {
    const int k = convt_class_k(p);
    return k >= 128 && convt_row_tiles(p, 32) * ((p.N + 63) / 64) <= (k > 128 || p.N > 64 ? 512 : 256) && ((int64_t)p.K + 128) * p.ldb * 2 < ((int64_t)1 << 31);
}
static bool convt_by_class(const Problem& p, bool wide) {
    return p.K - convt_class_k(p) >= (!wide ? 128 : p.conv.Cin % 64 == 0 ? 320 : 640) && convt_classes_fit(p);
}

// 16-bit types: the translation unit (group) that holds a configuration
typedef hipError_t GroupFn(const Problem&, hipStream_t, int, int);
static hipError_t launch_group16(int cfg, GroupFn* const (&groups)[kNumGroups16], const Problem& p, hipStream_t stream, int group_m) {
    if (cfg < 0 || cfg > 31) return hipErrorInvalidValue;
    for (int g = 0; g < kNumGroups16; ++g)
        if ((kGroupMask16[g] >> cfg) & 1u) return groups[g](p, stream, cfg, group_m);
    return hipErrorInvalidValue;
}
hipError_t launch_mfma_bf16(const Problem& p, hipStream_t stream, int cfg, int group_m) {
    static GroupFn* const g[kNumGroups16] = {launch_mfma_bf16_g0, launch_mfma_bf16_g1, launch_mfma_bf16_g2,
                                             launch_mfma_bf16_g3, launch_mfma_bf16_g4, launch_mfma_bf16_g5, launch_mfma_bf16_g6, launch_mfma_bf16_g7};
    return launch_group16(cfg, g, p, stream, group_m);
}
hipError_t launch_mfma_f16(const Problem& p, hipStream_t stream, int cfg, int group_m) {
    static GroupFn* const g[kNumGroups16] = {launch_mfma_f16_g0, launch_mfma_f16_g1, launch_mfma_f16_g2,
                                             launch_mfma_f16_g3, launch_mfma_f16_g4, launch_mfma_f16_g5, launch_mfma_f16_g6, launch_mfma_f16_g7};
    return launch_group16(cfg, g, p, stream, group_m);
}

static hipError_t launch_convt(const Problem& p_in, hipStream_t stream, int force_cfg, const char** name) {
    Problem p = p_in;
    const long long t = (long long)((p.M + 127) / 128) * ((p.N + 255) / 256);
    const bool wide = p.M >= 128 && p.N >= 256 && t >= 256;
    const bool classes = force_cfg == 2 ? convt_classes_fit(p) : force_cfg != 0 && force_cfg != 6 && convt_by_class(p, wide && force_cfg != 1);
    p.conv.transposed = classes ? 2 : 1;
    int cfg = force_cfg;
    if (classes) {
        static const char* const names[] = {"mfma16_256x128x32_w4x2_a64_b6_pair_classes", "mfma16_320x128x32_w4x2_a64_b6_pair_classes",
                                            "mfma16_384x128x32_w4x2_a64_b6_pair_classes", "mfma16_448x128x32_w4x2_a64_b6_pair_classes"};
        if (force_cfg < 0 && convt_tile64(p)) {
            *name = "mfma16_tile64_32x64_s3_classes";
            return p.in_dtype == DT_BF16 ? launch_tile64_bf16(p, stream, kTile64Classes, 1, nullptr) : launch_tile64_f16(p, stream, kTile64Classes, 1, nullptr);
        }
        const bool tall = cfg >= 14 && cfg < kNumMfmaConfigs && p.conv.Cin % 64 == 0;
        if (cfg != 1 && cfg != 2 && !tall) {
            cfg = tall_config(p, convt_class_k(p));
            if (!cfg) cfg = square_config(p);
        }
        *name = cfg >= 14 ? names[cfg - 14] : cfg == 1 ? "mfma16_128x128x64_w2x4_s2_classes" : "mfma16_128x128x64_w2x4_s4_classes";
    } else {
        if (cfg != 0 && cfg != 1 && cfg != 6) cfg = wide || square_tiles(p) >= kTilesOf512 ? 6 : 1;
        *name = mfma_config_name(cfg, false);
    }
    const int group_m = group_m_override() > 0 ? group_m_override() : 8;
    return p.in_dtype == DT_BF16 ? launch_mfma_bf16(p, stream, cfg, group_m) : launch_mfma_f16(p, stream, cfg, group_m);
}

hipError_t launch_mfma(const Problem& p, hipStream_t stream, int force_cfg, const char** name) {
    const bool fp8 = p.in_dtype == DT_FP8_E4M3 || p.in_dtype == DT_FP8_E5M2;
    if (p.in_dtype == DT_F32) {
        long long t = (long long)((p.M + 127) / 128) * ((p.N + 255) / 256) * p.batch;
        int c = (force_cfg == 0 || force_cfg == 1) ? force_cfg : (p.M >= 128 && p.N >= 256 && t >= 256) ? 0 : 1;
        *name = c == 0 ? "mfma_f32_128x256x16_w1x4_s3_occ2" : "mfma_f32_128x128x32_w2x2_s2";
        return launch_mfma_f32(p, stream, c, 8);
    }
    if (p.in_dtype == DT_INT8) {
        // Up to two 128x128 tiles per compute unit those: they fill each other's waits in the long epilogue (32 x 28 x 28 x 128 -> 256, 3 x 3, 392
        // tiles: 17.8 us, with 256x256 28.3, with 128x256 23.3).  More tiles: both operands k-major the pair pipeline; a convolution 128x256, two per unit (64 x 28 x 28 x 64 -> 256, 3 x 3: 27.4 with 128x128, 26.8 with 256x256, 23.0; 48 x 56 x 56 x 128 ->
        // 256: 75, 88, 74; 64 x 56 x 56 x 256 -> 256: 164, 180, 154); a row-major product 256x256, but 128x128 where the epilogue is most of the time
        // (200704 x 256, K = 64: 52 and 68, 256: 65 and 87).
        const long long t128 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
        const bool kmajor = p.trans_b && !p.is_conv;
        const bool large = p.M >= 256 && p.N >= 256 && t128 > 512;
        // (k-major: the height of the pair pipeline's tiles as in 16 bits: 4608 x 4864 x 4480 104.9 and 88.7 us, 7590 x 2176 x 3712 90 and 65; from the second
        // 128x128 tile per unit on from K = 1024: 2048 x 4096 x 1024 15.0 and 14.8, x 4096 38.5 and 32.3)
        const int pair = pair_config8(p, t128, 1024);
        int c = (force_cfg == 0 || force_cfg == 1 || force_cfg == 2 || force_cfg == 4 || (force_cfg >= 8 && force_cfg <= 13)) ? force_cfg
                : pair ? pair : !large || kmajor || p.K < (p.is_conv ? 256 : 512) ? square_config(p) : p.is_conv ? 0 : 4;
        if (c >= 8 && !kmajor) c = 4;       // the 16x16 blocks are built for k-major operands only
        *name = mfma_config_name(c, true);
        const int gm = group_m_override() > 0 ? group_m_override() : 8;
        return launch_mfma_int8(p, stream, c, gm);
    }
    if (p.is_conv && p.conv.transposed) return launch_convt(p, stream, force_cfg, name);
    int cfg = (force_cfg >= 0 && force_cfg < kNumMfmaConfigs) ? force_cfg : choose_config(p);
    if (!fp8 && (cfg == 4 || cfg == 8 || (cfg == 3 && p.is_conv) || (cfg >= 14 && !p.is_conv))) cfg = choose_config(p);   // not built for 16-bit types, for plain products only, for convolutions only
    // 9 takes a convolution whose channel count is a multiple of 64
    if (cfg >= 9 && p.is_conv && p.conv.Cin % 64 != 0) cfg = 7;
    if (fp8) {
        // the FP8 instruction consumes a 64-deep k-tile (in 2-byte units) in two steps:
        // only the 64-deep configurations are built for it
        const bool kmajor = p.trans_b && !p.is_conv;
        if (force_cfg != 1 && force_cfg != 2 && force_cfg != 4 && !(force_cfg >= 9 && force_cfg <= 13 && kmajor)) {       // (also a forced 5-8)
            // k-major B: the pair pipeline as in 16 bits, up to two 128x128 tiles per compute unit from K = 384 on (e4m3 4222 x 1024 x 384: 8.1 and 7.9 us,
            // 2146 x 2688 x 256: 8.0 and 8.1, 4475 x 1664 x 768: 11.5 and 11.2, 1676 x 3328 x 2176: 18.9 and 16.3).  With a row-major B, whose 8-bit transposing reads two small workgroups
            // hide from each other, they stay ahead until the traffic of many tiles and a long contraction decides (3072 x 2048 x 4096: 58.2 and 29.2;
            // 8192 x 8192 x 2048: 187 and 143; 4096 x 4096 x 8192: 128 and 118; 8192 x 4096 x 4096: 153 and 154; 8192^3: 451 and 461).
            // A convolution's 256x256 tiles spill registers (32 x 56 x 56 x 256 -> 256, 3 x 3: 560 and 80 us).
            const long long t128 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
            const bool large = p.M >= 256 && p.N >= 256 && !kmajor && !p.is_conv && t128 > 2048 && p.K >= 4096;
            const int pair = pair_config8(p, t128, 384);
            cfg = pair ? pair : large ? 4 : square_config(p);
        } else {
            cfg = force_cfg;
        }
    }
    const int group_m = group_m_override() > 0 ? group_m_override() : 8;
    *name = mfma_config_name(cfg, fp8);
    if (fp8) return launch_mfma_fp8(p, stream, cfg, group_m);
    return p.in_dtype == DT_BF16 ? launch_mfma_bf16(p, stream, cfg, group_m)
                                 : launch_mfma_f16(p, stream, cfg, group_m);
}

}  // namespace pbk
