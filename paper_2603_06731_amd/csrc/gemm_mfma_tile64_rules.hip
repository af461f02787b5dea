// Which problems take the 64-wide tiles (gemm_mfma_tile64.hip), and which of their forms.
#include "gemm_mfma_tile64.h"
#include "gemm_mfma_8bit.h"
#include <algorithm>

namespace pbk {

// The alignment rules of the staged kernel (mfma_supported).  Transposed convolutions, which come here by their residue classes, are launch_convt's.
bool mfma_tile64_supported(const Problem& p) {
    if (p.in_dtype == DT_F32) return false;
    if (p.is_conv) {
        if (p.conv.transposed) return false;
        // the quotients k / Cin and tap / KW come from a 32-bit multiplication
        const int64_t lim = (int64_t)1 << 32;
        if (((int64_t)p.K + 256) * p.conv.Cin >= lim || ((int64_t)p.K / p.conv.Cin + 256) * p.conv.KW >= lim) return false;
    }
    return mfma_supported(p);
}

// Tile of a problem (the names in launch_type): where the 32 x 64 tiles, two workgroups per compute unit, make at
// most little more than one round of the 256 units, they win (512 x 1024 x 1024: 6.6 against 8.8 us for one 64 x 64 tile per
// unit; up to 256 tiles 0.70 to 0.83 of its time for K = 256 ... 4096; 257 to 320 tiles, twelve shapes with N = 512 ... 4160: K up to
// 1024 0.78 to 0.96, 2048 0.83 to 1.07, 4096 0.86 to 1.18 of the four-stage form; 577 x 1024 x 4096: 22.5 against 19.3 us with three stages; from
// 321 to 400 tiles K up to 1024 0.80 to 0.97, 4096 0.96 to 1.08), for a convolution, whose addresses cost vector instructions that a second
// workgroup hides, up to one round of 64 x 64 tiles (8 x 14 x 14 x 512 -> 512, 3 x 3: 24.0 against 33 us); then one 64 x 64
// tile per unit with a deep ring (256 x 4096 x 4096: 20.7 against 22.7 and 24.0 us; three stages are as good for short contractions and
// ahead for long ones: 577 x 1024 x 4096 20.1 against 19.3, k-major B 19.4 against 18.2, 256 x 1024 x 1024 8.6 and 8.5), beyond that two per unit
// (1024 x 2048 x 2048: 16.4 against 24.3 us).
// (8-bit types: K in 2-byte units)
static bool bits8(const Problem& p) { return p.in_dtype != DT_BF16 && p.in_dtype != DT_F16; }
static hipError_t launch_tile64(const Problem& p, hipStream_t stream, int cfg, int parts, const ScratchUse* use) {
    switch (p.in_dtype) {
    case DT_BF16: return launch_tile64_bf16(p, stream, cfg, parts, use);
    case DT_F16: return launch_tile64_f16(p, stream, cfg, parts, use);
    case DT_INT8: return launch_tile64_int8(to_k_units(p), stream, cfg, parts, use);
    case DT_FP8_E4M3: return launch_tile64_e4m3(to_k_units(p), stream, cfg, parts, use);
    default: return launch_tile64_e5m2(to_k_units(p), stream, cfg, parts, use);
    }
}
bool mfma_tile64_built(const Problem& p, int cfg) { return !bits8(p) || (cfg != 0 && cfg != 2); }       // 8-bit types: 32 x 64 only
static int tile64_k(const Problem& p) { return bits8(p) ? p.K / 2 : p.K; }
static int tile64_choice(const Problem& p) {
    const int K = tile64_k(p);
    const long long t32 = (long long)((p.M + 31) / 32) * ((p.N + 63) / 64) * p.batch;
    const long long t64 = (long long)((p.M + 63) / 64) * ((p.N + 63) / 64) * p.batch;
    if (p.M <= 32 || t32 <= 256 || (p.is_conv && t64 <= 256)) return 1;
    if (t32 <= 320 && K < 3072) return 1;
    return t64 > 256 ? 2 : K >= 2048 ? kTile64Deep : 0;
}

// Up to half a round of 128 x 128 tiles on the 256 compute units (measured against their deep ring: 64 tiles, K = 4096: 20.7
// against 27.5 us; 128 tiles, K = 2048: 16.4 against 17.3; 160 tiles, K = 1024: 18.0 against 11.7), and enough rounds of k:
// - one for the 32 x 64 tiles (577 x 1024 x 128: 4.9 against 5.7 us);
// - two for one 64 x 64 tile per unit (256 x 4096, k-major B: K = 128 5.8 against 5.7, 192 6.25 against 6.05, 256 6.2 against 6.6);
// - four for two of them, whose short rings do not fill before (1024 x 2048: K = 128 6.4 against 6.0, 192 7.2 against 6.5, 384
//   8.0 against 7.8, 512 8.6 against 9.1; 4 x 56 x 56 x 128 -> 512, 1 x 1, stride 2: 7.9 against 7.1);
// - nine for two of them in a convolution whose channels 64 divides, which costs the 128 x 128 tiles no address code (3 x 3 on 276 to 492 tiles of 64 x 64: K =
//   576 10.3 to 10.7 against 9.4 to 9.7, 1x1, stride 2, 256 8.1 against 6.9; 1152 13.5 to 14.5 against 13.3 to 14.7, 2304 20.5 against 21.6 to 22.0, 4608 34.1 against 38.9; 96 channels, K = 864
//   12.2 against 13.5).
// 8-bit types, 32 x 64 tiles against 128 x 128 ones (us, the latter first):
// - int8, whose quantised epilogue is a long chain for 128 x 128 elements: as long as two workgroups per unit hold all tiles (53 x 7 x 7 x 32 -> 128, 3 x 3:
//   9.2 and 5.4; 49 x 14 x 14 x 256 -> 128, stride 2 16.6 and 8.9; 4 x 56 x 56 x 256 -> 256, stride 2, 392 tiles 16.5 and 10.7; 20 x 28 x 28 x 256 -> 64, 1 x 1,
//   490: 7.4 and 6.2; 12 x 56 x 56 x 64 -> 128, stride 2, 588: 10.7 both; 25 x 28 x 28 x 256 -> 256, stride 2, 616: 16.5 and 18.1; 8 x 14 x 14 x 512 -> 512, 392: 25.2 and 18.0), long products
//   up to about one per unit;
// - FP8 up to about one per unit, from K = 256 on (211 x 1536 x 5376: 17.6 and 12.0; 134 x 1856 x 1024 6.7 and 5.7; 85 x 2304 x 512 5.5 and 4.9; 78 x 4032 x
//   128 4.3 and 4.6; 472 x 1216 x 512, 285 tiles, 5.6 and 5.7), with a k-major B and a long contraction up to one and a half (608 x 1280 x 4096, 380
//   tiles: 14.4 and 12.9; 397 x 1472 x 2048 9.0 and 8.7; 482 x 2304 x 7168, 576: 22.8 and 30.6; row-major 128 x 4352 x 3200, 272: 13.0 and 14.5).
bool mfma_tile64_preferred(const Problem& p) {
    if (bits8(p)) {
        const long long t32 = (long long)((p.M + 31) / 32) * ((p.N + 63) / 64) * p.batch;
        if (p.in_dtype == DT_INT8) return t32 <= (p.K <= 3072 || p.is_conv ? 512 : 272);
        const bool kmajor = p.trans_b && !p.is_conv;
        return p.K >= 256 && t32 <= (!kmajor ? 256 : p.K >= 2048 ? 384 : 272);
    }
    const long long t128 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
    const int c = tile64_choice(p), rounds = c == 1 ? 1 : c == 0 ? 2 : p.is_conv && p.conv.Cin % 64 == 0 ? 9 : 4;
    return t128 <= 128 && tile64_k(p) >= rounds * T64_BK;
}

// Workgroups that share a 32 x 64 tile (1: tiles are not split).  Times in us, "/": with the operands in the caches / from memory, as the
// weights of a model come.
//
// Matrices: the parts of all tiles fill the 256 compute units once (up to 128 tiles), each with at least four rounds.
// - Against whole tiles (ksplit up to 16 rows): 31 x 1344 x 13312, 21 tiles: 36.3 and 12.6 with 8 parts; 48 x 1024 x 16384: 45.4 and 13.1; 18 x 2112 x
//   4096: 13.7 and 8.6; 256 x 1024 x 3968, 128 tiles: 13.9 and 11.0 with 2.
// - The parts' meeting takes some 3 us and more with each part, which short contractions do not give back: 128 x 1024 x 1024: 6.4 and 6.9, 20 x 1024
//   x 1024: 6.3 and 6.3, 376 x 576 x 1856: 8.4 and 8.2; nor do they give back parts beyond 192 workgroups: 64 tiles with 3 and 4 parts,
//   32 x 4096 x 2048 8.5 and 9.2, 64 x 2048 x 4096 10.0/12.7 and 9.9/11.6, 123 x 1024 x 9216 14.4/19.3 and 13.2/16.5, but 1 x 4096 x 8192 14.7/18.5 and
//   14.9/19.4, x 13312 25.0 and 23.4; more than 256 workgroups lose (4 x 5632 x 13312, 88 tiles: 2 parts 39, 3 50).  78 to 85 tiles: 2 and 3 parts, 96 x
//   1664 x 2048 8.6/9.3 and 8.1/8.9, 59 x 2496 x 9216 17.6/22.7 and 14.6/18.4.
// - 129 to 170 tiles: three parts, two workgroups on nearly every unit, against whole tiles on little more than half of the units: 128 x 2304 x 6144
//   19.4/25.2 and 14.7/20.0, 64 x 5120 x 9216 44 and 33, 59 x 5440 x 2560 10.5 and 10.7, 64 x 4608 x 2048 9.1 and 9.4; up to 32 rows, whose whole tiles
//   read close to the rate of the memory, later: 32 x 8448 x 6144 29.9 and 26.0, 4 x 9216 x 8192 36.4 and 32.2, 16 x 10240 x 4096 15.2/21.5 and 17.5/20.0.
//   One or two rows over a row-major B, ksplit first, from memory / from the caches: 1 x 8640 x 6144 25.6/17.7 and 23.0/19.4, 2 x 9792 x 8192 33.9/24.4 and
//   32.2/26.1, x 15000 59.4/52.7 and 53.2/46.0, 1 x 10240 x 6144 31.1/21.7 and 31.8/24.6, 2 x 10816 x 8192 34.8/26.6 and 33.6/28.6.
//   (FP8 128 x 2304 x 8192: 16.1 and 12.5, 96 x 3200 x 6144 13.1 and 11.6, 160 x 2048 x 4096 10.1 and 10.0.)
// - Two parts only, from 86 tiles on, give back less: with operands in the caches, 256 x 1024 x 1536 7.7 and 8.7, x 1792 8.3 and 9.0, x 2304 9.6 and
//   9.7; from memory 9.95 and 9.24, 11.0 and 9.7, 12.8 and 10.7; 61 x 3328 x 1536 7.6 and 8.3, from memory 10.3 and 9.3.
// - Up to 16 rows, row-major B, against ksplit, which reads the same bytes without a meeting: 16 x 1664 x 3072 8.9/9.2 and 8.1/8.6, but 8 rows 8.0/8.3 and
//   8.1/8.6, one 7.0/7.4 and 8.0/8.4; one row, 3136 x 3072 7.0/10.2 and 8.7/9.7, but 8 11.6 and 9.8 from memory; 8 x 4096 x 3072 9.9/15.1 and 9.2/11.1, 4 x 1024 x 4096 7.1/15.2 and 8.9/9.7, 8 x 2560 x 2560 9.4/14.4 and 7.9/9.6 but 4 x 3072 x 2560 8.6/13.3 and 8.2/9.9,
//   2 x 4096 x 2560 8.2/12.4 and 9.2/10.2; 65 to 85 tiles: 2 x 4224 x 4096 9.2/14.1 and 10.2/11.6, x 5760 13.0/20.4 and 12.0/14.3, 8 x 5120 x
//   13312 78 and 32; 86 to 128: 1 x 7552 x 5760 15.4/19.9 and 17.1/18.6, 1 x 6208 x 8192 22.1/23.7 and 20.2/21.4, 8 x 4096 x 14336 57 and 28; 1 x 1152 x 4992 12.5/7.6 and 9.7/9.1; ksplit reads rows of B
//   a multiple of 512 bytes apart badly from memory, so that up to eight rows are split as early as nine there (4 x 2048 x 3584 15.6/6.4 and 9.8/8.6, 1 x 2560 x 3072
//   14.9/5.8 and 9.9/8.0, 4 x 3072 x 4032 19.0/10.8 and 11.3/8.9, 8 x 1024 x 5760 18.3/8.6 and 10.2/9.3, 1 x 4096 x 3584 15.6/6.2 and 11.6/8.8), and so are 8-bit
//   operands, which ksplit does not take (1 x 1408 x 4096, whole and split, 9.7 and 7.6); more than 8 rows
//   from 4096 on: 12 x 6976 x 5696 14.8/22.3 and 15.7/18.0, 16 x 8192 x 4096 16.9 and 15.4; k-major 8 x 1024 x 4096 7.0 and 8.0.
//   Results in fp32 only with four parts and more, whose four sums each are as many as ksplit's sixteen (its distance from 64 bits first, of the result: 16 x
//   8192 x 4096, two parts, 1.15e-7 and 1.35e-7, 3 x 8200 x 5640, three, 1.28e-7 and 1.31e-7, 8 x 4096 x 14336, four, 1.86e-7 and 1.81e-7).
//
// Convolutions, whose addresses cost vector instructions that a second workgroup hides: up to two workgroups per unit, each with about five rounds
// (batch x 14 x 14, 3 x 3; whole tiles, then by parts): 152 tiles, 36 rounds: 18.9 and 14.5 with 3; 104 tiles 18.8 and 12.5 with 4; 93 tiles, 36:
// 15.5 with 2, 12.2 with 5; 65 tiles, 27: 11.2 with 3, 10.7 with 5, 11.2 with 6; 56 tiles, 36: 12.5 with 3, 11.4 with 7; 42 tiles, 18: 9.3
// with 3, 8.9 with 5, 9.5 with 6; 150 tiles, 18 11.3 and 10.2 with 3, 152 tiles, 14 9.7 and 10.1; 104 tiles, 14 9.7 and 9.6; 76 tiles, 9: 7.7 and 8.2 with 3, 52
// tiles 7.6 and 7.9; from 171 tiles on 36 rounds 18.9 and 17.1 with 2, 27 15.2 and 14.9, 18 11.4 and 12.0.  (int8 4 x 14 x 14 x 512 -> 384, 18 rounds: 11.9
// and 11.2 with 3.)
//
// More 32 x 64 tiles than these rules split: 64 x 64 tiles, two workgroups per unit (512 of them; 32 x 64 tiles read more for the same product).  Products with
// N = 1024, bias and residual, whole and with 2 or 3 parts: 160 tiles, K = 3072 16.4, 16.6, 15.9 (k-major B 16.0 and 16.3 with 3), 4096 20.1, 18.9, 17.2,
// 6144 26.8, 24.0, 20.3; 208 tiles, 3072 15.4 and 15.6, 4096 18.9 and 18.0, 8192 32.9 and 27.5; 256 tiles 4096 20.2 and 20.0.  Where 32 x 64 tiles make
// one round, only longer ones: 128 tiles with 4, 4096 15.0 and 17.7, 6144 20.5 and 18.8, 8192 24.6 and 20.6; 96 with 5, 6144 20.1 and 17.6, 12288 36.1
// and 22.8; 207 x 2112 x 3648, 132 with 3, 13.9 and 15.9, 207 x 2240 x 5440 18.2 and 17.3.  Few rows of tiles, where B comes from memory: 100 x 6144 x
// 4096 18.9/26.0 and 20.1/28.9, 128 x 8192 x 8192 45.1 and 48.6, 196 x 3456 x 4608 21.9/25.6 and 20.2/27.0.
static int tile64_parts64(const Problem& p) {
    const long long t64 = (long long)((p.M + 63) / 64) * ((p.N + 63) / 64) * p.batch, t32 = (long long)((p.M + 31) / 32) * ((p.N + 63) / 64) * p.batch;
    if (bits8(p) || p.is_conv || p.M <= 192 || t32 <= 170 || t64 > 240) return 1;
    if (t32 <= 256) return p.K >= 5632 ? std::min(512 / (int)t64, 5) : 1;
    return t64 <= 170 ? (p.K >= 3328 ? 3 : 1) : p.K >= 4096 && p.M > 256 ? 2 : 1;
}
static int tile64_parts_of(const Problem& p, bool forced) {
    const long long all = (long long)((p.M + 31) / 32) * ((p.N + 63) / 64) * p.batch;
    const int rounds = (tile64_k(p) + T64_BK - 1) / T64_BK;
    if (all > 256) return 1;
    const int tiles = (int)all;
    if (p.is_conv) {
        const int once = std::min({256 / tiles, rounds / 3, 5});
        const int twice = std::min({512 / tiles, (rounds + 2) / 5, tiles <= 32 ? 8 : 6});
        return forced ? std::min({512 / tiles, rounds, 8}) : rounds < (tiles > 170 ? 24 : tiles > 128 ? 16 : 11) ? 1 : std::max(once, twice);
    }
    if (tiles > 128) return tiles <= 170 && rounds >= (p.M <= 32 ? 45 : 24) ? 3 : 1;
    if (!forced && rounds < 12) return 1;
    if (!forced && p.M <= 16) {
        const bool early = p.M > 8 || p.ldb % 256 == 0 || bits8(p);
        const bool fits = p.trans_b ? p.K >= 4096 && (int64_t)p.N * p.K >= 4000000
                                    : p.K >= (tiles <= 64 ? (p.M > 4 || early ? 3072 : 4096) : p.M > 8 ? 4096 : tiles <= 85 ? 4608 : 6144) && (int64_t)p.N * p.K >= (early ? 5000000 : 6000000);
        if (!fits) return 1;
    }
    int parts = std::min((192 + tiles / 2) / tiles, 8);
    if (parts == 2 && tiles <= 85 && rounds >= 14) parts = 3;
    if (rounds >= (p.M <= 16 ? 72 : 48)) parts = std::max(parts, std::min(256 / tiles, 5));
    if (!forced && parts == 2 && rounds < 14) return 1;
    return std::min(parts, forced ? rounds : rounds / 4);
}

static int tile64_parts(const Problem& p, bool forced) {
    const int parts = tile64_parts_of(p, forced);
    const bool ksplit_adds_sixteen = p.M <= 16 && !p.is_conv && !p.trans_b && !bits8(p) && p.out_dtype == DT_F32;
    return !forced && ksplit_adds_sixteen && parts < 4 ? 1 : parts;
}

bool mfma_tile64_split_preferred(const Problem& p) { return tile64_parts(p, false) > 1 || tile64_parts64(p) > 1; }

bool launch_mfma_tile64_split(const Problem& p, hipStream_t stream, bool forced, const char** name, hipError_t* e) {
    static_assert(256 <= kScratchTickets && 512 * 64 * T64_BN * 4 <= kScratchBytes, "what tile64_parts and tile64_parts64 ask for at most");
    const int parts32 = tile64_parts(p, forced), parts64 = parts32 > 1 || forced ? 1 : tile64_parts64(p);
    int dev = 0;
    if (std::max(parts32, parts64) <= 1 || hipGetDevice(&dev) != hipSuccess) return false;
    const ScratchUse use(dev, stream);
    if (!use) return false;
    *name = bits8(p) ? "mfma8_tile64_32x64_s3_split" : parts64 > 1 ? "mfma16_tile64_64x64_s2_split" : "mfma16_tile64_32x64_s3_split";
    *e = parts64 > 1 ? launch_tile64(p, stream, kTile64Split64, parts64, &use) : launch_tile64(p, stream, kSplitChoice, parts32, &use);
    return true;
}

hipError_t launch_mfma_tile64(const Problem& p, hipStream_t stream, int cfg, const char** name) {
    const int c = bits8(p) || cfg == kSplitChoice ? 1 : cfg >= 0 && cfg <= 2 ? cfg : tile64_choice(p);
    static const char* const names[4] = {"mfma16_tile64_64x64_s4", "mfma16_tile64_32x64_s3", "mfma16_tile64_64x64_s2", "mfma16_tile64_64x64_s3"};
    *name = bits8(p) ? "mfma8_tile64_32x64_s3" : names[c == kTile64Deep ? 3 : c];
    return launch_tile64(p, stream, c, 1, nullptr);
}

}  // namespace pbk
