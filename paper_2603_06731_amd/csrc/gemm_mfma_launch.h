// Instantiation and launch of the MFMA kernel for one element type.
// Included by one translation unit per dtype so they compile in parallel.
#pragma once
#include <atomic>
#include <cstdlib>
#include "gemm_mfma_kernel.h"

namespace pbk {

struct MfmaConfig {
    int id;
    int bm, bn, bk, wm, wn, stages;
    const char* name;
    const char* name8 = nullptr;       // 8-bit types, where their blocks are others
};

// Tile configurations (the static stand-in for the paper's analytical tile
// size model, Sec. 4.3): id -> workgroup tile and wave grid.
static const MfmaConfig kMfmaConfigs[] = {
    {0, 128, 256, 32, 1, 4, 3, "mfma_128x256x32_w1x4_s3_occ2"},
    {1, 128, 128, 64, 2, 4, 2, "mfma16_128x128x64_w2x4_s2", "mfma_128x128x64_w2x4_s2"},
    {2, 128, 128, 64, 2, 4, 4, "mfma16_128x128x64_w2x4_s4", "mfma_128x128x64_w2x4_s4"},      // 1 with a deeper ring: at most one tile per compute unit
    {3, 128, 128, 64, 2, 2, 2, "mfma_128x128x64_w2x2_s2"},          // 16-bit plain matrices of one or two k-tiles
    {4, 256, 256, 64, 2, 4, 2, "mfma_256x256x64_w2x4_s2"},          // 8-bit types only
    {5, 256, 256, 32, 2, 4, 4, "mfma16_256x256x32_w2x4_s4"},        // 16x16x32 MFMA blocks (16-bit types)
    {6, 128, 256, 32, 1, 4, 3, "mfma16_128x256x32_w1x4_s3_occ2"},
    {7, 256, 256, 32, 2, 4, 4, "mfma16_256x256x32_w2x4_s4_a64"},    // A staged 64 deep (plain matrices)
    {8, 256, 256, 64, 2, 4, 2, "mfma16_256x256x64_w2x4_s2"},        // int8, both operands k-major (16x16x64 blocks)
    {9, 256, 256, 32, 2, 4, 5, "mfma16_256x256x32_w2x4_a64_b6_pair"},   // as 7 with six B stages, one barrier per two k-tiles
    {10, 224, 256, 32, 2, 4, 5, "mfma16_224x256x32_w2x4_a64_b6_pair"},  // 9 with fewer rows, see pair_choice
    {11, 192, 256, 32, 2, 4, 5, "mfma16_192x256x32_w2x4_a64_b6_pair"},
    {12, 160, 256, 32, 2, 4, 5, "mfma16_160x256x32_w2x4_a64_b6_pair"},
    {13, 128, 256, 32, 2, 4, 5, "mfma16_128x256x32_w2x4_a64_b6_pair"},
    {14, 256, 128, 32, 4, 2, 5, "mfma16_256x128x32_w4x2_a64_b6_pair"},  // convolutions of up to 128 columns, transposed ones of any number, see tall_config
    {15, 320, 128, 32, 4, 2, 5, "mfma16_320x128x32_w4x2_a64_b6_pair"},
    {16, 384, 128, 32, 4, 2, 5, "mfma16_384x128x32_w4x2_a64_b6_pair"},
    {17, 448, 128, 32, 4, 2, 5, "mfma16_448x128x32_w4x2_a64_b6_pair"},
};
static const int kNumMfmaConfigs = sizeof(kMfmaConfigs) / sizeof(kMfmaConfigs[0]);
inline const char* mfma_config_name(int c, bool e8) { return e8 && kMfmaConfigs[c].name8 ? kMfmaConfigs[c].name8 : kMfmaConfigs[c].name; }

// XCD (accelerator complex die, each with its own L2) and compute unit counts of a device,
// asked once per device.  Workgroup ids are dealt round-robin to the XCDs, which the block
// mapping undoes.
struct DeviceShape { int xcds, cus; };
inline hipError_t device_shape(int dev, DeviceShape* out) {
    static std::atomic<unsigned> cache[32];          // xcds << 16 | cus; 0 = not asked yet
    const int slot = dev & 31;
    unsigned v = cache[slot].load(std::memory_order_acquire);
    if (!v) {
        int x = 0, c = 0;
        hipError_t e = hipDeviceGetAttribute(&x, hipDeviceAttributeNumberOfXccs, dev);
        if (e != hipSuccess || x < 1) { (void)hipGetLastError(); x = 1; }
        e = hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        v = ((unsigned)x << 16) | (unsigned)(c & 0xFFFF);
        cache[slot].store(v, std::memory_order_release);
    }
    out->xcds = (int)(v >> 16);
    out->cus = (int)(v & 0xFFFF);
    return hipSuccess;
}

// Tiles of bm rows of a transposed convolution: one set per residue class of the output, sized by the largest class.
inline long long convt_row_tiles(const Problem& p, int bm) {
    const ConvGeom& g = p.conv;
    const long long images = p.M / ((long long)g.OH * g.OW);
    const long long rows = images * ((g.OH + g.stride_h - 1) / g.stride_h) * ((g.OW + g.stride_w - 1) / g.stride_w);
    const long long classes = (long long)(g.stride_h < g.OH ? g.stride_h : g.OH) * (g.stride_w < g.OW ? g.stride_w : g.OW);
    return (rows + bm - 1) / bm * classes;
}

inline ConvTAxis convt_axis_of(int O, int stride, int dil, int ktaps) {
    int g = stride;
    for (int b = dil; b;) { const int r = g % b; g = b; b = r; }             // gcd(stride, dil)
    ConvTAxis a{};
    a.classes = stride < O ? stride : O;
    a.stride = FastDiv::of(stride);
    a.step = FastDiv::of(stride / g);
    a.d = -(dil / g);
    a.lift = (ktaps * dil + stride - 1) / stride;
    a.n = (O + stride - 1) / stride;
    a.full = O - (a.n - 1) * stride;
    return a;
}

inline void convt_geometry(const Problem& p, TileMapConvT* t) {
    const ConvGeom& g = p.conv;
    t->h = convt_axis_of(g.OH, g.stride_h, g.dil_h, g.KH);
    t->w = convt_axis_of(g.OW, g.stride_w, g.dil_w, g.KW);
    t->images = (int)(p.M / ((long long)g.OH * g.OW));
    t->classes = FastDiv::of(t->h.classes * t->w.classes);
    t->classes_w = FastDiv::of(t->w.classes);
    t->cin = FastDiv::of(g.Cin);
    auto at_least_1 = [](int v) { return v > 1 ? v : 1; };                   // (no class has none: not reached)
    for (int j = 0; j < 2; ++j) {
        const int cols = at_least_1(t->w.n - j);
        t->ow[j] = FastDiv::of(cols);
        for (int i = 0; i < 2; ++i) t->pix[i][j] = FastDiv::of(at_least_1(t->h.n - i) * cols);
        t->taps_w[j] = FastDiv::of(at_least_1(g.KW / t->w.step.d + j));
    }
}

template <typename T, typename TO, int BM, int BN, int BK, int WM, int WN, int MODE, int NSTAGE, int OCC, int MI = 32,
          int ASTG = 0>
hipError_t launch_one(const Problem& p, hipStream_t stream, int group_m) {
    constexpr int LDS_BYTES = mfma_lds_bytes(BM, BN, BK, WM * WN, NSTAGE, ASTG);
    auto kern = gemm_mfma_kernel<T, TO, BM, BN, BK, WM, WN, MODE, NSTAGE, OCC, MI, ASTG>;
    static std::atomic<unsigned> attr_done{0};      // bit per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    unsigned bit = 1u << (dev & 31);
    if (!(attr_done.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_done.fetch_or(bit, std::memory_order_release);
    }
    TileMapOf<MODE> tm{};
    tm.tiles_m = (p.M + BM - 1) / BM;
    tm.tiles_n = (p.N + BN - 1) / BN;
    if constexpr (MODE == MODE_CONVT) {
        const long long tiles = convt_row_tiles(p, BM);
        if (tiles * tm.tiles_n > 0x7FFFFFFFLL) return hipErrorInvalidValue;
        tm.tiles_m = (int)tiles;
        convt_geometry(p, &tm);
    }
    if constexpr (MODE == MODE_CONV || MODE == MODE_CONVT_ALL) {
        tm.pix = FastDiv::of(p.conv.OH * p.conv.OW);
        tm.ow = FastDiv::of(p.conv.OW);
        tm.cin = FastDiv::of(p.conv.Cin);
        tm.kw = FastDiv::of(p.conv.KW);
        tm.stride_h = FastDiv::of(p.conv.stride_h);
        tm.stride_w = FastDiv::of(p.conv.stride_w);
    }
    tm.tiles_per_batch = tm.tiles_m * tm.tiles_n;
    long long total = (long long)tm.tiles_per_batch * p.batch;
    if (total <= 0 || total > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    tm.total = (int)total;
    tm.group_m = group_m < 1 ? 1 : group_m;
    DeviceShape ds;
    e = device_shape(dev, &ds);
    if (e != hipSuccess) return e;
    tm.xcds = ds.xcds;
    // hipLaunchKernel reports this launch's own status; the per-thread "last error"
    // may hold an unrelated earlier failure of another library
    Problem pa = p;
    void* args[] = {&pa, &tm};
    return hipLaunchKernel((const void*)kern, dim3((unsigned)total), dim3(WM * WN * 64), args, LDS_BYTES, stream);
}

template <typename T, int BM, int BN, int BK, int WM, int WN, int NSTAGE, int OCC = 1, int MI = 32, int ASTG = 0>
hipError_t launch_modes(const Problem& p, hipStream_t stream, int group_m) {
    if constexpr (ASTG == 2) {            // 256 columns: plain matrices and convolutions; 128: convolutions and, by residue classes, transposed ones
        if (p.is_conv) {          // the image in 64-deep pieces: each must lie inside one filter tap
            if (p.conv.transposed == 1 || p.conv.Cin % 64 != 0) return hipErrorInvalidValue;
            if (p.conv.transposed) {
                if constexpr (BN == 128) return launch_one<T, T, BM, BN, BK, WM, WN, MODE_CONVT, NSTAGE, OCC, MI, ASTG>(p, stream, group_m);
                else return hipErrorInvalidValue;
            }
            return launch_one<T, T, BM, BN, BK, WM, WN, MODE_CONV, NSTAGE, OCC, MI, ASTG>(p, stream, group_m);
        }
        if constexpr (BN == 128) {
            return hipErrorInvalidValue;
        } else {
            if (p.trans_b) return launch_one<T, T, BM, BN, BK, WM, WN, MODE_TRANS_B, NSTAGE, OCC, MI, ASTG>(p, stream, group_m);
            return launch_one<T, T, BM, BN, BK, WM, WN, MODE_DENSE, NSTAGE, OCC, MI, ASTG>(p, stream, group_m);
        }
    } else {
    if constexpr (BM == 128 && BN == 128 && BK == 64 && WM == 2 && WN == 2) {
        if (p.is_conv) return hipErrorInvalidValue;
        if (p.trans_b) return launch_one<T, T, BM, BN, BK, WM, WN, MODE_TRANS_B, NSTAGE, OCC, MI>(p, stream, group_m);
        return launch_one<T, T, BM, BN, BK, WM, WN, MODE_DENSE, NSTAGE, OCC, MI>(p, stream, group_m);
    } else {
    if (p.is_conv && p.conv.transposed) {
        // by residue classes (2): configurations 1 and 2; all taps (1): configurations 0, 1 and 6
        if constexpr (BM == 128 && BN == 128 && BK == 64) {
            if (p.conv.transposed == 2) return launch_one<T, T, BM, BN, BK, WM, WN, MODE_CONVT, NSTAGE, OCC, MI>(p, stream, group_m);
        }
        if constexpr ((BM == 128 && BN == 256 && BK == 32) || (BM == 128 && BN == 128 && BK == 64 && NSTAGE == 2))
            return p.conv.transposed == 2 ? hipErrorInvalidValue
                                          : launch_one<T, T, BM, BN, BK, WM, WN, MODE_CONVT_ALL, NSTAGE, OCC, MI>(p, stream, group_m);
        else
            return hipErrorInvalidValue;
    }
    if (p.is_conv) return launch_one<T, T, BM, BN, BK, WM, WN, MODE_CONV, NSTAGE, OCC, MI>(p, stream, group_m);
    if (p.trans_b) return launch_one<T, T, BM, BN, BK, WM, WN, MODE_TRANS_B, NSTAGE, OCC, MI>(p, stream, group_m);
    return launch_one<T, T, BM, BN, BK, WM, WN, MODE_DENSE, NSTAGE, OCC, MI, ASTG>(p, stream, group_m);
    }
    }
}

// The 16-bit instantiations are split over several translation units (groups of configurations) so
// that they compile in parallel: MASK has bit i set where this unit builds configuration i.
// PBK_DEV_MASK (build-time, development only) removes configurations from every group.
#ifndef PBK_DEV_MASK
#define PBK_DEV_MASK 0xFFFFFFFFu
#endif
#define PBK_CASE(ID, ...) case ID: if constexpr (((MASK & (PBK_DEV_MASK)) >> ID) & 1u) return launch_modes<T, __VA_ARGS__>(p, stream, group_m); else return hipErrorInvalidValue;

template <typename T, unsigned MASK>
hipError_t launch_config(const Problem& p, hipStream_t stream, int cfg, int group_m) {
    switch (cfg) {
    PBK_CASE(0, 128, 256, 32, 1, 4, 3, 2)
    // 128 x 128 tiles on eight waves of 64 x 32: two waves per SIMD fill each other's waits for LDS, barriers and address code where one
    // workgroup has a compute unit, four where two have it.  With four waves of 64 x 64 on 32 x 32 blocks, before and after: 2048 x 2048 x 4096
    // 36.7 and 34.4 us, 2048 x 2048 x 256 8.8 and 7.7, 32 x 28 x 28 x 128 -> 128, 3 x 3, 16.7 and 14.4, 16 x 56 x 56 x 96 -> 64, 3 x 3 (two per unit), 22.1
    // and 18.1 (16.4 since waves without columns only fetch); 32 x 32 blocks on eight waves: 36.7, 7.8, 14.9, 21.2.  K-tiles of 32 in four stages for two per unit: 17.9 there, 8 to 25 % behind from
    // K = 1024 on (rows of 64 bytes).
    PBK_CASE(1, 128, 128, 64, 2, 4, 2, 2, 16)
    PBK_CASE(2, 128, 128, 64, 2, 4, 4, 1, 16)
    PBK_CASE(3, 128, 128, 64, 2, 2, 2)
    // 4 (32x32 blocks) is not built for the 16-bit types
    PBK_CASE(5, 256, 256, 32, 2, 4, 4, 1, 16)
    PBK_CASE(6, 128, 256, 32, 1, 4, 3, 2, 16)
    PBK_CASE(7, 256, 256, 32, 2, 4, 4, 1, 16, 1)
    PBK_CASE(9, 256, 256, 32, 2, 4, 5, 1, 16, 2)
    PBK_CASE(10, 224, 256, 32, 2, 4, 5, 1, 16, 2)
    PBK_CASE(11, 192, 256, 32, 2, 4, 5, 1, 16, 2)
    PBK_CASE(12, 160, 256, 32, 2, 4, 5, 1, 16, 2)
    PBK_CASE(13, 128, 256, 32, 2, 4, 5, 1, 16, 2)
    PBK_CASE(14, 256, 128, 32, 4, 2, 5, 1, 16, 2)
    PBK_CASE(15, 320, 128, 32, 4, 2, 5, 1, 16, 2)
    PBK_CASE(16, 384, 128, 32, 4, 2, 5, 1, 16, 2)
    PBK_CASE(17, 448, 128, 32, 4, 2, 5, 1, 16, 2)
    default: return hipErrorInvalidValue;
    }
}

// configuration groups of the 16-bit translation units (gemm_mfma_16bit.hip, once per type and group)
constexpr unsigned kGroupMask16[] = {
    (1u << 0) | (1u << 1) | (1u << 2),   // 0: the 32x32-block configuration and the 128 x 128 tiles
    (1u << 5) | (1u << 3),            // 1: 256x256x32, plain ring; 128 x 128 tiles on four waves
    (1u << 6),                        // 2: 128x256x32, two workgroups per compute unit
    (1u << 7),                        // 3: A staged 64 deep
    (1u << 9),                        // 4: ... with six B stages and one barrier per pair of k-tiles
    (1u << 10) | (1u << 12),          // 5: the same with 224 and 160 rows
    (1u << 11) | (1u << 13),          // 6: ... 192 and 128 rows
    (1u << 14) | (1u << 15) | (1u << 16) | (1u << 17),    // 7: ... and 128 columns
};
constexpr int kNumGroups16 = sizeof(kGroupMask16) / sizeof(kGroupMask16[0]);
#define PBK_DECLARE_GROUP16(NAME, G) hipError_t launch_mfma_##NAME##_g##G(const Problem& p, hipStream_t stream, int cfg, int group_m);
PBK_DECLARE_GROUP16(bf16, 0) PBK_DECLARE_GROUP16(bf16, 1) PBK_DECLARE_GROUP16(bf16, 2) PBK_DECLARE_GROUP16(bf16, 3) PBK_DECLARE_GROUP16(bf16, 4) PBK_DECLARE_GROUP16(bf16, 5) PBK_DECLARE_GROUP16(bf16, 6) PBK_DECLARE_GROUP16(bf16, 7)
PBK_DECLARE_GROUP16(f16, 0) PBK_DECLARE_GROUP16(f16, 1) PBK_DECLARE_GROUP16(f16, 2) PBK_DECLARE_GROUP16(f16, 3) PBK_DECLARE_GROUP16(f16, 4) PBK_DECLARE_GROUP16(f16, 5) PBK_DECLARE_GROUP16(f16, 6) PBK_DECLARE_GROUP16(f16, 7)

hipError_t launch_mfma_bf16(const Problem& p, hipStream_t stream, int cfg, int group_m);
hipError_t launch_mfma_fp8(const Problem& p, hipStream_t stream, int cfg, int group_m);
hipError_t launch_mfma_int8(const Problem& p, hipStream_t stream, int cfg, int group_m);
hipError_t launch_mfma_f32(const Problem& p, hipStream_t stream, int cfg, int group_m);
hipError_t launch_mfma_f16(const Problem& p, hipStream_t stream, int cfg, int group_m);

}  // namespace pbk
