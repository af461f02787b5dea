// A few rows against a weight matrix (decode; 16-bit types, M <= 16): the work is reading B once.
//
// Every wave of the workgroup owns the WHOLE 16 x 16 NF output tile and a share of the contraction: k is dealt to
// the waves in chunks of 64, so that the waves of a workgroup walk through memory side by side.  Nothing is shared
// between waves inside the loop, so operands go from global memory straight into the registers that the MFMA reads: no
// LDS round trip, no barrier, and four k32 steps of loads in flight per wave.  With 128-wide tiles such a problem occupies
// half the chip at best and walks K in one chain of barriers: 8 x 14336 x 4096 took 64 us, 28.1 here (24.0 with the 64-wide
// tiles, which take long contractions over many columns: mfma_ksplit_preferred).  At the end the waves' partial tiles meet in LDS once, are added in wave order (fixed: bit-exact from run to
// run) and leave through the fused epilogue.
//
// Layouts (v_mfma_f32_16x16x32: lane l supplies operand index l%16 and 8 k values of lane group l/16; it receives
// column l%16 of srcB's index and rows 4 (l/16) + 0..3 of srcA's):
//   A rows and a k-major B: one 16-byte load per lane is the fragment itself.
//   A row-major B: a lane loads NF neighbouring columns of 8 k rows and transposes them with one v_perm_b32 per
//   register; the column of lane l in fragment j is NF (l%16) + j, in the k-major form too, so that a lane ends up
//   with NF neighbouring columns of a row and stores them as one piece.
// Pieces outside the matrices are given an out-of-range buffer offset and arrive as zeros.
#include "gemm_mfma_launch.h"

namespace pbk {
namespace {

template <int N> struct VecN;
template <> struct VecN<2> { typedef int t; };
template <> struct VecN<4> { typedef int2v t; };

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const char* base) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)kOob, 0x00020000);
}

template <typename T, bool TRANS_B, int NF, int NW>
__global__ __launch_bounds__(NW * 64, NW / 4) void gemm_mfma_ksplit_kernel(Problem p, TileMap tm) {
    constexpr int DEPTH = 4;                        // k32 steps in flight
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;

    int b, tile_m, tile_n;
    map_tile(tm, blockIdx.x, b, tile_m, tile_n);
    const int m0 = tile_m * 16, n0 = tile_n * 16 * NF;
    const char* Ab = (const char*)p.A + ((int64_t)b * p.stride_a + (int64_t)m0 * p.lda) * 2;
    const char* Bb = (const char*)p.B + ((int64_t)b * p.stride_b + (TRANS_B ? (int64_t)n0 * p.ldb : (int64_t)n0)) * 2;

    // ---- per-lane offsets
    const unsigned a_voff = m0 + c < p.M ? (unsigned)(c * (int)p.lda * 2 + g * 16) : kOob;
    const int ldb2 = (int)p.ldb * 2;
    unsigned b_voff[TRANS_B ? NF : 1];
    if (TRANS_B) {
#pragma unroll
        for (int j = 0; j < NF; ++j) b_voff[j] = n0 + c * NF + j < p.N ? (unsigned)((c * NF + j) * ldb2 + g * 16) : kOob;
    } else {
        b_voff[0] = n0 + c * NF < p.N ? (unsigned)(8 * g * ldb2 + c * NF * 2) : kOob;
    }

    f32x4 acc[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    typedef typename VecN<NF>::t BVec;
    short8v af[DEPTH];
    BVec br[TRANS_B ? 1 : DEPTH][8];                // row-major B: NF columns of 8 k rows
    short8v bk[TRANS_B ? DEPTH : 1][NF];            // k-major B: the fragments themselves

    const int KS = (p.K + 63) / 64;                 // chunks of 64, dealt round-robin to the waves
    // k32 steps of this wave; the last chunk of all may consist of one step only
    const int steps = wave < KS ? 2 * ((KS - wave + NW - 1) / NW) - ((KS - 1) % NW == wave && p.K - (KS - 1) * 64 <= 32) : 0;

    auto load = [&](int u, int s) {
        const int k0 = ((wave + (s >> 1) * NW) * 2 + (s & 1)) * 32;
        if (s >= steps) return;                     // wave-uniform; a step that is not loaded is not multiplied either
        const bool k_in = k0 + 8 * g < p.K;         // K % 8 == 0: the lane's 8 values are all inside or all outside
        const __amdgpu_buffer_rsrc_t ra = buffer_of(Ab + (int64_t)k0 * 2);
        af[u] = __builtin_bit_cast(short8v, __builtin_amdgcn_raw_buffer_load_b128(ra, k_in ? (int)a_voff : (int)kOob, 0, 0));
        if constexpr (TRANS_B) {
            const __amdgpu_buffer_rsrc_t rb = buffer_of(Bb + (int64_t)k0 * 2);
#pragma unroll
            for (int j = 0; j < NF; ++j)
                bk[u][j] = __builtin_bit_cast(short8v, __builtin_amdgcn_raw_buffer_load_b128(rb, k_in ? (int)b_voff[j] : (int)kOob, 0, 0));
        } else {
            const __amdgpu_buffer_rsrc_t rb = buffer_of(Bb + (int64_t)k0 * ldb2);
            const int off = k_in ? (int)b_voff[0] : (int)kOob;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                if constexpr (NF == 4) br[u][r] = __builtin_bit_cast(BVec, __builtin_amdgcn_raw_buffer_load_b64(rb, off, r * ldb2, 0));
                else br[u][r] = __builtin_bit_cast(BVec, __builtin_amdgcn_raw_buffer_load_b32(rb, off, r * ldb2, 0));
            }
        }
    };
    auto compute = [&](int u) {
        short8v bf[NF];
        if constexpr (TRANS_B) {
#pragma unroll
            for (int j = 0; j < NF; ++j) bf[j] = bk[u][j];
        } else {
            // columns 2 i and 2 i + 1 of k rows 2 t and 2 t + 1 sit in register i of rows 2 t, 2 t + 1
#pragma unroll
            for (int i = 0; i < NF / 2; ++i) {
                int4v lo, hi;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    unsigned e, o;
                    if constexpr (NF == 2) { e = (unsigned)br[u][2 * t]; o = (unsigned)br[u][2 * t + 1]; }
                    else { e = (unsigned)br[u][2 * t][i]; o = (unsigned)br[u][2 * t + 1][i]; }
                    lo[t] = (int)__builtin_amdgcn_perm(o, e, 0x05040100u);
                    hi[t] = (int)__builtin_amdgcn_perm(o, e, 0x07060302u);
                }
                bf[2 * i] = __builtin_bit_cast(short8v, lo);
                bf[2 * i + 1] = __builtin_bit_cast(short8v, hi);
            }
        }
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[j] = MfmaOp16<T>::run(af[u], bf[j], acc[j]);
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) load(u, u);
    for (int s = 0; s < steps; s += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (s + u < steps) compute(u);
            load(u, s + u + DEPTH);
        }
    }

    // ---- partial tiles meet in LDS: entry r * 64 + lane holds row 4 g + r, columns NF c .. + NF
    typedef __attribute__((ext_vector_type(NF))) float FVec;
    constexpr int E = 4 * 64;
    static_assert(E <= NW * 64, "one entry per thread");
    FVec* red = (FVec*)lds;
    float bias_v[NF];
    unsigned res_v[NF];                             // as they lie in memory: converted after the barrier, not behind every load
    const bool has_bias = epi_has_bias(p.epi), out_f32 = p.out_dtype == DT_F32;
    const int64_t c_batch = (int64_t)b * p.stride_c;
    const int e = threadIdx.x, row = m0 + ((e & 63) >> 4) * 4 + ((e >> 6) & 3), col = n0 + (e & 15) * NF;
    const bool mine = e < E && row < p.M && col < p.N;
#pragma unroll
    for (int j = 0; j < NF; ++j) {                  // requested before the barrier, used after it
        const bool in = mine && col + j < p.N;
        bias_v[j] = has_bias && in ? p.bias[col + j] : 0.0f;
        res_v[j] = 0;
        if (p.R && in) {
            const int64_t o = c_batch + (int64_t)row * p.ldr + col + j;
            if (out_f32) res_v[j] = ((const unsigned*)p.R)[o]; else res_v[j] = ((const uint16_t*)p.R)[o];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        FVec v;
#pragma unroll
        for (int j = 0; j < NF; ++j) v[j] = acc[j][r];
        red[wave * E + r * 64 + lane] = v;
    }
    __syncthreads();
    if (!mine) return;
    FVec v = red[e];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w * E + e];
    float t[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const float res = out_f32 ? __uint_as_float(res_v[j]) : widen<T>(__builtin_bit_cast(T, (uint16_t)res_v[j]));
        t[j] = apply_epilogue(v[j], p.alpha, bias_v[j], p.epi, p.R ? p.beta : 0.0f, res);
    }
    const int osz = p.out_dtype == DT_F32 ? 4 : 2;
    const bool vec = col + NF <= p.N && p.ldc % NF == 0 && ((uintptr_t)p.C + (uintptr_t)c_batch * osz) % (NF * osz) == 0;
    const int64_t o = c_batch + (int64_t)row * p.ldc + col;
    if (p.out_dtype == DT_F32) {
        float* cp = (float*)p.C + o;
        if (vec) {
            FVec w;
#pragma unroll
            for (int j = 0; j < NF; ++j) w[j] = t[j];
            *(FVec*)cp = w;
        } else {
#pragma unroll
            for (int j = 0; j < NF; ++j) if (col + j < p.N) cp[j] = t[j];
        }
    } else {
        uint16_t* cp = (uint16_t*)p.C + o;
        if (vec) {
            BVec w;
            if constexpr (NF == 2) w = (int)pack2<T>(t[0], t[1]);
            else
#pragma unroll
                for (int j = 0; j < NF / 2; ++j) w[j] = (int)pack2<T>(t[2 * j], t[2 * j + 1]);
            *(BVec*)cp = w;
        } else {
#pragma unroll
            for (int j = 0; j < NF; ++j) if (col + j < p.N) cp[j] = to_bits16<T>(t[j]);
        }
    }
}

template <typename T, bool TRANS_B, int NF, int NW>
hipError_t launch_tile(const Problem& p, hipStream_t stream) {
    constexpr int LDS_BYTES = NW * NF * 1024;
    auto kern = gemm_mfma_ksplit_kernel<T, TRANS_B, NF, NW>;
    static std::atomic<unsigned> attr_done{0};      // bit per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned bit = 1u << (dev & 31);
    if (!(attr_done.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_done.fetch_or(bit, std::memory_order_release);
    }
    DeviceShape ds;
    e = device_shape(dev, &ds);
    if (e != hipSuccess) return e;
    TileMap tm{};
    tm.tiles_m = (p.M + 15) / 16;
    tm.tiles_n = (p.N + 16 * NF - 1) / (16 * NF);
    const long long total = (long long)tm.tiles_m * tm.tiles_n * p.batch;
    if (total <= 0 || total > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    tm.tiles_per_batch = tm.tiles_m * tm.tiles_n;
    tm.total = (int)total;
    tm.group_m = 8;
    tm.xcds = ds.xcds;
    Problem pa = p;
    void* args[] = {&pa, &tm};
    return hipLaunchKernel((const void*)kern, dim3((unsigned)total), dim3(NW * 64), args, LDS_BYTES, stream);
}

template <typename T>
hipError_t launch_type(const Problem& p, hipStream_t stream, int cfg, const char** name) {
    switch (cfg) {
    case 0:
        *name = "mfma16_ksplit_16x64_w16";
        return p.trans_b ? launch_tile<T, true, 4, 16>(p, stream) : launch_tile<T, false, 4, 16>(p, stream);
    case 1:
        *name = "mfma16_ksplit_16x32_w16";
        return p.trans_b ? launch_tile<T, true, 2, 16>(p, stream) : launch_tile<T, false, 2, 16>(p, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

static bool al(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Widest piece of a row of B (columns per lane) that N, the strides and the base allow: 4, 2 or none (0).
static int ksplit_columns(const Problem& p) {
    if (p.trans_b) return al(p.B, 16) && p.ldb % 8 == 0 && p.stride_b % 8 == 0 ? 4 : 0;
    for (int nf = 4; nf >= 2; nf /= 2)
        if (al(p.B, 2 * nf) && p.N % nf == 0 && p.ldb % nf == 0 && p.stride_b % nf == 0) return nf;
    return 0;
}

// 64 columns per workgroup, 32 where that would leave more than half of the 256 compute units without one (N = 14336: 28.6
// against 36.7 us; N = 4096, K = 4096: 15.1 against 13.1; N = 1024, K = 16384: 36 against 30) or pieces of 8 bytes are not aligned.
static int ksplit_choice(const Problem& p) {
    if (ksplit_columns(p) == 2) return 1;
    return (long long)((p.N + 63) / 64) * ((p.M + 15) / 16) * p.batch >= 128 ? 0 : 1;
}

// Plain matrices.  A (and a k-major B) is read in aligned 16-byte pieces that lie entirely inside or outside K, a row-major B in
// pieces of 8 or 4 bytes, so that N need only be even; per-lane buffer offsets are 32-bit and must stay below 2^31.
// A launch holds fewer than 2^32 threads, 1024 here per tile: a batch of small products that share B can ask for more.
bool mfma_ksplit_supported(const Problem& p) {
    if ((p.in_dtype != DT_BF16 && p.in_dtype != DT_F16) || p.is_conv) return false;
    if (p.K < 8 || p.K % 8 || p.lda % 8 || p.stride_a % 8 || !al(p.A, 16)) return false;
    const int64_t lim = (int64_t)1 << 31;
    if (256 * p.lda * 2 + 256 >= lim || 256 * p.ldb * 2 + 1024 >= lim || ksplit_columns(p) == 0) return false;
    const int cols = ksplit_choice(p) == 0 ? 64 : 32;
    return (long long)((p.N + cols - 1) / cols) * ((p.M + 15) / 16) * p.batch * 1024 < (1LL << 32);
}

// One row of tiles, and a contraction that gives half of the 16 waves a chunk.  A k-major B is read here in pieces of 64 bytes from
// 16 rows at once, which costs load rate: over enough columns the 64-wide tiles staged in LDS are faster (N = 14336, K =
// 4096: 26.2 against 29.3 us; N = 4096: 16.8 against 13.4; N = 1024, K = 16384: 44 against 34).  Over a row-major B of 128 to 256
// tiles of 64 columns those read better too, once the contraction is long (us, this kernel first: 8 x 14336 x 4096 28.1 and 24.0, 16 x 13184 x 4992 27.3
// and 24.8, 16 x 15296 x 14272 73 and 67, 12 x 10112 x 2944 11.9 and 11.4, 8 x 8768 x 960 5.9 and 6.2); up to four rows, whose A costs
// this kernel less, later (4 x 12800 x 5120 31.4 and 28.3, but 4 x 8960 x 3072 11.1 and 11.6), and one or two of them only from 193 tiles on, which leave
// few units without one (1 x 14336 x 4096, 224 tiles, 27.0 and 24.0 from memory, 21.3 and 20.2 from the caches, 13888, 217, 20.5 and 20.2, 17.9 and 18.0; 12288,
// 192, 23.0 and 23.7, 17.8 and 18.4; 10240, 160, 21.8 and 23.2, 15.6 and 15.7; 8448, 132, 19.4 and 21.6, 13.5 and 14.5; 1 x 12288 x 8192 42.5 and 43.6), unless
// rows of B are a multiple of 1 KiB apart that is none of 4 KiB (11776 25.8 and 23.5, 18.9 and 17.8, 11264 24.9 and 23.2, 8704 24.6 and 22.5); with more columns the two-per-unit tiles fill their last round badly (8 x 24576 x 4096 45.4 and 48.4).
// Results in fp32 stay here: sixteen sums of k / 16 values are nearer to 64 bits than four of k / 4 (8 x 14336 x 4096: 1.15e-7 and 1.88e-7 of the result, 16 x
// 15296 x 14272 1.87e-7 and 3.69e-7); rounded to 16 bits both are 1.6615e-3 away.
bool mfma_ksplit_preferred(const Problem& p) {
    if (p.M > 16 || p.K < 512) return false;
    if (ksplit_choice(p) == 1) return true;
    const long long tiles = (long long)((p.N + 63) / 64) * p.batch;
    const bool odd_kib = p.ldb % 512 == 0 && p.ldb % 2048 != 0;
    return !p.trans_b && (tiles <= (p.M <= 2 && !odd_kib ? 192 : 128) || tiles > 256 || p.out_dtype == DT_F32 || p.K < (p.M <= 4 ? 4096 : 2048) || !mfma_tile64_supported(p) || !mfma_tile64_preferred(p));
}

hipError_t launch_mfma_ksplit(const Problem& p, hipStream_t stream, int cfg, const char** name) {
    const int c = cfg > 0 || (cfg == 0 && ksplit_columns(p) == 4) ? cfg : ksplit_choice(p);
    return p.in_dtype == DT_BF16 ? launch_type<bf16_t>(p, stream, c, name) : launch_type<f16_t>(p, stream, c, name);
}

}  // namespace pbk
