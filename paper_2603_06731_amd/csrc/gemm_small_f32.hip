// Small fp32 contractions (the 256^3 case of the paper's Sec. 4.3 walk-through and its kind): up to some
// thousand output tiles, where the time is launch plus one memory latency, or a tile-per-workgroup kernel of
// the usual size would leave most compute units idle.
//
// A workgroup of up to 16 waves computes a 16 x 16 tile of C with v_mfma_f32_16x16x4_f32 (true binary32 products and sums), each
// wave over a contiguous share of k; the waves' sums meet in LDS and are added in wave order.  Nothing else is staged: a lane
// loads its operand values straight into the registers the matrix instruction reads, 64 k at a time into one of two register sets.
// What bounds it: launch, one memory latency and the meeting; the chain of matrix instructions (16 per 64 k, 32 clocks each)
// and the loads are split over the waves.  With one wave per tile, and every load behind a test of its lane, a tile took 30 ns for every k: 256 x
// 256 x 256 7.0 against 4.0 us, 71 x 128 x 804 24.5 against 5.7.
// Many tiles are bound by the loads of operands that other tiles load too, and take 32 x 32 ones: 1024 x 1024 x 1024 53 against 33 us (69 on
// 128 x 128 tiles, which then occupy a quarter of the chip).
//
// Operand layout of the instruction (k = 4 per issue): lane l supplies, for the operand whose tile index is
// l % 16, the value at k = l / 16.  The sum over k is order-free, so lane group q = l / 16 takes the k
// positions 16 J + 4 q + i (i = 0..3) of each block of 16: one 16-byte load per block from a k-major operand.
// The accumulator is computed transposed (B^T A^T), which leaves a lane with four neighbouring columns of
// one row of C: a 16-byte store.
#include <hip/hip_runtime.h>
#include "pbk_problem.h"
#include "pbk_epilogue.h"

namespace pbk {
namespace {

typedef float __attribute__((ext_vector_type(4))) f32x4s;

constexpr int SKC = 64;                  // k per register set
constexpr int SBLK = SKC / 16;           // blocks of 16 k per set

// N neighbouring floats from an address that is only known to be 4-byte aligned, as one load
template <int N> __device__ __forceinline__ auto ld_floats(const float* p) {
    typedef __attribute__((ext_vector_type(N))) float V;
    V v;
    __builtin_memcpy(&v, (const __attribute__((address_space(1))) char*)p, sizeof(V));
    return v;
}

// four consecutive k of a k-major row, zero beyond kend
__device__ __forceinline__ f32x4s ld_k4(const float* row, int k, int kend) {
    f32x4s v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (k + 4 <= kend) return ld_floats<4>(row + k);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (k + i < kend) v[i] = row[k + i];
    return v;
}

// F x F blocks of 16 x 16 per workgroup (F = 1 or 2); waves: of the workgroup (1 to 16); per_wave: k of each but the last, a multiple of 16.
// Column c of block j is n0 + F c + j, so that a lane loads F neighbouring values of a row-major B at once and ends up with 4 F neighbouring
// columns of C.
template <bool TRANS_B, int F>
__global__ __launch_bounds__(F == 1 ? 1024 : 512) void gemm_small_f32_kernel(Problem p, int tiles_m, int tiles_n, int waves, int per_wave) {
    typedef __attribute__((ext_vector_type(F))) float BVec;
    __shared__ f32x4s sums[(F == 1 ? 16 : 8) * 64 * F * F];
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bid = blockIdx.x;
    const int tn = bid % tiles_n;
    bid /= tiles_n;
    const int tm = bid % tiles_m;
    const int b = bid / tiles_m;
    const int m0 = tm * 16 * F, n0 = tn * 16 * F;
    const float* A = (const float*)p.A + (int64_t)b * p.stride_a;
    const float* B = (const float*)p.B + (int64_t)b * p.stride_b;

    // (rows beyond M and columns beyond N repeat the last ones: what comes of them is not stored)
    const float* a_row[F];
    const float* b_row[F];             // k-major B (trans_b): rows of B like rows of A; otherwise columns of its k-rows
#pragma unroll
    for (int i = 0; i < F; ++i) {
        a_row[i] = A + (int64_t)(m0 + 16 * i + r < p.M ? m0 + 16 * i + r : p.M - 1) * p.lda;
        const int n = n0 + F * r + i < p.N ? n0 + F * r + i : p.N - 1;
        b_row[i] = TRANS_B ? B + (int64_t)n * p.ldb : B + n;
    }
    // a pair of a row-major B at the edge of an odd N starts one column earlier and gives its second value to both
    const bool pairs = F == 1 || p.N >= F;
    const float* b_pair = TRANS_B ? nullptr : B + (n0 + F * r + F <= p.N || !pairs ? n0 + F * r : p.N - F);
    const bool edge = F == 2 && n0 + F * r + 1 == p.N;
    const int k_begin = wave * per_wave, k_end = wave + 1 == waves ? p.K : k_begin + per_wave;      // (the last one has what is left)

    f32x4s av[2][F][SBLK], bv[2][F][SBLK];
    auto load = [&](int s, int kb) __attribute__((always_inline)) {
        if (kb + SKC <= k_end && (TRANS_B || pairs)) {            // wave-uniform; no load behind a test of its lane
#pragma unroll
            for (int J = 0; J < SBLK; ++J) {
                const int k = kb + 16 * J + 4 * q;
#pragma unroll
                for (int f = 0; f < F; ++f) av[s][f][J] = ld_floats<4>(a_row[f] + k);
                if (TRANS_B) {
#pragma unroll
                    for (int f = 0; f < F; ++f) bv[s][f][J] = ld_floats<4>(b_row[f] + k);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const BVec v = ld_floats<F>(b_pair + (int64_t)(k + i) * p.ldb);
#pragma unroll
                        for (int f = 0; f < F; ++f) bv[s][f][J][i] = edge ? v[F - 1] : v[f];
                    }
                }
            }
            return;
        }
#pragma unroll
        for (int J = 0; J < SBLK; ++J) {
            const int k = kb + 16 * J + 4 * q;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                av[s][f][J] = ld_k4(a_row[f], k, k_end);
                if (TRANS_B) {
                    bv[s][f][J] = ld_k4(b_row[f], k, k_end);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) bv[s][f][J][i] = k + i < k_end ? b_row[f][(int64_t)(k + i) * p.ldb] : 0.0f;
                }
            }
        }
    };
    f32x4s acc[F][F];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = f32x4s{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int J = 0; J < SBLK; ++J)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < F; ++i)
#pragma unroll
                    for (int j = 0; j < F; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[s][j][J][e], av[s][i][J][e], acc[i][j], 0, 0, 0);
    };
    load(0, k_begin);
    if (k_begin + SKC < k_end) load(1, k_begin + SKC);
    for (int kb = k_begin; kb < k_end; kb += 2 * SKC) {
        multiply(0);
        if (kb + 2 * SKC < k_end) load(0, kb + 2 * SKC);
        if (kb + SKC < k_end) {
            multiply(1);
            if (kb + 3 * SKC < k_end) load(1, kb + 3 * SKC);
        }
    }
    if (waves > 1) {
#pragma unroll
        for (int i = 0; i < F * F; ++i) sums[(wave * F * F + i) * 64 + lane] = acc[i / F][i % F];
        __syncthreads();
        if (wave > 0) return;
        for (int w = 1; w < waves; ++w)
#pragma unroll
            for (int i = 0; i < F * F; ++i) acc[i / F][i % F] += sums[(w * F * F + i) * 64 + lane];
    }

    // lane: rows m0 + 16 i + r, columns n0 + 4 F q .. + 4 F - 1
    const bool has_bias = epi_has_bias(p.epi);
    const bool c_vec = (p.ldc & 3) == 0 && (((uintptr_t)p.C & 15) == 0) && ((p.stride_c & 3) == 0);
#pragma unroll
    for (int i = 0; i < F; ++i) {
        const int gm = m0 + 16 * i + r;
#pragma unroll
        for (int h = 0; h < F; ++h) {                 // four columns at a time
            const int gn = n0 + 4 * F * q + 4 * h;
            if (gm >= p.M || gn >= p.N) continue;
            float* c_row = (float*)p.C + (int64_t)b * p.stride_c + (int64_t)gm * p.ldc + gn;
            const float* r_row = p.R ? (const float*)p.R + (int64_t)b * p.stride_c + (int64_t)gm * p.ldr + gn : nullptr;
            f32x4s out;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 4 * h + e;              // column c of the lane's: block c % F, element c / F
                const bool in = gn + e < p.N;
                const float bias = (has_bias && in) ? p.bias[gn + e] : 0.0f;
                const float res = (r_row && in) ? r_row[e] : 0.0f;
                out[e] = apply_epilogue(acc[i][c % F][c / F], p.alpha, bias, p.epi, p.beta, res);
            }
            if (gn + 4 <= p.N && c_vec) {
                *(f32x4s*)c_row = out;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (gn + e < p.N) c_row[e] = out[e];
            }
        }
    }
}

}  // namespace

// fp32 in and out, plain (batched) matmul
bool small_f32_supported(const Problem& p) {
    if (p.in_dtype != DT_F32 || p.out_dtype != DT_F32 || p.is_conv) return false;
    if (p.M < 1 || p.N < 1 || p.K < 1) return false;
    const long long tiles = (long long)((p.M + 15) / 16) * ((p.N + 15) / 16) * p.batch;
    return tiles <= 0x7FFFFFFFLL;
}

static long long tiles_of(const Problem& p, int n) { return (long long)((p.M + n - 1) / n) * ((p.N + n - 1) / n) * p.batch; }

// 32 x 32 tiles from some 2400 tiles of 16 x 16 on (2025 tiles, 720 x 720 x 1024: 25 against 31 us; 2304, 768 x 768 x 256: 9.8 and 11.7; 2500, 800 x 800 x
// 800: 34 and 28; 4096: 53 and 33, K = 64: 7.5 and 7.4), except (their time first)
// - where half of them would be empty (16 x 38416 x 64 10.6 and 7.0, 65536 x 16 x 256 31 and 19), unless a row-major B of many columns is read for a long
//   time (5 x 60001 x 512 50 and 53, 1000 of 3 x 50 x 1024 85 and 113; 1 x 65536 x 256 27 and 25, 16 x 50000 x 1024 77 and 63);
// - where there are more of them than the SIMDs have waves for at once, unless not by much and a row-major B is read for long (40 x 21001 x 64, 1314 of
//   them, 11.4 and 9.5, x 256 25.5 and 28.5, k-major 23.5 and 19.5; 450 of 33 x 46 x 64, 1800 of them, 15.0 and 10.7).
static bool blocks32(const Problem& p) {
    const long long t16 = tiles_of(p, 16), t32 = tiles_of(p, 32);
    if (t16 <= 2400) return false;
    if (p.M <= 16 || p.N <= 16) return p.M <= 16 && !p.trans_b && t16 > 3500 && p.K >= 512;
    return t32 <= 1024 || (t32 <= 1320 && !p.trans_b && p.K > 100);
}

// Up to 4096 tiles of 16 x 16, which are 1024 waves of 32 x 32, one per SIMD (in us, against 128 x 128 tiles of the main kernel):
// 512 x 512 x 512: 7.9 against 35.5, 800 x 800 x 800: 28 against 56, 1024 x 1024 x 1024: 33 against 69, x 64: 7.4 against 9.2, but x 32: 7.5 and 7.2 (1000 x
// 1001 x 32, k-major B, rows of C not aligned: 9.7 and 13.5); 1280 x 1280 x 1024: 75 against 70, 1536 x 1536 x 512: 57 against 39.
// With more than nine tiles per compute unit the generic kernel, whose tiles are 64 x 64, is ahead in some cases (its time first):
// - short contractions, and one to three rows or columns, so that most of every tile is empty: 1 x 38416 x 16 5.0 and 5.8, x 32: 6.4 and 7.0, x 40: 7.5 and
//   7.4; 2 x 65536 x 16 6.4 and 8.1; 65536 x 1 x 16 6.2 and 7.0; 1000 of 3 x 50 x 16 7.0 and 8.1; but 1 x 36000 x 16 5.0 and 4.5, 4 x 65536 x 16 8.4 and 8.1, 2000 of
//   2 x 30 x 16 8.6 and 7.5;
// - short contractions, whose time are the stores, if rows of C are not aligned and the generic kernel's tiles not empty either: 4000 x 250 x 16 8.3 and
//   9.6, x 32: 9.5 and 9.8, x 40: 10.5 and 9.9; 250 of 60 x 63 x 40 9.4 and 10.2, x 64: 10.5 and 9.9; 64 x 16001 x 40 10.7 and 11.0; but aligned, 48 x 16384 x
//   16, 7.8 and 7.0, and 1000 of 30 x 30 x 16 8.4 and 7.8;
// - far more 32 x 32 tiles than waves at once, except for a middling contraction or with a k-major B: 450 of 33 x 46, K = 16 7.3 and 8.7, 64 10.7 and 10.7,
//   128 15.3 and 18.0, 512 43 and 62 (k-major 15 and 12, 42 and 36).
bool small_f32_preferred(const Problem& p) {
    const long long t = tiles_of(p, 16);
    if (t > 4096 || p.K > 4096) return false;
    if (t <= 2304) return true;
    const bool aligned = p.ldc % 4 == 0 && p.stride_c % 4 == 0 && (uintptr_t)p.C % 16 == 0;
    if (mfma_supported(p) && mfma_preferred(p)) return p.K > 32 || !aligned;         // (otherwise against the generic kernel)
    if (p.M < 4 || p.N < 4) return p.K > 32 || (p.M < 48 && p.N < 48);
    if (t <= 2400 || p.M <= 16 || p.N <= 16) return true;
    const long long t32 = tiles_of(p, 32);
    if (t32 > 1320) return p.K >= 64 && (p.K == 64 || p.trans_b);
    if (t32 > 1024) return p.K > 40;
    return aligned || p.K > (!p.trans_b && (p.M <= 64 || p.N <= 64) ? 48 : 32) || 2ll * p.M * p.N * p.batch < 4096 * tiles_of(p, 64);
}

// Waves per tile: as many as the SIMDs (1024) have room for, with 128 k or more for each (256 x 256 x 256: 4.4 us with 1, 4.0 with 2 or 4, 4.7
// with 8; 128 x 128 x 1024: 10.7, 7.1, 5.4, 5.9; 512 x 512 x 512: 7.9, 8.0, 8.8, 8.9).
template <int F>
static hipError_t launch_blocks(const Problem& p, hipStream_t stream) {
    int tiles_m = (p.M + 16 * F - 1) / (16 * F), tiles_n = (p.N + 16 * F - 1) / (16 * F);
    const long long blocks = (long long)tiles_m * tiles_n * p.batch;
    if (blocks <= 0 || blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    int waves = 1;
    while (waves < (F == 1 ? 16 : 8) && waves * 2 * 128 <= p.K && blocks * waves * 2 <= 1024) waves *= 2;
    int per_wave = (int)(((long long)p.K + 15) / 16 + waves - 1) / waves * 16;
    waves = (int)(((long long)p.K + per_wave - 1) / per_wave);
    Problem pa = p;
    void* args[] = {&pa, &tiles_m, &tiles_n, &waves, &per_wave};
    const void* kern = p.trans_b ? (const void*)gemm_small_f32_kernel<true, F> : (const void*)gemm_small_f32_kernel<false, F>;
    return hipLaunchKernel(kern, dim3((unsigned)blocks), dim3(64 * waves), args, 0, stream);
}

hipError_t launch_small_f32(const Problem& p, hipStream_t stream, const char** name) {
    if (!blocks32(p)) {
        *name = "small_f32_16x16_mfma4";
        return launch_blocks<1>(p, stream);
    }
    *name = "small_f32_32x32_mfma4";
    return launch_blocks<2>(p, stream);
}

}  // namespace pbk
