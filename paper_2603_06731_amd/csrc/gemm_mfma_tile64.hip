// MFMA kernel with 64-wide output tiles for problems whose 128-wide tiles leave compute units idle (16-bit types): the
// layers of a block for some hundred tokens, convolutions over small images or with few output channels.
//
// A workgroup of 4 waves owns a BM x 64 tile.  The k axis advances in rounds of 128: the operands of a round are
// staged in LDS by all waves (direct-to-LDS loads of 16 bytes per lane along the rows, whole lines), and then every
// wave multiplies the WHOLE tile over its own 32 of the 128 k values, so that each staged byte is read from LDS once.
// The waves' partial tiles meet in LDS at the end and are added in wave order (fixed: bit-exact from run to run).
// With few tiles several workgroups share one, each with a run of the rounds (SPLIT); their sums meet in scratch memory (scratch.h).
// What bounds it: the chain of rounds of a workgroup that is alone on its compute unit (N = 1024: 64 x 64 tiles 5.4 us and
// 0.47 us per round, 32 x 64 tiles 4.2 and 0.34, with 32 workgroups on the chip as with 256); with two on a unit, its load
// path, 70 to 84 GB/s.  577 x 1024 x 4096 with bias and residual (304 tiles of 32 x 64, two on 48 of the units): 48.6 us with
// 128 x 128 tiles (40 of them), 20.1 here with 64 x 64 tiles.  Reading the next round's fragments under this
// round's MFMAs, with loads issued between them, was 10 % slower (its ring has one stage less in flight).
//
// LDS images: k-major operands (A, B with trans_b) [rows][128 k], 16-byte chunk index XORed with row % 16; row-major B
// [128 k][64 n], 32-byte slots XORed with bits 1 and 3 of k (the transposing read of one 16-column block touches rows
// k..k+3 and k+8..k+11 of one slot).  Both are free of bank conflicts.  The MFMA takes B as its first operand, so a lane
// holds 4 neighbouring columns of one row.
#include "gemm_mfma_launch.h"
#include "scratch.h"

namespace pbk {
namespace {

constexpr int T64_BN = 64, T64_BK = 128, T64_NW = 4;

__device__ __forceinline__ int t64_row_slot(int k) { return ((k >> 1) & 1) | (((k >> 3) & 1) << 1); }

// exact quotient by a divisor d for numerators n with n * d < 2^32: magic = ceil(2^32 / d) (d = 1: 0 stands for 2^32)
__device__ __forceinline__ int t64_div(int n, unsigned magic) { return magic ? (int)__umulhi((unsigned)n, magic) : n; }

// SPLIT: `parts` workgroups per tile, each with a run of the rounds of k
template <typename T, int MODE, int BM, int NSTAGE, bool SPLIT>
__global__ __launch_bounds__(T64_NW * 64, 1) void gemm_mfma_tile64_kernel(Problem p, TileMap tm, unsigned cin_magic, unsigned kw_magic, int parts,
                                                                          Scratch scratch) {
    constexpr bool TRANS_B = MODE == MODE_TRANS_B, CONV = MODE == MODE_CONV;
    constexpr int FM = BM / 16, FN = T64_BN / 16;
    constexpr int A_BYTES = BM * T64_BK * 2, STAGE = A_BYTES + T64_BN * T64_BK * 2;
    constexpr int CA = A_BYTES / 1024 / T64_NW, CB = (STAGE - A_BYTES) / 1024 / T64_NW;   // loads per wave and round
    constexpr int LOADS = CA + CB;
    static_assert(NSTAGE * STAGE <= 160 * 1024 && T64_NW * BM * T64_BN * 4 <= NSTAGE * STAGE, "LDS");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;

    int b, tile_m, tile_n;
    map_tile(tm, blockIdx.x, b, tile_m, tile_n);
    // (split: the map's batches are the parts, so that an XCD works on few runs of k, each of them on many tiles)
    const int part = SPLIT ? b / p.batch : 0;
    if (SPLIT) b -= part * p.batch;
    const int m0 = tile_m * BM, n0 = tile_n * T64_BN;
    // What the end of the kernel needs of the problem is read here and kept: left to the compiler, the scalar loads stand there, and their latency is
    // a twentieth of a small call (9 x 7 x 7 x 64 -> 256, 3 x 3, stride 2: 6.7 against 6.3 us).
    struct { float alpha, beta; int epi, out_dtype, M, N; int64_t ldc, ldr, stride_c; const float* bias; void* C; const void* R; } end =
        {p.alpha, p.beta, (int)p.epi, (int)p.out_dtype, (int)p.M, (int)p.N, p.ldc, p.ldr, p.stride_c, p.bias, p.C, p.R};
    asm volatile("" : "+s"(end.alpha), "+s"(end.beta), "+s"(end.epi), "+s"(end.out_dtype), "+s"(end.M), "+s"(end.N));
    asm volatile("" : "+s"(end.ldc), "+s"(end.ldr), "+s"(end.stride_c), "+s"(end.bias), "+s"(end.C), "+s"(end.R));
    const char* Ab = (const char*)p.A + (CONV ? 0 : ((int64_t)b * p.stride_a + (int64_t)m0 * p.lda) * 2);
    const char* Bb = (const char*)p.B + ((int64_t)b * p.stride_b + (TRANS_B ? (int64_t)n0 * p.ldb : (int64_t)n0)) * 2;

    // ---- per-lane sources of the staging loads: lane i of load r lands at byte 16 i of its KiB
    unsigned a_voff[CA], b_voff[CB];
    int a_k[CA], b_k[CB];                           // k of the piece inside the round
    int a_ih[CA], a_iw[CA];
#pragma unroll
    for (int r = 0; r < CA; ++r) {
        const int row = (wave * CA + r) * 4 + g, chunk = c ^ (row & 15), m = m0 + row;
        const bool ok = m < p.M;
        a_k[r] = chunk * 8;
        if (CONV) {
            const int pix = p.conv.OH * p.conv.OW;
            const int mc = ok ? m : 0;
            const int n = mc / pix, rem = mc - n * pix, oh = rem / p.conv.OW, ow = rem - oh * p.conv.OW;
            // (a row beyond M starts so far above the image that no tap reaches it)
            a_ih[r] = ok ? oh * p.conv.stride_h - p.conv.pad_h : -(1 << 30);
            a_iw[r] = ow * p.conv.stride_w - p.conv.pad_w;
            a_voff[r] = (unsigned)(((n * p.conv.H + oh * p.conv.stride_h - p.conv.pad_h) * p.conv.W + a_iw[r]) * p.conv.Cin * 2);
        } else {
            a_voff[r] = ok ? (unsigned)(row * (int)p.lda * 2 + chunk * 16) : kOob;
            a_ih[r] = a_iw[r] = 0;
        }
    }
#pragma unroll
    for (int r = 0; r < CB; ++r) {
        if (TRANS_B) {
            const int row = (wave * CB + r) * 4 + g, chunk = c ^ (row & 15);
            b_k[r] = chunk * 8;
            b_voff[r] = n0 + row < p.N ? (unsigned)(row * (int)p.ldb * 2 + chunk * 16) : kOob;
        } else {
            const int krow = (wave * CB + r) * 8 + (lane >> 3), half = lane & 7;
            const int nb = (((half >> 1) ^ t64_row_slot(krow)) << 5) | ((half & 1) << 4);    // byte of the row
            b_k[r] = krow;
            b_voff[r] = n0 + (nb >> 1) < p.N ? (unsigned)(krow * (int)p.ldb * 2 + nb) : kOob;
        }
    }
    const unsigned lds_base = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_addr_of(lds));

    auto dma = [&](int4v rsrc, unsigned addr, unsigned voff) {
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(addr), "v"(voff), "s"(rsrc) : "memory", "m0");
    };
    const int all = (p.K + T64_BK - 1) / T64_BK;    // rounds; only the last can be ragged
    // this workgroup's: r0 .. r0 + R - 1
    const int each = SPLIT ? all / parts : all, rest = SPLIT ? all - each * parts : 0;
    const int r0 = SPLIT ? part * each + (part < rest ? part : rest) : 0, R = SPLIT ? each + (part < rest ? 1 : 0) : all;
    auto issue = [&](int r, int stage) {
        const int k0 = r * T64_BK;
        const bool tail = k0 + T64_BK > p.K;        // wave-uniform
        const unsigned sa = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_base + stage * STAGE + wave * CA * 1024));
        const unsigned sb = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_base + stage * STAGE + A_BYTES + wave * CB * 1024));
        const int4v ra = make_rsrc(CONV ? Ab : Ab + (int64_t)k0 * 2);
        const int4v rb = make_rsrc(TRANS_B ? Bb + (int64_t)k0 * 2 : Bb + (int64_t)k0 * p.ldb * 2);
#pragma unroll
        for (int q = 0; q < CA; ++q) {
            unsigned off = a_voff[q];
            if (CONV) {
                // (per lane: working the taps out once per round on the scalar unit, where Cin % 64 allows it, put a serial
                // chain in front of the loads: 39 against 33 us on 8 x 14 x 14 x 512 -> 512, 3 x 3)
                const int k = k0 + a_k[q];
                const int tap = t64_div(k, cin_magic), ch = k - tap * p.conv.Cin;
                const int kh = t64_div(tap, kw_magic), kw = tap - kh * p.conv.KW;
                const int dh = kh * p.conv.dil_h, dw = kw * p.conv.dil_w;
                const int ih = a_ih[q] + dh, iw = a_iw[q] + dw;
                const bool ok = k < p.K && ih >= 0 && ih < p.conv.H && iw >= 0 && iw < p.conv.W;
                off = ok ? off + (unsigned)(((dh * p.conv.W + dw) * p.conv.Cin + ch) * 2) : kOob;
            } else if (tail && k0 + a_k[q] >= p.K) {
                off = kOob;
            }
            dma(ra, sa + q * 1024, off);
        }
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            unsigned off = b_voff[q];
            if (tail && k0 + b_k[q] >= p.K) off = kOob;
            dma(rb, sb + q * 1024, off);
        }
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // fragment offsets inside a stage (the wave's k32 step of the round is part of them)
    const int kmaj = c * 256 + (((wave * 4 + g) ^ c) << 4);                      // row c; rows 16 i + c: + 4096 i
    const int tr_k = wave * 32 + 8 * g + (c >> 2);                               // second half of the 8 k: + 4 rows
    int b_off[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
        b_off[j] = A_BYTES + (TRANS_B ? kmaj + j * 4096 : tr_k * 128 + ((j ^ t64_row_slot(tr_k)) << 5) + (c & 3) * 8);

    for (int r = 0; r < NSTAGE - 1 && r < R; ++r) issue(r0 + r, r);
    int stage = 0, slot_in = NSTAGE - 1;
    for (int r = 0; r < R; ++r) {
        // round r has landed once only the younger rounds' loads are outstanding
        const int newer = R - 1 - r < NSTAGE - 2 ? R - 1 - r : NSTAGE - 2;
        switch (newer) {
        case 0: wait_vmcnt<0>(); break;
        case 1: wait_vmcnt<LOADS>(); break;
        default: wait_vmcnt<2 * LOADS>(); break;
        }
        static_assert(NSTAGE >= 2 && NSTAGE <= 4, "cases above");
        __syncthreads();                            // everyone's pieces landed; everyone is done with the stage refilled next
        if (r + NSTAGE - 1 < R) issue(r0 + r + NSTAGE - 1, slot_in);
        const char* s = lds + stage * STAGE;
        short8v af[FM], bf[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) af[i] = *(const short8v*)(s + kmaj + i * 4096);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            if (TRANS_B) {
                bf[j] = *(const short8v*)(s + b_off[j]);
            } else {
                short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PBK_LDS_PTR(short4v, s + b_off[j]));
                short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PBK_LDS_PTR(short4v, s + b_off[j] + 4 * 128));
                bf[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = MfmaOp16<T>::run(bf[j], af[i], acc[i][j]);
        stage = stage + 1 == NSTAGE ? 0 : stage + 1;
        slot_in = slot_in + 1 == NSTAGE ? 0 : slot_in + 1;
    }

    // ---- the waves' partial tiles meet: piece (i, j, lane) holds row 16 i + c, columns 16 j + 4 g + 0..3
    constexpr int PIECES = BM * T64_BN / 4, PPT = PIECES / (T64_NW * 64);
    const bool has_bias = epi_has_bias(end.epi), out_f32 = end.out_dtype == DT_F32;
    const int64_t c_batch = (int64_t)b * end.stride_c;
    const int osz = out_f32 ? 4 : 2;
    const bool vec = end.N % 4 == 0 && end.ldc % 4 == 0 && ((uintptr_t)end.C + (uintptr_t)c_batch * osz) % (4 * osz) == 0;
    const int col = n0 + (threadIdx.x & 15) * 4;    // the same columns in every piece of the thread
    const bool r_vec = end.R && end.N % 4 == 0 && end.ldr % 4 == 0 && ((uintptr_t)end.R + (uintptr_t)c_batch * osz) % (4 * osz) == 0;
    float bias_v[4];
    f32x4 res_v[PPT];                               // four values of the residual as they lie in memory (16-bit types: the first half)
    auto row_of = [&](int q) { return m0 + (int)(threadIdx.x >> 4) + q * 16; };
    // bias and residual of the thread's pieces.  Whole pieces, and nothing is converted here: with a conversion behind every load the
    // thread waited for each of its values in turn (577 x 1024 x 4096: 2.5 us).
    auto fetch_tail = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bias_v[e] = has_bias && col + e < end.N ? end.bias[col + e] : 0.0f;
#pragma unroll
        for (int q = 0; q < PPT; ++q) res_v[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (!end.R) return;
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int row = row_of(q);
            if (row >= end.M || col >= end.N) continue;
            const int64_t o = c_batch + (int64_t)row * end.ldr + col;
            if (r_vec && out_f32) {
                res_v[q] = *(const f32x4*)((const float*)end.R + o);
            } else if (r_vec) {
                const int2v w = *(const int2v*)((const uint16_t*)end.R + o);
                res_v[q][0] = __int_as_float(w[0]);
                res_v[q][1] = __int_as_float(w[1]);
            } else if (out_f32) {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (col + e < end.N) res_v[q][e] = ((const float*)end.R)[o + e];
            } else {
                unsigned w[2] = {0, 0};
#pragma unroll
                for (int e = 0; e < 4; ++e) if (col + e < end.N) w[e >> 1] |= (unsigned)((const uint16_t*)end.R)[o + e] << (16 * (e & 1));
                res_v[q][0] = __uint_as_float(w[0]);
                res_v[q][1] = __uint_as_float(w[1]);
            }
        }
    };
    auto res_of = [&](int q, int e) __attribute__((always_inline)) -> float {
        if (out_f32) return res_v[q][e];
        return widen<T>(__builtin_bit_cast(T, (uint16_t)(__float_as_uint(res_v[q][e >> 1]) >> (16 * (e & 1)))));
    };
    if constexpr (!SPLIT) fetch_tail();
    __syncthreads();                                // the ring is free
    f32x4* red = (f32x4*)lds;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)                // (slot XORed so that both the write and the read below spread over the banks)
            red[wave * PIECES + (i * FN + j) * 64 + g * 16 + (c ^ (j * 4 + g))] = acc[i][j];
    __syncthreads();
    const int rj = (threadIdx.x & 15) >> 2, rg = threadIdx.x & 3;
    f32x4 sum[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int at = (q * FN + rj) * 64 + rg * 16 + ((int)(threadIdx.x >> 4) ^ (rj * 4 + rg));
        sum[q] = red[at];
#pragma unroll
        for (int w = 1; w < T64_NW; ++w) sum[q] += red[w * PIECES + at];
    }
    if constexpr (SPLIT) {
        // the parts of the tile meet: part w, piece q, thread
        const int tile = b * tm.tiles_per_batch + tile_m * tm.tiles_n + tile_n;
        const __amdgpu_buffer_rsrc_t buf = scratch_buffer(scratch.data + (size_t)tile * parts * PIECES * 16);
        auto at = [&](int w, int q) { return (int)((w * PIECES + q * (T64_NW * 64) + threadIdx.x) * 16); };
#pragma unroll
        for (int q = 0; q < PPT; ++q) scratch_put(buf, at(part, q), sum[q]);
        if (!scratch_last(scratch.tickets + tile, parts, (int*)lds)) return;       // (the sums have been read by its first barrier)
        fetch_tail();
#pragma unroll
        for (int q = 0; q < PPT; ++q) sum[q] = scratch_get(buf, at(0, q));
        constexpr int AHEAD = 4;                    // parts requested together
        for (int w = 1; w < parts; w += AHEAD) {
            f32x4 v[AHEAD][PPT];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
#pragma unroll
                for (int q = 0; q < PPT; ++q) v[i][q] = scratch_get(buf, at(w + i < parts ? w + i : parts - 1, q));
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (w + i >= parts) break;
#pragma unroll
                for (int q = 0; q < PPT; ++q) sum[q] += v[i][q];
            }
        }
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const f32x4 v = sum[q];
        const int row = row_of(q);
        if (row >= end.M || col >= end.N) continue;
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = apply_epilogue(v[e], end.alpha, bias_v[e], end.epi, end.R ? end.beta : 0.0f, res_of(q, e));
        const int64_t o = c_batch + (int64_t)row * end.ldc + col;
        if (out_f32) {
            float* cp = (float*)end.C + o;
            if (vec) {
                *(f32x4*)cp = f32x4{t[0], t[1], t[2], t[3]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (col + e < end.N) cp[e] = t[e];
            }
        } else {
            uint16_t* cp = (uint16_t*)end.C + o;
            if (vec) {
                *(int2v*)cp = int2v{(int)pack2<T>(t[0], t[1]), (int)pack2<T>(t[2], t[3])};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (col + e < end.N) cp[e] = to_bits16<T>(t[e]);
            }
        }
    }
}

// parts: workgroups that share a tile's rounds, in scratch memory (1: none, no scratch memory)
template <typename T, int MODE, int BM, int NSTAGE, bool SPLIT>
hipError_t launch_tile(const Problem& p, hipStream_t stream, int parts, const ScratchUse* use) {
    constexpr int LDS_BYTES = NSTAGE * (BM + T64_BN) * T64_BK * 2;
    auto kern = gemm_mfma_tile64_kernel<T, MODE, BM, NSTAGE, SPLIT>;
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
    tm.tiles_m = (p.M + BM - 1) / BM;
    tm.tiles_n = (p.N + T64_BN - 1) / T64_BN;
    const long long total = (long long)tm.tiles_m * tm.tiles_n * p.batch * parts;
    if (total <= 0 || total > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    tm.tiles_per_batch = tm.tiles_m * tm.tiles_n;
    tm.total = (int)total;
    tm.group_m = 8;
    tm.xcds = ds.xcds;
    auto magic = [](int d) { return d > 1 ? (unsigned)(((1ull << 32) + d - 1) / d) : 0u; };
    unsigned cin_magic = p.is_conv ? magic(p.conv.Cin) : 0, kw_magic = p.is_conv ? magic(p.conv.KW) : 0;
    Problem pa = p;
    Scratch scratch = use ? use->mem() : Scratch{};
    void* args[] = {&pa, &tm, &cin_magic, &kw_magic, &parts, &scratch};
    return launch_with(use, (const void*)kern, dim3((unsigned)total), dim3(T64_NW * 64), args, LDS_BYTES, stream);
}

constexpr int kDeepK = 16;               // tile64_choice only

template <typename T, int BM, int NSTAGE, bool SPLIT = false>
hipError_t launch_mode(const Problem& p, hipStream_t stream, int parts = 1, const ScratchUse* use = nullptr) {
    if (p.is_conv) return launch_tile<T, MODE_CONV, BM, NSTAGE, SPLIT>(p, stream, parts, use);
    return p.trans_b ? launch_tile<T, MODE_TRANS_B, BM, NSTAGE, SPLIT>(p, stream, parts, use)
                     : launch_tile<T, MODE_DENSE, BM, NSTAGE, SPLIT>(p, stream, parts, use);
}

template <typename T>
hipError_t launch_type(const Problem& p, hipStream_t stream, int cfg, const char** name) {
    switch (cfg) {
    case 0: *name = "mfma16_tile64_64x64_s4"; return launch_mode<T, 64, 4>(p, stream);
    case 1: *name = "mfma16_tile64_32x64_s3"; return launch_mode<T, 32, 3>(p, stream);
    case 2: *name = "mfma16_tile64_64x64_s2"; return launch_mode<T, 64, 2>(p, stream);
    case kDeepK: *name = "mfma16_tile64_64x64_s3"; return launch_mode<T, 64, 3>(p, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// The alignment rules of the staged kernel (mfma_supported); the transposed convolution is not built.
bool mfma_tile64_supported(const Problem& p) {
    if (p.in_dtype != DT_BF16 && p.in_dtype != DT_F16) return false;
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
// workgroup hides, up to one round of 64 x 64 tiles (8 x 14 x 14 x 512 -> 512, 3 x 3: 25.6 against 33 us); then one 64 x 64
// tile per unit with a deep ring (256 x 4096 x 4096: 20.7 against 22.7 and 24.0 us; three stages are as good for short contractions and
// ahead for long ones: 577 x 1024 x 4096 20.1 against 19.3, k-major B 19.4 against 18.2, 256 x 1024 x 1024 8.6 and 8.5), beyond that two per unit
// (1024 x 2048 x 2048: 16.4 against 24.3 us).
static int tile64_choice(const Problem& p) {
    const long long t32 = (long long)((p.M + 31) / 32) * ((p.N + 63) / 64) * p.batch;
    const long long t64 = (long long)((p.M + 63) / 64) * ((p.N + 63) / 64) * p.batch;
    if (p.M <= 32 || t32 <= 256 || (p.is_conv && t64 <= 256)) return 1;
    if (t32 <= 320 && p.K < 3072) return 1;
    return t64 > 256 ? 2 : p.K >= 2048 ? kDeepK : 0;
}

// Up to half a round of 128 x 128 tiles on the 256 compute units (measured against their deep ring: 64 tiles, K = 4096: 20.7
// against 27.5 us; 128 tiles, K = 2048: 16.4 against 17.3; 160 tiles, K = 1024: 18.0 against 11.7), and enough rounds of k:
// - one for the 32 x 64 tiles (577 x 1024 x 128: 4.9 against 5.7 us);
// - two for one 64 x 64 tile per unit (256 x 4096, k-major B: K = 128 5.8 against 5.7, 192 6.25 against 6.05, 256 6.2 against 6.6);
// - four for two of them, whose short rings do not fill before (1024 x 2048: K = 128 6.4 against 6.0, 192 7.2 against 6.5, 384
//   8.0 against 7.8, 512 8.6 against 9.1; 4 x 56 x 56 x 128 -> 512, 1 x 1, stride 2: 7.9 against 7.1).
bool mfma_tile64_preferred(const Problem& p) {
    const long long t128 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128) * p.batch;
    const int c = tile64_choice(p), rounds = c == 1 ? 1 : c == 0 ? 2 : 4;
    return t128 <= 128 && p.K >= rounds * T64_BK;
}

// Workgroups that share a 32 x 64 tile (1: tiles are not split).  Up to 128 tiles, so that 192 to 256 workgroups share the work, each with at
// least four rounds.  Times in us, unsplit (ksplit up to 16 rows) first:
// - 31 x 1344 x 13312, 21 tiles: 36.3 against 12.6 with 8 parts; 48 x 1024 x 16384: 45.4 and 13.1; 18 x 2112 x 4096: 13.7 and 8.6; 256 x
//   1024 x 3968, 128 tiles: 13.9 and 11.0 with 2; 3 x 3 convolutions 196 x 512 x 4608: 21.3 and 11.3, 48 x 256 x 4608: 20.6 and 9.4;
// - the parts' meeting takes some 3 us, which short contractions do not give back: 128 x 1024 x 1024: 6.4 and 6.9, 20 x 1024 x 1024: 6.3 and
//   6.3, 376 x 576 x 1856: 8.4 and 8.2; a convolution, whose rounds take longer, 784 x 128 x 1152: 8.0 and 7.6;
// - up to 16 rows against ksplit: 8 x 1024 x 4096: 7.0 and 8.0, 14 x 1472 x 6144: 13.8 and 9.2, 16 x 4096 x 4096: 13.2 and 10.3, 8 x 1024 x
//   16384: 33.6 and 12.5, but 6 x 3456 x 2368: 6.7 and 7.9; with a row-major B of many columns its workgroups read at the rate of the memory
//   already: 1 x 4736 x 4672 10.1 and 11.4, 4 x 8192 x 4096 14.7 and 15.1 (8 x 4096 x 4096 12.0 and 10.5, 16 x 8192 x 4096 16.9 and 15.4);
// - more tiles: 1024 x 320 x 4096, 160 tiles: 14.2 and 13.8, 1024 x 480 x 4096: 14.9 and 15.8;
// - two parts only, from 77 tiles on, give back less: with operands in the caches, 256 x 1024 x 1536 7.7 and 8.7, x 1792 8.3 and 9.0, x 2304 9.6 and 9.7; from
//   memory, as the weights of a model come, 9.95 and 9.24, 11.0 and 9.7, 12.8 and 10.7; 61 x 3328 x 1536 7.6 and 8.3, from memory 10.3 and 9.3; 3 x 3
//   convolutions 8 x 14 x 14 x 128 -> 128 8.3 and 8.8, from memory 8.4 and 8.5, 6 x 14 x 14 x 160 -> 128 9.7 and 8.6.
static int tile64_parts(const Problem& p, bool forced) {
    const long long tiles = (long long)((p.M + 31) / 32) * ((p.N + 63) / 64) * p.batch;
    const int rounds = (p.K + T64_BK - 1) / T64_BK;
    if (tiles > 128) return 1;
    if (!forced && rounds < (p.is_conv ? 9 : 12)) return 1;
    if (!forced && p.M <= 16 && !p.is_conv && (p.K < 4096 || (int64_t)p.N * p.K < (p.trans_b ? 4000000 : 6000000))) return 1;
    if (!forced && p.M <= 8 && p.N > 4096 && !p.is_conv && !p.trans_b) return 1;
    int parts = (int)((192 + tiles / 2) / tiles);
    const int most = forced ? rounds : rounds / 4;
    parts = parts < 8 ? parts : 8;
    if (!forced && parts == 2 && rounds < (p.is_conv ? 11 : 14)) return 1;
    return parts < most ? parts : most;
}

bool mfma_tile64_split_preferred(const Problem& p) { return tile64_parts(p, false) > 1; }

bool launch_mfma_tile64_split(const Problem& p, hipStream_t stream, bool forced, const char** name, hipError_t* e) {
    static_assert(128 <= kScratchTickets && 256 * 32 * T64_BN * 4 <= kScratchBytes, "up to 192 + 128 / 2 parts");
    const int parts = tile64_parts(p, forced);
    int dev = 0;
    if (parts <= 1 || hipGetDevice(&dev) != hipSuccess) return false;
    const ScratchUse use(dev, stream);
    if (!use) return false;
    *name = "mfma16_tile64_32x64_s3_split";
    *e = p.in_dtype == DT_BF16 ? launch_mode<bf16_t, 32, 3, true>(p, stream, parts, &use) : launch_mode<f16_t, 32, 3, true>(p, stream, parts, &use);
    return true;
}

hipError_t launch_mfma_tile64(const Problem& p, hipStream_t stream, int cfg, const char** name) {
    const int c = cfg >= 0 && cfg <= 2 ? cfg : cfg == kSplitChoice ? 1 : tile64_choice(p);
    return p.in_dtype == DT_BF16 ? launch_type<bf16_t>(p, stream, c, name) : launch_type<f16_t>(p, stream, c, name);
}

}  // namespace pbk
