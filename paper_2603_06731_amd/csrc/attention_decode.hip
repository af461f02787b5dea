// Fused attention for a few queries against a long context (decode): up to 16 query rows per batch entry, 16-bit types.
//
// The work is reading K and V once.  With one workgroup per batch entry and one query tile, the kernel for whole
// sequences leaves most of the chip idle and walks the context in one serial chain.  Here the keys are split over
// the waves of a workgroup, 32 at a time and round-robin, each wave with a softmax of its own: no barrier inside the
// loop.  A wave fetches its K and V tiles straight into its own LDS slice (whole rows, 16 bytes per lane); the K slice is
// refilled as soon as its fragments are in registers, the V slice likewise, so that about 100 KiB are in flight per
// compute unit and its load path stays busy: that path bounds the kernel with few batch entries, memory with many.  16 entries,
// context 8192, D = 128: 122 -> 32 us; 64 entries 133 -> 61 us (4.4 TB/s).  With fewer batch entries than compute
// units, 2 or 4 workgroups share an entry: each computes all scores but multiplies only its own DV columns of V,
// and the re-read K comes out of the L2 they share.  At the end the waves' outputs are brought to one reference point and added in
// wave order in LDS.
// With up to 96 entries and a context long enough, the keys are split over workgroups as well (SPLIT): every workgroup reads its own
// keys and values only, and the parts of an entry meet in scratch memory (scratch.h).  16 entries, context 8192, D = 128, operands
// from memory: 53 -> 20 us (4 TB/s would be 17); 16 x 4096 x 64: 17.5 -> 10.3.  It then is bound by memory and by a chain of latencies:
// first loads, the waves' meeting, the parts' meeting (some 3 us).
//
// Layouts (v_mfma_f32_16x16x32: lane l supplies operand index l%16 and 8 contraction values of group l/16; it receives
// column l%16 and rows 4 (l/16) + 0..3):
//   S^T = K Q^T: a lane holds, for query l%16, keys 16 blk + 4 (l/16) + 0..3 of the two 16-key blocks;
//   O^T = V^T P^T: its own 8 weights are the B operand as they are; the transposing LDS read fetches V rows in
//   that key order.  No weight changes lane.
#include "gemm_mfma_launch.h"
#include "scratch.h"
#include <type_traits>

namespace pbk {
namespace {

constexpr int DEC_KB = 32;              // keys per step of a wave
constexpr float DEC_SLACK = 8.0f;       // log2 of how far a score may exceed the softmax reference point

// 16-byte chunk of a K row / 32-byte slot of a V row (swizzle terms, bank-conflict-free reads, period 16 keys)
template <int D> __device__ __forceinline__ int dec_kswz(int key) { return D == 128 ? key & 15 : D == 64 ? (key >> 1) & 7 : (key >> 2) & 3; }
template <int DV> __device__ __forceinline__ int dec_vswz(int key) { return DV == 128 ? key & 7 : DV == 64 ? (key >> 1) & 3 : (key >> 2) & 1; }

// SPLIT: `parts` workgroups per batch entry, each with a run of the steps of 32 keys
template <typename T, int D, int DV, int NW, bool CAUSAL, bool SPLIT>
__global__ __launch_bounds__(NW * 64, NW / 4) void attention_decode_kernel(AttnProblem p, int total, int xcds, int parts, Scratch scratch) {
    static_assert(!SPLIT || DV == D, "keys or columns are split, not both");
    const int DS = SPLIT ? parts : D / DV;         // workgroups per batch entry
    constexpr int KS = D / 32, JD = DV / 16;
    constexpr int K_BYTES = DEC_KB * D * 2, V_BYTES = DEC_KB * DV * 2, WLDS = K_BYTES + V_BYTES;
    constexpr int KL = K_BYTES / 1024, VL = V_BYTES / 1024;          // loads per step
    constexpr int KCPR = D / 8, VCPR = DV / 8;                       // 16-byte chunks per row
    constexpr float LOG2E = 1.4426950408889634f;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;

    // one XCD (one L2) owns a contiguous run of (batch entry, column group) pairs
    const int xq = total / xcds, xr = total % xcds, xcd = blockIdx.x % xcds, local = blockIdx.x / xcds;
    const int id = xcd * xq + (xcd < xr ? xcd : xr) + local;
    const int b = id / DS, part = id - b * DS, d0 = SPLIT ? 0 : part * DV;
    const int c_off = p.Nk - p.Nq;                 // causal: key visible iff key <= query + c_off

    const char* Kb = (const char*)p.K + (int64_t)b * p.stride_k * 2;
    const char* Vb = (const char*)p.V + ((int64_t)b * p.stride_v + d0) * 2;
    unsigned k_voff[KL], v_voff[VL];
    int k_row[KL], v_row[VL];
#pragma unroll
    for (int r = 0; r < KL; ++r) {
        const int row = r * (64 / KCPR) + lane / KCPR;
        k_row[r] = row;
        k_voff[r] = (unsigned)(row * (int)p.ldk * 2 + (((lane % KCPR) ^ dec_kswz<D>(row)) << 4));
    }
#pragma unroll
    for (int r = 0; r < VL; ++r) {
        const int row = r * (64 / VCPR) + lane / VCPR, slot = lane % VCPR;
        v_row[r] = row;
        v_voff[r] = (unsigned)(row * (int)p.ldv * 2 + ((((slot >> 1) ^ dec_vswz<DV>(row)) << 5) | ((slot & 1) << 4)));
    }
    char* kl = lds + wave * WLDS;
    char* vl = kl + K_BYTES;
    const unsigned k_lds = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_addr_of(kl)), v_lds = k_lds + K_BYTES;
    auto dma = [&](int4v rsrc, unsigned addr, unsigned voff) {
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(addr), "v"(voff), "s"(rsrc) : "memory", "m0");
    };
    // steps of 32 keys: this workgroup's are S0 .. S - 1, dealt round-robin to the waves
    const int all = (p.Nk + DEC_KB - 1) / DEC_KB, each = SPLIT ? all / parts : all, rest = SPLIT ? all - each * parts : 0;
    const int S0 = SPLIT ? part * each + (part < rest ? part : rest) : 0, S = SPLIT ? S0 + each + (part < rest ? 1 : 0) : all;
    auto issue_k = [&](int s) {
        const int key0 = s * DEC_KB;
        const int4v r = make_rsrc(Kb + (int64_t)key0 * p.ldk * 2);
        const bool tail = key0 + DEC_KB > p.Nk;
#pragma unroll
        for (int q = 0; q < KL; ++q) dma(r, k_lds + q * 1024, tail && key0 + k_row[q] >= p.Nk ? kOob : k_voff[q]);
    };
    auto issue_v = [&](int s) {
        const int key0 = s * DEC_KB;
        const int4v r = make_rsrc(Vb + (int64_t)key0 * p.ldv * 2);
        const bool tail = key0 + DEC_KB > p.Nk;
#pragma unroll
        for (int q = 0; q < VL; ++q) dma(r, v_lds + q * 1024, tail && key0 + v_row[q] >= p.Nk ? kOob : v_voff[q]);
    };

    short8v qf[KS];
    {
        const char* qp = (const char*)p.Q + ((int64_t)b * p.stride_q + (int64_t)c * p.ldq) * 2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qf[ks] = short8v{0, 0, 0, 0, 0, 0, 0, 0};
            if (c < p.Nq) qf[ks] = *(const short8v*)(qp + (ks * 32 + g * 8) * 2);
        }
    }
    // (the query rows are in registers before the first uncounted load is issued)
    wait_vmcnt<0>();
    if (S0 + wave < S) { issue_k(S0 + wave); issue_v(S0 + wave); }

    f32x4 o_acc[JD];
#pragma unroll
    for (int j = 0; j < JD; ++j) o_acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float c1 = p.alpha * LOG2E;              // > 0: the maximum commutes with the scaling
    float m_run = -INFINITY, neg_m = 0.0f, l_run = 0.0f;
    float thr = -INFINITY;                         // a raw score above this moves the reference point

    int koff[KS], voff[JD];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) koff[ks] = c * (D * 2) + (((ks * 4 + g) ^ dec_kswz<D>(c)) << 4);
    const int tr_key = 4 * g + (c >> 2);
#pragma unroll
    for (int j = 0; j < JD; ++j) voff[j] = tr_key * (DV * 2) + ((j ^ dec_vswz<DV>(tr_key)) << 5) + (c & 3) * 8;

    auto pair_sum = [&](int w, float acc) {        // acc + both 16-bit weights of w
        if constexpr (std::is_same<T, bf16_t>::value) {
            typedef __attribute__((ext_vector_type(2))) __bf16 b2;
            const b2 one = {(__bf16)1.0f, (__bf16)1.0f};
            return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, w), one, acc, false);
        } else {
            typedef __attribute__((ext_vector_type(2))) _Float16 h2;
            const h2 one = {(_Float16)1.0f, (_Float16)1.0f};
            return __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, w), one, acc, false);
        }
    };
    auto lds_reads_done = [&]() {                  // the slice may be overwritten after this
        __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0) only
        __builtin_amdgcn_sched_barrier(0);
    };

    for (int s = S0 + wave; s < S; s += NW) {
        const int key0 = s * DEC_KB;
        const bool more = s + NW < S;
        // ---- scores: K of this step is older than V of this step
        wait_vmcnt<VL>();
        __builtin_amdgcn_sched_barrier(0);
        short8v kf[2][KS];
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[blk][ks] = *(const short8v*)(kl + koff[ks] + blk * 16 * (D * 2));
        lds_reads_done();
        if (more) issue_k(s + NW);
        f32x4 sc[2];
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) sc[blk] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) sc[blk] = MfmaOp16<T>::run(kf[blk][ks], qf[ks], sc[blk]);
        if (key0 + DEC_KB > p.Nk || (CAUSAL && key0 + DEC_KB - 1 > c_off)) {        // wave-uniform
#pragma unroll
            for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = key0 + blk * 16 + g * 4 + e;
                    if (key >= p.Nk || (CAUSAL && key > c + c_off)) sc[blk][e] = -INFINITY;
                }
        }
        // ---- softmax.  The reference point only has to stay within 2^DEC_SLACK of the running maximum; it is moved
        // (with the sum and the output) when some lane finds a score beyond that.
        float mx = sc[0][0];
#pragma unroll
        for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sc[e >> 2][e & 3]);
        if (__builtin_amdgcn_ballot_w64(mx > thr) != 0) {
            float bmax = mx;
            bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
            bmax = fmaxf(bmax, __shfl_xor(bmax, 32)) * c1;
            const bool move = bmax > m_run + DEC_SLACK;             // the same in the four lanes of a query
            const float m_new = move ? bmax : m_run;
            const float m_sub = m_new == -INFINITY ? 0.0f : m_new;
            const float corr = __builtin_amdgcn_exp2f(m_run - m_sub);
            m_run = m_new;
            neg_m = -m_sub;
            thr = (m_new + DEC_SLACK) / c1;
            l_run *= corr;
#pragma unroll
            for (int j = 0; j < JD; ++j) o_acc[j] *= corr;
        }
        int4v pw;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[i >> 1][(i & 1) * 2], c1, neg_m));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[i >> 1][(i & 1) * 2 + 1], c1, neg_m));
            pw[i] = (int)pack2<T>(p0, p1);
            l_run = pair_sum(pw[i], l_run);
        }
        const short8v pf = __builtin_bit_cast(short8v, pw);
        // ---- weights times V: only the K tile just requested may still be in flight
        if (more) wait_vmcnt<KL>(); else wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        short8v vf[JD];
#pragma unroll
        for (int j = 0; j < JD; ++j) {
            short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PBK_LDS_PTR(short4v, vl + voff[j]));
            short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PBK_LDS_PTR(short4v, vl + voff[j] + 16 * (DV * 2)));
            vf[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        lds_reads_done();
        if (more) issue_v(s + NW);
#pragma unroll
        for (int j = 0; j < JD; ++j) o_acc[j] = MfmaOp16<T>::run(vf[j], pf, o_acc[j]);
    }

    // ---- the waves' results meet: reference points and sums [NW][16], outputs as pieces [NW][JD][64] of 4 columns
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    __syncthreads();                               // every slice has been read for the last time
    f32x4* red = (f32x4*)lds;
    constexpr int PIECES = JD * 64;
    float* m_all = (float*)(lds + NW * PIECES * 16);
    float* l_all = m_all + NW * 16;
    static_assert(NW % 8 == 0 && NW * (PIECES * 16 + 128) + 4 <= NW * WLDS, "LDS");
#pragma unroll
    for (int j = 0; j < JD; ++j) red[wave * PIECES + j * 64 + lane] = o_acc[j];
    if (g == 0) { m_all[wave * 16 + c] = m_run; l_all[wave * 16 + c] = l_run; }
    __syncthreads();
    // outputs of n parts brought to one reference point and added; `v` holds the first eight of them already, the others come from o_of
    constexpr int AHEAD = 8;
    auto combine = [&](int n, auto&& m_of, auto&& l_of, auto&& o_of, f32x4 (&v)[AHEAD], float& m, float& l, f32x4& o) __attribute__((always_inline)) {
        m = m_of(0);
        for (int w = 1; w < n; ++w) m = fmaxf(m, m_of(w));
        const float m_sub = m == -INFINITY ? 0.0f : m;
        l = 0.0f;
        o = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int w0 = 0; w0 < n; w0 += AHEAD) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (w0 + i >= n) break;
                const float f = __builtin_amdgcn_exp2f(m_of(w0 + i) - m_sub);
                l = fmaf(l_of(w0 + i), f, l);
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = fmaf(v[i][k], f, o[k]);
            }
            if (w0 + AHEAD >= n) break;
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) v[i] = o_of(w0 + AHEAD + i < n ? w0 + AHEAD + i : n - 1);
        }
    };
    auto store = [&](int q, int e, float l, f32x4 o) __attribute__((always_inline)) {
        const float inv = 1.0f / l;
        const int d = d0 + (e >> 6) * 16 + ((e & 63) >> 4) * 4;
        *(int2v*)((char*)p.O + ((int64_t)b * p.stride_o + (int64_t)q * p.ldo + d) * 2) =
            int2v{(int)pack2<T>(o[0] * inv, o[1] * inv), (int)pack2<T>(o[2] * inv, o[3] * inv)};
    };
    f32x4 v[AHEAD];
    const int e = threadIdx.x, q = e & 15;         // a piece of the output, its query
    static_assert(PIECES <= NW * 64, "one piece per thread");
    const bool mine = e < PIECES && q < p.Nq;
    float m, l;
    f32x4 o;
    if (mine) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) v[i] = red[i * PIECES + e];
        combine(NW, [&](int w) { return m_all[w * 16 + q]; }, [&](int w) { return l_all[w * 16 + q]; },
                [&](int w) { return red[w * PIECES + e]; }, v, m, l, o);
        if constexpr (!SPLIT) store(q, e, l, o);
    }
    if constexpr (SPLIT) {
        // scratch memory of a part: PIECES pieces of the output at its reference points, then reference point and sum per query
        constexpr int PART = PIECES * 4 + 64;
        const __amdgpu_buffer_rsrc_t entry = scratch_buffer(scratch.data + (size_t)b * parts * PART * 4);
        if (mine) {
            scratch_put(entry, (part * PART + e * 4) * 4, o);
            if (e < 16) scratch_put(entry, (part * PART + PIECES * 4 + q * 4) * 4, f32x4{m, l, 0.0f, 0.0f});
        }
        if (!scratch_last(scratch.tickets + b, parts, (int*)(l_all + NW * 16))) return;
        auto o_of = [&](int w) { return scratch_get(entry, (w * PART + e * 4) * 4); };
        if (mine) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) v[i] = o_of(i < parts ? i : parts - 1);
        }
        float* ml = (float*)lds;                   // (the waves' outputs have been read) reference points and sums of the parts
        for (int i = threadIdx.x; i < parts * 16; i += NW * 64) {
            if ((i & 15) >= p.Nq) continue;
            const f32x4 x = scratch_get(entry, ((i >> 4) * PART + PIECES * 4 + (i & 15) * 4) * 4);
            ml[i * 2] = x[0];
            ml[i * 2 + 1] = x[1];
        }
        __syncthreads();
        if (mine) {
            combine(parts, [&](int w) { return ml[(w * 16 + q) * 2]; }, [&](int w) { return ml[(w * 16 + q) * 2 + 1]; }, o_of, v, m, l, o);
            store(q, e, l, o);
        }
    }
}

// parts: workgroups that share an entry's keys, in scratch memory (1: none, no scratch memory)
template <typename T, int D, int DV, int NW, bool SPLIT = false>
hipError_t launch_split(const AttnProblem& p, hipStream_t stream, int parts = 1, const ScratchUse* use = nullptr) {
    constexpr int LDS_BYTES = NW * DEC_KB * (D + DV) * 2;
    const void* kern = p.causal ? (const void*)attention_decode_kernel<T, D, DV, NW, true, SPLIT>
                                : (const void*)attention_decode_kernel<T, D, DV, NW, false, SPLIT>;
    static std::atomic<unsigned> attr_done[2];     // bit per device, for either form
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned bit = 1u << (dev & 31);
    if (!(attr_done[p.causal ? 1 : 0].load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_done[p.causal ? 1 : 0].fetch_or(bit, std::memory_order_release);
    }
    DeviceShape ds;
    e = device_shape(dev, &ds);
    if (e != hipSuccess) return e;
    int xcds = ds.xcds;
    const long long n = (long long)p.batch * (SPLIT ? parts : D / DV);
    if (n <= 0 || n > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    int total = (int)n;
    AttnProblem pa = p;
    Scratch scratch = use ? use->mem() : Scratch{};
    void* args[] = {&pa, &total, &xcds, &parts, &scratch};
    return launch_with(use, kern, dim3((unsigned)total), dim3(NW * 64), args, LDS_BYTES, stream);
}

template <typename T>
hipError_t launch_type(const AttnProblem& p, hipStream_t stream, int split) {
    switch (p.D) {
    case 32: return launch_split<T, 32, 32, 16>(p, stream);
    case 64: return split >= 2 ? launch_split<T, 64, 32, 16>(p, stream) : launch_split<T, 64, 64, 16>(p, stream);
    case 128:
        if (split >= 4) return launch_split<T, 128, 32, 16>(p, stream);
        return split == 2 ? launch_split<T, 128, 64, 8>(p, stream) : launch_split<T, 128, 128, 8>(p, stream);
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_keys(const AttnProblem& p, hipStream_t stream, int parts, const ScratchUse* use) {
    switch (p.D) {
    case 32: return launch_split<T, 32, 32, 16, true>(p, stream, parts, use);
    case 64: return launch_split<T, 64, 64, 16, true>(p, stream, parts, use);
    case 128: return launch_split<T, 128, 128, 8, true>(p, stream, parts, use);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Workgroups per batch entry: K is read once by each of them, V once by all together.  With few entries a compute unit's load path
// (about 95 GB/s with 64 of them at work) bounds the kernel, and the more units take part in reading V the better (D = 128, context 8192: 16
// entries 44.4 / 34.3 / 32.2 us with 1 / 2 / 4, 64 entries 84 / 67 / 61); with 128 entries the chip is occupied and the
// second reading of K costs (240 x 1104: 25.5 / 27.9 / 42.3; 223 x 5327: 102 / 108 / 159).
static int decode_split(const AttnProblem& p) { return p.batch > 128 ? 1 : p.batch > 64 ? 2 : 4; }

// Workgroups that share an entry's keys (1: they are not split).  Up to 192 workgroups on the 256 compute units and at least 384 keys for
// each (16 entries, context 8192, D = 128, operands from memory: 33.3 us with 3 parts, 22.2 with 6, 19.4 with 10, 20.1 with 12, 21.0 with
// 16; context 2048: 13.1 with 2, 10.6 with 4, 10.1 with 6, 10.6 with 8).  The meeting costs some 3 us, which a short context
// does not give back, nor do two parts a middling one.  Unsplit first:
// - D = 128: 16 x 1024: 7.6 against 8.6, x 2048: 11.4 against 10.1; 64 x 2048: 19.0 against 17.6, 52 x 1932: 12.5 against 13.0; 96 x 2048: 22.3 against 23.0, x 4096: 41.1
//   against 40.2; 128 x 8192: 90 against 96;
// - D = 64: 16 x 2048: 8.5 against 8.7, x 4096: 17.5 against 10.3; 96 x 4096: 24.8 against 22.3; 128 x 8192: 49.5 and 49.5;
// - D = 32: 16 x 3072: 7.7 against 8.0, x 4096: 9.0 against 7.9; 96 x 4096: 15.0 against 13.4.
// Keys and values in the caches already shift the line up: near it the split then costs up to a tenth (D = 64, 64 x 2560: 10.3 against 11.5, from memory
// 15.7 against 12.8; 55 x 2867 10.8 against 11.3, from memory 16.6 against 12.6; D = 128, 64 x 2048 13.8 against 15.3, from memory 19.1 against 17.3).
static int decode_parts(const AttnProblem& p, int force) {
    if ((force > 0 && force < 8) || p.batch > 96) return 1;
    const int least = p.batch > 64 ? 4096 : p.D == 128 ? (p.batch > 32 ? 2048 : 1536) : p.D == 64 ? 2560 : 3584;
    if (force != 8 && p.Nk < least) return 1;
    const int most = force == 8 ? (p.Nk + DEC_KB - 1) / DEC_KB : p.Nk / 384;        // (chosen by hand: a step of keys is enough)
    int parts = 192 / p.batch;
    if (parts > most) parts = most;
    return parts > 64 ? 64 : parts < 1 ? 1 : parts;
}

// The operand rules of attention_mfma_supported, at most 16 queries, no bias.  A launch holds fewer than 2^32 threads, up to 1024 here
// per workgroup (more than 128 entries have one workgroup each).
bool attention_decode_supported(const AttnProblem& p) {
    return p.Nq <= 16 && !p.bias && p.alpha > 0.0f && p.batch < (1 << 22) && attention_mfma_supported(p);
}

// Against the kernel of whole sequences (bf16; times in us, that kernel's first; operands from memory, not from caches, unless noted).
// - Below four steps of keys there is nothing to split (48 x 1 x 149 x 64: 4.4 against 5.7; 16 x 8 x 130 x 32: 4.4 against 4.5).
// - Up to 128 entries: ahead everywhere (128 x 1 x 128 x 64: 4.7 against 4.2, cached).  Up to 256, one workgroup per compute unit: ahead
//   (256 x 1 x 128 x 128: 7.4 against 7.2; x 8192: 194 against 185), except that one or two queries at D = 64 cost the kernel 0.7 us that
//   three do not and a short context does not give back: 160 x 1 x 128: 5.1 against 5.6, x 192: 5.8 against 6.0, x 256: 6.4
//   against 6.3; 256 x 1 x 256: 7.5 against 7.8, x 512: 10.9 against 10.2.
// - Beyond 256 entries its 8 or 16 waves and up to 128 KiB of LDS still leave one workgroup per unit, and the other kernel keeps several: D = 64, 512 x 1 x
//   128: 7.0 against 10.1 (cached), x 512: 16.7 against 19.2, x 2048: 50 against 53; D = 128, 257 x 1 x 4096: 103 against 129,
//   448 x 2048: 85 against 86.  From 640 entries on the two take equally many rounds, and long contexts are ahead or equal (640 x
//   1024 x 128: 72 against 65; 768 x 1536 x 64: 58 and 58, 1024 x 2048 x 64: 116 against 101; but 1536 x 1024 x 64: 75 against 79).
// - At D = 32 it takes half of the LDS: ahead up to 512 entries (512 x 128: 5.0 against 4.9, cached), from 256 keys on with any number
//   (1024 x 128: 7.5 against 8.3, x 256: 10.8 against 10.0, cached).
bool attention_decode_preferred(const AttnProblem& p) {
    if (p.Nk < 4 * DEC_KB) return false;
    if (p.batch <= 128) return true;
    if (p.batch <= 256) return p.D != 64 || p.Nq > 2 || p.Nk >= (p.batch <= 192 ? 256 : 384);
    if (p.D == 32) return p.batch <= 512 || p.Nk >= 256;
    return p.batch >= 640 && p.Nk >= (p.D == 64 ? 1536 : 1024);
}

hipError_t launch_attention_decode(const AttnProblem& p, hipStream_t stream, int force_split, const char** name) {
    const int parts = decode_parts(p, force_split);
    int dev = 0;
    static_assert(96 <= kScratchTickets && 192 * (128 * 16 + 64) * 4 <= kScratchBytes, "what decode_parts asks for at most");
    if (parts > 1 && hipGetDevice(&dev) == hipSuccess) {
        if (const ScratchUse use(dev, stream); use) {
            *name = p.causal ? "attn_mfma_decode_q16_kv32_split_causal" : "attn_mfma_decode_q16_kv32_split";
            return p.dtype == DT_BF16 ? launch_keys<bf16_t>(p, stream, parts, &use) : launch_keys<f16_t>(p, stream, parts, &use);
        }
    }
    const int split = force_split > 0 && force_split < 8 ? force_split : decode_split(p);
    static const char* const names[3][2] = {{"attn_mfma_decode_q16_kv32_c1", "attn_mfma_decode_q16_kv32_c1_causal"},
                                            {"attn_mfma_decode_q16_kv32_c2", "attn_mfma_decode_q16_kv32_c2_causal"},
                                            {"attn_mfma_decode_q16_kv32_c4", "attn_mfma_decode_q16_kv32_c4_causal"}};
    const int groups = split < p.D / 32 ? split : p.D / 32;        // column groups of launch_type
    *name = names[groups >= 4 ? 2 : groups >= 2 ? 1 : 0][p.causal ? 1 : 0];
    return p.dtype == DT_BF16 ? launch_type<bf16_t>(p, stream, split) : launch_type<f16_t>(p, stream, split);
}

}  // namespace pbk
