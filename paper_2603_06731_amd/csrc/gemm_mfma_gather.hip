// Matrix-unit contraction for 16-bit operands that the direct-to-LDS kernel cannot take: K, leading
// dimensions, N (row-major B) or the channel count of a convolution that are not multiples of 8,
// or bases that are not 16-byte aligned.  The paper's own worked example is of this kind (127 input
// channels, K = 1143: Sec. 4.5, partial tiles padded with zeros on the fly).
//
// Same tiling idea as the main kernel (Sec. 4.3 / 4.5 / 4.6), with the staging done through
// registers.  A piece is eight elements that are neighbours in memory (eight k of a row of a k-major
// operand, eight n of a k-row of a row-major B); every piece is ONE 16-byte load from an address that is
// only 2-byte aligned, issued unconditionally (so that the loads of three k-tiles can be in flight at
// any time: the compiler counts them).  What a piece must not contain is removed afterwards, in
// registers, when it is moved to LDS: elements beyond the end of K or of a filter tap are cleared,
// pieces that lie in the padding, beyond K or beyond M / N are cleared entirely; a piece whose 16 bytes
// would run over the end of the operand is read from 16 bytes before that end and shifted down.
// A convolution runs over a K axis in which every filter tap is rounded up to a multiple of eight
// channels (k' = tap * ceil8(Cin) + c), so that a piece never spans two taps; the weight rows of the
// padding channels are cleared like the image's.
// Pieces go to LDS in the main kernel's layouts: k-major [rows][32 k] with the 16-byte chunk index
// XOR-swizzled by the row (A, the image, a k-major B), n-major [32 k][128 n] read with the transposing
// LDS read (row-major B, weights).
// 128 or 64 rows x 128 columns, k-tiles of 32 or, in the deep form, of 64 (the rules are gather_form and gather_parts), v_mfma_f32_16x16x32, LDS double-buffered: while
// k-tile t is multiplied, the pieces of k-tiles t+1 .. t+3 are in flight to registers; one barrier per k-tile.
// The epilogue is the main kernel's (registers, then the LDS shuffle or direct stores).
#include "gemm_mfma_launch.h"
#include "scratch.h"

namespace pbk {
namespace {

constexpr int GBN = 128, GWN = 2;                    // GBM: 128 or 64, a parameter of the kernel

// 16 bytes from an address that is only known to be 2-byte aligned (one global_load_dwordx4)
// (the pointer is stated to be a global-memory one: a generic load would also count as an LDS operation)
__device__ __forceinline__ int4v ld_vec16(const char* ptr) {
    typedef const __attribute__((address_space(1))) char* global_ptr;
    int4v w;
    __builtin_memcpy(&w, (global_ptr)ptr, 16);
    return w;
}

// sixteen zero bytes in device memory: what a piece in the padding of an image, or a weight row of a padding
// channel, is read from (the load stays unconditional and the piece needs no clearing afterwards)
__device__ const int4v kZeroPiece = {0, 0, 0, 0};

// Where a piece is read from and what is kept of it: `meta` = number of leading elements to keep (0 .. 8)
// + 16 * number of elements to drop at the front first (the piece was read from that many elements
// before its place because 16 bytes from its place would have run over the end of the operand).
// kPlain = keep everything.
constexpr int kPlain = 8;
constexpr int kAllPlain = kPlain * 0x01010101;       // one byte per piece, up to four
struct PieceSrc { const char* ptr; int meta; };

// want: address of the piece's first element (anything at or above the operand's base when !ok);
// last16: the last address of the operand from which 16 bytes can be read
__device__ __forceinline__ PieceSrc piece_src(const char* want, const char* last16, bool ok, int cnt) {
    PieceSrc s;
    s.ptr = want <= last16 ? want : last16;
    const int shift = (int)((want - s.ptr) >> 1);
    // a piece with at least one element inside the operand starts at most 14 bytes after last16
    s.meta = (ok && cnt > 0 && shift < 8) ? (cnt | (shift << 4)) : 0;
    return s;
}

__device__ __forceinline__ int4v piece_fix(int4v v, int meta) {
    const int cnt = meta & 15, shift = meta >> 4;
    unsigned w0 = (unsigned)v[0], w1 = (unsigned)v[1], w2 = (unsigned)v[2], w3 = (unsigned)v[3];
    if (shift) {
        if (shift & 4) { w0 = w2; w1 = w3; w2 = 0; w3 = 0; }
        if (shift & 2) { w0 = w1; w1 = w2; w2 = w3; w3 = 0; }
        if (shift & 1) {
            w0 = (w0 >> 16) | (w1 << 16); w1 = (w1 >> 16) | (w2 << 16);
            w2 = (w2 >> 16) | (w3 << 16); w3 >>= 16;
        }
    }
    auto keep = [&](unsigned w, int q) -> int {
        return (int)(cnt >= 2 * q + 2 ? w : cnt == 2 * q + 1 ? (w & 0xFFFFu) : 0u);
    };
    return int4v{keep(w0, 0), keep(w1, 1), keep(w2, 2), keep(w3, 3)};
}

// The same for a piece of a row of taps (ROWS): bits 4 .. 7 are the elements to drop at the front or, negative, to move up by (two's complement); zeros
// come in at the other end.
__device__ __forceinline__ int4v piece_fix_signed(int4v v, int meta) {
    const int cnt = meta & 15, drop = (int)((unsigned)meta << 24) >> 28;
    unsigned w0 = (unsigned)v[0], w1 = (unsigned)v[1], w2 = (unsigned)v[2], w3 = (unsigned)v[3];
    if (drop > 0) {
        if (drop & 4) { w0 = w2; w1 = w3; w2 = 0; w3 = 0; }
        if (drop & 2) { w0 = w1; w1 = w2; w2 = w3; w3 = 0; }
        if (drop & 1) {
            w0 = (w0 >> 16) | (w1 << 16); w1 = (w1 >> 16) | (w2 << 16);
            w2 = (w2 >> 16) | (w3 << 16); w3 >>= 16;
        }
    } else if (drop < 0) {
        const int up = -drop;
        if (up & 4) { w3 = w1; w2 = w0; w1 = 0; w0 = 0; }
        if (up & 2) { w3 = w2; w2 = w1; w1 = w0; w0 = 0; }
        if (up & 1) {
            w3 = (w3 << 16) | (w2 >> 16); w2 = (w2 << 16) | (w1 >> 16);
            w1 = (w1 << 16) | (w0 >> 16); w0 <<= 16;
        }
    }
    auto keep = [&](unsigned w, int q) -> int {
        return (int)(cnt >= 2 * q + 2 ? w : cnt == 2 * q + 1 ? (w & 0xFFFFu) : 0u);
    };
    return int4v{keep(w0, 0), keep(w1, 1), keep(w2, 2), keep(w3, 3)};
}

// FAST (convolutions whose image tensor and weights are below 2 GiB each; the others work out 64-bit addresses for every piece): the k-tiles before the careful ones are fetched with 32-bit
// offsets that only ever grow by constants from one k-tile to the next; what must not be read has the out-of-range offset, for
// which a buffer load gives zeros.  (With a tap worked out by multiplication, 64-bit addresses and the tests of a piece joined by && for
// every piece of every k-tile, the address code took longer than the loads: 8 x 44 x 44 x 127 -> 512, 3 x 3, stride 2: 25.4 against 24.0 us.)
// DEEP: eight waves and k-tiles of 64 instead of four and 32, for a workgroup that is alone on its compute unit: a k-tile of 32 takes one wave per
// SIMD some 0.5 us, most of it issuing instructions and waiting for LDS and the barrier in turn; two waves per SIMD take little longer for 64
// (8 x 44 x 44 x 127 -> 512, 3 x 3, stride 2, 224 tiles: 24.0 against 18.6 us; 1 x 68 x 68 x 127 -> 64, 7 x 7: 103 against 68).
// SPLIT: `parts` workgroups per tile, each with a run of the k-tiles.
// ROWS (a FAST convolution with no distance between the taps of a row): the taps of a row of the filter are neighbours in the image's row as well as in the
// weights, so the row is one tap of KW Cin channels, and the K axis is KH ceil8(KW Cin) long instead of KH KW ceil8(Cin) (3 channels, 7 x 7: 168 instead
// of 392).  A piece is read from inside its row of the image, which it may leave on either side, and moved to its place in registers.
template <typename T, int MODE, int GBM, bool FAST, bool DEEP, bool SPLIT, bool ROWS = false>
__global__ __launch_bounds__(DEEP ? 512 : 256, 2) void gemm_mfma_gather_kernel(Problem p, TileMapOf<MODE> tmap, int parts, Scratch scratch) {
    constexpr int GBK = DEEP ? 64 : 32, GWM = DEEP ? 4 : 2;
    constexpr bool CONV = MODE == MODE_CONV;
    static_assert(CONV || !FAST, "plain matrices advance by pointers");
    static_assert(FAST || !ROWS, "rows of taps are built on the offsets of FAST");
    constexpr bool TRANS_B = MODE == MODE_TRANS_B;
    constexpr int NT = GWM * GWN * 64;
    constexpr int WTM = GBM / GWM, WTN = GBN / GWN;
    constexpr int FM = WTM / 16, FN = WTN / 16;
    constexpr int A_TILE = GBM * GBK * 2, G_STAGE = A_TILE + GBN * GBK * 2;      // bytes
    // 16-byte pieces of the two tiles per thread (1 or 2, and 2)
    constexpr int PA = GBM * (GBK / 8) / NT, PB = GBN * (GBK / 8) / NT;
    static_assert(PA * NT == GBM * (GBK / 8) && PB * NT == GBN * (GBK / 8) && PA + PB <= 4, "tile geometry");

    extern __shared__ __attribute__((aligned(1024))) char lds[];        // 2 x (A tile | B tile)
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / GWN, wn = wave % GWN;

    int b, tile_m, tile_n;
    map_tile(tmap, blockIdx.x, b, tile_m, tile_n);
    // (split: the map's batches are the parts)
    const int part = SPLIT ? b / p.batch : 0;
    if (SPLIT) b -= part * p.batch;
    const int m0 = tile_m * GBM, n0 = tile_n * GBN;
    const char* Abase = (const char*)p.A + (int64_t)b * p.stride_a * 2;
    const char* Bbase = (const char*)p.B + (int64_t)b * p.stride_b * 2;
    // the K axis the loop runs over: a convolution's taps rounded up to whole pieces
    const int Ct = CONV ? (ROWS ? p.conv.KW * p.conv.Cin : p.conv.Cin) : 0, Cp = (Ct + 7) & ~7;       // values of a tap, rounded up to pieces
    const int KWt = ROWS ? 1 : p.conv.KW;          // taps of a row
    const int taps = CONV ? p.conv.KH * KWt : 0;
    const int Kloop = CONV ? taps * Cp : p.K;
    // this workgroup's k-tiles: kt0 .. kt1 - 1
    const int KT = (Kloop + GBK - 1) / GBK;
    const int each = SPLIT ? KT / parts : KT, rest = SPLIT ? KT - each * parts : 0;
    const int kt0 = SPLIT ? part * each + (part < rest ? part : rest) : 0, kt1 = SPLIT ? kt0 + each + (part < rest ? 1 : 0) : KT;
    // the last addresses from which 16 bytes can be read (each operand holds at least 8 elements)
    const int64_t a_elems = CONV ? (int64_t)(p.M / (p.conv.OH * p.conv.OW)) * p.conv.H * p.conv.W * p.conv.Cin
                                 : (int64_t)(p.M - 1) * p.lda + p.K;
    const int64_t b_elems = TRANS_B ? (int64_t)(p.N - 1) * p.ldb + p.K : (int64_t)(p.K - 1) * p.ldb + p.N;
    const char* a_last16 = Abase + a_elems * 2 - 16;
    const char* b_last16 = Bbase + b_elems * 2 - 16;

    // ---- A (k-major source): piece = (row, chunk of 8 k); CPR neighbouring threads cover a row of the k-tile.
    // The thread's pieces differ in the row only (+ NT / CPR).
    constexpr int CPR = GBK / 8, NPR = GBN / 8;       // pieces per row of a k-major tile, per k-row of an n-major one
    const int a_chunk = t % CPR;
    int a_row[PA];
    bool a_ok[PA];
    const char* a_cur[PA];       // dense: address of the piece in the next k-tile to fetch; conv: the pixel's image
    int a_ih0[PA], a_iw0[PA];
    unsigned a_off[FAST ? PA : 1];
    int a_first[FAST ? PA : 1];
    // conv: (channel, tap) of the thread's pieces in the next k-tile to fetch
    int a_c = 0, a_tap = 0;
    if (CONV) {
        const int k = kt0 * GBK + a_chunk * 8;        // the pieces' place on the padded K axis in the first k-tile
        a_tap = k / Cp;
        a_c = k - a_tap * Cp;
    }
    // FAST: the same place as offsets (of A's pieces from the row's first tap; of B's k-row from row 0) and as tap coordinates
    const int row_step = FAST ? (p.conv.dil_h * p.conv.W) * p.conv.Cin * 2 : 0, col_step = FAST ? p.conv.dil_w * p.conv.Cin * 2 : 0;
    int f_kw = 0, f_dh = 0, f_dw = 0;
    unsigned f_delta = 0;
    if constexpr (FAST) {
        const int kh = a_tap / KWt;
        f_kw = a_tap - kh * KWt;
        f_dh = kh * p.conv.dil_h;
        f_dw = f_kw * p.conv.dil_w;
        f_delta = (unsigned)(kh * row_step + f_kw * col_step + (ROWS ? 0 : a_c * 2));
    }
    auto next_tap = [&]() __attribute__((always_inline)) {         // one tap on, its first channel where the place was
        if constexpr (ROWS) {
            f_dh += p.conv.dil_h;
            f_delta += (unsigned)row_step;
            return;
        }
        const bool wrap = ++f_kw == KWt;
        f_kw = wrap ? 0 : f_kw;
        f_dw = wrap ? 0 : f_dw + p.conv.dil_w;
        f_dh += wrap ? p.conv.dil_h : 0;
        f_delta += wrap ? (unsigned)(row_step - (KWt - 1) * col_step) : (unsigned)col_step;
    };
    // one k-tile further on the padded K axis: adv_tap taps and adv_c channels, with at most one carry
    const int adv_tap = CONV ? GBK / Cp : 0, adv_c = CONV ? GBK - adv_tap * Cp : 0;
    // tap / KW by multiplication (exact for tap < 2^20 / KW)
    const unsigned kw_magic = CONV ? (1u << 20) / (unsigned)p.conv.KW + 1u : 0u;
    const char* zero_piece = (const char*)&kZeroPiece;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
        a_row[i] = t / CPR + (NT / CPR) * i;
        const int gm = m0 + a_row[i];
        a_ok[i] = gm < p.M;
        const int gmc = a_ok[i] ? gm : p.M - 1;       // rows beyond M read a row that exists
        if (CONV) {
            if constexpr (CONV) {
                int rem, ow;
                const int n = tmap.pix.div(gmc, rem), oh = tmap.ow.div(rem, ow);
                a_ih0[i] = oh * p.conv.stride_h - p.conv.pad_h;
                a_iw0[i] = ow * p.conv.stride_w - p.conv.pad_w;
                a_cur[i] = Abase + (int64_t)n * p.conv.H * p.conv.W * p.conv.Cin * 2;
                if constexpr (FAST) {
                    // (modulo 2^32: the row's first tap may lie in front of the image)
                    a_off[i] = (unsigned)(((n * p.conv.H + a_ih0[i]) * p.conv.W + (ROWS ? 0 : a_iw0[i])) * p.conv.Cin * 2);
                    a_first[i] = a_ok[i] ? a_ih0[i] : -(1 << 30);      // a row beyond M meets no tap
                }
            }
        } else {
            a_cur[i] = Abase + ((int64_t)gmc * p.lda + (int64_t)kt0 * GBK + a_chunk * 8) * 2;
        }
    }
    // ---- B: k-major source (trans_b): pieces like A's.  n-major source (row-major B, the weights of a
    // convolution): a piece is eight neighbouring n of one k-row: b_row = k-row in the tile, b_chunk = which
    // eight n; the thread's pieces differ in the k-row only (+ NT / NPR).
    const int b_chunk = TRANS_B ? t % CPR : t % NPR;
    int b_row[PB];
    bool b_ok[PB];
    const char* b_cur[PB];       // address of the piece in the next k-tile to fetch (conv: of its first n in row 0)
    int b_c[PB], b_tap[PB];  // conv: (channel, tap) of the piece's k-row in the next k-tile to fetch
    unsigned b_off[FAST ? PB : 1];
    const unsigned b_adv = FAST ? (unsigned)((adv_tap * Ct + adv_c) * (int)p.ldb * 2) : 0u;        // one k-tile on
    const unsigned b_carry = FAST ? (unsigned)((Cp - Ct) * (int)p.ldb * 2) : 0u;                  // less for every tap begun
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        if (TRANS_B) {
            b_row[i] = t / CPR + (NT / CPR) * i;
            b_ok[i] = n0 + b_row[i] < p.N;
            b_cur[i] = Bbase + ((int64_t)(b_ok[i] ? n0 + b_row[i] : p.N - 1) * p.ldb + (int64_t)kt0 * GBK + b_chunk * 8) * 2;
        } else {
            b_row[i] = t / NPR + (NT / NPR) * i;
            b_ok[i] = n0 + b_chunk * 8 < p.N;
            // (a piece beyond N reads column N - 1 onwards: it stays inside B wherever the careful path is not taken)
            b_cur[i] = Bbase + (int64_t)(b_ok[i] ? n0 + b_chunk * 8 : p.N - 1) * 2;
            if constexpr (CONV) {        // (b_cur stays in row 0: the padded K axis gives the row)
                b_tap[i] = (kt0 * GBK + b_row[i]) / Cp;
                b_c[i] = kt0 * GBK + b_row[i] - b_tap[i] * Cp;
                if constexpr (FAST)
                    b_off[i] = (unsigned)((b_tap[i] * Ct + b_c[i]) * (int)p.ldb * 2) + (unsigned)((b_ok[i] ? n0 + b_chunk * 8 : p.N - 1) * 2);
            } else {
                b_cur[i] += ((int64_t)kt0 * GBK + b_row[i]) * p.ldb * 2;
            }
        }
    }
    const int64_t b_step = TRANS_B ? GBK * 2 : (int64_t)GBK * p.ldb * 2;     // dense: B's advance per k-tile

    // k-tiles from kt_careful on are fetched by the careful path (it keeps every load inside its operand and
    // works out what to keep of each piece); before it no piece can run over the end of an operand:
    //  - dense: every piece of a k-tile before the last lies inside its row (k-major) or in a k-row that has
    //    a successor (n-major; the over-read of a piece that straddles N needs ldb >= 8 to stay in it);
    //  - conv: the same for the weights; the piece at the end of a tap of an image whose channel count is not a
    //    multiple of 8 is read as the tap's LAST eight channels and shifted down afterwards, so it never
    //    leaves its pixel (needs Cin >= 8).
    int kt_careful = KT - 1;
    if (!TRANS_B && p.ldb < 8) kt_careful = 0;
    if (CONV && Ct < 8) kt_careful = 0;

    // the pieces of NPF k-tiles are in flight to registers at any time: a workgroup is often alone on its
    // compute unit (these are the odd, small problems), so the memory latency is covered by depth
    constexpr int NPF = 3;
    int4v avs[NPF][PA], bvs[NPF][PB];
    int metas[NPF];                  // one byte per piece: A's, then B's

    // the k-tiles before the careful ones
    const __amdgpu_buffer_rsrc_t a_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Abase, 0, (int)kOob, 0x00020000);
    const __amdgpu_buffer_rsrc_t b_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Bbase, 0, (int)kOob, 0x00020000);
    // the thread's pieces of A on the padded K axis one k-tile on
    auto advance_fast = [&]() __attribute__((always_inline)) {
        a_c += adv_c;
        if (!ROWS) f_delta += 2 * adv_c;
        for (int n = 0; n < adv_tap; ++n) next_tap();                      // (channel counts below the depth of a k-tile)
        a_tap += adv_tap;
        const bool carry = a_c >= Cp;
        if (carry) {
            a_c -= Cp; ++a_tap;
            if (!ROWS) f_delta -= 2 * (unsigned)Cp;
            next_tap();
        }
    };
    // ROWS: the pieces of A of one k-tile, careful or not: a piece never leaves its row of the image.  Returns the bytes of `metas`.
    // place: of the piece's first value in the image's row, which the row may not hold; from: where its eight values are read.  What the piece has beyond
    // the row is zero after the move, what it has beyond the tap is dropped.
    auto gather_rows = [&](auto set_tag, bool beyond) __attribute__((always_inline)) -> int {
        int meta = 0;
        if constexpr (ROWS) {
            constexpr int S = decltype(set_tag)::value;
            const int row = p.conv.W * p.conv.Cin, cnt = Ct - a_c < 8 ? Ct - a_c : 8;
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                const int place = a_iw0[i] * p.conv.Cin + a_c;
                int from = place < row - 8 ? place : row - 8;
                from = from > 0 ? from : 0;
                const int drop = place - from;
                const bool ok = ((unsigned)(a_first[i] + f_dh) < (unsigned)p.conv.H) & (drop > -8) & (drop < 8) & !beyond;
                avs[S][i] = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(a_buf, ok ? (int)(a_off[i] + f_delta + 2 * (unsigned)from) : (int)kOob, 0, 0));
                meta |= (ok ? cnt | ((drop & 15) << 4) : kPlain) << (8 * i);
            }
            advance_fast();
        }
        return meta;
    };
    // the pieces of the weights.  CAREFUL (with ROWS): those that would run over the operand's end are read before it, and marked
    auto weights_fast = [&](auto set_tag, auto careful_tag) __attribute__((always_inline)) -> int {
        constexpr int S = decltype(set_tag)::value;
        constexpr bool CAREFUL = decltype(careful_tag)::value;
        int meta = 0;
        if constexpr (FAST) {
            const unsigned last = CAREFUL ? (unsigned)(b_elems * 2 - 16) : 0u;
#pragma unroll
            for (int i = 0; i < PB; ++i) {
                bool ok = b_c[i] < Ct;                                        // a weight row that exists
                unsigned off = b_off[i];
                int kept = kPlain;
                if (CAREFUL) {
                    ok = ok & (b_tap[i] < taps);
                    const unsigned from = off < last ? off : last, drop = (off - from) >> 1;
                    ok = ok & (drop < 8);
                    kept = ok ? kPlain | (int)(drop << 4) : kPlain;
                    off = from;
                }
                bvs[S][i] = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(b_buf, ok ? (int)off : (int)kOob, 0, 0));
                meta |= kept << (8 * (PA + i));
                b_c[i] += adv_c; b_tap[i] += adv_tap; b_off[i] += b_adv;
                const bool c = b_c[i] >= Cp;
                b_c[i] -= c ? Cp : 0; b_tap[i] += c ? 1 : 0; b_off[i] -= c ? b_carry : 0u;
            }
        }
        return meta;
    };
    auto gather_fast = [&](auto set_tag) __attribute__((always_inline)) {
        if constexpr (FAST) {
            constexpr int S = decltype(set_tag)::value;
            int meta = 0;
            if constexpr (ROWS) {
                meta |= gather_rows(set_tag, false);
            } else {
            // the piece at the end of a tap is read Cp - Cin channels earlier and marked to be shifted down by as many
            const int left = p.conv.Cin - a_c, back = left < 8 ? Cp - p.conv.Cin : 0;
            const unsigned at = f_delta - 2 * (unsigned)back;
            const int marked = 8 | (back << 4);
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                const bool ok = ((unsigned)(a_first[i] + f_dh) < (unsigned)p.conv.H) & ((unsigned)(a_iw0[i] + f_dw) < (unsigned)p.conv.W);
                avs[S][i] = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(a_buf, ok ? (int)(a_off[i] + at) : (int)kOob, 0, 0));
                meta |= (ok ? marked : kPlain) << (8 * i);
            }
            advance_fast();
            }
            meta |= weights_fast(set_tag, BoolTag<false>{});
            metas[S] = meta;
        }
    };
    // fetch the pieces of k-tile kt into register set S (loads are issued here and waited for at the first
    // use); called for kt = 0, 1, 2, ... in order, also for up to NPF k-tiles beyond the last (those pieces
    // are cleared).  No load sits under a branch.
    auto gather = [&](int kt, auto set_tag, auto careful_tag) __attribute__((always_inline)) {
        constexpr int S = decltype(set_tag)::value;
        constexpr bool CAREFUL = decltype(careful_tag)::value != 0;
        if constexpr (FAST && !CAREFUL) { gather_fast(set_tag); return; }
        if constexpr (ROWS) { metas[S] = gather_rows(set_tag, a_tap >= taps) | weights_fast(set_tag, BoolTag<true>{}); return; }
        const int k0 = kt * GBK;
        int meta = 0;
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const char* want;
            bool ok = true;
            int cnt = 8;
            if (CONV) {
                const int kh = (int)(((unsigned)a_tap * kw_magic) >> 20), kw = a_tap - kh * p.conv.KW;
                const int ih = a_ih0[i] + kh * p.conv.dil_h, iw = a_iw0[i] + kw * p.conv.dil_w;
                ok = a_ok[i] && a_tap < taps && (unsigned)ih < (unsigned)p.conv.H && (unsigned)iw < (unsigned)p.conv.W;
                want = a_cur[i] + (unsigned)(((ih * p.conv.W + iw) * p.conv.Cin + a_c) * 2);
                cnt = min(8, p.conv.Cin - a_c);
                if (!CAREFUL) {
                    // a piece in the padding is read from the zero piece and kept whole; a piece at the end of a
                    // tap is read Cp - Cin channels earlier and marked to be shifted down by as many
                    const int back = cnt < 8 ? Cp - p.conv.Cin : 0;
                    want = ok ? want - 2 * back : zero_piece;
                    cnt = ok ? (8 | (back << 4)) : 8;
                    ok = true;
                } else if (!ok) {
                    want = a_cur[i];
                }
            } else {
                want = a_cur[i];
                a_cur[i] += GBK * 2;
                if (CAREFUL) { ok = a_ok[i]; cnt = min(max(p.K - (k0 + a_chunk * 8), 0), 8); }
            }
            PieceSrc s;
            if (CAREFUL) s = piece_src(want, a_last16, ok, cnt);
            else { s.ptr = want; s.meta = ok ? cnt : 0; }
            avs[S][i] = ld_vec16(s.ptr);
            meta |= s.meta << (8 * i);
        }
        if (CONV) {                                   // advance the pieces' place by one k-tile
            a_c += adv_c; a_tap += adv_tap;
            if (a_c >= Cp) { a_c -= Cp; ++a_tap; }
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const char* want;
            bool ok = true;
            int cnt = 8;
            if (CONV) {
                ok = b_tap[i] < taps && b_c[i] < p.conv.Cin;      // a weight row that exists
                const int row = ok ? b_tap[i] * p.conv.Cin + b_c[i] : 0;
                want = b_cur[i] + (int64_t)row * p.ldb * 2;
                if (!CAREFUL) { want = ok ? want : zero_piece; ok = true; }
                else ok = ok && b_ok[i];
                int c = b_c[i] + adv_c, tap = b_tap[i] + adv_tap;
                if (c >= Cp) { c -= Cp; ++tap; }
                b_c[i] = c; b_tap[i] = tap;
            } else {
                want = b_cur[i];
                b_cur[i] += b_step;
                if (CAREFUL) {
                    ok = b_ok[i];
                    if (TRANS_B) cnt = min(max(p.K - (k0 + b_chunk * 8), 0), 8);
                    else ok = ok && k0 + b_row[i] < p.K;
                }
            }
            PieceSrc s;
            if (CAREFUL) s = piece_src(want, b_last16, ok, cnt);
            else { s.ptr = want; s.meta = ok ? cnt : 0; }
            bvs[S][i] = ld_vec16(s.ptr);
            meta |= s.meta << (8 * (PA + i));
        }
        metas[S] = meta;
    };
    // (careful: the pieces may come from the careful path)
    auto stash = [&](int stage, auto set_tag, auto careful_tag) __attribute__((always_inline)) {
        constexpr int S = decltype(set_tag)::value;
        constexpr bool CAREFUL = decltype(careful_tag)::value != 0;
        char* sa = lds + stage * G_STAGE;
        char* sb = sa + A_TILE;
        int4v va[PA], vb[PB];
#pragma unroll
        for (int i = 0; i < PA; ++i) va[i] = avs[S][i];
#pragma unroll
        for (int i = 0; i < PB; ++i) vb[i] = bvs[S][i];
        if (metas[S] != (int)((unsigned)kAllPlain >> (8 * (4 - PA - PB)))) {         // rare: one branch for the thread's pieces
#pragma unroll
            for (int i = 0; i < PA; ++i) va[i] = ROWS ? piece_fix_signed(va[i], (metas[S] >> (8 * i)) & 255) : piece_fix(va[i], (metas[S] >> (8 * i)) & 255);
            if constexpr (CAREFUL || !FAST) {
#pragma unroll
                for (int i = 0; i < PB; ++i) vb[i] = piece_fix(vb[i], (metas[S] >> (8 * (PA + i))) & 255);
            }
        }
#pragma unroll
        for (int i = 0; i < PA; ++i) *(int4v*)(sa + kmajor_offset<GBK, true>(a_row[i], a_chunk)) = va[i];
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            if (TRANS_B) *(int4v*)(sb + kmajor_offset<GBK, true>(b_row[i], b_chunk)) = vb[i];
            else *(int4v*)(sb + nmajor_offset<GBN>(b_row[i], b_chunk * 16)) = vb[i];
        }
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;

    constexpr int KS = GBK / 32;                      // MFMA k-steps per k-tile
    const int f_row = lane & 15, f_kc = lane >> 4;
    // transposing read of the n-major B tile: 16-lane block q covers k rows 8q .. 8q+3 (second read: +4);
    // lane -> row (lane % 16) / 4, n piece lane % 4
    const int t16_k = ((lane & 15) >> 2) + ((lane >> 4) << 3);
    const int t16_nbyte = (lane & 3) * 8;
    // k-tile kt (its pieces were gathered into set S): multiply it from LDS stage kt % 2, move k-tile kt+1
    // (set S+1) into the other stage, which was last read before the previous barrier, and start fetching
    // k-tile kt+3 into set S, which has just been emptied
    auto step = [&](int kt, auto set_tag, auto careful_tag) __attribute__((always_inline)) {
        constexpr int S = decltype(set_tag)::value;
        const char* sa = lds + (kt & 1) * G_STAGE;
        const char* sb = sa + A_TILE;
        short8v af[KS][FM], bf[KS][FN];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
                af[ks][i] = *(const short8v*)(sa + kmajor_offset<GBK, true>(wm * WTM + i * 16 + f_row, ks * 4 + f_kc));
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (TRANS_B) {
                    bf[ks][j] = *(const short8v*)(sb + kmajor_offset<GBK, true>(wn * WTN + j * 16 + f_row, ks * 4 + f_kc));
                } else {
                    const char* r0 = sb + nmajor_offset<GBN>(t16_k, (wn * WTN + j * 16) * 2 + t16_nbyte) + ks * 32 * (GBN * 2);
                    short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PBK_LDS_PTR(short4v, r0));
                    short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PBK_LDS_PTR(short4v, r0 + 4 * (GBN * 2)));
                    bf[ks][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            }
        }
        gather(kt + NPF, set_tag, careful_tag);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = MfmaOp16<T>::run(bf[ks][j], af[ks][i], acc[i][j]);
        stash((kt + 1) & 1, IntTag<(S + 1) % NPF>{}, careful_tag);
        __syncthreads();
    };
    int kt = kt0;
    if (kt0 + NPF <= kt_careful) {
        gather(kt0, IntTag<0>{}, IntTag<0>{});
        gather(kt0 + 1, IntTag<1>{}, IntTag<0>{});
        gather(kt0 + 2, IntTag<2>{}, IntTag<0>{});
    } else {
        gather(kt0, IntTag<0>{}, IntTag<1>{});
        gather(kt0 + 1, IntTag<1>{}, IntTag<1>{});
        gather(kt0 + 2, IntTag<2>{}, IntTag<1>{});
        kt_careful = 0;
    }
    stash(kt0 & 1, IntTag<0>{}, IntTag<1>{});
    __syncthreads();
    // steps whose fetches (k-tiles kt + 3 .. kt + 5) all come before the careful ones
    for (; kt + 2 * NPF - 1 < kt_careful && kt + NPF <= kt1; kt += NPF) {
        step(kt, IntTag<0>{}, IntTag<0>{});
        step(kt + 1, IntTag<1>{}, IntTag<0>{});
        step(kt + 2, IntTag<2>{}, IntTag<0>{});
    }
    for (; kt < kt1; kt += NPF) {
        step(kt, IntTag<0>{}, IntTag<1>{});
        if (kt + 1 >= kt1) break;
        step(kt + 1, IntTag<1>{}, IntTag<1>{});
        if (kt + 2 >= kt1) break;
        step(kt + 2, IntTag<2>{}, IntTag<1>{});
    }
    if constexpr (SPLIT) {
        // the parts of the tile meet: part w, block, thread.  A wave without rows of C has nothing to bring.
        const int tile = b * tmap.tiles_per_batch + tile_m * tmap.tiles_n + tile_n;
        const __amdgpu_buffer_rsrc_t buf = scratch_buffer(scratch.data + (size_t)tile * parts * (GBM * GBN * 4));
        const bool live = m0 + wm * WTM < p.M;
        auto at = [&](int w, int i, int j) { return w * (GBM * GBN * 4) + ((i * FN + j) * NT + t) * 16; };
        if (live) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) scratch_put(buf, at(part, i, j), acc[i][j]);
        }
        if (!scratch_last(scratch.tickets + tile, parts, (int*)lds)) return;
        if (live) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = scratch_get(buf, at(0, i, j));
            constexpr int AHEAD = 4;                // parts requested together
            for (int w = 1; w < parts; w += AHEAD) {
                f32x4 v[AHEAD][FM][FN];
#pragma unroll
                for (int u = 0; u < AHEAD; ++u)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j) v[u][i][j] = scratch_get(buf, at(w + u < parts ? w + u : parts - 1, i, j));
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    if (w + u >= parts) break;
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j) acc[i][j] += v[u][i][j];
                }
            }
        }
        __syncthreads();                            // (the flag's word is free for the epilogue)
    }

    const int act = (p.epi == EPI_RELU || p.epi == EPI_BIAS_RELU) ? 1
                  : (p.epi == EPI_GELU_TANH || p.epi == EPI_BIAS_GELU_TANH) ? 2 : 0;
    char* wlds = lds + wave * ((2 * G_STAGE) / (GWM * GWN));
    EpiCtx<T, f32x4, FM, FN, WTM, WTN, (2 * G_STAGE) / (GWM * GWN)> ctx{p, acc, wlds, m0 + wm * WTM, n0 + wn * WTN, lane,
                                                                      (int64_t)b * p.stride_c, RowsPlain::of(p)};
    if (p.out_dtype == DT_F32) {
        if (act == 0) ctx.template run<0, true>(); else if (act == 1) ctx.template run<1, true>();
        else ctx.template run<2, true>();
    } else {
        if (act == 0) ctx.template run<0, false>(); else if (act == 1) ctx.template run<1, false>();
        else ctx.template run<2, false>();
    }
}

// parts: workgroups that share a tile's k-tiles, in scratch memory (1: none, no scratch memory)
template <typename T, int MODE, int GBM, bool FAST, bool DEEP, bool SPLIT = false, bool ROWS = false>
hipError_t launch_gather_mode(const Problem& p, hipStream_t stream, int parts = 1, const ScratchUse* use = nullptr) {
    constexpr int GBK = DEEP ? 64 : 32, THREADS = DEEP ? 512 : 256;
    constexpr int LDS_BYTES = 2 * (GBM + GBN) * GBK * 2;
    static_assert(LDS_BYTES <= 64 * 1024, "launched without a raised limit");
    auto kern = gemm_mfma_gather_kernel<T, MODE, GBM, FAST, DEEP, SPLIT, ROWS>;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    DeviceShape ds;
    e = device_shape(dev, &ds);
    if (e != hipSuccess) return e;
    TileMapOf<MODE> tm{};
    if constexpr (MODE == MODE_CONV) {
        tm.pix = FastDiv::of(p.conv.OH * p.conv.OW);
        tm.ow = FastDiv::of(p.conv.OW);
    }
    tm.tiles_m = (p.M + GBM - 1) / GBM;
    tm.tiles_n = (p.N + GBN - 1) / GBN;
    tm.tiles_per_batch = tm.tiles_m * tm.tiles_n;
    const long long total = (long long)tm.tiles_per_batch * p.batch * parts;
    if (total <= 0 || total > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    tm.total = (int)total;
    tm.group_m = 8;
    tm.xcds = ds.xcds;
    Problem pa = p;
    Scratch scratch = use ? use->mem() : Scratch{};
    void* args[] = {&pa, &tm, &parts, &scratch};
    return launch_with(use, (const void*)kern, dim3((unsigned)total), dim3(THREADS), args, LDS_BYTES, stream);
}

// Every offset of FAST, the taps of the last k-tile and what the last rows reach beyond the image included, stays below 2^31.
bool gather_fast_offsets(const Problem& p) {
    const int64_t lim = ((int64_t)1 << 31) - ((int64_t)1 << 20), row = (int64_t)p.conv.W * p.conv.Cin * 2;
    return (int64_t)(p.M / (p.conv.OH * p.conv.OW)) * p.conv.H * row < lim && ((int64_t)p.K + 256) * p.ldb * 2 < lim;
}

// A row of taps as one tap of KW Cin channels (ROWS of the kernel)?  Where the rows are neighbours in memory and hold a piece, and that K axis is shorter.  One
// as long has fewer pieces at the end of a tap, which takes as much from the forms with two workgroups or fewer per unit (us, taps first: 8 x 44 x 44 x 127 ->
// 512, 3 x 3, stride 2 18.9 and 17.0; 8 x 56 x 56 x 64 -> 61, 3 x 3 19.3 and 16.2; two 128-row tiles per unit, 8 x 100 x 100 x 127 -> 127: 72.3 and 73.8).
// Shorter: 8 x 224 x 224 x 3 -> 64, 7 x 7, stride 2 45.8 and 28.5; 1 x 224 x 224 12.8 and 8.5; 8 x 102 x 102 x 3 -> 512, 5 x 5 81.7 and 52.6; 7 x 115 x 115 x
// 11 -> 32, 7 x 7 57 and 38; 5 x 64 x 64 x 35 -> 256, 3 x 3, stride 2 12.3 and 10.8; 2 x 101 x 101 x 100 -> 127, 5 x 5 45.3 and 40.5.
bool gather_rows_of_taps(const Problem& p, bool shorter) {
    const int64_t row = (int64_t)p.conv.KW * p.conv.Cin, ours = (row + 7) & ~7, theirs = (int64_t)p.conv.KW * ((p.conv.Cin + 7) & ~7);
    return p.conv.KW > 1 && p.conv.dil_w == 1 && row >= 8 && (int64_t)p.conv.W * p.conv.Cin >= 8 && (ours < theirs || (ours == theirs && !shorter));
}

// fast: a convolution with 32-bit offsets
template <typename T, int GBM, bool DEEP, bool SPLIT = false>
hipError_t launch_gather_type(const Problem& p, hipStream_t stream, bool fast, int parts = 1, const ScratchUse* use = nullptr) {
    if (p.is_conv && fast && gather_rows_of_taps(p, GBM == 128 && !DEEP)) return launch_gather_mode<T, MODE_CONV, GBM, true, DEEP, SPLIT, true>(p, stream, parts, use);
    if (p.is_conv) return fast ? launch_gather_mode<T, MODE_CONV, GBM, true, DEEP, SPLIT>(p, stream, parts, use)
                               : launch_gather_mode<T, MODE_CONV, GBM, false, DEEP, SPLIT>(p, stream, parts, use);
    if (p.trans_b) return launch_gather_mode<T, MODE_TRANS_B, GBM, false, DEEP, SPLIT>(p, stream, parts, use);
    return launch_gather_mode<T, MODE_DENSE, GBM, false, DEEP, SPLIT>(p, stream, parts, use);
}

}  // namespace

// 16-bit operands of any alignment and any K, N, leading dimensions and channel count; convolutions that
// are not transposed.  Each operand must hold the 16 bytes of one piece, and one image must stay below
// 2 GiB (32-bit offsets inside an image).
bool mfma_gather_supported(const Problem& p) {
    if (p.in_dtype != DT_BF16 && p.in_dtype != DT_F16) return false;
    if (p.K < 1 || p.M < 1 || p.N < 1) return false;
    int64_t a_elems, b_elems;
    if (p.is_conv) {
        if (p.conv.transposed) return false;
        // tap -> (kh, kw) by multiplication is exact below 2^20 / KW taps
        if ((int64_t)p.conv.KH * p.conv.KW + 64 >= ((int64_t)1 << 20) / p.conv.KW) return false;
        const int64_t img = (int64_t)p.conv.H * p.conv.W * p.conv.Cin;
        if (img * 2 + 64 >= ((int64_t)1 << 31)) return false;
        a_elems = (int64_t)(p.M / (p.conv.OH * p.conv.OW)) * img;
        // the loop runs over taps * ceil8(Cin)
        if ((int64_t)p.conv.KH * p.conv.KW * ((p.conv.Cin + 7) & ~7) + 4 * 64 >= ((int64_t)1 << 31)) return false;
    } else {
        a_elems = (int64_t)(p.M - 1) * p.lda + p.K;
    }
    b_elems = p.trans_b ? (int64_t)(p.N - 1) * p.ldb + p.K : (int64_t)(p.K - 1) * p.ldb + p.N;
    if ((int64_t)p.K + 4 * 64 >= ((int64_t)1 << 30)) return false;
    return a_elems >= 8 && b_elems >= 8;
}

// Against the generic kernel, whose tiles are 64 x 64 (its time in us first): with 4096 outputs or more per entry from 16 k on.  With fewer
// - from 64 k and 16 columns on, where most of a tile would be empty otherwise (a convolution of 81 x 32 outputs, K = 75: 19.1 and 9.3; 36 x 32,
//   K = 2989: 401 and 15; 1 x 17 x 65: 9.4 and 6.9, 1 x 4001 x 257: 27 and 8.7, 250 x 16 x 1001: 117 and 11);
// - but not many entries that fill as many of its tiles as of these ones, which are larger, with a short contraction (17 x 17 to 63 x 63: 400 of
//   K = 65 12.8 to 15.9 and 9.2 to 12.7, 520: 13.5 to 19.7 and 14.9 to 18.8, 1500: 21.2 to 26.1 and 24.2 to 36.3; K = 97: 1500 27.6 to 33.4 and 23.8 to 34.4,
//   k-major B 24.5 to 35.2 and 24.2 to 34.0, 4000 54 to 101 and 59 to 98; K = 129: 8000 135 to 237 and 136 to 208; with three of its tiles to two of these,
//   1 x 129 and 30 x 130, 2000 of K = 65: 62 to 78 and 59 to 70, k-major B 55 to 70 and 59 to 72; with more of them, 100 x 17, 1 x 70 and 3 x 513: 1.2 to 1.6 times
//   as fast with any number).
bool mfma_gather_preferred(const Problem& p) {
    if (p.K < 16) return false;
    if ((long long)p.M * p.N >= 4096) return true;
    if (p.K < 64 || p.N < 16) return false;
    const long long theirs = (long long)((p.M + 63) / 64) * ((p.N + 63) / 64), ours = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128);
    if (2 * theirs > 3 * ours || (2 * theirs == 3 * ours && !p.trans_b)) return true;
    return p.K >= (ours * p.batch <= 512 ? 64 : ours * p.batch <= 2048 ? 96 : 128);
}

// Tiles, by how many rounds of the 256 compute units they make (us):
// - one round of 64-row ones: those, because a workgroup alone on its unit is bound by latency (8 x 44 x 44 x 127 -> 512, 3 x 3, stride 2, 224 tiles: 33.4 ->
//   25.4; 577 x 1021 x 4096, 80 tiles: 49.9 -> 35.0), in the deep form (18.6); two or three of the other form share a unit (3 x 81 x 81 x 35 -> 512, 3 x 3,
//   stride 2, 316 tiles: 22.7 deep, 16.6; 6 x 108 x 108 x 3 -> 65: 15.9 and 10.8);
// - one round of 128-row ones: those in the deep form (64-row tiles, two or three per unit, first: 6 x 122 x 122 x 127 -> 127, 5 x 5, stride 2 61.6 and 54.7;
//   5 x 149 x 149 x 100 -> 64, 7 x 7, stride 2 93.2 and 80.4; 3 x 161 x 161 x 3 -> 64, 7 x 7, stride 2 19.1 and 16.3; 128-row tiles of four waves first: 1993 x
//   1146 x 3993, k-major B 63.9 and 52.3, 2363 x 1394 x 663 20.8 and 19.2), but a short product (942 x 2430 x 241: 14.0 and 14.1);
// - a convolution whose 64-row tiles a unit holds three of: those (2 x 134 x 134 x 100 -> 65, 7 x 7, 281 tiles of 128 rows: 126 and 117; 7 x 75 x 75 x 3 -> 65,
//   7 x 7 26.7 and 24.6; 392 tiles, 4 x 112 x 112 x 35 -> 128, 3 x 3: 21.4 and 27.2), unless they have up to 32 columns, a long contraction and taps that rows do
//   not shorten (128-row ones first: 3 x 113 x 113 x 127 -> 32, 5 x 5, 81.3 and 87.8; 2 x 150 x 150 x 119 -> 32, 7 x 7, 146 and 156; x 100, which they shorten, 122 and 115);
// - beyond that two 128-row ones per unit.
enum : int { GATHER_128 = 0, GATHER_64, GATHER_DEEP64, GATHER_DEEP128 };
static int gather_form(const Problem& p) {
    const long long cols = (p.N + GBN - 1) / GBN;
    const long long t128 = (long long)((p.M + 127) / 128) * cols * p.batch, t64 = (long long)((p.M + 63) / 64) * cols * p.batch;
    if (t64 <= 256) return GATHER_DEEP64;
    if (t128 <= 256) return p.is_conv || p.K > 512 ? GATHER_DEEP128 : GATHER_64;
    return p.is_conv && t64 <= 768 && !(p.N <= 32 && p.K >= 3072 && !gather_rows_of_taps(p, true)) ? GATHER_64 : GATHER_128;
}

// Workgroups that share a tile (1: tiles are not split): up to one per compute unit, and up to eight, p of them from p (p + 2) k-tiles of 64 on,
// because every part adds a k-tile's worth to the parts' meeting.  In us, unsplit first:
// - 3 x 1657 x 8403, 13 tiles: 59 and 16 with 8 parts; 14 x 4459 x 8768, 35 tiles: 66 and 21 with 6; 36 x 10083 x 11392, 79 tiles: 103 and 48
//   with 3; 640 x 448 x 1927: 20.3 and 13.7 with 3, 14.1 with 4, 15.6 with 6; convolutions 2 x 15 x 15 x 100 -> 64, 7 x 7: 60 and 17.6, 1 x 18 x 18 x
//   61 -> 32, 7 x 7, stride 2, one tile: 40 and 15.2; 3 x 21 x 21 x 100 -> 127, 3 x 3: 18.7 and 14.5;
// - what short ones do not give back: 64 x 1003 x 501: 11.6 and 11.9, 300 x 300 x 301: 9.7 and 10.7, 130 x 2496 x 970, 60 tiles: 10.7 and 10.7;
//   convolutions of 2 and 3 k-tiles: 9.3 and 9.8, 8.6 and 9.3.
// rows: a row of taps is one tap.  The k-tiles are those of the K axis that the kernel then walks, up to eight times shorter than with a tap each (8 x 8 over one
// channel: one k-tile for eight; two parts of it, one of them empty, 8.1, whole 5.9), and cost more each, so that three parts pay sooner with few tiles: up
// to 32 from six k-tiles on, up to 40 from nine, up to 64 from eleven (whole, 2 parts, 3: 11 tiles, 6 k-tiles, 11.7, 11.2 and 10.9; 18, 7 11.6, 11.5 and 11.1; 50, 7 11.2,
// 11.7 and 12.2; 22, 9 13.7, 12.2 and 11.3; 38, 9, 2 parts and 3, 12.3 and 11.9, 44 tiles 12.4 and 12.7; 48, 11 15.5, 13.5 and 13.2; 61, 13 16.5, 14.8 and 14.8; 81, 11 16.2,
// 15.5 and 16.9; 13, 5 11.2, 11.8 and 11.6; 112, 7 11.0 and 12.7), and more parts a twelfth sooner (45 k-tiles, 5 and 6 parts: 16.3 and 15.8; 77, 7 and 8: 16.9 and 16.4).
static int gather_parts(const Problem& p, bool rows) {
    const long long tiles = (long long)((p.M + 63) / 64) * ((p.N + GBN - 1) / GBN) * p.batch;
    const long long tap = rows ? (long long)p.conv.KW * p.conv.Cin : p.conv.Cin, taps = rows ? p.conv.KH : (long long)p.conv.KH * p.conv.KW;
    const long long kt = ((p.is_conv ? taps * ((tap + 7) & ~7LL) : p.K) + 63) / 64;
    if (rows && kt < 15 && kt >= (tiles <= 32 ? 6 : tiles <= 40 ? 9 : tiles <= 64 ? 11 : 15)) return 3;
    if (tiles > 128 || kt < (p.is_conv ? 8 : 12)) return 1;
    const long long room = (long long)kScratchBytes / (64 * GBN * 4) / tiles;        // the parts' sums have to fit
    int parts = 1;
    static_assert(3 * 64 * 64 * GBN * 4 <= kScratchBytes, "three parts of 64 tiles");
    const long long worth = rows ? kt + kt / 12 : kt;
    while (parts < 8 && (parts + 1) * tiles <= 256 && parts < room && (parts + 1) * (parts + 3) <= worth) ++parts;
    return parts;
}

// force_cfg: 0 the 128-row tiles, 1 the 64-row ones (deep or not by the rule), 4 the deep 128-row ones; 2, 3 and 5 the same with a convolution's 64-bit
// addresses; otherwise by the rule.
hipError_t launch_mfma_gather(const Problem& p, hipStream_t stream, int force_cfg, const char** name) {
    const bool forced_wide = force_cfg == 2 || force_cfg == 3 || force_cfg == 5;
    const bool bf16 = p.in_dtype == DT_BF16, fast = p.is_conv && !forced_wide && gather_fast_offsets(p);
    const int wide = p.is_conv && !fast;           // 64-bit addresses and rows of taps: by names of their own
    int form = gather_form(p);
    if (force_cfg == 0 || force_cfg == 2) form = GATHER_128;
    if (force_cfg == 1 || force_cfg == 3) form = form == GATHER_DEEP64 ? GATHER_DEEP64 : GATHER_64;
    if (force_cfg == 4 || force_cfg == 5) form = GATHER_DEEP128;
    const int kind = wide ? 1 : p.is_conv && gather_rows_of_taps(p, form == GATHER_128) ? 2 : 0;
    if (form == GATHER_DEEP64) {
        const int parts = gather_parts(p, kind == 2);
        int dev = 0;
        if (parts > 1 && hipGetDevice(&dev) == hipSuccess) {
            if (const ScratchUse use(dev, stream); use) {
                static const char* const split[3] = {"mfma16_gather_64x128x64_w4x2_split", "mfma16_gather_64x128x64_w4x2_a64_split", "mfma16_rows_gather_64x128x64_w4x2_split"};
                *name = split[kind];
                return bf16 ? launch_gather_type<bf16_t, 64, true, true>(p, stream, fast, parts, &use)
                            : launch_gather_type<f16_t, 64, true, true>(p, stream, fast, parts, &use);
            }
        }
    }
    static const char* const names[4][3] = {
        {"mfma16_gather_128x128x32_w2x2", "mfma16_gather_128x128x32_w2x2_a64", "mfma16_rows_gather_128x128x32_w2x2"},
        {"mfma16_gather_64x128x32_w2x2", "mfma16_gather_64x128x32_w2x2_a64", "mfma16_rows_gather_64x128x32_w2x2"},
        {"mfma16_gather_64x128x64_w4x2", "mfma16_gather_64x128x64_w4x2_a64", "mfma16_rows_gather_64x128x64_w4x2"},
        {"mfma16_gather_128x128x64_w4x2", "mfma16_gather_128x128x64_w4x2_a64", "mfma16_rows_gather_128x128x64_w4x2"}};
    *name = names[form][kind];
    switch (form) {
    case GATHER_DEEP64: return bf16 ? launch_gather_type<bf16_t, 64, true>(p, stream, fast) : launch_gather_type<f16_t, 64, true>(p, stream, fast);
    case GATHER_DEEP128: return bf16 ? launch_gather_type<bf16_t, 128, true>(p, stream, fast) : launch_gather_type<f16_t, 128, true>(p, stream, fast);
    case GATHER_64: return bf16 ? launch_gather_type<bf16_t, 64, false>(p, stream, fast) : launch_gather_type<f16_t, 64, false>(p, stream, fast);
    default: return bf16 ? launch_gather_type<bf16_t, 128, false>(p, stream, fast) : launch_gather_type<f16_t, 128, false>(p, stream, fast);
    }
}

}  // namespace pbk
