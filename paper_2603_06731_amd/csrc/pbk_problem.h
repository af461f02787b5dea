// Internal description of one contraction, shared by the dispatcher and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbk {

enum : int { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2, DT_FP8_E4M3 = 3, DT_FP8_E5M2 = 4, DT_INT8 = 5 };
enum : int { EPI_NONE = 0, EPI_BIAS = 1, EPI_RELU = 2, EPI_BIAS_RELU = 3,
             EPI_BIAS_GELU_TANH = 4, EPI_GELU_TANH = 5 };

// Geometry of the convolution whose im2col rows form the A operand
// (paper Sec. 4.5: row i = (n, oh, ow), column k = (kh, kw, c)).
struct ConvGeom {
    int H, W, Cin;
    int OH, OW;
    int KH, KW;
    int stride_h, stride_w, pad_h, pad_w, dil_h, dil_w;   // pad: near side (top, left)
    // 0: row (n, oh, ow) reads input rows oh*stride - pad + kh*dil.
    // 1: transposed convolution in gather form: it reads input row (oh + pad - kh*dil)/stride
    //    for the taps where the division is exact.
    // 2: the same, rows walked by residue classes (set inside the matrix-unit path only).
    int transposed;
};

struct Problem {
    const void* A;        // M x K (lda), or the NHWC image when is_conv
    const void* B;        // K x N (ldb), or N x K (ldb) when trans_b
    void* C;              // M x N (ldc)
    const float* bias;    // [N] or nullptr
    int M, N, K, batch;
    int64_t lda, ldb, ldc;
    int64_t stride_a, stride_b, stride_c;   // elements between batch entries
    int in_dtype, out_dtype;
    int trans_b;
    int is_conv;
    int epi;
    float alpha;
    ConvGeom conv;
    // residual-add epilogue: out = act(alpha*acc + bias + beta*R), R of out_dtype, M x N (ldr); nullptr = none
    const void* R;
    int64_t ldr;
    float beta;
    // int8 operands (in_dtype DT_INT8): integer accumulation and the quantised epilogue
    //   t = float(acc)*q_scale[n] (+ bias[n]); optional requantise/dequantise with q_mid;
    //   unfolded batch norm if q_mean: t = (t - q_mean[n]) * (1 / sqrt(q_var[n] + q_eps)), q_mul = gamma, q_add = beta;
    //   t = t*q_mul[n] + q_add[n] (each if given); ReLU if q_relu;
    //   out = int8(clamp(roundeven(t/q_out))) for out_dtype DT_INT8, else t as fp32.
    const float* q_scale;
    const float* q_mul;
    const float* q_add;
    float q_mid, q_out;
    int q_relu;
    const float* q_mean;
    const float* q_var;
    float q_eps;
};

// One attention layer call (paper Sec. 4.4): O = softmax(alpha Q K^T + bias) V
// per batch entry; Q, O [Nq][D], K, V [Nk][D], bias float [Nq][Nk] or nullptr.
struct AttnProblem {
    const void* Q;
    const void* K;
    const void* V;
    const float* bias;
    void* O;
    int batch, Nq, Nk, D;
    int64_t ldq, ldk, ldv, ldo;                          // row strides, elements
    int64_t stride_q, stride_k, stride_v, stride_o;      // batch strides, elements
    int64_t ld_bias, stride_bias;
    int dtype;                                           // of Q, K, V and O
    float alpha;
    int causal;                                          // 1: row i attends to keys j <= i + (Nk - Nq) only (no bias then)
};

__host__ __device__ inline bool epi_has_bias(int epi) {
    return epi == EPI_BIAS || epi == EPI_BIAS_RELU || epi == EPI_BIAS_GELU_TANH;
}

// Launchers.  Each returns hipSuccess or the launch error; `name` receives a
// static string naming the configuration that ran.
hipError_t launch_generic(const Problem& p, hipStream_t stream, const char** name);
// fp32 matmuls of up to some thousand 16 x 16 tiles: the operands go straight to registers
bool small_f32_supported(const Problem& p);
bool small_f32_preferred(const Problem& p);
hipError_t launch_small_f32(const Problem& p, hipStream_t stream, const char** name);

// Returns false if this problem cannot take the MFMA path (alignment, dtype).
bool mfma_supported(const Problem& p);
// Returns false where the generic kernel is the better choice although the MFMA path could run.
bool mfma_preferred(const Problem& p);
hipError_t launch_mfma(const Problem& p, hipStream_t stream, int force_cfg, const char** name);

// The matrix-unit kernel that stages its tiles through registers: 16-bit operands of any alignment, K, N, leading
// dimensions and channel counts.
bool mfma_gather_supported(const Problem& p);
bool mfma_gather_preferred(const Problem& p);
hipError_t launch_mfma_gather(const Problem& p, hipStream_t stream, int force_cfg, const char** name);

// Short contractions (K <= 256) over many rows: B stationary in registers, the workgroup walks down M.
bool mfma_bstat_supported(const Problem& p);
bool mfma_bstat_preferred(const Problem& p);
hipError_t launch_mfma_bstat(const Problem& p, hipStream_t stream, const char** name);

// Few rows, or too few 128-wide tiles for the chip: the contraction is split over the waves of a workgroup.
// ksplit: operands straight into registers, each wave on its own; tile64: 64-wide tiles staged in LDS by all waves.
bool mfma_ksplit_supported(const Problem& p);
bool mfma_ksplit_preferred(const Problem& p);
hipError_t launch_mfma_ksplit(const Problem& p, hipStream_t stream, int force_cfg, const char** name);
bool mfma_tile64_supported(const Problem& p);
bool mfma_tile64_built(const Problem& p, int force_cfg);       // the form of this id, for the problem's type (-1: any)
bool mfma_tile64_preferred(const Problem& p);
hipError_t launch_mfma_tile64(const Problem& p, hipStream_t stream, int force_cfg, const char** name);
// tile64 with the contraction split over workgroups as well, in scratch memory of the stream; launch: false where the problem is not
// split (forced: any that makes two parts of a round) or there is no scratch memory, and nothing was launched then.
constexpr int kSplitChoice = 8;          // its id behind "tile64:"
bool mfma_tile64_split_preferred(const Problem& p);
bool launch_mfma_tile64_split(const Problem& p, hipStream_t stream, bool forced, const char** name, hipError_t* e);

// PBK_GROUP_M of the environment as read at the process's first call (0 = not set): tile rows
// per group of the block mapping, a benchmarking override.
int group_m_override();

// Attention: generic kernel (any dtype/alignment, D <= 512) and the fused MFMA kernel.
hipError_t launch_attention_generic(const AttnProblem& p, hipStream_t stream, const char** name);
bool attention_mfma_supported(const AttnProblem& p);
hipError_t launch_attention_mfma(const AttnProblem& p, hipStream_t stream, int force_cfg, const char** name);
// A few queries against a long context: the keys are split over the waves of a workgroup.
bool attention_decode_supported(const AttnProblem& p);
bool attention_decode_preferred(const AttnProblem& p);
hipError_t launch_attention_decode(const AttnProblem& p, hipStream_t stream, int force_cfg, const char** name);

}  // namespace pbk
