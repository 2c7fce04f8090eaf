// Internal launch interface between the host orchestration and the gfx950 kernels.
#pragma once
#include "common.h"

// ---------------------------------------------------------------- GEMM (gemm_bf16.hip)
// C = alpha * (A B^T + A2 B2^T) (+ R), bf16 operands, fp32 accumulate (MFMA).
struct GemmNT {
    const bf16_t* A = nullptr;  long lda = 0;   // [M, K]
    const bf16_t* B = nullptr;  long ldb = 0;   // [N, K]
    int M = 0, N = 0, K = 0;
    const bf16_t* A2 = nullptr; long lda2 = 0;  // [M, K2]  (low-rank K-extension; may be null)
    const bf16_t* B2 = nullptr; long ldb2 = 0;  // [N, K2]
    int K2 = 0;
    float alpha = 1.f;
    const float* R = nullptr;                   // fp32 [M, N] residual (c_f32 only), row stride ldc
    void* C = nullptr;          long ldc = 0;   // bf16 or fp32 [M, N]
    int c_f32 = 0;
    int batch = 1;                              // grid.z; element offsets applied per batch index:
    long bA = 0, bB = 0, bA2 = 0, bB2 = 0, bC = 0;
    int split_k = 0;                            // 0 = choose; >1 needs `partial`
    float* partial = nullptr;                   // fp32 scratch, >= batch*split*M*N elements
    size_t partial_elems = 0;
    // If set (batch must be 1, alpha 1): when the launcher splits the contraction of a wide-output GEMM it leaves the
    // fp32 partial tiles in `partial` ([n_split][M][N]), does not write C (nor add R), and stores n_split here, so that
    // the consumer can add them up itself instead of a reduce pass; otherwise 0 is stored and C is written.
    int* deferred = nullptr;
};
hipError_t launch_gemm_nt(const GemmNT& g, hipStream_t s);
// name of the tile configuration launch_gemm_nt picks for g (a static string) and the contraction split it uses
const char* gemm_nt_plan(const GemmNT& g, int* n_split);
// cheaper as two launches over two ranges of the columns (of every batch) or rows (see gemm_bf16.hip): they are left in a and b, and
// g.deferred, if set, receives 0; false: one launch
bool gemm_nt_two_parts(const GemmNT& g, GemmNT* a, GemmNT* b);

// The same for the narrow bf16 output of a low-rank product, without a second operand pair: one launch where that is faster
hipError_t launch_low_rank(const GemmNT& g, hipStream_t s);
const char* low_rank_plan(const GemmNT& g);      // name of its tile, "general" where it goes to launch_gemm_nt

// launch_gemm_nt, or the kernel of the low-rank products where that is faster: few outputs, few weights
hipError_t launch_frozen(const GemmNT& g, hipStream_t s);
const char* frozen_plan(const GemmNT& g);

// Direct-to-LDS loads take addresses that are multiples of 4 bytes (4 and 8 give what 16 gives); operands that start anywhere else, which only a
// caller of a single kernel can pass, come through registers.
inline bool loads_to_lds(const void* p) { return ((uintptr_t)p & 3) == 0; }

// C[Mo, No] (fp32) = alpha * P[T, Mo]^T Q[T, No]
struct GemmTN {
    const bf16_t* P = nullptr; long ldp = 0;
    const bf16_t* Q = nullptr; long ldq = 0;
    int T = 0, Mo = 0, No = 0;
    float alpha = 1.f;
    float* C = nullptr; long ldc = 0;
    int batch = 1;
    long bP = 0, bQ = 0, bC = 0;
    float* partial = nullptr;                   // optional scratch for splitting the token dimension
    size_t partial_elems = 0;
};
hipError_t launch_gemm_tn(const GemmTN& g, hipStream_t s);

// Up to TN_GROUP_MAX products C_k[Mo_k, No_k] (fp32) = P_k[T, Mo_k]^T Q_k[T, No_k] over the same T tokens in one
// launch (the dA and dB of every projection of a decoder layer).  tile0 is filled in by the launcher.
constexpr int TN_GROUP_MAX = 12;
struct TnProblem {
    const bf16_t* P = nullptr; const bf16_t* Q = nullptr; float* C = nullptr;
    long ldp = 0, ldq = 0, ldc = 0;
    int Mo = 0, No = 0, tile0 = 0, pad = 0;
};
struct GemmTNGroup {
    TnProblem p[TN_GROUP_MAX];
    int n = 0, T = 0;
    int* flag = nullptr;   // if set: bit 1 of *flag is raised when any product entry is not finite
    void add(const bf16_t* P, long ldp, int Mo, const bf16_t* Q, long ldq, int No, float* C, long ldc) {
        if (n < TN_GROUP_MAX) { TnProblem& q = p[n]; q.P = P; q.ldp = ldp; q.Mo = Mo; q.Q = Q; q.ldq = ldq; q.No = No; q.C = C; q.ldc = ldc; }
        ++n;
    }
};
hipError_t launch_gemm_tn_grouped(GemmTNGroup& g, hipStream_t s);

// fp32 products of the single-layer fp32 step (gemm_f32.hip): C = alpha A B^T (+ alpha2 A2 B2^T), operands, outputs and sums in fp32.
enum F32Kind { F32_KK = 0, F32_KN = 1, F32_MN = 2 };   // A [M,K] B [N,K] / A [M,K] B [K,N] / A [K,M] B [K,N], row-major
// the first AdamW step of a parameter (moments zero before it)
struct AdamWFirst { float lr, b1, b2, eps, decay, inv_bc1, inv_bc2; };
__device__ __forceinline__ float adamw_first(float p, float g, const AdamWFirst& o) {
    const float m = (1.f - o.b1) * g, v = (1.f - o.b2) * g * g;
    return p * o.decay - o.lr * (m * o.inv_bc1) / (sqrtf(v * o.inv_bc2) + o.eps);
}
struct F32Product {
    int kind = F32_KK;
    const float* A = nullptr;  long lda = 0;
    const float* B = nullptr;  long ldb = 0;
    int M = 0, N = 0, K = 0;
    const float* A2 = nullptr; long lda2 = 0;   // second operand pair of the same layouts (the low-rank term), K2 elements
    const float* B2 = nullptr; long ldb2 = 0;
    int K2 = 0;
    float alpha = 1.f, alpha2 = 1.f;
    float* C = nullptr;        long ldc = 0;
    const float* p_old = nullptr;               // with p_new: the product is the gradient of p_old (same shape and row
    float* p_new = nullptr;                     // stride), and p_new receives p_old after its first AdamW step
    AdamWFirst opt = {};
    int tiles_m = 0, tiles_n = 0, tile0 = 0;    // filled in by the launcher
};
constexpr int F32_GROUP_MAX = 4;
// n independent products in one launch.  Outputs must not overlap any operand.
hipError_t launch_gemm_f32_group(const F32Product* prods, int n, hipStream_t s);
// The name of the instance that such a launch takes.
const char* gemm_f32_plan(const F32Product* prods, int n);
hipError_t launch_adamw_first(const float* g, const float* p, float* p_new, size_t n, const AdamWFirst& o, hipStream_t s);

// ---------------------------------------------------------------- attention (attention.hip)
hipError_t launch_attention_fwd(const bf16_t* q, const bf16_t* k, const bf16_t* v, long ldq, int T, int n_heads,
                                int d_head, bf16_t* o, long ldo, float* lse, hipStream_t s);
hipError_t launch_attention_bwd(const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* o, const bf16_t* d_o,
                                const float* lse, long ldq, long ldo, int T, int n_heads, int d_head, bf16_t* dq,
                                bf16_t* dk, bf16_t* dv, float* delta, const float2* rope, hipStream_t s);

// ---------------------------------------------------------------- elementwise / reductions (elementwise.hip)
// part != null: the input row is not read from h but formed as the sum of n_part fp32 arrays [T, d] lying part_stride
// elements apart plus resid (may be null), and written to h_write (the residual stream) on the way.
hipError_t launch_rmsnorm_fwd(const float* h, const float* g, int T, int d, float eps, bf16_t* y, hipStream_t s,
                              const float* part = nullptr, int n_part = 0, long part_stride = 0,
                              const float* resid = nullptr, float* h_write = nullptr);
// dy_part != null: dy is the sum of n_part fp32 arrays [T, d] that lie part_stride elements apart (the
// partial tiles a split GEMM left behind, see GemmNT::deferred); the bf16 dy is then not read.
hipError_t launch_rmsnorm_bwd(const bf16_t* dy, const float* h, const float* g, const float* dres, int T, int d,
                              float eps, float* dh_out, bf16_t* dh_bf, hipStream_t s, const float* dy_part = nullptr,
                              int n_part = 0, long part_stride = 0);
hipError_t launch_rope(bf16_t* x, long ld, int T, int n_heads, int d_head, float base, int pos0, int sign,
                       const float2* table, hipStream_t s);
hipError_t launch_rope_table(float2* table, int n_pos, int d_head, float base, hipStream_t s);
hipError_t launch_swiglu_fwd(const bf16_t* gu, int T, int f, bf16_t* a, hipStream_t s);
hipError_t launch_swiglu_bwd(const bf16_t* da, const bf16_t* gu, int T, int f, bf16_t* dgu, hipStream_t s);
// labels: one per position, read for target positions only
hipError_t launch_cross_entropy(const float* logits, const int* labels, int T, int V, int first_target,
                                int n_targets, float* nll, bf16_t* dlogits, float* loss_sum, hipStream_t s, int row0 = 0,
                                int* flag = nullptr);
hipError_t launch_adamw(float* p, const float* g, float* m, float* v, bf16_t* shadow, size_t n, long step, float lr,
                        float beta1, float beta2, float eps, float wd, hipStream_t s, const int* skip_flag = nullptr);
hipError_t launch_embed(const bf16_t* E, const int* tokens, int T, int d, float* h, hipStream_t s, int* tok_out = nullptr);
hipError_t launch_f32_to_bf16(const float* src, bf16_t* dst, size_t n, hipStream_t s);
hipError_t launch_fill_f32(float* p, size_t n, float value, hipStream_t s);
// rows [0, r0) and [r1, T) of x and y, both [T, d], d a multiple of 4, become zero
hipError_t launch_zero_rows_around(float* x, bf16_t* y, int T, int d, int r0, int r1, hipStream_t s);
hipError_t launch_init_normal(float* p, size_t n, float std, uint64_t seed, uint64_t stream_id, hipStream_t s);
// LoRA dropout: the mask is a function of (key, element index); key from (seed, optimizer step, layer, group)
uint64_t dropout_key(uint64_t seed, int64_t step, int layer, int group);
hipError_t launch_dropout_fwd(const bf16_t* x, bf16_t* y, size_t n, uint64_t key, float p, hipStream_t s);
// dx [T, d_in] += D o (dH A), dH [T, K], AT [d_in, K]
hipError_t launch_dropout_low_rank_add(const bf16_t* dH, long ldh, const bf16_t* AT, long lda, int K, bf16_t* dx, int T, int d_in, uint64_t key,
                                       float p, hipStream_t s);
// dst[c, r] = src[r, c] for a [rows, cols] bf16 matrix with row strides lds / ldd
hipError_t launch_transpose_bf16(const bf16_t* src, long lds, int rows, int cols, bf16_t* dst, long ldd,
                                 hipStream_t s);
// many transposes in one launch: descriptors live in device memory
struct TransposeDesc { long src_off, dst_off; int rows, cols, lds, ldd, tile0, pad; };
hipError_t launch_transpose_table(const bf16_t* src_base, bf16_t* dst_base, const TransposeDesc* table_dev,
                                  int n_desc, int n_tiles, hipStream_t s, int tile_begin = 0);
// copy rows [rows, cols] bf16 from src (stride lds) to dst (stride ldd)
hipError_t launch_copy2d_bf16(const bf16_t* src, long lds, int rows, int cols, bf16_t* dst, long ldd, hipStream_t s);

// ---------------------------------------------------------------- one-token decoding (decode.hip)
// Where a matrix-vector product takes its input vector from (see gemv_kernel; mode 2 and x_out serve single calls)
struct GemvPre {
    int mode = 0;                 // 0: x as given; 1: RMSNorm of h with gain; 2: SwiGLU of the gate|up row gu
    const float* h = nullptr;
    const float* gain = nullptr;
    float eps = 0.f;
    const bf16_t* gu = nullptr;
    bf16_t* x_out = nullptr;      // if set, workgroup 0 stores the input vector it formed
};
// The low-rank term of a matrix-vector product (see gemv_kernel): either b, with h given, or the rows of a beside those of W.
struct GemvLora {
    const bf16_t* b = nullptr;            // [N, r]: adds sum_j b[n, j] h[(n / rows_per_group) r + j]
    int r = 0, rows_per_group = 0;        // rows_per_group 0: one group
    const float* h = nullptr;             // n_parts 0: h as it is; else n_parts vectors of r, h = scale * their sum (one group)
    int n_parts = 0;
    const bf16_t* a = nullptr;            // [n_a, K]: h_out = scale * a x
    int n_a = 0;
    float* h_out = nullptr;
    float scale = 1.f;
};
// y[N] = alpha * (W[N, K] x[K] + low-rank term) (+ resid, fp32 output only)
hipError_t launch_gemv(const bf16_t* W, long ldw, const bf16_t* x, int N, int K, const GemvLora& lora, float alpha,
                       const float* resid, bf16_t* y_bf, float* y_f32, hipStream_t s, const GemvPre* pre = nullptr);
// act = SwiGLU of one token's gate|up (raw fp32 [2 f] + B h, B [2 f, r], h [2 r]), and the shares of A_down act, one vector of
// r per DECODE_SW columns
constexpr int DECODE_SW = 128;
hipError_t launch_decode_swiglu(const float* raw, const bf16_t* b, const float* h, int r, int f, bf16_t* act,
                                const bf16_t* a_down, float* part, hipStream_t s);
// one query row against cache rows 0 .. n_keys-1 (row stride ld), per head
constexpr int ATTN_DECODE_MAX_SPLIT = 32;   // key ranges per head in the split decode-attention path
// Keys that one workgroup takes on, a head's whole cache or one range of it.  The kernels would take any number; these are the
// limits the entry points have always had, so that a call with too little scratch is told so instead of leaving a long cache
// to a few workgroups.
constexpr int ATTN_DECODE_MAX_UNSPLIT = 30208, ATTN_DECODE_MAX_RANGE = 13312;
struct DecodeFresh {                      // the newest token, if its q, k, v are still to be formed: raw + B h
    const float* raw = nullptr;           // [3 d]
    const bf16_t* b = nullptr;            // [3 d, r]
    const float* h = nullptr;             // [3 r]
    int r = 0, d = 0;
    const float2* rope = nullptr;         // (cos, sin) of its position for i = 0 .. d_head / 2 - 1
};
struct DecodeOut {
    bf16_t* o = nullptr;                  // [n_heads * d_head]
    const bf16_t* a = nullptr;            // with [r, n_heads * d_head]: part[head * r + j] = that head's share of a o
    int r = 0;
    float* part = nullptr;
};
hipError_t launch_attention_decode(const bf16_t* q, bf16_t* k, bf16_t* v, long ld, int n_keys, int n_heads, int d_head,
                                   const DecodeOut& out, float* ws, size_t ws_elems, hipStream_t s,
                                   const DecodeFresh& fresh = DecodeFresh{});
// index of the largest of n floats, lowest index among equals
hipError_t launch_argmax(const float* x, int n, int* out, hipStream_t s);
