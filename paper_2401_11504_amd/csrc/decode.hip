// One-token kernels of the generation side of Algorithm 1 (greedy decoding with the temporary LoRA module and a
// key/value cache): matrix-vector products with the LoRA correction, attention of one query against the cache, and
// the greedy argmax.  All of them stream their operand once: at one token per step the decoder is bound by reading
// the 13.5 GB of frozen weights, not by arithmetic.
#include "kernels.h"
#include <type_traits>

typedef unsigned gemv_vu4 __attribute__((ext_vector_type(4)));
// 16 bytes of a weight row.  Every byte of the matrix is read exactly once per token, so the loads are marked
// non-temporal: measured 5 % faster per token than ordinary loads.
__device__ __forceinline__ uint4 load_w16(const bf16_t* p) {
    const gemv_vu4 v = __builtin_nontemporal_load((const gemv_vu4*)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float dot8(const uint4& w, const float (&b)[8], float acc) {
    float a[8];
    unpack8(w, a);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += a[e] * b[e];
    return acc;
}

// One piece's share of A x: part[j] = sum over the piece's C columns of a[j, c] x[c], j < r, by NT threads.  C / 8 lanes share a
// row of A (row stride lda, a points at the piece's first column); x is in LDS, zero past the `left` columns that exist.
// av: the first NA rows per thread, row j = thread / (C / 8) + i * (8 NT / C), fetched ahead by the caller.
template <int C, int NT, int NA>
__device__ __forceinline__ void lowrank_part(const bf16_t* a, long lda, int r, const float* x, int left, uint4 (&av)[NA], float* part) {
    constexpr int LPR = C / 8, STEP = NT / LPR;
    const int sub = threadIdx.x % LPR, jj = threadIdx.x / LPR;
    float xv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) xv[e] = x[sub * 8 + e];
    for (int j0 = 0; j0 < r; j0 += NA * STEP) {
        if (j0) {
#pragma unroll
            for (int i = 0; i < NA; ++i) av[i] = *(const uint4*)(a + (long)min(j0 + jj + i * STEP, r - 1) * lda + min(sub * 8, left - 8));
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            float v = dot8(av[i], xv, 0.f);
#pragma unroll
            for (int off = LPR >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            const int j = j0 + jj + i * STEP;
            if (sub == 0 && j < r) part[j] = v;
        }
    }
}

// ---------------------------------------------------------------- y = W x (+ s-scaled LoRA term) (+ residual)
// R output rows n per wave: a row W[n, :] is read with 16-byte loads, 64 lanes wide; x sits in LDS.  The first eight loads
// of each row (all of it up to 4096 columns) are issued before x is formed, so that the weights stream while the workgroup
// is busy with its prologue (lm_head of the 7B shape 51.7 -> 41.7 us, 6.3 TB/s; gate|up 30.9 us with its rows of A, 5.8 TB/s).
// The low-rank term of a projection costs no launch of its own (four of them per layer were 26 of 122 us: a few microseconds
// of latency each):
//   lora.a: the rows of A ride along behind the rows of W and leave h = scale A x in lora.h_out, for whoever reads y to add
//   B h (q|k|v: the attention launch; gate|up: decode_swiglu_kernel);
//   lora.b (bf16 [N, r]) adds B h, where h = scale * the sum of n_parts vectors that the launch before has left, each from its
//   own piece of x (attention: one per head; decode_swiglu_kernel: one per workgroup).
// (One launch that computes A x in its first workgroups and hands it to the others through tagged words was no faster than
// two: every wave waited for it at the end with its registers full.)
// Where x comes from (MODE = pre.mode): 0 a bf16 vector; 1 RMSNorm of an fp32 row, x = bf16(h rho gain), formed in every
// workgroup (the vector is a few KB out of L2); workgroup 0 stores it to pre.x_out if that is set.
constexpr int GEMV_AHEAD = 8;
// LDS (160 KB): x, and for the sum of the parts of h 2 KB behind it; a vector so long that it leaves no room for those (K above
// 80896) has them in its place once the product is done (PARTS_LAST).
constexpr size_t LDS_PER_CU = 160 * 1024;
constexpr int GEMV_MAX_K = (int)(LDS_PER_CU - 16 * sizeof(float)) / 2;     // x beside the block sums
__host__ __device__ constexpr size_t gemv_x_bytes(int K) { return ((size_t)K * 2 + 15) & ~(size_t)15; }
__host__ __device__ constexpr bool gemv_parts_fit(int K) { return gemv_x_bytes(K) + 512 * sizeof(float) <= LDS_PER_CU; }

// A long row's product with x, w0 holding this lane's share of its first 4096 columns: eight loads ahead of the eight that
// are being added up.  A last trip of fewer pieces of 512 columns loads two, four, six or eight of them (one token of two 5120-wide
// layers: 431 us with eight, 406 with two); what a lane or a piece has behind the end of the row is left out of the sum.
template <int NB>
__device__ __forceinline__ void gemv_load(uint4 (&wv)[GEMV_AHEAD], const bf16_t* w, int K, int lane, int k) {
#pragma unroll
    for (int u = 0; u < NB; ++u) wv[u] = load_w16(w + min(k + u * 512 + lane * 8, K - 8));
    __builtin_amdgcn_sched_barrier(0);
}
template <int NB>
__device__ __forceinline__ float gemv_add(const uint4 (&wv)[GEMV_AHEAD], const bf16_t* sx, int K, int lane, int k, float acc) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int kk = k + u * 512 + lane * 8;
        float b[8];
        unpack8(*(const uint4*)(sx + min(kk, K - 8)), b);
        acc = kk < K ? dot8(wv[u], b, acc) : acc;
    }
    return acc;
}
__device__ __forceinline__ float gemv_row(const bf16_t* w, const bf16_t* sx, int K, int lane, uint4 (&w0)[GEMV_AHEAD]) {
    constexpr int NB = GEMV_AHEAD, STEP = NB * 512;
    uint4 w1[NB];
    float acc = 0.f;
    // the trip at k, held in a, and behind it the last one, to be fetched into b; false if there is more than that
    auto last = [&](uint4 (&a)[NB], uint4 (&b)[NB], int k) {
        const int left = K - k - STEP;
        auto end = [&](auto n) {
            constexpr int NT = decltype(n)::value;
            gemv_load<NT>(b, w, K, lane, k + STEP);
            acc = gemv_add<NT>(b, sx, K, lane, k + STEP, gemv_add<NB>(a, sx, K, lane, k, acc));
        };
        if (left > STEP) return false;
        if (left <= 0) acc = gemv_add<NB>(a, sx, K, lane, k, acc);
        else if (left <= 1024) end(std::integral_constant<int, 2>{});
        else if (left <= 2048) end(std::integral_constant<int, 4>{});
        else if (left <= 3072) end(std::integral_constant<int, 6>{});
        else end(std::integral_constant<int, 8>{});
        return true;
    };
    for (int k = 0;; k += 2 * STEP) {
        if (last(w0, w1, k)) break;
        gemv_load<NB>(w1, w, K, lane, k + STEP);
        acc = gemv_add<NB>(w0, sx, K, lane, k, acc);
        if (last(w1, w0, k + STEP)) break;
        gemv_load<NB>(w0, w, K, lane, k + 2 * STEP);
        acc = gemv_add<NB>(w1, sx, K, lane, k + STEP, acc);
    }
    return acc;
}

template <int R, int MODE, bool PARTS_LAST = false>
__global__ __launch_bounds__(256, R == 1 ? 4 : 3) void gemv_kernel(const bf16_t* __restrict__ W, long ldw,
                                                                   const bf16_t* __restrict__ x, int N, int K, GemvLora lora,
                                                                   float alpha, const float* __restrict__ resid,
                                                                   bf16_t* __restrict__ y_bf, float* __restrict__ y_f32,
                                                                   GemvPre pre) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float red[16];
    bf16_t* sx = (bf16_t*)smem;
    float *hp = (float*)(smem + (PARTS_LAST ? 0 : gemv_x_bytes(K))), *hs = hp + 256;        // only with lora.n_parts
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows = N + lora.n_a, n0 = ((int)blockIdx.x * 4 + wave) * R;

    // A norm's operands are asked for first (loads return in order), if they fit; a longer row is normed first, instead of
    // waiting behind the weights for every piece of it (one token of two 4608-wide layers 376 -> 357 us, of one 8192-wide 486 ->
    // 478).
    constexpr int NV = 4;
    const bool short_row = MODE == 1 && K <= 1024 * NV;
    auto emit = [&](int i, const float4& v, const float4& g, float rho) {
        uint2 o;
        o.x = pack_bf16x2(v.x * rho * g.x, v.y * rho * g.y);
        o.y = pack_bf16x2(v.z * rho * g.z, v.w * rho * g.w);
        *(uint2*)(sx + i) = o;
    };
    if (MODE == 1 && !short_row) {
        float ss = 0.f;
        for (int i = threadIdx.x * 4; i < K; i += 1024) {
            const float4 v = *(const float4*)(pre.h + i);
            ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
        ss = block_sum(ss, red);
        const float rho = rsqrtf(ss / (float)K + pre.eps);
        for (int i = threadIdx.x * 4; i < K; i += 1024) emit(i, *(const float4*)(pre.h + i), *(const float4*)(pre.gain + i), rho);
    }
    float4 hv[NV], gv[NV];
    if (short_row) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x * 4 + 1024 * j;
            if (1024 * j >= K) break;
            hv[j] = *(const float4*)(pre.h + min(i, K - 4));
            gv[j] = *(const float4*)(pre.gain + min(i, K - 4));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const bf16_t* w[R];
    uint4 wv[R][GEMV_AHEAD];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const long n = min(n0 + i, rows - 1);        // rows past the end repeat the last one and are not stored
        w[i] = n < N ? W + n * ldw : lora.a + (n - N) * K;
#pragma unroll
        for (int u = 0; u < GEMV_AHEAD; ++u) {
            const int k = lane * 8 + u * 512;
            wv[i][u] = load_w16(w[i] + min(k, K - 8));      // (no branch around a load; left out of the sum below)
        }
    }
    // this lane's element of the rows of B
    bf16_t bv[R];
#pragma unroll
    for (int i = 0; i < R; ++i) bv[i] = lora.b ? lora.b[(long)min(n0 + i, rows - 1) * lora.r + min(lane, lora.r - 1)] : (bf16_t)0;
    // h from its parts: 256 / r threads per entry.  (All of it, and a given x, in registers ahead of the weights or right
    // behind them was slower, 9 -> 12 us for o and 21 -> 31 for down.)
    const int hg = lora.n_parts > 0 ? 256 / lora.r : 0;
    float hsum = 0.f;
    if ((int)threadIdx.x < hg * lora.r) {
        const int j = threadIdx.x % lora.r, g = threadIdx.x / lora.r;
        for (int p0 = g; p0 < lora.n_parts; p0 += 8 * hg) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = lora.h[(long)min(p0 + u * hg, lora.n_parts - 1) * lora.r + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) hsum += p0 + u * hg < lora.n_parts ? t[u] : 0.f;
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    if constexpr (MODE == 1) {
        if (short_row) {
            float ss = 0.f;
#pragma unroll
            for (int j = 0; j < NV; ++j)
                if ((int)threadIdx.x * 4 + 1024 * j < K) ss += hv[j].x * hv[j].x + hv[j].y * hv[j].y + hv[j].z * hv[j].z + hv[j].w * hv[j].w;
            ss = block_sum(ss, red);
            const float rho = rsqrtf(ss / (float)K + pre.eps);
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int i = threadIdx.x * 4 + 1024 * j;
                if (i < K) emit(i, hv[j], gv[j], rho);
            }
        }
    } else {
        for (int i = threadIdx.x * 8; i < K; i += 2048) *(uint4*)(sx + i) = *(const uint4*)(x + i);
    }
    if (hg && !PARTS_LAST) hp[threadIdx.x] = hsum;
    __syncthreads();
    if (pre.x_out && blockIdx.x == 0)
        for (int i = threadIdx.x * 8; i < K; i += 2048) *(uint4*)(pre.x_out + i) = *(const uint4*)(sx + i);
    auto add_parts = [&] {
        if ((int)threadIdx.x < lora.r) {
            float h = 0.f;
            for (int g = 0; g < hg; ++g) h += hp[g * lora.r + threadIdx.x];
            hs[threadIdx.x] = lora.scale * h;
        }
        __syncthreads();
    };
    if (hg && !PARTS_LAST) add_parts();
    if (n0 >= rows && !PARTS_LAST) return;      // (with PARTS_LAST the barriers below are for every wave)

    float acc[R];
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = 0.f;
    if (K > GEMV_AHEAD * 512) {
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i] = gemv_row(w[i], sx, K, lane, wv[i]);
    } else {
#pragma unroll
        for (int u = 0; u < GEMV_AHEAD; ++u) {
            const int k = lane * 8 + u * 512;
            float b[8];
            unpack8(*(const uint4*)(sx + min(k, K - 8)), b);
#pragma unroll
            for (int i = 0; i < R; ++i) acc[i] = k < K ? dot8(wv[i][u], b, acc[i]) : acc[i];
        }
    }
    if (PARTS_LAST) {
        __syncthreads();                                // x has been read
        hp[threadIdx.x] = hsum;
        __syncthreads();
        add_parts();
    }
    if (lora.b) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int n = min(n0 + i, rows - 1);
            const bf16_t* b = lora.b + (long)n * lora.r;
            if (lane < lora.r) acc[i] += bf16_to_f32(bv[i]) * hs[lane];
            for (int j = lane + 64; j < lora.r; j += 64) acc[i] += bf16_to_f32(b[j]) * hs[j];
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const float sum = wave_sum(acc[i]), v = alpha * sum;
        const int n = n0 + i;
        if (lane != 0 || n >= rows) continue;
        if (n >= N) lora.h_out[n - N] = lora.scale * sum;
        else if (y_f32) y_f32[n] = v + (resid ? resid[n] : 0.f);
        else y_bf[n] = f32_to_bf16(v);
    }
}

// The same product for a call that stands alone (a given vector or a SwiGLU; h, if any, is read as it is, one for every
// rows_per_group rows), and for few long rows behind a norm: x first, then one row per wave with four loads in flight, or one row
// per workgroup where there are at most 512 of them, so that a row's loads are all in flight at once instead of queued behind one
// wave.  Few registers, so that the next launch's workgroups are on the chip while this one's finish: back to back, cold
// weights, against gemv_kernel: 512 rows of 11008 5.8 and 7.3 us, 64 rows of 28672 8.5 and 12.7; 12288 rows of 256 6.1 and 8.5;
// 32000 rows of 4096 40.6 and 43.8.  In a chain of launches that wait for each other, as lm_head behind its norm, the other
// kernel's early loads are worth more (51.7 and 41.7 us; 1000 rows of 256: 6 us of a token's 95).
// pre.mode as for gemv_kernel, and 2: SwiGLU of a gate|up row, x = bf16(silu(g) u).
__global__ __launch_bounds__(256) void gemv_plain_kernel(const bf16_t* __restrict__ W, long ldw, const bf16_t* __restrict__ x,
                                                         int N, int K, GemvLora lora, float alpha, const float* __restrict__ resid,
                                                         bf16_t* __restrict__ y_bf, float* __restrict__ y_f32, GemvPre pre,
                                                         int row_per_block) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float red[16];
    bf16_t* sx = (bf16_t*)smem;
    if (pre.mode == 1) {
        float ss = 0.f;
        for (int i = threadIdx.x * 4; i < K; i += 1024) {
            const float4 v = *(const float4*)(pre.h + i);
            ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
        ss = block_sum(ss, red);
        const float rho = rsqrtf(ss / (float)K + pre.eps);
        for (int i = threadIdx.x * 4; i < K; i += 1024) {
            const float4 v = *(const float4*)(pre.h + i), w = *(const float4*)(pre.gain + i);
            uint2 o;
            o.x = pack_bf16x2(v.x * rho * w.x, v.y * rho * w.y);
            o.y = pack_bf16x2(v.z * rho * w.z, v.w * rho * w.w);
            *(uint2*)(sx + i) = o;
        }
    } else if (pre.mode == 2) {
        for (int i = threadIdx.x * 8; i < K; i += 2048) {
            float g[8], u[8], o[8];
            unpack8(*(const uint4*)(pre.gu + i), g);
            unpack8(*(const uint4*)(pre.gu + K + i), u);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = g[e] / (1.f + __expf(-g[e])) * u[e];
            *(uint4*)(sx + i) = pack8(o);
        }
    } else {
        for (int i = threadIdx.x * 8; i < K; i += 2048) *(uint4*)(sx + i) = *(const uint4*)(x + i);
    }
    __syncthreads();
    if (pre.x_out && blockIdx.x == 0)
        for (int i = threadIdx.x * 8; i < K; i += 2048) *(uint4*)(pre.x_out + i) = *(const uint4*)(sx + i);
    // the lanes of a row: t of nt
    const int nt = row_per_block ? 256 : 64, t = threadIdx.x & (nt - 1);
    const int n = row_per_block ? blockIdx.x : blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;                                  // (whole waves of the last workgroup, never of a row per workgroup)
    const bf16_t* w = W + (long)n * ldw;
    float acc = 0.f;
    auto add = [&](const uint4& wv, int k) {
        float b[8];
        unpack8(*(const uint4*)(sx + k), b);
        acc = dot8(wv, b, acc);
    };
    if (row_per_block) {
        for (int k = t * 8; k < K; k += 2048) add(*(const uint4*)(w + k), k);
    } else {
        int k = t * 8;
        for (; k + 3 * 512 < K; k += 4 * 512) {
            uint4 wv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) wv[u] = load_w16(w + k + u * 512);
#pragma unroll
            for (int u = 0; u < 4; ++u) add(wv[u], k + u * 512);
        }
        for (; k < K; k += 512) add(load_w16(w + k), k);
    }
    if (lora.b) {
        const float* h = lora.h + (long)(n / lora.rows_per_group) * lora.r;
        const bf16_t* b = lora.b + (long)n * lora.r;
        for (int j = t; j < lora.r; j += nt) acc += bf16_to_f32(b[j]) * h[j];
    }
    acc = row_per_block ? block_sum(acc, red) : wave_sum(acc);
    if (t == 0) {
        const float v = alpha * acc;
        if (y_f32) y_f32[n] = v + (resid ? resid[n] : 0.f);
        else y_bf[n] = f32_to_bf16(v);
    }
}

hipError_t launch_gemv(const bf16_t* W, long ldw, const bf16_t* x, int N, int K, const GemvLora& lora, float alpha,
                       const float* resid, bf16_t* y_bf, float* y_f32, hipStream_t s, const GemvPre* pre) {
    if (N <= 0) return hipSuccess;
    if ((K & 7) || (ldw & 7) || K <= 0 || K > GEMV_MAX_K || (!y_bf && !y_f32)) return hipErrorInvalidValue;
    GemvPre p = pre ? *pre : GemvPre{};
    if (p.mode < 0 || p.mode > 2 || (p.mode == 0 && !x) || (p.mode == 1 && (!p.h || !p.gain)) || (p.mode == 2 && !p.gu))
        return hipErrorInvalidValue;
    GemvLora lo = lora;
    if (lo.rows_per_group <= 0) lo.rows_per_group = N;
    if (lo.n_a > 0 ? (!lo.a || !lo.h_out || lo.b) : (lo.b && (!lo.h || lo.r < 1))) return hipErrorInvalidValue;
    if (lo.n_parts > 0 && (p.mode != 0 || !lo.b || lo.r > 256 || lo.rows_per_group < N)) return hipErrorInvalidValue;   // summed for one group
    const bool alone = lo.n_a == 0 && lo.n_parts == 0 && (lo.b || p.mode != 1 || (N <= 512 && K > 4096));
    const size_t lds = gemv_x_bytes(K) + (lo.n_parts > 0 && gemv_parts_fit(K) ? 512 * sizeof(float) : 0);
    auto run = [&](auto kern, int grid, auto... more) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        kern<<<grid, 256, lds, s>>>(W, ldw, x, N, K, lo, alpha, resid, y_bf, y_f32, p, more...);
        return hipGetLastError();
    };
    if (alone) return run(gemv_plain_kernel, N <= 512 ? N : cdiv(N, 4), (int)(N <= 512));
    if (p.mode == 2) return hipErrorInvalidValue;
    // Two rows per wave halve the number of times the input vector is formed; worth it while that leaves every CU a few
    // workgroups.
    const bool two = N >= 8192;
    const int grid = cdiv((long)N + lo.n_a, two ? 8 : 4);
    if (p.mode == 0 && !gemv_parts_fit(K)) return run(gemv_kernel<1, 0, true>, cdiv(N, 4));
    if (p.mode == 0) return two ? run(gemv_kernel<2, 0>, grid) : run(gemv_kernel<1, 0>, grid);
    return two ? run(gemv_kernel<2, 1>, grid) : run(gemv_kernel<1, 1>, grid);
}

// ---------------------------------------------------------------- SwiGLU of one token
// DECODE_SW columns of act per workgroup: gate and up rows get their low-rank term (raw + B h, rounded to bf16 as the chunk
// path keeps them), act = bf16(silu(g) u), and the piece's share of the down projection's A act goes to
// part[blockIdx.x * r + j] (summed by gemv_kernel).
__global__ __launch_bounds__(256) void decode_swiglu_kernel(const float* __restrict__ raw, const bf16_t* __restrict__ b,
                                                            const float* __restrict__ h, int r, int f, bf16_t* __restrict__ act,
                                                            const bf16_t* __restrict__ a_down, float* __restrict__ part) {
    static_assert(DECODE_SW == 128, "256 threads: gate and up of 128 columns; 16 lanes per row of A");
    __shared__ float gu[256], sa[DECODE_SW];
    const int c0 = blockIdx.x * DECODE_SW, c = threadIdx.x & 127, which = threadIdx.x >> 7;
    const int sub = threadIdx.x & 15, jj = threadIdx.x >> 4, left = f - c0;
    uint4 av[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        av[i] = *(const uint4*)(a_down + (long)min(jj + 16 * i, r - 1) * f + c0 + min(sub * 8, left - 8));
    {
        const long n = (long)which * f + min(c0 + c, f - 1);
        float v = 0.f;
        for (int j0 = 0; j0 < r; j0 += 64) {
            uint4 bv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) bv[i] = *(const uint4*)(b + n * r + min(j0 + 8 * i, r - 8));
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float t[8];
                unpack8(bv[i], t);
                if (j0 + 8 * i < r)
#pragma unroll
                    for (int e = 0; e < 8; ++e) v += t[e] * h[which * r + j0 + 8 * i + e];
            }
        }
        gu[threadIdx.x] = bf16_to_f32(f32_to_bf16(raw[n] + v));
    }
    __syncthreads();
    if (threadIdx.x < DECODE_SW) {
        const float g = gu[c], v = g / (1.f + __expf(-g)) * gu[128 + c];
        const bf16_t o = f32_to_bf16(v);
        if (c0 + c < f) act[c0 + c] = o;
        sa[c] = c0 + c < f ? bf16_to_f32(o) : 0.f;
    }
    __syncthreads();
    lowrank_part<DECODE_SW, 256, 4>(a_down + c0, f, r, sa, left, av, part + (long)blockIdx.x * r);
}
hipError_t launch_decode_swiglu(const float* raw, const bf16_t* b, const float* h, int r, int f, bf16_t* act,
                                const bf16_t* a_down, float* part, hipStream_t s) {
    if (f <= 0 || (f & 7) || r < 8 || (r & 7)) return hipErrorInvalidValue;
    decode_swiglu_kernel<<<cdiv(f, DECODE_SW), 256, 0, s>>>(raw, b, h, r, f, act, a_down, part);
    return hipGetLastError();
}

// ---------------------------------------------------------------- attention of one query against the cache
// q: the query row (already rotated); K, V: rows 0 .. n_keys-1 of the cache with row stride ld (the layout q|k|v of
// the chunk path, so the cache IS the forward pass's saved projections).  Scores and the softmax are fp32; the
// output row is written in bf16.
//
// attend_range: one head against nk consecutive keys, by one workgroup of NW waves.  A key (or value) row of the head is
// DH * 2 contiguous bytes, read by DH / 8 adjacent lanes with one 16-byte load each; such a group of lanes takes its keys
// NP at a time, keys and values all in flight together (the loop is bound by load latency, not by bytes), and keeps a
// running maximum, sum and output of its own.  The groups are merged at the end: one barrier in all.  Leaves the
// unnormalised output in out[0 .. DH) of the first DH threads' `o`, with the maximum and the sum of exponentials.
// (1024 keys, 32 heads of 128: 7.7 us, against 11.0 with the scores in LDS, two block reductions and the values fetched after
// them; with the fresh token's rows formed as well 11.8.)
//
// fresh.raw != null: the token being decoded.  Its q, k and v do not exist yet as bf16 rows: they are raw + B h (fp32 sums,
// rounded to bf16), formed here -- q by every workgroup of the head, k and v by the one whose range ends with key `new_key`
// (-1: another range) -- and q and k are rotated with the (cos, sin) pairs of the token's position (RoPE pairs elements i
// and i + d_head / 2) and rounded to bf16 once more, as the chunk path's separate kernels would have stored them.  k and v
// are written to the cache for the tokens to come.
__device__ __forceinline__ void rope8(const float* mine, const float* other, const float2 (&row)[8], int sub, int lpk, float* out) {
    const bool first = sub < (lpk >> 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float2 cs = row[e];
        const float a = first ? mine[e] : other[e], b = first ? other[e] : mine[e];   // a: first-half element of the pair
        out[e] = bf16_to_f32(f32_to_bf16(first ? a * cs.x - b * cs.y : b * cs.x + a * cs.y));
    }
}
template <int DH, int NW>
__device__ __forceinline__ void attend_range(const bf16_t* __restrict__ qh, bf16_t* __restrict__ kh,
                                             bf16_t* __restrict__ vh, long ld, int nk, float scale,
                                             float& o, float& mx_out, float& sum_out, const DecodeFresh& fresh, int head,
                                             int new_key) {
    constexpr int LPK = DH / 8, KPW = 64 / LPK, KPP = NW * KPW;   // lanes per key, keys per wave and per pass
    constexpr int NP = NW > 4 ? 4 : 8;                                    // passes in flight (sixteen waves: 128 registers)
    __shared__ float part[NW][DH + 2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = lane % LPK, kk = wave * KPW + lane / LPK;
    const int psub = sub ^ (LPK >> 1);                                    // the lanes holding the pair partners
    __shared__ float row[3][DH];                                          // fresh q, k, v
    float2 cs[8];                                                         // this lane's share of the position's (cos, sin)
    uint4 kr[NP], vr[NP];
    auto fetch = [&](int u0) {
#pragma unroll
        for (int i = 0; i < NP; ++i) kr[i] = *(const uint4*)(kh + (long)min(u0 + i * KPP + kk, nk - 1) * ld + sub * 8);
#pragma unroll
        for (int i = 0; i < NP; ++i) vr[i] = *(const uint4*)(vh + (long)min(u0 + i * KPP + kk, nk - 1) * ld + sub * 8);
    };
    float qv[8], kn[8] = {}, vn[8] = {};                                  // kn, vn: the new key's and value's share
    fetch(0);
    __builtin_amdgcn_sched_barrier(0);
    if (fresh.raw) {
        // TPR threads per row of the head, each with every TPR-th eight of the row of B
        constexpr int TPR = NW * 64 / DH;
        const int c = tid / TPR, p = tid % TPR;
        float v[3] = {0.f, 0.f, 0.f}, raw[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) raw[x] = fresh.raw[(long)x * fresh.d + head * DH + c];
#pragma unroll
        for (int e = 0; e < 8; ++e) cs[e] = fresh.rope[sub % (LPK >> 1) * 8 + e];
        constexpr int NC = TPR >= 8 ? 1 : 8 / TPR;                        // pieces of eight per thread and trip: 64 of a row
        auto low = [&](auto rows) {               // every load of a trip before the first is used
            constexpr int NR = decltype(rows)::value;
            for (int j0 = 0; j0 < fresh.r; j0 += NC * TPR * 8) {
                uint4 bv[NR][NC];
                float4 ha[NR][NC], hb[NR][NC];
#pragma unroll
                for (int x = 0; x < NR; ++x)
#pragma unroll
                    for (int i = 0; i < NC; ++i) {
                        const int j = min(j0 + (i * TPR + p) * 8, fresh.r - 8);
                        bv[x][i] = *(const uint4*)(fresh.b + ((long)x * fresh.d + head * DH + c) * fresh.r + j);
                        ha[x][i] = *(const float4*)(fresh.h + x * fresh.r + j);
                        hb[x][i] = *(const float4*)(fresh.h + x * fresh.r + j + 4);
                    }
#pragma unroll
                for (int x = 0; x < NR; ++x)
#pragma unroll
                    for (int i = 0; i < NC; ++i) {
                        const float4 a = ha[x][i], b = hb[x][i];
                        const float hh[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                        v[x] = j0 + (i * TPR + p) * 8 < fresh.r ? dot8(bv[x][i], hh, v[x]) : v[x];
                    }
            }
        };
        if (new_key >= 0) low(std::integral_constant<int, 3>{}); else low(std::integral_constant<int, 1>{});
#pragma unroll
        for (int x = 0; x < 3; ++x) {
#pragma unroll
            for (int off = TPR >> 1; off > 0; off >>= 1) v[x] += __shfl_xor(v[x], off, 64);
            if (p == 0) row[x][c] = bf16_to_f32(f32_to_bf16(raw[x] + v[x]));
        }
        __syncthreads();
        rope8(row[0] + sub * 8, row[0] + psub * 8, cs, sub, LPK, qv);
        if (new_key >= 0) {
            rope8(row[1] + sub * 8, row[1] + psub * 8, cs, sub, LPK, kn);
#pragma unroll
            for (int e = 0; e < 8; ++e) vn[e] = row[2][sub * 8 + e];
            if (tid < LPK) {
                *(uint4*)(kh + (long)new_key * ld + sub * 8) = pack8(kn);
                *(uint4*)(vh + (long)new_key * ld + sub * 8) = pack8(vn);
            }
        }
    } else {
        unpack8(*(const uint4*)(qh + sub * 8), qv);
    }
    float m = -1.0e30f, l = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int u0 = 0; u0 < nk; u0 += NP * KPP) {
        if (u0 > 0) fetch(u0);
        __builtin_amdgcn_sched_barrier(0);
        float sc[NP], mloc = m;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int u = u0 + i * KPP + kk;
            float a[8], sdot = 0.f;
            unpack8(kr[i], a);
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] = u == new_key ? kn[e] : a[e];
#pragma unroll
            for (int e = 0; e < 8; ++e) sdot += a[e] * qv[e];
#pragma unroll
            for (int off = LPK >> 1; off > 0; off >>= 1) sdot += __shfl_xor(sdot, off, 64);
            sc[i] = u < nk ? sdot * scale : -1.0e30f;
            mloc = fmaxf(mloc, sc[i]);
        }
        const float alpha = __expf(m - mloc);
        m = mloc;
        l *= alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= alpha;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float pr = u0 + i * KPP + kk < nk ? __expf(sc[i] - m) : 0.f;
            float a[8];
            unpack8(vr[i], a);
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] = u0 + i * KPP + kk == new_key ? vn[e] : u0 + i * KPP + kk < nk ? a[e] : 0.f;
            l += pr;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = fmaf(pr, a[e], acc[e]);
        }
    }
    // merge the lane groups of a wave, then the waves (a group that had no key has m = -1e30 and zeros)
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
        const float mo = __shfl_xor(m, off, 64), lo = __shfl_xor(l, off, 64), mn = fmaxf(m, mo);
        const float a0 = __expf(m - mn), a1 = __expf(mo - mn);
        m = mn;
        l = l * a0 + lo * a1;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = acc[e] * a0 + __shfl_xor(acc[e], off, 64) * a1;
    }
    if (lane < LPK) {
#pragma unroll
        for (int e = 0; e < 8; ++e) part[wave][sub * 8 + e] = acc[e];
        if (lane == 0) { part[wave][DH] = m; part[wave][DH + 1] = l; }
    }
    __syncthreads();
    float mt = part[0][DH], lt = 0.f, ot = 0.f;
#pragma unroll
    for (int w = 1; w < NW; ++w) mt = fmaxf(mt, part[w][DH]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float a = __expf(part[w][DH] - mt);
        lt += a * part[w][DH + 1];
        ot += a * part[w][tid % DH];
    }
    o = ot;
    mx_out = mt;
    sum_out = lt;
}

// A head's output row, rounded, to memory, and with out.a its share of the output projection's A o (see lowrank_part).
// c: this thread's column; every thread of the workgroup (NT of them) takes part.
template <int DH, int NT, int NA>
__device__ __forceinline__ void head_output(float v, int c, int head, int n_heads, const DecodeOut& out, uint4 (&av)[NA]) {
    __shared__ float so[DH];
    const bf16_t b = f32_to_bf16(v);
    if ((int)threadIdx.x < DH) {
        out.o[(long)head * DH + c] = b;
        so[c] = bf16_to_f32(b);
    }
    if (!out.a) return;
    __syncthreads();
    lowrank_part<DH, NT, NA>(out.a + (long)head * DH, (long)n_heads * DH, out.r, so, DH, av, out.part + (long)head * out.r);
}
template <int DH, int NT, int NA>
__device__ __forceinline__ void head_output_fetch(int head, int n_heads, const DecodeOut& out, uint4 (&av)[NA]) {
    constexpr int LPR = DH / 8;
    if (!out.a) return;
#pragma unroll
    for (int i = 0; i < NA; ++i)
        av[i] = *(const uint4*)(out.a + (long)min((int)threadIdx.x / LPR + i * (NT / LPR), out.r - 1) * n_heads * DH + head * DH +
                                threadIdx.x % LPR * 8);
}

// One workgroup per head over the whole cache.
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64) void attn_decode_kernel(const bf16_t* __restrict__ q, bf16_t* __restrict__ k,
                                                              bf16_t* __restrict__ v, long ld, int n_keys, float scale,
                                                              DecodeOut out, DecodeFresh fresh) {
    const int head = blockIdx.x;
    float mx, sum, o;
    attend_range<DH, NW>(q + (long)head * DH, k + (long)head * DH, v + (long)head * DH, ld, n_keys, scale, o, mx, sum, fresh,
                         head, fresh.raw ? n_keys - 1 : -1);
    uint4 av[1];
    head_output_fetch<DH, NW * 64>(head, gridDim.x, out, av);
    head_output<DH, NW * 64>(o / sum, threadIdx.x % DH, head, gridDim.x, out, av);
}

// Long windows: the keys are cut into n_split ranges, one workgroup per (head, range), so that the cache is read by
// hundreds of workgroups instead of one per head.  Each writes its unnormalised output, its score maximum and its
// sum of exponentials to ws[(head * n_split + range) * (d_head + 2)]; attn_decode_combine_kernel merges the ranges.
template <int DH>
__global__ __launch_bounds__(256) void attn_decode_split_kernel(const bf16_t* __restrict__ q, bf16_t* __restrict__ k,
                                                                bf16_t* __restrict__ v, long ld, int n_keys, float scale,
                                                                int chunk, float* __restrict__ ws, DecodeFresh fresh) {
    const int head = blockIdx.x;
    const int k0 = blockIdx.y * chunk, nk = min(chunk, n_keys - k0);   // nk >= 1 by the launch geometry
    float mx, sum, o;
    const int new_key = n_keys - 1 - k0;                             // inside this range only for the last one
    attend_range<DH, 4>(q + (long)head * DH, k + (long)k0 * ld + (long)head * DH, v + (long)k0 * ld + (long)head * DH, ld, nk,
                        scale, o, mx, sum, fresh, head, fresh.raw && new_key < nk ? new_key : -1);
    float* out = ws + ((long)head * gridDim.y + blockIdx.y) * (DH + 2);
    if ((int)threadIdx.x < DH) out[threadIdx.x] = o;
    if (threadIdx.x == 0) { out[DH] = mx; out[DH + 1] = sum; }
}

// One workgroup per head, one thread per column.  Lane i holds range i's maximum and sum, and every load is issued before
// the first is used (one range after another, 32 of them took 15.9 us; now 8, with the share of A o).
template <int DH>
__global__ __launch_bounds__(DH) void attn_decode_combine_kernel(const float* __restrict__ ws, int n_split, DecodeOut out) {
    static_assert(ATTN_DECODE_MAX_SPLIT <= 32, "one lane per range");
    const int head = blockIdx.x, c = threadIdx.x, lane = threadIdx.x & 63, r = lane < n_split ? lane : n_split - 1;
    const float* w = ws + (long)head * n_split * (DH + 2);
    const float m = w[r * (DH + 2) + DH], l = w[r * (DH + 2) + DH + 1];
    float t[ATTN_DECODE_MAX_SPLIT];
#pragma unroll
    for (int i = 0; i < ATTN_DECODE_MAX_SPLIT; ++i) t[i] = w[min(i, n_split - 1) * (DH + 2) + c];
    uint4 av[8];
    head_output_fetch<DH, DH>(head, gridDim.x, out, av);
    __builtin_amdgcn_sched_barrier(0);
    const float M = wave_max(m);             // (all lanes take part in the exchange)
    const float e = lane < n_split ? __expf(m - M) : 0.f;
    const float L = wave_sum(e * l);
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < ATTN_DECODE_MAX_SPLIT; ++i) {
        const float ei = __shfl(e, i, 64);
        acc += i < n_split ? ei * t[i] : 0.f;
    }
    head_output<DH, DH>(acc / L, c, head, gridDim.x, out, av);
}

// ws (may be null): scratch of ws_elems floats for the split path; n_heads * n_split * (d_head + 2) of them are used.
// q is not read if `fresh` describes the newest token (then row n_keys - 1 of k and v is written).
template <int DH>
static hipError_t run_attention_decode(const bf16_t* q, bf16_t* k, bf16_t* v, long ld, int n_keys, int n_heads, int n_split,
                                       const DecodeOut& out, float* ws, hipStream_t s, const DecodeFresh& fresh) {
    const float scale = 1.f / sqrtf((float)DH);
    if (n_split >= 2) {
        const int chunk = cdiv(n_keys, n_split);
        if (chunk > ATTN_DECODE_MAX_RANGE) return hipErrorInvalidValue;
        n_split = cdiv(n_keys, chunk);            // no empty range
        attn_decode_split_kernel<DH><<<dim3(n_heads, n_split), 256, 0, s>>>(q, k, v, ld, n_keys, scale, chunk, ws, fresh);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        attn_decode_combine_kernel<DH><<<n_heads, DH, 0, s>>>(ws, n_split, out);
        return hipGetLastError();
    }
    if (n_keys > ATTN_DECODE_MAX_UNSPLIT) return hipErrorInvalidValue;
    if (n_keys > 128) attn_decode_kernel<DH, 16><<<n_heads, 1024, 0, s>>>(q, k, v, ld, n_keys, scale, out, fresh);
    else attn_decode_kernel<DH, 4><<<n_heads, 256, 0, s>>>(q, k, v, ld, n_keys, scale, out, fresh);
    return hipGetLastError();
}
hipError_t launch_attention_decode(const bf16_t* q, bf16_t* k, bf16_t* v, long ld, int n_keys, int n_heads, int d_head,
                                   const DecodeOut& out, float* ws, size_t ws_elems, hipStream_t s, const DecodeFresh& fresh) {
    if (n_keys <= 0 || n_heads <= 0) return hipErrorInvalidValue;
    if ((d_head != 64 && d_head != 128) || (ld & 7) || (out.a && (out.r & 7))) return hipErrorInvalidValue;
    // ranges of at least 128 keys, at most ATTN_DECODE_MAX_SPLIT of them, as many as the scratch holds
    // (below about 400 keys one workgroup per head is as fast and saves the second launch)
    int n_split = ws && n_keys >= 384 ? min(cdiv(n_keys, 128), ATTN_DECODE_MAX_SPLIT) : 1;
    if (ws && (size_t)n_heads * n_split * (d_head + 2) > ws_elems) n_split = (int)(ws_elems / ((size_t)n_heads * (d_head + 2)));
    // no more of them than are on the chip at once (two workgroups per CU), if that leaves none too long: those of a second round form
    // q and ask for their keys when the first is done (3800 keys, 32 heads: 30 ranges 22.2 us, 16 17.7)
    const int round = n_heads < 512 ? 512 / n_heads : 1;
    if (n_split > round && round >= 2 && cdiv(n_keys, round) <= ATTN_DECODE_MAX_RANGE) n_split = round;
    return d_head == 128 ? run_attention_decode<128>(q, k, v, ld, n_keys, n_heads, n_split, out, ws, s, fresh)
                         : run_attention_decode<64>(q, k, v, ld, n_keys, n_heads, n_split, out, ws, s, fresh);
}

// ---------------------------------------------------------------- greedy choice: index of the largest logit
// The lowest index wins among equal values.  One workgroup.
__global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ x, int n, int* __restrict__ out) {
    __shared__ float bv[16];
    __shared__ int bi[16];
    float best = -INFINITY;
    int idx = 0x7fffffff;
    auto take = [&](float v, int i) {
        if (v > best || (v == best && i < idx)) { best = v; idx = i; }
    };
    // sixteen bytes a time, eight loads in flight, one after another below 16384, where a trip of that is not worth it: 32000 values
    // 8.8 and 6.4 us, 16384 6.2 and 6.3, 8192 4.8 and 6.3, 100 3.4 and 4.6
    const int n4 = n >= 16384 && ((size_t)x & 15) == 0 ? n & ~3 : 0;
    for (int i0 = threadIdx.x * 4; i0 < n4; i0 += 8 * 4096) {
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = *(const float4*)(x + min(i0 + 4096 * j, n4 - 4));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = min(i0 + 4096 * j, n4 - 4);
            take(v[j].x, i); take(v[j].y, i + 1); take(v[j].z, i + 2); take(v[j].w, i + 3);
        }
    }
    for (int i = n4 + threadIdx.x; i < n; i += blockDim.x) take(x[i], i);
    for (int off = 32; off > 0; off >>= 1) {
        const float ov = __shfl_xor(best, off, 64);
        const int oi = __shfl_xor(idx, off, 64);
        if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { bv[w] = best; bi[w] = idx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < (int)(blockDim.x >> 6); ++k)
            if (bv[k] > best || (bv[k] == best && bi[k] < idx)) { best = bv[k]; idx = bi[k]; }
        *out = idx;
    }
}

hipError_t launch_argmax(const float* x, int n, int* out, hipStream_t s) {
    if (n <= 0) return hipErrorInvalidValue;
    argmax_kernel<<<1, 1024, 0, s>>>(x, n, out);
    return hipGetLastError();
}
