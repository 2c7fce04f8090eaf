// fp32 products of the single fp32 LoRA-adapted linear step, on the fp32 matrix instructions (inputs, products and sums all
// fp32).  Several independent products C = alpha (A B^T + A2 B2^T) of three operand layouts share a launch:
//   F32_KK  A [M, K], B [N, K]: the contraction is contiguous in both          (X A^T;  X W^T + H B^T)
//   F32_KN  A [M, K], B [K, N]                                                 (dY B;   dY W + dH A)
//   F32_MN  A [K, M], B [K, N]                                                 (dH^T X; dY^T H)
//
// v_mfma_f32_16x16x4_f32 adds its four products in ascending order, each as one fused multiply-add: an output is the plain
// chain fma(a[k], b[k], ..) over k, the same value wherever its tile boundaries lie.  (So no contraction is split, and the
// low-rank term is a chain of its own, added to the stored main term.)  Lane (l16, g) holds row l16, element g of the four:
// one float per operand.  An operand whose contraction is contiguous is kept in LDS as it comes, [row][k], with a stride
// that lets the 64 lanes of a read touch 64 banks; one whose rows (or columns) are contiguous as [k][row], and a lane reads
// F neighbouring rows at once, one for each of the F fragments of its wave's share (the output is written with that order
// undone).  Neither is transposed on the way.
//
// The bound is the matrix unit: 256 flop per clock and CU, a sixteenth of the bf16 rate, so that LDS reads are cheap beside
// it and tiles staged through registers are enough.  Measured, one step of 1024 tokens, 4096 x 4096, rank 64: 3.89 ms with
// 4 x 4 outputs per thread on the vector unit and thirteen launches, 0.69 ms here in two (100 of 157 TFLOP/s); the same bits.
// 128 tokens, 256 x 256, rank 8: 263 -> 36 us, of which the two kernels are 15.
#include "kernels.h"
#include <type_traits>

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // rows start at any multiple of a float

struct F32Batch {
    F32Product p[F32_GROUP_MAX];
    int n;
};

// The gradients of the factors (F32_MN) have a side of rank elements: 64 wide at most.  A few full tiles of them beside a
// chip's worth of large ones would also be the last to finish.
constexpr int F32_MN_TILE(int b) { return b < 64 ? b : 64; }

// BM x BN outputs per workgroup of 2 x 2 waves, BKF contraction elements per tile.
template <int BM, int BN, int BKF>
struct F32Tile {
    static constexpr int TM = BM / 2, TN = BN / 2, FM = TM / 16, FN = TN / 16;
    // floats per buffer, kept as [row][k + 4] or [k][row + 4]
    static constexpr int SA = BM * BKF + 4 * (BM > BKF ? BM : BKF), SB = BN * BKF + 4 * (BN > BKF ? BN : BKF);
    static constexpr int LDS_FLOATS = 3 * (SA + SB);
    static_assert(FM >= 1 && FN >= 1 && BKF % 16 == 0, "tile shape");
};

// One operand's share of a contraction tile, global memory -> registers -> LDS.  The loads go through a buffer resource that
// starts at the tile and ends with the operand: what lies behind its end reads as zero, so there is no branch around a load
// and the compiler can count exactly which of them a use has to wait for.  WIDE: rows of more than 2^22 floats, whose offsets
// within a tile do not fit the resource's 32 bits; plain loads with their own look at the operand's end (64 tokens, 4194312 x 64,
// rank 8: 0.21 s; one output per thread 2.9 to 3.2).
template <int B, int BKF, bool KC, bool WIDE>     // B rows (or columns); KC: the contraction is contiguous
struct F32Stage {
    static constexpr int CPR = (KC ? BKF : B) / 4, STEP = 256 / CPR, N = B * BKF / 1024;
    u32x4_t r[N];
    // rows r0 .. of `rows`, contraction elements k0 .. of kmax.  Columns past the end of a row of the [k][row] layout come
    // out of the next row: they, like rows past the end, only feed outputs that are never stored.
    __device__ __forceinline__ void load(const float* src, long ld, int r0, int rows, int k0, int kmax, int tid) {
        const long at = KC ? r0 * ld + k0 : k0 * ld + r0, end = KC ? (rows - 1) * ld + kmax : (kmax - 1) * ld + rows;
        if constexpr (WIDE) {
            const float* first = src + at;
            const long left = (unsigned)k0 < (unsigned)kmax ? end - at : 0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const long off = (tid / CPR + (long)STEP * i) * ld + (tid % CPR) * 4;
                f4u v = {0.f, 0.f, 0.f, 0.f};
                if (off + 4 <= left) {
                    v = *(const f4u*)(first + off);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (off + e < left) v[e] = first[off + e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) r[i][e] = __float_as_uint(v[e]);
            }
            return;
        }
        const long left = (unsigned)k0 < (unsigned)kmax ? (end - at) * 4 : 0;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(src + (left > 0 ? at : 0)), 0,
                                                            (int)(unsigned)(left > 0xffffffffL ? 0xffffffffL : left), 0x00020000);
        const unsigned off = ((unsigned)(tid / CPR) * (unsigned)ld + (tid % CPR) * 4) * 4, step = (unsigned)ld * (STEP * 4);
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + i * step, 0, 0);
    }
    __device__ __forceinline__ void store(float* tile, int k0, int kmax, int tid) {
        const int c = (tid % CPR) * 4, o = tid / CPR;
        constexpr int LD = KC ? BKF + 4 : B + 4;
        if (KC && k0 > kmax - BKF) {         // elements past the contraction's end belong to the next row: they count as zero
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) r[i][e] = c + e < kmax - k0 ? r[i][e] : 0u;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) *(u32x4_t*)(tile + (o + STEP * i) * LD + c) = r[i];
    }
};
// fragments of 16 contraction elements starting at k: v[i][j] = fragment i, element 4 j + g
template <int B, int BKF, int F, bool KC>
__device__ __forceinline__ void f32_fragments(const float* tile, int row0, int k, int l16, int g, float (&v)[F][4]) {
    if constexpr (KC) {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[i][j] = tile[(row0 + 16 * i + l16) * (BKF + 4) + k + 4 * j + g];
    } else {
        typedef float fvec __attribute__((ext_vector_type(F)));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const fvec t = *(const fvec*)(tile + (k + 4 * j + g) * (B + 4) + row0 + F * l16);
#pragma unroll
            for (int i = 0; i < F; ++i) v[i][j] = t[i];
        }
    }
}

template <int BM, int BN, int BKF, int PF, bool WIDE, bool AKC, bool BKC>
__device__ __forceinline__ void f32_tile(const F32Product& q, int tile, float* smem) {
    using T = F32Tile<BM, BN, BKF>;
    constexpr int FM = T::FM, FN = T::FN, KS = BKF / 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, g = lane >> 4;
    const int m0 = tile % q.tiles_m * BM, n0 = tile / q.tiles_m * BN;
    float *sA = smem, *sB = smem + 3 * T::SA;
    // First the main term, stored; then, for a product that has one, the low-rank term, added to what this thread stored.
#pragma unroll 1
    for (int term = 0; term < (q.K2 > 0 ? 2 : 1); ++term) {
        const float *A = term ? q.A2 : q.A, *B = term ? q.B2 : q.B;
        const long lda = term ? q.lda2 : q.lda, ldb = term ? q.ldb2 : q.ldb;
        const int K = term ? q.K2 : q.K, nk = (K + BKF - 1) / BKF;
        const int M = q.M, N = q.N;               // (values, not reloads behind every barrier)
        // Tile t goes from memory to the staging registers of slot t % PF, from there to place t % 3 of the LDS ring, and its
        // fragments to set t % 2: while tile t is multiplied the fragments of t + 1 are read, t + 2 is put into LDS and t + 3
        // .. t + 2 + PF are in flight.  One barrier per tile: it makes t + 2 visible and frees the place of t + 1.
        F32Stage<BM, BKF, AKC, WIDE> ra[PF];
        F32Stage<BN, BKF, BKC, WIDE> rb[PF];
        // (128-wide tiles have sixteen independent chains to hide the LDS behind, and no registers for a second set: they read
        // a tile's fragments when they multiply it)
        constexpr bool AHEAD = BM < 128;
        float a[AHEAD ? 2 : 1][KS][FM][4], b[AHEAD ? 2 : 1][KS][FN][4];
        f32x4_t acc[FM][FN];
        // (tiles behind the last one read as zeros and are never multiplied; their first element may lie beyond 2^31)
        auto tile_k = [](int t) { return (int)((unsigned)t * BKF); };
        auto load = [&](auto slot, int t) {
            ra[slot.value].load(A, lda, m0, M, tile_k(t), K, tid);
            rb[slot.value].load(B, ldb, n0, N, tile_k(t), K, tid);
        };
        auto park = [&](auto slot, int place, int t) {
            ra[slot.value].store(sA + place * T::SA, tile_k(t), K, tid);
            rb[slot.value].store(sB + place * T::SB, tile_k(t), K, tid);
        };
        auto fetch = [&](auto set, int place) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                f32_fragments<BM, BKF, FM, AKC>(sA + place * T::SA, wm * T::TM, ks * 16, l16, g, a[set.value][ks]);
                f32_fragments<BN, BKF, FN, BKC>(sB + place * T::SB, wn * T::TN, ks * 16, l16, g, b[set.value][ks]);
            }
        };
        using S0 = std::integral_constant<int, 0>; using S1 = std::integral_constant<int, 1>;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        using S2 = std::integral_constant<int, 2>; using S3 = std::integral_constant<int, 3>;
        load(S0{}, 0);
        load(S1{}, 1);
        if constexpr (PF == 4) { load(S2{}, 2); load(S3{}, 3); }
        park(S0{}, 0, 0);
        load(S0{}, PF);
        park(S1{}, 1, 1);
        load(S1{}, PF + 1);
        __syncthreads();
        if constexpr (AHEAD) fetch(S0{}, 0);
        int p0 = 0, p1 = 1, p2 = 2;               // places of tiles t, t + 1 and t + 2
        auto step = [&](auto u, int t) {          // u = t % PF
            using cur = std::integral_constant<int, AHEAD ? u.value & 1 : 0>;
            using slot = std::integral_constant<int, (u.value + 2) % PF>;
            if constexpr (AHEAD) fetch(std::integral_constant<int, cur::value ^ 1>{}, p1); else fetch(cur{}, p0);
            park(slot{}, p2, t + 2);
            load(slot{}, t + 2 + PF);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int jn = 0; jn < FN; ++jn)   // B first: a lane then holds row l16 of A's fragment, four columns
                            acc[i][jn] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[cur::value][ks][jn][j], a[cur::value][ks][i][j],
                                                                              acc[i][jn], 0, 0, 0);
            __syncthreads();
            const int p = p0;
            p0 = p1; p1 = p2; p2 = p;
        };
        for (int t = 0; t < nk; t += PF) {
            step(S0{}, t);
            if (t + 1 >= nk) break;
            step(S1{}, t + 1);
            if constexpr (PF == 4) {
                if (t + 2 >= nk) break;
                step(S2{}, t + 2);
                if (t + 3 >= nk) break;
                step(S3{}, t + 3);
            }
        }
        __syncthreads();                          // the places of the ring are free for the next term
        const float alpha = term ? q.alpha2 : q.alpha;

        // Output, four neighbouring columns of a row at a time: run r of row fragment i holds fragment r's columns 4 g .. 4 g + 3
        // (contiguous contraction), or columns FN (4 g) + 4 r .. + 3 of the wave's share, which interleaves the fragments.
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int r = 0; r < FN; ++r) {
                const int m = m0 + wm * T::TM + (AKC ? 16 * i + l16 : FM * l16 + i);
                const int n = n0 + wn * T::TN + (BKC ? 16 * r + 4 * g : 4 * FN * g + 4 * r);
                if (m >= q.M || n >= q.N) continue;
                float* dst = q.C + (long)m * q.ldc + n;
                const bool vec = n + 4 <= q.N;
                f4u v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = alpha * (BKC ? acc[i][r][e] : acc[i][(4 * r + e) % FN][(4 * r + e) / FN]);
                if (term) {
                    if (vec) {
                        const f4u c = *(const f4u*)dst;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += c[e];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (n + e < q.N) v[e] += dst[e];
                    }
                }
                if (vec) {
                    *(f4u*)dst = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < q.N) dst[e] = v[e];
                }
                if (q.p_new) {
                    const float* po = q.p_old + (long)m * q.ldc + n;
                    float* pn = q.p_new + (long)m * q.ldc + n;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < q.N) pn[e] = adamw_first(po[e], v[e], q.opt);
                }
            }
    }
}

template <int BM, int BN, int BKF, int PF, bool WIDE>
__global__ __launch_bounds__(256, 2) void f32_group_kernel(F32Batch grp) {
    extern __shared__ __align__(16) float smem_f32[];
    const int b = blockIdx.x;
    int k = 0;
    while (k + 1 < grp.n && b >= grp.p[k + 1].tile0) ++k;
    const F32Product& q = grp.p[k];
    // Workgroup ids go round-robin over the 8 XCDs: each gets a contiguous range of the product's tiles (rows fastest), so
    // that the CUs of one XCD share operand rows in its L2.
    const int n = q.tiles_m * q.tiles_n, id = b - q.tile0;
    const int c = id & 7, per = n >> 3, tile = c * per + min(c, n & 7) + (id >> 3);
    if (q.kind == F32_KK) f32_tile<BM, BN, BKF, PF, WIDE, true, true>(q, tile, smem_f32);
    else if (q.kind == F32_KN) f32_tile<BM, BN, BKF, PF, WIDE, true, false>(q, tile, smem_f32);
    else f32_tile<F32_MN_TILE(BM), F32_MN_TILE(BN), BKF, PF, WIDE, false, false>(q, tile, smem_f32);
}

__global__ __launch_bounds__(256) void adamw_first_kernel(const float* __restrict__ g, const float* p, float* p_new, size_t n,
                                                          AdamWFirst o) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p_new[i] = adamw_first(p[i], g[i], o);
}
hipError_t launch_adamw_first(const float* g, const float* p, float* p_new, size_t n, const AdamWFirst& o, hipStream_t s) {
    if (n == 0) return hipSuccess;
    adamw_first_kernel<<<cdiv((long)n, 256), 256, 0, s>>>(g, p, p_new, n, o);
    return hipGetLastError();
}

template <int BM, int BN, int BKF, int PF, bool WIDE = false>
static hipError_t run_f32(F32Batch& grp, hipStream_t s) {
    long tiles = 0;
    for (int k = 0; k < grp.n; ++k) {
        F32Product& q = grp.p[k];
        q.tiles_m = cdiv(q.M, q.kind == F32_MN ? F32_MN_TILE(BM) : BM);
        q.tiles_n = cdiv(q.N, q.kind == F32_MN ? F32_MN_TILE(BN) : BN);
        q.tile0 = (int)tiles;
        tiles += (long)q.tiles_m * q.tiles_n;
        if (tiles > 0x7fffffffL) return hipErrorInvalidValue;
    }
    const int lds = F32Tile<BM, BN, BKF>::LDS_FLOATS * (int)sizeof(float);
    auto kern = f32_group_kernel<BM, BN, BKF, PF, WIDE>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kern<<<(unsigned)tiles, 256, lds, s>>>(grp);
    return hipGetLastError();
}

hipError_t launch_gemm_f32_group(const F32Product* prods, int n, hipStream_t s) {
    if (n < 1 || n > F32_GROUP_MAX) return hipErrorInvalidValue;
    F32Batch grp;
    grp.n = n;
    int order[F32_GROUP_MAX];
    for (int k = 0; k < n; ++k) order[k] = k;
    for (int k = 1; k < n; ++k)               // longest contraction first: what is left for the end are short tiles
        for (int j = k; j > 0 && prods[order[j]].K > prods[order[j - 1]].K; --j) { int t = order[j]; order[j] = order[j - 1]; order[j - 1] = t; }
    long t128 = 0, t64 = 0;
    bool wide = false;
    for (int k = 0; k < n; ++k) {
        F32Product& q = grp.p[k];
        q = prods[order[k]];
        if (q.M <= 0 || q.N <= 0 || q.K <= 0) return hipErrorInvalidValue;
        wide |= q.lda > (1L << 22) || q.ldb > (1L << 22) || q.lda2 > (1L << 22) || q.ldb2 > (1L << 22);
        if (q.kind == F32_MN) continue;
        t128 += (long)cdiv(q.M, 128) * cdiv(q.N, 128);
        t64 += (long)cdiv(q.M, 64) * cdiv(q.N, 64);
    }
    // (rows that wide are long chains on few tiles, or next to no arithmetic: no 128-wide instance for them)
    if (wide) return t64 >= 256 ? run_f32<64, 64, 32, 2, true>(grp, s) : run_f32<32, 32, 64, 2, true>(grp, s);
    // The largest tile that gives every CU one.  Below that smaller tiles, down to one chain of 16 x 16 outputs per wave: the
    // low-rank products of 1024 tokens (K 4096) take 45 us on 128 workgroups, a third of it the chain itself.
    if (t128 >= 256) return run_f32<128, 128, 16, 2>(grp, s);
    if (t64 >= 256) return run_f32<64, 64, 32, 2>(grp, s);
    return run_f32<32, 32, 64, 4>(grp, s);
}
