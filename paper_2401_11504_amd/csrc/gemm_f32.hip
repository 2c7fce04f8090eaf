// Products of the single fp32 LoRA-adapted linear step: fp32 operands and outputs, sums in fp32.  Several independent products
// C = alpha (A B^T + A2 B2^T) of three operand layouts share a launch:
//   F32_KK  A [M, K], B [N, K]: the contraction is contiguous in both          (X A^T;  X W^T + H B^T)
//   F32_KN  A [M, K], B [K, N]                                                 (dY B;   dY W + dH A)
//   F32_MN  A [K, M], B [K, N]                                                 (dH^T X; dY^T H)
// Small ones go through the fp32 matrix instructions (f32_direct_kernel, f32_group_kernel; f32_waves_kernel: low-rank ones of long contractions), large ones through the bf16 ones with every operand cut into
// three parts (f32_split_kernel); f32_cost holds what the line between them was timed on.
//
// v_mfma_f32_16x16x4_f32 adds its four products one after another, each as one fused multiply-add: in f32_group_kernel an output is a chain
// fma(a[k], b[k], ..) over k, the same value wherever its tile boundaries lie (the low-rank term a chain of its own, added to the
// stored main term), in f32_direct_kernel the sum of eight of them.  Lane (l16, g) holds row l16, element g of the four, one float per operand: elements 4 g .. 4 g + 3 of sixteen,
// for four instructions, so that they are one LDS read where the contraction is contiguous (64x64 tiles, 128 tokens, 4096 x 4096:
// 174 us for the step, 147 as four reads became one).  An operand whose contraction is contiguous is kept in LDS as it comes, [row][k], with a stride
// that lets the 64 lanes of a read touch 64 banks; one whose rows (or columns) are contiguous as [k][row], and a lane reads
// F neighbouring rows at once, one for each of the F fragments of its wave's share (the output is written with that order
// undone).  Neither is transposed on the way.
//
// The bound of f32_group_kernel, where the chip is full, is the matrix unit: 256 flop per clock and CU, a sixteenth of the bf16 rate, so that
// LDS reads are cheap beside it and tiles staged through registers are enough.  The two others say theirs.
#include "kernels.h"
#include "tiles.h"
#include <type_traits>
#include <utility>

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
// PAST: the first row may lie behind the operand's end (then there is nothing to load).
template <int B, int BKF, bool KC, bool WIDE, bool PAST>     // B rows (or columns); KC: the contraction is contiguous
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
        const long left = (unsigned)k0 < (unsigned)kmax && (!PAST || end > at) ? (end - at) * 4 : 0;
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
// fragments of 16 contraction elements starting at k: v[i][j] = fragment i, element 4 g + j
template <int B, int BKF, int F, bool KC>
__device__ __forceinline__ void f32_fragments(const float* tile, int row0, int k, int l16, int g, float (&v)[F][4]) {
    if constexpr (KC) {
#pragma unroll
        for (int i = 0; i < F; ++i) {
            const f32x4_t t = *(const f32x4_t*)(tile + (row0 + 16 * i + l16) * (BKF + 4) + k + 4 * g);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[i][j] = t[j];
        }
    } else {
        typedef float fvec __attribute__((ext_vector_type(F)));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const fvec t = *(const fvec*)(tile + (k + 4 * g + j) * (B + 4) + row0 + F * l16);
#pragma unroll
            for (int i = 0; i < F; ++i) v[i][j] = t[i];
        }
    }
}

template <int BM, int BN, int BKF, bool WIDE, bool AKC, bool BKC, bool PAST = false>
__device__ __forceinline__ void f32_tile(const F32Product& q, int m0, int n0, float* smem, int tid) {
    using T = F32Tile<BM, BN, BKF>;
    constexpr int FM = T::FM, FN = T::FN, KS = BKF / 16, PF = 2;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, g = lane >> 4;
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
        F32Stage<BM, BKF, AKC, WIDE, PAST> ra[PF];
        F32Stage<BN, BKF, BKC, WIDE, PAST> rb[PF];
        float a[2][KS][FM][4], b[2][KS][FN][4];
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
        load(S0{}, 0);
        load(S1{}, 1);
        park(S0{}, 0, 0);
        load(S0{}, PF);
        park(S1{}, 1, 1);
        load(S1{}, PF + 1);
        __syncthreads();
        fetch(S0{}, 0);
        int p0 = 0, p1 = 1, p2 = 2;               // places of tiles t, t + 1 and t + 2
        auto step = [&](auto u, int t) {          // u = t % PF
            using cur = std::integral_constant<int, u.value & 1>;
            using slot = std::integral_constant<int, (u.value + 2) % PF>;
            fetch(std::integral_constant<int, cur::value ^ 1>{}, p1);
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
        // Whole rounds of PF tiles, then the rest: with exits between the steps the compiler sees a way from each of them to the next
        // round and has step 0 wait for the loads just issued (2 to 6 % of a small step).
        int t = 0;
        for (; t + PF <= nk; t += PF) {
            step(S0{}, t);
            step(S1{}, t + 1);
        }
        if (t < nk) step(S0{}, t);
        __syncthreads();                          // the places of the ring are free for the next term
        const float alpha = term ? q.alpha2 : q.alpha;

        // Output, four neighbouring columns of a row at a time: run r of row fragment i holds fragment r's columns 4 g .. 4 g + 3
        // (contiguous contraction), or columns FN (4 g) + 4 r .. + 3 of the wave's share, which interleaves the fragments.
        int lo = l16, go = g;                     // (as new values: the addresses are not to be held through the loop above)
        asm volatile("" : "+v"(lo), "+v"(go));
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int r = 0; r < FN; ++r) {
                const int m = m0 + wm * T::TM + (AKC ? 16 * i + lo : FM * lo + i);
                const int n = n0 + wn * T::TN + (BKC ? 16 * r + 4 * go : 4 * FN * go + 4 * r);
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

template <int BM, int BN, int BKF, bool WIDE>
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
    const int im = tile % q.tiles_m, in = tile / q.tiles_m, tid = threadIdx.x;
    constexpr int MM = F32_MN_TILE(BM), MN = F32_MN_TILE(BN);
    if (q.kind == F32_KK) f32_tile<BM, BN, BKF, WIDE, true, true>(q, im * BM, in * BN, smem_f32, tid);
    else if (q.kind == F32_KN) f32_tile<BM, BN, BKF, WIDE, true, false>(q, im * BM, in * BN, smem_f32, tid);
    else f32_tile<MM, MN, BKF, WIDE, false, false>(q, im * MM, in * MN, smem_f32, tid);
}

// ---------------------------------------------------------------- small steps: fragments straight from memory
// 16 F x 16 F outputs per workgroup of eight waves; wave w takes pieces w, w + 8, .. of sixteen contraction elements, and the eight sums are
// added in that order through LDS.  Each wave loads its own fragments, PF pieces ahead, with no LDS, no barrier and next to no address
// arithmetic in the loop (a base that moves in scalar registers, lane offsets that stay).  A small step is two chains over the whole
// width on few CUs.  Staged through LDS in 32x32 tiles with a barrier per 64 elements they took 11.5 ns an element, 2700 clocks of which
// 1024 were matrix instructions; this way it is 7 in 32x32 tiles and 3.6 in 16x16 ones, which is what a CU gets of its operands (40 to 60
// GB/s from beyond its L2), so that the smaller tile, on more CUs, is the faster one until the chip is full.  (Fragments through LDS of the
// wave's own, for loads of whole 64-byte runs, changed nothing; two groups of four waves in the staged kernel 9 ns, and slower where the
// chip is full.)  us: 128 tokens, 256 x 256, rank 8 36 -> 31; 37, 3349 x 142, rank 16 92 -> 46; 36, 563 x 4006, rank 4 100 -> 51.
constexpr int DIRECT_WAVES = 8;

template <int F, int PF, bool AKC, bool BKC>
__device__ __forceinline__ void f32_direct_sum(const float* A, long lda, const float* B, long ldb, int rows_a, int rows_b, int K,
                                               f32x4_t (&acc)[F][F], int wave, int lane) {
    const int l16 = lane & 15, g = lane >> 4;
    // byte offsets of fragment i within a piece; rows (columns) past the end are the last one again, and only feed what is never stored
    unsigned oa[F], ob[F];
#pragma unroll
    for (int i = 0; i < F; ++i) {
        const unsigned ra = min(16 * i + l16, rows_a - 1), rb = min(16 * i + l16, rows_b - 1);
        oa[i] = (AKC ? ra * (unsigned)lda + 4 * g : 4 * g * (unsigned)lda + ra) * 4;
        ob[i] = (BKC ? rb * (unsigned)ldb + 4 * g : 4 * g * (unsigned)ldb + rb) * 4;
    }
    float a[PF][F][4], b[PF][F][4];
    auto fragments = [&](auto kc, const float* base, long ld, int k, const unsigned (&off)[F], float (&v)[F][4]) {
        if constexpr (kc.value) {
            const char* at = (const char*)(base + k);
#pragma unroll
            for (int i = 0; i < F; ++i) {
                const f4u t = *(const f4u*)(at + off[i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = t[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const char* at = (const char*)(base + (k + e) * ld);
#pragma unroll
                for (int i = 0; i < F; ++i) v[i][e] = *(const float*)(at + off[i]);
            }
        }
    };
    using KA = std::integral_constant<bool, AKC>;
    using KB = std::integral_constant<bool, BKC>;
    auto multiply = [&](int u) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < F; ++i)
#pragma unroll
                for (int j = 0; j < F; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u][j][e], a[u][i][e], acc[i][j], 0, 0, 0);
    };
    const int full = K / 16, mine = full > wave ? (full - wave + DIRECT_WAVES - 1) / DIRECT_WAVES : 0;
    if (mine > 0) {
        auto load = [&](int u, int t) {           // (past the wave's last piece: that one again, never multiplied)
            const int k = 16 * (wave + DIRECT_WAVES * min(t, mine - 1));
            fragments(KA{}, A, lda, k, oa, a[u]);
            fragments(KB{}, B, ldb, k, ob, b[u]);
        };
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            load(u, u);
            __builtin_amdgcn_sched_barrier(0);    // (in this order: what a use waits for is counted)
        }
        int t = 0;
        for (; t + PF <= mine; t += PF)
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                multiply(u);
                load(u, t + u + PF);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
        for (int u = 0; u + 1 < PF; ++u)
            if (t + u < mine) multiply(u);
    }
    const int rest = K - 16 * full;
    if (rest > 0 && wave == full % DIRECT_WAVES) {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[0][i][e] = b[0][i][e] = 0.f;
                if (4 * g + e < rest) {
                    a[0][i][e] = *(const float*)((const char*)(A + (AKC ? 16 * full + e : (16 * full + e) * lda)) + oa[i]);
                    b[0][i][e] = *(const float*)((const char*)(B + (BKC ? 16 * full + e : (16 * full + e) * ldb)) + ob[i]);
                }
            }
        multiply(0);
    }
}

template <int F, int PF, bool AKC, bool BKC>
__device__ __forceinline__ void f32_direct_tile(const F32Product& q, int m0, int n0, float* smem) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};             // of the first STORING threads: four columns of a row
    constexpr int SIDE = 16 * F, LD = SIDE + 4, STORING = SIDE * SIDE / 4;
    const int row = tid / (SIDE / 4), col = tid % (SIDE / 4) * 4;
#pragma unroll 1
    for (int term = 0; term < (q.K2 > 0 ? 2 : 1); ++term) {
        const float *A = term ? q.A2 : q.A, *B = term ? q.B2 : q.B;
        const long lda = term ? q.lda2 : q.lda, ldb = term ? q.ldb2 : q.ldb;
        f32x4_t acc[F][F];
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        f32_direct_sum<F, PF, AKC, BKC>(A + (AKC ? m0 * lda : m0), lda, B + (BKC ? n0 * ldb : n0), ldb, q.M - m0, q.N - n0,
                                     term ? q.K2 : q.K, acc, wave, lane);
        if (term) __syncthreads();                // the other term's sums have been read
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j)           // (B first in the matrix instruction: a lane has row l16 of A's fragment, columns 4 g .. of B's)
                *(f32x4_t*)(smem + (wave * SIDE + 16 * i + l16) * LD + 16 * j + 4 * g) = acc[i][j];
        __syncthreads();
        if (tid < STORING) {
            f32x4_t sum = *(const f32x4_t*)(smem + row * LD + col);
#pragma unroll
            for (int w = 1; w < DIRECT_WAVES; ++w) sum += *(const f32x4_t*)(smem + (w * SIDE + row) * LD + col);
            const float alpha = term ? q.alpha2 : q.alpha;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = term ? v[e] + alpha * sum[e] : alpha * sum[e];
        }
    }
    const int m = m0 + row, n = n0 + col;
    if (tid >= STORING || m >= q.M || n >= q.N) return;
    const long at = (long)m * q.ldc + n;
    if (n + 4 <= q.N) {
        *(f4u*)(q.C + at) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + e < q.N) q.C[at + e] = v[e];
    }
    if (q.p_new) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + e < q.N) q.p_new[at + e] = adamw_first(q.p_old[at + e], v[e], q.opt);
    }
}

template <int F>
__global__ __launch_bounds__(DIRECT_WAVES * 64, 4) void f32_direct_kernel(F32Batch grp) {
    __shared__ __align__(16) float sums[DIRECT_WAVES * 16 * F * (16 * F + 4)];
    const int b = blockIdx.x;
    int k = 0;
    while (k + 1 < grp.n && b >= grp.p[k + 1].tile0) ++k;
    const F32Product& q = grp.p[k];
    const int n = q.tiles_m * q.tiles_n, id = b - q.tile0;      // (the same order of tiles as in f32_group_kernel)
    const int c = id & 7, per = n >> 3, tile = c * per + min(c, n & 7) + (id >> 3);
    const int m0 = tile % q.tiles_m * (16 * F), n0 = tile / q.tiles_m * (16 * F);
    if (q.kind == F32_KK) f32_direct_tile<F, 4, true, true>(q, m0, n0, sums);
    else if (q.kind == F32_KN) f32_direct_tile<F, 4, true, false>(q, m0, n0, sums);
    else f32_direct_tile<F, 3, false, false>(q, m0, n0, sums);
}

// ---------------------------------------------------------------- the low-rank products of larger steps
// 16 x 16 FN outputs per workgroup of eight waves, each with an eighth of the contraction in 32-wide pieces through a ring of its own:
// f32_direct_kernel's loads touch 16 rows with every instruction (and take one element a lane where the contraction is not contiguous), and a CU gets 40
// to 60 GB/s of them; direct-to-LDS loads of whole 128-byte rows (64-byte ones of the [K, N] operand) bring 88.  The eight sums are added in order
// through LDS.  H and dH of 1024 tokens, 4096 x 4096, rank 64: 34.7 and 18 us (in 16x16 tiles 23; rings of two and three pieces 19 to 20).  Operands and rows start at multiples of 16 bytes.
//   contiguous contraction: row r's chunk c (four elements) lies at position c ^ (r / 2 % 8)
//   [K, N]: of sixteen rows k, row 4 g + e lies at place 4 e + g, so that the 64 lanes that read element e of their four touch 64 banks
template <int FN, int ST>
__global__ __launch_bounds__(512, 2) void f32_waves_kernel(F32Batch grp) {
    constexpr int NL = 2 + 2 * FN, STAGE = NL * 1024, RING = ST * STAGE;
    static_assert((ST - 1) * NL <= 63 && 8 * RING <= 160 * 1024, "ring");
    extern __shared__ __align__(16) unsigned char smem_waves[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    int k = 0;
    while (k + 1 < grp.n && (int)blockIdx.x >= grp.p[k + 1].tile0) ++k;
    const F32Product& q = grp.p[k];
    const int n = q.tiles_m * q.tiles_n, id = blockIdx.x - q.tile0;
    const int c8 = id & 7, per = n >> 3, tile = c8 * per + min(c8, n & 7) + (id >> 3);
    const int m0 = tile / q.tiles_n * 16, n0 = tile % q.tiles_n * (16 * FN);       // the column tiles of a row tile on one XCD
    const bool kn = q.kind == F32_KN;
    const int M = q.M, N = q.N, K = q.K;
    const unsigned lda = (unsigned)q.lda * 4, ldb = (unsigned)q.ldb * 4;
    const char* A = (const char*)(q.A + (long)m0 * q.lda);
    const char* B = (const char*)(q.B + (kn ? 0 : (long)n0 * q.ldb));
    const long step_b = kn ? 32 * (long)ldb : 128;
    unsigned off[NL];          // of the fetches of a piece: two of A, two per fragment of B
    int at_k[NL];              // the first contraction element that this lane brings
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int r = (i & 1) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7), f = i / 2 - 1;
        if (i < 2 || !kn) {
            const int row = i < 2 ? min(r, M - 1 - m0) : min(16 * f + r, N - 1 - n0);
            off[i] = (unsigned)row * (i < 2 ? lda : ldb) + chunk * 16;
            at_k[i] = chunk * 4;
        } else {
            const int place = lane >> 2, kk = (i & 1) * 16 + (place & 3) * 4 + (place >> 2);
            off[i] = (unsigned)kk * ldb + (unsigned)min(n0 + 16 * f + 4 * (lane & 3), N - 4) * 4;
            at_k[i] = kk;
        }
    }
    const int nk = (K + 31) / 32, first = nk * wave >> 3, mine = (nk * (wave + 1) >> 3) - first;
    const bool narrow = (K & 31) && first + mine == nk;
    const unsigned ring0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)smem_waves + wave * RING);
    auto fetch = [&](int t, unsigned st) {
        const int kt = first + t;
        const char *pa = A + (long)kt * 128, *pb = B + kt * step_b;
        const int left = K - kt * 32;
        if (left >= 32) {
#pragma unroll
            for (int i = 0; i < NL; ++i) load_lds16(off[i], i < 2 ? pa : pb, __builtin_amdgcn_readfirstlane(ring0 + st + i * 1024));
        } else {                                   // zeros beyond the end
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                if (at_k[i] < left) load_lds16(off[i], i < 2 ? pa : pb, __builtin_amdgcn_readfirstlane(ring0 + st + i * 1024));
                else *(uint4*)(smem_waves + wave * RING + st + i * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
            }
        }
    };
    f32x4_t acc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int t = 0; t < min(ST, mine); ++t) fetch(t, t * STAGE);
    const unsigned char* ring = smem_waves + wave * RING;
    unsigned st = 0;
    for (int t = 0; t < mine; ++t) {
        if (t + ST <= mine && !narrow) wait_vmcnt<(ST - 1) * NL>();
        else wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        f32x4_t a[2], b[2][FN];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int at = l16 * 128 + (((4 * h + g) ^ (l16 >> 1)) << 4);
            a[h] = *(const f32x4_t*)(ring + st + at);
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (!kn) {
                    b[h][j] = *(const f32x4_t*)(ring + st + (j + 1) * 2048 + at);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[h][j][e] = *(const float*)(ring + st + (j + 1) * 2048 + h * 1024 + ((4 * e + g) * 16 + l16) * 4);
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // its place may be filled again
        if (t + ST < mine) fetch(t + ST, st);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[h][j][e], a[h][e], acc[j], 0, 0, 0);
        st = st + STAGE == RING ? 0 : st + STAGE;
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) *(f32x4_t*)(smem_waves + wave * RING + j * 1024 + lane * 16) = acc[j];
    __syncthreads();
    for (int i = tid; i < FN * 64; i += 512) {
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 8; ++w) v += *(const f32x4_t*)(smem_waves + w * RING + i * 16);
        const int el = i & 63, row = m0 + (el & 15), col = n0 + (i >> 6) * 16 + 4 * (el >> 4);
        if (row >= M || col >= N) continue;        // N is a multiple of 4
        f4u o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = q.alpha * v[e];
        *(f4u*)(q.C + (long)row * q.ldc + col) = o;
    }
}

// ---------------------------------------------------------------- split operands on the bf16 matrix instructions
// The same products with every operand cut into three bf16 parts, x = x1 + x2 + x3 (each the nearest bf16 to what is left, which the
// third holds exactly), and a b taken as (a1 b3 + a2 b2 + a1 b2 + a3 b1 + a2 b1) + a1 b1, each of the two in fp32 accumulators of its own.
// What is left out, a2 b3 + a3 b2 + a3 b3, is below 2^-26 of a product and of either sign.  The matrix instruction rounds to nearest,
// some four times for its 32 elements: K / 8 roundings at the size of the result instead of K.
// Distance from fp64, 2-norm, chain of fp32 products / parts: 1024 tokens, 4096 x 4096, rank 64 Y 1.15e-6 / 4.0e-7, dA 1.28e-6 / 4.5e-7,
// operands of one sign Y 1.8e-7 / 5.4e-8, a dY that is a softmax dX 6.3e-8 / 9.4e-8; 700, 2500 x 2500, rank 32 Y 8.9e-7 / 3.1e-7, of one sign
// 1.7e-7 / 5.3e-8.  (With all six products in one accumulator: Y 1.01e-6, the softmax's dX 1.9e-7, the same time.  With a sum of each tile by itself and
// added to the accumulator: 2.3e-7, 7.3e-8, 385 instead of 367 us.  Parts cut off instead of rounded have all the sign of x, and what a large
// sum drops of their products, each below half an ulp of it, adds up: with operands of one sign 2.1e-6 to 4e-5.)
//
// The bf16 unit has sixteen times the rate, so that six products take 6/16 of the time of one in fp32.  What is cut is cut on
// its way from the staging registers to LDS, seven vector operations an element, in slices between the matrix instructions.
// (A matrix instruction of 16 clocks hides two vector operations, from whichever wave: twice as many waves that cut in one go and multiply in
// another were slower, 465 against 430 us for a step of 1024 tokens, 4096 x 4096, rank 64; in fp32 tiles of 128x128 it was 690.)
//
// (Two fp16 halves an operand, scaled by a power of two for the whole array, take three products instead of six and 280 us instead of 390.
// But fp16 has five bits of exponent: an element below 2^-17 of the array's largest loses bits, and is nothing below 2^-40, where it may be all that an output is made of --
// the other operand may be zero, or small, where this one is large.  To find that out takes a look at every element, and among normal draws some always lie that low.)
//
// Operands are scaled by 2^24 on the way, so that the parts hold every value down to fp32's smallest (2^-149: the third part of one below 2^-110
// would be out of bf16's range otherwise), and outputs by 2^-48 at the end.  What does not fit then -- operands that are not finite or above
// 2^104, sums above 2^80 -- leaves an accumulator that is not finite: such a workgroup does its outputs again with f32_tile, in two halves of 256
// threads.  us for a step of 1024 tokens, 4096 x 4096, rank 64: 380; with a softmax for dY, most of it far below 1, 380 (674 all in fp32, 716
// where a value below 2^-110 sends a workgroup there); with one infinity in X, 957.
//
// Order of the 32 contraction elements of a tile within the matrix instruction: lane group g takes 4 g .. 4 g + 3 and
// 16 + 4 g .. 16 + 4 g + 3, in both operands.
constexpr int SPLIT_BK = 32, SPLIT_NT = 512, SPLIT_HEAD = 16;     // (bytes of LDS ahead of the planes)
constexpr float SPLIT_SCALE = 0x1p24f;
// One operand: memory -> registers (`N` items of four floats a thread) -> three planes of LDS per tile.
//   KC: [row][32], 8-byte piece p of a row (elements 4 p .. 4 p + 3) as half p / 4 of 16-byte chunk (p % 4) ^ (row / 4 % 4), so that
//       a lane's elements are one chunk, sixteen rows' chunks lie in distinct banks, and so do the pieces that are written
//   otherwise [k][B + 16], read by the LDS transpose read (eight consecutive k x 32 bytes lie in distinct banks)
template <int B, bool KC>
struct SplitOperand {
    static constexpr int LD = KC ? SPLIT_BK : B + 16, PLANE = KC ? B * LD : SPLIT_BK * LD, ELEMS = 3 * PLANE;
    static constexpr int CPR = (KC ? SPLIT_BK : B) / 4, STEP = SPLIT_NT / CPR, N = B * SPLIT_BK / (4 * SPLIT_NT);
    static_assert(N >= 1 && (!KC || STEP % 16 == 0), "tile shape");
    unsigned off;         // byte offset of item 0 within a tile in memory
    int dst;              // and where its parts go within a plane
    __device__ __forceinline__ void init(long ld, int tid) {
        const int c = tid % CPR, o = tid / CPR;
        off = ((unsigned)o * (unsigned)ld + c * 4) * 4;
        dst = KC ? o * LD + (((c & 3) ^ ((o >> 2) & 3)) * 8) + (c >> 2) * 4 : o * LD + c * 4;
    }
    // (what lies behind the operand's end reads as zero; see F32Stage)
    static __device__ __forceinline__ auto rsrc(const float* src, long ld, int r0, int rows, int k0, int kmax) {
        const long at = KC ? r0 * ld + k0 : k0 * ld + r0, end = KC ? (rows - 1) * ld + kmax : (kmax - 1) * ld + rows;
        const long left = (unsigned)k0 < (unsigned)kmax ? (end - at) * 4 : 0;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(src + (left > 0 ? at : 0)), 0,
                                                 (int)(unsigned)(left > 0xffffffffL ? 0xffffffffL : left), 0x00020000);
    }
    template <class R>
    __device__ __forceinline__ u32x4_t load(R rs, int i, long ld) const {
        return __builtin_amdgcn_raw_buffer_load_b128(rs, off + (unsigned)i * ((unsigned)ld * (STEP * 4)), 0, 0);
    }
    // elements past the contraction's end belong to the next row: they count as zero
    static __device__ __forceinline__ u32x4_t mask(u32x4_t r, int left, int tid) {
        const int c = (tid % CPR) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = !KC || c + e < left ? r[e] : 0u;
        return r;
    }
    // fragment of 16 rows from row0 on: lane (l16, g) holds row l16
    static __device__ __forceinline__ int lane_offset(int row0, int lane) {
        const int l16 = lane & 15, g = lane >> 4;
        return KC ? (row0 + l16) * LD + ((g ^ (l16 >> 2)) * 8) : (4 * g + (l16 >> 2)) * LD + row0 + 4 * (l16 & 3);
    }
    static __device__ __forceinline__ bf16x8_t fragment(const bf16_t* at, int i) {
        if constexpr (KC) {
            return *(const bf16x8_t*)(at + 16 * i * LD);
        } else {          // (lane q + 4 e of a group of sixteen points at element e, rows 4 q .. 4 q + 3: see tr_frag_at in tiles.h)
            typedef __attribute__((address_space(3))) bf16x4v_t* lds_ptr_t;
            const bf16x4v_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(at + 16 * i));
            const bf16x4v_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(at + 16 * i + 16 * LD));
            bf16x8_t v;
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
            return v;
        }
    }
};
// the parts of four floats times a scale, made in seven slices: two per pair of elements, then one per plane
struct SplitParts {
    unsigned x[3][2];
    float y[2];            // what the first part leaves of a pair
    static __device__ __forceinline__ float first(unsigned pair) { return __uint_as_float(pair << 16); }
    static __device__ __forceinline__ float second(unsigned pair) { return __uint_as_float(pair & 0xffff0000u); }
    __device__ __forceinline__ void pair(unsigned b0, unsigned b1, int j, float scale) {
        const float v0 = __uint_as_float(b0), v1 = __uint_as_float(b1);
        x[0][j] = pack_bf16x2(v0 * scale, v1 * scale);
        y[0] = fmaf(v0, scale, -first(x[0][j]));
        y[1] = fmaf(v1, scale, -second(x[0][j]));
    }
    __device__ __forceinline__ void rest(int j) {
        x[1][j] = pack_bf16x2(y[0], y[1]);
        x[2][j] = __builtin_amdgcn_perm(__float_as_uint(y[1] - second(x[1][j])), __float_as_uint(y[0] - first(x[1][j])), 0x07060302u);
    }
    __device__ __forceinline__ void put(bf16_t* dst, int p) const { *(uint2*)dst = make_uint2(x[p][0], x[p][1]); }
};

// f(0), f(1), .. with the index as a constant: registers that are picked by it stay registers
template <class F, int... I>
__device__ __forceinline__ void for_each_index(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void unrolled(F f) { for_each_index(f, std::make_integer_sequence<int, N>{}); }

template <int BM, int BN>
struct SplitTile {
    static constexpr int MAX(int a, int b) { return a > b ? a : b; }
    static constexpr int STAGE = MAX(SplitOperand<BM, true>::ELEMS + MAX(SplitOperand<BN, true>::ELEMS, SplitOperand<BN, false>::ELEMS),
                                     2 * SplitOperand<64, false>::ELEMS);
    // the halves that are taken in fp32 instead
    static constexpr int F32_BYTES = 2 * (int)sizeof(float) * MAX(F32Tile<64, BN, 16>::LDS_FLOATS, F32Tile<32, 64, 32>::LDS_FLOATS);
    static constexpr int LDS_BYTES = MAX(SPLIT_HEAD + 2 * STAGE * (int)sizeof(bf16_t), F32_BYTES);
};

// BM x BN outputs per workgroup of WM x WN waves.  Tile t + 1 of the contraction is cut and written to the other LDS stage while
// tile t is multiplied, and the loads of t + 2 follow into the registers that this frees: one barrier per tile, behind the last
// write, with an eighth of the matrix instructions left to cover the first fragments of t + 1.
template <int BM, int BN, int WM, int WN, bool AKC, bool BKC>
__device__ __forceinline__ bool split_tile(const F32Product& q, int m0, int n0, unsigned char* smem) {
    constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
    static_assert(WM * WN * 64 == SPLIT_NT && FM >= 1 && FN >= 1, "waves");
    using OA = SplitOperand<BM, AKC>;
    using OB = SplitOperand<BN, BKC>;
    constexpr int STAGE = OA::ELEMS + OB::ELEMS, NG = FM * FN, NMF = 6 * NG, NI = OA::N + OB::N, NS = 8 * NI;
    constexpr int AT_BARRIER = NMF - (NMF + 7) / 8, SLICED = NMF * 3 / 4;      // matrix instructions ahead of the barrier, and among slices
    const int M = q.M, N = q.N;
    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    int* overflow = (int*)smem;            // an accumulator is not finite
    bf16_t* planes = (bf16_t*)(smem + SPLIT_HEAD);
    const int a_off = OA::lane_offset(wm * TM, lane), b_off = OA::ELEMS + OB::lane_offset(wn * TN, lane);
    // The largest products (first parts) go into acc, the five others into `small`, which joins acc at the end: there each rounding is one of
    // 2^-8 of the result.  Fragments are taken BLOCK at a time, A's of the next block read beside the matrix instructions of this one
    // (254 registers; A's third parts are read in their own block, with them it would be scratch memory).
    constexpr int RB = FN >= 4 ? 1 : FN == 2 ? 2 : 1, BLOCK = RB * FN, NB = FM / RB;
    static_assert(FM % RB == 0 && NB % 2 == 0, "A's fragments of block b are in set b % 2");
    f32x4_t small[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) small[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bf16x8_t fa[2][2][RB], fa2[RB], fb[3][FN];
    auto read_a = [&](const bf16_t* stage, auto set, int b, int f) { fa[set.value][f % 2][f / 2] = OA::fragment(stage + a_off + f % 2 * OA::PLANE, b * RB + f / 2); };
    auto read_a2 = [&](const bf16_t* stage, int b, int f) { fa2[f] = OA::fragment(stage + a_off + 2 * OA::PLANE, b * RB + f); };
    auto read_b = [&](const bf16_t* stage, int s, int i) { fb[s][i] = OB::fragment(stage + b_off + s * OB::PLANE, i); };
    using S0 = std::integral_constant<int, 0>;
    // the main term, and the low-rank one on top of it, with alpha2 in its first operand.  (A large low-rank term below a long main one would be
    // rounded at each of its steps: 512 tokens, 1024 x 1024, rank 64, operands of one sign, Y 4.6e-7 from fp64 that way.)
#pragma unroll 1
    for (int term = 0; term < (q.K2 > 0 ? 2 : 1); ++term) {
        const float *A = term ? q.A2 : q.A, *B = term ? q.B2 : q.B;
        const long lda = term ? q.lda2 : q.lda, ldb = term ? q.ldb2 : q.ldb;
        const int K = term ? q.K2 : q.K;
        auto tile_k = [](int t) { return (int)((unsigned)t * SPLIT_BK); };     // (beyond the end: reads as zeros, never multiplied)
        OA oa;
        OB ob;
        oa.init(lda, tid);
        ob.init(ldb, tid);
        SplitParts parts;
        u32x4_t r[NI];                     // the items of A, then those of B
        auto item_dst = [&](bf16_t* stage, int i, int p) {
            return i < OA::N ? stage + (oa.dst + p * OA::PLANE + i * OA::STEP * OA::LD)
                             : stage + (OA::ELEMS + ob.dst + p * OB::PLANE + (i - OA::N) * OB::STEP * OB::LD);
        };
        auto mask = [&](int left) {
#pragma unroll
            for (int i = 0; i < NI; ++i) r[i] = i < OA::N ? OA::mask(r[i], left, tid) : OB::mask(r[i], left, tid);
        };
        const float scale_a = term ? q.alpha2 * SPLIT_SCALE : SPLIT_SCALE;
        {
            const auto rsa = OA::rsrc(A, lda, m0, M, 0, K);
            const auto rsb = OB::rsrc(B, ldb, n0, N, 0, K);
#pragma unroll
            for (int i = 0; i < NI; ++i) r[i] = i < OA::N ? oa.load(rsa, i, lda) : ob.load(rsb, i - OA::N, ldb);
            __syncthreads();               // the other term's tiles have been read
            if (tid == 0) *overflow = 0;
            mask(K);
            const auto rsa1 = OA::rsrc(A, lda, m0, M, tile_k(1), K);
            const auto rsb1 = OB::rsrc(B, ldb, n0, N, tile_k(1), K);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    parts.pair(r[i][2 * j], r[i][2 * j + 1], j, i < OA::N ? scale_a : SPLIT_SCALE);
                    parts.rest(j);
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) parts.put(item_dst(planes, i, p), p);
                r[i] = i < OA::N ? oa.load(rsa1, i, lda) : ob.load(rsb1, i - OA::N, ldb);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < FN; ++i) read_b(planes, 2, i);
#pragma unroll
            for (int i = 0; i < FN; ++i) read_b(planes, 1, i);
#pragma unroll
            for (int f = 0; f < 2 * RB; ++f) read_a(planes, S0{}, 0, f);
        }
        bf16_t *stage = planes, *other = planes + STAGE;
        const int nk = (K + SPLIT_BK - 1) / SPLIT_BK;
        for (int t = 0; t < nk; ++t) {
            const auto rsa = OA::rsrc(A, lda, m0, M, tile_k(t + 2), K);
            const auto rsb = OB::rsrc(B, ldb, n0, N, tile_k(t + 2), K);
            if (t + 2 >= nk) mask(K - tile_k(t + 1));
            // slice x of NS: half of the work on a pair of an item, one of its planes, or the load that replaces it
            auto slice = [&](auto xc) {
                constexpr int i = xc.value / 8, y = xc.value % 8;
                if constexpr (y < 4 && y % 2 == 0) parts.pair(r[i][y], r[i][y + 1], y / 2, i < OA::N ? scale_a : SPLIT_SCALE);
                else if constexpr (y < 4) parts.rest(y / 2);
                else if constexpr (y < 7) parts.put(item_dst(other, i, y - 4), y - 4);
                else if constexpr (i < OA::N) r[i] = oa.load(rsa, i, lda);
                else r[i] = ob.load(rsb, i - OA::N, ldb);
            };
            auto hand_over = [&] {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            };
            unrolled<NMF>([&](auto ec) {
                constexpr int e = ec.value, b = e / (6 * BLOCK), at = e % (6 * BLOCK), gr = at / BLOCK, x = at % BLOCK, i = x / FN, jn = x % FN;
                constexpr int left = NMF - AT_BARRIER, set = b % 2;
                constexpr int pa = gr == 1 || gr == 4 ? 1 : gr == 3 ? 2 : 0, pb = gr == 0 ? 2 : gr == 1 || gr == 2 ? 1 : 0;
                // B first: a lane then holds row l16 of A's fragment, columns 4 g .. 4 g + 3 of B's
                f32x4_t& sum = gr == 5 ? acc[b * RB + i][jn] : small[b * RB + i][jn];
                sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[pb][jn], pa == 2 ? fa2[i] : fa[set][pa % 2][i], sum, 0, 0, 0);
                // the fragments that are needed next: B's first parts, A's third ones, the others of A's next block
                unrolled<FN>([&](auto f) {
                    if constexpr (f.value == e) read_b(stage, 0, f.value);
                });
                unrolled<RB>([&](auto f) {
                    if constexpr (f.value == at) read_a2(stage, b, f.value);
                });
                unrolled<2 * RB>([&](auto f) {
                    if constexpr (b + 1 < NB && 3 * BLOCK + f.value * BLOCK / RB == at) read_a(stage, std::integral_constant<int, set ^ 1>{}, b + 1, f.value);
                });
                unrolled<NS>([&](auto y) {
                    if constexpr (y.value * SLICED / NS == e) slice(y);
                });
                if constexpr (e + 1 == AT_BARRIER) hand_over();
                unrolled<2 * FN + 2 * RB>([&](auto f) {
                    if constexpr (AT_BARRIER - 1 + f.value * left / (2 * FN + 2 * RB) == e) {
                        if constexpr (f.value < 2 * FN) read_b(other, 2 - f.value / FN, f.value % FN);
                        else read_a(other, S0{}, 0, f.value - 2 * FN);
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
            });
            bf16_t* const s = stage;
            stage = other; other = s;
        }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] += small[i][j];
    float zero = 0.f;                      // (stays that where every accumulator is finite)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) zero = fmaf(acc[i][j][e], 0.f, zero);
    if (!(zero == 0.f)) *overflow = 1;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(*overflow)) return false;
    const float alpha = q.alpha / (SPLIT_SCALE * SPLIT_SCALE);
    int out = threadIdx.x;                 // (as a new value: the output's addresses are not to be held through the loops above)
    asm volatile("" : "+v"(out));
    const int l16 = out & 15, g = (out >> 4) & 3;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int r = 0; r < FN; ++r) {
            const int m = m0 + wm * TM + 16 * i + l16, n = n0 + wn * TN + 16 * r + 4 * g;
            if (m >= M || n >= N) continue;
            const long at = (long)m * q.ldc + n;
            f4u v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = alpha * acc[i][r][e];
            if (n + 4 <= N) {
                *(f4u*)(q.C + at) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) q.C[at + e] = v[e];
            }
            if (q.p_new) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) q.p_new[at + e] = adamw_first(q.p_old[at + e], v[e], q.opt);
            }
        }
    return true;
}

template <int BM, int BN, int WM, int WN, int BKF, bool AKC, bool BKC>
__device__ __forceinline__ void split_or_f32_tile(const F32Product& q, int m0, int n0, unsigned char* smem) {
    if (split_tile<BM, BN, WM, WN, AKC, BKC>(q, m0, n0, smem)) return;
    __syncthreads();                       // every wave has read the flag that lies in this memory
    const int tid = threadIdx.x, half = __builtin_amdgcn_readfirstlane(tid >> 8);
    constexpr int B = BM / 2 < 64 ? BM / 2 : 64;      // (rows at once: 128 would take more registers than there are)
#pragma unroll 1
    for (int m = 0; m < BM / 2; m += B) {
        if (m) __syncthreads();
        f32_tile<B, BN, BKF, false, AKC, BKC, true>(q, m0 + half * (BM / 2) + m, n0,
                                                       (float*)smem + half * F32Tile<B, BN, BKF>::LDS_FLOATS, tid & 255);
    }
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(SPLIT_NT, 2) void f32_split_kernel(F32Batch grp) {
    extern __shared__ __align__(16) unsigned char smem_split[];
    const int b = blockIdx.x;
    int k = 0;
    while (k + 1 < grp.n && b >= grp.p[k + 1].tile0) ++k;
    const F32Product& q = grp.p[k];
    const int n = q.tiles_m * q.tiles_n, id = b - q.tile0;      // (the same order of tiles as in f32_group_kernel)
    const int c = id & 7, per = n >> 3, tile = c * per + min(c, n & 7) + (id >> 3);
    const int im = tile % q.tiles_m, in = tile / q.tiles_m;
    if (q.kind == F32_KK) split_or_f32_tile<BM, BN, WM, WN, 16, true, true>(q, im * BM, in * BN, smem_split);
    else if (q.kind == F32_KN) split_or_f32_tile<BM, BN, WM, WN, 16, true, false>(q, im * BM, in * BN, smem_split);
    else split_or_f32_tile<64, 64, 2, 4, 32, false, false>(q, im * 64, in * 64, smem_split);
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

template <int BM, int BN>
static hipError_t place_f32(F32Batch& grp, int* n_tiles) {
    long tiles = 0;
    for (int k = 0; k < grp.n; ++k) {
        F32Product& q = grp.p[k];
        q.tiles_m = cdiv(q.M, q.kind == F32_MN ? F32_MN_TILE(BM) : BM);
        q.tiles_n = cdiv(q.N, q.kind == F32_MN ? F32_MN_TILE(BN) : BN);
        q.tile0 = (int)tiles;
        tiles += (long)q.tiles_m * q.tiles_n;
        if (tiles > 0x7fffffffL) return hipErrorInvalidValue;
    }
    *n_tiles = (int)tiles;
    return hipSuccess;
}
template <int BM, int BN, int BKF, bool WIDE = false>
static hipError_t run_f32(F32Batch& grp, hipStream_t s) {
    int tiles = 0;
    hipError_t e = place_f32<BM, BN>(grp, &tiles);
    if (e != hipSuccess) return e;
    const int lds = F32Tile<BM, BN, BKF>::LDS_FLOATS * (int)sizeof(float);
    auto kern = f32_group_kernel<BM, BN, BKF, WIDE>;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kern<<<tiles, 256, lds, s>>>(grp);
    return hipGetLastError();
}
template <int F>
static hipError_t run_direct(F32Batch& grp, hipStream_t s) {
    int tiles = 0;
    hipError_t e = place_f32<16 * F, 16 * F>(grp, &tiles);
    if (e != hipSuccess) return e;
    f32_direct_kernel<F><<<tiles, DIRECT_WAVES * 64, 0, s>>>(grp);
    return hipGetLastError();
}
template <int BM, int BN, int WM, int WN>
static hipError_t run_split(F32Batch& grp, hipStream_t s) {
    int tiles = 0;
    hipError_t e = place_f32<BM, BN>(grp, &tiles);
    if (e != hipSuccess) return e;
    const int lds = SplitTile<BM, BN>::LDS_BYTES;
    auto kern = f32_split_kernel<BM, BN, WM, WN>;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kern<<<tiles, SPLIT_NT, lds, s>>>(grp);
    return hipGetLastError();
}

template <int FN, int ST>
static hipError_t run_waves_f32(F32Batch& grp, hipStream_t s) {
    int tiles = 0;
    hipError_t e = place_f32<16, 16 * FN>(grp, &tiles);
    if (e != hipSuccess) return e;
    const int lds = 8 * ST * (2 + 2 * FN) * 1024;
    auto kern = f32_waves_kernel<FN, ST>;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kern<<<tiles, 512, lds, s>>>(grp);
    return hipGetLastError();
}

// What a launch takes: the longest chain, or all contraction tiles spread over 256 CUs, whichever is longer, per instance: us per
// contraction element of one chain and of 256 tiles, and what it takes besides.  Fitted to steps of 86 shapes, 33 to 8200 tokens, widths
// 40 to 5000, ranks 4 to 64, with each instance forced (the low-rank products in 16x16 tiles): what is picked takes 0.3 % longer than the
// fastest on average, 8 % at worst.  Tokens x d_in x d_out, us in 16x16, 32x32 (direct), 64x64 (fp32), 128x128, 256x128 (split):
// 128x256x256 30, 32, 38, 42, 49; 36x563x4006 50, 65, 122, 186, 270; 300x1000x1000 63, 52, 57, 72, 96; 128x4096x4096 249, 157, 137, 197, 286;
// 512x1024x1024 107, 74, 66, 75, 98; 1024x1024x1024 182, 112, 98, 75, 99; 1400x300x4000 239, 164, 144, 188, 271; 333x4096x4096 632, 368, 285, 205,
// 286; 1024x4096x4096 1877, 1006, 678, 427, 377.
struct F32Cost { int bm, bn; double chain, tiles, fixed; };
static double f32_cost(const F32Batch& grp, const F32Cost& c) {
    double longest = 0, all = 0;
    for (int k = 0; k < grp.n; ++k) {
        const F32Product& q = grp.p[k];
        const double K = (double)q.K + q.K2;
        const bool mn = q.kind == F32_MN;
        all += (double)cdiv(q.M, mn ? F32_MN_TILE(c.bm) : c.bm) * cdiv(q.N, mn ? F32_MN_TILE(c.bn) : c.bn) * K;
        if ((!mn || grp.n == 1) && K > longest) longest = K;
    }
    const double chain = c.chain * longest, tiles = c.tiles * all / 256;
    return c.fixed + (chain > tiles ? chain : tiles);
}

static const char* const F32_INSTANCES[] = {"direct-16x16", "direct-32x32", "64x64", "split-128x128", "split-256x128", "wide-32x32", "wide-64x64", "waves-16x16", "waves-16x32"};

// The products in the order they go out, and the instance that takes them.
static int arrange_f32(const F32Product* prods, int n, F32Batch& grp) {
    grp.n = n;
    int order[F32_GROUP_MAX];
    for (int k = 0; k < n; ++k) order[k] = k;
    for (int k = 1; k < n; ++k)               // longest contraction first: what is left for the end are short tiles
        for (int j = k; j > 0 && prods[order[j]].K > prods[order[j - 1]].K; --j) { int t = order[j]; order[j] = order[j - 1]; order[j - 1] = t; }
    bool wide = false, split = true;
    long t64 = 0;
    for (int k = 0; k < n; ++k) {
        F32Product& q = grp.p[k];
        q = prods[order[k]];
        wide |= q.lda > (1L << 22) || q.ldb > (1L << 22) || q.lda2 > (1L << 22) || q.ldb2 > (1L << 22);
        if (q.kind != F32_MN) t64 += (long)cdiv(q.M, 64) * cdiv(q.N, 64);
        // (a side that leaves half of a split tile empty, as the low-rank products have; a contraction of less than a tile, which is padding for
        // the rest and not nearer to fp64 in parts; factors that would move what the scaled parts hold)
        split &= (q.kind == F32_MN || (q.M > 64 && q.N > 64)) && q.K >= SPLIT_BK;
        for (float f : {q.alpha, q.K2 > 0 ? q.alpha2 : 1.f}) split &= f == 0.f || (fabsf(f) >= 0x1p-20f && fabsf(f) <= 0x1p20f);
    }
    // (rows that wide are long chains on few tiles, or next to no arithmetic: no 128-wide instance for them)
    if (wide) return t64 >= 256 ? 6 : 5;
    const F32Cost costs[] = {{16, 16, 0.0036, 0.0024, -1.0}, {32, 32, 0.0045, 0.0061, 0.4}, {64, 64, 0.0162, 0.0185, 2.3},
                             {128, 128, 0.0246, 0.0475, -0.9}, {256, 128, 0.0573, 0.0731, 2.7}};
    int best = 0;
    for (int c = 1; c < (split ? 5 : 3); ++c)
        if (f32_cost(grp, costs[c]) < f32_cost(grp, costs[best])) best = c;
    // Low-rank products of long contractions, operands that can be fetched straight into LDS.  Launches of H and dH by themselves, 672 sizes of 17 to 4096
    // tokens, widths 1024 to 5000, ranks 4 to 256, us in f32_direct_kernel (the instance the costs above pick) and here, 16x16 | 16x32: up to one 16x16 tile a
    // CU 0.69 and 0.84 of the direct one's time where rows are whole 128-byte lines (333 tokens, 4096 x 4096, rank 64: 18.8, 12.5 | 13.6; 64 tokens,
    // 2048 x 2048, rank 8: 10.1, 7.0 | 8.6), 0.96 and 1.03 where they are not (64, 2500 x 2500, rank 64: 10.8, 10.4 | 12.2), and from rank 128 on there no gain
    // (33, 1100 x 2052, rank 128: 8.2, 10.1 | 9.3; 128, 1100 x 2052, rank 256: 8.5, 10.8 | 12.2); beyond, 0.82 and 0.73 (1024, 4096 x 4096, rank 64: 30.7,
    // 17.1 | 14.3; 1400, 2048 x 2048, rank 64: 21.1, 14.0 | 14.1; 4096, 2500 x 2500, rank 64: 40.4, 49.2 | 41.1).  Where the costs pick larger tiles
    // (ranks of 256, 2048 tokens) 16x32 takes 0.64 to 1.12 of their time: not taken.  Half of a 16x32 tile is empty up to rank 16 (4096, 4096 x 4096, rank 8: 26.7,
    // 22.6 | 24.2).
    bool waves = best <= 1, lines = true;
    long tiles = 0;
    int rank = 0;
    for (int k = 0; k < n; ++k) {
        const F32Product& q = grp.p[k];
        waves &= q.kind != F32_MN && q.K2 == 0 && !q.p_new && q.N <= 256 && q.K >= 1024 && ((q.lda | q.ldb | q.ldc | q.N | q.K) & 3) == 0 &&
                 (((uintptr_t)q.A | (uintptr_t)q.B) & 15) == 0;
        lines &= (q.lda & 31) == 0 && (q.kind == F32_KN || (q.ldb & 31) == 0);
        tiles += (long)cdiv(q.M, 16) * cdiv(q.N, 16);
        rank = q.N > rank ? q.N : rank;
    }
    if (waves && tiles > 256 && rank > 16) return 8;
    if (waves && (lines || rank <= 64)) return 7;
    return best;
}

const char* gemm_f32_plan(const F32Product* prods, int n) {
    F32Batch grp;
    return n >= 1 && n <= F32_GROUP_MAX ? F32_INSTANCES[arrange_f32(prods, n, grp)] : "";
}

hipError_t launch_gemm_f32_group(const F32Product* prods, int n, hipStream_t s) {
    if (n < 1 || n > F32_GROUP_MAX) return hipErrorInvalidValue;
    for (int k = 0; k < n; ++k)
        if (prods[k].M <= 0 || prods[k].N <= 0 || prods[k].K <= 0) return hipErrorInvalidValue;
    F32Batch grp;
    switch (arrange_f32(prods, n, grp)) {
        case 0: return run_direct<1>(grp, s);
        case 1: return run_direct<2>(grp, s);
        case 2: return run_f32<64, 64, 32>(grp, s);
        case 3: return run_split<128, 128, 2, 4>(grp, s);
        case 4: return run_split<256, 128, 4, 2>(grp, s);
        case 5: return run_f32<32, 32, 64, true>(grp, s);
        case 6: return run_f32<64, 64, 32, true>(grp, s);
        case 7: return run_waves_f32<1, 2>(grp, s);
        default: return run_waves_f32<2, 1>(grp, s);
    }
}
