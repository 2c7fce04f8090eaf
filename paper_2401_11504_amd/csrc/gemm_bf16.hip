// bf16 MFMA GEMMs for the LoRA-adapted linear layers (gfx950).
//
//  gemm_nt : C = alpha (A B^T + A2 B2^T) (+ R)      both operand pairs are K-contiguous.
//            Forward:  Y  = X W^T  + Hs B^T           (A2 = Hs = s X A^T, K2 = r)
//            Backward: dX = dY Wt^T + dH At^T          (Wt, At = transposed copies, K2 = r)
//            Low-rank: Hs = s X A^T, dH = s dY Bt^T    (N = r: mostly nt_waves_kernel)
//            The low-rank term rides along as extra K tiles of the same accumulator, so the
//            frozen product and the LoRA correction are one pass over the output.
//  gemm_tn : C = alpha P^T Q, contraction over the token dimension (dA = dH^T X, dB = dY^T Hs),
//            fp32 output.  Operand tiles lie in LDS as in memory and are read transposed.
//
// LDS tiles hold 64 contraction elements per row, padded to 72 so that the 16-byte fragment
// reads of 8 consecutive rows fall into distinct banks.
#include "kernels.h"
#include "tiles.h"
#include <algorithm>
#include <type_traits>

// ======================================================================== NT
// Workgroup ids go round-robin over the 8 XCDs (each with its own L2).  XCD c therefore runs ids c, c + 8, ..: give
// it the contiguous tile range that starts after the ranges of XCDs 0 .. c-1 (the first n % 8 XCDs hold one tile
// more), so that the CUs of one XCD work on neighbouring tiles and share operand rows in their L2.
__device__ __forceinline__ int xcd_contiguous(int id, int n) {
    const int c = id & 7, q = n >> 3, rem = n & 7;
    return c * q + min(c, rem) + (id >> 3);
}

template <int BM, int BN, int WM, int WN, bool PARTIAL>
__global__ __launch_bounds__(256) void gemm_nt_kernel(GemmNT p, int tiles_m, int tiles_n, int split_k) {
    extern __shared__ __align__(16) unsigned char smem[];
    bf16_t* sA = (bf16_t*)smem;       // [2][BM * LS]
    bf16_t* sB = sA + 2 * BM * LS;    // [2][BN * LS]
    constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32;
    constexpr int CA = BM / 32, CB = BN / 32;  // 16-byte chunks per thread per tile
    static_assert(WM * WN == 4 && FM >= 1 && FN >= 1, "4 waves");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int l32 = lane & 31, g = lane >> 5;

    // XCD-aware tile order: consecutive workgroup ids go round-robin over the 8 XCDs, so give
    // XCD x the contiguous tile range [x * n/8, (x+1) * n/8): its CUs then share W columns in its L2.
    const int ntiles = tiles_m * tiles_n;
    int pid = blockIdx.x;
    pid = xcd_contiguous(pid, ntiles);
    const int tile_m = pid % tiles_m, tile_n = pid / tiles_m;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int z = blockIdx.z, split = blockIdx.y;

    const bf16_t* A = p.A + (long)z * p.bA;
    const bf16_t* B = p.B + (long)z * p.bB;
    const bf16_t* A2 = p.A2 ? p.A2 + (long)z * p.bA2 : nullptr;
    const bf16_t* B2 = p.B2 ? p.B2 + (long)z * p.bB2 : nullptr;

    const int nk1 = (p.K + BK - 1) / BK, nk2 = (p.K2 + BK - 1) / BK;
    const int nk = nk1 + nk2;
    const int kt_begin = (int)((long)nk * split / split_k), kt_end = (int)((long)nk * (split + 1) / split_k);

    uint4 ra[CA], rb[CB];
    auto gload = [&](int kt) {
        const bf16_t *pa, *pb;
        long la, lb;
        int k0, kmax;
        if (kt < nk1) { pa = A; pb = B; la = p.lda; lb = p.ldb; k0 = kt * BK; kmax = p.K; }
        else { pa = A2; pb = B2; la = p.lda2; lb = p.ldb2; k0 = (kt - nk1) * BK; kmax = p.K2; }
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int c = tid + 256 * i, row = c >> 3, kk = k0 + (c & 7) * 8;
            ra[i] = (m0 + row < p.M && kk < kmax) ? *(const uint4*)(pa + (long)(m0 + row) * la + kk)
                                                  : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int c = tid + 256 * i, row = c >> 3, kk = k0 + (c & 7) * 8;
            rb[i] = (n0 + row < p.N && kk < kmax) ? *(const uint4*)(pb + (long)(n0 + row) * lb + kk)
                                                  : make_uint4(0, 0, 0, 0);
        }
    };
    auto sstore = [&](int buf) {
        bf16_t* a = sA + buf * BM * LS;
        bf16_t* b = sB + buf * BN * LS;
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int c = tid + 256 * i;
            *(uint4*)(a + (c >> 3) * LS + (c & 7) * 8) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int c = tid + 256 * i;
            *(uint4*)(b + (c >> 3) * LS + (c & 7) * 8) = rb[i];
        }
    };

    f32x16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    if (kt_begin < kt_end) {
        gload(kt_begin);
        sstore(0);
    }
    __syncthreads();
    for (int kt = kt_begin; kt < kt_end; ++kt) {
        const int buf = (kt - kt_begin) & 1;
        if (kt + 1 < kt_end) gload(kt + 1);
        const bf16_t* a = sA + buf * BM * LS + (wm * TM + l32) * LS + g * 8;
        const bf16_t* b = sB + buf * BN * LS + (wn * TN + l32) * LS + g * 8;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8_t fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[i] = *(const bf16x8_t*)(a + i * 32 * LS + ks * 16);
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = *(const bf16x8_t*)(b + j * 32 * LS + ks * 16);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = mfma32(fa[i], fb[j], acc[i][j]);
        }
        if (kt + 1 < kt_end) sstore(buf ^ 1);
        __syncthreads();
    }

    // epilogue: lane holds column l32 and rows 8*(v/4) + 4*g + v%4 of each 32x32 fragment
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = n0 + wn * TN + j * 32 + l32;
            if (col >= p.N) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm * TM + i * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                if (row >= p.M) continue;
                if (PARTIAL) {
                    p.partial[(((long)z * split_k + split) * p.M + row) * p.N + col] = acc[i][j][v];
                } else {
                    const long off = (long)z * p.bC + (long)row * p.ldc + col;
                    float val = p.alpha * acc[i][j][v];
                    if (p.c_f32) {
                        if (p.R) val += p.R[off];
                        ((float*)p.C)[off] = val;
                    } else {
                        ((bf16_t*)p.C)[off] = f32_to_bf16(val);
                    }
                }
            }
        }
}


__global__ void splitk_reduce_kernel(GemmNT p, int split_k);

// ======================================================================== NT, direct-to-LDS pipeline
// Same contract as gemm_nt_kernel.  Operand tiles go from global memory straight into LDS (global_load_lds_dwordx4: each
// lane's 16 bytes land at M0 + 16 * lane), so whole rings of tiles are in flight without staging registers.  A tile row
// is 64 bf16 = one 128-byte cache line = 8 chunks of 16 bytes; chunk c of row r is kept at position c ^ ((r / 2) % 8),
// chosen by which global chunk each lane fetches.  The LDS serves 16 lanes x 16 bytes per clock from 64 banks, and two
// rows span the 64 banks once, so 16 consecutive rows reading the same logical chunk must land on 8 distinct positions
// in the even rows and 8 in the odd rows: that is what the (r / 2) term gives.
// Rows beyond M / N are clamped to the last valid row: they only feed outputs that are never stored.
// Accumulates in place, in accumulation registers.  As a builtin the compiler renames the accumulators of the 192- and
// 128-column instances from one k-step to the next and moves every one of them (a quarter of the loop's issue slots).
__device__ __forceinline__ void mfma16_acc(f32x4_t& c, bf16x8_t a, bf16x8_t b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// How a launch maps workgroup ids to tiles and contraction ranges, worked out on the host: the kernel's prologue is
// exposed time on every launch, and integer divisions by run-time values cost it dozens of scalar instructions each.
// q = n / d for the small n that occur here is umulhi(n, ceil(2^32 / d)) (exact while n * d < 2^32).
struct NtMap {
    int tiles_m, tiles_n;
    unsigned inv_tiles_m;    // ceil(2^32 / tiles_m)
    unsigned inv_n_split;    // ceil(2^32 / n_split)
    int xcd_split;           // 1: the XCD a workgroup runs on also fixes its split (n_split 2, 4 or 8 and tiles divide evenly)
    int xs_log2;             // log2 of the XCDs per split in that case
    int tiles_per_xs;        // tiles / XCDs per split
};
static NtMap make_nt_map(int tiles_m, int tiles_n, int n_split, int batch, bool splitk) {
    NtMap m;
    m.tiles_m = tiles_m;
    m.tiles_n = tiles_n;
    m.inv_tiles_m = (unsigned)((0x100000000ull + (unsigned)tiles_m - 1) / (unsigned)tiles_m);
    m.inv_n_split = (unsigned)((0x100000000ull + (unsigned)n_split - 1) / (unsigned)n_split);
    const int ntiles = tiles_m * tiles_n, xs = 8 / (n_split > 0 ? n_split : 1);
    m.xcd_split = splitk && batch == 1 && (n_split == 2 || n_split == 4 || n_split == 8) && ntiles % xs == 0;
    m.xs_log2 = xs == 4 ? 2 : xs == 2 ? 1 : 0;
    m.tiles_per_xs = m.xcd_split ? ntiles / xs : 0;
    return m;
}
__device__ __forceinline__ unsigned div_by(unsigned n, unsigned inv) { return inv == 0 ? n : __umulhi(n, inv); }   // inv == 0 encodes d = 1

// Four waves, each with a (BM / 2) x (BN / 2) share of the tile, one wave per SIMD for the large tiles.
//
// The order of the contraction: first the "edge" tiles -- the low-rank pair A2 B2^T, and the last K % 64 elements of
// A B^T -- then the whole 64-wide tiles of A B^T.  Edge tiles may be narrower than 64: lanes with nothing to fetch store zeros
// to LDS instead.  With the usual ranks they are all fetched by the prologue, and the loop proper fetches only whole tiles
// through pointers that advance by a constant.
//
// The A operand has AST tiles of LDS, the B operand (the weights, which come from HBM) one more: a tile of B is fetched
// AST tiles ahead of its use during the first k-step, a tile of A at the end of the tile whose place it takes.  One
// barrier per tile ("hand-over"): before the second k-step every wave has read the whole tile (its places may be
// refilled) and the next tile has landed.  Nothing is issued in bursts: the fragments of the next k-step and the fetches
// are spread between the MFMAs, at most as fast as the LDS (one 16-byte read per wave and three MFMAs) and the address
// unit take them, so that with the 256-wide tiles the matrix pipe is what the wave waits for (256x128 and 128x128 tiles
// request more bytes per flop: 53 to 58 GB/s per CU of the 60 that the loads reach alone with cold weights).
//
// Measured, M = 2048, N = 32000, K = 4096, weights cold: 455 us (1180 TFLOP/s) with 256x256 tiles of eight waves,
// v_mfma_f32_32x32x16_bf16, a barrier every 32 contraction elements; 413 us with four waves and one barrier every 64;
// 370 us (1450 TFLOP/s) with v_mfma_f32_16x16x32_bf16, which draws less power (the chip is power-limited here: it then
// runs at 2.0 instead of 1.8 GHz), and the reads spread over the k-step.
template <int BM, int BN, int AST, bool SPLITK>
__global__ __launch_bounds__(256, 1) void gemm_nt_dl_kernel(GemmNT p, NtMap map) {
    constexpr int NT = 256, BST = AST + 1;
    constexpr int ROWB = BK * 2;                                // bytes per tile row
    constexpr int LA = BM * 8 / NT, LB = BN * 8 / NT;           // 16-byte fetches per thread per tile
    constexpr int A_STAGE = BM * ROWB, B_STAGE = BN * ROWB, B_RING = AST * A_STAGE;
    constexpr int TM = BM / 2, TN = BN / 2, FM = TM / 16, FN = TN / 16;
    static_assert(LA >= 1 && LB >= 1 && FM >= 1 && FN >= 1 && AST >= 2, "tile shape");
    extern __shared__ __align__(16) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)smem;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, g = lane >> 4;

    // Workgroup ids go round-robin over the 8 XCDs (x fastest, then y), each with its own L2: XCD c gets a contiguous
    // range of tiles (m fastest), so that its CUs share weight rows.  With the contraction split 2, 4 or 8 ways the
    // XCD also fixes the split: XCD c works on split c / (8 / n_split) only, so an XCD fetches just its share of the
    // contraction range of the activations instead of all of it.
    const int tiles_m = map.tiles_m;
    const int ntiles = tiles_m * map.tiles_n;
    const int n_split = SPLITK ? (int)gridDim.y : 1;
    int pid = blockIdx.x, split = SPLITK ? (int)blockIdx.y : 0;
    if (SPLITK && map.xcd_split) {
        const int id = blockIdx.y * gridDim.x + blockIdx.x, c = id & 7, j = id >> 3;
        split = c >> map.xs_log2;
        pid = (c & ((1 << map.xs_log2) - 1)) * map.tiles_per_xs + j;
    } else {
        pid = xcd_contiguous(pid, ntiles);
    }
    const int tile_n = (int)div_by((unsigned)pid, map.inv_tiles_m), tile_m = pid - tile_n * tiles_m;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int z = blockIdx.z;

    const bf16_t* A = p.A + (long)z * p.bA;
    const bf16_t* B = p.B + (long)z * p.bB;
    const bf16_t* A2 = p.A2 ? p.A2 + (long)z * p.bA2 : nullptr;
    const bf16_t* B2 = p.B2 ? p.B2 + (long)z * p.bB2 : nullptr;
    // edge tiles: the low-rank pair, then the ragged end of the main pair
    const int n_low = (p.K2 + BK - 1) / BK, nk1 = p.K / BK;
    const int n_edge_all = n_low + ((p.K & (BK - 1)) ? 1 : 0), nk_all = n_edge_all + nk1;
    // with SPLITK, n_split workgroups share one output tile: this one takes tiles [kt0, kt0 + nk) of that order
    const int kt0 = SPLITK ? (int)div_by((unsigned)(nk_all * split), map.inv_n_split) : 0;
    const int nk = (SPLITK ? (int)div_by((unsigned)(nk_all * (split + 1)), map.inv_n_split) : nk_all) - kt0;
    const int n_edge = max(0, min(nk, n_edge_all - kt0));
    const bf16_t* Am = A + (long)max(0, kt0 - n_edge_all) * BK;       // first whole tile of this workgroup
    const bf16_t* Bm = B + (long)max(0, kt0 - n_edge_all) * BK;

    // byte offsets of this thread's chunks within a tile of the main pair; its logical chunk is the same in every row
    const int chunk = (tid & 7) ^ ((tid >> 4) & 7), trow = tid >> 3;
    unsigned va[LA], vb[LB];
#pragma unroll
    for (int j = 0; j < LA; ++j)   // 32-bit arithmetic: the launcher only takes this path for operands below 2^30 elements
        va[j] = ((unsigned)min(m0 + trow + 32 * j, p.M - 1) * (unsigned)p.lda + chunk * 8) * 2;
#pragma unroll
    for (int j = 0; j < LB; ++j)
        vb[j] = ((unsigned)min(n0 + trow + 32 * j, p.N - 1) * (unsigned)p.ldb + chunk * 8) * 2;
    const unsigned wdst = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);

    // fetch an edge tile's A rows or B rows (t counts from this workgroup's first tile); zeros where there is nothing
    auto fetch_edge = [&](int t, auto side, unsigned slot) {
        constexpr bool b_side = decltype(side)::value;
        const int e = kt0 + t;
        int valid;          // chunks
        const bf16_t* src;
        long ld;
        if (e < n_low) {
            const int k0 = e * BK;
            valid = min(BK, p.K2 - k0) >> 3;
            src = (b_side ? B2 : A2) + k0;
            ld = b_side ? p.ldb2 : p.lda2;
        } else {
            valid = (p.K & (BK - 1)) >> 3;
            src = (b_side ? B : A) + (long)nk1 * BK;
            ld = b_side ? p.ldb : p.lda;
        }
        const int r0 = (b_side ? n0 : m0) + trow, last = (b_side ? p.N : p.M) - 1;
#pragma unroll
        for (int j = 0; j < (b_side ? LB : LA); ++j) {
            const int row = min(r0 + 32 * j, last);
            const unsigned dst = slot + wave * 1024 + j * NT * 16;      // LDS offset of this wave's 64 chunks
            if (chunk < valid)
                load_lds16(((unsigned)row * (unsigned)ld + chunk * 8) * 2, src, __builtin_amdgcn_readfirstlane(lds0 + dst));
            else
                *(uint4*)(smem + dst + lane * 16) = make_uint4(0, 0, 0, 0);
        }
    };

    using T_ = std::true_type; using F_ = std::false_type;
    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // fragment reads: row (w * T + l16), chunk 4 ks + g, swizzled by the row
    const int coff0 = (g ^ (l16 >> 1)) << 4, coff1 = ((4 + g) ^ (l16 >> 1)) << 4;
    const unsigned char* a_ptr = smem + (wm * TM + l16) * ROWB;
    const unsigned char* b_ptr = smem + B_RING + (wn * TN + l16) * ROWB;
    constexpr int NMF = FM * FN, NRD = FM + FN;
    constexpr int RSP = NMF / NRD >= 3 ? 3 : NMF >= 32 ? 2 : 1;           // MFMAs per fragment read
    constexpr int BSP = NMF / LB >= 6 ? 6 : NMF / LB, ASP = NMF / LA;     // MFMAs per fetch
    static_assert(BSP >= 1 && ASP >= 1 && RSP * NRD <= NMF, "every read and fetch of a k-step has a slot");

    // prologue: the first AST tiles of both operands (rolled: code that a launch jumps over is an instruction-cache miss)
#pragma unroll 1
    for (int s = 0; s < min(AST, nk); ++s) {
        const unsigned as = s * A_STAGE, bs = B_RING + s * B_STAGE;
        if (s < n_edge) {
            fetch_edge(s, F_{}, as);
            fetch_edge(s, T_{}, bs);
        } else {
            const bf16_t *pa = Am + (long)(s - n_edge) * BK, *pb = Bm + (long)(s - n_edge) * BK;
#pragma unroll
            for (int j = 0; j < LA; ++j) load_lds16(va[j], pa, wdst + as + j * NT * 16);
#pragma unroll
            for (int j = 0; j < LB; ++j) load_lds16(vb[j], pb, wdst + bs + j * NT * 16);
        }
    }
    bf16x8_t fa[2][FM], fb[2][FN];
    unsigned sa = 0, sb = 0, sbw = AST * B_STAGE;     // LDS offsets: the current tile's places, the place of B to fill
    // wait until at most the fetches of the r youngest tiles are outstanding (exact: those are whole tiles, A before B)
    auto wait_tiles = [&](int r) {
        static_assert((AST - 1) * (LA + LB) <= 63, "s_waitcnt vmcnt is a 6-bit field");
        if (r <= 0) wait_vmcnt<0>();
        else if (r == 1 || AST == 2) wait_vmcnt<LA + LB>();
        else if (r == 2 || AST == 3) wait_vmcnt<(AST > 2 ? 2 : 1) * (LA + LB)>();
        else wait_vmcnt<(AST - 1) * (LA + LB)>();
    };
    // A wave may have skipped fetches of a narrow edge tile: those cannot be counted, and whoever needs a tile behind one waits
    // for everything in flight.
    const bool narrow = ((p.K | p.K2) & (BK - 1)) != 0;
    wait_tiles(n_edge == 0 || !narrow ? min(nk, AST) - 1 : 0);      // tile 0 has landed
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (nk > 0) {
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[0][i] = *(const bf16x8_t*)(a_ptr + i * 16 * ROWB + coff0);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[0][j] = *(const bf16x8_t*)(b_ptr + j * 16 * ROWB + coff0);
    }

    // One k-step on fragment set CUR: the slot behind MFMA e carries one fragment read of the next k-step (in the order
    // A0, B0 .. B(FN-1), A1 ..: what its first MFMAs need first) and, if FETCH, one fetch of the operand whose place is free:
    // B during the first k-step of a tile, A during the second.
    auto kstep = [&](auto cur_c, auto reads_c, auto fetch_c, const unsigned char* ra, const unsigned char* rb,
                     const bf16_t* src, unsigned dst) {
        constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1;
        constexpr bool READS = decltype(reads_c)::value, FETCH = decltype(fetch_c)::value;
#pragma unroll
        for (int e = 0; e < NMF; ++e) {
            // operands swapped: lane (l16, g) then holds row l16, columns 4 g .. 4 g + 3 of the fragment
            mfma16_acc(acc[e / FN][e % FN], fb[CUR][e % FN], fa[CUR][e / FN]);
            if constexpr (READS) {
                if (e % RSP == 0 && e / RSP < NRD) {
                    const int r = e / RSP;
                    if (r == 0) fa[NXT][0] = *(const bf16x8_t*)ra;
                    else if (r <= FN) fb[NXT][r - 1] = *(const bf16x8_t*)(rb + (r - 1) * 16 * ROWB);
                    else fa[NXT][r - FN] = *(const bf16x8_t*)(ra + (r - FN) * 16 * ROWB);
                }
            }
            if constexpr (FETCH) {
                if constexpr (CUR == 0) {
                    if (e % BSP == (BSP > 1 ? 1 : 0) && e / BSP < LB) load_lds16(vb[e / BSP], src, dst + (e / BSP) * NT * 16);
                } else {
                    if (e % ASP == (ASP > 1 ? 1 : 0) && e / ASP < LA) load_lds16(va[e / ASP], src, dst + (e / ASP) * NT * 16);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using C0 = std::integral_constant<int, 0>; using C1 = std::integral_constant<int, 1>;
    const bf16_t *pa = Am + (long)max(0, AST - n_edge) * BK, *pb = Bm + (long)max(0, AST - n_edge) * BK;   // next whole tiles to fetch
    // fetches that may still be outstanding at the hand-over of a steady-state tile (the younger tiles')
    constexpr int HW = (AST - 1) * LB + (AST - 2) * LA;
    static_assert(HW <= 63, "s_waitcnt vmcnt is a 6-bit field");
    // the last AST tiles fetch nothing, and the tiles still in flight can be counted unless they are narrow edge tiles from the
    // loop for those
    const bool counted = !narrow || n_edge <= AST || nk >= n_edge + AST;
    auto next = [](unsigned s, unsigned stage, unsigned ring) { return s + stage == ring ? 0u : s + stage; };
    // MODE 2: fetch whole tiles; 1: fetch edge tiles; 0: fetch nothing (the last AST tiles)
    auto tile = [&](auto mode_c, auto last_c, int kt) {
        constexpr int MODE = decltype(mode_c)::value;
        constexpr bool LAST = decltype(last_c)::value;
        const unsigned char *ra = a_ptr + sa, *rb = b_ptr + sb;
        using FETCH = std::integral_constant<bool, MODE == 2>;
        if constexpr (MODE == 1) fetch_edge(kt + AST, T_{}, B_RING + sbw);
        kstep(C0{}, T_{}, FETCH{}, ra + coff1, rb + coff1, pb, wdst + B_RING + sbw);
        const unsigned da = wdst + sa, sa_old = sa;
        sa = next(sa, A_STAGE, AST * A_STAGE);
        sb = next(sb, B_STAGE, BST * B_STAGE);
        sbw = next(sbw, B_STAGE, BST * B_STAGE);
        if constexpr (!LAST) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (MODE == 2 || (MODE == 1 && !narrow)) wait_vmcnt<HW>(); else wait_tiles(MODE == 0 && counted ? nk - 2 - kt : 0);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if constexpr (MODE == 1) fetch_edge(kt + AST, F_{}, sa_old);
            kstep(C1{}, T_{}, FETCH{}, a_ptr + sa + coff0, b_ptr + sb + coff0, pa, da);
        } else {
            kstep(C1{}, F_{}, F_{}, ra, rb, pa, da);
        }
        if constexpr (MODE == 2) { pa += BK; pb += BK; }
    };
    int kt = 0;
    // more edge tiles than the prologue fetches (ranks above 64 or so)
    for (; kt < n_edge - AST; ++kt) tile(C1{}, F_{}, kt);
    for (; kt < nk - AST; ++kt) tile(std::integral_constant<int, 2>{}, F_{}, kt);
    for (; kt < nk - 1; ++kt) tile(C0{}, F_{}, kt);
    if (nk > 0) tile(C0{}, T_{}, kt);

    // Ordinary instructions read the accumulators from here on.  The compiler does not see the matrix instructions inside
    // the asm statements, so the wait for their last results is spelled out, and every accumulator passes through a
    // statement behind it so that no read can be moved in front.
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));

    // Output.  A lane holds four neighbouring columns of one row per fragment; each wave turns its share of the tile around
    // in LDS so that rows leave as 16-byte pieces of TN contiguous columns.  The stores run in a rolled loop: unrolled over
    // the fragments with their bounds checks they were 50 KB of code.  (LDS operations of one wave execute in order, so the
    // slab needs no waits of its own.)
    __builtin_amdgcn_s_barrier();  // every wave is done reading operand tiles
    asm volatile("" ::: "memory");
    // (lane numbers formed anew: kept across the loop they cost the 256x256 instance a spill, and with it a scratch allocation)
    const int elane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), el16 = elane & 15, eg = elane >> 4;
    const int row0 = m0 + wm * TM, col0 = n0 + wn * TN;
    const bool whole = m0 + BM <= p.M && n0 + BN <= p.N;       // workgroup-uniform: no bounds checks
    constexpr int LDS_BYTES = AST * A_STAGE + BST * B_STAGE;
    if (SPLITK || p.c_f32) {
        // fp32: each split stores its raw tile (splitk_reduce_kernel or the consumer adds the splits in index order
        // afterwards: device-wide fences inside a kernel cost a full L2 write-back on this chip), or C = alpha acc (+ R)
        constexpr int SLD = TN + 4, CPR = TN / 4;
        constexpr int PI = 4 * TM * SLD * 4 <= LDS_BYTES ? FM : FM / 2;      // fragment rows per pass
        static_assert(4 * PI * 16 * SLD * 4 <= LDS_BYTES && FM % PI == 0, "the output slab fits");
        float* slab = (float*)smem + wave * PI * 16 * SLD;
        float* C;
        const float* R = nullptr;
        long ldc;
        float alpha = 1.f;
        if constexpr (SPLITK) {
            C = p.partial + ((long)z * n_split + split) * (long)p.M * p.N;
            ldc = p.N;
        } else {
            C = (float*)p.C + (long)z * p.bC;
            if (p.R) R = p.R + (long)z * p.bC;
            ldc = p.ldc;
            alpha = p.alpha;
        }
        const bool vec = (ldc & 3) == 0 && (((size_t)C | (size_t)R) & 15) == 0;
#pragma unroll
        for (int i0 = 0; i0 < FM; i0 += PI) {
#pragma unroll
            for (int i = 0; i < PI; ++i) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const f32x4_t v = acc[i0 + i][j];
                    *(float4*)(slab + (i * 16 + el16) * SLD + j * 16 + 4 * eg) =
                        make_float4(alpha * v[0], alpha * v[1], alpha * v[2], alpha * v[3]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_wave_barrier();
            auto store4 = [&](int c, bool check) {
                const int r = c / CPR, cc = (c % CPR) * 4;
                const int row = row0 + i0 * 16 + r, col = col0 + cc;
                if (check && (row >= p.M || col >= p.N)) return;
                const long off = (long)row * ldc + col;
                float4 v = *(const float4*)(slab + r * SLD + cc);
                if (!check || (vec && col + 4 <= p.N)) {
                    if (R) {
                        const float4 q = *(const float4*)(R + off);
                        v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
                    }
                    *(float4*)(C + off) = v;
                } else {
                    const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if (col + x < p.N) C[off + x] = e[x] + (R ? R[off + x] : 0.f);
                }
            };
            if (whole && vec) {
#pragma unroll 4
                for (int c = elane; c < PI * 16 * CPR; c += 64) store4(c, false);
            } else {
#pragma unroll 2
                for (int c = elane; c < PI * 16 * CPR; c += 64) store4(c, true);
            }
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        // bf16: C = alpha acc
        constexpr int SLD = TN + 8, CPR = TN / 8;
        static_assert(4 * TM * SLD * 2 <= LDS_BYTES, "the output slab fits");
        bf16_t* slab = (bf16_t*)smem + wave * TM * SLD;
        bf16_t* C = (bf16_t*)p.C + (long)z * p.bC;
        const long ldc = p.ldc;
        const float alpha = p.alpha;
        const bool vec = (ldc & 7) == 0 && ((size_t)C & 15) == 0;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4_t v = acc[i][j];
                uint2 w;
                w.x = pack_bf16x2(alpha * v[0], alpha * v[1]);
                w.y = pack_bf16x2(alpha * v[2], alpha * v[3]);
                *(uint2*)(slab + (i * 16 + el16) * SLD + j * 16 + 4 * eg) = w;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_wave_barrier();
        if (vec && whole) {
#pragma unroll 4
            for (int c = elane; c < TM * CPR; c += 64) {
                const int r = c / CPR, cc = (c % CPR) * 8;
                *(uint4*)(C + (long)(row0 + r) * ldc + col0 + cc) = *(const uint4*)(slab + r * SLD + cc);
            }
        } else {
#pragma unroll 1
            for (int c = elane; c < TM * CPR; c += 64) {
                const int r = c / CPR, cc = (c % CPR) * 8;
                const int row = row0 + r, col = col0 + cc;
                if (row >= p.M || col >= p.N) continue;
                bf16_t* dst = C + (long)row * ldc + col;
                if (vec && col + 8 <= p.N) {
                    *(uint4*)dst = *(const uint4*)(slab + r * SLD + cc);
                } else {
                    for (int x = 0; x < 8 && col + x < p.N; ++x) dst[x] = slab[r * SLD + cc + x];
                }
            }
        }
    }
}

template <int BM, int BN, int AST, bool SPLITK>
static hipError_t run_nt_dl(const GemmNT& g, hipStream_t s, int n_split = 1) {
    const int tiles_m = cdiv(g.M, BM), tiles_n = cdiv(g.N, BN);
    const size_t lds = (size_t)(AST * BM + (AST + 1) * BN) * BK * 2;
    dim3 grid(tiles_m * tiles_n, SPLITK ? n_split : 1, g.batch);
    auto kern = gemm_nt_dl_kernel<BM, BN, AST, SPLITK>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const bool defer = SPLITK && g.deferred;                         // the consumer adds the partial tiles up
    kern<<<grid, 256, lds, s>>>(g, make_nt_map(tiles_m, tiles_n, SPLITK ? n_split : 1, g.batch, SPLITK));
    if (defer) {
        *g.deferred = n_split;
    } else if (SPLITK) {
        const long n = (long)g.M * (g.N >> 2) * g.batch;
        splitk_reduce_kernel<<<cdiv(n, 256), 256, 0, s>>>(g, n_split);
    }
    return hipGetLastError();
}

// sum the split-K partials in a fixed order (deterministic), scale, add residual, convert.  One thread owns four
// consecutive columns; the partials are fetched eight splits at a time before they are added, so that the loads
// of a batch are all in flight together instead of one L2 round trip per split.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmNT p, int split_k) {
    const long mn = (long)p.M * p.N;
    const int n4 = p.N >> 2;                      // N % 4 == 0 (checked by the launcher)
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)p.M * n4 * p.batch) return;
    const int z = (int)(idx / ((long)p.M * n4));
    const long q = idx % ((long)p.M * n4);
    const int row = (int)(q / n4), col = (int)(q % n4) * 4;
    const float* src = p.partial + (long)z * split_k * mn + (long)row * p.N + col;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    int k = 0;
    for (; k + 8 <= split_k; k += 8) {
        float4 t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = *(const float4*)(src + (long)(k + j) * mn);
#pragma unroll
        for (int j = 0; j < 8; ++j) { s.x += t[j].x; s.y += t[j].y; s.z += t[j].z; s.w += t[j].w; }
    }
    for (; k < split_k; ++k) {
        const float4 t = *(const float4*)(src + (long)k * mn);
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    const long off = (long)z * p.bC + (long)row * p.ldc + col;
    const float v[4] = {p.alpha * s.x, p.alpha * s.y, p.alpha * s.z, p.alpha * s.w};
    if (p.c_f32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ((float*)p.C)[off + e] = v[e] + (p.R ? p.R[off + e] : 0.f);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) ((bf16_t*)p.C)[off + e] = f32_to_bf16(v[e]);
    }
}

template <int BM, int BN, int WM, int WN>
static hipError_t run_nt(const GemmNT& g, int split_k, hipStream_t s) {
    const int tiles_m = cdiv(g.M, BM), tiles_n = cdiv(g.N, BN);
    const size_t lds = (size_t)2 * (BM + BN) * LS * sizeof(bf16_t);
    dim3 grid(tiles_m * tiles_n, split_k, g.batch);
    hipError_t e;
    if (split_k > 1) {
        auto kern = gemm_nt_kernel<BM, BN, WM, WN, true>;
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        kern<<<grid, 256, lds, s>>>(g, tiles_m, tiles_n, split_k);
        const long n = (long)g.M * (g.N >> 2) * g.batch;
        splitk_reduce_kernel<<<cdiv(n, 256), 256, 0, s>>>(g, split_k);
    } else {
        auto kern = gemm_nt_kernel<BM, BN, WM, WN, false>;
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        kern<<<grid, 256, lds, s>>>(g, tiles_m, tiles_n, 1);
    }
    return hipGetLastError();
}

// what every kernel here asks of a product
static bool nt_valid(const GemmNT& g) {
    return !((g.K & 7) || (g.K2 & 7) || (g.lda & 7) || (g.ldb & 7) || (g.lda2 & 7) || (g.ldb2 & 7) || (g.bA & 7) || (g.bB & 7) || (g.bA2 & 7) ||
             (g.bB2 & 7)) && (g.c_f32 || !g.R);
}
// Operands that start where direct-to-LDS loads can take them
static bool nt_loads_to_lds(const GemmNT& g) { return loads_to_lds(g.A) && loads_to_lds(g.B) && loads_to_lds(g.A2) && loads_to_lds(g.B2); }
// Whether the direct-to-LDS kernel takes this product.  Its offsets within an operand are 32-bit.  A contraction that is no
// multiple of 64 (ranks below 64, ragged widths) costs it one edge tile, waited for before the loop starts: worth it from
// 256 elements on (1024 x 1024 x 1024 with rank 16: 8 us against 14 us register-staged, back to back), below that the whole contraction
// is one or two such waits.
static bool nt_direct(const GemmNT& g) {
    if (g.K <= 0 || !nt_loads_to_lds(g)) return false;
    if (((g.K % BK) || (g.K2 % BK)) && g.K < 256) return false;
    return (long)g.M * g.lda < (1L << 30) && (long)g.N * g.ldb < (1L << 30) && (long)g.M * g.lda2 < (1L << 30) &&
           (long)g.N * g.ldb2 < (1L << 30);
}
// the same for 64x64 tiles: a narrow output over a ragged contraction (a low-rank product of a ragged width) stays with the
// register-staged kernel, whose split it shares with every other rank
static bool nt_direct_small(const GemmNT& g) { return nt_direct(g) && ((g.K % BK) == 0 || g.N >= 128); }

// The tile configurations the launcher can pick (every one is reachable from launch_gemm_nt; the kernel tests name the
// shape that lands on each).
enum NtConfig {
    // tiles of 64 contraction elements; A / B tiles in LDS
    NT_128x128,         // 128x128, 4 / 5
    NT_128x128_SPLIT,   // with the contraction split 2 to 8 ways (partials reduced afterwards or by the consumer)
    NT_256x128,         // 256x128, 3 / 4
    NT_256x128_SPLIT,
    NT_256x192,         // 256x192, 2 / 3
    NT_256x256,         // 256x256, 2 / 3
    NT_256x256_SPLIT,
    NT_REG_128x128,     // register-staged, for what nt_direct refuses: ragged contractions below 256 elements, operands beyond 1 Gi or off by half a word
    NT_REG_128x64,
    NT_SKINNY           // N <= 64 per batch or few tiles: 64x64 tiles, contraction split over up to 16 workgroups
};

// A model of the time of one launch of the direct-to-LDS kernel: full rounds of 256 tiles (one per CU), then what is left, which
// takes less the fewer CUs it keeps busy (the chip clocks higher and its memory is shared by fewer): us per 1000 contraction
// elements of a round with next to no tiles (k_min) and with 256 (k_full).  Fitted to instances forced on the products of 4096-,
// 2048- and 1024-wide layers.  Against every instance forced on the products of six layers 1024 to 5120 wide at 64 to 5120 rows, weights
// cold, 11702 timings of 1100 products: what it picks takes 1.3 % longer than the fastest instance on average (10 % at the 95th percentile;
// at worst 37 %, some products of 256 to 384 rows and width 2560 that 64x64 tiles are taken for and 128x128 in four would be faster).  A rule
// that rated each instance by operand bytes and split 256x128 tiles only is 6 % behind it; 4096 x 22016 at 256 rows 106 us against 62,
// at 5120 rows 1000 against 787.
struct NtTile { NtConfig cfg, cfg_split; int bm, bn; double k_min, k_full; };
static const NtTile kNtTiles[] = {
    {NT_SKINNY, NT_SKINNY, 64, 64, 3.1, 3.75},
    {NT_128x128, NT_128x128_SPLIT, 128, 128, 7.1, 9.0},
    {NT_256x128, NT_256x128_SPLIT, 256, 128, 9.9, 12.6},
    {NT_256x192, NT_256x192, 256, 192, 12.2, 16.9},
    {NT_256x256, NT_256x256_SPLIT, 256, 256, 15.5, 20.2},
};
struct NtPick { NtConfig cfg; int split; double us; };
// for products that the direct-to-LDS kernel takes (gemm_nt_two_parts also prices with it what choose_nt keeps from it)
static NtPick pick_nt(const GemmNT& g) {
    const double k1000 = ((double)g.K + g.K2) * 1e-3, mn = (double)g.M * g.N * g.batch;
    const int nk = cdiv(g.K, BK) + cdiv(g.K2, BK);
    const bool many = (long)cdiv(g.M, 128) * cdiv(g.N, 128) * g.batch >= 128;      // (64x64 tiles: where 128x128 leave half the CUs idle)
    // the pass over the partial tiles of a split: a reduce launch that reads them and writes C (6.3 us and 1.4 us a million values),
    // or, when the consumer adds them up itself (g.deferred), the extra bytes written here and read there
    const double pass0 = g.deferred ? 0.0 : 6.3, pass1 = g.deferred ? 1.1e-6 : 1.41e-6;
    const bool may_split = g.split_k == 0 && g.partial && !(g.N & 3);
    NtPick whole = {NT_SKINNY, 1, 1e30}, split = {NT_SKINNY, 8, 1e30};
    for (const NtTile& t : kNtTiles) {
        if (t.bm == 64 && many) continue;
        const long tiles = (long)cdiv(g.M, t.bm) * cdiv(g.N, t.bn) * g.batch;
        for (int sp = 1; sp <= 8; sp = sp == 2 ? 3 : sp == 3 ? 4 : 2 * sp) {
            if (sp > 1 && (!may_split || t.cfg_split == t.cfg || nk / sp < 8 || mn * sp > (double)g.partial_elems)) break;
            const long n = tiles * sp, rem = n & 255;
            // Three ways: for the 72 to 85 tiles that two leave a third of the chip idle on and four need two rounds for.  us without and
            // with them in 128x128 and 256x128 tiles: 2048 x 11264 at 1280 rows 71 and 64, 2560 x 13824 at 1024 82 and 73, 3072 x 8192 at 700 60
            // and 50, 5120 x 13824 at 512 83 and 75; 256x256 tiles also beyond one round, 2560 x 13824 at 1700 rows 141 and 116.
            if (sp == 3 && t.bn < 256 && (n < 213 || n > 256)) continue;
            double us = (double)(n >> 8) * t.k_full;
            if (rem) us += t.k_min + (t.k_full - t.k_min) * rem * (1.0 / 256);
            us = 2.0 + us * k1000 / sp + (sp > 1 ? pass0 + pass1 * mn * sp : 0.0);
            NtPick& best = sp > 1 ? split : whole;
            if (us < (sp > best.split ? 0.96 : 1.0) * best.us) best = {sp > 1 ? t.cfg_split : t.cfg, sp, us};
        }
    }
    return split.us < 0.96 * whole.us ? split : whole;       // (what promises less than the model's error is not worth more partial tiles)
}

static NtConfig choose_nt(const GemmNT& g, int* n_split) {
    *n_split = 1;
    const int nk = cdiv(g.K, BK) + cdiv(g.K2, BK);
    const long t128 = (long)cdiv(g.M, 128) * cdiv(g.N, 128) * g.batch;
    const long t64n = (long)cdiv(g.M, 128) * cdiv(g.N, 64) * g.batch;
    if (g.N > 64 && nt_direct(g) && (t128 >= 128 || (g.N >= 256 && g.split_k == 0))) {
        const NtPick p = pick_nt(g);
        *n_split = p.split;
        return p.cfg;
    }
    if (g.N > 64 && t128 >= 200) return NT_REG_128x128;
    if (g.N > 64 && t64n >= 200) return NT_REG_128x64;
    // a narrow output (or one the direct-to-LDS kernel refuses): 64x64 tiles, and split the contraction when scratch is available
    const long t64 = (long)cdiv(g.M, 64) * cdiv(g.N, 64) * g.batch;
    int split = g.split_k;
    if (split == 0) {
        split = 1;
        if (g.partial && t64 < 256) {
            split = (int)(512 / t64);
            if (split > nk / 4) split = nk / 4;   // at least four k-tiles per split
            if (split < 1) split = 1;
            while (split > 1 && (size_t)split * g.M * g.N * g.batch > g.partial_elems) --split;
        }
    }
    if (split > nk) split = nk > 0 ? nk : 1;
    if (g.N & 3) split = 1;   // the reduce kernel works on groups of four columns
    *n_split = split;
    return NT_SKINNY;
}

// A GEMM whose tile count leaves its last round of workgroups poorly filled can be cheaper as two launches: whole rounds of tiles
// over the first columns (of every batch) or the first rows, and the rest on its own with whatever tile and split suits it.
// 5120 rows of 4096 x 22016: 320 tiles of 256x256, a round and a quarter that costs two, 819 us, 787 in 256x192 tiles; as 4096 rows (482 us)
// and 1024 (141) 623.  A rest of 64 to 255 columns and few rows is priced by the model too, though choose_nt runs it by the rule for narrow
// outputs; us in one launch and in two of that kind: 1024 x 16576 x 3072 106 and 88, 2048 x 8288 x 3072 104 and 86, 1024 x 16448 x 4096 131
// and 104, 3008 x 5520 x 1024 49 and 45, 3264 x 2560 x 13824 207 and 208.
bool gemm_nt_two_parts(const GemmNT& g, GemmNT* a, GemmNT* b) {
    if (g.split_k > 1 || g.M < 256 || g.N < 512 || g.batch <= 0 || !nt_direct(g)) return false;
    const double second_launch_us = 3.0;
    if ((long)cdiv(g.M, 256) * cdiv(g.N, 128) * g.batch <= 256) return false;      // one round as it is
    GemmNT h = g;
    double best = 0.96 * pick_nt(h).us;
    h.deferred = nullptr;
    int rows = 0, cols = 0;
    for (const NtTile& t : kNtTiles) {
        if (t.bm < 256) continue;
        const long tm = cdiv(g.M, t.bm), tn = cdiv(g.N, t.bn), rounds = tm * tn * g.batch / 256;
        for (long r = rounds; r >= 1 && r >= rounds - 1; --r) {
            for (int by_rows = 0; by_rows < 2; ++by_rows) {
                const long first = by_rows ? 256 * r / (tn * g.batch) * t.bm : 256 * r / (tm * g.batch) * t.bn;
                const int whole = by_rows ? g.M : g.N;
                if (first <= 0 || whole - first < 64) continue;
                int& n = by_rows ? h.M : h.N;
                n = (int)first;
                double us = pick_nt(h).us;
                n = whole - (int)first;
                us += pick_nt(h).us + second_launch_us;
                n = whole;
                if (us < best) { best = us; rows = by_rows ? (int)first : 0; cols = by_rows ? 0 : (int)first; }
            }
        }
    }
    if (!rows && !cols) return false;
    const size_t out = g.c_f32 ? sizeof(float) : sizeof(bf16_t);
    if (g.deferred) *g.deferred = 0;
    *a = *b = h;
    if (rows) {
        a->M = rows;
        b->M = g.M - rows;
        b->A = g.A + (long)rows * g.lda;
        if (g.K2 > 0) b->A2 = g.A2 + (long)rows * g.lda2;
        b->C = (char*)g.C + (size_t)rows * g.ldc * out;
        if (g.R) b->R = g.R + (long)rows * g.ldc;
    } else {
        a->N = cols;
        b->N = g.N - cols;
        b->B = g.B + (long)cols * g.ldb;
        if (g.K2 > 0) b->B2 = g.B2 + (long)cols * g.ldb2;
        b->C = (char*)g.C + (size_t)cols * out;
        if (g.R) b->R = g.R + cols;
    }
    return true;
}

const char* gemm_nt_plan(const GemmNT& g, int* n_split) {
    int sp = 1;
    const NtConfig c = choose_nt(g, &sp);
    if (n_split) *n_split = sp;
    switch (c) {
        case NT_128x128: return "128x128";
        case NT_128x128_SPLIT: return "128x128-split";
        case NT_256x256_SPLIT: return "256x256-split";
        case NT_256x128: return "256x128";
        case NT_256x128_SPLIT: return "256x128-split";
        case NT_256x192: return "256x192";
        case NT_256x256: return "256x256";
        case NT_REG_128x128: return "reg-128x128";
        case NT_REG_128x64: return "reg-128x64";
        case NT_SKINNY: break;
    }
    return nt_direct_small(g) ? (sp > 1 ? "64x64-split" : "64x64") : (sp > 1 ? "reg-64x64-split" : "reg-64x64");
}

hipError_t launch_gemm_nt(const GemmNT& g, hipStream_t s) {
    if (g.deferred) {
        *g.deferred = 0;
        if (g.batch != 1 || g.alpha != 1.f) return hipErrorInvalidValue;
    }
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
    if (!nt_valid(g)) return hipErrorInvalidValue;
    int split = 1;
    switch (choose_nt(g, &split)) {
        case NT_128x128: return run_nt_dl<128, 128, 4, false>(g, s);
        case NT_256x128: return run_nt_dl<256, 128, 3, false>(g, s);
        case NT_128x128_SPLIT: return run_nt_dl<128, 128, 4, true>(g, s, split);
        case NT_256x128_SPLIT: return run_nt_dl<256, 128, 3, true>(g, s, split);
        case NT_256x256_SPLIT: return run_nt_dl<256, 256, 2, true>(g, s, split);
        case NT_256x192: return run_nt_dl<256, 192, 2, false>(g, s);
        case NT_256x256: return run_nt_dl<256, 256, 2, false>(g, s);
        case NT_REG_128x128: return run_nt<128, 128, 2, 2>(g, 1, s);
        case NT_REG_128x64: return run_nt<128, 64, 2, 2>(g, 1, s);
        case NT_SKINNY: break;
    }
    if (split > 1 && (!g.partial || (size_t)split * g.M * g.N * g.batch > g.partial_elems)) return hipErrorInvalidValue;
    if (nt_direct_small(g)) {
        if (split > 1) return run_nt_dl<64, 64, 4, true>(g, s, split);
        return run_nt_dl<64, 64, 4, false>(g, s);
    }
    return run_nt<64, 64, 2, 2>(g, split, s);
}

// ======================================================================== NT, few tiles: the waves of a workgroup split the contraction
// The same contract as gemm_nt_kernel, for outputs too small to fill the chip with tiles that pay: the few columns of a low-rank product,
// Hs = s X A^T, dH = s dY B (N = the rank, or three of them), and every product of a small decoder or a short sample.
// One launch: a workgroup computes a (16 FM) x (16 FN) tile over the whole contraction, each of its eight waves an eighth of it in
// 64-wide pieces through a ring of its own (direct-to-LDS loads of whole 128-byte rows, ST pieces in flight, no barrier), and adds
// the eight sums up through LDS in a fixed order.  What bounds it, in calls back to back, is the operand stream of a CU (some 88 GB/s with the
// weights of the factor in the L2s): the tile is the one that leaves the busiest CU the fewest bytes, and up to 32x48 the rings (48 to 80 KB) are small
// enough for two workgroups per CU, whose loads, sums and stores then overlap; wider tiles (96 to 128 KB) have one.  Behind another kernel a launch takes
// 1 to 3 us more: in an update of 1024 tokens, 64 columns of 4096 behind attention and a norm 7.3 and 8.0, beside the dA/dB launch of the other stream
// 21.2, 64 of 11008 14.5, 192 of 4096 10.8, 64 x 3 12.4.
// us against 64x64 tiles with the contraction split over up to 16 workgroups and a reduce launch behind (operands cold, calls back to back;
// columns x batch of a contraction of 4096): 1024 rows, 192: 8.0 and 12.8; 64: 5.6 and 9.7; 64 x 3: 8.5 and 13.5; 2048 rows: 9.8 and 15.4,
// 6.7 and 12.9, 12.6 and 18.1; 5120 rows: 20 and 25, 16 and 16, 22 and 28; 64 of a contraction of 11008: 512 rows 9.9 and 14.3, 1024 rows
// 10.6 and 13.5, 2048 rows 19 and 17.  Rings of 96 to 160 KB (two to five pieces ahead): up to 1 us slower.
template <int FM, int FN, int ST>
__global__ __launch_bounds__(512, 2) void nt_waves_kernel(GemmNT p, int tiles_m, int tiles_n) {
    constexpr int NL = 2 * (FM + FN), STAGE = NL * 1024, RING = ST * STAGE;      // fetches per piece; bytes
    static_assert((ST - 1) * NL <= 63 && FM * FN * 1024 <= RING && 8 * RING <= 160 * 1024, "ring");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    // the column tiles of a row tile lie on one XCD: its L2 then fetches the rows of A once
    int id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int tile_n = id % tiles_n;
    id /= tiles_n;
    const int z = id / tiles_m, tile_m = id - z * tiles_m;
    const int m0 = tile_m * 16 * FM, n0 = tile_n * 16 * FN;
    const bf16_t* A = p.A + (long)z * p.bA;
    const bf16_t* B = p.B + (long)z * p.bB;

    // fetch i of a piece brings rows 8 i .. 8 i + 7 (first of A, then of B); chunk c of row r lies at position c ^ (r / 2 % 8)
    const int r8 = lane >> 3;
    unsigned off[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const bool a = i < 2 * FM;
        const int r = (a ? i : i - 2 * FM) * 8 + r8;
        const unsigned chunk = (unsigned)((lane & 7) ^ ((r >> 1) & 7));
        off[i] = (a ? (unsigned)min(m0 + r, p.M - 1) * (unsigned)p.lda : (unsigned)min(n0 + r, p.N - 1) * (unsigned)p.ldb) * 2 + chunk * 16;
    }
    // pieces of the contraction: the low-rank pair, then the main one; the last of each may be narrow
    const int n_low = (p.K2 + BK - 1) / BK, nk = n_low + (p.K + BK - 1) / BK;
    const int k_first = nk * wave >> 3, mine = (nk * (wave + 1) >> 3) - k_first;        // this wave's pieces
    const int whole = min(n_low + p.K / BK, k_first + mine);                            // n_low .. whole - 1 are fetched without a look
    const bool narrow = (((p.K | p.K2) & (BK - 1)) != 0) && (whole < k_first + mine || k_first < n_low);
    const unsigned ring0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)smem + wave * RING);
    auto fetch = [&](int t, unsigned st) {
        const int kt = k_first + t;
        if (kt >= n_low && kt < whole) {
            const bf16_t *pa = A + (long)(kt - n_low) * BK, *pb = B + (long)(kt - n_low) * BK;
#pragma unroll
            for (int i = 0; i < NL; ++i) load_lds16(off[i], i < 2 * FM ? pa : pb, __builtin_amdgcn_readfirstlane(ring0 + st + i * 1024));
            return;
        }
        const bool low = kt < n_low;                // zeros beyond the end
        const int k0 = (low ? kt : kt - n_low) * BK, valid = min(BK, (low ? p.K2 : p.K) - k0) >> 3;
        const bf16_t* pa = (low ? p.A2 + (long)z * p.bA2 : A) + k0;
        const bf16_t* pb = (low ? p.B2 + (long)z * p.bB2 : B) + k0;
        const unsigned la = (unsigned)(low ? p.lda2 : p.lda) * 2, lb = (unsigned)(low ? p.ldb2 : p.ldb) * 2;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const bool a = i < 2 * FM;
            const int r = (a ? i : i - 2 * FM) * 8 + r8, chunk = (lane & 7) ^ ((r >> 1) & 7);
            if (chunk < valid)
                load_lds16((unsigned)(a ? min(m0 + r, p.M - 1) : min(n0 + r, p.N - 1)) * (a ? la : lb) + chunk * 16, a ? pa : pb,
                           __builtin_amdgcn_readfirstlane(ring0 + st + i * 1024));
            else
                *(uint4*)(smem + wave * RING + st + i * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
        }
    };
    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int t = 0; t < min(ST, mine); ++t) fetch(t, t * STAGE);
    const unsigned char* row = smem + wave * RING + l16 * 128;
    const int c0 = (g ^ (l16 >> 1)) << 4, c1 = ((4 + g) ^ (l16 >> 1)) << 4;
    unsigned st = 0;
    for (int t = 0; t < mine; ++t) {
        // the pieces behind this one may be in flight; narrow ones have fetches that cannot be counted
        if (t + ST <= mine && !narrow) wait_vmcnt<(ST - 1) * NL>();
        else wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        bf16x8_t fa[2][FM], fb[2][FN];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[ks][i] = *(const bf16x8_t*)(row + st + i * 2048 + (ks ? c1 : c0));
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[ks][j] = *(const bf16x8_t*)(row + st + (FM + j) * 2048 + (ks ? c1 : c0));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // its place may be filled again
        if (t + ST < mine) fetch(t + ST, st);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)      // operands swapped: lane (l16, g) then holds row l16, columns 4 g .. 4 g + 3
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
        st = st + STAGE == RING ? 0 : st + STAGE;
    }
    // the eight sums, each in its wave's own ring
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) *(f32x4_t*)(smem + wave * RING + (i * FN + j) * 1024 + lane * 16) = acc[i][j];
    __syncthreads();
    for (int e = tid; e < FM * FN * 64; e += 512) {
        f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 8; ++w) s += *(const f32x4_t*)(smem + w * RING + e * 16);
        const int f = e >> 6, el = e & 63, r = m0 + f / FN * 16 + (el & 15), c = n0 + f % FN * 16 + 4 * (el >> 4);
        if (r >= p.M || c >= p.N) continue;       // N is a multiple of 4
        const long at = (long)z * p.bC + (long)r * p.ldc + c;
        if (p.c_f32) {
            float4 v = make_float4(p.alpha * s[0], p.alpha * s[1], p.alpha * s[2], p.alpha * s[3]);
            if (p.R) {
                const float4 q = *(const float4*)(p.R + at);
                v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
            }
            *(float4*)((float*)p.C + at) = v;
        } else {
            uint2 w;
            w.x = pack_bf16x2(p.alpha * s[0], p.alpha * s[1]);
            w.y = pack_bf16x2(p.alpha * s[2], p.alpha * s[3]);
            *(uint2*)((bf16_t*)p.C + at) = w;
        }
    }
}
template <int FM, int FN, int ST>
static hipError_t run_waves(const GemmNT& g, hipStream_t s) {
    const int tiles_m = cdiv(g.M, 16 * FM), tiles_n = cdiv(g.N, 16 * FN);
    const int lds = 8 * ST * 2 * (FM + FN) * 1024;
    auto kern = nt_waves_kernel<FM, FN, ST>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kern<<<tiles_m * tiles_n * g.batch, 512, lds, s>>>(g, tiles_m, tiles_n);
    return hipGetLastError();
}
// What a tile costs: launch, ends and first loads (2.5 us), the stream of the busiest CU, and what the way from memory adds: for low-rank products the
// rows of A (us; within 15 % of the timings above but for long contractions of few rows, which are faster), for frozen ones, whose weights are
// cold, the operands of all tiles (see pick_small).
struct WavesTile { int fm, fn; const char* name; };
static const WavesTile kWavesTiles[] = {{1, 1, "16x16"}, {1, 2, "16x32"}, {2, 2, "32x32"}, {2, 3, "32x48"}, {2, 4, "32x64"}, {3, 4, "48x64"}, {4, 4, "64x64"}};
// index into kWavesTiles of the fastest of the first n_tiles that promises less than `best` us, or -1
static int pick_waves(const GemmNT& g, double best, int n_tiles, double rows_us, double all_us) {
    const size_t align = g.c_f32 ? 15 : 7;
    if (g.K <= 0 || (g.N & 3) || (g.ldc & 3) || (g.bC & 3) || ((size_t)g.C & align) || ((size_t)g.R & 15) || !nt_loads_to_lds(g))
        return -1;
    if ((long)g.M * g.lda >= (1L << 30) || (long)g.N * g.ldb >= (1L << 30) || (long)g.M * g.lda2 >= (1L << 30) || (long)g.N * g.ldb2 >= (1L << 30))
        return -1;
    int pick = -1;
    for (int i = 0; i < n_tiles; ++i) {
        const WavesTile& t = kWavesTiles[i];
        const long n = (long)cdiv(g.M, 16 * t.fm) * cdiv(g.N, 16 * t.fn) * g.batch;
        const double bytes = 32.0 * (t.fm + t.fn) * (g.K + g.K2);
        const double us = 2.5 + 11.4e-6 * bytes * (double)((n + 255) / 256) + rows_us + all_us * bytes * n;
        if (us < best) { best = us; pick = i; }
    }
    return pick;
}
static hipError_t launch_waves(const GemmNT& g, int tile, hipStream_t s) {
    switch (tile) {
        case 0: return run_waves<1, 1, 2>(g, s);
        case 1: return run_waves<1, 2, 1>(g, s);
        case 2: return run_waves<2, 2, 1>(g, s);
        case 3: return run_waves<2, 3, 1>(g, s);
        case 4: return run_waves<2, 4, 1>(g, s);
        case 5: return run_waves<3, 4, 1>(g, s);
        default: return run_waves<4, 4, 1>(g, s);
    }
}
// What the general kernel promises for a low-rank product, by the route choose_nt takes with the scratch there is: whole, for short contractions, 2.5 us
// and 3.5 per 1000 elements; long ones split and reduced 10 us and 0.095 per million operand bytes (no less than a part takes), whole 2.5
// per 1000 elements and the rows of A for every column tile, 3.5 where tiles queue; many 128-wide tiles by their own model.  us whole and here:
// 64 columns of 11008, two at once, 2048 rows 33.6 and 20.2, 64 rows 30.6 and 10.5; 192 columns of 4096, 5120 rows 22.8 and 19.1, 12000 rows 35.2
// and 38.3, 16384 rows 48.8 and 54.3; 64 columns, 16384 rows 24.6 and 25.7.
static double general_low_rank_us(const GemmNT& g) {
    if (g.split_k == 1) return 2.5 + 3.5e-3 * g.K;
    int split = 1;
    if (choose_nt(g, &split) != NT_SKINNY) return pick_nt(g).us;
    const long t64 = (long)cdiv(g.M, 64) * cdiv(g.N, 64) * g.batch;
    if (split > 1) return std::max(10.0 + 0.095e-6 * 256.0 * g.K * t64, 5.5 + 2.5e-3 * g.K / split);
    const double rows_us = 0.1e-6 * 2.0 * g.M * g.K * g.batch * cdiv(g.N, 64);
    return 2.5 + rows_us + (t64 <= 256 ? 2.5e-3 * g.K : 3.5e-3 * g.K * cdiv(t64, 256));
}
// index into kWavesTiles, or -1 for the general kernel (what that refuses is refused there)
static int pick_low_rank(const GemmNT& g) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || g.deferred || !nt_valid(g)) return -1;
    return pick_waves(g, general_low_rank_us(g), (int)(sizeof(kWavesTiles) / sizeof(kWavesTiles[0])), 0.1e-6 * 2.0 * g.M * g.K * g.batch, 0.0);
}
const char* low_rank_plan(const GemmNT& g) {
    const int i = pick_low_rank(g);
    return i < 0 ? "general" : kWavesTiles[i].name;
}
hipError_t launch_low_rank(const GemmNT& g, hipStream_t s) {
    const int i = pick_low_rank(g);
    return i < 0 ? launch_gemm_nt(g, s) : launch_waves(g, i, s);
}
// A frozen product of a small decoder or a short sample: up to half a million outputs and, each of a batch, four million weights (us in the general kernel
// and here: 200 x 256 x 688 7.0 and 4.9, 300 x 512 x 1408 8.3 and 5.8, 16 x 2048 x 2048 8.4 and 4.9; three at once, 33 x 1024 x 1024 6.4 and 5.5, 16 x 2048 x
// 2048 8.6 and 6.9; beyond, 128 x 4096 x 4096 22.8 and 22.9, 1024 x 1024 x 1024 7.8 and 9.6, 1024 x 1024 x 2816 14.3 and 15.2).  Tiles whose weights are cold get
// 67 MB a us on top of the stream of a CU, and 32x64 ones lose to the general kernel where few rows share many columns: 200 x 2048 x 2048
// 9.0 and 12.0, three times 85 x 2048 x 2048 9.4 and 14.4.  The general kernel's model is that of launches that follow one another closely;
// behind another kernel's end its chain of barriers costs 1 us more.  us of a layer with every product in the general kernel, with all five tiles by the
// stream of a CU alone, and so: 512 wide, 200 tokens 165, 153, 154; 1024 wide, 512 tokens 208, 202, 203; 1792 wide, 200 tokens 234, 238, 235; 2048 wide, 256
// tokens 281, 288, 281 (ten lengths of 64 to 900 tokens, nine widths: no layer slower than in the general kernel by more than 1.1 %, the noise).
static int pick_small(const GemmNT& g) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || !nt_valid(g) || (g.deferred && (g.batch != 1 || g.alpha != 1.f))) return -1;
    if (g.K <= 0 || g.split_k > 1 || (long)g.M * g.N * g.batch > (1L << 19) || (long)g.N * g.K > (1L << 22)) return -1;
    const double general = nt_direct(g) ? pick_nt(g).us : 2.0 + 4.2e-3 * (g.K + g.K2);
    return pick_waves(g, general + 1.0, 2L * g.N * g.batch <= 9L * g.M ? 5 : 4, 0.0, 1.5e-8);
}
const char* frozen_plan(const GemmNT& g) {
    const int i = pick_small(g);
    return i < 0 ? "general" : kWavesTiles[i].name;
}
hipError_t launch_frozen(const GemmNT& g, hipStream_t s) {
    const int i = pick_small(g);
    if (i < 0) return launch_gemm_nt(g, s);
    if (g.deferred) *g.deferred = 0;
    return launch_waves(g, i, s);
}

// ======================================================================== TN
// One 64x64 output tile of P^T Q over the 64-token tiles [it0, it1).  The operand tiles stay in LDS as they lie in
// memory, [t][i] with the token index t as rows, and the matrix unit's operands (contraction over t) come out of the
// LDS transpose read (read_tr_frag in tiles.h): no transposing stores, no bank conflicts.  Both operands use the
// same slot order, so the permutation of the 16 contraction slots of a step cancels.  Returns this wave's 32x32 accumulator.
// What bounds it: four MFMAs a wave and tile are a tenth of the time a tile takes to arrive, so it is the bytes in flight and, with many
// tokens, memory: a ring of TN_ST tiles of both operands by direct-to-LDS loads, TN_ST - 1 of them on their way, one barrier a tile.
// us of a layer's launch with one tile ahead in registers and with this: 1024 tokens of width 1024 (260 tiles) 17.6 and 11.6, 200 tokens
// (65 tiles) 8.9 and 7.0; 7B shapes (1220 tiles), 5120 tokens 235 and 211 (3.8 TB/s of operands), 1536 tokens 62 and 60.  Three tiles (and
// three workgroups on a CU) or a contiguous range of the tiles on each XCD measure the same within 3 %.
constexpr int TN_ST = 4, TN_TILE = 64 * 128, TN_STAGE = 2 * TN_TILE;     // bytes of a tile, of P's and Q's
// DIRECT: the operands start at multiples of 4 bytes; else they come through registers, a tile at a time.
template <bool DIRECT>
__device__ __forceinline__ f32x16_t tn_tile(const bf16_t* P, long ldp, int Mo, const bf16_t* Q, long ldq, int No, int T,
                                            int i0, int j0, int it0, int it1) {
    __shared__ __align__(16) unsigned char ring[TN_ST * TN_STAGE];
    const unsigned lds0 = (unsigned)(size_t)ring;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wi = wave >> 1, wj = wave & 1;
    const unsigned tr_at = tr_frag_at<64>(lane);
    // a wave brings rows 8 wave .. and 32 further of both tiles (fetches wave and wave + 4), each lane the chunk that belongs at its place;
    // a chunk behind the last column is that one again (its products are columns or rows that nobody stores), a row behind the last token
    // that one again, cleared below
    const int fr = 8 * wave + (lane >> 3), fc = (lane & 7) ^ tile_swz<64>(fr);
    const unsigned pc = (unsigned)min(i0 + fc * 8, Mo - 8) * 2, qc = (unsigned)min(j0 + fc * 8, No - 8) * 2;
    auto fetch = [&](int it) {
        const bf16_t *pb = P + (long)it * 64 * ldp, *qb = Q + (long)it * 64 * ldq;
        const unsigned st = lds0 + (unsigned)((it - it0) % TN_ST * TN_STAGE) + wave * 1024;
        const int last = T - 1 - it * 64;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const unsigned row = (unsigned)min(fr + 32 * h, last);
            bring_lds16<DIRECT>(row * (unsigned)(ldp * 2) + pc, pb, st + h * 4096, lane);
            bring_lds16<DIRECT>(row * (unsigned)(ldq * 2) + qc, qb, st + TN_TILE + h * 4096, lane);
        }
    };
    f32x16_t acc = zero16();
#pragma unroll
    for (int i = 0; i < TN_ST - 1; ++i)
        if (it0 + i < it1) fetch(it0 + i);
    for (int it = it0; it < it1; ++it) {
        if (it + TN_ST - 2 < it1) wait_vmcnt<4 * (TN_ST - 2)>();     // this tile has landed (the last ones: all have),
        else wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // the one before has been read
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (it + TN_ST - 1 < it1) fetch(it + TN_ST - 1);
        unsigned char* st = ring + (it - it0) % TN_ST * TN_STAGE;
        if (it * 64 + 64 > T) {                                      // a ragged last tile: rows behind the last token are zero
            for (int c = (T - it * 64) * 8 + (int)threadIdx.x; c < 64 * 8; c += 256) {
                *(uint4*)(st + c * 16) = make_uint4(0, 0, 0, 0);
                *(uint4*)(st + TN_TILE + c * 16) = make_uint4(0, 0, 0, 0);
            }
            __syncthreads();
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bf16x8_t a = read_tr_frag<64>(st + ks * 16 * 128, tr_at, wi);
            const bf16x8_t b = read_tr_frag<64>(st + TN_TILE + ks * 16 * 128, tr_at, wj);
            acc = mfma32(a, b, acc);
        }
    }
    return acc;
}

template <bool DIRECT>
__global__ __launch_bounds__(256) void gemm_tn_kernel(GemmTN p, int n_split) {
    // grid.y = Mo tiles x n_split: each split covers a contiguous token range; with n_split > 1 the splits are
    // stored as fp32 partials and added by tn_reduce_kernel.
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = wave >> 1, wj = wave & 1, l32 = lane & 31, g = lane >> 5;
    const int tiles_i = (p.Mo + 63) / 64;
    const int ti = blockIdx.y % tiles_i, split = blockIdx.y / tiles_i;
    const int i0 = ti * 64, j0 = blockIdx.x * 64, z = blockIdx.z;
    const int nt_all = (p.T + 63) / 64;
    const int it0 = (int)((long)nt_all * split / n_split), it1 = (int)((long)nt_all * (split + 1) / n_split);
    const f32x16_t acc = tn_tile<DIRECT>(p.P + (long)z * p.bP, p.ldp, p.Mo, p.Q + (long)z * p.bQ, p.ldq, p.No, p.T, i0, j0, it0, it1);
    const int col = j0 + wj * 32 + l32;
    if (n_split == 1) {
        if (col < p.No) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = i0 + wi * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                if (row < p.Mo) p.C[(long)z * p.bC + (long)row * p.ldc + col] = p.alpha * acc[v];
            }
        }
        return;
    }
    const long mn = (long)p.Mo * p.No;
    float* part = p.partial + ((long)z * n_split + split) * mn;
    if (col < p.No) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = i0 + wi * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
            if (row < p.Mo) part[(long)row * p.No + col] = acc[v];
        }
    }
}

// Several independent P^T Q products over the same T tokens in one launch: workgroup b takes output tile
// b - tile0 of the problem whose tile range holds b.  Every tile runs over all tokens, so nothing is split or reduced.
template <bool DIRECT>
__global__ __launch_bounds__(256) void gemm_tn_grouped_kernel(GemmTNGroup grp) {
    const int b = blockIdx.x;
    int k = 0;
    while (k + 1 < grp.n && b >= grp.p[k + 1].tile0) ++k;
    const TnProblem& q = grp.p[k];
    const int t = b - q.tile0, tiles_j = (q.No + 63) / 64;
    const int i0 = (t / tiles_j) * 64, j0 = (t % tiles_j) * 64;
    const f32x16_t acc = tn_tile<DIRECT>(q.P, q.ldp, q.Mo, q.Q, q.ldq, q.No, grp.T, i0, j0, 0, (grp.T + 63) / 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = wave >> 1, wj = wave & 1, l32 = lane & 31, g = lane >> 5;
    const int col = j0 + wj * 32 + l32;
    bool bad = false;
    if (col < q.No) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = i0 + wi * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
            if (row < q.Mo) {
                q.C[(long)row * q.ldc + col] = acc[v];
                bad |= !isfinite(acc[v]);
            }
        }
    }
    // a gradient that is not finite must not reach the optimizer: raise bit 1 of the update's flag (one vector atomic
    // per wave that saw one; never in a healthy update)
    if (grp.flag && __builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) atomicOr(grp.flag, 2);
}

// adds the token splits of gemm_tn_kernel in index order
__global__ __launch_bounds__(256) void tn_reduce_kernel(GemmTN p, int n_split) {
    const long mn = (long)p.Mo * p.No;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= mn * p.batch) return;
    const int z = (int)(idx / mn);
    const long r = idx % mn;
    float sum = 0.f;
    for (int sp = 0; sp < n_split; ++sp) sum += p.partial[((long)z * n_split + sp) * mn + r];
    p.C[(long)z * p.bC + (r / p.No) * p.ldc + (r % p.No)] = p.alpha * sum;
}

hipError_t launch_gemm_tn(const GemmTN& g, hipStream_t s) {
    if (g.Mo <= 0 || g.No <= 0 || g.batch <= 0) return hipSuccess;
    if ((g.ldp & 7) || (g.ldq & 7) || (g.Mo & 7) || (g.No & 7) || (g.bP & 7) || (g.bQ & 7)) return hipErrorInvalidValue;
    const long tiles = (long)cdiv(g.No, 64) * cdiv(g.Mo, 64) * g.batch;
    int split = 1;
    if (g.partial && tiles < 512) {
        split = (int)(768 / tiles);
        const int max_split = cdiv(g.T, 64) / 2;   // at least two token tiles per split
        if (split > max_split) split = max_split;
        if (split > 8) split = 8;
        if (split < 1) split = 1;
        while (split > 1 && (size_t)split * g.Mo * g.No * g.batch > g.partial_elems) --split;
    }
    dim3 grid(cdiv(g.No, 64), cdiv(g.Mo, 64) * split, g.batch);
    if (loads_to_lds(g.P) && loads_to_lds(g.Q)) gemm_tn_kernel<true><<<grid, 256, 0, s>>>(g, split);
    else gemm_tn_kernel<false><<<grid, 256, 0, s>>>(g, split);
    if (split > 1) {
        const long n = (long)g.Mo * g.No * g.batch;
        tn_reduce_kernel<<<cdiv(n, 256), 256, 0, s>>>(g, split);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_tn_grouped(GemmTNGroup& g, hipStream_t s) {
    if (g.n <= 0 || g.T <= 0) return hipSuccess;
    if (g.n > TN_GROUP_MAX) return hipErrorInvalidValue;
    int tiles = 0;
    bool direct = true;
    for (int k = 0; k < g.n; ++k) {
        TnProblem& q = g.p[k];
        direct &= loads_to_lds(q.P) && loads_to_lds(q.Q);
        if (q.Mo <= 0 || q.No <= 0 || (q.ldp & 7) || (q.ldq & 7) || (q.Mo & 7) || (q.No & 7)) return hipErrorInvalidValue;
        q.tile0 = tiles;
        tiles += cdiv(q.Mo, 64) * cdiv(q.No, 64);
    }
    if (direct) gemm_tn_grouped_kernel<true><<<tiles, 256, 0, s>>>(g);
    else gemm_tn_grouped_kernel<false><<<tiles, 256, 0, s>>>(g);
    return hipGetLastError();
}
