// Causal self-attention within one chunk, forward and backward, on bf16 MFMA (gfx950).
//
// Forward and backward work on the TRANSPOSED score tile where that keeps the softmax row in one lane:
//   forward / dQ :  S^T[u][t] = K[u] . Q[t]   -> a lane owns one query t (and its partner lane t too),
//                   so the running max, the row sum, lse[t] and delta[t] are per-lane scalars;
//                   O^T[d][t] += V^T[d][u] P^T[u][t]   and   dQ^T[d][t] += K^T[d][u] dS^T[u][t]
//                   reuse the score fragment directly as the B operand (see tiles.h); their A operands V^T, K^T (and
//                   dO^T, Q^T below) are never built: the tiles stay as they lie in memory and are read through the
//                   LDS transpose read of gfx950 (read_tr_frag), without transposing stores.
//   dK / dV      :  S[t][u] = Q[t] . K[u]     -> a lane owns one key u;
//                   dV^T[d][u] += dO^T[d][t] P[t][u],  dK^T[d][u] += Q^T[d][t] dS[t][u].
// P is never stored: the backward pass rebuilds it from the saved log-sum-exp.
// No access of the loops over tiles has a bank conflict.  What SQ_LDS_BANK_CONFLICT counts grows with the blocks, not with their tiles: it is the slabs that
// results leave through, 384 cycles a workgroup at d_head 128 (192 at 64) forward, 768 (192) for a dK/dV and a dQ part together
// backward: 15, 9 and 5 % of the LDS cycles at 1024, 2048 and 4096 tokens forward, 13, 8 and 5 % backward.
// The two parts of the backward launch (dK and dV; dQ) write disjoint outputs, so no atomics are needed and results
// are bit-reproducible.
#include <type_traits>
#include <utility>

#include "kernels.h"
#include "tiles.h"

#define NEG_BIG (-1.0e30f)

template <int DH>
struct AttnCfg {
    static constexpr int NKS = DH / 16; // MFMA steps over d
    static constexpr int ND = DH / 32;  // 32-wide d tiles
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// write a D fragment set holding X^T[d][row] (lane = row) as bf16 rows of X
template <int DH>
__device__ __forceinline__ void write_rows_from_dT(bf16_t* __restrict__ dst, const f32x16_t* acc, float mul, int g) {
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            uint2 w;
            w.x = pack_bf16x2(acc[dt][4 * vq] * mul, acc[dt][4 * vq + 1] * mul);
            w.y = pack_bf16x2(acc[dt][4 * vq + 2] * mul, acc[dt][4 * vq + 3] * mul);
            *(uint2*)(dst + dt * 32 + 8 * vq + 4 * g) = w;
        }
}

// ======================================================================== forward
// Two key groups of four waves each; a wave owns 32 queries, and the key tiles (64 keys) of the causal range are dealt
// out to the key groups in turn (group kg takes tiles kg, kg + 2, ..).  Every group keeps its own running max, row
// sum and output accumulator over its tiles and the groups are merged once at the end through LDS (the usual
// two-state softmax merge).  With KG = 2 a SIMD runs two waves, so one wave's softmax arithmetic overlaps the other's
// MFMAs; at T = 1024 with 32 heads there are otherwise only as many 32-query waves as the chip has SIMDs.  Four waves a group
// beat two there (a K/V tile is shared by more queries; the extra workgroups of two do not overlap enough).
// K and V tiles come by direct-to-LDS loads, one tile ahead in the group's other buffer, with one barrier a tile; Q and O pass through LDS
// too (straight from and to memory every instruction touches 32 rows).  us with tiles staged through registers (two barriers a tile, Q and
// O by rows) and with this, heads of 128 / 64: 1024 tokens, 32 heads 28.8 and 25.4 / 16 heads 17.3 and 15.3; 2048 tokens 54.8 and 47.5 /
// 30.8 and 28.9; 5120 tokens, 32 heads of 128 277 and 246 (870 TFLOP/s; the rest is the softmax between the two products of a tile, and at
// 1024 tokens the heaviest block: 8 passes of two tiles where the mean is 4.5).  The order of every sum is the same in both.
// DIRECT: q, k and v start at multiples of 4 bytes (else their tiles come through registers)
constexpr int ATTN_NW = 4, ATTN_KG = 2;      // waves a group, groups
template <int DH, bool DIRECT>
__global__ __launch_bounds__(ATTN_KG * ATTN_NW * 64, 2) void attn_fwd_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                                const bf16_t* __restrict__ v, long ldq, int T,
                                                                bf16_t* __restrict__ o, long ldo, float* __restrict__ lse,
                                                                float scale_log2e) {
    using C = AttnCfg<DH>;
    constexpr int NW = ATTN_NW, KG = ATTN_KG, NT = NW * 64, QB = NW * 32;
    constexpr int RB = DH * 2, TB = 64 * RB, NI = TB / 4096;      // bytes of a row, of a tile; fetches per wave and tile
    static_assert(NW == 4 && KG == 2, "four waves fetch a tile; the block's queries fit one buffer");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int kg = __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
    const int tid = threadIdx.x % NT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, g = lane >> 5;
    const unsigned lds0 = (unsigned)(size_t)smem_raw;
    const unsigned group_at = kg * 4 * TB;                        // two buffers of a K and a V tile each
    const unsigned row_at = row_frag_at<DH>(lane), tr_at = tr_frag_at<DH>(lane);
    const TileFetch<DH, DIRECT> fetch_rows(lane);
    // Heaviest (latest) query blocks first, every head's before any head's second heaviest (longest job first).  The blocks of a head are
    // gridDim.y workgroups apart in dispatch order (x fastest), so with a multiple of eight heads they lie on one XCD, whose L2 fetches the
    // head's keys and values once; with a head's blocks side by side all eight XCDs fetch them (1024 tokens, 32 heads of 128:
    // 25 MB fetched and 22.8 us, 84 MB and 25.4).
    const int idx = blockIdx.y * gridDim.x + blockIdx.x;
    const int qb = (int)gridDim.x - 1 - idx / (int)gridDim.y, head = idx % (int)gridDim.y;
    const int q0 = qb * QB, tq0 = q0 + 32 * wave, t_abs = tq0 + l32;
    const bf16_t* qh = q + (long)head * DH;
    const bf16_t* kh = k + (long)head * DH;
    const bf16_t* vh = v + (long)head * DH;

    f32x16_t oacc[C::ND];
#pragma unroll
    for (int dt = 0; dt < C::ND; ++dt) oacc[dt] = zero16();
    float m = NEG_BIG, lpart = 0.f;

    const int kend = min(q0 + QB, T);
    const int n_tiles = (kend + 63) / 64;
    const int n_iter = (n_tiles + KG - 1) / KG;   // a group's surplus tile lies wholly in the future and is skipped
    auto fetch = [&](int it) {
        const int u0 = min((it * KG + kg) * 64, (T - 1) & ~63);   // (a surplus tile may begin behind the last key: any other instead)
        const unsigned at = lds0 + group_at + (it & 1) * 2 * TB;
#pragma unroll
        for (int j = 0; j < NI; ++j) fetch_rows(kh + (long)u0 * ldq, (unsigned)ldq * 2, wave * NI + j, T - 1 - u0, at);
#pragma unroll
        for (int j = 0; j < NI; ++j) fetch_rows(vh + (long)u0 * ldq, (unsigned)ldq * 2, wave * NI + j, T - 1 - u0, at + TB);
    };
    // the block's queries (128 rows, 16 a wave) through the first group's second buffer
    const int w0 = 16 * (kg * NW + wave), qr = min(q0 + w0, T - 1);
#pragma unroll
    for (int j = 0; j < NI; ++j) fetch_rows(qh + (long)qr * ldq, (unsigned)ldq * 2, j, T - 1 - qr, lds0 + 2 * TB + w0 * RB);
    fetch(0);
    wait_vmcnt<DIRECT ? 2 * NI : 0>();
    if constexpr (!DIRECT) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bf16x8_t qf[C::NKS];
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) qf[ks] = *(const bf16x8_t*)(smem_raw + 2 * TB + wave * 32 * RB + (row_at ^ (unsigned)(ks << 5)));
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) asm volatile("" : "+v"(qf[ks]));
    for (int it = 0; it < n_iter; ++it) {
        const int u0 = (it * KG + kg) * 64;
        wait_vmcnt<0>();                                          // the tile has landed,
        if (u0 + 64 > T) clear_rows<DH>(smem_raw + group_at + (it & 1) * 2 * TB + TB, max(16 * wave, T - u0), 16 * wave + 16, lane);     // (V: P is 0 there)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // the one before (and Q) has been read
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (it + 1 < n_iter) fetch(it + 1);
        const unsigned char* sK = smem_raw + group_at + (it & 1) * 2 * TB;
        const unsigned char* sV = sK + TB;
        if (u0 > tq0 + 31) continue;  // wave-uniform: every key of this tile is in the future
        // both 32-key halves of the tile at once: two independent MFMA chains, one softmax update
        f32x16_t s0 = zero16(), s1 = zero16();
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            const bf16x8_t a0 = *(const bf16x8_t*)(sK + (row_at ^ (unsigned)(ks << 5)));
            const bf16x8_t a1 = *(const bf16x8_t*)(sK + 32 * RB + (row_at ^ (unsigned)(ks << 5)));
            s0 = mfma32(a0, qf[ks], s0);
            s1 = mfma32(a1, qf[ks], s1);
        }
        // the running max m is kept in units of the raw scores (the scale is positive, so it commutes with max) and
        // the scale is folded into the exponent's multiply-add: one instruction per score less
        float x[32];
        float mloc = NEG_BIG;
        if (u0 + 63 > tq0) {  // the tile touches the diagonal: causal mask
#pragma unroll
            for (int vv = 0; vv < 16; ++vv) {
                const int u = u0 + 8 * (vv >> 2) + 4 * g + (vv & 3);
                x[vv] = (u > t_abs) ? NEG_BIG : s0[vv];
                x[16 + vv] = (u + 32 > t_abs) ? NEG_BIG : s1[vv];
            }
        } else {
#pragma unroll
            for (int vv = 0; vv < 16; ++vv) {
                x[vv] = s0[vv];
                x[16 + vv] = s1[vv];
            }
        }
#pragma unroll
        for (int vv = 0; vv < 32; ++vv) mloc = fmaxf(mloc, x[vv]);
        mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
        const float m_new = fmaxf(m, mloc);
        const float alpha = fast_exp2((m - m_new) * scale_log2e);
        const float mb = m_new * scale_log2e;
        float psum = 0.f;
#pragma unroll
        for (int vv = 0; vv < 32; ++vv) {
            x[vv] = fast_exp2(fmaf(x[vv], scale_log2e, -mb));
            psum += x[vv];
        }
        lpart = lpart * alpha + psum;
        m = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {  // skip the rescale once the running max has settled
#pragma unroll
            for (int dt = 0; dt < C::ND; ++dt)
#pragma unroll
                for (int vv = 0; vv < 16; ++vv) oacc[dt][vv] *= alpha;
        }
#pragma unroll
        for (int us = 0; us < 2; ++us)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bf16x8_t b = pack_b_from_d(x + 16 * us, h);
#pragma unroll
                for (int dt = 0; dt < C::ND; ++dt) {
                    const bf16x8_t a = read_tr_frag<DH>(sV + (us * 32 + 16 * h) * RB, tr_at, dt);
                    oacc[dt] = mfma32(a, b, oacc[dt]);
                }
            }
    }
    // merge the key groups into group 0: values of thread `tid` are kept NT apart (no bank conflicts)
    float* mg = (float*)smem_raw;
    __syncthreads();                            // every group is done with its K / V tiles
    if (kg == 1) {
#pragma unroll
        for (int dt = 0; dt < C::ND; ++dt)
#pragma unroll
            for (int vv = 0; vv < 16; ++vv) mg[(dt * 16 + vv) * NT + tid] = oacc[dt][vv];
        mg[(C::ND * 16) * NT + tid] = m;
        mg[(C::ND * 16 + 1) * NT + tid] = lpart;
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = mg[(C::ND * 16) * NT + tid], l1 = mg[(C::ND * 16 + 1) * NT + tid];
    const float mt = fmaxf(m, m1);
    const float a0 = fast_exp2((m - mt) * scale_log2e), a1 = fast_exp2((m1 - mt) * scale_log2e);
#pragma unroll
    for (int dt = 0; dt < C::ND; ++dt)
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) oacc[dt][vv] = oacc[dt][vv] * a0 + mg[(dt * 16 + vv) * NT + tid] * a1;
    lpart = lpart * a0 + l1 * a1;
    m = mt;
    const float ltot = lpart + __shfl_xor(lpart, 32, 64), inv = 1.f / ltot;
    if (t_abs < T && g == 0) lse[(long)head * T + t_abs] = (m * scale_log2e + log2f(ltot)) * 0.6931471805599453f;
    // the wave's 32 rows leave through LDS (behind what the merge reads), so that a row is written in 16-byte pieces.  (Bank
    // conflicts: 96 cycles a wave.)
    constexpr int LD = DH + 8;
    bf16_t* slab = (bf16_t*)(smem_raw + NT * (C::ND * 16 + 2) * sizeof(float)) + wave * 32 * LD;
    static_assert(NT * (C::ND * 16 + 2) * 4 + NT / 2 * LD * 2 <= 8 * TB, "the output slab fits");
    write_rows_from_dT<DH>(slab + l32 * LD, oacc, inv, g);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = lane; i < 32 * DH / 8; i += 64) {
        const int row = i / (DH / 8), c = i % (DH / 8) * 8;
        if (tq0 + row < T) *(uint4*)(o + (long)(tq0 + row) * ldo + (long)head * DH + c) = *(const uint4*)(slab + row * LD + c);
    }
}

// ======================================================================== backward
// One part of the backward pass: either dK and dV of a block of keys (the streamed rows are the queries from it on) or dQ of a block
// of queries (DQ; the streamed rows are the keys up to it).  A wave keeps NG groups of 32 rows of its block, their first operand
// P1 (K; Q) in registers, and takes every second 32-row piece of the streamed matrices X1 (Q; K) and X2 (dO; V):
//   S[x][p] = X1[x] . P1[p],  dP[x][p] = X2[x] . P2[p]       a lane owns row p of the block, registers run over x
//   acc1^T[d][p] += X1^T[d][x] dS[x][p]  (dK; dQ),           acc2^T[d][p] += X2^T[d][x] P[x][p]  (dV)
// with the score fragments reused as B operands (see tiles.h).  Four waves: two row groups of the block, two halves of a 64-row
// streamed tile; what the two halves gathered is added at the end through LDS.
//
// What bounds it: at d_head 128 and long samples the energy of the matrix instructions (a loop of nothing else on random operands runs
// at 1.6 to 1.85 of 2.4 GHz here, 18 to 20 ns an MFMA; a 64-row tile takes 64 of them a wave for dK and dV, 1.2 us, and 1.7 in all), at
// 1024 tokens also the two ends of a part (3 us of loads, 1.5 us of exchange and stores).  d_head 128 has one wave per SIMD (256
// accumulators, 64 registers of K, 64 of S and dP, 32 of P and dS), so nothing but the order of its instructions keeps the matrix unit
// busy: a wave has 64 rows, so that a fragment of X feeds two MFMAs, and the probabilities are formed between the MFMAs of dP, dS
// between those of dV.  V of a key block stays in LDS for want of registers.  d_head 64 has two waves of 32 rows per SIMD.  Tiles come by
// direct-to-LDS loads two tiles ahead, one copy of each: 16-byte chunk c of row x lies at position c ^ swz(x), so that both the reads of
// 16 rows at one chunk and the transposing reads of four rows x 64 bytes fall into distinct banks.
// us without and with this (before: waves of 32 rows, two copies of each tile, loads and stores of 32 rows at a time), heads of 128 / 64:
// 1024 tokens, 32 heads 62 and 46 / 16 heads 39 and 18; 2048 tokens 189 and 138 / 78 and 47; 5120 tokens, 32 heads of 128 1000 and 745.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

__device__ const float kBeyond[2] = {1.0e30f, 0.f};       // log-sum-exp and delta of a query that does not exist: every probability is 0

template <int DH> struct BwdCfg {
    static constexpr int NG = DH / 64;                     // 32-row groups per wave
    static constexpr int PB = 64 * NG;                     // rows of a block
    static constexpr int RB = DH * 2, TB = 64 * RB;        // bytes of a row, of a tile
    static constexpr int STAGE = 2 * TB + 512, NST = 3;    // X1, X2, lse and delta of the 64 rows
    static constexpr int V0 = DH == 128 ? PB * RB : 0;     // V of the block, in front of them
    static constexpr int LDS = V0 + NST * STAGE;
    static_assert(LDS <= 160 * 1024 && LDS >= 4 * NG * (DH / 32) * 16 * 256, "the exchange of the accumulators fits");
};
__device__ __forceinline__ void mfma32_acc(f32x16_t& c, bf16x8_t a, bf16x8_t b) {
    // in place, in accumulation registers; two wait states have to pass between a vector instruction that writes an operand and this
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// the same in vector registers, for scores: FIRST starts from zero.  Their last results may be read once two more MFMAs have been
// issued, or behind score_ready.
template <bool FIRST>
__device__ __forceinline__ void mfma32_score(f32x16_t& c, bf16x8_t a, bf16x8_t b) {
    if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// DIRECT: q, k, v and dO start at multiples of 4 bytes (else their tiles come through registers, ahead of the products instead of between them)
template <int DH, bool DQ, bool DIRECT>
__device__ __forceinline__ void attn_bwd_part(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, const bf16_t* __restrict__ d_o,
    const float* __restrict__ lse, const float* __restrict__ delta, long ldq, long ldo, int T, bf16_t* __restrict__ dq,
    bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, float scale, const float2* __restrict__ rope, int block, int head,
    unsigned char* smem) {
    using C = BwdCfg<DH>;
    constexpr int NG = C::NG, KS = DH / 16, ND = DH / 32, RB = C::RB, TB = C::TB, STAGE = C::STAGE, NST = C::NST;
    constexpr int NI = TB / 4096;                                      // fetches per wave and tile
    constexpr int NF = 2 * NI + (DQ ? 0 : 1);                          // fetches per wave and stage
    constexpr bool V_LDS = !DQ && NG == 2;
    static_assert(KS == 2 * ND, "as many MFMAs for each product");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5, pg = wave >> 1, sg = wave & 1;
    const unsigned lds0 = (unsigned)(size_t)smem;
    const int p0 = block * C::PB, pw0 = p0 + 32 * NG * pg;             // first row of the block, of this wave's share
    // first row of group j of this wave: the waves of the two halves count their groups in opposite order, so that each hands its last
    // one to the other in the end
    auto group_row = [&](int j) { return pw0 + 32 * (NG == 2 ? j ^ sg : 0); };
    const float scale_log2e = scale * 1.4426950408889634f;
    const long hd = (long)head * DH;
    const bf16_t* x1 = (DQ ? k : q) + hd;
    const bf16_t* x2 = (DQ ? v : d_o) + hd;
    const bf16_t* p1 = (DQ ? q : k) + hd;
    const bf16_t* p2 = (DQ ? d_o : v) + hd;
    const long ldx2 = DQ ? ldq : ldo, ldp2 = DQ ? ldo : ldq;
    const float* lse_h = lse + (long)head * T;
    const float* delta_h = delta + (long)head * T;

    float dlt[NG], lse2[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
        const int p = min(group_row(j) + l32, T - 1);      // rows beyond the last are never stored, and each has a lane of its own
        dlt[j] = DQ ? delta_h[p] : 0.f;
        lse2[j] = DQ ? lse_h[p] * 1.4426950408889634f : 0.f;
    }

    const TileFetch<DH, DIRECT> fetch_rows(lane);
    const unsigned ld1b = (unsigned)ldq * 2, ldx2b = (unsigned)ldx2 * 2;
    struct Fetch { const bf16_t *a, *b; const float* stats; int last; unsigned st; };
    auto fetch_of = [&](int tile, unsigned st) {
        const long r0 = (long)tile * 64;
        return Fetch{x1 + r0 * ldq, x2 + r0 * ldx2, (sg ? delta_h : lse_h) + r0, T - 1 - tile * 64, st};
    };
    // piece n of the NF a wave issues per tile (two waves each bring lse and delta, so that every wave has as many in flight)
    auto fetch_piece = [&](const Fetch& f, int n) {
        if (n < NI) fetch_rows(f.a, ld1b, wave * NI + n, f.last, lds0 + f.st);
        else if (n < 2 * NI) fetch_rows(f.b, ldx2b, wave * NI + n - NI, f.last, lds0 + f.st + TB);
        else load_lds4(lane <= f.last ? f.stats + lane : kBeyond + sg, __builtin_amdgcn_readfirstlane(lds0 + f.st + 2 * TB + sg * 256));
    };
    auto fetch = [&](const Fetch& f) {
#pragma unroll
        for (int n = 0; n < NF; ++n) fetch_piece(f, n);
    };

    const int n_tiles = (T + 63) / 64;
    const int tile0 = DQ ? 0 : p0 / 64, tile1 = DQ ? min((p0 + C::PB + 63) / 64, n_tiles) : n_tiles;
    // The operands of the block come through LDS too, and the results leave through it: 16 bytes a lane straight from and to memory touch
    // 32 rows with every instruction (loads and stores of one part 8.5 us; 4.5 like this).  P1 takes the place of the third tile.
    constexpr unsigned P1_AT = C::V0 + 2 * STAGE, P2_AT = DH == 128 ? 0 : P1_AT + TB;
    auto fetch_block = [&](const bf16_t* x, long ld, unsigned at) {    // a quarter each, from its own first row: offsets between rows are 32-bit
        const int w0 = wave * (C::PB / 4), r0 = min(p0 + w0, T - 1);
#pragma unroll
        for (int j = 0; j < C::PB * RB / 4096; ++j)
            fetch_rows(x + (long)r0 * ld, (unsigned)ld * 2, j, T - 1 - r0, lds0 + at + w0 * RB);
    };
    fetch_block(p1, ldq, P1_AT);
    fetch_block(p2, ldp2, P2_AT);
    // dK and dV take the tiles from the last one down, dQ from the first one up: the blocks of a head that start together then read the
    // same ones (5120 tokens: 764 us with both upwards, 755 with both downwards, 745 like this)
    const int n_steps = tile1 - tile0;
    auto tile_of = [&](int i) { return DQ ? min(i, n_steps - 1) : tile1 - 1 - min(i, n_steps - 1); };
    fetch(fetch_of(tile_of(0), C::V0));
    fetch(fetch_of(tile_of(1), C::V0 + STAGE));
    // this lane's place in the fragments of block rows (chunk 2 ks + g of row l32 of a group)
    const unsigned p_at = (unsigned)((pg * 32 * NG + (NG == 2 ? 32 * sg : 0)) * RB) + row_frag_at<DH>(lane);
    auto p_frag = [&](unsigned at, int j, int ks) { return *(const bf16x8_t*)(smem + at + (p_at ^ (unsigned)(ks << 5 | j * 32 * RB))); };
    wait_vmcnt<DIRECT ? 2 * NF : 0>();
    if constexpr (!DIRECT) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bf16x8_t p1f[NG][KS], p2f[V_LDS ? 1 : NG][V_LDS ? 1 : KS];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            p1f[j][ks] = p_frag(P1_AT, j, ks);
            if constexpr (!V_LDS) p2f[j][ks] = p_frag(P2_AT, j, ks);
        }
    }
    // the compiler's own loads are waited for here and not in the loop
#pragma unroll
    for (int j = 0; j < NG; ++j) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            asm volatile("" : "+v"(p1f[j][ks]));
            if constexpr (!V_LDS) asm volatile("" : "+v"(p2f[j][ks]));
        }
        asm volatile("" : "+v"(dlt[j]), "+v"(lse2[j]));
    }

    // zeros by MFMAs with nothing in them: sixteen instructions instead of 256 (code that runs once is paid for in instruction cache misses)
    f32x16_t acc1[NG][ND], acc2[DQ ? 1 : NG][DQ ? 1 : ND];
    bf16x8_t nothing = __builtin_bit_cast(bf16x8_t, make_uint4(0, 0, 0, 0));
    asm volatile("s_nop 1" : "+v"(nothing));
#pragma unroll
    for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %1, 0" : "=a"(acc1[j][dt]) : "v"(nothing));
            if constexpr (!DQ) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %1, 0" : "=a"(acc2[j][dt]) : "v"(nothing));
        }

    // this lane's place in a fragment read of rows (chunk 2 ks + g) and in a transposing read (read_tr_frag)
    const unsigned row_at = (unsigned)(sg * 32 * RB) + row_frag_at<DH>(lane), tr_at = (unsigned)(sg * 32 * RB) + tr_frag_at<DH>(lane);
    auto row_frag = [&](unsigned tile, int ks) { return *(const bf16x8_t*)(smem + tile + (row_at ^ (unsigned)(ks << 5))); };
    auto tr_frag = [&](unsigned tile, int i) {       // i = h ND + dt: contraction rows 16 h .., columns 32 dt ..
        return read_tr_frag<DH>(smem + tile + (i / ND) * 16 * RB, tr_at, i % ND);
    };

    // J: groups of rows that take part (the others keep what they have: not even a weight of 0 meets a row that does not belong to them)
    auto compute = [&](auto masked, auto groups, unsigned st, int xs0, const Fetch& next) {
        constexpr bool MASK = decltype(masked)::value;
        constexpr int J = decltype(groups)::value;
        // One fragment of X and NG MFMAs a slot, KS slots each of S, dP, dV and dK (of S, dP and dQ).  Fragments are asked for AHEAD slots
        // before they are used, and the vector work on the scores, in items of four values a lane, goes between the MFMAs behind them.
        constexpr int B0 = KS, C0 = 2 * KS, NS = (DQ ? 3 : 4) * KS, D0 = NS - KS;
        constexpr int AHEAD = 4, AHEAD_V = 3;
        static_assert(J == NG || !DQ, "only key blocks leave a group out");
        f32x16_t s[NG], dp[NG];
        bf16x8_t pb[NG][2], dsb[NG][2], fx[NS], fv[NG][KS];
        float4 l4[4], d4[4];
        const unsigned t1 = st, t2 = st + TB;
        auto read = [&](auto slot) {
            constexpr int i = decltype(slot)::value, n = i % KS;
            if constexpr (i < B0) fx[i] = row_frag(t1, n);
            else if constexpr (i < C0) {
                fx[i] = row_frag(t2, n);
                if constexpr (V_LDS) {
#pragma unroll
                    for (int j = 0; j < J; ++j) fv[j][n] = p_frag(P2_AT, j, n);
                }
            } else fx[i] = tr_frag(i >= D0 ? t1 : t2, n);
        };
        auto mfma = [&](auto slot) {
            constexpr int i = decltype(slot)::value, n = i % KS;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                if constexpr (i < B0) mfma32_score<n == 0>(s[j], fx[i], p1f[j][n]);
                else if constexpr (i < C0) mfma32_score<n == 0>(dp[j], fx[i], V_LDS ? fv[j][n] : p2f[V_LDS ? 0 : j][V_LDS ? 0 : n]);
                else if constexpr (i >= D0) mfma32_acc(acc1[j][n % ND], fx[i], dsb[j][n / ND]);
                else mfma32_acc(acc2[DQ ? 0 : j][DQ ? 0 : n % ND], fx[i], pb[j][n / ND]);
            }
        };
        auto read_stats = [&](int which, int vq) {       // lse (0) or delta (1) of the rows of item vq
            if constexpr (!DQ) (which ? d4 : l4)[vq] = *(const float4*)((const float*)(smem + st + 2 * TB) + which * 64 + sg * 32 + 8 * vq + 4 * g);
        };
        auto probs = [&](int j, int vq) {          // four probabilities, in place of their scores
            const float ll[4] = {l4[vq].x, l4[vq].y, l4[vq].z, l4[vq].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float sub = DQ ? lse2[j] : ll[e] * 1.4426950408889634f;
                float pe = fast_exp2(s[j][4 * vq + e] * scale_log2e - sub);
                if (MASK) {
                    const int x_p = xs0 + 8 * vq + 4 * g + e - group_row(j) - l32;          // a key must not follow its query
                    pe = (DQ ? x_p > 0 : x_p < 0) ? 0.f : pe;
                }
                s[j][4 * vq + e] = pe;
                if constexpr (!DQ) pb[j][vq >> 1][4 * (vq & 1) + e] = (__bf16)pe;
            }
        };
        auto dscores = [&](int j, int vq) {
            const float dd[4] = {d4[vq].x, d4[vq].y, d4[vq].z, d4[vq].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                dsb[j][vq >> 1][4 * (vq & 1) + e] = (__bf16)(s[j][4 * vq + e] * (dp[j][4 * vq + e] - (DQ ? dlt[j] : dd[e])));
        };
        // The compiler does not see the matrix instructions inside the asm statements: what reads their results comes behind a statement
        // that passes them through, two MFMAs or enough wait states later.
        auto ready = [&](f32x16_t* x, auto wait) {
            if constexpr (decltype(wait)::value) asm volatile("s_nop 15\n\ts_nop 3");
#pragma unroll
            for (int j = 0; j < J; ++j) asm volatile("" : "+v"(x[j]));
        };
        using Wait = std::true_type; using SlotWait = std::bool_constant<J == 1>;
        // item n: group n % NG, rows 8 (n / NG) ..; dV needs the first half of the probabilities KS / 2 slots before the second
        constexpr int NI_P = 4 * NG;
        auto p_item = [](int i) -> int {           // the item of probabilities behind the MFMAs of slot i
            if (NG == 1) return i >= B0 && i < B0 + 4 ? i - B0 : -1;
            if (DQ) return i >= B0 + 1 && i < B0 + 8 ? i - B0 - 1 : -1;
            return i >= B0 + 1 && i <= B0 + 3 ? i - B0 - 1 : i >= B0 + 5 && i <= B0 + 6 ? i - B0 - 2 : i >= C0 && i <= C0 + 2 ? i - C0 + 5 : -1;
        };
        auto d_item = [](int i) -> int {           // of dS
            if (DQ) return -1;
            if (NG == 1) return i >= C0 && i < C0 + 4 ? i - C0 : -1;
            return i >= C0 + 3 && i < C0 + 7 ? i - C0 - 3 : i >= D0 && i < D0 + 4 ? i - D0 + 4 : -1;
        };
        static_for<AHEAD>([&](auto slot) { read(slot); });
        static_for<NS>([&](auto slot) {
            constexpr int i = decltype(slot)::value;
            static_for<AHEAD>([&](auto more) {
                constexpr int r = i + 1 + decltype(more)::value;
                if constexpr (r < NS && r - (V_LDS && r >= B0 && r < C0 ? AHEAD_V : AHEAD) == i) read(std::integral_constant<int, r>{});
            });
            if (DIRECT && i < NF - NI) fetch_piece(next, NI + i);
            if (DIRECT && i >= NS - NI) fetch_piece(next, i - (NS - NI));
#pragma unroll
            for (int x = 0; x < NI_P; ++x) {
                if (p_item(i + 2) == x && x % NG == 0) read_stats(0, x / NG);
                if (d_item(i + 2) == x && x % NG == 0) read_stats(1, x / NG);
            }
            mfma(slot);
            if constexpr (i == B0) ready(s, SlotWait{});
            if constexpr (i == C0 && !DQ) ready(dp, SlotWait{});
            if (p_item(i) >= 0 && p_item(i) % NG < J) probs(p_item(i) % NG, p_item(i) / NG);
            if (d_item(i) >= 0 && d_item(i) % NG < J) dscores(d_item(i) % NG, d_item(i) / NG);
            if constexpr (DQ) {
                if (i == D0 - 1) {
                    if (NG == 2) probs(1, 3);
                    ready(dp, Wait{});
#pragma unroll
                    for (int x = 0; x < 2 * NG; ++x) dscores(x % NG, x / NG);
                }
                if (i >= D0 && i < D0 + ND) {
#pragma unroll
                    for (int x = 0; x < 2 * NG / ND; ++x) dscores((2 * NG + (i - D0) * (2 * NG / ND) + x) % NG, (2 * NG + (i - D0) * (2 * NG / ND) + x) / NG);
                }
            }
            // two wait states between a vector instruction and the MFMA that takes its result
            if constexpr (i == C0 - 1 || i == D0 - 1 || i == D0 + ND - 1 || (!DQ && i == C0 + ND - 1)) asm volatile("s_nop 1");
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    unsigned st = C::V0, st_next = C::V0 + 2 * STAGE;
    int i_step = 0;
    auto step = [&](auto what) {           // 0: nothing to do for this wave, 1: every score counts, 2: with the causal mask, 3: the first group only
        constexpr int WHAT = decltype(what)::value;
        wait_vmcnt<DIRECT ? NF : 0>();                                     // this tile has landed (the next may be in flight)
        if constexpr (!DQ) {                                               // (the last tile is the first; dO: P is 0 there)
            if (i_step == 0 && tile1 * 64 > T) clear_rows<DH>(smem + st + TB, max(16 * wave, T - (tile1 - 1) * 64), 16 * wave + 16, lane);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                 // and every read of the one before is done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const Fetch next = fetch_of(tile_of(i_step + 2), st_next);         // (behind the last tile: that one again, unused)
        if constexpr (WHAT && !DIRECT) fetch(next);
        if constexpr (WHAT) compute(std::bool_constant<(WHAT >= 2)>{}, std::integral_constant<int, WHAT == 3 ? 1 : NG>{}, st, tile_of(i_step) * 64 + 32 * sg, next);
        else fetch(next);
        st = st == C::V0 + (NST - 1) * STAGE ? C::V0 : st + STAGE;
        st_next = st_next == C::V0 + (NST - 1) * STAGE ? C::V0 : st_next + STAGE;
        ++i_step;
    };
    using Skip = std::integral_constant<int, 0>; using Plain = std::integral_constant<int, 1>; using Masked = std::integral_constant<int, 2>;
    using First = std::integral_constant<int, 3>;
    // Wave-uniform ranges of tiles: those in which every query precedes every key of this wave are left out, those on the diagonal need
    // the mask.  (Rows beyond T need none: as queries their log-sum-exp is beyond any score, as keys they follow every query.)
    const int w = pw0 - 32 * sg;
    if constexpr (DQ) {
        const int plain_end = min(tile1, (w + 33) >> 6), mask_end = min(tile1, (w + 32 * NG + 63) >> 6);
        while (i_step < plain_end) step(Plain{});
        while (i_step < mask_end) step(Masked{});
        while (i_step < n_steps) step(Skip{});
    } else {
        const int plain_end = tile1 - min(tile1, (w + 32 * NG + 62) >> 6), mask_end = tile1 - min(tile1, (w + 32) >> 6);
        while (i_step < plain_end) step(Plain{});
        // (the piece of queries at the keys of the first of two groups precedes every key of the second)
        if constexpr (NG == 2) { if (sg == 0 && i_step < mask_end) step(First{}); }
        while (i_step < mask_end) step(Masked{});
        while (i_step < n_steps) step(Skip{});
    }
    wait_vmcnt<0>();
    // Ordinary instructions read the accumulators from here on (see gemm_nt_dl_kernel)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
            asm volatile("" : "+a"(acc1[j][dt]));
            if constexpr (!DQ) asm volatile("" : "+a"(acc2[j][dt]));
        }
    // add the two halves: each wave hands over one half of what it holds (NG 2: the other's group of rows; else dK or dV, or all of dQ)
    // and finishes the other; values of one thread are kept 64 apart
    // (lane numbers formed anew: kept across the loop they cost a spill)
    const int elane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), el32 = elane & 31, eg = elane >> 5;
    __syncthreads();
    constexpr int HALF = C::LDS / (1024 * 4) * 1024;       // bytes of LDS per wave
    float4* mine = (float4*)(smem + wave * HALF) + elane;
    const float4* other = (const float4*)(smem + (wave ^ 1) * HALF) + elane;
    auto put = [&](const f32x16_t* a, int n0) {
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                mine[(n0 + dt * 4 + vq) * 64] = make_float4(a[dt][4 * vq], a[dt][4 * vq + 1], a[dt][4 * vq + 2], a[dt][4 * vq + 3]);
    };
    auto add = [&](f32x16_t* a, int n0) {
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const float4 o = other[(n0 + dt * 4 + vq) * 64];
                a[dt][4 * vq] += o.x; a[dt][4 * vq + 1] += o.y; a[dt][4 * vq + 2] += o.z; a[dt][4 * vq + 3] += o.w;
            }
    };
    // one group of rows leaves through LDS, so that a row is written in 16-byte pieces (and its RoPE angles read so).  (Bank conflicts:
    // 64 cycles a group of rows.)
    auto out = [&](const f32x16_t* a, bf16_t* dst, float mul, const float2* table) {
        constexpr int LD = DH + 4, HALF_D = DH / 2, CPH = HALF_D / 8;       // floats per row, 8-column chunks per half
        float* slab = (float*)(smem + wave * HALF);
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                *(float4*)(slab + el32 * LD + dt * 32 + 8 * vq + 4 * eg) = make_float4(a[dt][4 * vq], a[dt][4 * vq + 1], a[dt][4 * vq + 2], a[dt][4 * vq + 3]);
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int i = elane; i < 32 * CPH; i += 64) {
            const int row = i / CPH, c = i % CPH * 8, p = group_row(0) + row;
            if (p >= T) continue;
            float lo[8], hi[8];
#pragma unroll
            for (int e = 0; e < 8; e += 4) {
                *(float4*)(lo + e) = *(const float4*)(slab + row * LD + c + e);
                *(float4*)(hi + e) = *(const float4*)(slab + row * LD + HALF_D + c + e);
            }
            if (table) {       // the inverse rotation of the pairs (d, d + DH / 2), the adjoint of the forward one
                const float2* cs = table + (long)p * HALF_D + c;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = lo[e], y = hi[e], sn = -cs[e].y;
                    lo[e] = x * cs[e].x - y * sn;
                    hi[e] = y * cs[e].x + x * sn;
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) { lo[e] *= mul; hi[e] *= mul; }
            *(uint4*)(dst + (long)p * ldq + hd + c) = pack8(lo);
            *(uint4*)(dst + (long)p * ldq + hd + HALF_D + c) = pack8(hi);
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto out1 = [&](const f32x16_t* a) { out(a, DQ ? dq : dk, scale, rope); };
    auto out2 = [&](const f32x16_t* a) { out(a, dv, 1.f, nullptr); };
    if constexpr (NG == 2) {
        put(acc1[1], 0);
        if constexpr (!DQ) put(acc2[1], 4 * ND);
        __syncthreads();
        add(acc1[0], 0);
        if constexpr (!DQ) add(acc2[0], 4 * ND);
        __syncthreads();
        out1(acc1[0]);
        if constexpr (!DQ) out2(acc2[0]);
    } else if constexpr (DQ) {
        if (sg == 1) put(acc1[0], 0);
        __syncthreads();
        if (sg == 0) { add(acc1[0], 0); out1(acc1[0]); }
    } else {
        if (sg == 0) put(acc2[0], 0); else put(acc1[0], 0);
        __syncthreads();
        if (sg == 0) add(acc1[0], 0); else add(acc2[0], 0);
        __syncthreads();
        if (sg == 0) out1(acc1[0]); else out2(acc2[0]);
    }
}

// Both kinds of part in one launch.  Every workgroup does ONE part -- the dK/dV of a key block (all queries from it on) or the dQ of a
// query block (all keys up to it) -- and the parts are handed out longest first: level j of the grid holds the dK/dV part of key
// block j and the dQ part of query block n - 1 - j of every head, and levels run from the heaviest down.  As two launches each part
// list has an 8:1 causal imbalance between its workgroups at 1024 tokens, and the chip waits for the longest one twice; in one launch a
// CU that finishes a light part picks up the next.  delta must already be in memory (the dK/dV parts read rows that other
// workgroups' dQ parts own).  grid = (n blocks, heads, 2).
template <int DH, bool DIRECT>
__global__ __launch_bounds__(256, DH == 128 ? 1 : 2) void attn_bwd_fused_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ delta, long ldq, long ldo,
    int T, bf16_t* __restrict__ dq, bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, float scale,
    const float2* __restrict__ rope) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int n = gridDim.x, heads = gridDim.y;
    const int idx = (blockIdx.z * heads + blockIdx.y) * n + blockIdx.x;   // position in dispatch order (x fastest)
    const int level = idx / (2 * heads), r = idx % (2 * heads), head = r % heads;
    if (r < heads) attn_bwd_part<DH, false, DIRECT>(q, k, v, d_o, lse, delta, ldq, ldo, T, dq, dk, dv, scale, rope, level, head, smem);
    else attn_bwd_part<DH, true, DIRECT>(q, k, v, d_o, lse, delta, ldq, ldo, T, dq, dk, dv, scale, rope, n - 1 - level, head, smem);
}

// ======================================================================== launchers
template <int DH>
static hipError_t run_fwd(dim3 grid, const bf16_t* q, const bf16_t* k, const bf16_t* v, long ldq, int T, bf16_t* o,
                          long ldo, float* lse, float sl2, hipStream_t s) {
    const size_t lds = (size_t)ATTN_KG * 4 * 64 * DH * sizeof(bf16_t);
    const bool direct = loads_to_lds(q) && loads_to_lds(k) && loads_to_lds(v);
    auto kern = direct ? attn_fwd_kernel<DH, true> : attn_fwd_kernel<DH, false>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kern<<<grid, ATTN_KG * ATTN_NW * 64, lds, s>>>(q, k, v, ldq, T, o, ldo, lse, sl2);
    return hipGetLastError();
}

hipError_t launch_attention_fwd(const bf16_t* q, const bf16_t* k, const bf16_t* v, long ldq, int T, int n_heads,
                                int d_head, bf16_t* o, long ldo, float* lse, hipStream_t s) {
    if (T <= 0 || n_heads <= 0) return hipSuccess;
    if ((ldq & 7) || (ldo & 7)) return hipErrorInvalidValue;
    const float sl2 = (1.f / sqrtf((float)d_head)) * 1.4426950408889634f;
    dim3 grid(cdiv(T, ATTN_NW * 32), n_heads);
    if (d_head == 128) return run_fwd<128>(grid, q, k, v, ldq, T, o, ldo, lse, sl2, s);
    if (d_head == 64) return run_fwd<64>(grid, q, k, v, ldq, T, o, ldo, lse, sl2, s);
    return hipErrorInvalidValue;
}

// delta[head][t] = dO[t, head, :] . O[t, head, :] on its own, for the one-launch backward, whose dK/dV parts cannot
// wait for the dQ parts of other workgroups to produce it: DH / 8 lanes per (t, head), 16 bytes each.
template <int DH>
__global__ __launch_bounds__(256) void attn_delta_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o,
                                                         long ldo, int T, int n_heads, float* __restrict__ delta) {
    // grid: x over the heads of a token (256 / LPR heads per workgroup), y over tokens
    constexpr int LPR = DH / 8;
    const int head_raw = (int)(blockIdx.x * 256 + threadIdx.x) / LPR, sub = threadIdx.x % LPR;
    const bool live = head_raw < n_heads;
    const int head = live ? head_raw : 0;
    for (long t = blockIdx.y; t < T; t += gridDim.y) {
        float a[8], b[8], dot = 0.f;
        unpack8(*(const uint4*)(o + t * ldo + (long)head * DH + sub * 8), a);
        unpack8(*(const uint4*)(d_o + t * ldo + (long)head * DH + sub * 8), b);
#pragma unroll
        for (int e = 0; e < 8; ++e) dot += a[e] * b[e];
        for (int off = LPR >> 1; off > 0; off >>= 1) dot += __shfl_xor(dot, off, 64);
        if (live && sub == 0) delta[(long)head * T + t] = dot;
    }
}

// delta from its own small kernel, then one launch that holds every dK/dV and every dQ part, longest first.
template <int DH>
static hipError_t run_bwd(const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* o, const bf16_t* d_o,
                          const float* lse, float* delta, long ldq, long ldo, int T, int n_heads, bf16_t* dq, bf16_t* dk,
                          bf16_t* dv, const float2* rope, hipStream_t s) {
    using C = BwdCfg<DH>;
    const float scale = 1.f / sqrtf((float)DH);
    dim3 grid(cdiv(T, C::PB), n_heads, 2);
    const dim3 dgrid(cdiv((long)n_heads * (DH / 8), 256), T < 65535 ? T : 65535);
    attn_delta_kernel<DH><<<dgrid, 256, 0, s>>>(o, d_o, ldo, T, n_heads, delta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool direct = loads_to_lds(q) && loads_to_lds(k) && loads_to_lds(v) && loads_to_lds(d_o);
    auto kern = direct ? attn_bwd_fused_kernel<DH, true> : attn_bwd_fused_kernel<DH, false>;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e != hipSuccess) return e;
    kern<<<grid, 256, C::LDS, s>>>(q, k, v, d_o, lse, delta, ldq, ldo, T, dq, dk, dv, scale, rope);
    return hipGetLastError();
}

// delta (fp32 [n_heads, T]) = rowsum(dO * O), workspace written here and read by the dK/dV part.  rope != null: q and k
// were rotated by RoPE (table of (cos, sin) per position and pair, positions 0 .. T-1) before the forward pass, and dq,
// dk come out as gradients with respect to the UNROTATED projections.
hipError_t launch_attention_bwd(const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* o, const bf16_t* d_o,
                                const float* lse, long ldq, long ldo, int T, int n_heads, int d_head, bf16_t* dq,
                                bf16_t* dk, bf16_t* dv, float* delta, const float2* rope, hipStream_t s) {
    if (T <= 0 || n_heads <= 0) return hipSuccess;
    if ((ldq & 7) || (ldo & 7)) return hipErrorInvalidValue;
    if (d_head == 128) return run_bwd<128>(q, k, v, o, d_o, lse, delta, ldq, ldo, T, n_heads, dq, dk, dv, rope, s);
    if (d_head == 64) return run_bwd<64>(q, k, v, o, d_o, lse, delta, ldq, ldo, T, n_heads, dq, dk, dv, rope, s);
    return hipErrorInvalidValue;
}
