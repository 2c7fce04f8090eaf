// MFMA tile helpers shared by the GEMM and attention kernels (gfx950).
//
// v_mfma_f32_32x32x16_bf16 operand layout (lane = 32*g + l32):
//   A fragment: row  i = l32, contraction slots k = 8g .. 8g+7   (8 bf16 = 16 bytes per lane)
//   B fragment: col  j = l32, contraction slots k = 8g .. 8g+7
//   D fragment: col  j = l32, rows i = 8*(v/4) + 4g + v%4 for v = 0..15
// Because the contraction is a sum, any permutation of the 16 slots is allowed as long as A and B
// use the same one.  A D fragment reused as a B operand (keeping j) supplies, for registers
// v = 8h .. 8h+7, the slot order  i = 16h + {4g..4g+3, 8+4g..8+4g+3}; the A operand is then read
// as two 4-slot pieces at i = 16h+4g and 16h+8+4g (read_tr_frag below).
#pragma once
#include "common.h"

#define BK 64
#define LS 72  // LDS row stride (elements) of a 64-wide K-contiguous bf16 tile read with 16-byte accesses

__device__ __forceinline__ f32x16_t mfma32(bf16x8_t a, bf16x8_t b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16_t zero16() {
    f32x16_t z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
}

// registers v = 8h .. 8h+7 of a D fragment, rounded to bf16, as a B operand
__device__ __forceinline__ bf16x8_t pack_b_from_d(const float* d, int h) {
    bf16x8_t b;
#pragma unroll
    for (int e = 0; e < 8; ++e) b[e] = (__bf16)d[8 * h + e];
    return b;
}

// Direct-to-LDS loads: each lane's 16 (4) bytes land at lds_addr + 16 (4) * lane.
__device__ __forceinline__ void load_lds16(unsigned voff, const void* sbase, unsigned lds_addr) {
    // M0 carries the LDS destination: bound as a physical-register operand, so the compiler sets it and knows it is used
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "{m0}"(lds_addr) : "memory");
}
__device__ __forceinline__ void load_lds4(const void* p, unsigned lds_addr) {
    asm volatile("global_load_lds_dword %0, off" ::"v"(p), "{m0}"(lds_addr) : "memory");
}
// 16 bytes a lane to lds_addr + 16 lane, by such a load (DIRECT) or, where the address may be no multiple of 4, through registers (waited for at once)
template <bool DIRECT>
__device__ __forceinline__ void bring_lds16(unsigned voff, const void* sbase, unsigned lds_addr, int lane) {
    if constexpr (DIRECT) {
        load_lds16(voff, sbase, __builtin_amdgcn_readfirstlane(lds_addr));
    } else {
        typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) u32x4_t* lds_ptr_t;
        *(lds_ptr_t)(uintptr_t)(lds_addr + 16 * lane) = *(const u32x4_t*)((const char*)sbase + voff);
    }
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A [rows][DH] tile by direct-to-LDS loads, one copy: 16-byte chunk c of row x lies at position c ^ tile_swz(x), so that both the reads of
// 16 rows at one chunk and the transposing reads of four rows x 64 bytes (read_tr_frag) fall into distinct banks.
template <int DH>
__device__ __forceinline__ int tile_swz(int row) {
    return DH == 128 ? 4 * (row & 3) | ((row >> 2) & 3) : 4 * ((row >> 1) & 1) | ((row >> 2) & 3);
}
// fetch i of a tile brings its rows i RPI .. (beyond `last`: that one again), each lane the chunk that belongs at its place; base: row 0, or a row that
// is a multiple of 16 further (rows up to 63 from it: the offset has 32 bits)
// DIRECT: the operand starts at a multiple of 4 bytes, else through registers
template <int DH, bool DIRECT>
struct TileFetch {
    static constexpr int CPR = DH / 8, RPI = 64 / CPR;         // chunks per row, rows per fetch
    int lane, fr;
    unsigned fc;
    __device__ __forceinline__ TileFetch(int lane) : lane(lane), fr(lane / CPR), fc((unsigned)((lane % CPR) ^ tile_swz<DH>(lane / CPR)) << 4) {}
    __device__ __forceinline__ void operator()(const bf16_t* base, unsigned ldb, int i, int last, unsigned lds) const {
        const unsigned c = fc ^ (unsigned)((i * (RPI / 4) & 3) << 4);                  // swz of rows i RPI + fr
        bring_lds16<DIRECT>((unsigned)min(i * RPI + fr, last) * ldb + c, base, lds + i * 1024, lane);
    }
};
// rows first .. end - 1 of such a tile made zero by one wave.  Fetches bring the last row again in the place of rows behind it; where the products
// take those with weights of 0, an infinity in the last row would turn into 0 x inf.
template <int DH>
__device__ __forceinline__ void clear_rows(unsigned char* tile, int first, int end, int lane) {
    for (int at = first * DH * 2 + lane * 16; at < end * DH * 2; at += 1024) *(uint4*)(tile + at) = make_uint4(0, 0, 0, 0);
}
// this lane's share of the address of a fragment of rows (row l32, chunk 2 ks + g: ^ ks << 5) ..
template <int DH>
__device__ __forceinline__ unsigned row_frag_at(int lane) {
    const int l32 = lane & 31, g = lane >> 5;
    return (unsigned)(l32 * DH * 2 + ((g ^ tile_swz<DH>(l32)) << 4));
}
// .. and of a transposing read (contraction rows 0 .. 15, columns 32 dt ..: ^ dt << 6; rows 8 further: ^ 32, + 8 rows).
// A operand for a D-fragment-as-B product (contraction slots 16h + {4g..4g+3, 8+4g..8+4g+3}, see the top of this
// file) taken from the tile as it lies in memory, [k][n] row-major with n contiguous, by the LDS transpose read of
// gfx950 (ds_read_b64_tr_b16): within each group of 16 lanes, lane 4q + c receives element c of the four 8-byte rows
// that lanes q, q + 4, q + 8, q + 12 of the group point at.  Lane q + 4e therefore points at row k0 + e, columns
// n0 + 4q .. 4q + 3, and lane 4q + c ends up with column n0 + 4q + c of rows k0 .. k0 + 3: four consecutive contraction
// slots of one operand row, which is what the matrix unit wants.  Lane groups 0 / 1 cover columns n0 .. 15 /
// n0 + 16 .. 31 (l32), groups 2 / 3 the same columns for g = 1.  Used for both operands of a product, the slot
// permutation cancels, so the same read serves ordinary P^T Q products (tn_tile).
template <int DH>
__device__ __forceinline__ unsigned tr_frag_at(int lane) {
    const int G = lane >> 4, te = (lane & 15) >> 2, tq = lane & 3;
    return (unsigned)((4 * (G >> 1) + te) * DH * 2 + ((DH == 128 ? te : te >> 1) << 6) + (((2 * (G & 1) + (tq >> 1)) ^ (G >> 1)) << 4) + ((tq & 1) << 3));
}
typedef __bf16 bf16x4v_t __attribute__((ext_vector_type(4)));
template <int DH>
__device__ __forceinline__ bf16x8_t read_tr_frag(const unsigned char* rows, unsigned at, int dt) {
    typedef __attribute__((address_space(3))) bf16x4v_t* lds_ptr_t;
    at ^= (unsigned)(dt << 6);
    const bf16x4v_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(rows + at));
    const bf16x4v_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(rows + (at ^ 32u) + 8 * DH * 2));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
