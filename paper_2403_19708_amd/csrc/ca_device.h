// Device helpers shared by the attention kernels.
#pragma once

#include "ca_internal.h"

namespace ca {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

__device__ inline float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ inline uint32_t pack_bf16(float a, float b) {
    bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in bits 3:0 and
// 15:14, expcnt 6:4 and lgkmcnt 11:8 left at "don't wait")
#define CA_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// *p through the scalar cache: p is uniform and nothing writes *p while the kernel runs
__device__ inline int32_t load_uniform(const int32_t *p) {
    return *reinterpret_cast<const __attribute__((address_space(4))) int32_t *>(reinterpret_cast<uintptr_t>(p));
}

// 16 bytes per lane, global -> LDS at lds_base + lane*16, no register in between.  Written as inline
// assembly on purpose: the compiler then knows nothing of the outstanding load and does not guard
// every later LDS read with s_waitcnt vmcnt(0) (it cannot tell which LDS bytes the load will write);
// the waits are placed by hand with CA_WAIT_VMCNT, which the in-order completion of these loads
// makes exact.  lds_base must be wave-uniform.
__device__ inline void dma16(const void *src, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"(src) : "memory", "m0");
}

// same, with the address split into a wave-uniform 64-bit base (scalar registers) and a 32-bit
// per-lane byte offset: no vector arithmetic per load
__device__ inline void dma16_sbase(const void *base_uniform, uint32_t lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 : : "s"(lds_base), "v"(lane_off), "s"(base_uniform) : "memory", "m0");
}

// same, for data that is read once
__device__ inline void dma16_sbase_nt(const void *base_uniform, uint32_t lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 : : "s"(lds_base), "v"(lane_off), "s"(base_uniform) : "memory", "m0");
}

__device__ inline uint32_t lds_offset(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// Results that a workgroup on another die reads inside the same launch: written through and read past the dies' own caches
// (agent scope).  A release fence instead would write back a die's whole L2, once per wavefront.
// Through a buffer descriptor (`base` wave-uniform, `at` in bytes): one instruction moves 16 bytes, where an atomic access
// moves 8 at most.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
constexpr int kAgentScope = 16;                    // sc1
__device__ inline __amdgpu_buffer_rsrc_t buffer_at(float *base) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000); }
__device__ inline void store_agent4(__amdgpu_buffer_rsrc_t b, int at, f32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, at, 0, kAgentScope);
}
__device__ inline void store_agent2(__amdgpu_buffer_rsrc_t b, int at, float2 v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, at, 0, kAgentScope);
}
__device__ inline f32x4 load_agent4(__amdgpu_buffer_rsrc_t b, int at) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, kAgentScope));
}
__device__ inline float2 load_agent2(__amdgpu_buffer_rsrc_t b, int at) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(b, at, 0, kAgentScope));
}
// Counts a workgroup in whose stores of this kind are done; true in the one that is the n-th (which may then read the
// others').  Called by every thread of the workgroup; `flag` is in LDS.  The n-th brings the count back to zero in the same
// atomic operation: no count in between can be lost.
__device__ inline bool arrive_last(uint32_t *count, int n, int32_t *flag) {
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");    // this wavefront's stores have been acknowledged
    __syncthreads();
    if (threadIdx.x == 0) *flag = atomicInc(count, (unsigned)(n - 1)) == (unsigned)(n - 1);
    __syncthreads();
    return *flag != 0;
}

// (cos, sin) of position pos for the eight rotary pairs that the 16-byte pieces `piece` and `piece` + D/16 of a row hold
template <int D, int STYLE>
__device__ inline void load_cs(const float2 *__restrict__ rope, int pos, int piece, float2 (&cs)[8]) {
    constexpr int HALF = D / 2;
    const float2 *row = rope + (int64_t)pos * HALF;
    if (STYLE == 0) {
        const float4 *p = reinterpret_cast<const float4 *>(row + 8 * piece);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 v = p[w];
            cs[2 * w] = make_float2(v.x, v.y);
            cs[2 * w + 1] = make_float2(v.z, v.w);
        }
    } else {
        const float4 *p = reinterpret_cast<const float4 *>(row + 4 * piece);
        const float4 *q = reinterpret_cast<const float4 *>(row + HALF / 2 + 4 * piece);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const float4 v = p[w], u = q[w];
            cs[2 * w] = make_float2(v.x, v.y);
            cs[2 * w + 1] = make_float2(v.z, v.w);
            cs[4 + 2 * w] = make_float2(u.x, u.y);
            cs[4 + 2 * w + 1] = make_float2(u.z, u.w);
        }
    }
}

// one dword (2 elements) of each of the two 16-byte pieces a (dims d0..) and b (dims d0 + D/2..)
// (f = a factor applied to the rotated values before they are rounded)
template <int STYLE>
__device__ inline void rotate_dword(uint32_t &pa, uint32_t &pb, const float2 (&cs)[8], int w, float f = 1.0f) {
    const float a0 = bf_lo(pa), a1 = bf_hi(pa);
    const float b0 = bf_lo(pb), b1 = bf_hi(pb);
    if (STYLE == 0) {
        const float2 c0 = cs[2 * w], c1 = cs[2 * w + 1];
        pa = pack_bf16((a0 * c0.x - b0 * c0.y) * f, (a1 * c1.x - b1 * c1.y) * f);
        pb = pack_bf16((b0 * c0.x + a0 * c0.y) * f, (b1 * c1.x + a1 * c1.y) * f);
    } else {
        const float2 ca_ = cs[w], cb_ = cs[4 + w];
        pa = pack_bf16((a0 * ca_.x - a1 * ca_.y) * f, (a1 * ca_.x + a0 * ca_.y) * f);
        pb = pack_bf16((b0 * cb_.x - b1 * cb_.y) * f, (b1 * cb_.x + b0 * cb_.y) * f);
    }
}

// What lanes of a wavefront wrote to LDS in front of this, its other lanes read behind it.  The hardware keeps the LDS accesses of a
// wavefront in order; the compiler sees the addresses of one lane only and has to be told (no instruction comes of it).
__device__ inline void lds_handover() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The 32 stacked query rows row_first .. of a wavefront, rotated, scaled by `f` and rounded, as B operand of S^T = K Q^T (lane ->
// row lane % 32, k-step ks -> piece 2 ks + lane / 32).  A lane that fetches its own row touches 32 cache lines in every
// instruction, each line in four instructions, for the queries and again for the rotary table, and the first level cache does not hold
// the lines of eight wavefronts that long: 10.6 us from the start of a workgroup of 256 rows to its first tile (32 heads, one
// row per position).  Here D / 4 lanes fetch a row and its table row side by side, two rotary pairs each, and the rotated row goes
// through LDS to the lanes that want it.  `fetch` only asks for the data; `finish` needs stage(): kQueryBytes of LDS that nobody else uses.
template <int D, int STYLE>
struct QueryRows {
    static constexpr int kStride = 2 * D + 16;             // bytes of a row in LDS: 16-byte reads of 32 rows are free of bank conflicts
    static constexpr int kQueryBytes = 32 * kStride;
    static constexpr int LPR = D / 4;                      // lanes per row
    static constexpr int RPS = 64 / LPR;                   // rows per step
    static constexpr int STEPS = 32 / RPS;
    float4 cs[STEPS];                                      // (cos, sin) of pairs 2 c and 2 c + 1, c = lane % LPR
    uint32_t x[STEPS], y[STEPS];

    __device__ inline void fetch(const AttnArgs &a, int q0, int g, int G, int n, int row_first, int row_last) {
        const int lane = threadIdx.x & 63, c = lane % LPR;
        const int j0 = row_first / G, r0 = j0 * G;               // (wave-uniform)
        const float per_g = 1.0f / (float)G;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int r = min(row_first + i * RPS + lane / LPR, row_last);
            const int j = j0 + (int)(((float)(r - r0) + 0.5f) * per_g);      // r / G (the operand is below G + 32)
            const uint16_t *row = a.q + ((int64_t)(q0 + j) * a.n_q_heads + g * G + (r - j * G)) * D;
            cs[i] = *reinterpret_cast<const float4 *>(a.rope + (int64_t)(n + j) * (D / 2) + 2 * c);
            if (STYLE == 0) {
                x[i] = *reinterpret_cast<const uint32_t *>(row + 2 * c);
                y[i] = *reinterpret_cast<const uint32_t *>(row + D / 2 + 2 * c);
            } else {
                const uint2 v = *reinterpret_cast<const uint2 *>(row + 4 * c);
                x[i] = v.x;
                y[i] = v.y;
            }
        }
    }
    __device__ inline void finish(uint8_t *stage, float f, bf16x8 (&Qf)[D / 16]) {
        const int lane = threadIdx.x & 63, c = lane % LPR;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const float2 first = make_float2(cs[i].x, cs[i].y), second = make_float2(cs[i].z, cs[i].w);
            const float2 both[8] = {first, second, first, second, second, second, second, second};
            rotate_dword<STYLE>(x[i], y[i], both, 0, f);         // (STYLE 0: pairs both[0], both[1]; 1: both[0], both[4])
            uint8_t *at = stage + (i * RPS + lane / LPR) * kStride;
            if (STYLE == 0) {
                *reinterpret_cast<uint32_t *>(at + 4 * c) = x[i];
                *reinterpret_cast<uint32_t *>(at + D + 4 * c) = y[i];
            } else {
                *reinterpret_cast<uint2 *>(at + 8 * c) = make_uint2(x[i], y[i]);
            }
        }
        lds_handover();
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            Qf[ks] = *reinterpret_cast<const bf16x8 *>(stage + lane % 32 * kStride + 16 * (2 * ks + lane / 32));
    }
};

// The 32 stacked rows of a wavefront, normalised and rounded, from the C layout of O^T (lane -> row lane % 32, dims 32 db + 8 i +
// 4 (lane / 32) .. + 3 in registers 4 i .. of block db) to `out`.  A lane that stores its own row writes 16 bytes of 32 lines in every
// instruction; through LDS (`stage`: kQueryBytes that nobody else uses) an instruction writes whole lines.
template <int D>
__device__ inline void store_rows(const AttnArgs &a, int q0, int g, int G, int row_first, int row_last, uint8_t *stage, const f32x16 (&O)[D / 32], float inv) {
    constexpr int kStride = QueryRows<D, 0>::kStride, LPR = D / 8, RPS = 64 / LPR;      // lanes per row, rows per instruction
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint2 o = make_uint2(pack_bf16(O[db][4 * i] * inv, O[db][4 * i + 1] * inv), pack_bf16(O[db][4 * i + 2] * inv, O[db][4 * i + 3] * inv));
            *reinterpret_cast<uint2 *>(stage + lane % 32 * kStride + 2 * (32 * db + 8 * i + 4 * (lane / 32))) = o;
        }
    lds_handover();
    const int j0 = row_first / G, r0 = j0 * G;                   // (wave-uniform)
    const float per_g = 1.0f / (float)G;
#pragma unroll
    for (int i = 0; i < 32 / RPS; ++i) {
        const int at = i * RPS + lane / LPR, r = row_first + at;
        const uint4 o = *reinterpret_cast<const uint4 *>(stage + at * kStride + 16 * (lane % LPR));
        const int j = j0 + (int)(((float)(r - r0) + 0.5f) * per_g);          // r / G (the operand is below G + 32)
        if (r <= row_last) *reinterpret_cast<uint4 *>(a.out + ((int64_t)(q0 + j) * a.n_q_heads + g * G + (r - j * G)) * D + 8 * (lane % LPR)) = o;
    }
}

// four head dimensions d.. of stacked row `row` of a (conversation with first new token q0, kv head g), normalised
template <int D>
__device__ inline void store_out_row4(const AttnArgs &a, int q0, int g, int G, int row, int d, f32x4 o, float inv) {
    const int j = row / G;
    const int head = g * G + (row - j * G);
    uint2 b;
    b.x = pack_bf16(o[0] * inv, o[1] * inv);
    b.y = pack_bf16(o[2] * inv, o[3] * inv);
    *reinterpret_cast<uint2 *>(a.out + ((int64_t)(q0 + j) * a.n_q_heads + head) * D + d) = b;
}

}  // namespace

}  // namespace ca
