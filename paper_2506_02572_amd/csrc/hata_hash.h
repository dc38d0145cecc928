// HashEncode of a few vectors (Alg. 2 of the paper: Sign(x . W_H), BitPack) on the fp64 matrix instructions: query
// vectors and appended keys.
//
// Four bf16 vectors at a time against 64 (or 32) hash columns of a KV head's weights [128][r], by a workgroup of
// 256 threads, in fp64 (every product of a bf16 and an fp32 value is exact there, so the sign agrees with an
// exact evaluation unless |projection| is below ~1e-13) on v_mfma_f64_4x4x4_4b: four blocks of [4 hash columns x
// 4 channels] . [4 channels x 4 vectors], operands one value a lane -- A: column lane % 16, B: vector
// lane % 4, both: channel lane / 16; result: vector lane % 4, column lane / 16 + 4 (lane / 4 % 4).  The vectors
// are few, so the narrow instruction wastes nothing, and the contraction needs no sums across lanes.  A
// wave owns 16 columns, and lane / 16 stands for 32 consecutive channels.  16.6 cycles per instruction and
// SIMD: the 32 of a set of four vectors take 0.22 us, the conversions in their shadow.
#pragma once
#include "hata_device.h"

namespace hata {

// The 32 weights a lane needs: its column, its 32 channels.
template <int COLS>
struct HashWeights {
    static_assert(COLS == 64 || COLS == 32, "four waves of 16 columns, or two (the other two repeat them)");
    float w[32];
    // W: the first of the columns, r: the weights' row pitch
    __device__ __forceinline__ void fetch(const float* __restrict__ W, int r) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        uint32_t at = 4u * (uint32_t)(32 * (lane >> 4) * r + (COLS == 64 ? wave : wave & 1) * 16 + (lane & 15));
        asm volatile("" : "+v"(at));  // (addresses are made anew for every fetch instead of being kept)
        const char* base = reinterpret_cast<const char*>(W);
#pragma unroll
        for (int s = 0; s < 32; ++s) w[s] = *reinterpret_cast<const float*>(base + s * r * 4 + at);
    }
};

// this lane's 32 channels of a vector
__device__ __forceinline__ void hash_load_x(const uint16_t* __restrict__ x, uint4 (&r)[4]) {
    const uint16_t* p = x + 32 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = reinterpret_cast<const uint4*>(p)[i];
}

// or over the lanes that hold the other columns of this lane's vector (lane bits 2..5)
__device__ __forceinline__ uint32_t or_columns(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false);  // row_ror:4
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);  // row_ror:8
    float x, y;
    swap16(__uint_as_float(v), x, y);
    v = __float_as_uint(x) | __float_as_uint(y);
    swap32(__uint_as_float(v), x, y);
    return __float_as_uint(x) | __float_as_uint(y);
}

// Four vectors: x holds this lane's part of vector first + lane % 4.  Vector v's code words for these columns go to
// s_codes[v * pitch ...] where v is below `last`; complete after the caller's next barrier.
template <int COLS>
__device__ __forceinline__ void hash_pass(const HashWeights<COLS>& W, const uint4 (&x)[4], uint32_t* s_codes, int pitch,
                                          int first, int last) {
    double acc = 0.0;
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        // (without the barriers the compiler converts right behind the loads, or ahead of a loop around this:
        // waits early, and twice the registers)
        float w = W.w[s];
        asm volatile("" : "+v"(w));
        const uint4 q = x[s >> 3];
        uint32_t pair = ((s >> 1) & 3) == 0 ? q.x : ((s >> 1) & 3) == 1 ? q.y : ((s >> 1) & 3) == 2 ? q.z : q.w;
        asm volatile("" : "+v"(pair));
        const double xd = (double)((s & 1) ? bf16_hi(pair) : bf16_lo(pair));
        acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)w, xd, acc, 0, 0, 0);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = (lane >> 4) + (lane & 12);  // column of the result
    const int v = first + lane;
    const uint32_t bits = or_columns((acc >= 0.0 ? 1u : 0u) << m);
    if (lane < 4 && v < last && wave < COLS / 16) reinterpret_cast<uint16_t*>(s_codes)[v * pitch * 2 + wave] = (uint16_t)bits;
}

// One vector alone, over the vector ALU: a lane its column and its 32 channels of x.  The matrix instruction takes one vector as long
// as four, and a wave alone on its SIMD waits 31 cycles for each before the next; an fp64 FMA takes 4.4.
template <int COLS>
__device__ __forceinline__ void hash_one(const HashWeights<COLS>& W, const uint4 (&x)[4], uint32_t* s_codes, int pitch, int vector) {
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        float w = W.w[s];
        asm volatile("" : "+v"(w));  // (as above)
        const uint4 q = x[s >> 3];
        uint32_t pair = ((s >> 1) & 3) == 0 ? q.x : ((s >> 1) & 3) == 1 ? q.y : ((s >> 1) & 3) == 2 ? q.z : q.w;
        asm volatile("" : "+v"(pair));
        acc[s & 1] = fma((double)w, (double)((s & 1) ? bf16_hi(pair) : bf16_lo(pair)), acc[s & 1]);
    }
    double t = acc[0] + acc[1];
    t += __shfl_xor(t, 16, 64);
    t += __shfl_xor(t, 32, 64);
    const unsigned long long bits = __builtin_amdgcn_ballot_w64(t >= 0.0);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0 && wave < COLS / 16) reinterpret_cast<uint16_t*>(s_codes)[vector * pitch * 2 + wave] = (uint16_t)bits;
}

// ---- the same by 16 waves, each 16 columns and a part of the channels (r = 32 .. 256: 8, 4, 2 or 1 parts) ----
template <int R>
struct UnitHash {
    static constexpr int GROUPS = R / 16, PARTS = 16 / GROUPS;  // groups of 16 columns; waves of a group
    static constexpr int CH = HATA_D / PARTS / 4;               // channels of a lane
    float w[CH];
    // the wave's first channel, and this lane's
    static __device__ __forceinline__ int channel() {
        return (threadIdx.x >> 6) / GROUPS * (HATA_D / PARTS) + CH * ((threadIdx.x & 63) >> 4);
    }
    __device__ __forceinline__ void fetch(const float* __restrict__ W) {
        const float* p = W + (int64_t)channel() * R + (threadIdx.x >> 6) % GROUPS * 16 + (threadIdx.x & 15);
#pragma unroll
        for (int s = 0; s < CH; ++s) w[s] = p[s * R];
    }
    struct Vector { uint32_t x[CH / 2]; };
    static __device__ __forceinline__ Vector fetch_x(const uint16_t* __restrict__ x) {
        Vector v;
        const uint16_t* p = x + channel();
        if constexpr (CH == 4) {
            const uint2 a = *reinterpret_cast<const uint2*>(p);
            v.x[0] = a.x; v.x[1] = a.y;
        } else {
#pragma unroll
            for (int i = 0; i < CH / 8; ++i) {
                const uint4 a = reinterpret_cast<const uint4*>(p)[i];
                v.x[4 * i] = a.x; v.x[4 * i + 1] = a.y; v.x[4 * i + 2] = a.z; v.x[4 * i + 3] = a.w;
            }
        }
        return v;
    }
    // this wave's part of four projections (result: vector lane % 4, column lane / 16 + 4 (lane / 4 % 4) of the group)
    __device__ __forceinline__ double project(const Vector& v) const {
        double acc = 0.0;
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const double xd = (double)((s & 1) ? bf16_hi(v.x[s >> 1]) : bf16_lo(v.x[s >> 1]));
            acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)w[s], xd, acc, 0, 0, 0);
        }
        return acc;
    }
    // This lane's part of ONE vector's projection (v: that vector's channels in every lane) on the vector ALU: column lane % 16, its
    // own channels.  A pass of one vector takes the matrix instruction as long as one of four, this a quarter of that.
    __device__ __forceinline__ double project_one(const Vector& v) const {
        double acc = 0.0;
#pragma unroll
        for (int s = 0; s < CH; ++s)
            acc = fma((double)w[s], (double)((s & 1) ? bf16_hi(v.x[s >> 1]) : bf16_lo(v.x[s >> 1])), acc);
        return acc;
    }
    // sign bits of such a projection, the waves' parts added up
    static __device__ __forceinline__ void store_bits_one(double acc, uint32_t* s_codes, int group, int vector) {
        acc += __shfl_xor(acc, 16, 64);
        acc += __shfl_xor(acc, 32, 64);
        const unsigned long long bits = __builtin_amdgcn_ballot_w64(acc >= 0.0);
        if ((threadIdx.x & 63) == 0) reinterpret_cast<uint16_t*>(s_codes)[vector * (R / 16) + group] = (uint16_t)bits;
    }
    // sign bits of a whole projection: 16 bits of vector first + lane % 4 (below `last`), into s_codes[vector][R / 32]
    static __device__ __forceinline__ void store_bits(double acc, uint32_t* s_codes, int group, int first, int last) {
        const int lane = threadIdx.x & 63, v = first + lane;
        const uint32_t bits = or_columns((acc >= 0.0 ? 1u : 0u) << ((lane >> 4) + (lane & 12)));
        if (lane < 4 && v < last) reinterpret_cast<uint16_t*>(s_codes)[v * (R / 16) + group] = (uint16_t)bits;
    }
};

}  // namespace hata
