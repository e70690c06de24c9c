// What the kernels that stream weights past a handful of tokens share: their fragment reads, and the rows such a product
// multiplies, computed by every workgroup from what they are made of (SkinnySource).
#pragma once
#include "blr_common.h"

namespace blr {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));   // (arrays of HIP's uint4 struct stay in scratch memory)

__device__ __attribute__((aligned(16))) const unsigned char zero_piece[16] = {0};   // the source of operand pieces past the contraction index

__device__ __forceinline__ bf16x8 lds_read_frag(unsigned addr) {   // (reads the compiler can see wait for all direct loads)
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr) : "memory");
    return v;
}

__device__ __forceinline__ void unpack8(u32x4 v, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[2 * i] = __uint_as_float(v[i] << 16); f[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u); }
}
__device__ __forceinline__ u32x4 pack8(const float (&f)[8]) {
    return u32x4{pack2_bf16(f[0], f[1]), pack2_bf16(f[2], f[3]), pack2_bf16(f[4], f[5]), pack2_bf16(f[6], f[7])};
}

// Rows [M][K] of batch entry g, bf16, row pitch xs bytes, from their source.
// Every thread of the workgroup takes part; the caller's barrier follows. `red`: 8 M floats of scratch.
template <int SRC, int NW>
__device__ __forceinline__ void source_rows(const SkinnySource& q, int M, int K, int g, unsigned char* rows, unsigned xs, float* red) {
    const int tid = threadIdx.x;
    if constexpr (SRC == kSrcNorm) {
        // H' = H + Y rounded to storage, n = H' / rms(H'): the whole row for the sum, the slice [g K, g K + K) for the product
        const int wave = tid >> 6, k0 = g * K;
        for (int m = 0; m < M; ++m) {
            const bf16_t* h = q.a + (int64_t)m * q.d;
            float ss = 0.f;
            for (int c = tid * 8; c < q.d; c += NW * 64 * 8) {
                u32x4 v = *(const u32x4*)(h + c);
                float f[8];
                unpack8(v, f);
                if (q.y) {
                    float y[8];
                    unpack8(*(const u32x4*)(q.y + (int64_t)m * q.d + c), y);
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] += y[i];
                    v = pack8(f);
                    unpack8(v, f);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) ss += f[i] * f[i];
                if (c >= k0 && c < k0 + K) *(u32x4*)(rows + m * xs + (c - k0) * 2) = v;
                if (q.out && (blockIdx.x | blockIdx.y | blockIdx.z) == 0) *(u32x4*)(q.out + (int64_t)m * q.d + c) = v;   // (a buffer nobody reads in this launch)
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
            if ((tid & 63) == 0) red[m * 8 + wave] = ss;
        }
        __syncthreads();
        for (int it = tid; it < M * (K >> 3); it += NW * 64) {
            const int m = it / (K >> 3), c = it - m * (K >> 3);
            float ss = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) ss += red[m * 8 + w];
            const float scale = rsqrtf(ss / (float)q.d + q.scale);             // scale: eps
            unsigned char* p = rows + m * xs + c * 16;
            float f[8];
            unpack8(*(const u32x4*)p, f);
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] *= scale;
            *(u32x4*)p = pack8(f);
        }
    }
}

}  // namespace
}  // namespace blr
