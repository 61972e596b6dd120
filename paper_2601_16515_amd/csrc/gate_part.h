// Gate pass 1 as device code: the gate kernel and the kernels that do the gate next to the linear state share it.
#pragma once
#include "salad_internal.h"

namespace salad {

// ------------------------------------------------------------------------------------------------
// Gate pass 1 (Alg. 1 Level 2): sum over a strided set of tokens of sigmoid(x.w + bias).
// One wave per token at a time; a lane owns 8-element chunks lane, lane+64, ... of the row and the
// matching gate weights in registers.  HBM-bound: x_t is read exactly once, 16 bytes per lane per
// load for bf16 (32 for fp32).  Partial sums are written per workgroup and added up in a fixed
// order by the finalize kernel, so the result does not depend on scheduling.
// ------------------------------------------------------------------------------------------------
constexpr int GATE_MAX_CHUNKS = 10;   // D <= 8*64*10 = 5120

// Raw 8-element chunk of a row: 16 bytes (bf16) or 32 bytes (fp32) per lane.
template <bool BF16> struct Chunk8;
template <> struct Chunk8<true> {
    uint4 u;
    __device__ inline void load(const void *row, int chunk) { u = *reinterpret_cast<const uint4 *>(reinterpret_cast<const u16 *>(row) + chunk * 8); }
    __device__ inline void zero() { u = make_uint4(0, 0, 0, 0); }
    __device__ inline float dot(const float (&w)[8], float acc) const
    {
        const uint32_t v[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc = fmaf(__uint_as_float(v[i] << 16), w[2 * i], acc);
            acc = fmaf(__uint_as_float(v[i] & 0xffff0000u), w[2 * i + 1], acc);
        }
        return acc;
    }
};
template <> struct Chunk8<false> {
    float v[8];
    __device__ inline void load(const void *row, int chunk)
    {
        const float4 *p = reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(row) + chunk * 8);
        const float4 a = p[0], b = p[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
    __device__ inline void zero()
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.f;
    }
    __device__ inline float dot(const float (&w)[8], float acc) const
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fmaf(v[i], w[i], acc);
        return acc;
    }
};

// NCH: 8-element chunks per lane (D <= 512 * NCH); TOK: tokens a wave handles per step.  The loads of the
// next step are issued before the current step is reduced (two register buffers), so a wave always has
// TOK*NCH 16-byte loads per lane in flight while it runs the dot products, the wave reduction and the
// sigmoid of the previous tokens.
// Called by all threads of a workgroup; 4 waves (`wave` 0..3) share one partial sum: number `part` of sample b, nothing if
// part >= nparts.  wave_sum: 4 floats of LDS.
template <bool BF16, int NCH, int TOK>
__device__ inline __attribute__((always_inline)) void gate_part(const void *x_t, const float *__restrict__ w, float bias, int N, int D,
                                                                float *__restrict__ partial, int nparts, int b, int part, int wave,
                                                                float *wave_sum)
{
    const int lane = threadIdx.x & 63;
    const int nch = D >> 3;
    float wr[NCH][8];
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        int c = lane + 64 * j;
#pragma unroll
        for (int e = 0; e < 8; ++e) wr[j][e] = (c < nch) ? w[c * 8 + e] : 0.f;
    }
    const size_t esz = BF16 ? 2 : 4;
    const char *xb = reinterpret_cast<const char *>(x_t) + (size_t)b * N * D * esz;
    const int stride = nparts * 4 * TOK;
    float acc = 0.f;
    Chunk8<BF16> bufA[TOK][NCH], bufB[TOK][NCH];
    auto issue = [&](Chunk8<BF16> (&buf)[TOK][NCH], int n0) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < TOK; ++t) {
            const int n = n0 + t < N ? n0 + t : N - 1;
            const void *row = xb + (size_t)n * D * esz;
#pragma unroll
            for (int j = 0; j < NCH; ++j) {
                const int c = lane + 64 * j;
                if (c < nch) buf[t][j].load(row, c);
                else buf[t][j].zero();
            }
        }
    };
    auto consume = [&](const Chunk8<BF16> (&buf)[TOK][NCH], int n0) __attribute__((always_inline)) {
        float dot[TOK];
#pragma unroll
        for (int t = 0; t < TOK; ++t) {
            dot[t] = 0.f;
#pragma unroll
            for (int j = 0; j < NCH; ++j) dot[t] = buf[t][j].dot(wr[j], dot[t]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int t = 0; t < TOK; ++t) dot[t] += __shfl_xor(dot[t], o);
#pragma unroll
        for (int t = 0; t < TOK; ++t)
            if (n0 + t < N) acc += 1.f / (1.f + __expf(-(dot[t] + bias)));   // identical in every lane
    };
    int n0 = part < nparts ? (part * 4 + wave) * TOK : N;
    if (n0 < N) issue(bufA, n0);
    while (n0 < N) {
        if (n0 + stride < N) issue(bufB, n0 + stride);
        consume(bufA, n0);
        n0 += stride;
        if (n0 >= N) break;
        if (n0 + stride < N) issue(bufA, n0 + stride);
        consume(bufB, n0);
        n0 += stride;
    }
    if (lane == 0) wave_sum[wave] = acc;
    __syncthreads();
    if (lane == 0 && wave == 0 && part < nparts)
        partial[(size_t)b * nparts + part] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
}

}  // namespace salad
