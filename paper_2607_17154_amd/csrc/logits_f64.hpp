// fp32 storage: router logits of 16 tokens by v_mfma_f64_16x16x4_f64, shared by
// the routing kernel and the similarity model.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ordermoe {

constexpr int LF_TOKENS = 16, LF_THREADS = 512, LF_WAVES = LF_THREADS / 64;

// LDS bytes of the K slices' fp64 sums (none with 8 or 16 expert blocks)
__host__ __device__ inline int logits_f64_part_bytes(int Epad) { return Epad <= 64 ? LF_WAVES * 256 * 8 : 0; }

// Logits of tokens t0 .. t0 + 15 of x [T][d] against all E experts of w [E][d]:
// out[token * ld + expert].  Called by a whole block of LF_THREADS; NBT, a power
// of two, is at least the number of 16-expert blocks.  The 8 waves take the
// expert blocks and, with fewer than 8 of them, KW slices of the K steps of 16;
// the slices' fp64 sums meet in `part` (LDS) and are added in slice order, then
// rounded once to fp32 (the products of fp32 values are exact in fp64).  A lane
// reads four consecutive K values of its token row and of its expert row (16
// bytes each) and feeds them to four MFMAs.  Rows past the batch and experts
// past E re-read the last one; their logits mean nothing.  With KW > 1 the
// logits are complete after the caller's next barrier, as they are with KW = 1.
// What bounds it is the latency of a few dependent rounds of reads: a thread per
// logit with a serial fp64 chain over d kept one read in flight.
template <int NBT>
__device__ inline void logits_f64(const float* x, int64_t T, const float* w, int E, int d, int64_t t0, int tid,
                                  float* out, int ld, double* part) {
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int EG = NBT < LF_WAVES ? NBT : LF_WAVES;      // expert groups
    constexpr int KW = LF_WAVES / EG;                        // K slices
    constexpr int NB = NBT / EG;                             // 16-expert blocks per wave
    constexpr int U = 4;                                     // K steps per set of reads
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Epad = (E + 15) & ~15;
    const int eg = wave / KW, kw = wave % KW;
    const int r16 = lane & 15, kq = (lane >> 4) * 4;
    const int64_t tok = t0 + r16 < T ? t0 + r16 : T - 1;
    const float* xr = x + tok * (int64_t)d + kq;
    const float* wr[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int e = (eg * NB + n) * 16 + r16;
        wr[n] = w + (int64_t)(e < E ? e : E - 1) * d + kq;
    }
    const int nsteps = d / 16;
    const int ns = (nsteps - kw + KW - 1) / KW;              // steps of this wave
    f64x4 acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = f64x4{0.0, 0.0, 0.0, 0.0};
    f32x4 xv[2][U], wv[2][U][NB];
    auto load = [&](int b, int i0) {                         // (past the end: the last step, not multiplied)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t o = (int64_t)(kw + KW * (i0 + u < ns ? i0 + u : ns - 1)) * 16;
            xv[b][u] = *(const f32x4*)(xr + o);
#pragma unroll
            for (int n = 0; n < NB; ++n) wv[b][u][n] = *(const f32x4*)(wr[n] + o);
        }
    };
    auto mma = [&](int b, int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u < ns)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xv[b][u][q], (double)wv[b][u][n][q],
                                                                      acc[n], 0, 0, 0);
    };
    if (ns > 0) {
        load(0, 0);
        for (int i = 0; i < ns; i += 2 * U) {
            load(1, i + U);
            mma(0, i);
            load(0, i + 2 * U);
            mma(1, i + U);
        }
    }
    // acc[n][i]: token 4 i + lane / 16, expert lane % 16 of the block
    if constexpr (KW == 1) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int e = (eg * NB + n) * 16 + r16;
            if (e < Epad)
#pragma unroll
                for (int i = 0; i < 4; ++i) out[(4 * i + (lane >> 4)) * ld + e] = (float)acc[n][i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wave * 256 + (4 * i + (lane >> 4)) * 16 + r16] = acc[0][i];
        __syncthreads();
        for (int p = tid; p < LF_TOKENS * Epad; p += LF_THREADS) {
            const int tr = p / Epad, e = p - tr * Epad;
            const double* q = part + (e >> 4) * KW * 256 + tr * 16 + (e & 15);
            double v = q[0];
#pragma unroll
            for (int s = 1; s < KW; ++s) v += q[s * 256];
            out[tr * ld + e] = (float)v;
        }
    }
}

}  // namespace ordermoe
