// Lookup tables: ComputeLookupTable (Alg. 2) + 8-bit quantisation, for the batch kernel and the
// few-query kernel.
#pragma once
#include "device_util.h"

// A workgroup (256 threads) builds the tables of queries [q0, q0 + count), one after the other.  A thread owns groups of
// four consecutive codes of one sub-quantizer (group eg = tid + WG r: sub-quantizer eg / 4, codes
// 4 (eg % 4) ..+3), so the 16 entries of a sub-quantizer sit in four neighbouring lanes: its
// offset and width are a minimum and a maximum over those lanes (register moves), the largest
// width a maximum over the wave and then over the waves (one barrier per query), and a group's
// four bytes leave as one store.  The codewords of a thread's groups are the same for every query
// and stay in registers when a sub-vector has at most four dimensions.  The arithmetic per entry
// is unchanged: squared differences (or products) summed in dimension order.
#define LUT_GROUPS_MAX (RAIRS_MAX_M * 4 / WG)           // groups per thread at the largest M
struct LutShared {
    float wave_span[2][WG / 64];                        // alternating by query: one barrier per query
    float bias_s[RAIRS_MAX_M];                          // only for the stage call's sum of the offsets
};
template <bool IP, int DSUB>                            // DSUB: dimensions of a sub-vector, 0 = any (codewords re-read)
static __device__ __forceinline__ void lut_build_wg(const float *__restrict__ q,
                                                    const float *__restrict__ codebook, int d, int M,
                                                    int64_t nq, int64_t q0, int count,
                                                    uint8_t *__restrict__ lut,
                                                    float *__restrict__ bias_sum,
                                                    float *__restrict__ scale, LutShared &sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int dsub = DSUB > 0 ? DSUB : d / M;
    const int ngroups = M * 4;
    constexpr int CW = DSUB > 0 ? DSUB : 1;
    float cw[LUT_GROUPS_MAX][4][CW];
    if (DSUB > 0) {
#pragma unroll
        for (int r = 0; r < LUT_GROUPS_MAX; r++) {
            const int eg = tid + WG * r;
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int t = 0; t < CW; t++)
                    cw[r][k][t] = eg < ngroups ? codebook[((size_t)eg * 4 + k) * DSUB + t] : 0.0f;
        }
    }
    for (int qi = 0; qi < count && q0 + qi < nq; qi++) {
        const int64_t qid = q0 + qi;
        const float *qq = q + (size_t)qid * d;
        float T[LUT_GROUPS_MAX][4], lo[LUT_GROUPS_MAX], span = 0.0f;
#pragma unroll
        for (int r = 0; r < LUT_GROUPS_MAX; r++) {
            const int eg = tid + WG * r;
            lo[r] = 0.0f;
            if (eg < ngroups) {                         // (r = 0: every thread when M >= 64)
                const int m = eg >> 2;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    float acc;
                    if (DSUB > 0) {
                        const float x0 = qq[m * DSUB];
                        const float a = x0 - cw[r][k][0];
                        acc = IP ? x0 * cw[r][k][0] : a * a;
#pragma unroll
                        for (int t = 1; t < CW; t++) {
                            const float xt = qq[m * DSUB + t];
                            const float b = xt - cw[r][k][t];
                            const float sq = IP ? xt * cw[r][k][t] : b * b;
                            acc = acc + sq;
                        }
                    } else {
                        const float *c = codebook + ((size_t)eg * 4 + k) * dsub;
                        const float a = qq[m * dsub] - c[0];
                        acc = IP ? qq[m * dsub] * c[0] : a * a;
                        for (int t = 1; t < dsub; t++) {
                            const float b = qq[m * dsub + t] - c[t];
                            const float sq = IP ? qq[m * dsub + t] * c[t] : b * b;
                            acc = acc + sq;
                        }
                    }
                    T[r][k] = IP ? -acc : acc;          // inner product: minus the product, smaller is better
                }
                float mn = T[r][0], mx = T[r][0];
#pragma unroll
                for (int k = 1; k < 4; k++) {
                    mn = T[r][k] < mn ? T[r][k] : mn;
                    mx = T[r][k] > mx ? T[r][k] : mx;
                }
                // over the four lanes of the sub-quantizer (a minimum and a maximum: order-free)
                float o = lane_xor1(mn); mn = o < mn ? o : mn;
                o = lane_xor2(mn); mn = o < mn ? o : mn;
                o = lane_xor1(mx); mx = o > mx ? o : mx;
                o = lane_xor2(mx); mx = o > mx ? o : mx;
                lo[r] = mn;
                const float width = mx - mn;
                span = width > span ? width : span;
                if (bias_sum && (tid & 3) == 0) sh.bias_s[m] = mn;
            }
        }
        // the largest width over the workgroup
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float o = __shfl_xor(span, off);
            span = o > span ? o : span;
        }
        float *ws = sh.wave_span[qi & 1];
        if (lane == 0) ws[wave] = span;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WG / 64; w++) span = ws[w] > span ? ws[w] : span;
        const float s = span > 0.0f ? __fdiv_rn(255.0f, span) : 0.0f;
        if (tid == 0 && scale) scale[qid] = s;
        if (tid == 64 && bias_sum) {
            // the sum of the offsets is defined in sub-quantizer order; only the stage call asks for it
            float bsum = 0.0f;
            for (int m = 0; m < M; m++) bsum = bsum + sh.bias_s[m];
            bias_sum[qid] = bsum;
        }
#pragma unroll
        for (int r = 0; r < LUT_GROUPS_MAX; r++) {
            const int eg = tid + WG * r;
            if (eg < ngroups) {
                uint32_t packed = 0;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const float x = T[r][k] - lo[r];
                    const float y = x * s;
                    float rr = rintf(y);
                    rr = rr > 255.0f ? 255.0f : rr;
                    packed |= (uint32_t)rr << (8 * k);
                }
                ((uint32_t *)(lut + (size_t)qid * M * 16))[eg] = packed;
            }
        }
        if (bias_sum) __syncthreads();                  // the offsets are rewritten by the next query
    }
}

