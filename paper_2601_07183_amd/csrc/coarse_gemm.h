// Scores of the coarse quantizer's shortlist route on the matrix cores: keys[q][l] =
// f32_key(|c'_l|^2 - 2 q'.c'_l), where q' = fl(q - cmean) and c' = fl(c - cmean) are the centred query
// and centroid, and the smallest key of every half tile (16 lists, see below) in
// hmin[q][2 * tile + half].
//
// The products run on the bf16 matrix cores at fp32's precision: a value is the exact sum of three
// bf16 pieces (8 significant bits each, rounded to nearest), and of the nine products of pieces the
// six with the larger factors are summed (v_mfma_f32_32x32x16_bf16), the leading ones apart from the
// others; what is left out is below 2^-23 |q_i||c_i|, and a sum over 128 dimensions is rounded 16
// times instead of 64.  Against the fp32 instruction (v_mfma_f32_32x32x2f32) that is 48 instructions
// of 32 cycles instead of 64 of 64 for a 32 x 32 tile at d = 128.  Measured (fp32 instruction / this):
// 10,000 queries against 16,384 x 128 centroids 530 / 358 us, 4,096 x 96 113 / 86, 1,000 against
// 1,024 x 960 90 / 38, 65,536 against 1,024 x 128 189 / 127; bound now by the operand fetch and the
// store of the keys next to the products.  Error of the scores against 64 bits over 700 queries and all
// lists (root mean square and largest, fp32 instruction / this): d = 128 1.2e-3, 2.6e-2 / 8.5e-4, 9.2e-3 at
// scores of 2e4; d = 96 2.5e-8, 3.8e-7 / 1.5e-8, 1.1e-7 at 0.4; d = 960 4.7e-9, 1.5e-7 / 2.8e-9, 3.7e-8 at
// 0.07; d = 32 5.8e-7, 6.3e-6 / 4.4e-7, 3.0e-6 at 12; of nine shapes and both metrics none is further off.
//
// A workgroup takes 128 queries, 32 per wave, whose pieces stay in registers; the lists' pieces are
// laid out at upload in operand order ([tile][step of 16 dimensions][piece][lane] 16-byte operands,
// zero beyond the last list and dimension), staged in LDS and read from there by all four waves;
// the next tile is fetched into registers while the current one is multiplied (two LDS buffers,
// one barrier per tile).  Lists are the rows of the result: lane (half k, query j) gets lists
// 8 g + 4 k + r of the tile, g and r from 0 to 3, so that the minimum of a half tile is a lane's own.
#pragma once
#include "device_util.h"

typedef float v16f __attribute__((ext_vector_type(16)));
// (clang's own vectors: arrays of HIP's vector structs ended up in scratch memory here)
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
#define GEMM_QWG 128
#define GEMM_CHUNK_KS 8             // steps of 16 dimensions whose operands a workgroup holds at a time

// the three pieces of eight values
static __device__ __forceinline__ void split_bf16x3(const float (&x)[8], v8bf (&out)[3])
{
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const __bf16 a = (__bf16)x[e];
        const float ra = x[e] - (float)a;                // exact
        const __bf16 b = (__bf16)ra;
        const float rb = ra - (float)b;                  // exact
        out[0][e] = a;
        out[1][e] = b;
        out[2][e] = (__bf16)rb;
    }
}

// Eight centred values of a row, dimensions i0 .. i0 + 7 (zero from d on; d is a multiple of 4).
static __device__ __forceinline__ void load_centred8(const float *row, const float *mean, int i0, int d, float (&x)[8])
{
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int i = i0 + 4 * h;
        const bool in = i < d;
        const v4f a = *(const v4f *)(row + (in ? i : 0)), m = *(const v4f *)(mean + (in ? i : 0));
#pragma unroll
        for (int e = 0; e < 4; e++) x[4 * h + e] = in ? a[e] - m[e] : 0.0f;
    }
}

// The lists' operands (at upload): one wave per tile and step.
__global__ __launch_bounds__(64) void pack_centroids_kernel(const float *__restrict__ cent, const float *__restrict__ cmean,
                                                            int d, int nlist, int ksteps, v4u *__restrict__ cop)
{
    const int lane = threadIdx.x, s = blockIdx.x % ksteps, tile = blockIdx.x / ksteps;
    const int l = tile * 32 + (lane & 31), i0 = 16 * s + 8 * (lane >> 5);
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const bool in = l < nlist && i0 + e < d;
        x[e] = in ? cent[(size_t)l * d + i0 + e] - cmean[i0 + e] : 0.0f;
    }
    v8bf p[3];
    split_bf16x3(x, p);
#pragma unroll
    for (int u = 0; u < 3; u++) cop[((size_t)blockIdx.x * 3 + u) * 64 + lane] = __builtin_bit_cast(v4u, p[u]);
}

int rairs_launch_pack_centroids(const float *cent, const float *cmean, int d, int nlist, void *cop, hipStream_t s)
{
    const int ksteps = (d + 15) / 16, ntiles = (nlist + 31) / 32;
    hipLaunchKernelGGL(pack_centroids_kernel, dim3((unsigned)(ksteps * ntiles)), dim3(64), 0, s, cent, cmean, d, nlist,
                       ksteps, (v4u *)cop);
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}

// A tile (or a chunk of one): six products a step, the operands of a step read from LDS while the step
// before it is multiplied (the fences keep the compiler from putting the reads in front of their use).
template <int KS>
static __device__ __forceinline__ void gemm_tile(const v4u *b, int lane, const v8bf (&A)[KS][3], v16f &hi, v16f &lo)
{
    v4u n0 = b[lane], n1 = b[64 + lane], n2 = b[128 + lane];
#pragma unroll
    for (int s = 0; s < KS; s++) {
        const v8bf b0 = __builtin_bit_cast(v8bf, n0), b1 = __builtin_bit_cast(v8bf, n1), b2 = __builtin_bit_cast(v8bf, n2);
        if (s + 1 < KS) {
            n0 = b[(s + 1) * 192 + lane];
            n1 = b[(s + 1) * 192 + 64 + lane];
            n2 = b[(s + 1) * 192 + 128 + lane];
        }
        __builtin_amdgcn_sched_barrier(0);
        lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b2, A[s][0], lo, 0, 0, 0);
        lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, A[s][1], lo, 0, 0, 0);
        lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, A[s][2], lo, 0, 0, 0);
        hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, A[s][0], hi, 0, 0, 0);
        lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, A[s][0], lo, 0, 0, 0);
        lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, A[s][1], lo, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Norms of this lane's lists of a tile (there are whole tiles of them).
static __device__ __forceinline__ void gemm_norms(const float *cnorm, int tile, int k, v4f (&c4)[4])
{
#pragma unroll
    for (int g = 0; g < 4; g++) c4[g] = *(const v4f *)(cnorm + tile * 32 + 4 * k + 8 * g);
}

// A wave's way out: a tile's keys turned so that a store instruction writes whole 128-byte lines (as
// they come, a lane's 16 bytes are a quarter line, 32 rows apart: 690 us instead of 600 for
// 10,000 queries and 16,384 lists when measured), and the half tiles' minima of up to four tiles.
#define KEY_ROW 36                  // words: 16-byte aligned rows in different banks
struct GemmOut {
    uint32_t key[32][KEY_ROW];
    uint32_t least[32][12];         // [query][2 * (tile - first tile of the four) + half]
};

// Keys of one tile of this wave's 32 queries (from row q0 of the key matrix on).  alpha = 2:
// |c'|^2 - 2 q'.c'; alpha = 1 with zero norms: -q.c.
static __device__ __forceinline__ void gemm_keys(const v16f &hi, const v16f &lo, const v4f (&c4)[4], int tile, int lane,
                                                 int nlist, int64_t q0, int64_t nq, uint32_t *keys, float alpha,
                                                 GemmOut &out, int of_four)
{
    const int j = lane & 31, k = lane >> 5, l0 = tile * 32 + 4 * k;
    const bool part = tile * 32 + 32 > nlist;            // uniform: the last tile
    uint32_t least = 0xFFFFFFFFu;
#pragma unroll
    for (int g = 0; g < 4; g++) {
        const float cn[4] = {c4[g].x, c4[g].y, c4[g].z, c4[g].w};
        uint32_t key[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float dot = hi[4 * g + r] + lo[4 * g + r];
            key[r] = f32_key(cn[r] - alpha * dot);
            if (part && l0 + 8 * g + r >= nlist) key[r] = 0xFFFFFFFFu;
            least = key[r] < least ? key[r] : least;
        }
        *(v4u *)&out.key[j][8 * g + 4 * k] = (v4u){key[0], key[1], key[2], key[3]};
    }
    out.least[j][2 * of_four + k] = least;
    wave_lds_sync();
    const int n = nq - q0 < 32 ? (int)(nq - q0) : 32;    // rows that are queries (uniform; none: <= 0)
    uint32_t *first = keys + (size_t)q0 * nlist + tile * 32;
    if ((nlist & 3) == 0) {                              // uniform: rows are 16-byte aligned, four lists exist or none
        const int row = lane >> 3, col = 4 * (lane & 7);
        const int rows = !part || tile * 32 + col < nlist ? n : 0;
        const uint32_t off = (uint32_t)row * (uint32_t)nlist + (uint32_t)col;        // (one 32-bit offset from uniform rows)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const v4u x = *(const v4u *)&out.key[row + 8 * i][col];
            uint32_t *rowp = first + (size_t)(8 * i) * nlist;
            if (row + 8 * i < rows) *(v4u *)(rowp + off) = x;
        }
    } else {
#pragma unroll 1
        for (int i = k; i < n; i += 2)
            if (tile * 32 + j < nlist) first[(size_t)i * nlist + j] = out.key[i][j];
    }
    wave_lds_sync();                                     // (the region is the next tile's)
}

// The minima of tiles t0 .. t0 + n - 1, n <= 4.
static __device__ __forceinline__ void gemm_minima(const GemmOut &out, int t0, int n, int lane, int64_t q0, int64_t nq,
                                                   uint32_t *hmin, int nhalf)
{
    const int j = lane & 31, k = lane >> 5;
    if (!hmin || q0 + j >= nq) return;
    uint32_t *dst = hmin + (size_t)(q0 + j) * nhalf + 2 * t0 + 4 * k;
    if (n == 4 && (nhalf & 3) == 0 && (t0 & 1) == 0)     // uniform
        *(v4u *)dst = *(const v4u *)&out.least[j][4 * k];
    else
#pragma unroll
        for (int e = 0; e < 4; e++)
            if (4 * k + e < 2 * n) dst[e] = out.least[j][4 * k + e];
}

template <int KS>                                       // steps of 16 dimensions, at least the row's
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(KS <= 4 ? 4 : KS <= 6 ? 3 : 2))) void coarse_gemm_kernel(const float *__restrict__ q, const v4u *__restrict__ cop,
                                                         const float *__restrict__ cmean,
                                                         const float *__restrict__ cnorm, int d, int nlist, int ksteps,
                                                         int csplits, int tiles_per_split, int64_t nq,
                                                         uint32_t *__restrict__ keys, uint32_t *__restrict__ hmin,
                                                         float alpha)
{
    constexpr int OPS = KS * 3 * 64, PER = (OPS + WG - 1) / WG;
    __shared__ v4u Bs[2][PER * WG];
    __shared__ __align__(16) GemmOut out_s[WG / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 31, k = lane >> 5;
    // workgroups that share an L2 (consecutive ids go round the 8 dies) take the same lists
    int qblock, csplit;
    if ((csplits & 7) == 0) {
        const int per = csplits >> 3, x = blockIdx.x & 7, y = blockIdx.x >> 3;
        csplit = x * per + y % per;
        qblock = y / per;
    } else {
        csplit = blockIdx.x % csplits;
        qblock = blockIdx.x / csplits;
    }
    const int ntiles = (nlist + 31) >> 5;
    const int t_begin = csplit * tiles_per_split;
    const int t_end = t_begin + tiles_per_split < ntiles ? t_begin + tiles_per_split : ntiles;
    if (t_begin >= t_end) return;                       // uniform for the workgroup
    v4u st[PER];
    const int tile_ops = ksteps * 192;                  // (steps of KS beyond the row multiply zeros of the query)
    auto fetch = [&](int t) {
        const v4u *src = cop + (size_t)t * tile_ops;
#pragma unroll
        for (int e = 0; e < PER; e++) {
            const int i = threadIdx.x + WG * e;
            st[e] = src[i < tile_ops ? i : 0];
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int e = 0; e < PER; e++) Bs[buf][threadIdx.x + WG * e] = st[e];
    };
    fetch(t_begin);
    const int64_t q0 = (int64_t)qblock * GEMM_QWG + wave * 32, qj = q0 + j;
    const float *qrow = q + (size_t)(qj < nq ? qj : nq - 1) * d;
    v8bf A[KS][3];
#pragma unroll
    for (int s = 0; s < KS; s++) {
        float x[8];
        load_centred8(qrow, cmean, 16 * s + 8 * k, d, x);
        split_bf16x3(x, A[s]);
    }
    stage(0);
    __syncthreads();
    int buf = 0;
    const int nhalf = 2 * ntiles;
    for (int t = t_begin; t < t_end; t++) {
        const bool more = t + 1 < t_end;
        fetch(more ? t + 1 : t);
        v4f c4[4];
        gemm_norms(cnorm, t, k, c4);
        v16f hi, lo;
#pragma unroll
        for (int r = 0; r < 16; r++) hi[r] = lo[r] = 0.0f;
        gemm_tile<KS>(Bs[buf], lane, A, hi, lo);
        // (staged ahead of the keys' stores: the wait for the operands would be one for the stores too,
        // 250 us instead of 237 for 65,536 queries and 1,024 lists)
        stage(buf ^ 1);
        const int of_four = (t - t_begin) & 3;
        gemm_keys(hi, lo, c4, t, lane, nlist, q0, nq, keys, alpha, out_s[wave], of_four);
        if (of_four == 3 || !more) {
            gemm_minima(out_s[wave], t - of_four, of_four + 1, lane, q0, nq, hmin, nhalf);
            wave_lds_sync();
        }
        __syncthreads();
        buf ^= 1;
    }
}

// The same scores for longer rows: the dimensions are taken in chunks of 16 * GEMM_CHUNK_KS, and the
// NT tiles of the workgroup keep their accumulators across the chunks.
template <int NT>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2))) void coarse_gemm_chunk_kernel(const float *__restrict__ q,
                                                               const v4u *__restrict__ cop,
                                                               const float *__restrict__ cmean,
                                                               const float *__restrict__ cnorm, int d,
                                                               int nlist, int ksteps, int ngroups, int64_t nq,
                                                               uint32_t *__restrict__ keys,
                                                               uint32_t *__restrict__ hmin, float alpha)
{
    constexpr int KS = GEMM_CHUNK_KS, OPS = KS * 192, PER = OPS / WG;
    __shared__ v4u Bs[2][OPS];
    __shared__ __align__(16) GemmOut out_s[WG / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 31, k = lane >> 5;
    const int qblock = blockIdx.x / ngroups, grp = blockIdx.x % ngroups;
    const int64_t q0 = (int64_t)qblock * GEMM_QWG + wave * 32, qj = q0 + j;
    const float *qrow = q + (size_t)(qj < nq ? qj : nq - 1) * d;
    const int ntiles = (nlist + 31) >> 5, nchunks = (ksteps + KS - 1) / KS;
    const int nt = ntiles - grp * NT < NT ? ntiles - grp * NT : NT;          // this workgroup's tiles
    v16f hi[NT], lo[NT];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int r = 0; r < 16; r++) hi[t][r] = lo[t][r] = 0.0f;
    v4u st[PER];
    auto fetch = [&](int c, int t) {
        const int s0 = c * KS, n = (ksteps - s0 < KS ? ksteps - s0 : KS) * 192;
        const v4u *src = cop + ((size_t)(grp * NT + t) * ksteps + s0) * 192;
#pragma unroll
        for (int e = 0; e < PER; e++) {
            const int i = threadIdx.x + WG * e;
            st[e] = src[i < n ? i : 0];                 // (beyond the row: multiplied by zeros of the query)
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int e = 0; e < PER; e++) Bs[buf][threadIdx.x + WG * e] = st[e];
    };
    fetch(0, 0);
    int buf = 0;
    for (int c = 0; c < nchunks; c++) {
        v8bf A[KS][3];
#pragma unroll
        for (int s = 0; s < KS; s++) {
            float x[8];
            load_centred8(qrow, cmean, 16 * (c * KS + s) + 8 * k, d, x);
            split_bf16x3(x, A[s]);
        }
#pragma unroll
        for (int t = 0; t < NT; t++) {
            if (t < nt) {                               // uniform for the workgroup
                // (the buffer's last readers are behind the barrier of the other one)
                stage(buf);
                __syncthreads();
                const bool next_c = t + 1 >= nt;
                fetch(next_c && c + 1 < nchunks ? c + 1 : c, next_c ? 0 : t + 1);
                gemm_tile<KS>(Bs[buf], lane, A, hi[t], lo[t]);
                buf ^= 1;
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NT; t++)
        if (t < nt) {
            v4f c4[4];
            gemm_norms(cnorm, grp * NT + t, k, c4);
            gemm_keys(hi[t], lo[t], c4, grp * NT + t, lane, nlist, q0, nq, keys, alpha, out_s[wave], t);
        }
    gemm_minima(out_s[wave], grp * NT, nt, lane, q0, nq, hmin, 2 * ntiles);
}
