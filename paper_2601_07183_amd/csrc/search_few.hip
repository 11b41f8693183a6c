// RairsSearch (Alg. 2) for small batches: one query, a handful, some hundreds over many lists.  The
// list-major path of scan_mfma.hip fills the 32 columns of a matrix tile with queries that probe
// the same list and needs some fifteen kernels to set that up; with a few queries per list most
// columns are empty and the set-up is the cost.  Here every query keeps its own workgroups and
// the whole search is four kernels (the rule that chooses is few_pays in api.hip):
//
//   front:  distances of all (query, list) pairs in the direct form, and the lookup tables;
//   probe:  per query the nprobe smallest, the probe bitmap, the blocks of its lists (reference cells
//           of probed owners left out), and a bound: the bigK-th smallest score of a sample of its
//           nearest lists;
//   scan:   scores by table lookups in LDS, several workgroups per query; items at or below the
//           bound that the duplicate rule keeps are collected per workgroup, cut to the bigK best
//           whenever they fill the workgroup's buffer, so no query can overflow;
//   finish: the bigK best (score, id) of a query's workgroups, their exact distances, the K best.
//
// The results are those of the list-major path bit for bit: the coarse distances are the defining
// direct form itself (no shortlist needed), the scores are integers, and selections are by the
// total orders (distance, list id), (score, id), (distance, id).  Nothing here is shared between
// queries, so there are no global atomics and nothing has to be cleared beforehand.
//
// What bounds it: for one query the chain of launches, barriers and memory round trips (1M x 128
// index, nprobe 23: 4 + 12 + 5 + 9 us of kernels, 30 to 35 us a search; 147 us list-major), for a
// hundred the scan's lookups -- 1.9 vector instructions and one two-cycle LDS read each, 7 to 8 *
// 10^12 lookups/s on the chip (100 queries at nprobe 32: 386 -> 115 us).
#include "device_util.h"
#include "lut_build.h"

// ---- selection in a workgroup -------------------------------------------------------------------

#define PICK_BINS 1024
struct PickShared {
    uint32_t hist[3][PICK_BINS];
};
template <int NT>
static __device__ __forceinline__ void pick_clear(PickShared &sh)
{
    for (int i = threadIdx.x; i < 3 * PICK_BINS; i += NT) sh.hist[0][i] = 0u;
}

// A threshold t such that at least k and at most `most` of the workgroup's values are <= t, given
// that at least k exist, all distinct, in [lo, hi].  each(f) calls f(value) for every value that the
// thread holds (values outside the range are ignored).  One histogram of PICK_BINS equal bins over
// [lo, hi] finds the bin of the k-th smallest; as long as the bins up to there hold more than
// `most`, the range narrows to that bin.  Bins end up one value wide, so this always ends.
// The time of this kernel family is barriers and round trips, so a round has one barrier: three
// histograms take turns (`turn`, kept by the caller from call to call; all clear at the start) --
// behind the barrier of a round everybody has read the previous one, which is cleared for the
// round after the next -- and every wave derives the bin by itself.  Bin b sits at word
// (b % 16) * 64 + b / 16: a lane sums 16 consecutive bins without bank conflicts.
template <int NT, typename Each>
static __device__ __forceinline__ uint64_t wg_pick(Each each, uint32_t k, uint32_t most, uint64_t lo, uint64_t hi,
                                                   PickShared &sh, int &turn)
{
    static_assert(PICK_BINS == 16 * 64, "sixteen bins per lane");
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t base = 0;                                   // values below lo
    for (;;) {
        const uint64_t range = hi - lo;
        const int bits = range ? 64 - __clzll((long long)range) : 0;
        const int shift = bits > 10 ? bits - 10 : 0;
        uint32_t *hist = sh.hist[turn], *old = sh.hist[turn == 0 ? 2 : turn - 1];
        turn = turn == 2 ? 0 : turn + 1;
        each([&](uint64_t x) {
            if (x >= lo && x <= hi) {
                const uint32_t b = (uint32_t)((x - lo) >> shift);
                atomicAdd(&hist[(b & 15u) * 64u + (b >> 4)], 1u);
            }
        });
        __syncthreads();
        for (int i = tid; i < PICK_BINS; i += NT) old[i] = 0u;
        uint32_t h[16], mine = 0;
#pragma unroll
        for (int u = 0; u < 16; u++) { h[u] = hist[u * 64 + lane]; mine += h[u]; }
        const uint32_t incl = wave_incl_sum_u32(mine);
        uint32_t cum = base + incl - mine, bin = 0, upto = 0, before = 0;
        const bool here = cum < k && cum + mine >= k;    // one lane
#pragma unroll
        for (int u = 0; u < 16; u++) {
            if (cum < k && cum + h[u] >= k) { bin = 16u * (uint32_t)lane + u; upto = cum + h[u]; before = cum; }
            cum += h[u];
        }
        const unsigned long long who = __ballot(here);
        const int src = who ? __ffsll((long long)who) - 1 : 63;
        const uint64_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, src);
        upto = (uint32_t)__builtin_amdgcn_readlane((int)upto, src);
        before = (uint32_t)__builtin_amdgcn_readlane((int)before, src);
        const uint64_t last = lo + ((b0 + 1) << shift) - 1ull;
        if (upto <= most || shift == 0) return last < hi ? last : hi;
        base = before;
        lo = lo + (b0 << shift);
        hi = last < hi ? last : hi;
    }
}

// Places of m <= NT distinct values in ascending order: use(i, place) is called once for every value
// i, by one thread.  A value's place is the number of smaller ones; up to 16 neighbouring threads
// share the counting.
template <int NT, typename Use>
static __device__ __forceinline__ void wg_rank(const uint64_t *x, int m, Use use)
{
    int sh = 0;                                          // log2 of the threads per value
    while (sh < 4 && (m << (sh + 1)) <= NT) sh++;
    const int i = (int)threadIdx.x >> sh, sub = (int)threadIdx.x & ((1 << sh) - 1);
    const uint64_t mine = i < m ? x[i] : 0ull;
    int place = 0;
#pragma unroll 4
    for (int j = sub; j < m; j += 1 << sh) place += x[j] < mine ? 1 : 0;
    for (int off = 1; off < (1 << sh); off <<= 1) place += __shfl_xor(place, off);
    if (i < m && sub == 0) use(mine, place);
}

// ---- front: direct-form distances and lookup tables --------------------------------------------

// The first nq workgroups build one query's tables each; the others take Q queries x 16 LS lists.
// A group of 16 lanes takes LS lists: lane l sums the dimensions of the classes l, l + 16, l + 32,
// l + 48 (mod 64), so the strides 32 and 16 of the defined butterfly are sums inside the lane and
// only strides 8 to 1 cross lanes (the re-scoring arithmetic of the coarse shortlist).
template <bool IP, int DSUB, int Q, int LS>
__global__ __launch_bounds__(WG) void few_front_kernel(IndexView v, FewArgs a, int list_groups)
{
    __shared__ LutShared lsh;
    if ((int64_t)blockIdx.x < a.nq) {
        lut_build_wg<IP, DSUB>(a.q, v.codebook, v.d, v.M, a.nq, blockIdx.x, 1, a.lut, nullptr, nullptr, lsh);
        return;
    }
    const uint32_t b = blockIdx.x - (uint32_t)a.nq;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, l16 = lane & 15;
    const int64_t q0 = (int64_t)(b / list_groups) * Q;
    const int l0 = (int)(b % list_groups) * 16 * LS + wave * 4 * LS + grp;    // this group's lists: l0 + 4 u
    const int d = v.d;
    const float *qr[Q];
    const float *cr[LS];
    float p[Q][LS][4];
#pragma unroll
    for (int j = 0; j < Q; j++) qr[j] = a.q + (size_t)(q0 + j < a.nq ? q0 + j : a.nq - 1) * d;
#pragma unroll
    for (int u = 0; u < LS; u++) {
        const int l = l0 + 4 * u;
        cr[u] = v.centroids + (size_t)(l < v.nlist ? l : v.nlist - 1) * d;
    }
#pragma unroll
    for (int j = 0; j < Q; j++)
#pragma unroll
        for (int u = 0; u < LS; u++)
#pragma unroll
            for (int cc = 0; cc < 4; cc++) p[j][u][cc] = 0.0f;
    int i0 = 0;
#pragma unroll 2
    for (; i0 + 64 <= d; i0 += 64) {                     // whole rounds of 64 dimensions
        float x[LS][4], y[Q][4];
#pragma unroll
        for (int cc = 0; cc < 4; cc++) {
#pragma unroll
            for (int u = 0; u < LS; u++) x[u][cc] = cr[u][i0 + l16 + 16 * cc];
#pragma unroll
            for (int j = 0; j < Q; j++) y[j][cc] = qr[j][i0 + l16 + 16 * cc];
        }
#pragma unroll
        for (int j = 0; j < Q; j++)
#pragma unroll
            for (int u = 0; u < LS; u++)
#pragma unroll
                for (int cc = 0; cc < 4; cc++) {
                    float sq;
                    if (IP) sq = y[j][cc] * x[u][cc];
                    else { const float diff = y[j][cc] - x[u][cc]; sq = diff * diff; }
                    p[j][u][cc] = p[j][u][cc] + sq;
                }
    }
    if (i0 < d) {                                        // the last, partial round
#pragma unroll
        for (int cc = 0; cc < 4; cc++) {
            const int i = i0 + l16 + 16 * cc;
            if (i < d) {
#pragma unroll
                for (int u = 0; u < LS; u++) {
                    const float x = cr[u][i];
#pragma unroll
                    for (int j = 0; j < Q; j++) {
                        const float y = qr[j][i];
                        float sq;
                        if (IP) sq = y * x;
                        else { const float diff = y - x; sq = diff * diff; }
                        p[j][u][cc] = p[j][u][cc] + sq;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < Q; j++)
#pragma unroll
        for (int u = 0; u < LS; u++) {
            const float s02 = p[j][u][0] + p[j][u][2], s13 = p[j][u][1] + p[j][u][3];    // stride 32
            float t = s02 + s13;                         // stride 16
            t = t + lane_xor8(t);
            t = t + lane_xor4(t);
            t = t + lane_xor2(t);
            t = t + lane_xor1(t);
            const int l = l0 + 4 * u;
            if (l16 == 0 && l < v.nlist && q0 + j < a.nq)
                a.keys[(size_t)(q0 + j) * v.nlist + l] = f32_key(IP ? -t : t);
        }
}

// ---- scores by table lookups -------------------------------------------------------------------

// Tables of one query in LDS: the M * 16 bytes as they are (sub-quantizer m at 16 m), zero up to the
// nd * 256 bytes that whole code dwords address.
template <int NT>
static __device__ __forceinline__ void few_load_tables(const IndexView &v, const uint8_t *lut, uint8_t *lq)
{
    const uint4 *src = (const uint4 *)lut;
    uint4 *dst = (uint4 *)lq;
    for (int i = threadIdx.x; i < v.nd * 16; i += NT) dst[i] = i < v.M ? src[i] : make_uint4(0, 0, 0, 0);
}

// Eight lookups of one code dword: nibble t of the lane's parity g addresses byte 32 t + 16 g +
// code.  The nibbles are first spread to bytes that already carry the 16 g.
static __device__ __forceinline__ uint32_t few_lookup8(const uint8_t *lq, uint32_t c, uint32_t gm)
{
    // (as instructions: the compiler otherwise merges the mask into the byte selections, which
    // takes a third more of them; the loop is bound by vector instruction issue)
    uint32_t e, o = c >> 4;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(e) : "v"(c), "s"(0x0F0F0F0Fu), "v"(gm));
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(o) : "v"(o), "s"(0x0F0F0F0Fu), "v"(gm));
    uint32_t s = 0;
#pragma unroll
    for (int n = 0; n < 4; n++) {
        s += lq[64 * n + ((e >> (8 * n)) & 255u)];
        s += lq[64 * n + 32 + ((o >> (8 * n)) & 255u)];
    }
    return s;
}

// Scores of NB blocks, NB even: lane (half h, item i) gets in out[p] the score of item i of block
// 2 p + h.  blk: the blocks (wave-uniform).  ND: code dwords per block and lane when at most four
// (fetch requests them all), 0: any number, four at a time and four ahead.
template <int ND, int NB>
struct FewCodes {
    static constexpr int NDS = ND > 0 ? ND : 4;
    uint32_t c[NB][NDS];
    __device__ __forceinline__ void fetch(const IndexView &v, const int32_t (&blk)[NB], int lane)
    {
        const int nd = ND > 0 ? ND : v.nd;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const uint32_t *cp = v.codes + (size_t)blk[b] * (nd * 64);       // uniform
#pragma unroll
            for (int w = 0; w < NDS; w++) c[b][w] = cp[(ND > 0 || w < nd ? w : nd - 1) * 64 + lane];
        }
    }
    __device__ __forceinline__ void scores(const IndexView &v, const uint8_t *lq, const int32_t (&blk)[NB], int lane,
                                           uint32_t (&out)[NB / 2])
    {
        const uint32_t gm = lane >= 32 ? 0x10101010u : 0u;
        uint32_t part[NB];
#pragma unroll
        for (int b = 0; b < NB; b++) part[b] = 0;
        if (ND > 0) {
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int w = 0; w < NDS; w++) part[b] += few_lookup8(lq + 256 * w, c[b][w], gm);
        } else {
            const int nd = v.nd;
            for (int w0 = 0; w0 < nd; w0 += 4) {
                uint32_t x[NB][NDS];
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    const uint32_t *cp = v.codes + (size_t)blk[b] * (nd * 64);
#pragma unroll
                    for (int w = 0; w < NDS; w++) {
                        x[b][w] = c[b][w];
                        c[b][w] = cp[(w0 + 4 + w < nd ? w0 + 4 + w : nd - 1) * 64 + lane];
                    }
                }
#pragma unroll
                for (int w = 0; w < NDS; w++)
                    if (w0 + w < nd) {                   // uniform
#pragma unroll
                        for (int b = 0; b < NB; b++) part[b] += few_lookup8(lq + 256 * (w0 + w), x[b][w], gm);
                    }
            }
        }
        // the two halves of the wave hold the two parities of the sub-quantizers: after the swap of
        // one register's upper with the other's lower half both addends of an item are in one lane
#pragma unroll
        for (int p = 0; p < NB / 2; p++) {
            uint32_t x = part[2 * p], y = part[2 * p + 1];
            asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
            out[p] = x + y;
        }
    }
};

// ---- probe: lists, units and bound of a query --------------------------------------------------

#define PROBE_NT 1024
#define PROBE_WAVES (PROBE_NT / 64)
#define PROBE_MOST (FEW_MAX_NPROBE + 64)
#define SAMPLE_NB 4                                      // sample blocks that a wave takes at a time
struct ProbeShared {
    uint8_t lq[RAIRS_MAX_M * 16];                        // first: at address zero a lookup needs no base added
    PickShared pick;
    uint64_t sel[PROBE_MOST];
    int32_t list[FEW_MAX_NPROBE], blk_begin[FEW_MAX_NPROBE], seg_begin[FEW_MAX_NPROBE];
    uint32_t segpre[FEW_MAX_NPROBE + 1], ownpre[FEW_MAX_NPROBE + 1];
    uint32_t bm[FEW_MAX_NLIST / 32];
    uint16_t sc[RAIRS_SAMPLE_MAX_BLOCKS * 32];
    uint32_t cnt, blocks, valid, smin, smax, lo[PROBE_WAVES], hi[PROBE_WAVES];
};
template <int KPT, int ND>                               // list keys per thread; code dwords (0: any)
__global__ __launch_bounds__(PROBE_NT) void few_probe_kernel(IndexView v, FewArgs a)
{
    __shared__ __align__(16) ProbeShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t qi = blockIdx.x;
    const int nlist = v.nlist, nprobe = a.nprobe;
    const uint32_t *row = a.keys + (size_t)qi * nlist;

    // the nprobe smallest (key, list id)
    uint32_t key[KPT];
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int u = 0; u < KPT; u++) {
        const int l = tid + PROBE_NT * u;
        key[u] = row[l < nlist ? l : nlist - 1];
    }
    few_load_tables<PROBE_NT>(v, a.lut + (size_t)qi * v.M * 16, sh.lq);
    for (int i = tid; i < a.bmwords; i += PROBE_NT) sh.bm[i] = 0u;
    pick_clear<PROBE_NT>(sh.pick);
    int turn = 0;
#pragma unroll
    for (int u = 0; u < KPT; u++) {
        kmin = key[u] < kmin ? key[u] : kmin;
        kmax = key[u] > kmax ? key[u] : kmax;
    }
    wave_min_max_u32(kmin, kmax);
    if (lane == 0) { sh.lo[wave] = kmin; sh.hi[wave] = kmax; }
    if (tid == 0) { sh.cnt = 0; sh.blocks = 0; sh.valid = 0; sh.smin = 0xFFFFu; sh.smax = 0u; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < PROBE_WAVES; w++) {
        kmin = sh.lo[w] < kmin ? sh.lo[w] : kmin;
        kmax = sh.hi[w] > kmax ? sh.hi[w] : kmax;
    }
    auto each_key = [&](auto f) {
#pragma unroll
        for (int u = 0; u < KPT; u++) {
            const int l = tid + PROBE_NT * u;
            if (l < nlist) f(((uint64_t)key[u] << 16) | (uint32_t)l);
        }
    };
    const uint64_t thr = wg_pick<PROBE_NT>(each_key, (uint32_t)nprobe, (uint32_t)nprobe + 64u, (uint64_t)kmin << 16,
                                           ((uint64_t)kmax << 16) | 0xFFFFu, sh.pick, turn);
    each_key([&](uint64_t x) {
        if (x <= thr) sh.sel[atomicAdd(&sh.cnt, 1u)] = x;    // at most nprobe + 64
    });
    __syncthreads();
    wg_rank<PROBE_NT>(sh.sel, (int)sh.cnt, [&](uint64_t x, int place) {
        if (place < nprobe) {
            const int l = (int)(x & 0xFFFFu);
            sh.list[place] = l;
            atomicOr(&sh.bm[l >> 5], 1u << (l & 31));
        }
    });
    __syncthreads();

    // segments and own blocks of the probed lists, numbered through (two prefixes side by side)
    uint32_t nseg, nown;
    {
        uint32_t x = 0, y = 0;
        if (tid < nprobe) {
            const ListEntry le = v.lists[sh.list[tid]];
            x = (uint32_t)le.seg_cnt;
            y = (uint32_t)(le.shared_cnt + le.misc_cnt);
            sh.blk_begin[tid] = le.blk_begin;
            sh.seg_begin[tid] = le.seg_begin;
        }
        for (int i = tid; i < a.bmwords; i += PROBE_NT) a.bitmap[(size_t)qi * a.bmwords + i] = sh.bm[i];
        const uint32_t xi = wave_incl_sum_u32(x), yi = wave_incl_sum_u32(y);
        if (lane == 63) { sh.lo[wave] = xi; sh.hi[wave] = yi; }
        __syncthreads();
        uint32_t xb = 0, yb = 0;
        nseg = nown = 0;
#pragma unroll
        for (int w = 0; w < FEW_MAX_NPROBE / 64; w++) {  // only these waves hold lists
            const uint32_t p = sh.lo[w], q = sh.hi[w];
            if (w < wave) { xb += p; yb += q; }
            nseg += p;
            nown += q;
        }
        if (tid < nprobe) { sh.segpre[tid] = xb + xi - x; sh.ownpre[tid] = yb + yi - y; }
    }
    __syncthreads();
    // the last list whose prefix is <= x (lists without entries share their successor's prefix)
    auto list_of = [&](const uint32_t *pre, uint32_t x) {
        int lo = 0, hi = nprobe - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pre[mid] <= x) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    // The bound: bigK-th smallest score over the first own blocks of the nearest lists.  Every item
    // counted is one that the duplicate rule keeps, so it is an entry of the query's candidate
    // queue and no two are the same vector.  A wave takes consecutive blocks, SAMPLE_NB at a time;
    // the first ones are requested here and scored behind the block list, whose own round trips
    // run meanwhile.
    const uint32_t ns = nown < (uint32_t)a.sample_blocks ? nown : (uint32_t)a.sample_blocks;
    const uint32_t per = (ns + PROBE_WAVES - 1) / PROBE_WAVES;
    const uint32_t s1 = ((uint32_t)wave + 1u) * per < ns ? ((uint32_t)wave + 1u) * per : ns;
    uint32_t s0 = (uint32_t)wave * per;
    const int h = lane >> 5, i32 = lane & 31, hm = -h;
    int32_t blk[SAMPLE_NB];
    int Lb[SAMPLE_NB];
    uint2 it[SAMPLE_NB / 2];
    FewCodes<ND, SAMPLE_NB> codes;
    int sp = 0;                                          // the list of the next block
    // (by bits: an array indexed per lane would go through memory)
#define SAMPLE_HALF(x_) ((x_)[b] ^ (((x_)[b] ^ (x_)[b + 1]) & hm))
    auto fetch_sample = [&]() {
#pragma unroll
        for (int b = 0; b < SAMPLE_NB; b++) {
            const uint32_t s = s0 + b < s1 ? s0 + b : s1 - 1;
            while (sp + 1 < nprobe && sh.ownpre[sp + 1] <= s) sp++;          // uniform
            Lb[b] = __builtin_amdgcn_readfirstlane(sh.list[sp]);
            blk[b] = __builtin_amdgcn_readfirstlane(sh.blk_begin[sp] + (int)(s - sh.ownpre[sp]));
        }
#pragma unroll
        for (int b = 0; b < SAMPLE_NB; b += 2) it[b / 2] = v.idtag[(size_t)SAMPLE_HALF(blk) * 32 + i32];
        codes.fetch(v, blk, lane);
    };
    if (s0 < s1) {                                       // uniform for the wave
        sp = __builtin_amdgcn_readfirstlane(list_of(sh.ownpre, s0));
        fetch_sample();
    }
    // the blocks to score, in no particular order
    int32_t *blocks = a.blocks + (size_t)qi * a.max_blocks;
    for (uint32_t i0 = 0; i0 < nseg; i0 += PROBE_NT) {   // (a wave-wide prefix and one LDS atomic per wave)
        const uint32_t i = i0 + (uint32_t)tid;
        int first = 0, n = 0;
        if (i < nseg) {
            const int p = list_of(sh.segpre, i);
            const SegEntry se = v.segs[sh.seg_begin[p] + (int)(i - sh.segpre[p])];
            first = se.blk_begin;
            n = se.nblk;
            if (se.owner >= 0 && ((sh.bm[se.owner >> 5] >> (se.owner & 31)) & 1u)) n = 0;     // scored through its owner
        }
        const uint32_t incl = wave_incl_sum_u32((uint32_t)n);
        uint32_t at = 0;
        if (lane == 63) at = atomicAdd(&sh.blocks, incl);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - (uint32_t)n;
        if (at + (uint32_t)n <= (uint32_t)a.max_blocks)
            for (int b = 0; b < n; b++) blocks[at + b] = first + b;
    }
    {
        uint32_t valid_n = 0, smin = 0xFFFFu, smax = 0u;
        const bool any = s0 < s1;
        while (s0 < s1) {
            uint32_t out[SAMPLE_NB / 2];
            codes.scores(v, sh.lq, blk, lane, out);
#pragma unroll
            for (int b = 0; b < SAMPLE_NB; b += 2) {
                const uint32_t s = s0 + b + h;
                const int o = (int)it[b / 2].y, L = SAMPLE_HALF(Lb);
                bool keep = s < s1 && it[b / 2].x != RAIRS_EMPTY_ID;
                if (keep && o >= 0 && o < L && ((sh.bm[o >> 5] >> (o & 31)) & 1u)) keep = false;
                if (s < s1) sh.sc[s * 32 + i32] = keep ? (uint16_t)out[b / 2] : (uint16_t)0xFFFFu;
                valid_n += (uint32_t)__popcll(__ballot(keep));
                if (keep) {
                    smin = out[b / 2] < smin ? out[b / 2] : smin;
                    smax = out[b / 2] > smax ? out[b / 2] : smax;
                }
            }
            s0 += SAMPLE_NB;
            if (s0 < s1) fetch_sample();
        }
#undef SAMPLE_HALF
        wave_min_max_u32(smin, smax);
        if (any && lane == 0) { atomicMin(&sh.smin, smin); atomicMax(&sh.smax, smax); atomicAdd(&sh.valid, valid_n); }
    }
    __syncthreads();
    uint32_t bound = 0xFFFFu;
    if (sh.valid >= (uint32_t)a.refine_k) {              // uniform
        auto each_score = [&](auto f) {
            for (uint32_t e = (uint32_t)tid; e < ns * 32u; e += PROBE_NT) {
                const uint32_t x = sh.sc[e];
                if (x != 0xFFFFu) f(((uint64_t)x << 16) | e);
            }
        };
        // (a bound a few entries looser than the exact one is as good: up to an eighth more)
        bound = (uint32_t)(wg_pick<PROBE_NT>(each_score, (uint32_t)a.refine_k, (uint32_t)a.refine_k + (uint32_t)a.refine_k / 8u,
                                             (uint64_t)sh.smin << 16, ((uint64_t)sh.smax << 16) | 0xFFFFu, sh.pick, turn) >> 16);
    }
    if (tid == 0) {
        a.bound[qi] = (int32_t)bound;
        a.nblocks[qi] = sh.blocks < (uint32_t)a.max_blocks ? sh.blocks : (uint32_t)a.max_blocks;
    }
}

// ---- scan ----------------------------------------------------------------------------------------

#define FEW_ROUND (4 * (WG / 64) * 32)                   // most items that a workgroup adds between two looks at its buffer
static_assert(FEW_CAP >= RAIRS_MAX_REFINE_K + FEW_ROUND, "the bigK best and one round's items fit the buffer");

template <int ND>
struct FewScanShared {
    uint8_t lq[(ND > 0 ? ND : RAIRS_MAX_M / 16) * 256];  // first: at address zero a lookup needs no base added
    uint64_t buf[FEW_CAP];
    uint64_t tau;
    uint32_t cnt, items;
};
template <int ND>
__global__ __launch_bounds__(WG) void few_scan_kernel(IndexView v, FewArgs a)
{
    __shared__ __align__(16) FewScanShared<ND> sh;
    uint64_t *buf = sh.buf;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t qi = blockIdx.y;
    const uint32_t nb = a.nblocks[qi];
    const int32_t *blocks = a.blocks + (size_t)qi * a.max_blocks;            // 16-byte aligned
    const uint32_t *bmq = a.bitmap + (size_t)qi * a.bmwords;
    // a wave takes four blocks at a time
    uint32_t u = 4u * (blockIdx.x * (WG / 64) + (uint32_t)__builtin_amdgcn_readfirstlane(wave));
    const uint32_t step = 4u * gridDim.x * (WG / 64);
    int4 be = *(const int4 *)(blocks + (u < nb ? u : 0u));
    few_load_tables<WG>(v, a.lut + (size_t)qi * v.M * 16, sh.lq);
    if (tid == 0) {
        sh.tau = ((uint64_t)(uint32_t)a.bound[qi] << 32) | 0xFFFFFFFFull;
        sh.cnt = 0;
        sh.items = 0;
    }
    __syncthreads();
    // keep the bigK best of the n entries (all threads together)
    auto cut = [&](uint32_t n) {
        const int n2 = next_pow2((int)n);
        for (int e = (int)n + tid; e < n2; e += WG) buf[e] = ~0ull;
        __syncthreads();
        bitonic_sort_lds(buf, n2);
        if (tid == 0 && n >= (uint32_t)a.refine_k) {
            sh.cnt = (uint32_t)a.refine_k;
            sh.tau = buf[a.refine_k - 1];
        }
        __syncthreads();
    };
    uint32_t items = 0;
    for (uint32_t u0 = 4u * blockIdx.x * (WG / 64); u0 < nb; u0 += step) {   // uniform for the workgroup
        const uint64_t tau = sh.tau;
        if (u < nb) {
            int32_t blk[4] = {be.x, be.y, be.z, be.w};
            uint32_t vm[4];
#pragma unroll
            for (int b = 0; b < 4; b++) {
                const bool in = u + b < nb;
                blk[b] = __builtin_amdgcn_readfirstlane(in ? blk[b] : blk[0]);
                vm[b] = in ? v.vmask[blk[b]] : 0u;
                items += (uint32_t)__popc(vm[b]);
            }
            u += step;
            be = *(const int4 *)(blocks + (u < nb ? u : 0u));
            uint32_t s2[2];
            FewCodes<ND, 4> codes;
            codes.fetch(v, blk, lane);
            codes.scores(v, sh.lq, blk, lane, s2);
            const int i = lane & 31;
            const uint32_t hm = lane >= 32 ? 0xFFFFFFFFu : 0u;   // (by bits: an array indexed per lane would go through memory)
            bool pass[2];
#pragma unroll
            for (int p = 0; p < 2; p++)
                pass[p] = (((vm[2 * p] ^ ((vm[2 * p] ^ vm[2 * p + 1]) & hm)) >> i) & 1u) && s2[p] <= (uint32_t)(tau >> 32);
            if (__ballot(pass[0] || pass[1]) != 0ull) {
                uint2 it[2];
                int L[2];
#pragma unroll
                for (int p = 0; p < 2; p++) {
                    it[p] = make_uint2(RAIRS_EMPTY_ID, 0xFFFFFFFFu);
                    L[p] = -1;
                    const uint32_t bk = (uint32_t)blk[2 * p] ^ (uint32_t)((blk[2 * p] ^ blk[2 * p + 1]) & (int)hm);
                    if (pass[p]) {
                        it[p] = v.idtag[(size_t)bk * 32 + i];
                        L[p] = v.blk_list[bk];           // the list that stores the block: a tagged item is scanned through it
                    }
                }
#pragma unroll
                for (int p = 0; p < 2; p++) {
                    const int o = (int)it[p].y;
                    // RemoveVectorIfVisited: the item is taken from list o
                    if (pass[p] && o >= 0 && o < L[p] && ((bmq[o >> 5] >> (o & 31)) & 1u)) pass[p] = false;
                    const uint64_t x = ((uint64_t)s2[p] << 32) | it[p].x;
                    const bool in = pass[p] && x < tau;
                    const unsigned long long m = __ballot(in);
                    if (m) {
                        uint32_t at = 0;
                        if (lane == 0) at = atomicAdd(&sh.cnt, (uint32_t)__popcll(m));
                        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                        if (in) buf[at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = x;
                    }
                }
            }
        }
        __syncthreads();
        const uint32_t fill = sh.cnt;
        __syncthreads();
        if (fill > FEW_CAP - FEW_ROUND) cut(fill);       // uniform
    }
    if (lane == 0 && items) atomicAdd(&sh.items, items);
    __syncthreads();
    if (sh.cnt > (uint32_t)a.region) cut(sh.cnt);      // (read by everybody before cut's first barrier)
    const uint32_t n = sh.cnt;
    uint64_t *out = a.surv + ((size_t)qi * gridDim.x + blockIdx.x) * a.region;
    for (uint32_t e = (uint32_t)tid; e < n; e += WG) out[e] = buf[e];
    if (tid == 0) a.counts[(size_t)qi * gridDim.x + blockIdx.x] = make_uint2(n, sh.items);
}

// ---- finish: the bigK best, their exact distances, the K best ----------------------------------

#define FIN_NT 1024
#define FIN_KEYS 4096
#define FIN_SLACK 64
template <bool IP, typename RowT>
__global__ __launch_bounds__(FIN_NT) void few_finish_kernel(IndexView v, FewArgs a)
{
    __shared__ PickShared pick;
    __shared__ uint64_t keys[FIN_KEYS];
    __shared__ uint64_t sel[RAIRS_MAX_REFINE_K + FIN_SLACK];
    __shared__ uint32_t cand[RAIRS_MAX_REFINE_K];
    __shared__ uint32_t reg_n[FEW_MAX_WGS], reg_at[FEW_MAX_WGS];             // entries of each workgroup, and of those before it
    __shared__ uint64_t wave_sum[FEW_MAX_WGS / 64];
    __shared__ uint32_t s_cnt, s_min, s_max;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t qi = blockIdx.x;
    const int W = a.wgs, refine_k = a.refine_k, k = a.k;
    static_assert(FEW_MAX_WGS <= FIN_NT, "a thread per region");
    // entries of each workgroup in the low, items scored in the high word: one prefix sum for both
    uint2 cn = make_uint2(0u, 0u);
    if (tid < W) cn = a.counts[(size_t)qi * W + tid];
    const uint32_t incl = wave_incl_sum_u32(cn.x), incl_items = wave_incl_sum_u32(cn.y);
    if (lane == 63 && wave < FEW_MAX_WGS / 64) wave_sum[wave] = ((uint64_t)incl_items << 32) | incl;
    pick_clear<FIN_NT>(pick);
    int turn = 0;
    if (tid == 0) { s_cnt = 0; s_min = 0xFFFFFFFFu; s_max = 0u; }
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < FEW_MAX_WGS / 64; w++) {
        const uint64_t x = wave_sum[w];
        if (w < wave) before += x;
        all += x;
    }
    const uint32_t total = (uint32_t)all;
    if (tid < W) { reg_n[tid] = cn.x; reg_at[tid] = (uint32_t)before + incl - cn.x; }
    if (tid == 0) {
        if (a.dco) a.dco[qi] = (int64_t)(all >> 32);
        a.flags[qi] = 0u;
        a.surv_cnt[qi] = total;
    }
    __syncthreads();
    const uint64_t *src = a.surv + (size_t)qi * W * a.region;
    const bool in_lds = total <= FIN_KEYS;               // uniform
    uint32_t smin = 0xFFFFFFFFu, smax = 0u;              // over this thread's scores
    if (in_lds) {
        // numbered through, so that a thread's loads do not wait for each other
#pragma unroll
        for (int u = 0; u < FIN_KEYS / FIN_NT; u++) {
            const uint32_t e = (uint32_t)(tid + FIN_NT * u);
            if (e < total) {
                int lo = 0, hi = W - 1;                  // the last region that starts at or before e
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (reg_at[mid] <= e) lo = mid; else hi = mid - 1;
                }
                const uint64_t x = src[(size_t)lo * a.region + (e - reg_at[lo])];
                keys[e] = x;
                smin = (uint32_t)(x >> 32) < smin ? (uint32_t)(x >> 32) : smin;
                smax = (uint32_t)(x >> 32) > smax ? (uint32_t)(x >> 32) : smax;
            }
        }
        wave_min_max_u32(smin, smax);
        if (lane == 0) { atomicMin(&s_min, smin); atomicMax(&s_max, smax); }
        __syncthreads();
        smin = s_min;
        smax = s_max;
    } else {
        smin = 0u;
        smax = 255u * (uint32_t)v.M;
    }
    auto each = [&](auto f) {
        if (in_lds) {
            for (uint32_t e = (uint32_t)tid; e < total; e += FIN_NT) f(keys[e]);
        } else {
            for (int r = wave; r < W; r += FIN_NT / 64) {
                const uint32_t n = reg_n[r];
                for (uint32_t e = (uint32_t)lane; e < n; e += 64) f(src[(size_t)r * a.region + e]);
            }
        }
    };
    uint32_t nc = total;                                 // candidates
    if (total > (uint32_t)refine_k) {
        const uint64_t thr = wg_pick<FIN_NT>(each, (uint32_t)refine_k, (uint32_t)refine_k + FIN_SLACK, (uint64_t)smin << 32,
                                             ((uint64_t)smax << 32) | 0xFFFFFFFFull, pick, turn);
        each([&](uint64_t x) {
            if (x <= thr) sel[atomicAdd(&s_cnt, 1u)] = x;
        });
        __syncthreads();
        const int m = (int)s_cnt;
        if (m <= FIN_NT)                                 // uniform
            wg_rank<FIN_NT>(sel, m, [&](uint64_t x, int place) {
                if (place < refine_k) cand[place] = (uint32_t)x;
            });
        else
            for (int i = tid; i < m; i += FIN_NT) {
                const uint64_t mine = sel[i];
                int place = 0;
                for (int j = 0; j < m; j++) place += sel[j] < mine ? 1 : 0;
                if (place < refine_k) cand[place] = (uint32_t)mine;
            }
        nc = (uint32_t)refine_k;
    } else {
        for (uint32_t e = (uint32_t)tid; e < total; e += FIN_NT) cand[e] = (uint32_t)keys[e];   // (bigK <= 1024: in LDS)
    }
    __syncthreads();
    // exact distances: a candidate per group of 16 lanes, two in flight (see refine_kernel)
    const float *qq = a.q + (size_t)qi * v.d;
    const int grp = tid >> 4, l16 = lane & 15;
    constexpr int NG = FIN_NT / 16, RU = 2;
    for (uint32_t c0 = 0; c0 < nc; c0 += NG * RU) {
        uint32_t id[RU];
        float p[RU][4];
        const RowT *row[RU];
#pragma unroll
        for (int u = 0; u < RU; u++) {
            const uint32_t c = c0 + NG * u + grp;
            id[u] = cand[c < nc ? c : nc - 1];
            row[u] = (const RowT *)v.raw + (size_t)id[u] * v.d;
            p[u][0] = p[u][1] = p[u][2] = p[u][3] = 0.0f;
        }
        int i0 = 0;
#pragma unroll 3
        for (; i0 + 64 <= v.d; i0 += 64) {
            float qv[4], x[RU][4];
#pragma unroll
            for (int cc = 0; cc < 4; cc++) {
                qv[cc] = qq[i0 + l16 + 16 * cc];
#pragma unroll
                for (int u = 0; u < RU; u++) x[u][cc] = (float)row[u][i0 + l16 + 16 * cc];
            }
#pragma unroll
            for (int u = 0; u < RU; u++)
#pragma unroll
                for (int cc = 0; cc < 4; cc++) {
                    float sq;
                    if (IP) sq = qv[cc] * x[u][cc];
                    else { const float diff = qv[cc] - x[u][cc]; sq = diff * diff; }
                    p[u][cc] = p[u][cc] + sq;
                }
        }
        if (i0 < v.d) {
#pragma unroll
            for (int cc = 0; cc < 4; cc++) {
                const int i = i0 + l16 + 16 * cc;
                if (i < v.d) {
                    const float qv = qq[i];
#pragma unroll
                    for (int u = 0; u < RU; u++) {
                        const float x = (float)row[u][i];
                        float sq;
                        if (IP) sq = qv * x;
                        else { const float diff = qv - x; sq = diff * diff; }
                        p[u][cc] = p[u][cc] + sq;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < RU; u++) {
            const uint32_t c = c0 + NG * u + grp;
            const float s02 = p[u][0] + p[u][2], s13 = p[u][1] + p[u][3];
            float t = s02 + s13;
            t = t + lane_xor8(t);
            t = t + lane_xor4(t);
            t = t + lane_xor2(t);
            t = t + lane_xor1(t);
            const float dist = IP ? -t : t;
            if (l16 == 0 && c < nc) sel[c] = ((uint64_t)f32_key(dist) << 32) | id[u];
        }
    }
    __syncthreads();
    // a candidate's place in the (distance, id) order is the number of smaller ones
    static_assert(FIN_NT >= RAIRS_MAX_REFINE_K, "a thread per candidate");
    wg_rank<FIN_NT>(sel, (int)nc, [&](uint64_t x, int place) {
        if (place < k) {
            a.out_ids[(size_t)qi * k + place] = (int64_t)(uint32_t)x;
            const float sc = key_f32((uint32_t)(x >> 32));
            a.out_dists[(size_t)qi * k + place] = IP ? -sc : sc;
        }
    });
    for (int r = (int)nc + tid; r < k; r += FIN_NT) {    // fewer than k candidates exist
        a.out_ids[(size_t)qi * k + r] = -1;
        a.out_dists[(size_t)qi * k + r] = IP ? -__builtin_inff() : __builtin_inff();
    }
}

// ---- launch --------------------------------------------------------------------------------------

int rairs_launch_few(const IndexView &v, const FewArgs &a, hipStream_t s, hipEvent_t *ev, const FewEvents &se)
{
    if (a.nq < 1 || a.nq > 65535 || a.nprobe > FEW_MAX_NPROBE || v.nlist > FEW_MAX_NLIST || a.wgs < 1 ||
        a.wgs > FEW_MAX_WGS || a.max_blocks < 4 || (a.max_blocks & 3) != 0 || a.sample_blocks > RAIRS_SAMPLE_MAX_BLOCKS) {
        rairs_set_error("few-query search outside its limits");
        return RAIRS_EINVAL;
    }
    const int dsub = v.d / v.M;
    if (se.lut0) RAIRS_HIP(hipEventRecord(se.lut0, s));
#define FRONT_LAUNCH(IP_, DS_, Q_, LS_)                                                           \
    do {                                                                                          \
        const int groups = (v.nlist + 16 * LS_ - 1) / (16 * LS_);                                 \
        hipLaunchKernelGGL((few_front_kernel<IP_, DS_, Q_, LS_>),                                 \
                           dim3((unsigned)(a.nq + (a.nq + Q_ - 1) / Q_ * groups)), dim3(WG), 0, s, v, a, groups); \
    } while (0)
#define FRONT_SHAPE(IP_, DS_)                                                                     \
    do { if (a.nq >= 4) FRONT_LAUNCH(IP_, DS_, 4, 2); else FRONT_LAUNCH(IP_, DS_, 1, 1); } while (0)
#define FRONT_METRIC(DS_)                                                                         \
    do { if (v.metric) FRONT_SHAPE(true, DS_); else FRONT_SHAPE(false, DS_); } while (0)
    switch (dsub) {
    case 1: FRONT_METRIC(1); break;
    case 2: FRONT_METRIC(2); break;
    case 4: FRONT_METRIC(4); break;
    default: FRONT_METRIC(0); break;
    }
#undef FRONT_METRIC
#undef FRONT_SHAPE
#undef FRONT_LAUNCH
    if (se.lut1) RAIRS_HIP(hipEventRecord(se.lut1, s));
    const dim3 qgrid((unsigned)a.nq);
#define PROBE_LAUNCH(KPT_, ND_) hipLaunchKernelGGL((few_probe_kernel<KPT_, ND_>), qgrid, dim3(PROBE_NT), 0, s, v, a)
#define PROBE_KEYS(ND_)                                                                           \
    do {                                                                                          \
        if (v.nlist <= PROBE_NT) PROBE_LAUNCH(1, ND_);                                            \
        else if (v.nlist <= 4 * PROBE_NT) PROBE_LAUNCH(4, ND_);                                   \
        else PROBE_LAUNCH(16, ND_);                                                               \
    } while (0)
    static_assert(16 * PROBE_NT >= FEW_MAX_NLIST, "a thread's keys cover the largest directory");
    switch (v.nd) {
    case 1: PROBE_KEYS(1); break;
    case 2: PROBE_KEYS(2); break;
    case 3: PROBE_KEYS(3); break;
    case 4: PROBE_KEYS(4); break;
    default: PROBE_KEYS(0); break;
    }
#undef PROBE_KEYS
#undef PROBE_LAUNCH
    if (se.probed) RAIRS_HIP(hipEventRecord(se.probed, s));
    const dim3 sgrid((unsigned)a.wgs, (unsigned)a.nq);
    if (ev) RAIRS_HIP(hipEventRecord(ev[0], s));
#define SCAN_LAUNCH(ND_)                                                                          \
    hipLaunchKernelGGL(few_scan_kernel<ND_>, sgrid, dim3(WG), 0, s, v, a)
    switch (v.nd) {
    case 1: SCAN_LAUNCH(1); break;
    case 2: SCAN_LAUNCH(2); break;
    case 3: SCAN_LAUNCH(3); break;
    case 4: SCAN_LAUNCH(4); break;
    default: SCAN_LAUNCH(0); break;
    }
#undef SCAN_LAUNCH
    if (ev) RAIRS_HIP(hipEventRecord(ev[1], s));
    if (se.scanned) RAIRS_HIP(hipEventRecord(se.scanned, s));
#define FINISH_LAUNCH(IP_, ROW_) hipLaunchKernelGGL((few_finish_kernel<IP_, ROW_>), qgrid, dim3(FIN_NT), 0, s, v, a)
    if (v.metric) { if (v.raw_u8) FINISH_LAUNCH(true, uint8_t); else FINISH_LAUNCH(true, float); }
    else          { if (v.raw_u8) FINISH_LAUNCH(false, uint8_t); else FINISH_LAUNCH(false, float); }
#undef FINISH_LAUNCH
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}
