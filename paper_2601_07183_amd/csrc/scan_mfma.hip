// List-major SEIL scan on the matrix cores (SeilSearch of Alg. 5 for the whole query batch, with
// the list-grouped task order of the "cache optimisation for query batch" paragraph of
// Section 5.2 taken to its conclusion: a block is fetched once for 32 queries).
//
// score(query, item) = sum_m lut[query][m][code[item][m]] is a contraction of the lookup tables
// with a 0/1 expansion of the codes, which the kernels give to the sparse matrix
// instruction v_smfmac_i32_32x32x64_i8 in a form that has nothing to look up (selectors, below).
// The LDS-table kernel (other M) does the same with the tables in LDS.
// Integer arithmetic throughout, so the scores equal the plain 16-bit sums bit for bit.
//
// Work is cut into units (list L, tile of <= 32 queries probing L, run of parts of the list; a part
// is a run of segments of about 32 blocks); waves of a persistent grid draw units from a counter.
// The dedup rules are the order-free ones of scan_exact.hip.  A score passes when it is <= the
// query's bound; passing pairs are staged per wave, logged in bulk and cut to bigK afterwards by
// collect_kernel and the select kernels.
//
// The bound.  tau0 = bigK-th smallest score in a sample, the head of the query's first list (scored
// by the bound kernel of scan_exact.hip, or, for large batches, by sample_group_kernel and
// sample_mfma_kernel below with the same matrix instruction, queries grouped by first list).  Every
// survivor that the duplicate rule can never drop (an item of a shared block, or a miscellaneous
// item whose other list has the larger id; the index keeps one bit per slot for this) is counted in
// a per-query histogram of RAIRS_HIST_BINS equal score bins over [0, tau0] (over a guessed range
// when the sample had fewer than bigK items; scores beyond it share the last bin, which proves
// nothing).  Each counted slot is an entry of the query's candidate
// queue, so once bins 0..b hold >= bigK of them, no item scoring above the top edge of bin b can be
// among the bigK best: that edge is a valid, tighter bound.  Lanes that file survivors re-derive
// the query's bound now and then and lower it with an atomic minimum; scanning waves re-read it
// every few blocks, and once the scan has ended final_bound_kernel derives it from all counts.  A stale view is only looser.
#include <limits.h>

#include <type_traits>

#include "device_util.h"
#include "select_wg.h"

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));


// ---- grouping queries by list ----------------------------------------------------------------

// Where there are fewer units than waves, a unit's blocks are cut into a power of two of slices, a wave for each (as
// many as the log has chunks for: split_max).
static __device__ __forceinline__ uint32_t unit_slices(uint32_t nunits, uint32_t starters, uint32_t split_max)
{
    uint32_t s = 1;
    while (2u * s <= split_max && nunits * 2u * s <= starters) s *= 2u;
    return s;
}
// Chunks of the survivor log that the scanning waves start with: `starters` waves (with the tables
// in registers) or workgroups (tables in LDS, `waves_each` waves) begin on the slices of units numbered by
// their own index, and each wave of those that get one owns the chunk of its index.  The cursor for later
// chunks starts behind them.  (Handing out the first chunks by a counter instead makes 2,048 waves hit
// one address as the kernel starts: 20 us on a 0.56 ms kernel.)
static __device__ __forceinline__ uint32_t log_first_free(uint32_t nunits, uint32_t starters, uint32_t waves_each, uint32_t split_max)
{
    const uint32_t n = nunits * unit_slices(nunits, starters, split_max);
    return (n < starters ? n : starters) * waves_each;
}

__global__ void lm_count_kernel(const int32_t *__restrict__ probe_ids, int64_t nq, int nprobe,
                                int p_first, int nlist, int32_t *lcount)
{
    const int np = nprobe - p_first;
    int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= nq * np) return;
    int64_t q = gid / np;
    int p = p_first + (int)(gid % np);
    int L = probe_ids[q * nprobe + p];
    if (L >= 0 && L < nlist) atomicAdd(&lcount[L], 1);
}

// A unit of work is (list, tile of <= 32 of the queries probing it, run of unit_parts consecutive
// parts of the list; a part is about 32 blocks, unit_parts is 1..4, smaller when there is little
// work).  Exclusive prefixes over lists of queries (loff) and units
// (toff); one workgroup of 1024.
// Parts per unit of list L: the lists from `tail_from` on are cut into single parts.  Waves take
// units in order, so the last ones taken are small and the waves finish closer together (the
// kernel ends with its slowest wave, and a two-part unit is 0.08 ms of work on the 1M x 128 workload).
static __device__ __forceinline__ int list_unit_parts(int L, int unit_parts, int tail_from)
{
    return L >= tail_from ? 1 : unit_parts;
}

static __device__ __forceinline__ int units_of(int nqueries, int part_cnt, int unit_parts)
{
    return ((nqueries + 31) >> 5) * ((part_cnt + unit_parts - 1) / unit_parts);
}

// Everything a scanning wave needs to start on unit `u` of list L in one look-up, so that it does
// not walk unit -> list -> directory entry -> parts at the head of every unit: the list, the tile,
// the unit's segments [seg0, seg1) as absolute segment numbers, and where the list's queries are.
#define UNIT_REC_WORDS 8
#define UNIT_MAX_SEGS 32     // runs per unit: up to 4 parts of RAIRS_PART_SEGS runs
static_assert(4 * RAIRS_PART_SEGS == UNIT_MAX_SEGS, "a unit's runs fit half a wave");
static __device__ __forceinline__ void write_unit_rec(const IndexView &v, int32_t *unit_rec, int u, int L,
                                                      int first_unit_of_list, int qbase, int qn, int unit_parts)
{
    const ListEntry le = v.lists[L];
    const int rem = u - first_unit_of_list;
    const int runs = (le.part_cnt + unit_parts - 1) / unit_parts;
    const int tile = rem / runs;
    const int p0 = (rem % runs) * unit_parts;
    const int p1 = p0 + unit_parts < le.part_cnt ? p0 + unit_parts : le.part_cnt;
    int4 lo = make_int4(L, tile, v.parts[le.part_begin + p0], v.parts[le.part_begin + p1]);
    int4 hi = make_int4(qbase, qn, 0, 0);
    *(int4 *)(unit_rec + (size_t)u * UNIT_REC_WORDS) = lo;
    *(int4 *)(unit_rec + (size_t)u * UNIT_REC_WORDS + 4) = hi;
}

__global__ __launch_bounds__(1024) void lm_prefix_kernel(IndexView v,
                                                         const int32_t *__restrict__ lcount,
                                                         int32_t *loff, int32_t *lcursor,
                                                         int32_t *toff,
                                                         int unit_parts, int tail_from, int32_t *unit_rec,
                                                         uint32_t *log_cursor, uint32_t starters, uint32_t waves_each, uint32_t split_max)
{
    __shared__ int sc[1024], st[1024];
    // one workgroup on the critical path of the grouping, usually next to a kernel that fills the
    // chip: let its waves issue first on the compute unit they share
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x;
    const int per = (v.nlist + 1023) / 1024;
    const int lo = tid * per < v.nlist ? tid * per : v.nlist;
    const int hi = lo + per < v.nlist ? lo + per : v.nlist;
    int c = 0, t = 0;
    for (int L = lo; L < hi; L++) {
        int n = lcount[L];
        c += n;
        t += units_of(n, v.lists[L].part_cnt, list_unit_parts(L, unit_parts, tail_from));
    }
    sc[tid] = c;
    st[tid] = t;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int x = tid >= off ? sc[tid - off] : 0;
        int y = tid >= off ? st[tid - off] : 0;
        __syncthreads();
        sc[tid] += x;
        st[tid] += y;
        __syncthreads();
    }
    int cb = sc[tid] - c, tb = st[tid] - t;
    for (int L = lo; L < hi; L++) {
        int n = lcount[L];
        loff[L] = cb;
        toff[L] = tb;
        lcursor[L] = 0;
        cb += n;
        tb += units_of(n, v.lists[L].part_cnt, list_unit_parts(L, unit_parts, tail_from));
    }
    if (tid == 1023) {
        loff[v.nlist] = sc[1023];
        toff[v.nlist] = st[1023];
        *log_cursor = log_first_free((uint32_t)st[1023], starters, waves_each, split_max);
    }
}

// The unit table of the large-directory route, one thread per list (inside the single workgroup of
// the prefix kernel these writes took 1.5 ms for 16,384 lists and 100,000 units).
__global__ __launch_bounds__(256) void lm_units_kernel(IndexView v, const int32_t *__restrict__ lcount,
                                                       const int32_t *__restrict__ loff,
                                                       const int32_t *__restrict__ toff,
                                                       int unit_parts, int tail_from,
                                                       int32_t *unit_rec)
{
    const int L = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (L >= v.nlist) return;
    const int n = lcount[L], tb = toff[L], cb = loff[L];
    const int up = list_unit_parts(L, unit_parts, tail_from);
    const int nu = units_of(n, v.lists[L].part_cnt, up);
    for (int u = 0; u < nu; u++) write_unit_rec(v, unit_rec, tb + u, L, tb, cb, n, up);
}

__global__ void lm_fill_kernel(const int32_t *__restrict__ probe_ids, int64_t nq, int nprobe,
                               int p_first, int nlist, const int32_t *__restrict__ loff,
                               int32_t *lcursor, int32_t *qlist)
{
    const int np = nprobe - p_first;
    int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= nq * np) return;
    int64_t q = gid / np;
    int p = p_first + (int)(gid % np);
    int L = probe_ids[q * nprobe + p];
    if (L >= 0 && L < nlist) {
        int pos = atomicAdd(&lcursor[L], 1);
        qlist[loff[L] + pos] = (int32_t)q;
    }
}

// The same two steps for directories of up to LM_LDS_NLIST lists: a workgroup first groups its
// LM_PAIRS (query, probe) pairs by list in LDS and then touches each list's global counter once,
// instead of once per pair (a list is probed by hundreds of queries of a batch).
#define LM_PAIRS 4096
#define LM_LDS_NLIST 16384
#define LM_UNIT_WGS 8        // workgroups of the fill kernel that build the unit table
__global__ __launch_bounds__(256) void lm_count_lds_kernel(const int32_t *__restrict__ probe_ids,
                                                           int64_t nq, int nprobe, int p_first,
                                                           int nlist, int32_t *lcount, int qb)
{
    extern __shared__ int32_t lm_hist[];
    const int tid = threadIdx.x;
    for (int i = tid; i < nlist; i += 256) lm_hist[i] = 0;
    __syncthreads();
    const int np = nprobe - p_first;
    const int64_t q0 = (int64_t)blockIdx.x * qb;
    const int pairs = qb * np;
    for (int i = tid; i < pairs; i += 256) {
        const int64_t q = q0 + i / np;
        if (q >= nq) continue;
        const int L = probe_ids[q * nprobe + p_first + i % np];
        if (L >= 0 && L < nlist) atomicAdd(&lm_hist[L], 1);
    }
    __syncthreads();
    for (int i = tid; i < nlist; i += 256) {
        const int c = lm_hist[i];
        if (c) atomicAdd(&lcount[i], c);
    }
}

// Exclusive prefix sums, by a workgroup of 256 threads, of x[0 .. n): thread t owns the contiguous
// run [t per, (t+1) per); `mine` is the sum over its run.  Returns the sum over the runs before
// this thread's and leaves the total in *total (LDS).  wsum: LDS, 4 words.
static __device__ __forceinline__ int wg256_exclusive(int mine, int32_t *wsum, int32_t *total)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_up(incl, off);
        if (lane >= off) incl += x;
    }
    __syncthreads();                                   // wsum may still be read from an earlier call
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        const int x = wsum[w];
        if (w < wave) before += x;
        all += x;
    }
    if (tid == 0) *total = all;
    return before + incl - mine;
}

// Second step for directories of up to LM_LDS_NLIST lists.  No separate prefix kernel sits between
// counting and filling: every workgroup derives the list offsets from the counts itself (a few KB,
// from L2), and LM_UNIT_WGS extra workgroups (the last ones) write them out for the scan together
// with the unit table (toff, unit_rec).
__global__ __launch_bounds__(256) void lm_fill_lds_kernel(IndexView v, const int32_t *__restrict__ probe_ids,
                                                          int64_t nq, int nprobe, int p_first,
                                                          const int32_t *__restrict__ lcount,
                                                          int32_t *loff, int32_t *lcursor, int32_t *qlist,
                                                          int qb, int32_t *toff,
                                                          int unit_parts, int tail_from, int32_t *unit_rec,
                                                          uint32_t *log_cursor, uint32_t starters, uint32_t waves_each, uint32_t split_max)
{
    extern __shared__ int32_t lm_lds[];                // [nlist] ranks / run starts, [nlist + 1] offsets
    __shared__ int32_t wsum[4], total;
    const int nlist = v.nlist;
    int32_t *lm_hist = lm_lds, *loff_s = lm_lds + nlist;
    const int tid = threadIdx.x;
    const int per = (nlist + 255) / 256;
    const int lo = tid * per < nlist ? tid * per : nlist;
    const int hi = lo + per < nlist ? lo + per : nlist;
    {
        int mine = 0;
        for (int L = lo; L < hi; L++) mine += lcount[L];
        int run = wg256_exclusive(mine, wsum, &total);
        for (int L = lo; L < hi; L++) {
            loff_s[L] = run;
            run += lcount[L];
        }
    }
    __syncthreads();
    const int nfill = (int)gridDim.x - LM_UNIT_WGS;
    if ((int)blockIdx.x >= nfill) {
        // The unit table: every one of these workgroups derives the unit offsets of all lists
        // (into LDS), the first writes the offsets out, and each fills its share of the records,
        // finding a unit's list by bisection on the offsets.
        const int ub = (int)blockIdx.x - nfill;
        int32_t *toff_s = lm_hist;                     // [nlist]
        if (ub == 0) {
            if (tid == 0) loff[nlist] = total;
            for (int L = lo; L < hi; L++) loff[L] = loff_s[L];
        }
        int mine = 0;
        for (int L = lo; L < hi; L++) mine += units_of(lcount[L], v.lists[L].part_cnt, list_unit_parts(L, unit_parts, tail_from));
        int run = wg256_exclusive(mine, wsum, &total);
        for (int L = lo; L < hi; L++) {
            toff_s[L] = run;
            if (ub == 0) toff[L] = run;
            run += units_of(lcount[L], v.lists[L].part_cnt, list_unit_parts(L, unit_parts, tail_from));
        }
        __syncthreads();
        const int nunits = total;
        if (ub == 0 && tid == 0) {
            toff[nlist] = nunits;
            *log_cursor = log_first_free((uint32_t)nunits, starters, waves_each, split_max);
        }
        const int share = (nunits + LM_UNIT_WGS - 1) / LM_UNIT_WGS;
        const int e1 = (ub + 1) * share < nunits ? (ub + 1) * share : nunits;
        for (int e = ub * share + tid; e < e1; e += 256) {
            // the last list whose first unit is <= e (lists without units share their successor's offset)
            int a0 = 0, b0 = nlist - 1;
            while (a0 < b0) {
                const int mid = (a0 + b0 + 1) >> 1;
                if (toff_s[mid] <= e) a0 = mid; else b0 = mid - 1;
            }
            write_unit_rec(v, unit_rec, e, a0, toff_s[a0], loff_s[a0], lcount[a0], list_unit_parts(a0, unit_parts, tail_from));
        }
        return;
    }
    for (int i = tid; i < nlist; i += 256) lm_hist[i] = 0;
    __syncthreads();
    const int np = nprobe - p_first;
    const int64_t q0 = (int64_t)blockIdx.x * qb;
    const int pairs = qb * np;                         // <= LM_PAIRS
    int myL[LM_PAIRS / 256], myr[LM_PAIRS / 256];
#pragma unroll
    for (int k = 0; k < LM_PAIRS / 256; k++) {
        const int i = tid + 256 * k;
        myL[k] = -1;
        myr[k] = 0;
        if (i < pairs) {
            const int64_t q = q0 + i / np;
            if (q < nq) {
                const int L = probe_ids[q * nprobe + p_first + i % np];
                if (L >= 0 && L < nlist) {
                    myL[k] = L;
                    myr[k] = atomicAdd(&lm_hist[L], 1);        // rank within this workgroup
                }
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < nlist; i += 256) {
        const int c = lm_hist[i];
        if (c) lm_hist[i] = loff_s[i] + atomicAdd(&lcursor[i], c);   // where this workgroup's run starts
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < LM_PAIRS / 256; k++)
        if (myL[k] >= 0) qlist[lm_hist[myL[k]] + myr[k]] = (int32_t)(q0 + (tid + 256 * k) / np);
}

// ---- the scan ----------------------------------------------------------------------------------

// Element at a 32-bit byte offset from a uniform base (one register of address per lane instead of two).
// The offset is made opaque where it is used: widened outside of a loop it would be a pair of registers again.
template <typename T>
static __device__ __forceinline__ T *at32(T *base, uint32_t bytes)
{
    asm volatile("" : "+v"(bytes));
    return (T *)((char *)base + bytes);
}
// The same value, but made anew where this stands: what is derived from it does not stay in registers
// across the loops around it.
static __device__ __forceinline__ int here(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// counter++ by the calling lane.  (Through an address per lane: where the compiler sees one address it adds up over
// the lanes first and waits for the answer at once.)
static __device__ __forceinline__ uint32_t take_next(uint32_t *counter) { return atomicAdd(at32(counter, 0u), 1u); }

// Bin of a score: floor(score * mul / 2^32) with mul close to BINS 2^32 / (range + 1), range >= BINS, so
// that scores 0 .. range fall into bins 0 .. BINS - 1 (larger scores, and whatever rounding puts beyond
// the last bin, are put into it by the caller).
static __device__ __forceinline__ uint32_t hist_range(uint32_t range)
{
    return range < (uint32_t)RAIRS_HIST_BINS ? (uint32_t)RAIRS_HIST_BINS : range;
}
static __device__ __forceinline__ uint32_t hist_mul(uint32_t range)
{
    return (uint32_t)((float)RAIRS_HIST_BINS * 4294967296.0f * __builtin_amdgcn_rcpf((float)(range + 1u)));
}

// The bound once bins 0 .. b are the first with bigK entries (0xFFFF: none, the last bin also holds scores beyond the range).
// A score of bin <= b is below (b + 1) 2^32 / mul.  The reciprocal, its two roundings and the
// truncation leave mul within 2^-21 of BINS 2^32 / (range + 1), which is at least 2^22, so that is less than
// x + 0.05, x = (b + 1) (range + 1) / BINS <= 65536, and the score at most floor(x + 4 / 64).
static_assert(RAIRS_HIST_BINS == 64, "the slack is in 64ths");
static __device__ __forceinline__ uint32_t bound_at_bin(uint32_t b, uint32_t range)
{
    if (b >= RAIRS_HIST_BINS - 1) return 0xFFFFu;
    const uint32_t edge = ((b + 1u) * (range + 1u) + 4u) / RAIRS_HIST_BINS;
    return edge < 0xFFFFu ? edge : 0xFFFFu;
}

// Tightest bound the histogram of query `qid` proves: the histogram counts queue entries, so once
// bins 0..b hold >= bigK of them nothing scoring above the top edge of bin b can be among the
// bigK best.
static __device__ __forceinline__ uint32_t histogram_bound(const MfmaScanArgs &a, uint32_t qid,
                                                           uint32_t range)
{
    const uint4 *hq = (const uint4 *)at32(a.hist, qid * (RAIRS_HIST_BINS * 4u));
    const uint32_t need = (uint32_t)a.refine_k;
    uint32_t cum = 0;
    int b = 0;                                         // bins with fewer than bigK counted up to them: the first with enough
    // (16 bins in flight at a time: all 64 at once take 64 registers, which the scan loop around
    // this call then pays for with spills)
    constexpr int HB = 4;
    for (int i0 = 0; i0 < RAIRS_HIST_BINS / 4; i0 += HB) {
        uint4 h[HB];
#pragma unroll
        for (int i = 0; i < HB; i++) h[i] = hq[i0 + i];
#pragma unroll
        for (int i = 0; i < HB; i++) {
            cum += h[i].x; b += cum < need ? 1 : 0;
            cum += h[i].y; b += cum < need ? 1 : 0;
            cum += h[i].z; b += cum < need ? 1 : 0;
            cum += h[i].w; b += cum < need ? 1 : 0;
        }
    }
    return bound_at_bin((uint32_t)b, range);
}

// A passing (item, query) pair waits in a per-wave LDS queue until enough have gathered; then the
// wave appends them to its current chunk of a global survivor log with plain stores, counts them
// in the queries' histograms and, for some, lowers the query's bound.  The wave owns its chunk and
// takes a number for the next one when it is full (only waves with work own chunks, so the log of a
// small batch is small).  That waits for an atomic's answer, once in 2,048 entries; asked for at an
// earlier flush, the answer's register was copied, and so waited for together with the flush's stores, in
// every round of survivors (6,000 queries, bigK = 400, lists of 3,800 items: 292 us instead of 253).  Chunks of 2,048 entries: with 256 the scan kernel of the 1M x 128 workload took
// 0.610 ms instead of 0.558 (1,024 and more: the same) and the collect step, whose atomics go by
// chunk and query, 49 us instead of 35.  Ids, tags and the duplicate rule are resolved afterwards,
// in bulk, by collect_kernel and the select kernels.
#define LOG_CHUNK RAIRS_LOG_CHUNK
static_assert((LOG_CHUNK & (LOG_CHUNK - 1)) == 0, "places in a chunk are taken by masking");
#define LOG_COUNTED 0x80000000u    // bit 31 of a staged slot: the entry counts in the histogram
struct StageEntry {
    uint2 log;                     // the log entry: {block * 32 + item (| LOG_COUNTED), score << 16 | query of the pass}
    uint32_t range, unused;        // of the query's histogram
};
struct StageQueue {
    static constexpr int CAP = 256;         // a multiple of 64: a flush takes the queue in rows of 64
    StageEntry ent[CAP + 64];        // the last 64 take what lanes without an entry write
    __device__ __forceinline__ uint2 &log(int i) { return ent[i].log; }
    __device__ __forceinline__ uint32_t range(const MfmaScanArgs &, int i, uint32_t) { return ent[i].range; }
};
// the same for the kernel with the tables in LDS, where every KB counts: the range is looked up again
struct SmallStageQueue {
    static constexpr int CAP = 128;
    uint2 ent[CAP];
    __device__ __forceinline__ uint2 &log(int i) { return ent[i]; }
    __device__ __forceinline__ uint32_t range(const MfmaScanArgs &a, int, uint32_t qid) { return hist_range((uint32_t)*at32(a.tau, qid * 4u)); }
};

struct LogCursor {
    uint32_t chunk, used;               // wave-uniform
};

// When a wave refreshes bounds: every `gap`-th flush.  The gap starts at 4, doubles (up to 16)
// each time a refresh lowers no bound -- late in the scan the bounds have settled and reading
// histograms is wasted time -- and returns to 4 when one does.  (With the bound that the sample
// gives, a start of 2 is 1 % slower on the 1M x 128 workload and 3 % on the 960-dimension one,
// a start of 8 is slower again.)
// (measured on the 1M x 128 workload: all or half of the lanes refreshing, at any pacing, is slower
// than a quarter -- a refresh costs memory traffic per lane, not only latency)
#define REFRESH_LANES_MASK 3
#define REFRESH_GAP_MIN 4u
#define REFRESH_GAP_MAX 16u
struct RefreshPace {
    uint32_t gap, since, turn;          // wave-uniform
};

template <typename Queue>
static __device__ __forceinline__ void stage_flush(const MfmaScanArgs &a, Queue &sq, int n,
                                                   int lane0, LogCursor &lc, RefreshPace &rp)
{
    const int lane = here(lane0);
    const uint32_t end = lc.used + (uint32_t)n;
    uint32_t next = lc.chunk;
    if (end > LOG_CHUNK) {
        // the chunk fills up: the rest goes to another (with no other left this flush is not stored at all, and the
        // chunk ends where it stood: what reads the log takes a fill's word for it that its entries were written)
        if (lane == 0) {
            next = take_next(a.log_cursor);
            if (lc.chunk < (uint32_t)a.log_chunks) a.chunk_fill[lc.chunk] = next < (uint32_t)a.log_chunks ? LOG_CHUNK : lc.used;
        }
        next = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
    }
    const bool room = lc.chunk < (uint32_t)a.log_chunks && next < (uint32_t)a.log_chunks;
    if (!room && lane == 0) *a.log_overflow = 1u;      // every query is then redone exactly
#pragma unroll
    for (int u = 0; u < Queue::CAP / 64; u++) {
        const int i = lane + 64 * u;
        if (i < n) {
            const uint2 e = sq.log(i);
            const uint32_t qid = e.y & 0xFFFFu;
            const uint32_t at = lc.used + (uint32_t)i;
            if (room) a.log[(size_t)(at < LOG_CHUNK ? lc.chunk : next) * LOG_CHUNK + (at & (LOG_CHUNK - 1u))] = make_uint2(e.x & ~LOG_COUNTED, e.y);
            if (e.x & LOG_COUNTED) {
                // scores beyond the histogram's range share the last bin
                const uint32_t bin = __umulhi(e.y >> 16, hist_mul(sq.range(a, i, qid)));
                atomicAdd(at32(a.hist, (qid * RAIRS_HIST_BINS + (bin < RAIRS_HIST_BINS - 1 ? bin : RAIRS_HIST_BINS - 1)) * 4u), 1u);
            }
        }
    }
    if (++rp.since >= rp.gap) {
        // a quarter of the first row's entries, a different quarter each time, refresh their
        // query's bound.  A stale histogram only gives a looser bound; the bound itself only
        // ever shrinks.
        rp.since = 0;
        bool lowered = false;
        if (lane < n && ((lane + rp.turn) & (REFRESH_LANES_MASK)) == 0) {
            const uint32_t qid = sq.log(lane).y & 0xFFFFu;
            int32_t *bq = at32(a.bound, qid * 4u);
            const int32_t cur = __hip_atomic_load(bq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t nb = histogram_bound(a, qid, sq.range(a, lane, qid));
            if (nb < 0xFFFFu && (int32_t)nb < cur) {
                atomicMin(bq, (int32_t)nb);
                lowered = true;
            }
        }
        rp.turn++;
        rp.gap = __ballot(lowered) != 0ull ? REFRESH_GAP_MIN : (rp.gap < REFRESH_GAP_MAX ? rp.gap * 2u : REFRESH_GAP_MAX);
    }
    lc.used = end > LOG_CHUNK ? end - LOG_CHUNK : end;
    lc.chunk = next;
}

// The accumulators of a block start at -(th + 1), th the lane's threshold in the matrix core's
// signed units, so a row passes (score <= th) exactly when its accumulator ends up negative, and
// the mask of passing rows is the 16 sign bits: one funnel shift per row, no compare, no select.
// Lanes that must not pass anything start at a large positive value instead.
#define ACC_NEVER 0x40000000        // (the bits of 2.0f, which an instruction can hold)
static __device__ __forceinline__ uint32_t negative_rows(const v16i &acc)
{
    uint32_t pm = 0;
#pragma unroll
    for (int r = 15; r >= 0; r--) pm = __builtin_amdgcn_alignbit(pm, (uint32_t)acc[r], 31);   // pm << 1 | sign
    return pm;
}

// Mask of the accumulator rows r whose item, 8 (r / 4) + r % 4 in a lane's own count, is below n.
static __device__ __forceinline__ uint32_t rows_below(int n)
{
    uint32_t rows = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int m = n - 8 * k < 0 ? 0 : n - 8 * k > 4 ? 4 : n - 8 * k;
        rows |= ((1u << m) - 1u) << (4 * k);
    }
    return rows;
}
// ---- selectors: a code as five picks of one out of four ------------------------------------------
//
// The sparse instruction takes, per group of four positions, two kept values and their positions
// 0 .. 3.  With the kept values constant (a one in one of the two slots, a zero in the other) a group
// picks one of its four table entries by position.  A code c = 4 h + l becomes five such picks:
//   group g < 4:  entry l of T[4 g .. 4 g + 3] if h == g, else its entry f_g (f = 3, 0, 0, 0),
//   group 4:      entry h of {T[f_0], T[4 + f_1], T[8 + f_2], T[12 + f_3]},
// whose sum is T[c] + sum_g T[4 g + f_g]: the score plus a number that depends on the query alone, which
// goes into the threshold.  (Four groups cannot do: every pattern takes one entry of each group, so the
// 16 x 16 matrix of picks has rank 13.)  The picks of all codes of a dword are bitwise functions of
// it: with X the l and Y the h of sixteen codes as 2-bit fields (eight codes in the fields of one
// slot, eight in those of the other), R1 and R0 the bits of h doubled, the five position words are
//   X | R1 | R0,  X & R0 & ~R1,  X & R1 & ~R0,  X & R1 & R0,  Y
// -- a dozen vector instructions for ten matrix instructions, and no table to look anything up in.
// Position words: nibble n of a lane's word belongs to its group n, low two bits the first slot.
#define SEL_F0 3                    // f_0; f_1, f_2 and f_3 are 0
#define SEL_FIRST 0x00010001        // kept values: the pick is the first slot's ...
#define SEL_SECOND 0x01000100       // ... or the second one's
// bit by bit m ? a : b
static __device__ __forceinline__ uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

static __device__ __forceinline__ void select_words(uint32_t X, uint32_t Y, uint32_t R1, uint32_t R0, uint32_t (&w)[5])
{
    w[0] = X | R1 | R0;
    w[1] = X & R0 & ~R1;
    w[2] = X & R1 & ~R0;
    w[3] = X & R1 & R0;
    w[4] = Y;
}
// sixteen codes of a lane: those of dword a in the first slots, those of dword b in the second ones
static __device__ __forceinline__ void select_words_pair(uint32_t a, uint32_t b, uint32_t (&w)[5])
{
    const uint32_t X = bit_select(0x33333333u, a, b << 2), Y = bit_select(0x33333333u, a >> 2, b);
    select_words(X, Y, bit_select(0x55555555u, Y >> 1, Y), bit_select(0x55555555u, Y, Y << 1), w);
}
// eight codes, first slots (the second ones hold anything)
static __device__ __forceinline__ void select_words_one(uint32_t a, uint32_t (&w)[5])
{
    const uint32_t Y = a >> 2;
    select_words(a, Y, bit_select(0x55555555u, a >> 3, Y), bit_select(0x55555555u, Y, a >> 1), w);
}

// An instruction (v_smfmac_i32_32x32x64_i8: 32 items x 32 queries x 16 groups) takes one group of eight codes
// of either parity: 5 nd of them a block, instruction 5 w + g group g of the codes of dword w.  Lane (item,
// parity) gives positions for its eight groups; the instruction's K order, checked entry by entry, takes groups
// 0 - 3 of parity p from registers 4 p .. + 3 of the table operand's lower half wave, groups 4 - 7 from its
// upper one.  (The one-hot expansion took 4 nd instructions, each fed by four LDS look-ups and five vector
// instructions.)

// The table operand straight from the bytes T (the sample's kernel): lane (query, half) holds, for dword w,
// sub-quantizers 16 w + 8 half .. + 7, even ones in the first four registers, four table entries (signed:
// value - 128) to a register.  M must be 16 ND: all of 16 ND rows are read and picked from.  Returns what a
// contraction is above the score (the same number in both lanes of a query).
template <int ND>
static __device__ __forceinline__ int load_byte_tables(const uint8_t *lut, uint32_t qid, int M, int half, v8i (&B)[5 * ND])
{
    const uint8_t *lq = lut + (size_t)qid * (size_t)(M * 16) + half * 128;
    int extra = 0;                                     // sum of the (signed) entries that the groups not meant pick
#pragma unroll
    for (int w = 0; w < ND; w++) {
        v4i x[8];
#pragma unroll
        for (int k = 0; k < 8; k++) x[k] = *(const v4i *)(lq + w * 256 + k * 16) ^ (int)0x80808080;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int r = (k >> 1) + 4 * (k & 1);
#pragma unroll
            for (int g = 0; g < 4; g++) B[5 * w + g][r] = x[k][g];
            // bytes f_0 of group 0, 0 of groups 1, 2, 3
            const int e = (int)(__builtin_amdgcn_perm((uint32_t)x[k].y, (uint32_t)x[k].x, 0x0C0C0400u + SEL_F0) |
                                __builtin_amdgcn_perm((uint32_t)x[k].w, (uint32_t)x[k].z, 0x04000C0Cu));
            B[5 * w + 4][r] = e;
            extra = __builtin_amdgcn_sdot4(e, 0x01010101, extra, false);
        }
        __builtin_amdgcn_sched_barrier(0);             // (32 registers of loads in flight at a time, not 32 ND)
    }
    extra += __shfl_xor(extra, 32);
    // a contraction is the sum over the sub-quantizers of T[c] + sum_g T[4 g + f_g], less 5 * 128; extra is that
    // of the T[4 g + f_g], less 4 * 128
    return extra - 128 * M;
}

// The scan's own form of the tables, made once per query.  A group's entries may be shifted by a number of
// its own, so the entry that the groups not meant pick is made zero wherever the other three fit into a
// signed byte then: four of five picks are zeros.  What a matrix instruction costs is power: with random
// table bytes picked everywhere the chip holds 1.66 GHz (19.7 ns each, every SIMD at it), with four of five
// picks zero 2.03 GHz (16.1 ns; the one-hot expansion 1.72 GHz, 19.0 ns).
// Per query scan_tables_stride bytes: for dword w and half the five registers of eight words each that
// load_byte_tables describes, then what a contraction is above the score.
static __host__ __device__ __forceinline__ int scan_tables_stride(int nd) { return nd * 320 + 16; }

// One wave makes those of query q, a lane per sub-quantizer.
static __device__ __forceinline__ void write_scan_tables(const uint8_t *__restrict__ lut, int M, int nd, int64_t q,
                                                         uint8_t *__restrict__ tables)
{
    const int lane = threadIdx.x & 63;
    const int stride = scan_tables_stride(nd);
    uint32_t *out = (uint32_t *)(tables + (size_t)q * stride);
    int above = 0;
    for (int m = lane; m < 16 * nd; m += 64) {
        uint32_t e[5] = {0u, 0u, 0u, 0u, 0u};          // (sub-quantizers from M on: zeros)
        if (m < M) {
            const v4i x = *(const v4i *)(lut + (size_t)q * (size_t)(M * 16) + (size_t)m * 16);
            above -= 128;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                int t[4];
#pragma unroll
                for (int l = 0; l < 4; l++) t[l] = (int)(((uint32_t)x[g] >> (8 * l)) & 255u);
                const int lo = min(min(t[0], t[1]), min(t[2], t[3])), hi = max(max(t[0], t[1]), max(t[2], t[3]));
                const int tf = t[g == 0 ? SEL_F0 : 0];
                const int shift = min(max(tf, hi - 127), lo + 128);
                above += tf - shift;
#pragma unroll
                for (int l = 0; l < 4; l++) e[g] |= ((uint32_t)(t[l] - shift) & 255u) << (8 * l);
                e[4] |= ((uint32_t)(tf - 128) & 255u) << (8 * g);
            }
        }
        const int k = m & 7, r = (k >> 1) + 4 * (k & 1);
        uint32_t *p = out + (m >> 3) * 40 + r;
#pragma unroll
        for (int g = 0; g < 5; g++) p[8 * g] = e[g];
    }
    const uint32_t sum = wave_sum_u32((uint32_t)above);
    if (lane == 0) out[nd * 80] = sum;
}

// First kernel of the grouping: `zero_wgs` workgroups clear the counters, the others make the scan's tables, a wave per
// query.  (Nobody before the scan reads either.  A launch of its own for the tables is 5 us more on the way to the scan.)
// The scanning waves start on the units numbered by their own index (a second one each at index +
// nwaves with the tables in registers), so the unit counter starts behind those.
__global__ __launch_bounds__(WG) void lm_begin_kernel(int zero_wgs, IndexView v, MfmaScanArgs a, uint32_t first_task)
{
    if ((int)blockIdx.x >= zero_wgs) {
        const int64_t q = (int64_t)(blockIdx.x - zero_wgs) * (WG / 64) + (threadIdx.x >> 6);
        if (q < a.nq) write_scan_tables(a.lut, v.M, v.nd, q, a.tables);
        return;
    }
    const int64_t gid = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (gid < v.nlist) { a.lcount[gid] = 0; a.lcursor[gid] = 0; }
    if (gid < a.nq) { a.surv_cnt[gid] = 0; if (a.dco) a.dco[gid] = 0ull; }
    if (gid < a.log_chunks) a.chunk_fill[gid] = 0;
    if (gid == 0) { *a.next_task = first_task; *a.log_cursor = 0u; a.log_overflow[0] = 0; a.log_overflow[1] = 0; }   // (the cursor: set again with the unit count)
    if (gid == 0) { a.work[0] = 0u; a.work[1 + a.nq] = 0u; }   // the two lists of queries for the kernels behind the scan
}

template <int ND>
static __device__ __forceinline__ void load_scan_tables(const uint8_t *tables, uint32_t qid, int half, v8i (&B)[5 * ND])
{
    const uint32_t row = qid * (uint32_t)scan_tables_stride(ND);        // < 2^29: a pass has at most 65,536 queries
    const char *p = (const char *)at32(tables, row + (uint32_t)half * 160u);
#pragma unroll
    for (int t = 0; t < 5 * ND; t++) {
        const v4i x = *(const v4i *)(p + (t / 5 * 320 + t % 5 * 32)), y = *(const v4i *)(p + (t / 5 * 320 + t % 5 * 32 + 16));
        B[t] = (v8i){x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    }
}

// acc += the contraction of a block's codes with the tables, in two parts.
template <int ND>
struct Contraction {
    static_assert(ND == 1 || ND == 3 || ND == 4, "the kernels' shapes");
    static constexpr int FRONT = ND >= 3 ? 10 : 5, BACK = 5 * ND - FRONT;      // matrix instructions
    uint32_t s[2][5];                                  // position words of the two parts
    __device__ __forceinline__ void front_words(const uint32_t (&c)[ND])
    {
        if (ND >= 3) select_words_pair(c[0], c[ND >= 3 ? 1 : 0], s[0]);
        else select_words_one(c[0], s[0]);
    }
    __device__ __forceinline__ void back_words(const uint32_t (&c)[ND])
    {
        if (ND == 3) select_words_one(c[ND - 1], s[1]);
        if (ND == 4) select_words_pair(c[ND > 2 ? 2 : 0], c[ND - 1], s[1]);
    }
    __device__ __forceinline__ void front(const v8i (&B)[5 * ND], v16i &acc)
    {
        five<0>(s[0], B, acc);
        if (ND >= 3) five<1>(s[0], B, acc);
    }
    __device__ __forceinline__ void back(const v8i (&B)[5 * ND], v16i &acc)
    {
        if (ND >= 3) five<(ND >= 3 ? 2 : 0)>(s[1], B, acc);
        if (ND == 4) five<(ND == 4 ? 3 : 0)>(s[1], B, acc);
    }
    template <int W>
    static __device__ __forceinline__ void five(const uint32_t (&w)[5], const v8i (&B)[5 * ND], v16i &acc)
    {
        constexpr int kept = W & 1 ? SEL_SECOND : SEL_FIRST;
        const v4i slot = {kept, kept, kept, kept};
#pragma unroll
        for (int g = 0; g < 5; g++) acc = __builtin_amdgcn_smfmac_i32_32x32x64_i8(slot, B[5 * W + g], acc, (int)w[g], 0, 0);
    }
};
template <int ND>
static __device__ __forceinline__ void contract_block(const uint32_t (&c)[ND], const v8i (&B)[5 * ND], v16i &acc)
{
    Contraction<ND> k;
    k.front_words(c);
    k.front(B, acc);
    k.back_words(c);
    k.back(B, acc);
}
// Lets the instruction scheduler put N vector instructions behind each of M matrix instructions.
template <int M, int N>
static __device__ __forceinline__ void interleave()
{
#pragma unroll
    for (int i = 0; i < M; i++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, N, 0);
    }
}

// Number of set bits of `mask` below this lane.
static __device__ __forceinline__ int lanes_below(unsigned long long mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// acc[r] for a row index that differs from lane to lane: four levels of bitwise selection on the
// bits of r, in registers (an indexed array would go through memory).
static __device__ __forceinline__ int select_row(const v16i &acc, int r)
{
    const int m0 = -(r & 1), m1 = -((r >> 1) & 1), m2 = -((r >> 2) & 1), m3 = -((r >> 3) & 1);
    int s8[8], s4[4];
#pragma unroll
    for (int k = 0; k < 8; k++) s8[k] = (acc[2 * k + 1] & m0) | (acc[2 * k] & ~m0);
#pragma unroll
    for (int k = 0; k < 4; k++) s4[k] = (s8[2 * k + 1] & m1) | (s8[2 * k] & ~m1);
    const int s2a = (s4[1] & m2) | (s4[0] & ~m2), s2b = (s4[3] & m2) | (s4[2] & ~m2);
    return (s2b & m3) | (s2a & ~m3);
}

// Read-only words at a wave-uniform address, by scalar loads.
template <typename T>
using scalar_ptr = const __attribute__((address_space(4))) T *;
template <typename T>
static __device__ __forceinline__ scalar_ptr<T> as_scalar(const T *p) { return (scalar_ptr<T>)(uintptr_t)p; }

// What bounds it: the matrix cores' power (2 waves a SIMD; see write_scan_tables) and the survivors' vector
// instructions, which run beside them a block behind.  Before (one-hot rows looked up in LDS, survivors after
// each block): 1M x 128, M = 64, 10,000 queries, 23 probes: 695 us, now 645; 2,999 queries, bigK = 400: 515, 460;
// 1M x 96, M = 48: 430, 400; 100 probes of 16,384 lists: 3.96 ms, 3.75.
// ND: code dwords of an item and parity (M <= 16 ND).  SLICED: units may be cut into slices (compiled in where they
// never are, that costs 3 % of the 1M x 128 workload's kernel).
template <int ND, bool SLICED>
__global__ __launch_bounds__(WG, 2) void scan_mfma_kernel(IndexView v, MfmaScanArgs a)
{
    __shared__ StageQueue stage[WG / 64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    StageQueue &sq = stage[wave];
    int nstaged = 0;                                   // wave-uniform fill of the stage queue
    const uint32_t nunits = (uint32_t)as_scalar(a.toff)[v.nlist];
    if (nunits == 0u) return;                          // nothing was written: all chunk fills stay 0
    // first unit and first log chunk by wave index; the counters start behind them
    const uint32_t gwave = blockIdx.x * (WG / 64) + (uint32_t)wave, nwaves = gridDim.x * (WG / 64);
    LogCursor lc;
    lc.chunk = gwave;                                  // (a wave without a unit never writes)
    lc.used = 0;
    RefreshPace pace = {REFRESH_GAP_MIN, REFRESH_GAP_MIN - 1u, 0u};
#define FLUSH_STAGE()                                                   \
    do {                                                                \
        stage_flush(a, sq, nstaged, lane, lc, pace);     \
        nstaged = 0;                                                    \
    } while (0)

    // Unit u below is slice u % slices of unit u / slices.
    const uint32_t slices = SLICED ? unit_slices(nunits, nwaves, (uint32_t)a.split_max) : 1u, nslices = nunits * slices;
    const uint32_t slice_shift = (uint32_t)__builtin_ctz(slices);
    // A wave works on unit u, already knows the one after it (u_next) and asks the counter for
    // the one after that: so the record of the next unit can be fetched a whole unit ahead and a
    // unit starts with its queries and segments in registers instead of a chain of look-ups.
    // A flush costs much the same for one row of 64 entries and for three; but what waits in the queues is not
    // counted, so bounds fall later, and with few units a wave or a small bigK so many entries gather above the
    // final bound that buffers overflow.  (1M x 128, 2,999 queries, bigK = 400: 514 us with one row, 473 with two, 460 with
    // three; 300,000 x 96, 2,048 lists, 10,000 queries, 16 probes, bigK = 100, 5,500 units: 235, 204; 200,000 x 128, 400 lists,
    // 3,000 queries, bigK = 40, 2,000 units: 146, 142, but then the selection takes 20 us more.  At M = 16 a survivor
    // costs more than the contraction of a block, so bounds come first: 200,000 x 32, 10,000 queries, 32 probes, bigK = 10: 603
    // with one row, 640 with two.)
    const int flush_above = ND == 1 ? 64 : a.refine_k >= 256 ? 192 : nunits >= (a.refine_k >= 64 ? 1u : 3u) * nwaves ? 128 : 64;
    // A unit's bounds are looked up every second block, at M = 16 every one, and with many units a wave every fourth: by then they
    // have settled.  (Every fourth / second: M = 48, 500 queries, 64 of 400 lists, bigK = 1,000 2,700 us, the log runs out, 768;
    // M = 64, 2,000 queries, 32 of 400 lists, bigK = 400 308, 289; 2M x 96, 4,096 lists, 10,000 queries, 39 probes 382, 402; M = 16,
    // 10,000 queries, 16 of 400 lists 807, 727 and with every one 703.  At M = 48 and 64 there are no registers for every one.)
    const int bound_mask = ND == 1 ? 0 : nunits >= 3u * nwaves ? 3 : 1;
    uint32_t u = gwave, u_next = gwave + nwaves;       // the counter starts behind both
    auto record = [&](uint32_t i) {
        const scalar_ptr<int32_t> p = as_scalar(a.unit_rec) + (size_t)(i >> slice_shift) * UNIT_REC_WORDS;
        return make_int4(p[4] + 32 * p[1], p[5] - 32 * p[1], p[2], p[3]);      // {first query of the tile, queries from there on, segments}
    };
    // ... and the query of this lane's column there (an absent column takes query 0's tables and never passes), the
    // range of its histogram, and what its contractions are above its scores
    struct Column {
        int qid;
        uint32_t range;
        int above;
    };
    auto tile_query = [&](const int4 &r) { const int j = here(lane) & 31; return j < r.y ? *at32(a.qlist + r.x, (uint32_t)j * 4u) : -1; };
    auto query_facts = [&](Column &c) {
        const uint32_t q = (uint32_t)(c.qid >= 0 ? c.qid : 0);
        c.range = hist_range((uint32_t)*at32(a.tau, q * 4u));
        c.above = *(const int *)at32(a.tables, q * (uint32_t)scan_tables_stride(ND) + (uint32_t)(ND * 320));
    };
    int4 rec = record(u < nslices ? u : 0u);
    Column next;
    next.qid = tile_query(rec);
    query_facts(next);
    while (u < nslices) {                              // every wave leaves: the counter only grows
        uint32_t u_next2 = 0;
        if (lane == 0) u_next2 = take_next(a.next_task);
        int seg0 = rec.z, first = 0, left = INT_MAX;   // the slice: from block `first` of run seg0 on, `left` blocks
        const int seg1 = rec.w;
        const int qid = next.qid, above = next.above;
        const uint32_t range = next.range;
        rec = record(u_next < nslices ? u_next : u);
        next.qid = tile_query(rec);
        // run entries go two ahead and the owner's bitmap word one ahead, so that neither is waited for at
        // the head of a run
        auto segment = [&](int i) {
            const scalar_ptr<SegEntry> p = as_scalar(v.segs) + i;
            SegEntry e;
            e.blk_begin = p->blk_begin; e.nblk = p->nblk; e.misc_from = p->misc_from; e.owner = p->owner; e.tail_valid = p->tail_valid;
            return e;
        };
        if (slices > 1u) {                             // uniform
            // (a run per lane: one after the other, their lengths are a chain of up to 32 scalar loads)
            const int i = here(lane), runs = seg1 - seg0;
            int upto = i < runs ? v.segs[seg0 + i].nblk : 0;           // blocks of runs 0 .. i
#pragma unroll
            for (int off = 1; off < UNIT_MAX_SEGS; off <<= 1) {
                const int x = __shfl_up(upto, off);
                if (i >= off) upto += x;
            }
            const int n = __builtin_amdgcn_readlane(upto, UNIT_MAX_SEGS - 1), s = (int)(u & (slices - 1u));
            first = (n * s) >> slice_shift;
            left = ((n * (s + 1)) >> slice_shift) - first;
            const int over = __popcll(__builtin_amdgcn_ballot_w64(i < runs && upto <= first));     // runs before the slice
            if (over > 0 && left > 0) {
                first -= __builtin_amdgcn_readlane(upto, over - 1);
                seg0 += over;
            }
        }
        if (left > 0) {
        const int unit_lane = here(lane);
        const uint32_t q0 = (uint32_t)(qid >= 0 ? qid : 0);
        v8i B[5 * ND];
        load_scan_tables<ND>(a.tables, q0, unit_lane >> 5, B);
        query_facts(next);
        // the query's bound: other waves keep lowering it, so it is looked up again during the
        // run, ahead of the block that uses it (a stale bound is only looser)
        // per-lane addresses stay 32-bit offsets from uniform bases (a 64-bit pointer per lane
        // costs two of the registers this kernel is short of)
        const uint32_t bm0 = q0 * (uint32_t)a.bmwords;   // < 2^27: a pass has at most 65,536 queries of at most 2,048 words
        int bound_next = __hip_atomic_load(at32(a.bound, q0 * 4u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // Codes and masks {countable slots, slots in use} of a block are fetched a block before they are
        // scored: the fetches walk through the unit's runs on their own (and stay on its last block).  (Two or
        // three blocks ahead: no faster.)
        int fseg = seg0;
        SegEntry fs = segment(seg0);
        int fblk = fs.blk_begin + first, fend = fs.blk_begin + fs.nblk;
        fs = segment(seg0 + 1 < seg1 ? seg0 + 1 : seg0);       // the run behind the one that is being fetched
        uint32_t cn[ND];
        uint2 cmn;
        auto fetch = [&]() {
            const char *p = (const char *)at32(v.codes + (size_t)fblk * ND * 64, (uint32_t)lane * 4u);    // (a uniform base)
#pragma unroll
            for (int w = 0; w < ND; w++) cn[w] = *(const uint32_t *)(p + w * 256);
            const scalar_ptr<uint2> m = as_scalar(v.bmask) + fblk;
            cmn = make_uint2(m->x, m->y);
            if (fblk + 1 < fend) fblk++;
            else if (fseg + 1 < seg1) {
                fseg++;
                fblk = fs.blk_begin;
                fend = fblk + fs.nblk;
                fs = segment(fseg + 1 < seg1 ? fseg + 1 : fseg);
            }
        };
        fetch();
        // The blocks in turn.  A block's survivors are looked for while the next one is contracted: two sets of
        // accumulators, and with each set what its survivors need to know of the block.
        struct Scored {
            v16i acc;                                  // acc[r]: item row 8 (r / 4) + 4 half + r % 4, query column j
            int negth;                                 // what the accumulators started at
            uint32_t rows;                             // this lane's rows whose slots can hold an item
            int blk;                                   // wave-uniform
            uint32_t cmask;
        };
        int seg = seg0, b = first;
        SegEntry se = segment(seg0), sen = segment(seg0 + 1 < seg1 ? seg0 + 1 : seg0);
        auto owner_word = [&](const SegEntry &e) { return *at32(a.bitmap, (bm0 + (uint32_t)(e.owner >= 0 ? e.owner >> 5 : 0)) * 4u); };
        uint32_t owner_bits = owner_word(se);          // of the run to be entered
        uint32_t scored = 0, seg_items = 0;            // items this lane's query was scored against in this unit; slots in use of the run's blocks
        bool live = false;
        int negth = ACC_NEVER;
        auto enter_run = [&]() {
            // cell (owner, L) is scored through list `owner` for queries that probe it
            live = qid >= 0 && !(se.owner >= 0 && ((owner_bits >> (se.owner & 31)) & 1u));
            // (the next run's word into the same register: into another one, it is copied and waited for here)
            __builtin_amdgcn_sched_barrier(0);
            owner_bits = owner_word(sen);
            negth = ACC_NEVER;
            seg_items = 0;
        };
        // the block behind the present one, if the unit has one
        auto advance = [&]() __attribute__((always_inline)) {
            if (--left > 0 && ++b < se.nblk) return true;
            // the distance computations of this run (Section 6.1's DCO): every slot in use of every block
            // that was contracted, for each query the run was live for
            scored += live ? seg_items : 0u;
            if (left == 0 || ++seg >= seg1) return false;
            se = sen;
            sen = segment(seg + 1 < seg1 ? seg + 1 : seg);
            b = first = 0;
            enter_run();
            return true;
        };
        // one survivor of every lane that has any (pm: its rows that pass), no branches
        auto stage_round = [&](const Scored &x, uint32_t &pm, int lane_) __attribute__((always_inline)) {
            const int half = lane_ >> 5;
            const unsigned long long mask = __builtin_amdgcn_ballot_w64(pm != 0u);
            int at = nstaged + lanes_below(mask);
            asm volatile("" : "+v"(at));               // (or a branch goes around its two instructions)
            const int pos = pm != 0u ? at : StageQueue::CAP + lane_;
            const int r = __builtin_ctz(pm | 0x10000u);
            pm &= pm - 1u;
            const int sc = select_row(x.acc, r & 15) - x.negth - above;      // the row's score
            const uint32_t item = 8u * (uint32_t)(r >> 2) + (uint32_t)(r & 3) + 4u * half;
            sq.log(pos) = make_uint2(((uint32_t)x.blk * 32u + item) | (((x.cmask >> (item & 31u)) & 1u) << 31),
                                         ((uint32_t)sc << 16) | (uint32_t)qid);
            sq.ent[pos].range = range;
            nstaged += __popcll(mask);
        };
        auto stage_rest = [&](const Scored &x, uint32_t &pm) __attribute__((always_inline)) {
            for (;;) {
                if (nstaged > flush_above) FLUSH_STAGE();
                if (__builtin_amdgcn_ballot_w64(pm != 0u) == 0ull) break;
                stage_round(x, pm, here(lane));
            }
        };
        auto step = [&](Scored &x, const Scored &before) __attribute__((always_inline)) {
            uint32_t c[ND];
            const uint2 masks = cmn;
#pragma unroll
            for (int w = 0; w < ND; w++) c[w] = cn[w];
            fetch();
            seg_items += (uint32_t)__popc(masks.y);
            if (((b - first) & bound_mask) == 0) {
                // the accumulators start at -(threshold + 1): a row passes iff it ends up negative
                if (live) negth = -(bound_next + above + 1);
                bound_next = __hip_atomic_load(at32(a.bound, q0 * 4u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            x.negth = negth;
            x.blk = se.blk_begin + b;
            x.cmask = masks.x;
            x.rows = 0xFFFFu;
            // the list's last block: drop rows whose slot holds no item
            if (b == se.nblk - 1 && se.tail_valid < 32) x.rows = rows_below(se.tail_valid - 4 * (here(lane) >> 5));
            Contraction<ND> k;
            k.front_words(c);
            // (a copy the compiler cannot see through: the accumulators' start value must not stay tied to the
            // register that the survivors need later, or the whole tuple is built elsewhere and moved)
            int acc0 = negth;
            asm volatile("" : "+v"(acc0));
#pragma unroll
            for (int r = 0; r < 16; r++) x.acc[r] = acc0;
            __builtin_amdgcn_sched_barrier(0);
            k.front(B, x.acc);
            k.back_words(c);
            uint32_t pm = negative_rows(before.acc) & before.rows;     // rows of this lane that pass
            interleave<Contraction<ND>::FRONT, 3>();
            __builtin_amdgcn_sched_barrier(0);
            k.back(B, x.acc);
            // (the first round without a look whether there is one to make: five matrix instructions leave no room for it)
            if (ND > 1) stage_round(before, pm, here(lane));
            interleave<Contraction<ND>::BACK, 4>();
            __builtin_amdgcn_sched_barrier(0);
            // (the next block's codes are waited for here: behind a flush it would be a wait for its stores and
            // atomics too, which are counted with the loads)
#pragma unroll
            for (int w = 0; w < ND; w++) asm volatile("" : "+v"(cn[w]));
            stage_rest(before, pm);
        };
        Scored x0, x1;
        x1.negth = ACC_NEVER; x1.rows = 0u; x1.blk = 0; x1.cmask = 0u;
#pragma unroll
        for (int r = 0; r < 16; r++) x1.acc[r] = ACC_NEVER;
        enter_run();
        for (;;) {
            step(x0, x1);
            if (!advance()) break;
            step(x1, x0);
            if (!advance()) { x0 = x1; break; }
        }
        uint32_t pm = negative_rows(x0.acc) & x0.rows;
        stage_rest(x0, pm);
        if (a.dco && here(lane) < 32 && scored) atomicAdd(at32(a.dco, (uint32_t)qid * 8u), (unsigned long long)scored);
        } else
            query_facts(next);
        // do not sit on survivors for long: their histogram counts tighten everyone's bound
        if (nstaged >= 32 || (u_next >= nslices && nstaged > 0)) FLUSH_STAGE();
        u = u_next;
        u_next = (uint32_t)__builtin_amdgcn_readfirstlane((int)u_next2);
    }
    // (a wave that never had a unit wrote nothing, and the chunk of its index may be another wave's)
    if (lane == 0 && lc.used > 0 && lc.chunk < (uint32_t)a.log_chunks) a.chunk_fill[lc.chunk] = lc.used;
}

// The bounds once more before the log is read, a wave per query: by now every survivor is counted.  The scanning waves
// refresh a bound now and then, and a batch of few units is over before most of them have: of what they logged so
// much stays at or below a stale bound that queries leave the wave's select for the workgroup's, or for the exact redo.
// (28,000 x 100, M = 50, 500 queries, 64 of 97 lists, bigK = 1,000: 1,400 us, two queries redone, now 630; M = 48, 3,000 queries, 4 probes,
// bigK = 40: 183 us, now 166.)  Few lists and a small bigK cannot fill a buffer: there its launch, 3 us, is saved.
static bool final_bound_pays(const MfmaScanArgs &a) { return a.refine_k >= 32 || a.nprobe >= 8; }
__global__ __launch_bounds__(WG) void final_bound_kernel(MfmaScanArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * (WG / 64) + (threadIdx.x >> 6);
    if (q >= a.nq) return;
    uint32_t upto = a.hist[q * RAIRS_HIST_BINS + lane];        // a bin per lane
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = __shfl_up(upto, off);
        if (lane >= off) upto += x;
    }
    const uint32_t b = (uint32_t)__popcll(__ballot(upto < (uint32_t)a.refine_k));
    if (lane == 0) {
        const int32_t nb = (int32_t)bound_at_bin(b, hist_range((uint32_t)a.tau[q]));
        if (nb < 0xFFFF && nb < a.bound[q]) a.bound[q] = nb;
    }
}

// Distribute the survivor log to the per-query buffers (a workgroup takes one chunk at a time).  A chunk holds
// entries of a few dozen queries; they are grouped in LDS first so that each query's counter is
// bumped once per chunk, not once per entry.
#define COLLECT_WG 1024
#define COLLECT_EPT (LOG_CHUNK / COLLECT_WG)            // entries of a chunk per thread
#define COLLECT_SLOTS 512
static_assert(LOG_CHUNK % COLLECT_WG == 0, "a chunk is a whole number of entries per thread");
static_assert(COLLECT_WG >= COLLECT_SLOTS, "a thread per slot clears and publishes the tables");
__global__ __launch_bounds__(COLLECT_WG) void collect_kernel(MfmaScanArgs a)
{
    __shared__ int32_t key[COLLECT_SLOTS];
    __shared__ uint32_t cnt[COLLECT_SLOTS], base[COLLECT_SLOTS];
    const int tid = threadIdx.x;
    const uint32_t lim = log_chunks_used(a);
    for (uint32_t c = blockIdx.x; c < lim; c += gridDim.x) {
    const uint32_t n = a.chunk_fill[c];
    if (n == 0) continue;                               // uniform
    if (tid < COLLECT_SLOTS) { key[tid] = -1; cnt[tid] = 0; }
    __syncthreads();
    uint2 e[COLLECT_EPT];                               // {slot, score << 16 | query}
    int slot[COLLECT_EPT];
    uint32_t rank[COLLECT_EPT];
    // an entry logged under an earlier, looser bound is dropped when its score is above the
    // query's final bound: it cannot be among the bigK best
    bool live[COLLECT_EPT];
#pragma unroll
    for (int k = 0; k < COLLECT_EPT; k++) {
        const int i = tid + COLLECT_WG * k;
        e[k] = make_uint2(0, 0);
        if (i < (int)n) e[k] = a.log[(size_t)c * LOG_CHUNK + i];
    }
#pragma unroll
    for (int k = 0; k < COLLECT_EPT; k++) {
        const int i = tid + COLLECT_WG * k;
        live[k] = i < (int)n && (int32_t)(e[k].y >> 16) <= a.bound[e[k].y & 0xFFFFu];
        slot[k] = -1;
        rank[k] = 0;
    }
#pragma unroll
    for (int k = 0; k < COLLECT_EPT; k++) {
        if (live[k]) {
            const int qid = (int)(e[k].y & 0xFFFFu);
            // open addressing on the query id; a full table falls back to a direct atomic below
            int h = (int)(((uint32_t)qid * 2654435761u) >> 23);          // 9 bits
            for (int probe = 0; probe < COLLECT_SLOTS; probe++) {
                const int prev = atomicCAS(&key[h], -1, qid);
                if (prev == -1 || prev == qid) { slot[k] = h; break; }
                h = (h + 1) & (COLLECT_SLOTS - 1);
            }
            if (slot[k] >= 0) rank[k] = atomicAdd(&cnt[slot[k]], 1u);
        }
    }
    __syncthreads();
    if (tid < COLLECT_SLOTS && cnt[tid] > 0) base[tid] = atomicAdd(&a.surv_cnt[key[tid]], cnt[tid]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < COLLECT_EPT; k++) {
        if (live[k]) {
            const uint32_t qid = e[k].y & 0xFFFFu;
            const uint32_t pos = slot[k] >= 0 ? base[slot[k]] + rank[k] : atomicAdd(&a.surv_cnt[qid], 1u);
            if (pos < (uint32_t)a.surv_cap)
                a.surv_buf[(size_t)qid * a.surv_cap + pos] = ((uint64_t)(e[k].y >> 16) << 48) | e[k].x;
            else if (pos < SURV_CAP_MAX) {              // rare: see LogSpill
                const LogSpill spill = log_spill(a, (uint32_t)qid);
                const uint32_t at = atomicAdd(spill.count, 1u);
                if (at < spill.room) spill.ent[at] = e[k];
            }
        }
    }
    __syncthreads();                                    // the tables are reused for the next chunk
    }
}

// Per query with at most `cap` survivors (the usual case): one wave resolves them (id,
// duplicate rule of the miscellaneous area), sorts them by (score, id) in its own LDS region and
// writes the bigK smallest.  No workgroup barrier is used: a wave only touches its own region, and
// LDS operations of one wave complete in issue order.
#define SELW_STRIKE_MAX 8           // ties beyond bigK that are struck out one by one; more: a full sort
template <int NU>
static __device__ __forceinline__ uint32_t selw_cut(const uint64_t (&mine)[SELW_CAP_MAX / 64], uint32_t k)
{
    uint32_t cut = 0;
    for (int bit = 15; bit >= 0; bit--) {
        const uint32_t cand = cut | (1u << bit);
        uint32_t below = 0;
#pragma unroll
        for (int u = 0; u < NU; u++) below += (uint32_t)__popcll(__ballot((uint32_t)(mine[u] >> 32) < cand));
        if (below < k) cut = cand;
    }
    return cut;
}

__global__ __launch_bounds__(WG) void select_wave_kernel(IndexView v, MfmaScanArgs a, int cap)
{
    extern __shared__ __align__(16) uint64_t selw_keys[];      // [WG / 64][cap]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t q = (int64_t)blockIdx.x * (WG / 64) + wave;
    if (q >= a.nq) return;
    // the first 256 slots of the query's buffer (it has at least 1024) are requested together
    // with the count; slots beyond the count hold stale bits and are replaced below
    const uint64_t *sb = a.surv_buf + (size_t)q * a.surv_cap;
    uint64_t e_first[4];
#pragma unroll
    for (int u = 0; u < 4; u++) e_first[u] = sb[64 * u + lane];
    const uint32_t n = a.surv_cnt[q];
    // (queries that this kernel leaves to the two kernels behind it go on a list each, so that those
    // kernels, which normally have nothing to do, are a few workgroups looking at a count)
    bool redo_it = n > SURV_CAP_MAX || *a.log_overflow != 0u;
    if (!redo_it && n > (uint32_t)a.surv_cap) {
        const LogSpill spill = log_spill(a, (uint32_t)q);
        redo_it = *spill.count > spill.room;
    }
    if (redo_it) {
        if (lane == 0) {
            a.flags[q] = 1;                 // redone by the exact kernel
            uint32_t *redo = a.work + 1 + a.nq;
            redo[1 + atomicAdd(&redo[0], 1u)] = (uint32_t)q;
        }
        return;
    }
    if (n > (uint32_t)cap) {                // the workgroup-wide select's case
        if (lane == 0) a.work[1 + atomicAdd(&a.work[0], 1u)] = (uint32_t)q;
        return;
    }
    if (lane == 0) a.flags[q] = 0;
    uint64_t *keys = selw_keys + (size_t)wave * cap;
    const uint32_t *bm = a.bitmap + (size_t)q * a.bmwords;
    for (uint32_t i0 = 0; i0 < n; i0 += 256) {
        uint64_t e[4];
        uint32_t id[4], Lb[4];
        int o[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint32_t i = i0 + 64 * u + lane;
            if (i0 == 0) e[u] = i < n ? e_first[u] : 0ull;      // slot 0 of block 0: read and discarded
            else e[u] = sb[i < n ? i : n - 1];
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint2 it = v.idtag[(uint32_t)e[u]];
            Lb[u] = (uint32_t)v.blk_list[(uint32_t)e[u] >> 5];      // the list that stores the block
            id[u] = it.x;
            o[u] = (int)it.y;
        }
        uint32_t bw[4];                     // the tags' probe-bitmap words, all fetched together
#pragma unroll
        for (int u = 0; u < 4; u++) bw[u] = bm[o[u] >= 0 ? o[u] >> 5 : 0];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint32_t i = i0 + 64 * u + lane;
            // a tagged item sits in a miscellaneous block, which is only ever scanned through the
            // list that stores it
            const uint32_t score = (uint32_t)(e[u] >> 48), L = Lb[u];
            bool keep = id[u] != RAIRS_EMPTY_ID;
            // RemoveVectorIfVisited: the item was already taken from list o
            if (keep && o[u] >= 0 && (uint32_t)o[u] < L && ((bw[u] >> (o[u] & 31)) & 1u)) keep = false;
            if (i < n) keys[i] = keep ? (((uint64_t)score << 32) | id[u]) : ~0ull;
        }
    }
    wave_lds_sync();
    // Only entries up to the score of the bigK-th best need sorting: take the kept keys back into
    // registers, find that score by bisection on its 16 bits, and pack the entries up to it.
    uint64_t mine[SELW_CAP_MAX / 64];
#pragma unroll
    for (int u = 0; u < SELW_CAP_MAX / 64; u++) {
        mine[u] = ~0ull;
        if (64 * u < (int)n) {                          // uniform
            const uint32_t i = 64 * u + lane;
            if (i < n) mine[u] = keys[i];
        }
    }
    // largest t with fewer than bigK scores below it (over the rows of 64 that hold entries)
    const uint32_t cut = n <= 128   ? selw_cut<2>(mine, (uint32_t)a.refine_k)
                         : n <= 256 ? selw_cut<4>(mine, (uint32_t)a.refine_k)
                         : n <= 512 ? selw_cut<8>(mine, (uint32_t)a.refine_k)
                                    : selw_cut<SELW_CAP_MAX / 64>(mine, (uint32_t)a.refine_k);
    // (dropped entries carry score 0xFFFFFFFF and are never below a candidate; with fewer than bigK
    // kept entries cut ends at 0xFFFF and everything kept is packed)
    wave_lds_sync();                                    // every lane has its keys in registers
    uint32_t m = 0;
#pragma unroll
    for (int u = 0; u < SELW_CAP_MAX / 64; u++) {
        if (64 * u < (int)n) {
            const bool in = (uint32_t)(mine[u] >> 32) <= cut;
            const unsigned long long bal = __ballot(in);
            if (in) keys[m + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull))] = mine[u];
            m += (uint32_t)__popcll(bal);
        }
    }
    // The whole search does not need the candidates in order (refine orders by exact distance):
    // of the m entries up to the cut all but m - bigK are results, and those few -- entries that
    // tie on the cut's score -- are struck out largest (score, id) first.
    if (a.any_order && (int)m - a.refine_k <= SELW_STRIKE_MAX) {
        wave_lds_sync();
        for (int extra = (int)m - a.refine_k; extra > 0; extra--) {
            uint64_t mine_max = 0ull;
            for (int i = lane; i < (int)m; i += 64) {
                const uint64_t x = keys[i];
                if (x != ~0ull && x > mine_max) mine_max = x;
            }
            const uint64_t largest = ~wave_min_u64(~mine_max);
            for (int i = lane; i < (int)m; i += 64)
                if (keys[i] == largest) keys[i] = ~0ull;     // keys are distinct: one lane, one slot
            wave_lds_sync();
        }
        uint32_t out = 0;
        for (int i0 = 0; i0 < (int)m; i0 += 64) {
            const int i = i0 + lane;
            const uint64_t key = i < (int)m ? keys[i] : ~0ull;
            const bool ok = key != ~0ull;
            const unsigned long long bal = __ballot(ok);
            if (ok) {
                const uint32_t pos = out + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
                a.cand_ids[(size_t)q * a.refine_k + pos] = (int64_t)(uint32_t)key;
                if (a.cand_score) a.cand_score[(size_t)q * a.refine_k + pos] = (int32_t)(key >> 32);
            }
            out += (uint32_t)__popcll(bal);
        }
        for (int i = (int)out + lane; i < a.refine_k; i += 64) {   // fewer than bigK entries exist
            a.cand_ids[(size_t)q * a.refine_k + i] = -1;
            if (a.cand_score) a.cand_score[(size_t)q * a.refine_k + i] = -1;
        }
        return;
    }
    const int n2 = next_pow2(m < 2 ? 2 : (int)m);
    for (int i = (int)m + lane; i < n2; i += 64) keys[i] = ~0ull;
    wave_lds_sync();
    wave_bitonic_sort_lds(keys, n2, lane);
    for (int i = lane; i < a.refine_k; i += 64) {
        const uint64_t key = i < n2 ? keys[i] : ~0ull;
        const bool ok = key != ~0ull;
        a.cand_ids[(size_t)q * a.refine_k + i] = ok ? (int64_t)(uint32_t)key : -1;
        if (a.cand_score) a.cand_score[(size_t)q * a.refine_k + i] = ok ? (int32_t)(key >> 32) : -1;
    }
}

// (Queries with more survivors than a wave holds are left on a list for the workgroup-wide select,
// select_wg.h, which runs in the launch behind this one together with the exact redo.)

// ---- the same scan with the tile's tables in LDS -----------------------
//
// For tables too large for registers (M = 240: 37.5 KB per half wave of queries) the eight waves of a workgroup
// share one tile.  Its tables sit in LDS as [instruction][16-byte half][lane] (of sixteen dwords of codes
// the last one's in registers, or 160 KB would not do), the unit's blocks go to the waves in groups of
// four, and a wave's instruction operand is read once for its group: two LDS reads to four matrix instructions, 16 of the
// LDS's cycles for 132 of a SIMD's, so four SIMDs keep it half busy.  (Units of few blocks are dealt in groups of
// two.)  Codes come a pair of dwords ahead.  Survivors, bounds and the log work as in scan_mfma_kernel.
// The dense instruction with one-hot rows from LDS, two reads each, took all of the LDS's time: 200,000 x 960,
// M = 240, 1,000 queries, 45 probes: 865 us, now 570.
#define LDSK_WAVES 8
// matrix instructions a block whose tables are in LDS
static __host__ __device__ __forceinline__ int ldsk_lds_ops(int nd) { return 5 * (nd < 16 ? nd : 15); }
template <bool LAST_IN_REGS>                           // sixteen dwords of codes
__global__ __launch_bounds__(64 * LDSK_WAVES, 2) void scan_mfma_lds_kernel(IndexView v, MfmaScanArgs a)
{
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    __shared__ SegEntry segs_s[UNIT_MAX_SEGS];
    __shared__ uint32_t s_unit;
    const int ND = v.nd, ops = ldsk_lds_ops(ND);
    v4i *Bl = (v4i *)dyn_lds;                           // [ops][2][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), half = lane >> 5, j = lane & 31;
    SmallStageQueue &sq = ((SmallStageQueue *)(dyn_lds + (size_t)ops * 2048))[wave];
    int nstaged = 0;
    RefreshPace pace = {REFRESH_GAP_MIN, REFRESH_GAP_MIN - 1u, 0u};
    const uint32_t nunits = (uint32_t)a.toff[v.nlist];
    if (nunits == 0u) return;                          // uniform; nothing was written
    LogCursor lc;
    lc.chunk = blockIdx.x * LDSK_WAVES + wave;         // (a workgroup without a unit never writes)
    lc.used = 0;
    for (bool first = true;; first = false) {
        __syncthreads();                               // everyone is done with the previous tile
        if (threadIdx.x == 0) s_unit = first ? blockIdx.x : atomicAdd(a.next_task, 1u);
        __syncthreads();
        const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_unit);
        if (u >= nunits) break;                        // uniform for the workgroup; the counter only grows
        const int32_t *rec = a.unit_rec + (size_t)u * UNIT_REC_WORDS;
        const int tile = rec[1], seg0 = rec[2], nseg = rec[3] - seg0;      // nseg <= UNIT_MAX_SEGS
        const int q_at = rec[4] + tile * 32, qn = rec[5] - tile * 32;
        if ((int)threadIdx.x < nseg) segs_s[threadIdx.x] = v.segs[seg0 + threadIdx.x];
        const int qid = j < qn ? a.qlist[q_at + j] : -1;
        const uint32_t q0 = (uint32_t)(qid >= 0 ? qid : 0);     // (an absent column takes query 0's tables and never passes)
        const char *row = (const char *)a.tables + (size_t)q0 * scan_tables_stride(ND);
        const int above = *(const int *)(row + ND * 320);
        const char *mine = row + half * 160;
        for (int t = wave; t < ops; t += LDSK_WAVES) {
            const char *p = mine + t / 5 * 320 + t % 5 * 32;
            const v4i x = *(const v4i *)p, y = *(const v4i *)(p + 16);
            Bl[t * 128 + lane] = x;
            Bl[t * 128 + 64 + lane] = y;
        }
        v8i Br[LAST_IN_REGS ? 5 : 1];
        if (LAST_IN_REGS)
#pragma unroll
            for (int g = 0; g < 5; g++) {
                const char *p = mine + 15 * 320 + g * 32;
                const v4i x = *(const v4i *)p, y = *(const v4i *)(p + 16);
                Br[LAST_IN_REGS ? g : 0] = (v8i){x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
            }
        const int32_t *bq = a.bound + q0;
        const uint32_t *bmq = a.bitmap + (size_t)q0 * a.bmwords;
        __syncthreads();
        int nblocks = 0;
        for (int i = 0; i < nseg; i++) nblocks += segs_s[i].nblk;
        nblocks = __builtin_amdgcn_readfirstlane(nblocks);
        uint32_t scored = 0;                           // items this lane's query was scored against, by this wave
        int wseg = 0, wbase = 0;                       // run that holds the next block, blocks before it
        auto group_of = [&](auto width, int first_block) __attribute__((always_inline)) {
            constexpr int N = decltype(width)::value;
            int blk[N], negth[N];                      // (uniform; per lane)
            uint32_t cmask[N], rows[N];                // (uniform; per lane)
            const int bound = __hip_atomic_load(bq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int i = 0; i < N; i++) {
                const bool there = first_block + i < nblocks;              // (behind the last block: the last one again, nobody passes)
                const int at = there ? first_block + i : nblocks - 1;
                while (at >= wbase + segs_s[wseg].nblk) { wbase += segs_s[wseg].nblk; wseg++; }
                const SegEntry se = segs_s[wseg];
                const int b = at - wbase;
                blk[i] = __builtin_amdgcn_readfirstlane(se.blk_begin + b);
                // cell (owner, L) is scored through list `owner` for queries that probe it
                const uint32_t ob = bmq[se.owner >= 0 ? se.owner >> 5 : 0];
                const bool live = there && qid >= 0 && !(se.owner >= 0 && ((ob >> (se.owner & 31)) & 1u));
                negth[i] = live ? -(bound + above + 1) : ACC_NEVER;
                const uint2 masks = v.bmask[blk[i]];
                cmask[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)masks.x);
                scored += live ? (uint32_t)__popc(masks.y) : 0u;           // the block is contracted now: its DCO
                // the list's last block: drop rows whose slot holds no item
                rows[i] = b == se.nblk - 1 && se.tail_valid < 32 ? rows_below(se.tail_valid - 4 * half) : 0xFFFFu;
            }
            v16i acc[N];
#pragma unroll
            for (int i = 0; i < N; i++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc[i][r] = negth[i];
            uint32_t c[N][2], n[N][2];
            auto codes = [&](uint32_t (&to)[N][2], int w) {
#pragma unroll
                for (int i = 0; i < N; i++) {
                    const uint32_t *p = at32(v.codes + ((size_t)blk[i] * ND + w) * 64, (uint32_t)lane * 4u);
                    to[i][0] = p[0];
                    to[i][1] = p[w + 1 < ND ? 64 : 0];  // uniform
                }
            };
            codes(c, 0);
            v4i b0 = Bl[lane], b1 = Bl[64 + lane];
            const v4i one = {SEL_FIRST, SEL_FIRST, SEL_FIRST, SEL_FIRST}, two = {SEL_SECOND, SEL_SECOND, SEL_SECOND, SEL_SECOND};
            auto five = [&](const v4i &slot, const uint32_t (&s)[N][5], int t) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < 5; g++) {
                    const v8i B = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
                    const int tn = t + g + 1 < ops ? t + g + 1 : ops - 1;
                    b0 = Bl[tn * 128 + lane];
                    b1 = Bl[tn * 128 + 64 + lane];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < N; i++) acc[i] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(slot, B, acc[i], (int)s[i][g], 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            int w = 0;
#pragma unroll 1                                       // (laid out fourteen times it spills)
            for (; w + 2 <= (LAST_IN_REGS ? 14 : ND); w += 2) {
                codes(n, w + 2 < ND ? w + 2 : w);
                uint32_t s[N][5];
#pragma unroll
                for (int i = 0; i < N; i++) select_words_pair(c[i][0], c[i][1], s[i]);
                five(one, s, 5 * w);
                five(two, s, 5 * w + 5);
#pragma unroll
                for (int i = 0; i < N; i++) { c[i][0] = n[i][0]; c[i][1] = n[i][1]; }
            }
            if (LAST_IN_REGS || w < ND) {              // uniform: the last pair, or an odd last dword
                uint32_t s[N][5];
#pragma unroll
                for (int i = 0; i < N; i++) {
                    if (LAST_IN_REGS) select_words_pair(c[i][0], c[i][1], s[i]);
                    else select_words_one(c[i][0], s[i]);
                }
                five(one, s, 5 * w);
                if (LAST_IN_REGS)
#pragma unroll
                    for (int g = 0; g < 5; g++)
#pragma unroll
                        for (int i = 0; i < N; i++) acc[i] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(two, Br[LAST_IN_REGS ? g : 0], acc[i], (int)s[i][g], 0, 0);
            }
#pragma unroll
            for (int i = 0; i < N; i++) {
                uint32_t pm = negative_rows(acc[i]) & rows[i];
                for (;;) {
                    const unsigned long long mask = __builtin_amdgcn_ballot_w64(pm != 0u);
                    if (mask == 0ull) break;
                    const int r = __builtin_ctz(pm | 0x10000u);
                    const int sc = select_row(acc[i], r & 15) - negth[i] - above;      // the row's score
                    const uint32_t item = 8u * (uint32_t)(r >> 2) + (uint32_t)(r & 3) + 4u * half;
                    if (pm != 0u)
                        sq.ent[nstaged + lanes_below(mask)] = make_uint2(((uint32_t)blk[i] * 32u + item) | (((cmask[i] >> (item & 31u)) & 1u) << 31),
                                                                         ((uint32_t)sc << 16) | (uint32_t)qid);
                    pm &= pm - 1u;
                    nstaged += __popcll(mask);
                    if (nstaged > SmallStageQueue::CAP - 64) {
                        stage_flush(a, sq, nstaged, lane, lc, pace);
                        nstaged = 0;
                    }
                }
            }
        };
        // groups of four where that gives all waves something, else of two
        if (nblocks >= 3 * LDSK_WAVES)
            for (int b = 4 * wave; b < nblocks; b += 4 * LDSK_WAVES) group_of(std::integral_constant<int, 4>(), b);
        else
            for (int b = 2 * wave; b < nblocks; b += 2 * LDSK_WAVES) group_of(std::integral_constant<int, 2>(), b);
        if (nstaged >= 32) {
            stage_flush(a, sq, nstaged, lane, lc, pace);
            nstaged = 0;
        }
        if (a.dco && half == 0 && scored) atomicAdd(&a.dco[q0], (unsigned long long)scored);
    }
    if (nstaged > 0) stage_flush(a, sq, nstaged, lane, lc, pace);
    // (a wave that never had a unit wrote nothing, and the chunk of its index may be another wave's)
    if (lane == 0 && lc.used > 0 && lc.chunk < (uint32_t)a.log_chunks) a.chunk_fill[lc.chunk] = lc.used;
}

// ---- the bound sample on the matrix cores -----------------------------------------------------
//
// The sample that seeds a query's bound is the head of its first probed list.  Queries that share
// a first list are scored together: one workgroup groups the batch by first list, then a wave
// scores the head of a list for a tile of up to 32 such queries with the scan's matrix
// instruction, and writes every (query, item) score out for the rank kernel.  About ten queries
// share a first list in a 10,000-query batch over 1,024 lists, so the tiles are a third full --
// still several times cheaper than one table lookup per code on the vector units.
#define SAMPLE_GROUP_MAX_NLIST 8192
#define SAMPLE_GROUP_MIN_QUERIES 1024
#define SG_HELD 12

// s_off: exclusive prefix over lists of the queries whose first probe is the list; s_q: those
// queries, list by list; s_toff: exclusive prefix of tiles (32 queries); s_tiles: list of every tile.
__global__ __launch_bounds__(1024) void sample_group_kernel(const int32_t *__restrict__ probe_ids,
                                                            int64_t nq, int nprobe, int nlist,
                                                            int32_t *s_off, int32_t *s_toff,
                                                            int32_t *s_q, int32_t *s_tiles)
{
    extern __shared__ int32_t sg_lds[];                // [nlist] counts, then cursors; [nlist] offsets
    __shared__ int sc[16], st[16];
    int32_t *cnt_s = sg_lds, *off_s = sg_lds + nlist;
    const int tid = threadIdx.x;
    for (int i = tid; i < nlist; i += 1024) cnt_s[i] = 0;
    __syncthreads();
    // the first SG_HELD queries of a thread stay in registers: their loads are all in flight at
    // once and the second pass does not fetch them again
    int myL[SG_HELD];
#pragma unroll
    for (int k = 0; k < SG_HELD; k++) {
        const int64_t q = tid + 1024 * k;
        int L = q < nq ? probe_ids[q * nprobe] : -1;
        myL[k] = L >= 0 && L < nlist ? L : -1;
    }
#pragma unroll
    for (int k = 0; k < SG_HELD; k++)
        if (myL[k] >= 0) atomicAdd(&cnt_s[myL[k]], 1);
    for (int64_t q = tid + 1024 * SG_HELD; q < nq; q += 1024) {
        const int L = probe_ids[q * nprobe];
        if (L >= 0 && L < nlist) atomicAdd(&cnt_s[L], 1);
    }
    __syncthreads();
    const int per = (nlist + 1023) / 1024;
    const int lo = tid * per < nlist ? tid * per : nlist;
    const int hi = lo + per < nlist ? lo + per : nlist;
    int c = 0, t = 0;
    for (int L = lo; L < hi; L++) {
        const int n = cnt_s[L];
        c += n;
        t += (n + 31) >> 5;
    }
    // exclusive prefixes of (c, t) over the 1024 threads: a scan inside each wave, then the totals
    // of the 16 waves through LDS
    const int lane = tid & 63, wave = tid >> 6;
    int ci = c, ti = t;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_up(ci, off), y = __shfl_up(ti, off);
        if (lane >= off) { ci += x; ti += y; }
    }
    if (lane == 63) { sc[wave] = ci; st[wave] = ti; }
    __syncthreads();
    int cw = 0, tw = 0, call = 0, tall = 0;
#pragma unroll
    for (int w2 = 0; w2 < 16; w2++) {
        const int x = sc[w2], y = st[w2];
        if (w2 < wave) { cw += x; tw += y; }
        call += x;
        tall += y;
    }
    int cb = cw + ci - c, tb = tw + ti - t;
    for (int L = lo; L < hi; L++) {
        const int n = cnt_s[L], nt = (n + 31) >> 5;
        s_off[L] = cb;
        off_s[L] = cb;
        s_toff[L] = tb;
        for (int u = 0; u < nt; u++) s_tiles[tb + u] = L;
        cb += n;
        tb += nt;
    }
    if (tid == 0) {
        s_off[nlist] = call;
        s_toff[nlist] = tall;
    }
    __syncthreads();
    for (int i = tid; i < nlist; i += 1024) cnt_s[i] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SG_HELD; k++)
        if (myL[k] >= 0) s_q[off_s[myL[k]] + atomicAdd(&cnt_s[myL[k]], 1)] = tid + 1024 * k;
    for (int64_t q = tid + 1024 * SG_HELD; q < nq; q += 1024) {
        const int L = probe_ids[q * nprobe];
        if (L >= 0 && L < nlist) s_q[off_s[L] + atomicAdd(&cnt_s[L], 1)] = (int32_t)q;
    }
}

// scores[q][b * 32 + i] = score of item i of block b of the first `sample_blocks` own blocks of
// q's first list (0xFFFF: the slot holds no item); blocks the list does not have are not written.
template <int ND>
__global__ __launch_bounds__(WG) void sample_mfma_kernel(IndexView v, const uint8_t *__restrict__ lut,
                                                            int sample_blocks,
                                                            const int32_t *__restrict__ s_off,
                                                            const int32_t *__restrict__ s_toff,
                                                            const int32_t *__restrict__ s_q,
                                                            const int32_t *__restrict__ s_tiles,
                                                            uint16_t *__restrict__ scores)
{
    const int lane = threadIdx.x & 63, g = lane >> 5, j = lane & 31;
    const uint32_t ntiles = (uint32_t)s_toff[v.nlist];
    const uint32_t gwave = blockIdx.x * (WG / 64) + (threadIdx.x >> 6), nwaves = gridDim.x * (WG / 64);
    v8i B[5 * ND];
    for (uint32_t u = gwave; u < ntiles; u += nwaves) {
        const int L = __builtin_amdgcn_readfirstlane(s_tiles[u]);
        const ListEntry le = v.lists[L];
        const int tile = (int)u - __builtin_amdgcn_readfirstlane(s_toff[L]);
        const int base = s_off[L], n = s_off[L + 1] - base;
        const int qi = tile * 32 + j;
        const int qid = qi < n ? s_q[base + qi] : -1;
        const int above = load_byte_tables<ND>(lut, (uint32_t)(qid >= 0 ? qid : 0), v.M, g, B);
        int cnt = le.shared_cnt + le.misc_cnt;
        cnt = cnt < sample_blocks ? cnt : sample_blocks;
        if (cnt <= 0) continue;                        // uniform for the wave
        const uint32_t *cp = v.codes + (size_t)le.blk_begin * ND * 64 + lane;
        uint32_t cn[ND];
#pragma unroll
        for (int w = 0; w < ND; w++) cn[w] = cp[w * 64];
        uint32_t vmn = v.vmask[le.blk_begin];
        uint16_t *row = scores + (size_t)(qid >= 0 ? qid : 0) * sample_blocks * 32;
        for (int b = 0; b < cnt; b++) {
            uint32_t c[ND];
#pragma unroll
            for (int w = 0; w < ND; w++) c[w] = cn[w];
            const uint32_t vm = vmn;
            if (b + 1 < cnt) {
#pragma unroll
                for (int w = 0; w < ND; w++) cn[w] = cp[(size_t)(b + 1) * ND * 64 + w * 64];
                vmn = v.vmask[le.blk_begin + b + 1];
            }
            // the accumulators end as the scores themselves (below 2^16)
            v16i acc;
#pragma unroll
            for (int r = 0; r < 16; r++) acc[r] = -above;
            contract_block<ND>(c, B, acc);
            // acc[r]: item 8 * (r / 4) + 4 * g + r % 4, query column j: four consecutive items
            // per group of four registers, written as one 8-byte store.  A block whose 32 slots
            // all hold items (every block but a list's last, unless items were deleted) needs no
            // look at the slot mask: two scores to a word and out.
            if (qid >= 0) {
                if (vm == 0xFFFFFFFFu) {               // uniform
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        *(uint2 *)(row + b * 32 + 8 * k + 4 * g) =
                            make_uint2((uint32_t)acc[4 * k] | ((uint32_t)acc[4 * k + 1] << 16),
                                       (uint32_t)acc[4 * k + 2] | ((uint32_t)acc[4 * k + 3] << 16));
                } else {
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        const int item = 8 * k + 4 * g;
                        uint32_t sc4[4];
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            sc4[e] = ((vm >> (item + e)) & 1u) ? (uint32_t)acc[4 * k + e] : 0xFFFFu;
                        *(uint2 *)(row + b * 32 + item) = make_uint2(sc4[0] | (sc4[1] << 16), sc4[2] | (sc4[3] << 16));
                    }
                }
            }
        }
    }
}

bool rairs_sample_scores_supported(const IndexView &v, int64_t nq)
{
    return v.M == 16 * v.nd && (v.nd == 1 || v.nd == 3 || v.nd == 4) && v.nlist <= SAMPLE_GROUP_MAX_NLIST &&
           nq >= SAMPLE_GROUP_MIN_QUERIES;
}

int rairs_launch_sample_group(const IndexView &v, const int32_t *probe_ids, int nprobe, int64_t nq,
                              int32_t *s_off, int32_t *s_toff, int32_t *s_q, int32_t *s_tiles,
                              hipStream_t s)
{
    if (!rairs_sample_scores_supported(v, nq)) {
        rairs_set_error("matrix-core sample not available for this index or batch");
        return RAIRS_EINVAL;
    }
    const size_t lds = (size_t)2 * v.nlist * 4;
    if (lds > 32 * 1024)
        RAIRS_HIP(hipFuncSetAttribute((const void *)sample_group_kernel,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(sample_group_kernel, dim3(1), dim3(1024), lds, s, probe_ids, nq, nprobe, v.nlist,
                       s_off, s_toff, s_q, s_tiles);
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}

int rairs_launch_sample_scores(const IndexView &v, const uint8_t *lut, int sample_blocks, int64_t nq,
                               const int32_t *s_off, const int32_t *s_toff, const int32_t *s_q,
                               const int32_t *s_tiles, uint16_t *scores, hipStream_t s)
{
    if (!rairs_sample_scores_supported(v, nq) || sample_blocks < 1 || sample_blocks > RAIRS_SAMPLE_MAX_BLOCKS) {
        rairs_set_error("matrix-core sample not available for this index or batch");
        return RAIRS_EINVAL;
    }
    const int64_t tiles_max = nq / 32 + v.nlist;
    unsigned grid = (unsigned)((tiles_max + WG / 64 - 1) / (WG / 64));
    if (grid > 512u) grid = 512u;
#define SAMPLE_MFMA(ND_)                                                                          \
    hipLaunchKernelGGL(sample_mfma_kernel<ND_>, dim3(grid), dim3(WG), 0, s, v, lut, sample_blocks, s_off, \
                       s_toff, s_q, s_tiles, scores)
    switch (v.nd) {
    case 1: SAMPLE_MFMA(1); break;
    case 3: SAMPLE_MFMA(3); break;
    default: SAMPLE_MFMA(4); break;
    }
#undef SAMPLE_MFMA
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}

bool rairs_mfma_supported(const IndexView &v) { return v.T >= 1 && v.nd <= 16; }

// Up to 64 sub-quantizers the tables fit into registers.  Which kernel is faster then is more a matter of load than of M: a
// wave with a tile of its own contracts faster, eight waves that share one work a crowded unit's survivors off sooner and are
// at fewer units at once, so bounds come earlier.  At two dwords of codes the second weighs more, from three on the first; at
// sixteen sub-quantizers it is about even, and the smaller bigK counts.  (us in registers / in LDS.  10,000 queries, 32 probes, bigK =
// 10: M = 16 771 / 910, 32 428 / 565, 48 409 / 556, 64 489 / 670; 10,000, 16, 100: M = 16 990 / 1,030, 24 1,253 / 1,103 and 1,193 / 1,265, 32
// 488 / 600, 48 463 / 532; 3,000, 16, 40: M = 16 418 / 406 and 346 / 270, 24 597 / 472 and 453 / 512, 32 265 / 241, 48 246 / 229, 64 281 / 256;
// 300, 16, 100: M = 16 277 / 330, 24 430 / 421 and 324 / 405, 48 190 / 200; 2,000, 8, 40: M = 8 227 / 188, 16 311 / 289, 24 399 / 331, 32 199 / 191.)
bool rairs_mfma_reg_tables(const IndexView &v) { return v.nd <= 4 && (v.nd >= 3 || v.M == 16); }

// persistent grids: 256 compute units x 2 workgroups of 4 waves with the tables in registers; one
// workgroup of LDSK_WAVES waves per compute unit with the tables in LDS
static void scan_launch_shape(const IndexView &v, bool *reg_tables, unsigned *grid)
{
    *reg_tables = rairs_mfma_reg_tables(v);
    *grid = *reg_tables ? 512u : 256u;
}

// Half of the chunks of the survivor log beyond those for the entries themselves, when the pass has at most `units` units.
int64_t rairs_scan_log_waves(const IndexView &v, int64_t units)
{
    // At most 2,048 waves hold a chunk, whichever kernel.  That many and once more are for those with three shapes, and twice that
    // for the others (sixteen waves a workgroup once): what waves leave is where survivors beyond their buffers go, and
    // programs size workspaces by it, which the few-query search has to fit as well.
    if (v.M == 16 || v.M == 48 || v.M == 64) return units < 2048 ? units : 2048;
    return (units < 256 ? units : 256) * 16;
}

int rairs_launch_group(const IndexView &v, const MfmaScanArgs &a, hipStream_t s)
{
    const int np = a.nprobe - a.p_first;
    if (np <= 0) return RAIRS_OK;
    bool reg_tables;
    unsigned gridx;
    scan_launch_shape(v, &reg_tables, &gridx);
    const uint32_t nwaves = gridx * (reg_tables ? WG / 64 : LDSK_WAVES);
    // who starts on a unit of its own index, and with how many waves (see log_first_free)
    const uint32_t starters = reg_tables ? nwaves : gridx, waves_each = reg_tables ? 1u : (uint32_t)LDSK_WAVES;
    if (a.log_chunks < 2) {
        rairs_set_error("survivor log of %d chunks", a.log_chunks);
        return RAIRS_EINVAL;
    }
    const int64_t pairs = a.nq * np;
    int64_t nz = v.nlist > a.nq ? v.nlist : a.nq;
    nz = nz > a.log_chunks ? nz : a.log_chunks;
    const unsigned zero_wgs = (unsigned)((nz + WG - 1) / WG), table_wgs = (unsigned)((a.nq + WG / 64 - 1) / (WG / 64));
    hipLaunchKernelGGL(lm_begin_kernel, dim3(zero_wgs + table_wgs), dim3(WG), 0, s, (int)zero_wgs, v, a, reg_tables ? 2 * nwaves : gridx);
    const bool lds_group = v.nlist <= LM_LDS_NLIST;
    const int qb = LM_PAIRS / np > 0 ? LM_PAIRS / np : 1;
    const unsigned lgrid = (unsigned)((a.nq + qb - 1) / qb);
    if (lds_group) {
        if ((size_t)v.nlist * 4 > 48 * 1024)
            RAIRS_HIP(hipFuncSetAttribute((const void *)lm_count_lds_kernel,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, v.nlist * 4));
        hipLaunchKernelGGL(lm_count_lds_kernel, dim3(lgrid), dim3(256), (size_t)v.nlist * 4, s,
                           a.probe_ids, a.nq, a.nprobe, a.p_first, v.nlist, a.lcount, qb);
    } else
        hipLaunchKernelGGL(lm_count_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, s,
                           a.probe_ids, a.nq, a.nprobe, a.p_first, v.nlist, a.lcount);
    if (lds_group) {
        const size_t lds = ((size_t)2 * v.nlist + 1) * 4;
        if (lds > 48 * 1024)
            RAIRS_HIP(hipFuncSetAttribute((const void *)lm_fill_lds_kernel,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(lm_fill_lds_kernel, dim3(lgrid + LM_UNIT_WGS), dim3(256), lds, s, v, a.probe_ids, a.nq,
                           a.nprobe, a.p_first, a.lcount, a.loff, a.lcursor, a.qlist, qb, a.toff,
                           a.unit_parts, a.unit_tail_from, a.unit_rec, a.log_cursor, starters, waves_each, (uint32_t)a.split_max);
    } else {
        hipLaunchKernelGGL(lm_prefix_kernel, dim3(1), dim3(1024), 0, s, v, a.lcount, a.loff, a.lcursor,
                           a.toff, a.unit_parts, a.unit_tail_from, a.unit_rec, a.log_cursor, starters, waves_each, (uint32_t)a.split_max);
        hipLaunchKernelGGL(lm_units_kernel, dim3((unsigned)((v.nlist + 255) / 256)), dim3(256), 0, s, v, a.lcount,
                           a.loff, a.toff, a.unit_parts, a.unit_tail_from, a.unit_rec);
        hipLaunchKernelGGL(lm_fill_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, s,
                           a.probe_ids, a.nq, a.nprobe, a.p_first, v.nlist, a.loff, a.lcursor, a.qlist);
    }
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}

size_t rairs_scan_tables_bytes(const IndexView &v, int64_t nq) { return (size_t)nq * scan_tables_stride(v.nd); }

int rairs_launch_scan_mfma(const IndexView &v, const MfmaScanArgs &a, hipStream_t s, hipEvent_t *ev)
{
    if (a.nprobe - a.p_first <= 0) return RAIRS_OK;
    if (a.surv_cap > SURV_CAP_MAX) {
        rairs_set_error("survivor capacity %d above %d", a.surv_cap, SURV_CAP_MAX);
        return RAIRS_EINVAL;
    }
    if (a.nq > 65536) {                                // a log entry has 16 bits for the query of the pass
        rairs_set_error("a scan pass takes at most 65536 queries, got %lld", (long long)a.nq);
        return RAIRS_EINVAL;
    }
    bool reg_tables;
    unsigned gridx;
    scan_launch_shape(v, &reg_tables, &gridx);
    const dim3 grid(gridx);
    if (ev) RAIRS_HIP(hipEventRecord(ev[0], s));
    switch (reg_tables ? v.nd : 0) {
    case 1: hipLaunchKernelGGL((a.split_max > 1 ? scan_mfma_kernel<1, true> : scan_mfma_kernel<1, false>), grid, dim3(WG), 0, s, v, a); break;
    case 3: hipLaunchKernelGGL((a.split_max > 1 ? scan_mfma_kernel<3, true> : scan_mfma_kernel<3, false>), grid, dim3(WG), 0, s, v, a); break;
    case 4: hipLaunchKernelGGL((a.split_max > 1 ? scan_mfma_kernel<4, true> : scan_mfma_kernel<4, false>), grid, dim3(WG), 0, s, v, a); break;
    default: {
        const size_t lds = (size_t)ldsk_lds_ops(v.nd) * 2048 + LDSK_WAVES * sizeof(SmallStageQueue);
        const auto kernel = v.nd < 16 ? scan_mfma_lds_kernel<false> : scan_mfma_lds_kernel<true>;
        RAIRS_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kernel, grid, dim3(64 * LDSK_WAVES), lds, s, v, a);
    }
    }
    if (ev) RAIRS_HIP(hipEventRecord(ev[1], s));
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}

int rairs_launch_select(const IndexView &v, const MfmaScanArgs &a, hipStream_t s)
{
    if (final_bound_pays(a))
        hipLaunchKernelGGL(final_bound_kernel, dim3((unsigned)((a.nq + WG / 64 - 1) / (WG / 64))), dim3(WG), 0, s, a);
    hipLaunchKernelGGL(collect_kernel, dim3((unsigned)(a.log_chunks < 4096 ? a.log_chunks : 4096)),
                       dim3(COLLECT_WG), 0, s, a);
    const int cap = rairs_select_wave_cap(a.refine_k);
    hipLaunchKernelGGL(select_wave_kernel, dim3((unsigned)((a.nq + WG / 64 - 1) / (WG / 64))), dim3(WG),
                       (size_t)cap * 8 * (WG / 64), s, v, a, cap);
    RAIRS_HIP(hipGetLastError());
    return RAIRS_OK;
}
