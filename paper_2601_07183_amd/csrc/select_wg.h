// Workgroup-wide select of a query's survivors, for the queries that select_wave_kernel leaves on
// its list (more survivors than a wave holds): resolve the survivors and keep the bigK smallest
// (score, id).  A two-pass radix select on the 16-bit score finds the score of the bigK-th
// survivor; only entries up to that score are sorted.  A query's survivors beyond its buffer come
// from the spill (up to SURV_CAP_MAX in all; more than that, or a full bucket of the spill, and the wave
// kernel puts the query on the list of the exact redo instead).
#pragma once
#include "device_util.h"

// Survivors that do not fit their query's buffer go, as log entries, to the unused chunks at the end of
// the survivor log.  A buffer is sized so that one query in some ten thousand needs this where a bound
// exists, and the alternative, the exact redo, is one workgroup's walk through all lists of the query:
// 19 ms on an 8M x 128 index with 98 probes and 17 ms on 200,000 x 960 with 45, for batches of 5.8 and
// 1.2 ms.  Where lists are shorter than bigK there is no bound and whole batches come here, so the chunks
// are dealt out to the queries in buckets of SPILL_CHUNKS, counted in the fill word of their first
// chunk: a query walks only the bucket that it shares with every so-many-th other query.  (12,800
// queries, 32 probes of lists of some 50 items, 5,267 of them over: 3.9 ms with all of those redone, 15.7
// with a walk over everything that was spilled for each, 2.3 with buckets.)  A bucket holds what two to four queries can spill; a
// full one sends its queries to the redo.
#define SPILL_CHUNKS 4
struct LogSpill {
    uint2 *ent;                   // {slot, score << 16 | query of the pass}
    uint32_t *count;              // entries that wanted to go there, `room` of them did
    uint32_t room;
};
static __device__ __forceinline__ uint32_t log_chunks_used(const MfmaScanArgs &a)
{
    const uint32_t lim = *a.log_cursor;                 // chunks handed out
    return lim < (uint32_t)a.log_chunks ? lim : (uint32_t)a.log_chunks;
}
static __device__ __forceinline__ LogSpill log_spill(const MfmaScanArgs &a, uint32_t q)
{
    const uint32_t lim = log_chunks_used(a), left = (uint32_t)a.log_chunks - lim, buckets = left / SPILL_CHUNKS;
    if (left == 0) return {a.log, a.log_overflow + 1, 0u};
    const uint32_t c = buckets ? lim + q % buckets * SPILL_CHUNKS : lim;
    return {a.log + (size_t)c * RAIRS_LOG_CHUNK, a.chunk_fill + c, (buckets ? SPILL_CHUNKS : left) * RAIRS_LOG_CHUNK};
}

struct SelectShared {
    uint64_t keys[SURV_CAP_MAX];
    uint32_t hist[256];
    uint32_t prefix, need, kept;
};

// All threads of the workgroup call this together; the shared state may be reused on return.
static __device__ __forceinline__ void select_query_wg(const IndexView &v, const MfmaScanArgs &a, int wave_cap,
                                                        int64_t q, SelectShared &sh)
{
    uint64_t *keys = sh.keys;
    uint32_t *hist = sh.hist;
    const int tid = threadIdx.x;
    const uint32_t n = a.surv_cnt[q];
    if (n <= (uint32_t)wave_cap || n > SURV_CAP_MAX || *a.log_overflow != 0u) return;   // (uniform; not on the list)
    if (tid == 0) { a.flags[q] = 0; sh.kept = (uint32_t)a.surv_cap; }
    auto resolve = [&](uint32_t slot, uint32_t score) {
        uint64_t key = ~0ull;
        const uint32_t L = (uint32_t)v.blk_list[slot >> 5];
        const uint2 it = v.idtag[slot];
        const uint32_t id = it.x;
        const int o = (int)it.y;
        bool keep = id != RAIRS_EMPTY_ID;
        if (keep && o >= 0 && (uint32_t)o < L) {
            // RemoveVectorIfVisited: the item was already taken from list o
            const uint32_t wbits = a.bitmap[(size_t)q * a.bmwords + (o >> 5)];
            if ((wbits >> (o & 31)) & 1u) keep = false;
        }
        if (keep) key = ((uint64_t)score << 32) | id;
        return key;
    };
    for (int i = tid; i < (int)n && i < a.surv_cap; i += WG) {
        const uint64_t e = a.surv_buf[(size_t)q * a.surv_cap + i];
        keys[i] = resolve((uint32_t)e, (uint32_t)(e >> 48));
    }
    if (n > (uint32_t)a.surv_cap) {         // uniform: the rest of them is in the spill, among other queries' entries
        const LogSpill spill = log_spill(a, (uint32_t)q);
        const uint32_t ns = *spill.count;   // (at most spill.room, or the query would be on the other list)
        __syncthreads();
        for (uint32_t i = (uint32_t)tid; i < ns; i += WG) {
            const uint2 e = spill.ent[i];
            if ((int64_t)(e.y & 0xFFFFu) == q) keys[atomicAdd(&sh.kept, 1u)] = resolve(e.x, e.y >> 16);
        }
        __syncthreads();
    }
    // score of the bigK-th smallest kept key: radix select, high byte then low byte
    uint32_t prefix = 0, need = (uint32_t)a.refine_k;
    bool all = false;                       // fewer than bigK kept: everything is sorted
    for (int pass = 0; pass < 2 && !all; pass++) {
        const int shift = pass == 0 ? 8 : 0;
        hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < (int)n; i += WG) {
            const uint64_t key = keys[i];
            if (key != ~0ull) {
                const uint32_t sc = (uint32_t)(key >> 32);
                if (pass == 0 || (sc >> 8) == prefix) atomicAdd(&hist[(sc >> shift) & 255u], 1u);
            }
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t cum = 0;
            sh.need = 0xFFFFFFFFu;
            for (int b = 0; b < 256; b++) {
                if (cum + hist[b] >= need) { sh.prefix = (uint32_t)b; sh.need = need - cum; break; }
                cum += hist[b];
            }
        }
        __syncthreads();
        if (sh.need == 0xFFFFFFFFu) all = true;
        else { prefix = pass == 0 ? sh.prefix : ((prefix << 8) | sh.prefix); need = sh.need; }
        __syncthreads();
    }
    const uint32_t cut = all ? 0xFFFFu : prefix;          // keep scores <= cut
    // compact the kept keys with score <= cut to the front (order is irrelevant before the sort)
    if (tid == 0) sh.kept = 0;
    __syncthreads();
    uint64_t mine[SURV_CAP_MAX / WG];
    int nm = 0;
    for (int i = tid; i < (int)n; i += WG) {
        const uint64_t key = keys[i];
        if (key != ~0ull && (uint32_t)(key >> 32) <= cut) mine[nm++] = key;
    }
    __syncthreads();
    uint32_t at = nm ? atomicAdd(&sh.kept, (uint32_t)nm) : 0u;
    for (int i = 0; i < nm; i++) keys[at + i] = mine[i];
    __syncthreads();
    const int kept = (int)sh.kept;
    const int n2 = next_pow2(kept < 2 ? 2 : kept);
    for (int i = kept + tid; i < n2; i += WG) keys[i] = ~0ull;
    __syncthreads();
    bitonic_sort_lds(keys, n2);
    for (int i = tid; i < a.refine_k; i += WG) {
        const uint64_t key = i < n2 ? keys[i] : ~0ull;
        const bool ok = key != ~0ull;
        a.cand_ids[(size_t)q * a.refine_k + i] = ok ? (int64_t)(uint32_t)key : -1;
        if (a.cand_score) a.cand_score[(size_t)q * a.refine_k + i] = ok ? (int32_t)(key >> 32) : -1;
    }
    __syncthreads();                        // the keys are the next query's
}
