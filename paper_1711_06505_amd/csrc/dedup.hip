// dedup.hip -- ams_dedup: the batch's image IDs reduced to one sorted set with
// inverse index and stable occurrence order (section 4.2: requests for the
// same image are processed once; Algorithm 1: an image's gradients are
// collected in one place).
//
// Method: a stable LSD radix sort of (ID, occurrence index) over the
// ceil(log2 n_ids) significant bits, at most 8 bits per pass, then head flags
// and a scan give the unique set, its CSR offsets and the inverse index.
//
// Kernels (P = number of radix passes):
//   dd_small       the whole dedup in one block (at most 8192 occurrences);
//                  else
//   dd_prep        global digit histograms of every pass in one read of the
//                  IDs, the ID range check, and zeroing of the look-back words
//                  (from 2^20 occurrences on zeroed by dd_zero);
//   dd_pass  x P   per 2048-key (4096) tile: local ranks from 64-lane ballots
//                  (lanes holding the same digit find each other bit by bit)
//                  and per-wave running counters in LDS; the tile in digit
//                  order in LDS; its position among earlier tiles by decoupled
//                  look-back over the per-tile digit counts they publish; then
//                  a stable scatter;
//   dd_unique      head flags of the sorted keys, rank by the same look-back,
//                  and the outputs; the tile that completes a count of
//                  finished tiles writes the device status (the passes' error
//                  flag, the unique pass's own look-back bound hits carried in
//                  the count, and the range check);
//   dd_inverse     from 2^21 occurrences on, the inverse index bucket by bucket.
// Tiles, waves, rows and lanes are visited in index order, so the sort is
// stable and every output bit-exact.  A tile only waits for earlier tiles to
// publish, and blocks are dispatched in index order, so every wait ends.
#include "ams_device.h"

#include <climits>
#include <mutex>

namespace {

constexpr int kThreads = 256;                 // 4 waves
constexpr int kWaves = kThreads / AMS_WAVE;
constexpr int kRows = 8;                      // rows of 64 keys per wave
constexpr int kTile = kThreads * kRows;       // 2048 keys per tile
constexpr int kMaxBits = 8;
constexpr int kRadix = 1 << kMaxBits;
constexpr int kMaxPasses = 4;
constexpr int kPrepBlocks = 32;                // partial histograms a pass sums

// look-back words: 2-bit state in the top bits, count below
constexpr uint32_t kAgg = 1u << 30;           // this tile's own count is published
constexpr uint32_t kPrefix = 2u << 30;        // the inclusive prefix up to this tile
constexpr uint32_t kValMask = (1u << 30) - 1;
constexpr int64_t kMaxOcc = (1 << 30) - 1;    // prefix counts stay below the state bits

__device__ __forceinline__ uint32_t ld_relaxed(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The look-back words carry everything they communicate (no other data is
// published through them), so relaxed device-scope atomics suffice; they go
// around the per-XCD caches without the cache write-back/invalidate that
// release/acquire ordering would add.
__device__ __forceinline__ void st_relaxed(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive prefix of this tile's count over all earlier tiles (decoupled
// look-back).  words[t * stride] is this tile's word, earlier tiles' words at
// words[(t - 1) * stride], ...; with stride = the radix, the threads of a
// block (one digit each) read consecutive words.  lookback_publish has
// published the aggregate (tile 0: the prefix); the inclusive prefix is
// published here.  Every tile publishes before it waits, so
// each wait ends; the wait is nevertheless bounded (`limit` re-reads), and a
// bound that is hit is recorded in *err instead of spinning on.  What follows
// such a give-up is wrong but stays in bounds: the passes drop positions past
// the buffers, and dd_unique clamps the occurrences that it uses as indexes
// (positions that nothing was written to hold whatever the workspace held).
constexpr int kSpinLimit = 1 << 22;

__device__ __forceinline__ void lookback_publish(uint32_t *words, int stride, int t, uint32_t count)
{
    st_relaxed(&words[(size_t)t * stride], (t == 0 ? kPrefix : kAgg) | count);
}

__device__ uint32_t lookback(uint32_t *words, int stride, int t, uint32_t count, int limit, int32_t *err)
{
    if (t == 0) return 0;
    // walk back in batches of independent reads (one round trip each); the
    // nearest inclusive prefix is usually a few tiles back, so a batch of 16
    // (measured against 8, 32, 64 and 128: 20.3 against 21.5, 22.6, 32.7 and
    // 42.9 us per pass on 750k keys) keeps the reads that are not needed few
    constexpr int kBatch = 16;
    uint32_t excl = 0;
    int spins = 0;
    for (int hi = t - 1; hi >= 0;) {
        const int nb = hi + 1 < kBatch ? hi + 1 : kBatch;
        uint32_t w[kBatch];
        bool ready = true;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            w[i] = i < nb ? ld_relaxed(&words[(size_t)(hi - i) * stride]) : kPrefix;
            ready &= (w[i] & ~kValMask) != 0;
        }
        if (!ready) {                             // some tile of the batch has not published
            if (++spins < limit) continue;
            __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
        spins = 0;
        bool done = false;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (done || i >= nb) continue;
            excl += w[i] & kValMask;
            done = (w[i] & ~kValMask) == kPrefix;
        }
        if (done) break;
        hi -= nb;
    }
    st_relaxed(&words[(size_t)t * stride], kPrefix | (excl + count));
    return excl;
}

// The same look-back walked by one whole wave: lane i reads the word of tile
// (hi - i), so 64 earlier tiles cost one round trip.  The lowest lane holding
// an inclusive prefix is the nearest one; the sum runs up to it.
__device__ uint32_t lookback_wave(uint32_t *words, int t, uint32_t count, int limit, bool &hit)
{
    const int lane = ams_lane();
    if (t == 0) {
        if (lane == 0) st_relaxed(&words[0], kPrefix | count);
        return 0;
    }
    if (lane == 0) st_relaxed(&words[t], kAgg | count);
    uint32_t excl = 0;
    int spins = 0;
    for (int hi = t - 1; hi >= 0;) {
        const int j = hi - lane;
        const uint32_t w = j >= 0 ? ld_relaxed(&words[j]) : kPrefix;   // before tile 0: prefix 0
        if (ams_ballot((w & ~kValMask) == 0) != 0) {                   // not all published yet
            if (++spins < limit) continue;
            hit = true;
            break;
        }
        spins = 0;
        const uint64_t pre = ams_ballot((w & ~kValMask) == kPrefix);
        const int stop = pre ? __ffsll((unsigned long long)pre) - 1 : AMS_WAVE - 1;
        const int v = lane <= stop ? (int)(w & kValMask) : 0;
        excl += (uint32_t)__shfl(ams_wave_incl_scan(v), AMS_WAVE - 1, AMS_WAVE);
        if (pre) break;
        hi -= AMS_WAVE;
    }
    if (lane == 0) st_relaxed(&words[t], kPrefix | (excl + count));
    return excl;
}

struct Plan {
    int bits, passes, width, ntiles;
    int limit;                                 // re-reads of a bounded wait (kSpinLimit)
};

__device__ __forceinline__ int pass_bits(const Plan &P, int pass)
{
    const int shift = pass * P.width;
    return (P.bits - shift) < P.width ? (P.bits - shift) : P.width;
}

// Global digit histograms (partials per prep block), range check, zeroing.
// 1024 threads per block: one LDS histogram per wave (a hot ID's digit then
// contends within one wave only), 16 waves adding at once.
// WIDE (large batches): any number of blocks add their counts to one histogram
// per pass with integer atomics (the sums do not depend on their order), which
// dd_zero has cleared along with the words; else each block writes a partial
// of its own and clears its share of the words.
constexpr int kPrepThreads = 1024;
constexpr int kPrepWaves = kPrepThreads / AMS_WAVE;
template <bool WIDE>
__global__ __launch_bounds__(kPrepThreads) void dd_prep(const uint32_t *__restrict__ keys, int n, Plan P,
                                                        uint32_t n_ids, int32_t *__restrict__ hpart,
                                                        int32_t *__restrict__ bad,
                                                        uint32_t *__restrict__ words, int n_words)
{
    // eight keys per thread are loaded before their counts are added
    constexpr int U = 8;
    __shared__ int h[kPrepWaves][kMaxPasses][kRadix];
    const int t = threadIdx.x, wave = t / AMS_WAVE;
    for (int i = t; i < kPrepWaves * kMaxPasses * kRadix; i += kPrepThreads) (&h[0][0][0])[i] = 0;
    if (!WIDE)
        for (int i = blockIdx.x * kPrepThreads + t; i < n_words; i += gridDim.x * kPrepThreads) words[i] = 0;
    __syncthreads();
    bool out = false;
    const int stride = gridDim.x * kPrepThreads;
    for (int i0 = blockIdx.x * kPrepThreads + t; i0 < n; i0 += U * stride) {
        uint32_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * stride;
            k[u] = i < n ? keys[i] : 0xffffffffu;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k[u] == 0xffffffffu && i0 + u * stride >= n) continue;
            out |= (k[u] >= n_ids);
            for (int p = 0; p < P.passes; ++p) {
                const uint32_t mask = (1u << pass_bits(P, p)) - 1u;
                atomicAdd(&h[wave][p][(k[u] >> (p * P.width)) & mask], 1);
            }
        }
    }
    const int any_out = __syncthreads_or(out);
    if (t < kRadix)
        for (int p = 0; p < P.passes; ++p) {
            int c = 0;
            for (int w = 0; w < kPrepWaves; ++w) c += h[w][p][t];
            if (!WIDE) hpart[((size_t)blockIdx.x * kMaxPasses + p) * kRadix + t] = c;
            else if (c) atomicAdd(&hpart[p * kRadix + t], c);
        }
    if (t == 0) {
        if (!WIDE) bad[blockIdx.x] = any_out;
        else if (any_out) atomicOr(bad, 1);
    }
}

__global__ __launch_bounds__(kThreads) void dd_zero(uint32_t *__restrict__ words, int n_words,
                                                    int32_t *__restrict__ hpart, int n_hpart,
                                                    int32_t *__restrict__ bad)
{
    const int i0 = blockIdx.x * kThreads + threadIdx.x, stride = gridDim.x * kThreads;
    for (int i = i0; i < n_words; i += stride) words[i] = 0;
    for (int i = i0; i < n_hpart; i += stride) hpart[i] = 0;
    if (i0 == 0) *bad = 0;
}

// ------------------------------------------------------- small batches
// The whole dedup of at most 8192 occurrences in one block: the same stable
// radix passes with the keys in registers between LDS exchanges (wave w holds
// positions [w ROWS 64, (w + 1) ROWS 64), row by row), then the unique pass.
// A batch this small is bound by launches.  IDs of 18 bits, whole call: 576
// occurrences 24.0 us in five launches, 8.6 us so; 2000: 26.6 and 9.6; 4000:
// 32.8 and 14.5; 8000: 33.0 and 23.1 (one compute unit ranks 8192 keys in the
// time five launches take for 16384, hence the line at 8192).  At 31 bits, four
// passes: 2048 37.8 and 12.5; 8192 48.3 and 32.7, with 44.8 in tiles at 8193.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / AMS_WAVE;
constexpr int kSmallMax = 8 * kSmallThreads;


template <int ROWS>
__global__ __launch_bounds__(kSmallThreads) void dd_small(const uint32_t *__restrict__ ids, int n, Plan P,
                                                          uint32_t n_ids, int32_t *__restrict__ uniq,
                                                          int32_t *__restrict__ inv, int32_t *__restrict__ occ_perm,
                                                          int32_t *__restrict__ uniq_off,
                                                          int32_t *__restrict__ n_uniq,
                                                          int32_t *__restrict__ dev_status)
{
    __shared__ int cnt[kSmallWaves][kRadix];
    __shared__ int wsum[kSmallWaves];
    __shared__ uint32_t ks[ROWS * kSmallThreads];
    __shared__ int32_t vs[ROWS * kSmallThreads];
    const int t = threadIdx.x, lane = ams_lane(), wave = t / AMS_WAVE;
    const int tbase = wave * (ROWS * AMS_WAVE) + lane;
    const uint64_t lt = ams_lanemask_lt();
    uint32_t key[ROWS];
    int32_t val[ROWS];
    bool out = false;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = tbase + r * AMS_WAVE;
        key[r] = ids[min(i, n - 1)];
        val[r] = i;
        out |= key[r] >= n_ids;
    }
    const int any_out = __syncthreads_or(out);
    for (int pass = 0; pass < P.passes; ++pass) {
        const int shift = pass * P.width, bits = pass_bits(P, pass);
        const uint32_t mask = (1u << bits) - 1u;
        int rank[ROWS];
        for (int d = lane; d < kRadix; d += AMS_WAVE) cnt[wave][d] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const bool valid = tbase + r * AMS_WAVE < n;
            const uint32_t d = (key[r] >> shift) & mask;
            uint64_t peers = ams_ballot(valid);
            for (int b = 0; b < bits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bb = ams_ballot(bit);
                peers &= bit ? bb : ~bb;
            }
            const int below = __popcll(peers & lt);
            const int c = valid ? cnt[wave][d] : 0;
            rank[r] = c + below;
            __builtin_amdgcn_wave_barrier();
            if (valid && below == 0) cnt[wave][d] = c + __popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // where each wave's keys of a digit start: the digits' counts scanned
        // over four waves, then the waves' counts in order
        int tot = 0, incl = 0;
        if (t < kRadix) {
            for (int w = 0; w < kSmallWaves; ++w) tot += cnt[w][t];
            incl = ams_wave_incl_scan(tot);
            if (lane == AMS_WAVE - 1) wsum[wave] = incl;
        }
        __syncthreads();
        if (t < kRadix) {
            int run = incl - tot;
            for (int w = 0; w < wave; ++w) run += wsum[w];
            for (int w = 0; w < kSmallWaves; ++w) {
                const int c = cnt[w][t];
                cnt[w][t] = run;
                run += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (tbase + r * AMS_WAVE < n) {
                const int pos = cnt[wave][(key[r] >> shift) & mask] + rank[r];
                ks[pos] = key[r];
                vs[pos] = val[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int i = min(tbase + r * AMS_WAVE, n - 1);
            key[r] = ks[i];
            val[r] = vs[i];
        }
    }
    // head flags row by row; a wave's heads before a position: earlier rows'
    // and, by ballot, earlier lanes'
    uint64_t heads[ROWS];
    int c = 0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = tbase + r * AMS_WAVE;
        heads[r] = ams_ballot(i < n && (i == 0 || ks[i - 1] != key[r]));
        c += __popcll(heads[r]);
    }
    if (lane == 0) wsum[wave] = c;
    __syncthreads();
    int run = 0;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = tbase + r * AMS_WAVE;
        const bool head = (heads[r] >> lane) & 1;
        const int u = run + __popcll(heads[r] & lt) + (head ? 1 : 0) - 1;
        run += __popcll(heads[r]);
        if (i >= n) continue;
        occ_perm[i] = val[r];
        inv[val[r]] = u;
        if (head) {
            uniq[u] = (int32_t)key[r];
            uniq_off[u] = i;
        }
        if (i == n - 1) {
            uniq_off[u + 1] = n;
            *n_uniq = u + 1;
            *dev_status = any_out ? AMS_ERR_ID_RANGE : AMS_OK;
        }
    }
}

// One stable radix pass over tiles of ROWS x 256 keys.  vin == nullptr means
// the identity (first pass).  The tile's keys and values are first put in
// digit order in LDS (which needs only the tile's own counts, so it runs
// before the look-back), then written out from there: the keys of one digit
// are consecutive in the output, so a wave's 64 stores fall in a few runs
// where stores straight from the ranks meet up to 64 lines.  Per pass, 12.1M
// keys of 21 bits: 109 us with stores from the ranks, 84 us so, 68 us (2.9
// TB/s) in tiles of 4096 keys; 57k keys of 18 bits: 12.0 and 11.8 us (14.8 in
// the larger tiles: too few blocks).
template <int ROWS>
__global__ __launch_bounds__(kThreads) void dd_pass(const uint32_t *__restrict__ kin,
                                                    const int32_t *__restrict__ vin,
                                                    uint32_t *__restrict__ kout, int32_t *__restrict__ vout,
                                                    int n, Plan P, int pass,
                                                    const int32_t *__restrict__ hpart, int n_prep,
                                                    uint32_t *__restrict__ words, int32_t *__restrict__ err)
{
    constexpr int TILE = ROWS * kThreads;
    __shared__ int cnt[kWaves][kRadix];
    __shared__ int gofs[kRadix];
    __shared__ int scan_tmp[2][kWaves];
    __shared__ uint32_t ks[TILE];
    __shared__ int32_t vs[TILE];
    const int t = threadIdx.x, lane = ams_lane(), wave = t / AMS_WAVE;
    const int shift = pass * P.width, bits = pass_bits(P, pass);
    const uint32_t mask = (1u << bits) - 1u;
    const int tile0 = blockIdx.x * TILE;
    const int tbase = tile0 + wave * (ROWS * AMS_WAVE);
    const uint64_t lt = ams_lanemask_lt();
    uint32_t key[ROWS];
    int32_t val[ROWS];
    int rank[ROWS];
    // every load of the block first, all independent (one memory round trip):
    // the tile's keys and values (clamped, branch-free), then this pass's
    // per-block digit partials
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int idx = min(tbase + r * AMS_WAVE + lane, n - 1);
        key[r] = kin[idx];
        val[r] = vin ? vin[idx] : idx;
    }
    int tot = 0;
    if (n_prep == 1) {
        tot = hpart[pass * kRadix + t];
    } else {
        int part[kPrepBlocks];
#pragma unroll
        for (int b = 0; b < kPrepBlocks; ++b)
            part[b] = hpart[((size_t)min(b, n_prep - 1) * kMaxPasses + pass) * kRadix + t];
#pragma unroll
        for (int b = 0; b < kPrepBlocks; ++b) tot += b < n_prep ? part[b] : 0;
    }
    for (int d = lane; d < kRadix; d += AMS_WAVE) cnt[wave][d] = 0;

#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int idx = tbase + r * AMS_WAVE + lane;
        const bool valid = idx < n;
        const uint32_t d = (key[r] >> shift) & mask;
        uint64_t peers = ams_ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = ams_ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const int below = __popcll(peers & lt);
        const int c = valid ? cnt[wave][d] : 0;
        rank[r] = c + below;
        // every lane of the wave has read its counter before the leader of
        // each digit group advances it (one wave, LDS ops in program order)
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) cnt[wave][d] = c + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // this tile's count of digit t (2^width look-back words per tile; digits
    // past this pass's bits are empty everywhere)
    const int R = 1 << P.width;
    uint32_t *const lb = words + ((size_t)pass * P.ntiles) * R + t;
    int tile_cnt = 0;
    for (int w = 0; w < kWaves; ++w) tile_cnt += cnt[w][t];
    if (t < (1 << bits)) lookback_publish(lb, R, blockIdx.x, (uint32_t)tile_cnt);
    // exclusive digit offsets over all keys (the same in every tile) and
    // within the tile
    const int incl = ams_wave_incl_scan(tot), tincl = ams_wave_incl_scan(tile_cnt);
    if (lane == AMS_WAVE - 1) {
        scan_tmp[0][wave] = incl;
        scan_tmp[1][wave] = tincl;
    }
    __syncthreads();
    int gbase = incl - tot, tstart = tincl - tile_cnt;
    for (int w = 0; w < wave; ++w) {
        gbase += scan_tmp[0][w];
        tstart += scan_tmp[1][w];
    }
    // where each wave's keys of digit t start in the tile
    int run = tstart;
    for (int w = 0; w < kWaves; ++w) {
        const int c = cnt[w][t];
        cnt[w][t] = run;
        run += c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (tbase + r * AMS_WAVE + lane < n) {
            const int pos = cnt[wave][(key[r] >> shift) & mask] + rank[r];
            ks[pos] = key[r];
            vs[pos] = val[r];
        }
    uint32_t before = 0;
    if (t < (1 << bits)) before = lookback(lb, R, blockIdx.x, (uint32_t)tile_cnt, P.limit, err);
    gofs[t] = gbase + (int)before - tstart;
    __syncthreads();
    const int m = min(TILE, n - tile0);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = r * kThreads + t;
        if (i < m) {
            const uint32_t k = ks[i];
            const int pos = gofs[(k >> shift) & mask] + i;
            // (a bounded wait that gave up leaves a wrong offset, here or in a
            // pass before: the status says so, and this store stays inside)
            if ((unsigned)pos < (unsigned)n) {
                kout[pos] = k;
                vout[pos] = vs[i];
            }
        }
    }
}

// Unique set, CSR offsets, stable occurrence order, inverse index, count,
// and the device status: each tile adds 1 + (hit << 32) to *done (one
// relaxed 64-bit add: tiles finished in the low word, look-back bound hits of
// this pass in the high word); the tile whose add completes the count reads
// the passes' error flag and the range check (earlier launches, ordered by
// the kernel boundaries) and writes the status.  Only the count itself is
// communicated between tiles, so no ordering beyond the add's atomicity is
// needed.
//
// BUCKET (batches whose inverse index leaves the caches): inv[occ] = rank at
// random positions moves a whole line per 4 bytes.  Instead a tile puts its
// (occ, rank) pairs in the order of occ's bucket (32768 consecutive
// occurrences) in LDS, takes a run of each bucket's array with one atomic add
// and writes the runs; dd_inverse then places each bucket in LDS and stores
// inv whole.  Where a pair lands within its bucket depends on the order of
// the adds, inv does not.  12.1M occurrences: 194 us
// with the random stores, 100 + 27 us so; 3M: 52 and 35 + 10; 1.5M: 31 and
// 24 + 10 (the line is at 2M).
constexpr int kBucketBits = 15, kMaxBuckets = 512;
constexpr int kBucketStride = 16;              // counters 64 bytes apart

template <int THREADS, bool BUCKET>
__global__ __launch_bounds__(THREADS) void dd_unique(const uint32_t *__restrict__ k,
                                                      const int32_t *__restrict__ v, int n,
                                                      uint32_t *__restrict__ words, int limit,
                                                      const int32_t *__restrict__ err,
                                                      unsigned long long *__restrict__ done,
                                                      const int32_t *__restrict__ bad, int n_prep,
                                                      int32_t *__restrict__ uniq, int32_t *__restrict__ inv,
                                                      int32_t *__restrict__ occ_perm,
                                                      int32_t *__restrict__ uniq_off,
                                                      int32_t *__restrict__ n_uniq, int32_t *__restrict__ dev_status,
                                                      int32_t *__restrict__ fill, int32_t *__restrict__ pair_occ,
                                                      int32_t *__restrict__ pair_rank)
{
    constexpr int kItems = 8;                  // consecutive positions per thread
    constexpr int TILE = THREADS * kItems, WAVES = THREADS / AMS_WAVE;
    __shared__ int ws[WAVES];
    __shared__ int bcnt[BUCKET ? kMaxBuckets : 1], bofs[BUCKET ? kMaxBuckets : 1];
    __shared__ int32_t po[BUCKET ? TILE : 1], pr[BUCKET ? TILE : 1];
    __shared__ uint32_t tile_base;
    const int t = threadIdx.x, w = t / AMS_WAVE;
    const int i0 = blockIdx.x * TILE + t * kItems;
    static_assert(kItems == 8, "two 16-byte loads per thread");
    // a thread's 8 keys and values: two 16-byte loads each when all 8 are in
    // range (i0 is a multiple of 8), else one by one
    const bool full = i0 + kItems <= n;
    uint32_t kk[kItems];
    int32_t vv[kItems];
    if (full) {
        const uint4 a = *(const uint4 *)(k + i0), b = *(const uint4 *)(k + i0 + 4);
        const int4 x = *(const int4 *)(v + i0), y = *(const int4 *)(v + i0 + 4);
        kk[0] = a.x; kk[1] = a.y; kk[2] = a.z; kk[3] = a.w; kk[4] = b.x; kk[5] = b.y; kk[6] = b.z; kk[7] = b.w;
        vv[0] = x.x; vv[1] = x.y; vv[2] = x.z; vv[3] = x.w; vv[4] = y.x; vv[5] = y.y; vv[6] = y.z; vv[7] = y.w;
    } else {
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            kk[q] = i0 + q < n ? k[i0 + q] : 0u;
            vv[q] = i0 + q < n ? v[i0 + q] : 0;
        }
    }
    // an index from here on (inv, the buckets, and through occ_perm the pooling
    // backward's records): inside the batch also where a pass gave up a wait
#pragma unroll
    for (int q = 0; q < kItems; ++q) vv[q] = (int32_t)min((uint32_t)vv[q], (uint32_t)(n - 1));
    const uint32_t kprev = (i0 > 0 && i0 < n) ? k[i0 - 1] : 0u;
    if (BUCKET)
        for (int i = t; i < kMaxBuckets; i += THREADS) bcnt[i] = 0;
    int flag[kItems];
    int c = 0;
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        const int i = i0 + q;
        const uint32_t before = q == 0 ? kprev : kk[q - 1];
        flag[q] = (i < n && (i == 0 || kk[q] != before)) ? 1 : 0;
        c += flag[q];
    }
    const int incl = ams_wave_incl_scan(c);
    if (ams_lane() == AMS_WAVE - 1) ws[w] = incl;
    __syncthreads();
    bool hit = false;                          // (wave 0: this tile's look-back bound)
    if (w == 0) {
        int tot = 0;
        for (int x = 0; x < WAVES; ++x) tot += ws[x];
        const uint32_t b = lookback_wave(words, blockIdx.x, (uint32_t)tot, limit, hit);
        if (t == 0) tile_base = b;
    }
    __syncthreads();
    int run = (int)tile_base + incl - c;      // heads strictly before position i0
    for (int x = 0; x < w; ++x) run += ws[x];
    // (the caller's occ_perm may start anywhere: 16-byte stores only when aligned)
    const bool vec_out = full && (((uintptr_t)occ_perm & 15) == 0);
    if (vec_out) {
        *(int4 *)(occ_perm + i0) = make_int4(vv[0], vv[1], vv[2], vv[3]);
        *(int4 *)(occ_perm + i0 + 4) = make_int4(vv[4], vv[5], vv[6], vv[7]);
    }
    int rk[kItems], bpos[kItems];              // BUCKET: ranks, places within the tile's bucket runs
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        const int i = i0 + q;
        if (i >= n) break;
        run += flag[q];
        const int rank = run - 1;
        const int32_t occ = vv[q];
        if (!vec_out) occ_perm[i] = occ;
        if (BUCKET) {
            rk[q] = rank;
            bpos[q] = atomicAdd(&bcnt[(occ >> kBucketBits) & (kMaxBuckets - 1)], 1);
        } else {
            inv[occ] = rank;
        }
        if (flag[q]) {
            uniq[rank] = (int32_t)kk[q];
            uniq_off[rank] = i;
        }
        if (i == n - 1) {
            uniq_off[rank + 1] = n;
            *n_uniq = rank + 1;
        }
    }
    if constexpr (BUCKET) {
        static_assert(!BUCKET || THREADS >= kMaxBuckets, "a thread per bucket");
        __syncthreads();
        // the tile's runs: starts in LDS (a scan of the counts), places in the
        // buckets (one add each)
        const int b = t < kMaxBuckets ? t : 0;
        const int cb = t < kMaxBuckets ? bcnt[b] : 0;
        const int bincl = ams_wave_incl_scan(cb);
        int place = 0;
        if (cb) place = (b << kBucketBits) + atomicAdd(&fill[b * kBucketStride], cb);
        if (ams_lane() == AMS_WAVE - 1) ws[w] = bincl;
        __syncthreads();
        int start = bincl - cb;
        for (int x = 0; x < w; ++x) start += ws[x];
        if (t < kMaxBuckets) {
            bcnt[b] = start;
            bofs[b] = place - start;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kItems; ++q)
            if (i0 + q < n) {
                const int x = bcnt[(vv[q] >> kBucketBits) & (kMaxBuckets - 1)] + bpos[q];
                po[x] = vv[q];
                pr[x] = rk[q];
            }
        __syncthreads();
        const int m = min(TILE, n - (int)blockIdx.x * TILE);
        for (int i = t; i < m; i += THREADS) {
            const int occ = po[i], pos = bofs[(occ >> kBucketBits) & (kMaxBuckets - 1)] + i;
            if ((unsigned)pos < (unsigned)n) {
                pair_occ[pos] = occ;
                pair_rank[pos] = pr[i];
            }
        }
    }
    if (t == 0) {
        const unsigned long long old = __hip_atomic_fetch_add(done, 1ull + ((unsigned long long)hit << 32),
                                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)old == gridDim.x - 1) {
            const bool lb = (old >> 32) != 0 || hit ||
                            __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            int any_bad = 0;
            for (int b = 0; b < n_prep; ++b) any_bad |= bad[b];
            *dev_status = lb ? AMS_ERR_HIP : (any_bad ? AMS_ERR_ID_RANGE : AMS_OK);
        }
    }
}

// inv of one bucket of occurrences from its (occ, rank) pairs.
constexpr int kInvThreads = 1024;
__global__ __launch_bounds__(kInvThreads) void dd_inverse(const int32_t *__restrict__ pair_occ,
                                                          const int32_t *__restrict__ pair_rank, int n,
                                                          int32_t *__restrict__ inv)
{
    constexpr int SIZE = 1 << kBucketBits, U = 8;
    __shared__ int32_t x[SIZE];
    const int b0 = blockIdx.x << kBucketBits, m = min(SIZE, n - b0);
    for (int i0 = threadIdx.x; i0 < m; i0 += U * kInvThreads) {
        int32_t o[U], r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = b0 + min(i0 + u * kInvThreads, m - 1);
            o[u] = pair_occ[i];
            r[u] = pair_rank[i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kInvThreads < m) x[o[u] & (SIZE - 1)] = r[u];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += kInvThreads) inv[b0 + i] = x[i];
}

__global__ void dd_empty(int32_t *n_uniq, int32_t *dev_status, int32_t *uniq_off)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        *dev_status = AMS_OK;
        *n_uniq = 0;
        uniq_off[0] = 0;
    }
}

constexpr int id_bits(int32_t n_ids)
{
    int b = 1;
    while (b < 31 && (1ll << b) < (long long)n_ids) ++b;
    return b;
}

// From kWideOcc occurrences on: tiles of 4096 keys in the radix passes, one
// histogram per pass (dd_zero, dd_prep<true>).  Whole call, 21-bit IDs, without
// and with: 750k occurrences 83.3 and 83.8 us (the extra launch costs what the
// wider histogram saves), 1.5M 117.5 and 105.5, 12.1M 576 and 418.
constexpr int64_t kWideOcc = 1 << 20;
constexpr int kWideRows = 2 * kRows;
// From kBucketOcc on, while the buckets are enough, the inverse index goes by
// buckets; their counters follow the histograms.  Past 2^24 occurrences there are
// not, and the random stores come back (2M IDs: 506 us at 2^24, 638 past it).
constexpr int64_t kBucketOcc = 1 << 21;
static_assert(kMaxPasses * kRadix + kMaxBuckets * kBucketStride <= kPrepBlocks * kMaxPasses * kRadix &&
                  kBucketOcc >= kWideOcc && kWideOcc >= kPrepBlocks * kTile,
              "the partial histograms' room holds one histogram and the counters");

struct Layout {
    Plan P;
    bool wide, bucket;
    int n_prep, n_words, i_err, i_done, utiles;
    size_t off_kb, off_va, off_vb, off_hpart, off_bad, off_words, total;
};

constexpr Layout layout(int64_t n_occ, int32_t n_ids)
{
    Layout L{};
    L.P.bits = id_bits(n_ids);
    L.P.passes = (L.P.bits + kMaxBits - 1) / kMaxBits;
    L.P.width = (L.P.bits + L.P.passes - 1) / L.P.passes;
    L.P.limit = kSpinLimit;
    L.utiles = (int)((n_occ + kTile - 1) / kTile);
    L.wide = n_occ >= kWideOcc;
    L.bucket = n_occ >= kBucketOcc && n_occ <= (int64_t)kMaxBuckets << kBucketBits;
    L.P.ntiles = L.wide ? (int)((n_occ + 2 * kTile - 1) / (2 * kTile)) : L.utiles;
    L.n_prep = L.utiles < kPrepBlocks ? (L.utiles > 0 ? L.utiles : 1) : kPrepBlocks;
    // look-back words (1 << width per tile and pass, then one per tile for
    // the unique pass), the passes' error flag, and the unique pass's 64-bit
    // completion count at an even word (the region is 256-byte aligned)
    const int n_lb = L.P.passes * L.P.ntiles * (1 << L.P.width) + L.utiles;
    L.i_err = n_lb;
    L.i_done = (n_lb + 2) & ~1;
    L.n_words = L.i_done + 2;
    auto al = [](size_t x) constexpr { return (x + 255) & ~(size_t)255; };
    const size_t nb = al((size_t)n_occ * 4);
    size_t o = nb;                           // keys ping (pong is the caller's ids on pass 0)
    L.off_kb = o; o += nb;
    L.off_va = o; o += nb;
    L.off_vb = o; o += nb;
    L.off_hpart = o; o += al((size_t)L.n_prep * kMaxPasses * kRadix * 4);
    L.off_bad = o; o += al((size_t)L.n_prep * 4);
    // (room for the words of 2048-key tiles in any case: the size has to serve
    // every smaller batch)
    const size_t most = (size_t)L.P.passes * L.utiles * (1 << L.P.width) + L.utiles + 4;
    L.off_words = o; o += al(most * 4);
    L.total = o;
    return L;
}

// Workspace that serves every ID range up to n_ids (and, the layout growing
// with n_occ, every smaller batch): the look-back words grow with the digit
// width, which is not monotonic in n_ids (100 IDs: one 7-bit pass; 1000: two
// of 5), so the largest layout over the bit counts up to n_ids's.
constexpr size_t workspace_bound(int64_t n_occ, int32_t n_ids)
{
    size_t t = 0;
    const int B = id_bits(n_ids);
    for (int b = 1; b <= B; ++b) {
        const size_t x = layout(n_occ, b == B ? n_ids : (int32_t)(1u << b)).total;
        t = x > t ? x : t;
    }
    return t;
}

// Enqueues the whole dedup with its workspace at `w` (layout L).
ams_status dedup_enqueue(const int32_t *ids, int n, int32_t n_ids, int32_t *uniq, int32_t *inv,
                         int32_t *occ_perm, int32_t *uniq_off, int32_t *n_uniq, int32_t *dev_status,
                         char *w, const Layout &L, hipStream_t st)
{
    if (n == 0) {
        AMS_LAUNCH("dd_empty", st, dd_empty<<<1, 64, 0, st>>>(n_uniq, dev_status, uniq_off));
        return ams_launch_status();
    }
    if (n <= kSmallMax) {
#define DD_SMALL(R)                                                                                                 \
    AMS_LAUNCH("dd_small", st, dd_small<R><<<1, kSmallThreads, 0, st>>>((const uint32_t *)ids, n, L.P, (uint32_t)n_ids, \
                                                                       uniq, inv, occ_perm, uniq_off, n_uniq, dev_status))
        if (n <= kSmallThreads) DD_SMALL(1);
        else if (n <= 2 * kSmallThreads) DD_SMALL(2);
        else if (n <= 4 * kSmallThreads) DD_SMALL(4);
        else DD_SMALL(8);
#undef DD_SMALL
        return ams_launch_status();
    }
    uint32_t *ka = (uint32_t *)w;
    uint32_t *kb = (uint32_t *)(w + L.off_kb);
    int32_t *va = (int32_t *)(w + L.off_va);
    int32_t *vb = (int32_t *)(w + L.off_vb);
    int32_t *hpart = (int32_t *)(w + L.off_hpart);
    int32_t *bad = (int32_t *)(w + L.off_bad);
    uint32_t *words = (uint32_t *)(w + L.off_words);
    int32_t *err = (int32_t *)(words + L.i_err);
    unsigned long long *done = (unsigned long long *)(words + L.i_done);

    if (L.wide) {
        const int zg = L.n_words / (4 * kThreads) + 1;
        AMS_LAUNCH("dd_zero", st, dd_zero<<<zg < 1024 ? zg : 1024, kThreads, 0, st>>>(
                                      words, L.n_words, hpart,
                                      kMaxPasses * kRadix + (L.bucket ? kMaxBuckets * kBucketStride : 0), bad));
        // one block per 16384 keys, at most one per compute unit
        const int g = (n + 16 * kPrepThreads - 1) / (16 * kPrepThreads);
        AMS_LAUNCH("dd_prep", st, dd_prep<true><<<g < 256 ? g : 256, kPrepThreads, 0, st>>>(
                                      (const uint32_t *)ids, n, L.P, (uint32_t)n_ids, hpart, bad, words, L.n_words));
    } else {
        // dd_prep also zeroes every look-back word, the error flag and the count
        AMS_LAUNCH("dd_prep", st, dd_prep<false><<<L.n_prep, kPrepThreads, 0, st>>>(
                                      (const uint32_t *)ids, n, L.P, (uint32_t)n_ids, hpart, bad, words, L.n_words));
    }
    const int n_prep = L.wide ? 1 : L.n_prep;
    const uint32_t *kin = (const uint32_t *)ids;
    const int32_t *vin = nullptr;
    uint32_t *bufk[2] = {ka, kb};
    int32_t *bufv[2] = {va, vb};
    for (int pass = 0; pass < L.P.passes; ++pass) {
        uint32_t *kout = bufk[pass & 1];
        int32_t *vout = bufv[pass & 1];
        if (L.wide)
            AMS_LAUNCH("dd_pass", st, dd_pass<kWideRows><<<L.P.ntiles, kThreads, 0, st>>>(
                                          kin, vin, kout, vout, n, L.P, pass, hpart, n_prep, words, err));
        else
            AMS_LAUNCH("dd_pass", st, dd_pass<kRows><<<L.P.ntiles, kThreads, 0, st>>>(
                                          kin, vin, kout, vout, n, L.P, pass, hpart, n_prep, words, err));
        kin = kout;
        vin = vout;
    }
    uint32_t *uw = words + (size_t)L.P.passes * L.P.ntiles * (1 << L.P.width);
    if (L.bucket) {
        // the pass buffers that do not hold the sorted keys and values
        int32_t *po = (int32_t *)bufk[L.P.passes & 1], *pr = bufv[L.P.passes & 1];
        const int tiles = (n + 8 * kInvThreads - 1) / (8 * kInvThreads);
        AMS_LAUNCH("dd_unique", st, (dd_unique<kInvThreads, true><<<tiles, kInvThreads, 0, st>>>(
                                        kin, vin, n, uw, L.P.limit, err, done, bad, n_prep, uniq, inv, occ_perm, uniq_off, n_uniq,
                                        dev_status, hpart + kMaxPasses * kRadix, po, pr)));
        AMS_LAUNCH("dd_inverse", st, dd_inverse<<<((n - 1) >> kBucketBits) + 1, kInvThreads, 0, st>>>(po, pr, n, inv));
    } else {
        AMS_LAUNCH("dd_unique", st, (dd_unique<kThreads, false><<<L.utiles, kThreads, 0, st>>>(
                                        kin, vin, n, uw, L.P.limit, err, done, bad, n_prep, uniq, inv, occ_perm, uniq_off, n_uniq,
                                        dev_status, nullptr, nullptr, nullptr)));
    }
    return ams_launch_status();
}

// ------------------------------------------------ no-allocation variant ----
// Scratch of ams_dedup_noalloc: the workspace of the largest batch it takes
// (kNoAllocMaxOcc occurrences, IDs of up to 31 bits: four radix passes),
// 19.0 MB in every GPU's copy of the library's code object.  Host code never
// passes `scratch` itself to a kernel (on the host it names a stand-in, not
// device memory): the device address comes from hipGetSymbolAddress, looked
// up once per device with that device current.
constexpr int64_t kNoAllocMaxOcc = AMS_DEDUP_NOALLOC_MAX_OCC;
constexpr size_t kScratchBytes = workspace_bound(kNoAllocMaxOcc, INT32_MAX);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];

// Device address of this device's scratch (nullptr on failure).
void *scratch_on_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

extern "C" size_t ams_dedup_workspace(int64_t n_occ, int32_t n_ids)
{
    if (n_occ < 0 || n_ids < 1) return 0;
    return workspace_bound(n_occ, n_ids);
}

namespace {

ams_status dedup_limited(const int32_t *ids, int64_t n_occ, int32_t n_ids, int32_t *uniq, int32_t *inv,
                         int32_t *occ_perm, int32_t *uniq_off, int32_t *n_uniq, int32_t *dev_status, void *ws,
                         size_t ws_bytes, int limit, void *stream)
{
    if (n_occ < 0 || n_occ > kMaxOcc || n_ids < 1) return AMS_ERR_SIZE;
    if (!uniq_off || !n_uniq || !dev_status) return AMS_ERR_NULL;
    if (n_occ > 0 && (!ids || !uniq || !inv || !occ_perm || !ws)) return AMS_ERR_NULL;
    Layout L = layout(n_occ, n_ids);
    if (n_occ > 0 && ws_bytes < L.total) return AMS_ERR_WORKSPACE;
    L.P.limit = limit;
    return dedup_enqueue(ids, (int)n_occ, n_ids, uniq, inv, occ_perm, uniq_off, n_uniq, dev_status, (char *)ws, L,
                         (hipStream_t)stream);
}

}  // namespace

extern "C" ams_status ams_dedup(const int32_t *ids, int64_t n_occ, int32_t n_ids, int32_t *uniq,
                                int32_t *inv, int32_t *occ_perm, int32_t *uniq_off,
                                int32_t *n_uniq, int32_t *dev_status, void *ws, size_t ws_bytes,
                                void *stream)
{
    return dedup_limited(ids, n_occ, n_ids, uniq, inv, occ_perm, uniq_off, n_uniq, dev_status, ws, ws_bytes, kSpinLimit,
                         stream);
}

// ams_dedup with the waits bounded at `limit` re-reads: not part of the
// interface (the header does not declare it).  With a limit of 1 a tile gives
// up as soon as an earlier one is not ready, which is how the tests reach what
// follows a give-up.
extern "C" ams_status amsi_dedup_limit(const int32_t *ids, int64_t n_occ, int32_t n_ids, int32_t *uniq, int32_t *inv,
                                       int32_t *occ_perm, int32_t *uniq_off, int32_t *n_uniq, int32_t *dev_status,
                                       void *ws, size_t ws_bytes, int32_t limit, void *stream)
{
    return dedup_limited(ids, n_occ, n_ids, uniq, inv, occ_perm, uniq_off, n_uniq, dev_status, ws, ws_bytes, limit,
                         stream);
}

extern "C" ams_status ams_dedup_noalloc(const int32_t *ids, int64_t n_occ, int32_t n_ids, int32_t *uniq,
                                        int32_t *inv, int32_t *occ_perm, int32_t *uniq_off,
                                        int32_t *n_uniq, int32_t *dev_status, void *stream)
{
    if (n_occ < 0 || n_ids < 1) return AMS_ERR_SIZE;
    if (n_occ > kNoAllocMaxOcc) return AMS_ERR_CAPACITY;
    if (!uniq_off || !n_uniq || !dev_status) return AMS_ERR_NULL;
    if (n_occ > 0 && (!ids || !uniq || !inv || !occ_perm)) return AMS_ERR_NULL;
    const Layout L = layout(n_occ, n_ids);
    if (L.total > kScratchBytes) return AMS_ERR_CAPACITY;
    char *w = (char *)scratch_on_current_device();
    if (!w) return AMS_ERR_HIP;
    return dedup_enqueue(ids, (int)n_occ, n_ids, uniq, inv, occ_perm, uniq_off, n_uniq, dev_status, w, L,
                         (hipStream_t)stream);
}
