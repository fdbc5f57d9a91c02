// Top-k per appended token (the selection half of Eq. 1's Idx) over the
// causal candidates [0, M+i] of each score row, exact under the strict order
// (score descending, id ascending).
//
// One block per row.  A row (up to 557 KB at a 128K history) does not fit in
// LDS, so the block streams it from HBM once, keeping only candidates that
// beat a running threshold in an LDS buffer of CAP (key, id) pairs:
//   1. threshold seed: a sample of 8-element groups spread over the row (1/32
//      of a 128K row) gives the key of a rank a little above k * (sample
//      share), so that in expectation ~1.3k elements pass.  (Whole 128-byte
//      lines, four times as far apart, hit spans of high scores too unevenly: a
//      row whose seed came out above its k-th key is streamed again);
//   2. streaming filter: each wave takes 1 KB chunks of its own, TK_RING of
//      them in flight in registers, and appends what it accepts with one LDS
//      atomic per chunk that has any.  The waves meet only when the row is
//      done or the buffer full: a wave that finds no room stops at its chunk;
//      the buffer is then cut to exactly the k best, the threshold rises to
//      the k-th best (key, id), and the stopped waves go on, so no member of
//      the answer is lost.  If the seed was above the k-th key (fewer than k
//      passed), the row is streamed again with a looser one, then with none;
//   3. exact selection from registers: the keys' range is narrowed to one of
//      2048 equal bins, and again, until the bin holding the k-th key has few
//      enough entries to be ranked pairwise, or is a single key, whose ties
//      the same narrowing on ids resolves (smallest first);
//   4. ordered output: the winners are set in an LDS bitmap over [0, n), a
//      block scan of its words' popcounts gives each winner its rank, and the
//      ids are staged by rank in LDS and written out coalesced.
//
// What bounds it: the stream (HBM at long rows of many tokens), and with few
// or short rows the fixed phases, whose cost is barriers and LDS round trips.
// Narrowing between the data's own extremes takes one histogram pass where
// 8-bit digits from the top took four (the first ones all but one bin wide,
// their atomics serialised), register scans replace shuffles, and waves that
// stream on their own need no barrier per stage.  Measured (k = 2048 unless
// stated): 4096 rows of 135K 500 -> 397 us (5.6 TB/s of scores, 6.2 with the
// sample; behind the prefill indexer 8192 rows of 139K take 870 us as before,
// alone 992 -> 813), 64 rows of 32K-158K 55 -> 24, 512 shards of 16K (k = 256)
// 21 -> 13, one row of 13K 27 -> 14, 2048 rows of 8.2K (k = 512) 90 -> 48.
#include "janus_device.hpp"
#include "janus_host.hpp"
#include "launch_rules.hpp"

#include <algorithm>
#include <type_traits>

namespace janus {

constexpr int TK_THREADS = 512;
constexpr int TK_RING = 8;                // 1 KB chunks in flight per wave
constexpr int TK_MAX_K = 6144;            // with CAP = 8192: >= 2048 free slots after a cut
constexpr int TK_SMALL_K = 2048;          // with CAP = 4096
constexpr int TK_BINS = 2048;
constexpr int TK_FEW = 64;                // entries of a bin that are ranked pairwise
constexpr int TK_TIES = 512;              // a bin of more values is narrowed as ties

constexpr int tk_max_k(int cap) { return cap <= 4096 ? TK_SMALL_K : TK_MAX_K; }

template <int CAP>
struct alignas(16) TopkShared {
    static constexpr int WAVES = TK_THREADS / kWave;
    uint32_t key[CAP];
    int32_t id[CAP];   // directly behind key: the output bitmap spans both
    union {
        uint32_t hist[TK_BINS];
        uint16_t pre[2 * CAP];  // set bits before each word of the output bitmap
    };
    int32_t stage[tk_max_k(CAP)];  // ids by rank
    uint32_t few_key[TK_FEW];
    int32_t few_id[TK_FEW];
    int32_t wsum[WAVES];
    uint32_t wmin[WAVES], wmax[WAVES];
    int32_t count;
    int32_t nfew;
    int32_t sel_bin, sel_rem, sel_cnt;
    uint32_t thr_key;  // accept (key, id) > (thr_key, thr_id) in the strict order:
    int32_t thr_id;    //   key > thr_key, or key == thr_key and id < thr_id
    float thr_f;       // thr_key as a score (the same test on floats)
};

// Score of an order-preserving key (inverse of score_key).  Keys below that of
// -inf are not scores; they map to -inf, which only makes a threshold looser.
JANUS_DEV float key_score(uint32_t key)
{
    if (key < 0x007fffffu)
        return -INFINITY;
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// Sets the running threshold (one thread; the caller synchronises).
template <class SM>
JANUS_DEV void set_threshold(SM &sm, uint32_t key, int32_t id)
{
    sm.thr_key = key;
    sm.thr_id = key < 0x007fffffu ? 0x7fffffff : id;
    sm.thr_f = key_score(key);
}

// Wave-uniform buffer resource over [base, base + bytes): loads past the end
// return zeros.
JANUS_DEV __amdgpu_buffer_rsrc_t row_rsrc(const void *base, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    void *p = reinterpret_cast<void *>(((uint64_t)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(p, (short)0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// Exclusive prefix sum over the block; also returns the total.  Ends without
// a barrier: the caller has one before wsum's next use.
template <class SM>
JANUS_DEV int block_exclusive_scan(SM &sm, int v, int &total)
{
    const int wave = threadIdx.x >> 6;
    const int incl = wave_sum_scan(v);
    if ((threadIdx.x & 63) == 63)
        sm.wsum[wave] = incl;
    lds_sync();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < SM::WAVES; ++w) {
        const int s = sm.wsum[w];
        off += (w < wave) ? s : 0;
        tot += s;
    }
    total = tot;
    return off + incl - v;
}

// Smallest and largest of the block's values (two barriers).
template <class SM>
JANUS_DEV void block_extremes(SM &sm, uint32_t &lo, uint32_t &hi)
{
    auto umin = [](int a, int b) { return (int)min((uint32_t)a, (uint32_t)b); };
    auto umax = [](int a, int b) { return (int)max((uint32_t)a, (uint32_t)b); };
    const uint32_t mn = (uint32_t)wave_scan((int)lo, -1, umin), mx = (uint32_t)wave_scan((int)hi, 0, umax);
    if ((threadIdx.x & 63) == 63) {
        sm.wmin[threadIdx.x >> 6] = mn;
        sm.wmax[threadIdx.x >> 6] = mx;
    }
    lds_sync();
    lo = 0xffffffffu;
    hi = 0u;
#pragma unroll
    for (int w = 0; w < SM::WAVES; ++w) {
        lo = min(lo, sm.wmin[w]);
        hi = max(hi, sm.wmax[w]);
    }
    lds_sync();
}

// Narrows [lo, hi], which holds at least `want` of the block's values v (those
// flagged in on), to the bin that holds the want-th largest: at most `few`
// values, or a single value of the range.  On return [lo, hi] is that bin,
// `want` how many of its largest values make up the asked number, and the
// result how many values it holds.
template <int NI, class SM>
JANUS_DEV int narrow(SM &sm, const uint32_t (&v)[NI], uint32_t on, uint32_t &lo, uint32_t &hi, int &want, int few)
{
    constexpr int PER = TK_BINS / TK_THREADS;  // bins per thread of the scan
    int cnt = 0;
    for (int pass = 0; pass < 3; ++pass) {  // 11 bits a pass
        const int bits = 32 - __clz((int)(hi - lo) | 1);
        const int sh = max(0, bits - 11);  // (hi - lo) >> sh < 2048
#pragma unroll
        for (int j = 0; j < PER; ++j)
            sm.hist[threadIdx.x * PER + j] = 0u;
        lds_sync();
        if (__builtin_amdgcn_readfirstlane(cnt) > TK_TIES) {
            // so many values in one bin are mostly ties, which go on to one bin
            // again: a wave of those makes one addition (additions to one
            // address run one after another: 512 rows of 25K, 0.2% of them
            // above zero, 82 -> 57 us, of 131K 112 -> 89)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const bool hit = ((on >> i) & 1u) && v[i] >= lo && v[i] <= hi;
                const uint32_t bin = (v[i] - lo) >> sh;
                const uint64_t act = __ballot(hit);
                if (act == 0)
                    continue;
                const int l = __builtin_ctzll(act);
                const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)bin, l);
                const bool one = __ballot(hit && bin == first) == act;
                if (one ? (int)(threadIdx.x & 63) == l : hit)
                    atomicAdd(&sm.hist[bin], one ? (uint32_t)__popcll(act) : 1u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i)
                if (((on >> i) & 1u) && v[i] >= lo && v[i] <= hi)
                    atomicAdd(&sm.hist[(v[i] - lo) >> sh], 1u);
        }
        lds_sync();
        // thread t holds bins from TK_BINS - 1 - PER t down
        int h[PER], sum = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            h[j] = (int)sm.hist[TK_BINS - 1 - PER * (int)threadIdx.x - j];
            sum += h[j];
        }
        int tot;
        int c = block_exclusive_scan(sm, sum, tot);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (c < want && c + h[j] >= want) {
                sm.sel_bin = TK_BINS - 1 - PER * (int)threadIdx.x - j;
                sm.sel_rem = want - c;
                sm.sel_cnt = h[j];
            }
            c += h[j];
        }
        lds_sync();
        lo += (uint32_t)sm.sel_bin << sh;
        hi = lo + min(hi - lo, (1u << sh) - 1u);
        want = sm.sel_rem;
        cnt = sm.sel_cnt;
        if (cnt <= few || sh == 0)
            break;
        // (the next pass writes sel_* after three more barriers)
    }
    return cnt;
}

// Flags of the k best of the block's buffered entries (those flagged in on, at
// least k of them), and the threshold set to the k-th best or, where all of
// a bin wins, to the bin's lower end.  Ends with a barrier.
template <int NI, class SM>
JANUS_DEV uint32_t best(SM &sm, const uint32_t (&key)[NI], const int32_t (&id)[NI], uint32_t on, int k)
{
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if ((on >> i) & 1u) {
            lo = min(lo, key[i]);
            hi = max(hi, key[i]);
        }
    if (threadIdx.x == 0)
        sm.nfew = 0;
    block_extremes(sm, lo, hi);
    int want = k;
    const int cnt = narrow(sm, key, on, lo, hi, want, TK_FEW);
    uint32_t win = 0, in = 0;  // above the bin, inside it
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        win |= (((on >> i) & 1u) && key[i] > hi ? 1u : 0u) << i;
        in |= (((on >> i) & 1u) && key[i] >= lo && key[i] <= hi ? 1u : 0u) << i;
    }
    if (want == cnt) {  // the whole bin
        win |= in;
        if (threadIdx.x == 0)
            set_threshold(sm, lo, 0x7fffffff);
    } else if (cnt <= TK_FEW) {
        // rank the bin's entries against each other
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if ((in >> i) & 1u) {
                const int at = atomicAdd(&sm.nfew, 1);
                sm.few_key[at] = key[i];
                sm.few_id[at] = id[i];
            }
        lds_sync();
        // (one thread per entry: by their owners, a wave's entries one after
        // another, a bin of 60 ties took 65 us)
        if ((int)threadIdx.x < cnt) {
            const uint32_t mk = sm.few_key[threadIdx.x];
            const int32_t mi = sm.few_id[threadIdx.x];
            int rank = 0;
#pragma unroll 4
            for (int j = 0; j < cnt; ++j)
                rank += sm.few_key[j] > mk || (sm.few_key[j] == mk && sm.few_id[j] < mi);
            if (rank == want - 1)
                set_threshold(sm, mk, mi);
        }
        lds_sync();
        const uint32_t T = sm.thr_key;
        const int32_t I = sm.thr_id;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            win |= (((in >> i) & 1u) && (key[i] > T || (key[i] == T && id[i] <= I)) ? 1u : 0u) << i;
    } else {
        // many ties on one key: its smallest ids, the largest of ~id
        uint32_t inv[NI], ilo = 0xffffffffu, ihi = 0u;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            inv[i] = ~(uint32_t)id[i];
            if ((in >> i) & 1u) {
                ilo = min(ilo, inv[i]);
                ihi = max(ihi, inv[i]);
            }
        }
        block_extremes(sm, ilo, ihi);
        narrow(sm, inv, in, ilo, ihi, want, 1);  // ids differ: a bin of one
#pragma unroll
        for (int i = 0; i < NI; ++i)
            win |= (((in >> i) & 1u) && inv[i] >= ilo ? 1u : 0u) << i;
        if (threadIdx.x == 0)
            set_threshold(sm, lo, (int32_t)~ilo);
    }
    lds_sync();
    return win;
}

// The buffer's entries of this thread (e = threadIdx.x + i TK_THREADS), flagged.
template <int NI, class SM>
JANUS_DEV uint32_t load_entries(const SM &sm, int cnt, uint32_t (&key)[NI], int32_t (&id)[NI])
{
    uint32_t on = 0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int e = (int)threadIdx.x + i * TK_THREADS;
        key[i] = e < cnt ? sm.key[e] : 0u;
        id[i] = e < cnt ? sm.id[e] : -1;
        on |= (id[i] >= 0 ? 1u : 0u) << i;  // (slots left by a stopped wave hold -1)
    }
    return on;
}

// Cuts the full buffer to exactly its k best entries and raises the threshold
// to the k-th best.  Begins and ends with a barrier.
template <int CAP>
__device__ __noinline__ void compact(TopkShared<CAP> &sm, int k)
{
    constexpr int NI = CAP / TK_THREADS;
    uint32_t key[NI];
    int32_t id[NI];
    lds_sync();
    const uint32_t on = load_entries(sm, CAP, key, id);
    const uint32_t win = best(sm, key, id, on, k);
    int tot;
    int pos = block_exclusive_scan(sm, __popc(win), tot);  // (every entry is in registers by now)
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if ((win >> i) & 1u) {
            sm.key[pos] = key[i];
            sm.id[pos] = id[i];
            ++pos;
        }
    if (threadIdx.x == 0)
        sm.count = tot;  // == k
    lds_sync();
}

// Appends this wave's accepted elements among x[0..3] (lane's ids id0 ..
// id0+3, those flagged in pend); false if they found no room (then none is
// in the buffer, and its last slots are marked unused).
template <int CAP, class SM>
JANUS_DEV bool append4(SM &sm, v4f x, uint32_t pend, int id0, float tf, int32_t ti)
{
    bool a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        a[j] = x[j] >= tf && ((pend >> j) & 1u);
    if (__ballot(a[0] || a[1] || a[2] || a[3]) == 0)
        return true;
    // an element equal to the threshold passes only with a smaller id
    uint64_t m[4];
    int tot = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a[j] = a[j] && !(x[j] == tf && id0 + j >= ti);
        m[j] = __ballot(a[j]);
        tot += __popcll(m[j]);
    }
    if (tot == 0)
        return true;
    int base = 0;
    if ((threadIdx.x & 63) == 0)
        base = atomicAdd(&sm.count, tot);
    base = __builtin_amdgcn_readfirstlane(base);
    if (base + tot > CAP) {
        for (int e = base + (int)(threadIdx.x & 63); e < CAP; e += kWave)
            sm.id[e] = -1;
        return false;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int slot = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[j], 0));
        if (a[j]) {
            sm.key[slot] = score_key(x[j]);
            sm.id[slot] = id0 + j;
        }
        base += __popcll(m[j]);
    }
    return true;
}

// One pass over [0, n) of the row, filtering against the running threshold;
// with seed > 0 the threshold is first set from a sample of the row, so that
// about seed * k elements pass.  Ends with a barrier.
template <int CAP>
JANUS_DEV void stream_row(TopkShared<CAP> &sm, const float *__restrict__ row, int n, int k, float seed)
{
    constexpr int NW = TK_THREADS / kWave;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // unaligned head (< 4 elements), 16-byte aligned body of float4s, tail (< 4)
    const int head = min(n, (int)(((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15) >> 2));
    const int nbody4 = (n - head) >> 2;
    const int tail0 = head + (nbody4 << 2);
    const __amdgpu_buffer_rsrc_t body = row_rsrc(row + head, 16u * (uint32_t)nbody4);
    const int nch = (nbody4 + kWave - 1) / kWave;  // 1 KB chunks: wave w takes w, w + NW, ..
    // this lane's float4 at index i of the body (zeros past it)
    auto load4 = [&](int i) {
        return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(body, 16 * i, 0, 0));
    };

    // the sample goes out first, then the head and tail elements and the
    // wave's first chunks; the sample is ranked under their latency
    constexpr int SPT = TK_SAMPLE_GROUPS * 2 / TK_THREADS;  // float4s of the sample per thread
    const int ngroups = nbody4 >> 1;
    const int m4 = seed > 0.f ? min(TK_SAMPLE_GROUPS, ngroups) * 2 : 0;
    v4f smp[SPT];
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        const int e = (int)threadIdx.x + j * TK_THREADS;
        smp[j] = load4(e < m4 ? 2 * tk_sample_group(e >> 1, ngroups) + (e & 1) : nbody4);
    }
    // lanes 0..2 of the first wave take the head, 4..6 the tail
    const int hti = lane < 4 ? lane : tail0 + lane - 4;
    const bool ht = wave == 0 && (lane < 4 ? lane < head : lane < 8 && hti < n);
    const float htv = ht ? row[hti] : 0.f;
    v4f x[TK_RING];
#pragma unroll
    for (int u = 0; u < TK_RING; ++u)
        x[u] = load4((wave + u * NW) * kWave + lane);

    if (seed > 0.f) {
        uint32_t key[4 * SPT], on = 0, lo = 0xffffffffu, hi = 0u;
#pragma unroll
        for (int j = 0; j < SPT; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t kk = score_key(smp[j][c]);
                key[4 * j + c] = kk;
                if ((int)threadIdx.x + j * TK_THREADS < m4) {
                    on |= 1u << (4 * j + c);
                    lo = min(lo, kk);
                    hi = max(hi, kk);
                }
            }
        block_extremes(sm, lo, hi);
        // rank ~ seed * k * (sample / n) + 8; the bin's lower end suffices once
        // the bin holds few of that rank's entries
        int r = min(4 * m4, (int)(seed * (float)k * (float)(4 * m4) / (float)n) + 8);
        narrow(sm, key, on, lo, hi, r, max(4, r >> 3));
        if (threadIdx.x == 0)
            set_threshold(sm, lo, 0x7fffffff);  // accept key >= seed
        lds_sync();
    }

    bool edge = wave == 0;  // the head and tail are still to be appended
    int j = wave;           // this wave's next chunk
    for (bool first = true;; first = false) {
        const float tf = sm.thr_f;
        const int32_t ti = sm.thr_id;
        if (!first) {
#pragma unroll
            for (int u = 0; u < TK_RING; ++u)
                x[u] = load4((j + u * NW) * kWave + lane);
        }
        bool room = true;
        if (edge) {
            room = append4<CAP>(sm, v4f{htv, 0.f, 0.f, 0.f}, ht ? 1u : 0u, hti, tf, ti);
            edge = !room;
        }
        // (one exit: with an early one the compiler moves the loads to the
        // end of the loop and waits for all of them there)
        while (room && j < nch) {
#pragma unroll
            for (int u = 0; u < TK_RING; ++u) {
                const int v4 = j * kWave + lane;
                // (chunks past the row have nothing pending)
                if (room)
                    room = append4<CAP>(sm, x[u], v4 < nbody4 ? 0xfu : 0u, head + 4 * v4, tf, ti);
                x[u] = load4(v4 + TK_RING * NW * kWave);
                j += room ? NW : 0;
            }
        }
        lds_sync();
        if (sm.count <= CAP)
            break;
        compact(sm, k);
    }
}

// After a seed above the k-th key: the row again with a looser seed, then with
// none.  Begins with a barrier.  512 rows of 131K: 65 us with the first seed,
// 91 with the second, 132 where the sample misleads both (two streams, the
// second without a threshold, would be one less, but the streams that filter
// are the cheap ones, and with one seed alone the middle case took the last's).
template <int CAP>
__device__ __noinline__ void stream_again(TopkShared<CAP> &sm, const float *row, int n, int k)
{
    for (float seed = n > CAP ? 3.f : 0.f;; seed = 0.f) {
        lds_sync();
        if (threadIdx.x == 0) {
            sm.count = 0;
            set_threshold(sm, 0u, 0x7fffffff);
        }
        lds_sync();
        stream_row<CAP>(sm, row, n, k, seed);
        if (sm.count >= k || seed == 0.f)
            break;
    }
}

template <int CAP>
__global__ __launch_bounds__(TK_THREADS, CAP <= 4096 ? 4 : 2) void topk_rows(
    const int32_t *__restrict__ q_start, const int32_t *__restrict__ hist_len,
    const int64_t *__restrict__ score_start, int num_seqs, int es,
    const float *__restrict__ scores, int k_row, int32_t *__restrict__ topk_idx, int shards, int align)
{
    __shared__ TopkShared<CAP> sm;
    // causal rows (shards == 0): block g selects k_row of its candidates
    // (tokens: [0, M+i]);
    // sharded rows: block g*shards + n selects k_row/shards of history shard n
    const int g = shards ? blockIdx.x / shards : blockIdx.x;
    const int b = __builtin_amdgcn_readfirstlane(session_of_row_wave(q_start, num_seqs, g));
    const int i = g - q_start[b];
    const int N = q_start[b + 1] - q_start[b];
    const int M = hist_len[b];
    const int ctx = entries_of(M + N, es);
    const int Mh = entries_of(M, es);  // history candidates
    int base = 0, n = last_cand(M, i, es) + 1, k = k_row;
    int32_t *out = topk_idx + (int64_t)g * k_row;
    if (shards) {
        const int sh = blockIdx.x - g * shards;
        const int units = (Mh + align - 1) / align;        // pages of the history
        const int L = align * ((units + shards - 1) / shards);  // candidates per shard
        base = min(Mh, sh * L);
        n = min(Mh, base + L) - base;
        k = k_row / shards;
        out += sh * k;
    }
    const float *row = scores + score_start[b] + (int64_t)i * ctx + base;

    if (n <= k) {
        for (int j = threadIdx.x; j < k; j += TK_THREADS)
            out[j] = j < n ? base + j : -1;
        return;
    }
    if (threadIdx.x == 0) {
        sm.count = 0;
        set_threshold(sm, 0u, 0x7fffffff);  // accept everything
    }
    lds_sync();

    // 1., 2. one streaming pass (more if the seed was above the k-th key)
    stream_row<CAP>(sm, row, n, k, n > CAP ? 1.3f : 0.f);
    if (sm.count < k)
        stream_again<CAP>(sm, row, n, k);
    // 3. the k best of the buffered candidates
    const int cnt = sm.count;
    constexpr int NI = CAP / TK_THREADS;
    uint32_t key[NI], win;
    int32_t id[NI];
    win = load_entries(sm, cnt, key, id);
    if (cnt > k)
        win = best(sm, key, id, win, k);
    else
        lds_sync();
    // 4. ascending output (the bitmap lies over the key and id arrays)
    uint32_t *bm = sm.key;
    const int nwords = (n + 31) >> 5;                          // <= 2 * CAP (checked by the launcher)
    const int wpt = ((nwords + TK_THREADS - 1) / TK_THREADS + 3) & ~3;       // words per thread, whole 16-byte reads
    for (int wd = 4 * threadIdx.x; wd < nwords; wd += 4 * TK_THREADS)
        *(v4i *)(bm + wd) = v4i{0, 0, 0, 0};
    lds_sync();
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if ((win >> i) & 1u)
            atomicOr(&bm[id[i] >> 5], 1u << (id[i] & 31));
    lds_sync();
    const int w0 = threadIdx.x * wpt, w1 = min((nwords + 3) & ~3, w0 + wpt);
    int c = 0;
    for (int wd = w0; wd < w1; wd += 4) {
        const v4i x = *(const v4i *)(bm + wd);
        c += __popc((uint32_t)x[0]) + __popc((uint32_t)x[1]) + __popc((uint32_t)x[2]) + __popc((uint32_t)x[3]);
    }
    int tot;
    int pos = block_exclusive_scan(sm, c, tot);
    for (int wd = w0; wd < w1; wd += 4) {
        const v4i x = *(const v4i *)(bm + wd);
        const uint32_t p0 = pos, p1 = p0 + __popc((uint32_t)x[0]), p2 = p1 + __popc((uint32_t)x[1]),
                       p3 = p2 + __popc((uint32_t)x[2]);
        *(v2i *)(sm.pre + wd) = v2i{(int)(p0 | (p1 << 16)), (int)(p2 | (p3 << 16))};
        pos = (int)(p3 + __popc((uint32_t)x[3]));
    }
    lds_sync();
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if ((win >> i) & 1u) {
            const int wd = id[i] >> 5;
            sm.stage[sm.pre[wd] + __popc(bm[wd] & ((1u << (id[i] & 31)) - 1u))] = base + id[i];
        }
    lds_sync();
    for (int j = threadIdx.x; j < k; j += TK_THREADS)
        out[j] = j < tot ? sm.stage[j] : -1;
}

} // namespace janus

using namespace janus;

// Launch over total_q rows (shards == 0) or total_q * shards (row, shard) pairs.
static int launch_topk(const janus_batch *bt, const float *scores, int k, int32_t *topk_idx, int shards,
                       int align, void *stream)
{
    const int kk = shards ? k / shards : k;
    // the output bitmap spans the key and id arrays: max_ctx <= 2 * CAP * 32
    if (kk > TK_MAX_K || bt->max_ctx > 2 * 8192 * 32)
        return JANUS_ERR_UNSUPPORTED;
    if (bt->total_q == 0)
        return JANUS_OK;
    const dim3 grid((unsigned)bt->total_q * (unsigned)(shards ? shards : 1));
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(TK_THREADS), 0, as_stream(stream), bt->q_start, bt->hist_len,
                           bt->score_start, bt->num_seqs, bt->entry_shift, scores, k, topk_idx, shards, align);
    };
    if (kk <= TK_SMALL_K && bt->max_ctx <= 2 * 4096 * 32)
        go(topk_rows<4096>);
    else
        go(topk_rows<8192>);
    return launch_status();
}

extern "C" int janus_topk(const janus_batch *bt, const float *scores, int k, int32_t *topk_idx,
                          void *workspace, size_t *workspace_bytes, void *stream)
{
    (void)workspace;
    if (workspace_bytes)
        *workspace_bytes = 0;
    if (!batch_ok(bt) || !bt->score_start || !scores || !topk_idx || k < 1)
        return JANUS_ERR_INVALID_ARG;
    return launch_topk(bt, scores, k, topk_idx, 0, 1, stream);
}

extern "C" int janus_topk_sharded(const janus_batch *bt, const float *scores, int k, int num_shards, int align,
                                  int32_t *topk_idx, void *workspace, size_t *workspace_bytes, void *stream)
{
    (void)workspace;
    if (workspace_bytes)
        *workspace_bytes = 0;
    if (!batch_ok(bt) || !bt->score_start || !scores || !topk_idx || k < 1 || num_shards < 1 ||
        k % num_shards != 0 || align < 1)
        return JANUS_ERR_INVALID_ARG;
    return launch_topk(bt, scores, k, topk_idx, num_shards, align, stream);
}
