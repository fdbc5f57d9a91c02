// Page demand (the union of the per-token selections, mapped through the page
// table to physical pages), read packing (Sec. 4.3: one read per maximal run
// of selected, physically adjacent pages, split from the low end at max_run)
// and the corrective-read set of Eq. (2) (actual minus predicted pages).
//
// Union: each block takes a contiguous range of query rows, four rows' ids in
// flight at a time, maps every valid id to its physical page and sets it in
// an LDS bitmap (read-before-set, so the hot pages that every row selects cost
// one LDS read, not an atomic; ids of one thread on one logical page, as
// ascending selections have them, are looked up once); the block then ORs its
// non-empty words into the global bitmap.
// Lists and runs: a block stages the whole bitmap in LDS (at most 64 KB) and
// emits a slice of RUN_THREADS words, one word per thread: what lies before
// the slice (pages, run starts, the last unset page) it counts itself, so that
// the slices need nothing from each other.
// Few rows: one block does all of it, in one launch instead of three (pd_one_block).
//
// What bounds all of these is latency: chains of loads and barriers, and the
// launches.  Measured: the union of 4096 rows of 2048 ids 28 -> 10 us, of 64
// rows 20 -> 5; list and runs of 81K pages 12 -> 10.6; two rows in one launch 7.1
// us instead of 1 + 7 + 12 in three.
#include "janus_device.hpp"
#include "janus_host.hpp"
#include "launch_rules.hpp"

#include <algorithm>

namespace janus {

constexpr int PD_THREADS = 512;
constexpr int PD_MAX_BLOCKS = 1024;
constexpr int RUN_WAVES = RUN_THREADS / kWave;
constexpr int PD_MAX_PAGES = 1 << 19;  // 64 KB LDS bitmap

__global__ void bitmap_zero(uint32_t *__restrict__ bm, int nwords)
{
    int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w < nwords)
        bm[w] = 0u;
}

struct UnionArgs {
    const int32_t *q_start, *hist_len;
    int num_seqs, es;
    const int32_t *topk_idx;
    int k, vec;  // vec: rows of ids may be read 16 bytes at a time
    const int32_t *page_table;
    int pt_ld, page_shift;
    const int32_t *limit;
};

// Sets the pages of rows [r0, r1) in the LDS bitmap; T threads.
template <int T>
JANUS_DEV void union_rows(const UnionArgs &u, int r0, int r1, uint32_t *sbm)
{
    if (r0 >= r1)
        return;
    int b = __builtin_amdgcn_readfirstlane(session_of_row_wave(u.q_start, u.num_seqs, r0));
    int next = u.q_start[b + 1];
    // the session's id limit and page table
    auto limit_of = [&](int s, int begin, int end) {
        const int ctx = entries_of(u.hist_len[s] + (end - begin), u.es);
        return min(ctx, u.limit ? u.limit[s] : entries_of(u.hist_len[s], u.es));
    };
    int lim = limit_of(b, u.q_start[b], next);
    const int32_t *pt = u.page_table + (int64_t)b * u.pt_ld;
    for (int r = r0; r < r1; r += PD_ROWS) {
        int lims[PD_ROWS];
        const int32_t *pts[PD_ROWS];
#pragma unroll
        for (int i = 0; i < PD_ROWS; ++i) {
            lims[i] = 0;  // rows past the end select nothing
            pts[i] = pt;
            if (r + i < r1) {
                if (r + i >= next) {
                    while (r + i >= next) {
                        ++b;
                        next = u.q_start[b + 1];
                    }
                    lim = limit_of(b, u.q_start[b], next);
                    pt = u.page_table + (int64_t)b * u.pt_ld;
                }
                lims[i] = lim;
                pts[i] = pt;
            }
        }
        for (int j0 = 0; j0 < u.k; j0 += 4 * T) {
            // this thread's four ids of each row: consecutive ones, or T apart
            v4i id[PD_ROWS];
            const int j = u.vec ? j0 + 4 * (int)threadIdx.x : j0 + (int)threadIdx.x;
#pragma unroll
            for (int i = 0; i < PD_ROWS; ++i) {
                id[i] = v4i{-1, -1, -1, -1};
                const int32_t *row = u.topk_idx + (int64_t)(r + i) * u.k;
                if (r + i < r1) {
                    if (u.vec) {
                        if (j < u.k)
                            id[i] = *(const v4i *)(row + j);
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (j + c * T < u.k)
                                id[i][c] = row[j + c * T];
                    }
                }
            }
            int page[PD_ROWS][4];
#pragma unroll
            for (int i = 0; i < PD_ROWS; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int s = id[i][c];
                    page[i][c] = -1;
                    const bool dup = c > 0 && id[i][c > 0 ? c - 1 : 0] >= 0 && id[i][c > 0 ? c - 1 : 0] < lims[i] &&
                                     (id[i][c > 0 ? c - 1 : 0] >> u.page_shift) == (s >> u.page_shift);
                    if (s >= 0 && s < lims[i] && !dup)
                        page[i][c] = pts[i][s >> u.page_shift];
                }
#pragma unroll
            for (int i = 0; i < PD_ROWS; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int p = page[i][c];
                    if (p >= 0) {
                        const uint32_t bit = 1u << (p & 31);
                        if (!(sbm[p >> 5] & bit))
                            atomicOr(&sbm[p >> 5], bit);
                    }
                }
        }
    }
}

__global__ __launch_bounds__(PD_THREADS) void page_union(UnionArgs u, int total_q, int nwords,
                                                         uint32_t *__restrict__ bitmap)
{
    extern __shared__ uint32_t sbm[];
    for (int w = threadIdx.x; w < nwords; w += PD_THREADS)
        sbm[w] = 0u;
    lds_sync();
    const int rows_per = (total_q + gridDim.x - 1) / gridDim.x;
    const int r0 = min(total_q, (int)blockIdx.x * rows_per);
    union_rows<PD_THREADS>(u, r0, min(total_q, r0 + rows_per), sbm);
    lds_sync();
    for (int w = threadIdx.x; w < nwords; w += PD_THREADS) {
        const uint32_t v = sbm[w];
        if (v && (__atomic_load_n(&bitmap[w], __ATOMIC_RELAXED) & v) != v)
            atomicOr(&bitmap[w], v);
    }
}

struct RunShared {
    int32_t a[RUN_WAVES], b[RUN_WAVES], c[RUN_WAVES], d[RUN_WAVES];
    int32_t fz[RUN_THREADS];  // first unset page from thread t's words on
};

JANUS_DEV int op_add(int a, int b) { return a + b; }
JANUS_DEV int op_max(int a, int b) { return max(a, b); }
JANUS_DEV int op_min(int a, int b) { return min(a, b); }

// Block-wide inclusive scans of two values over RUN_THREADS threads, with
// their totals and one barrier; s, t: one scratch value per wave each, free
// until the next barrier after this call.  before_a: a's scan over the threads
// before this one.
template <class OpA, class OpB>
JANUS_DEV void run_scan2(int32_t *s, int32_t *t, int &a, int unit_a, OpA op_a, int &b, int unit_b, OpB op_b,
                         int &before_a, int &total_a, int &total_b)
{
    const int wave = threadIdx.x >> 6;
    const int ia = wave_scan(a, unit_a, op_a), ib = wave_scan(b, unit_b, op_b);
    if ((threadIdx.x & 63) == 63) {
        s[wave] = ia;
        t[wave] = ib;
    }
    lds_sync();
    int ba = unit_a, bb = unit_b;
    total_a = unit_a;
    total_b = unit_b;
#pragma unroll
    for (int w = 0; w < RUN_WAVES; ++w) {
        const int x = s[w], y = t[w];
        ba = w < wave ? op_a(ba, x) : ba;
        bb = w < wave ? op_b(bb, y) : bb;
        total_a = op_a(total_a, x);
        total_b = op_b(total_b, y);
    }
    before_a = op_a(ba, dpp_move<0x138, 0xf>(unit_a, ia));  // lane - 1's scan (none in lane 0)
    a = op_a(ba, ia);
    b = op_b(bb, ib);
}

// Run starts among the pages of word w (bits v), and their pieces emitted: a
// maximal run of set pages is cut from its low end into pieces of max_run.
// last_zero: the last unset page before the word.
template <class Emit>
JANUS_DEV int run_starts(int w, uint32_t v, int last_zero, int max_run, Emit emit)
{
    int n = 0;
    while (v) {
        const int i = __ffs(v) - 1;
        const uint32_t rest = ~(v >> i);
        const int len = rest ? __ffs(rest) - 1 : 32;  // set pages from i on (at most 32 - i: zeros are shifted in)
        const int lo = (w << 5) + i, hi = lo + min(len, 32 - i);
        // the first piece that starts at or after lo: lo itself, unless the run began before this word
        int skip = 0;
        if (i == 0 && last_zero != lo - 1) {
            const int m = (lo - last_zero - 1) % max_run;
            skip = m ? max_run - m : 0;
        }
        if (skip < hi - lo) {
            for (int p = lo + skip;; p += max_run) {
                emit(n, p, hi);
                ++n;
                if (max_run >= hi - p)
                    break;
            }
        }
        if (i + len >= 32)
            break;
        v &= ~0u << (i + len);
    }
    return n;
}

// Run starts among the pages of word w: run_starts' count.  With max_run >= 32
// a word's runs have one start each, but the one that began before the word,
// which has one at most.
JANUS_DEV int count_starts(int w, uint32_t v, int last_zero, int max_run)
{
    if (max_run < 32)
        return run_starts(w, v, last_zero, max_run, [](int, int, int) {});
    int n = __popc(v & ~(v << 1));
    if ((v & 1u) && last_zero != (w << 5) - 1) {
        const int len = ~v ? __ffs(~v) - 1 : 32, m = ((w << 5) - last_zero - 1) % max_run;
        n -= m != 0 && max_run - m >= len ? 1 : 0;
    }
    return n;
}

// Walks the pages of the bitmap sw in LDS (nbits bits in whole 32-bit words,
// zeros past them): writes, for this block's slice of RUN_THREADS words, one per
// thread, the ascending page list (if list != NULL) and the packed runs, and in
// the first block the two counts.  ONE: the bitmap has at most RUN_THREADS words,
// and bits past nbits are ignored; that a thread's range is one word is then known
// to the compiler (page_demand_small of 2 rows 7.5 -> 7.1 us).
template <bool ONE>
JANUS_DEV void emit_list_runs(RunShared &sh, const uint32_t *sw, int nbits, int max_run, int32_t *list, int32_t *runs,
                              int32_t *n_pages_out, int32_t *n_runs_out)
{
    const int nwords = (nbits + 31) >> 5, tid = threadIdx.x;
    const int wpt = ONE ? 1 : max(1, (nwords + RUN_THREADS - 1) / RUN_THREADS);  // words of a thread's range
    const uint32_t last_mask = nbits & 31 ? (1u << (nbits & 31)) - 1u : ~0u;
    auto word = [&](int w) { return ONE && w == nwords - 1 ? sw[w] & last_mask : sw[w]; };
    auto last_unset = [&](int w, uint32_t v) { return (w << 5) + 31 - __clz((int)~v); };  // v not all ones
    // over ranges of wpt words: the first unset page from each range on
    // (ranges taken from the end), the last one before each
    int before;
    {
        const int t = RUN_THREADS - 1 - tid, e0 = min(nwords, t * wpt), e1 = min(nwords, e0 + wpt);
        int fz = nbits, lz = -1, tf, tl;
        for (int w = e1 - 1; w >= e0; --w)
            if (word(w) != 0xffffffffu)
                fz = min(nbits, (w << 5) + __ffs(~word(w)) - 1);
        const int a0 = min(nwords, tid * wpt), a1 = min(nwords, a0 + wpt);
        for (int w = a0; w < a1; ++w)
            if (word(w) != 0xffffffffu)
                lz = last_unset(w, word(w));
        run_scan2(sh.a, sh.b, lz, -1, op_max, fz, nbits, op_min, before, tl, tf);
        sh.fz[t] = fz;
    }
    // the first unset page after word w
    auto first_zero = [&](int w) {
        for (int x = w + 1; x < nwords; ++x) {
            if (wpt == 1 || x % wpt == 0)  // a range's first word
                return sh.fz[wpt == 1 ? x : x / wpt];
            if (word(x) != 0xffffffffu)
                return min(nbits, (x << 5) + __ffs(~word(x)) - 1);
        }
        return nbits;
    };
    // one slice, and what lies before it: nothing, or counted here
    const int s0 = blockIdx.x * RUN_THREADS, w = s0 + tid;
    const uint32_t v = w < nwords ? word(w) : 0u;
    int pages_before = 0, starts_before = 0, lb = before, unused;
    if (wpt > 1) {
        int pages = 0, starts = 0, L = before, zl = -1, zero_before, one = 0;
        const int a0 = min(nwords, tid * wpt), a1 = min(nwords, a0 + wpt);
        for (int x = a0; x < a1; ++x) {
            const uint32_t y = word(x);
            if (s0 == 0 || x < s0) {  // (the first block counts everything, for the totals)
                pages += __popc(y);
                starts += count_starts(x, y, L, max_run);
            }
            if (y != 0xffffffffu) {
                L = last_unset(x, y);
                if (x < s0)
                    zl = L;
            }
        }
        run_scan2(sh.c, sh.d, pages, 0, op_add, starts, 0, op_add, unused, pages_before, starts_before);
        run_scan2(sh.a, sh.b, zl, -1, op_max, one, 0, op_add, unused, zero_before, unused);
        if (s0 == 0) {
            if (tid == 0) {
                if (n_pages_out)
                    *n_pages_out = pages_before;
                *n_runs_out = starts_before;
            }
            pages_before = starts_before = 0;
        }
        int z = w < nwords && v != 0xffffffffu ? last_unset(w, v) : -1;
        run_scan2(sh.c, sh.d, z, -1, op_max, one, 0, op_add, lb, unused, unused);
        lb = max(lb, zero_before);
    }
    int np = __popc(v), ns = count_starts(w, v, lb, max_run), tp, ts, pages_at;
    const int own_starts = ns;
    run_scan2(wpt > 1 ? sh.a : sh.c, wpt > 1 ? sh.b : sh.d, np, 0, op_add, ns, 0, op_add, pages_at, tp, ts);
    if (wpt == 1 && s0 == 0 && tid == 0) {
        if (n_pages_out)
            *n_pages_out = tp;
        *n_runs_out = ts;
    }
    int pos = pages_before + pages_at;
    const int rpos = starts_before + ns - own_starts;
    if (list)
        for (uint32_t x = v; x; x &= x - 1u)
            list[pos++] = (w << 5) + __ffs(x) - 1;
    if (own_starts)
        run_starts(w, v, lb, max_run, [&](int n, int p, int hi) {
            const int end = (hi & 31) == 0 ? first_zero(w) : hi;  // a run up to the word's end may go on
            *(v2i *)(runs + 2 * (int64_t)(rpos + n)) = v2i{p, min(max_run, end - p)};
        });
}

// The bitmap's words, with zeros past nbits
JANUS_DEV uint32_t masked_word(const uint32_t *bm, int w, int nbits)
{
    const int hi = nbits - (w << 5);
    return hi < 32 ? bm[w] & ((1u << hi) - 1u) : bm[w];
}

__global__ __launch_bounds__(RUN_THREADS) void page_list_runs(const uint32_t *__restrict__ bitmap, int nbits,
                                                              int max_run, int32_t *__restrict__ list,
                                                              int32_t *__restrict__ runs, int32_t *n_pages,
                                                              int32_t *n_runs)
{
    __shared__ RunShared sh;
    extern __shared__ uint32_t sw[];  // the bitmap's words
    const int nwords = (nbits + 31) >> 5;
    for (int w = threadIdx.x; w < nwords; w += RUN_THREADS)
        sw[w] = masked_word(bitmap, w, nbits);
    lds_sync();
    emit_list_runs<false>(sh, sw, nbits, max_run, list, runs, n_pages, n_runs);
}

// All of page demand in one block
__global__ __launch_bounds__(RUN_THREADS) void page_demand_small(UnionArgs u, int total_q, int nbits, int max_run,
                                                                 uint32_t *__restrict__ bitmap,
                                                                 int32_t *__restrict__ list,
                                                                 int32_t *__restrict__ runs,
                                                                 int32_t *__restrict__ counts)
{
    __shared__ RunShared sh;
    extern __shared__ uint32_t sw[];
    const int nwords = (nbits + 31) >> 5;
    for (int w = threadIdx.x; w < nwords; w += RUN_THREADS)
        sw[w] = 0u;
    lds_sync();
    union_rows<RUN_THREADS>(u, 0, total_q, sw);
    lds_sync();
    for (int w = threadIdx.x; w < nwords; w += RUN_THREADS)
        bitmap[w] = sw[w];
    emit_list_runs<true>(sh, sw, nbits, max_run, list, runs, counts, counts + 1);
}

// A block reads both bitmaps whole before it writes anything, so that one
// block alone may write over them (in place: see the launch).
__global__ __launch_bounds__(RUN_THREADS) void predict_diff_kernel(const uint32_t *actual, const uint32_t *predicted,
                                                                   int nbits, int max_run, uint32_t *miss,
                                                                   int32_t *miss_runs, int32_t *counts)
{
    __shared__ RunShared sh;
    extern __shared__ uint32_t sw[];  // the miss set's words
    const int nwords = (nbits + 31) >> 5;
    int ca = 0, cp = 0, cap = 0;
    for (int w = threadIdx.x; w < nwords; w += RUN_THREADS) {
        const uint32_t a = masked_word(actual, w, nbits), p = masked_word(predicted, w, nbits);
        ca += __popc(a);
        cp += __popc(p);
        cap += __popc(a & p);
        sw[w] = a & ~p;
    }
    if (blockIdx.x == 0) {
        int na, np, nap, unused, one = 0;
        run_scan2(sh.a, sh.b, ca, 0, op_add, cp, 0, op_add, unused, na, np);
        run_scan2(sh.c, sh.d, cap, 0, op_add, one, 0, op_add, unused, nap, unused);
        if (threadIdx.x == 0) {
            counts[0] = na;
            counts[1] = np;
            counts[2] = nap;
            counts[3] = na - nap;
        }
    }
    lds_sync();  // the staged words are read from here on
    for (int w = blockIdx.x * RUN_THREADS + threadIdx.x; w < nwords; w += gridDim.x * RUN_THREADS)
        miss[w] = sw[w];
    emit_list_runs<false>(sh, sw, nbits, max_run, nullptr, miss_runs, nullptr, counts + 4);
}

} // namespace janus

using namespace janus;

// Blocks of the list and run kernels: one per slice of words
static int run_blocks(int nwords) { return std::max(1, ceil_div(nwords, RUN_THREADS)); }

extern "C" int janus_page_demand(const janus_batch *bt, const int32_t *topk_idx, int k,
                                 const int32_t *page_table, int pt_ld, int page_size, const int32_t *limit,
                                 int num_phys_pages, int max_run, uint32_t *bitmap, int32_t *page_list,
                                 int32_t *runs, int32_t *counts, void *workspace, size_t *workspace_bytes,
                                 void *stream)
{
    (void)workspace;
    if (workspace_bytes)
        *workspace_bytes = 0;
    if (!batch_ok(bt) || !topk_idx || !page_table || !bitmap || !page_list || !runs || !counts || k < 1 ||
        pt_ld < 1 || !pow2(page_size) || !table_covers(bt, pt_ld, page_size) || num_phys_pages < 0 || max_run < 1)
        return JANUS_ERR_INVALID_ARG;
    if (num_phys_pages > PD_MAX_PAGES)
        return JANUS_ERR_UNSUPPORTED;
    hipStream_t st = as_stream(stream);
    const int nwords = (num_phys_pages + 31) >> 5;
    const size_t lds = std::max(nwords, 1) * sizeof(uint32_t);
    const int vec = k % 4 == 0 && (reinterpret_cast<uintptr_t>(topk_idx) & 15) == 0;
    const UnionArgs u = {bt->q_start, bt->hist_len, bt->num_seqs, bt->entry_shift, topk_idx, k, vec, page_table,
                         pt_ld, __builtin_ctz((unsigned)page_size), limit};
    if (pd_one_block(bt->total_q, k, nwords)) {
        hipLaunchKernelGGL(page_demand_small, dim3(1), dim3(RUN_THREADS), lds, st, u, (int)bt->total_q,
                           num_phys_pages, max_run, bitmap, page_list, runs, counts);
        return launch_status();
    }
    if (nwords > 0)
        hipLaunchKernelGGL(bitmap_zero, dim3(ceil_div(nwords, 256)), dim3(256), 0, st, bitmap, nwords);
    if (bt->total_q > 0 && nwords > 0)
        hipLaunchKernelGGL(page_union, dim3(std::min<int>(PD_MAX_BLOCKS, bt->total_q)), dim3(PD_THREADS), lds, st, u,
                           (int)bt->total_q, nwords, bitmap);
    hipLaunchKernelGGL(page_list_runs, dim3(run_blocks(nwords)), dim3(RUN_THREADS), lds, st, bitmap, num_phys_pages,
                       max_run, page_list, runs, counts, counts + 1);
    return launch_status();
}

extern "C" int janus_predict_diff(const uint32_t *actual, const uint32_t *predicted, int num_phys_pages,
                                  int max_run, uint32_t *miss, int32_t *miss_runs, int32_t *counts, void *stream)
{
    if (!actual || !predicted || !miss || !miss_runs || !counts || num_phys_pages < 0 || max_run < 1)
        return JANUS_ERR_INVALID_ARG;
    if (num_phys_pages > PD_MAX_PAGES)
        return JANUS_ERR_UNSUPPORTED;
    const int nwords = (num_phys_pages + 31) >> 5, nblk = run_blocks(nwords);
    const size_t words = (size_t)nwords * sizeof(uint32_t), lds = std::max<size_t>(words, sizeof(uint32_t));
    auto over = [&](const void *out, size_t n, const void *in) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(out), b = reinterpret_cast<uintptr_t>(in);
        return a < b + words && b < a + n;
    };
    auto over_inputs = [&](const void *out, size_t n) { return over(out, n, actual) || over(out, n, predicted); };
    // an output over an input: the other blocks would still read what the
    // first one writes, so one block writes the miss set and the counts, and
    // a launch after it the runs of all slices
    const bool alone = nblk > 1 && (over_inputs(miss, words) || over_inputs(counts, 5 * sizeof(int32_t)) ||
                                    over_inputs(miss_runs, 2 * sizeof(int32_t) * (size_t)num_phys_pages));
    hipLaunchKernelGGL(predict_diff_kernel, dim3(alone ? 1 : nblk), dim3(RUN_THREADS), lds, as_stream(stream), actual,
                       predicted, num_phys_pages, max_run, miss, miss_runs, counts);
    if (alone)
        hipLaunchKernelGGL(page_list_runs, dim3(nblk), dim3(RUN_THREADS), lds, as_stream(stream), miss, num_phys_pages,
                           max_run, (int32_t *)nullptr, miss_runs, (int32_t *)nullptr, counts + 4);
    return launch_status();
}
