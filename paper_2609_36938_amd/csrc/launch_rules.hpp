// Rules by which the C ABI picks a kernel or the shape of a launch, as plain
// functions of sizes: they can be evaluated without a GPU.
#pragma once

#include <stdint.h>

namespace janus {

// ---- page demand: one block for all of it, or three launches -----------------

constexpr int PD_ROWS = 4;          // rows in flight per block
constexpr int RUN_THREADS = 1024;   // the one block, and the list and run kernel's
constexpr int PD_SMALL_STEPS = 2;

// Steps that one block takes over the ids, one after another: PD_ROWS rows at
// a time, four ids of each row per thread.
constexpr int64_t pd_steps(int64_t total_q, int64_t k)
{
    return ((total_q + PD_ROWS - 1) / PD_ROWS) * ((k + 4 * RUN_THREADS - 1) / (4 * RUN_THREADS));
}

// A step is a chain of dependent loads, about 2 us however few ids it has, and
// many rows would be walked by one block alone.  Measured, one block against
// three launches: 8 rows of 2048 ids 12.9 against 13 us (and two launches
// less for the host), 12 of 1024 14.9 against 12.9, 64 of 256 46 against 14,
// 256 of 64 162 against 18.  (The one block has a word of the bitmap per thread.)
constexpr bool pd_one_block(int64_t total_q, int64_t k, int nwords)
{
    return total_q > 0 && nwords > 0 && nwords <= RUN_THREADS && pd_steps(total_q, k) <= PD_SMALL_STEPS;
}

// ---- prefill indexer: key chunks of a session -----------------------------------

constexpr int IDX_XCD = 8;            // L2 domains (XCDs) of the chip
constexpr int IDX_STAGE = 128;        // keys per LDS stage
constexpr int IDX_KEY_CHUNK = 16384;  // target keys per block: long blocks spread each block's query and weight loads over more keys

// Chunks per XCD of every session: the longest session's are at most
// IDX_KEY_CHUNK keys long.  Contexts up to 2^24: at most 128.
constexpr int prefill_per_xcd(int max_ctx)
{
    const int per = ((max_ctx + IDX_XCD - 1) / IDX_XCD + IDX_KEY_CHUNK - 1) / IDX_KEY_CHUNK;
    return per > 1 ? per : 1;
}
// ceil(2^31 / n): the division by n that session_chunk makes, as a multiplication
constexpr unsigned prefill_recip(int n) { return ((1u << 31) + (unsigned)n - 1) / (unsigned)n; }

// Keys of one chunk of a session: its context over the launch's chunk count
// (IDX_XCD * n), in whole stages.  Every session has chunks on every XCD that
// way; with the chunk length of the longest session, a shorter one had only the
// first chunks, so that the last XCDs idled (eight sessions of 10K to 51K
// tokens, MXFP4 keys: 3995 -> 2998 us; sixteen of 0.5K to 131K, fp8 keys: 2948
// -> 950).  x = ceil(ctx / 8) + n - 1 is below 2^22 and the reciprocal's error
// below n <= 2^7 in 2^31, so that x * recip >> 31 is the exact quotient: a
// block's first loads wait for it, and with a division appends of 5 to 200
// tokens took 1% longer (fp8 keys, 16K tokens: 47.9 against 47.4 us).  About half
// of that is where the main loop then lay: its place against 32 bytes moves the
// three prefill kernels by up to 0.8%, and MXFP4's lies 0.7% better with the
// division (131K + 64 tokens: 172.5 and 173.5 us).
constexpr int session_chunk(int ctx, int n, unsigned recip)
{
    const unsigned x = (unsigned)((ctx + IDX_XCD - 1) / IDX_XCD + n - 1);
    const int keys = (int)((unsigned long long)x * recip >> 31);
    return (keys + IDX_STAGE - 1) / IDX_STAGE * IDX_STAGE;
}

// ---- decode indexer: blocks of a batch ----------------------------------------

// First block of session s, whose keys start at ctx_start, in chunks of 2^shift
// keys: each session has as many blocks as chunks, or one more, and no block
// needs the sessions before its own.
constexpr int rows_first(int ctx_start, int s, int shift) { return (ctx_start >> shift) + s; }

// Keys per block of a decode batch, and how its blocks are numbered.
struct RowsPlan {
    int chunk;       // keys per block, 4096 down to 256 (one 64-key group per wave)
    int per_seq;     // blocks of every session, or 0: numbered by rows_first
    int64_t blocks;
};
constexpr int ROWS_CHUNK_MIN = 256;
constexpr int64_t ROWS_MAX_BLOCKS = (1 << 24) - 1;  // a launch takes fewer than 2^32 threads

// The chunk with the shortest time estimated, in keys of one block alone on its
// CU, by the blocks that the fullest CU takes (a session of C keys makes about
// C / chunk + 1/2; one block more than the CUs is left out: the last key of a
// power of two and one).  The first block costs its start and its keys.  Each
// next one that is resident beside it (with one token per session 3 blocks a CU,
// 4 with FP4 keys, else 2) runs mostly under it, but for what the memory takes for its keys; with
// the CU full, the next one costs like the first.  The constants are fitted to
// 1071 batches of 1 to 4096 sessions of 500 to 1M keys, even and ragged, with 1,
// 2 and 4 tokens and both key types: the chunk taken is 0.9% off the best one in
// the mean with keys from HBM and 1.3% with keys in the cache.  The chunk that
// fills rounds of resident blocks best was 7.3% and 10% off, whole chunks per CU
// with a fixed cost per block 3.3% and 4.2% (us, the three in turn, fp8 keys: 16
// sessions of 15K to 60K 19.4, 19.4, 25.8; 48 of 8192 with 2 tokens 19.1, 18.8,
// 23.8; 256 of 4000 32.0, 40.6, 32.0; one of 1M with 63 of 1K and 2 tokens 42, 51,
// 42; 64 of 32K to 164K 151, 151, 150).
// Blocks are numbered by rows_first unless the grid of the longest session's
// chunks for each session needs no more of them, or has each on a CU of its own:
// it saves the search, 0.2 us.
constexpr RowsPlan rows_plan(int num_seqs, int max_ctx, int64_t total_ctx, int max_q, int cus, bool fp4)
{
    const bool one = max_q <= 1;
    const int resident = one ? fp4 ? 4 : 3 : 2;
    const int start = fp4 ? one ? 512 : 384 : 128, beside = fp4 ? one ? 384 : 256 : one ? 448 : 1024;
    RowsPlan best = {0, 0, 0};
    double best_cost = -1.0;
    for (int c = one ? 2048 : 4096; c >= ROWS_CHUNK_MIN; c /= 2) {
        const int per_seq = (max_ctx + c - 1) / c;
        const int64_t grid = (int64_t)num_seqs * per_seq, numbered = total_ctx / c + num_seqs;
        const bool even = grid <= numbered || grid <= cus;
        const int64_t blocks = even ? grid : numbered;
        if (best.chunk && blocks > ROWS_MAX_BLOCKS)
            break;
        const double about = (double)total_ctx / c + 0.5 * num_seqs;
        const double useful = about < (double)grid ? about : (double)grid;
        const double first = c + start, memory = 0.6 * c, under = 0.2 * c + beside;
        const double next = under > memory ? under : memory;
        int64_t n = (int64_t)((useful - 1.0) / cus);  // blocks after the fullest CU's first
        if (n > 0 && (double)n * cus >= useful - 1.0)
            --n;
        const int64_t refills = n / resident;
        const double cost = first + (double)(n - refills) * next + (double)refills * (first > next ? first : next);
        if (best_cost < 0.0 || cost < best_cost) {
            best_cost = cost;
            best = RowsPlan{c, even ? per_seq : 0, blocks};
        }
    }
    return best;
}

// ---- top-k: the sample that seeds a row's threshold ----------------------------

constexpr int TK_SAMPLE_GROUPS = 512;  // ~1/32 of a 128K row, in 8-element groups

// Group of a row of ngroups groups that is the sample's g-th, over the whole
// row.  A whole stride (ngroups / TK_SAMPLE_GROUPS) left out up to half of a
// short row, its end, and a row with its high scores ahead of that was streamed
// again: 512 rows of 8184 descending scores (k = 512) 31.3 us, now 10.9.
// (ngroups <= 2^16 by the launcher's bound on contexts: the product fits.)
constexpr int tk_sample_group(int g, int ngroups)
{
    return ngroups <= TK_SAMPLE_GROUPS ? g : (int)((unsigned)g * (unsigned)ngroups / TK_SAMPLE_GROUPS);
}

// ---- MQA attention: one token per wave, or the block's waves on one token ------

constexpr int MQA_WAVES = 4;  // waves per block

// Whether a block's four waves share one token.  A batch takes rounds of one
// block per CU, of which the whole chip has 256 (asking the device took 0.4 of
// the 12 us of a small call, and a part of a chip only gets the slower form).
// One round's time in ns, fitted to 270 batches of 8 to 6000 rows of 32 to 1024
// ids with 1, 8 and 16 heads (which differ by 5%): 3400 + 12 k for a shared
// token, 3800 + 49 k for four.  The rule takes the faster form of all of them to
// within 2% (256 ids: 500 rows 13.8 us shared, 18.6 else, 768 rows 19.5 and 19.1;
// 512 ids: 1024 rows 39 and 31, 1100 rows 46 and 58).  Up to 100 ids, three or
// four tiles for four waves, the forms take as long as each other in one round,
// and longer batches keep a token per wave.
constexpr bool mqa_shared(int64_t total_q, int64_t k)
{
    const int64_t one = (total_q + 255) / 256;
    const int64_t four = (total_q + 256 * MQA_WAVES - 1) / (256 * MQA_WAVES);
    return k > 100 && one * (3400 + 12 * k) < four * (3800 + 49 * k);
}

} // namespace janus
