"""The rules that pick kernels and launch shapes, compiled for the host and
checked on their own."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_36938_amd", "csrc")
WRAP = r"""
#include "launch_rules.hpp"
extern "C" {
int pd_one_block(long q, long k, int nwords) { return janus::pd_one_block(q, k, nwords); }
int prefill_per_xcd(int max_ctx) { return janus::prefill_per_xcd(max_ctx); }
int session_chunk(int ctx, int n) { return janus::session_chunk(ctx, n, janus::prefill_recip(n)); }
void rows_plan(int n, int max_ctx, long total, int max_q, int cus, int fp4, long *out)
{
    const janus::RowsPlan p = janus::rows_plan(n, max_ctx, total, max_q, cus, fp4);
    out[0] = p.chunk, out[1] = p.per_seq, out[2] = p.blocks;
}
int tk_sample_group(int g, int ngroups) { return janus::tk_sample_group(g, ngroups); }
int mqa_shared(long q, long k) { return janus::mqa_shared(q, k); }
int rows_first(int ctx_start, int s, int shift) { return janus::rows_first(ctx_start, s, shift); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(WRAP)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, str(d / "r.cpp"), "-o",
                           str(d / "r.so")])
    return ctypes.CDLL(str(d / "r.so"))


def test_page_demand_one_block(rules):
    one = lambda q, k, nw=40: bool(rules.pd_one_block(ctypes.c_long(q), ctypes.c_long(k), nw))  # noqa: E731
    for q, k in [(1, 1), (2, 2048), (8, 2048), (8, 1), (4, 8192)]:
        assert one(q, k), (q, k)
    # rows are walked one step after another, whatever their ids: many rows take blocks of their own
    for q, k in [(256, 64), (16384, 1), (4096, 4), (64, 256), (128, 128), (9, 1), (8, 8192), (0, 5)]:
        assert not one(q, k), (q, k)
    assert one(2, 64, 1024) and not one(2, 64, 1025) and not one(2, 64, 0)


@pytest.mark.parametrize("shift", [8, 10, 11])
def test_decode_blocks_cover_every_chunk(rules, shift):
    rng = np.random.default_rng(shift)
    for n in (1, 2, 63, 64, 65, 1000):
        ctx = np.where(rng.random(n) < 0.2, 0, np.exp(rng.uniform(0, 12, n)).astype(np.int64))
        ctx[rng.integers(n)] = 7 << shift
        start = np.concatenate([[0], np.cumsum(ctx)])
        first = [rules.rows_first(int(start[s]), s, shift) for s in range(n)] + [(int(start[-1]) >> shift) + n]
        for s in range(n):
            chunks = -(-int(ctx[s]) >> shift)
            assert chunks <= first[s + 1] - first[s] <= chunks + 1


def test_decode_plan(rules):
    def plan(ctx, fp4=0, q=1):
        out = (ctypes.c_long * 3)()
        rules.rows_plan(len(ctx), int(max(ctx)), ctypes.c_long(int(sum(ctx))), q, 256, fp4, out)
        chunk, per_seq, blocks = out
        assert chunk in (256, 512, 1024, 2048, 4096) and blocks < 1 << 24
        # every chunk of every session has a block
        assert per_seq * chunk >= max(ctx) and blocks == per_seq * len(ctx) if per_seq else \
            blocks == sum(ctx) // chunk + len(ctx)
        return chunk, per_seq, blocks, sum(-(-c // chunk) for c in ctx)
    rng = np.random.default_rng(3)
    between = lambda n, lo, hi: [int(c) for c in np.exp(rng.uniform(np.log(lo), np.log(hi), n))]  # noqa: E731
    # measured (sessions, keys of the longest, keys in all, tokens, FP4): the chunks within 5% of the fastest
    # (the rule is 0.9% off in the mean; former ones took up to 34% longer here)
    for n, longest, total, q, fp4, best in [
            (1, 131073, 131073, 1, 0, (512,)), (2, 15970, 27558, 1, 0, (256,)),
            (3, 163841, 491523, 1, 1, (1024,)), (12, 60001, 720012, 1, 0, (1024,)),
            (16, 55086, 509512, 1, 0, (1024,)), (24, 23285, 300492, 2, 0, (1024, 2048)),
            (32, 22841, 398418, 1, 0, (1024, 2048)), (32, 22844, 398514, 4, 0, (1024, 2048)),
            (32, 22844, 398514, 4, 1, (1024,)), (48, 8193, 393264, 1, 0, (1024, 2048)),
            (48, 8194, 393312, 2, 0, (1024, 2048)), (48, 8194, 393312, 2, 1, (1024,)),
            (48, 8196, 393408, 4, 0, (1024, 2048)), (64, 24001, 1536064, 1, 0, (1024, 2048)),
            (64, 23370, 795088, 1, 1, (1024, 2048)), (64, 163841, 2059473, 1, 0, (1024,))]:
        out = (ctypes.c_long * 3)()
        rules.rows_plan(n, longest, ctypes.c_long(total), q, 256, fp4, out)
        assert out[0] in best, (n, longest, total, q, fp4, out[0])
    # sessions of one length: no empty block
    for ctx in ([4000] * 256, [1000] * 4096, [100000] * 64):
        for q in (1, 2, 4):
            _, _, blocks, useful = plan(ctx, 0, q)
            assert blocks == useful
    # one long session among short ones does not set the grid of all
    ragged = [[1000000] + [1000] * 63, [1000000] + [500] * 1023]
    ragged += [between(n, 1000, 270000) for n in (3, 17, 64, 300, 2000) for _ in range(8)]
    for ctx in ragged:
        for fp4 in (0, 1):
            for q in (1, 2, 4):
                _, _, blocks, useful = plan(ctx, fp4, q)
                assert blocks <= max(256, 2 * useful + 16), (len(ctx), blocks, useful)
    for q in (1, 2, 4):
        assert plan([1 << 24], 0, q)[2] and plan([1] * 100000, 0, q)[2] == 100000
        assert plan([1], 0, q)[:3] == (256, 1, 1)


def test_prefill_chunks(rules):
    rng = np.random.default_rng(5)
    assert rules.prefill_per_xcd(1) == 1 and rules.prefill_per_xcd(131072) == 1 and rules.prefill_per_xcd(131073) == 2
    assert rules.prefill_per_xcd(1 << 24) == 128
    for n in list(range(1, 129)):
        for ctx in [0, 1, 7, 8, 9, 8 * n, 8 * n + 1, 1 << 24, (1 << 24) - 1] + list(rng.integers(1, 1 << 24, 200)):
            ctx = int(ctx)
            keys = -(-ctx // (8 * n))
            assert rules.session_chunk(ctx, n) == -(-keys // 128) * 128, (ctx, n)


def test_topk_sample_spans_the_row(rules):
    for n in list(range(513)) + [1022, 1023, 1024, 1025, 2047, 5000, 16384, 65535, 1 << 16]:
        g = [rules.tk_sample_group(j, n) for j in range(min(n, 512))]
        assert g == sorted(set(g)) and (not g or g[0] == 0 and g[-1] < n)
        # no stretch of the row longer than one and a half shares is left out, the end neither
        assert all(b - a <= 1.5 * n / 512 + 1 for a, b in zip(g, g[1:] + [n]))


def test_mqa_shared(rules):
    def shared(q, k):
        return bool(rules.mqa_shared(ctypes.c_long(q), ctypes.c_long(k)))
    # measured: one token per block faster, then one token per wave
    for q, k in [(8, 256), (250, 256), (500, 256), (512, 256), (1100, 256), (260, 512), (520, 512), (1100, 512),
                 (2100, 512), (256, 1024), (768, 1024), (1100, 1024), (1500, 1024), (2100, 1024)]:
        assert shared(q, k), (q, k)
    for q, k in [(1000, 32), (6000, 32), (1000, 100), (2048, 100), (1000, 256), (1500, 256), (3000, 256), (1024, 512),
                 (2048, 512), (4096, 512), (1000, 1024), (2048, 1024), (3000, 1024)]:
        assert not shared(q, k), (q, k)
