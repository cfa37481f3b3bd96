"""Which kernel a GEMM call takes, a host query: the calls below were measured on both
kernels, and the one named is the faster (the times are beside the rule)."""
import math
import random

import pytest

import paper_2409_20361_amd as rrs


@pytest.mark.parametrize("M,K,N,g,tiled,path", [
    # the eight-wave weight stream at K = 8192, 17 to 32 tokens
    (16, 8192, 28672, 128, False, "stream"), (17, 8192, 28672, 128, False, "stream"),
    (32, 8192, 256, 64, False, "stream"), (24, 8192, 16384, 512, False, "stream"),
    (33, 8192, 28672, 128, False, "mid"), (24, 8192, 1024, 128, True, "stream"),
    (20, 8192, 4096, 64, True, "stream"), (32, 8192, 4096, 64, True, "stream"),
    (32, 8192, 28672, 512, True, "stream"), (33, 8192, 4096, 128, True, "mid"),
    # the few-token kernel above 16 tokens
    (17, 2048, 28672, 512, False, "decode"), (32, 4096, 12288, 256, False, "decode"),
    (32, 4096, 8192, 256, False, "mid"), (32, 4096, 12288, 128, False, "mid"),
    (33, 4096, 12288, 256, False, "mid"), (64, 16384, 12288, 256, False, "decode"),
    (32, 16384, 20480, 512, True, "decode"), (48, 16384, 10192, 512, True, "decode"),
    (32, 2048, 20464, 256, False, "decode"), (32, 2048, 20400, 256, False, "mid"),
    (65, 16384, 12288, 256, False, "mid"), (32, 16384, 8208, 256, False, "decode"),
    (32, 16384, 8192, 512, False, "mid"), (64, 16384, 8208, 512, True, "decode"),
    (33, 16384, 10176, 256, False, "mid"), (64, 512, 28672, 64, True, "decode"),
    (33, 512, 8208, 64, False, "decode"), (33, 512, 8192, 64, False, "mid"),
    (32, 512, 28672, 64, True, "mid"),
])
def test_few_tokens(M, K, N, g, tiled, path):
    flags = rrs.WEIGHT_TILED if tiled else 0
    for scratch in (False, True):
        assert rrs.gemm_path(M, N, K, g, flags, scratch=scratch) == path


@pytest.mark.parametrize("M,K,N,g,kind,tiled,path", [
    # the main kernel where the token launch or idle tiles cost more than they save
    (4096, 2048, 1120, 128, None, False, "main"), (8192, 2048, 608, 512, None, True, "main"),
    (5953, 1024, 992, 128, None, True, "main"), (2048, 1024, 4096, 128, "per_channel", False, "main"),
    (2048, 4096, 4096, 128, "per_channel", False, "main"),
    (5346, 2048, 784, 64, "per_channel", False, "main"),
    (8192, 2048, 1024, 512, "reorder", False, "main"),
    (547, 8192, 23696, 256, "reorder", False, "main"), (89, 512, 22016, 512, None, False, "main"),
    (134, 8192, 18400, 128, "reorder", False, "main"),
    (134, 8192, 18400, 128, "reorder", True, "fp6_large"),
    # few columns and short K, where the fits err
    (7932, 2048, 400, 256, None, False, "main"), (7439, 2048, 992, 64, None, False, "main"),
    (6884, 2048, 464, 256, None, True, "main"), (771, 512, 2928, 64, None, False, "main"),
    (258, 512, 7952, 128, None, False, "main"), (1185, 512, 1744, 128, "per_channel", False, "main"),
    # and the others where they are ahead
    (618, 512, 3072, 512, None, True, "mid"), (4000, 8192, 1024, 128, None, False, "fp6_teams"),
    (5000, 4096, 640, 128, None, False, "fp6_teams"), (187, 4096, 17040, 128, "reorder", False, "fp6_large"),
    (173, 4096, 4096, 128, None, False, "mid"), (512, 8192, 8192, 128, None, False, "fp6_teams"),
    (1024, 4096, 12288, 128, "per_channel", False, "fp6_small"),
    (1500, 4096, 12288, 128, "reorder", False, "fp6_tail"),
    (2048, 4096, 12288, 128, None, False, "fp6_large"),
    (1867, 8192, 8512, 64, "reorder", False, "fp6_small"),
])
def test_many_tokens(M, K, N, g, kind, tiled, path):
    flags = rrs.WEIGHT_TILED if tiled else 0
    forms = {kind: True} if kind else {}
    assert rrs.gemm_path(M, N, K, g, flags, **forms) == path
    if path in ("main", "mid"):  # also the calls without scratch
        assert rrs.gemm_path(M, N, K, g, flags, scratch=False, **forms) == path


def test_order_of_the_sum_does_not_depend_on_the_layout():
    # one order each, but those of one entry share theirs
    order = {"main": 0, "fp6_small": 0, "fp6_large": 0, "mid_eighths": "stream"}
    rng = random.Random(3)
    for _ in range(20000):
        M = round(math.exp(rng.uniform(0, 9.1)))
        K, N = 512 << rng.randrange(6), 16 * round(math.exp(rng.uniform(0, 7.5)))
        g = rng.choice([64, 128, 256, 512])
        kw = {"reorder": rng.random() < 0.5, "scratch": rng.random() < 0.7}
        paths = [rrs.gemm_path(M, N, K, g, f, **kw) for f in (0, rrs.WEIGHT_TILED)]
        assert order.get(paths[0], paths[0]) == order.get(paths[1], paths[1]), (M, N, K, g, kw)


def test_other_forms_have_no_wide_few_token_kernel():
    for M, K, N, g in ((24, 8192, 1024, 128), (32, 16384, 12288, 512), (48, 512, 28672, 64)):
        for kind in ("reorder", "per_channel"):
            assert rrs.gemm_path(M, N, K, g, **{kind: True}, scratch=False) in ("mid", "main")


def test_scratch_of_a_call():
    # The shape's bytes where this call takes a kernel on scratch, 0 where it does not.
    rng, seen = random.Random(5), {}
    for _ in range(4000):
        M = round(math.exp(rng.uniform(0, 9.1)))
        K, N = 512 << rng.randrange(6), 16 * round(math.exp(rng.uniform(0, 7.5)))
        g, f = rng.choice([64, 128, 256, 512]), rng.choice([0, rrs.WEIGHT_TILED])
        kind = rng.choice([None, "reorder", "per_channel"])
        path = rrs.gemm_path(M, N, K, g, f, **({kind: True} if kind else {}))
        nbytes = rrs.lib().rrs_gemm_scratch_bytes_ex(M, N, K, g, f, int(kind != "per_channel"),
                                                     int(kind == "reorder"))
        assert nbytes == (rrs.gemm_scratch_bytes(M, N, K) if path.startswith("fp6") else 0)
        seen[path.startswith("fp6")] = seen.get(path.startswith("fp6"), 0) + 1
    assert len(seen) == 2
    assert rrs.lib().rrs_gemm_scratch_bytes_ex(520, 4112, 2048, 0, 0, 0, 0) == 0  # mid-size
    assert rrs.lib().rrs_gemm_scratch_bytes_ex(520, 4112, 2048, 96, 0, 1, 0) == 0  # no such group


@pytest.mark.parametrize("M,K,N,tiled,blocks", [
    # the larger tile from where the smaller one takes more than 256 workgroups
    (22, 16384, 8192, False, 1), (22, 16384, 8208, False, 2), (28, 4096, 9168, False, 2),
    (61, 8192, 4096, False, 1), (61, 8192, 4112, False, 2), (49, 8192, 8192, False, 2),
    (49, 8192, 8208, False, 4), (49, 8192, 8208, True, 4), (16, 4096, 28672, False, 1),
    (64, 4096, 4096, False, 1), (32, 16384, 4096, False, 1), (173, 4096, 4096, False, 4),
    (300, 8192, 1024, False, 2), (32, 4096, 12288, False, 2), (33, 4096, 28672, False, 4),
    # tiled and K up to 1024: from 160 of the larger
    (32, 1024, 8624, True, 1), (32, 1024, 10192, True, 2), (58, 512, 8944, True, 2),
    (32, 2048, 8624, True, 2),
])
def test_mid_size_tile(M, K, N, tiled, blocks):
    assert rrs.lib().rrs_test_gemm_mid_token_blocks(M, N, K, int(tiled)) == blocks


def test_invalid():
    assert rrs.gemm_path(0, 512, 512, 128) == "" == rrs.gemm_path(4, 512, 512, 96)
    assert rrs.gemm_path(4, 24, 512, 128) == "" == rrs.gemm_path(4, 512, 1000, 128)
    assert rrs.gemm_path(4, 512, 512, 0, per_channel=True) == "mid"
    assert rrs.gemm_path(4, 512, 512, 128, reorder=True, per_channel=True) == ""
