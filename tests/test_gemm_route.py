"""Which kernel a GEMM call takes, a host query: the calls below were measured on both
kernels, and the one named is the faster (the times are beside the rule)."""
import pytest

import paper_2409_20361_amd as rrs


@pytest.mark.parametrize("M,K,N,g,tiled,path", [
    # the eight-wave weight stream at K = 8192, 17 to 32 tokens
    (16, 8192, 28672, 128, False, "stream"), (17, 8192, 28672, 128, False, "stream"),
    (32, 8192, 256, 64, False, "stream"), (24, 8192, 16384, 512, False, "stream"),
    (33, 8192, 28672, 128, False, "mid"), (24, 8192, 1024, 128, True, "stream"),
    (20, 8192, 4096, 64, True, "stream"), (32, 8192, 4096, 64, True, "mid"),
    (32, 8192, 28672, 512, True, "stream"), (32, 8192, 28672, 128, True, "mid"),
    # the few-token kernel above 16 tokens
    (17, 2048, 28672, 512, False, "decode"), (32, 4096, 12288, 256, False, "decode"),
    (32, 4096, 8192, 256, False, "mid"), (32, 4096, 12288, 128, False, "mid"),
    (33, 4096, 12288, 256, False, "mid"), (64, 16384, 12288, 256, False, "decode"),
    (32, 16384, 20480, 512, True, "decode"), (48, 16384, 20480, 512, True, "mid"),
    (65, 16384, 12288, 256, False, "mid"), (64, 512, 28672, 64, True, "decode"),
    (32, 512, 28672, 64, True, "mid"),
])
def test_few_tokens(M, K, N, g, tiled, path):
    flags = rrs.WEIGHT_TILED if tiled else 0
    for scratch in (False, True):
        assert rrs.gemm_path(M, N, K, g, flags, scratch=scratch) == path


def test_other_forms_have_no_wide_few_token_kernel():
    for M, K, N, g in ((24, 8192, 1024, 128), (32, 16384, 12288, 512), (48, 512, 28672, 64)):
        for kind in ("reorder", "per_channel"):
            assert rrs.gemm_path(M, N, K, g, **{kind: True}, scratch=False) in ("mid", "main")


def test_invalid():
    assert rrs.gemm_path(0, 512, 512, 128) == "" == rrs.gemm_path(4, 512, 512, 96)
    assert rrs.gemm_path(4, 24, 512, 128) == "" == rrs.gemm_path(4, 512, 1000, 128)
    assert rrs.gemm_path(4, 512, 512, 0, per_channel=True) == "mid"
    assert rrs.gemm_path(4, 512, 512, 128, reorder=True, per_channel=True) == ""
