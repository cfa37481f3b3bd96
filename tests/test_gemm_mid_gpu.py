"""The GEMM for 17 to a few hundred tokens (small tiles whose waves split K), at
its edges: one, two and four blocks of 16 tokens, ragged rows and columns, K so
short that waves have no tile, every group size, both weight layouts, the
runtime reorder's block table and the per-channel scheme.

The partials hook must equal the integer products bit for bit. Y is compared
with the binary64 sum of the exact partials; the bound is one float16 rounding
(2^-11 of the value, the subnormal step below 2^-14) and the rounding of an
fp32 sum of G terms in any order, (G + 3) 2^-24 sum |s_b P_b| scaled like Y.
"""
import numpy as np
import pytest

from tests._gpu_util import tile_wq, to_gpu, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    rrs.lib()


def _pack(q):
    u = (q & 15).astype(np.uint8)
    return (u[:, 0::2] | (u[:, 1::2] << 4)).astype(np.uint8)


def _case(M, K, N, g, seed):
    rng = np.random.default_rng(seed)
    qx = rng.integers(-8, 8, (M, K)).astype(np.int8)   # -8 too: any nibble is a valid operand
    qw = rng.integers(-8, 8, (N, K)).astype(np.int8)
    a = rng.uniform(0.01, 0.1, M).astype(np.float32)
    s = np.exp(rng.uniform(-3, 3, K // g)).astype(np.float32)
    b = rng.uniform(1e-3, 1e-2, N).astype(np.float32)
    return qx, qw, a, s, b


def _partials(qx, qw, g):
    K = qx.shape[1]
    x = qx.reshape(len(qx), K // g, g).transpose(1, 0, 2).astype(np.float32)
    w = qw.reshape(len(qw), K // g, g).transpose(1, 2, 0).astype(np.float32)
    return np.matmul(x, w).astype(np.int64)  # |P| <= 64 * 512: exact in float32


def _check(y, P, a, s, b, K, label):
    sc = a.astype(np.float64)[:, None] * b.astype(np.float64)[None, :] / K
    ref = np.einsum("b,bmn->mn", s.astype(np.float64), P) * sc
    T = np.einsum("b,bmn->mn", s.astype(np.float64), np.abs(P)) * sc
    bound = np.maximum(np.abs(ref) * 2.0 ** -11, 2.0 ** -25) + (len(s) + 3) * 2.0 ** -24 * T
    err = np.abs(y.astype(np.float64) - ref)
    assert np.all(err <= bound * 1.001), f"{label}: {float((err / bound).max())} of the bound"


CASES = [
    (17, 512, 16, 64, False), (33, 512, 48, 128, True), (64, 1024, 1040, 512, False),
    (31, 2048, 2576, 256, True), (32, 16384, 64, 128, False), (65, 4096, 80, 64, True),
    (130, 1024, 5136, 128, False), (63, 2048, 10256, 64, False), (200, 2048, 2064, 512, True),
    (49, 8192, 176, 256, False),
    # the first columns where the larger tile is taken: 32 and 64 tokens
    (20, 1024, 8208, 64, False), (33, 2048, 8208, 128, True), (61, 4096, 4112, 512, False),
]


@pytest.mark.parametrize("M,K,N,g,tiled", CASES)
def test_mid_gemm(M, K, N, g, tiled):
    import paper_2409_20361_amd as rrs
    print(f"[case] mid GEMM M={M} K={K} N={N} g={g} tiled={tiled}", flush=True)
    fl = rrs.WEIGHT_TILED if tiled else 0
    for form in ({}, {"reorder": True}, {"per_channel": True}):
        assert rrs.gemm_path(M, N, K, g, fl, **form) == "mid"
    qx, qw, a, s, b = _case(M, K, N, g, M + K)
    P = _partials(qx, qw, g)
    X, A, S, B = to_gpu(_pack(qx)), to_gpu(a), to_gpu(s), to_gpu(b)
    rows = _pack(qw)
    assert np.array_equal(to_np(rrs.w4a4_gemm_partials(X, to_gpu(rows), g)), P)
    W = to_gpu(tile_wq(rows) if tiled else rows)
    _check(to_np(rrs.w4a4_gemm(X, A, S, W, B, g, flags=fl)), P, a, s, b, K, "plain")
    # per-channel: one exact sum over K
    y = to_np(rrs.w4a4_gemm_per_channel(X, A, W, B, flags=fl))
    _check(y, P.sum(0, keepdims=True), a, np.ones(1, np.float32), b, K, "per-channel")
    # block table: position block p pairs with natural block order[p]
    order = np.random.default_rng(K).permutation(K // 32).astype(np.int32)
    qr = qw.reshape(N, K // 32, 32)[:, order].reshape(N, K)
    y = to_np(rrs.w4a4_gemm_reorder(X, A, S, W, B, to_gpu(order), g, flags=fl))
    _check(y, _partials(qx, qr, g), a, s, b, K, "reorder")


@pytest.mark.parametrize("M", [1, 16])
def test_per_channel_few_tokens(M):
    import paper_2409_20361_amd as rrs
    K, N = 1024, 144
    print(f"[case] per-channel M={M}", flush=True)
    qx, qw, a, s, b = _case(M, K, N, 128, 5)
    y = to_np(rrs.w4a4_gemm_per_channel(to_gpu(_pack(qx)), to_gpu(a), to_gpu(_pack(qw)),
                                        to_gpu(b)))
    P = _partials(qx, qw, 512).sum(0, keepdims=True)
    _check(y, P, a, np.ones(1, np.float32), b, K, "per-channel")
