"""The few-token kernels above 16 tokens, where the route takes them: the eight-wave weight
stream (K = 8192, 17 to 32 tokens) and the few-token kernel with two and four blocks of
tokens, at the first and last token count and the narrowest N of each, with ragged last
column blocks. Partials bit for bit, Y within the mid-size kernel's bound."""
import numpy as np
import pytest

from tests._gpu_util import tile_wq, to_gpu, to_np
from tests.test_gemm_mid_gpu import _case, _check, _pack, _partials

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M,K,N,g,tiled,path", [
    (17, 8192, 16, 64, False, "stream"), (32, 8192, 4112, 128, False, "stream"),
    (25, 8192, 272, 256, False, "stream"), (32, 8192, 48, 512, True, "stream"),
    (20, 8192, 80, 64, True, "stream"), (19, 8192, 10256, 512, True, "stream"),
    (17, 2048, 20432, 256, False, "decode"), (32, 4096, 10192, 512, False, "decode"),
    (33, 16384, 10192, 256, False, "decode"), (64, 16384, 10224, 512, False, "decode"),
    (20, 16384, 10208, 512, True, "decode"), (64, 16384, 10192, 256, True, "decode"),
    (32, 4096, 10256, 256, True, "decode"), (33, 512, 10192, 64, True, "decode"),
    (64, 512, 10208, 64, False, "decode"),
])
def test_wide(M, K, N, g, tiled, path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    print(f"[case] wide M={M} K={K} N={N} g={g} tiled={tiled}", flush=True)
    fl = rrs.WEIGHT_TILED if tiled else 0
    assert rrs.gemm_path(M, N, K, g, fl) == path
    qx, qw, a, s, b = _case(M, K, N, g, M + K + N)
    qx[M // 2] = -8
    qw[:16] = -8
    P = _partials(qx, qw, g)
    X, rows = to_gpu(_pack(qx)), _pack(qw)
    if not tiled:
        assert np.array_equal(to_np(rrs.w4a4_gemm_partials(X, to_gpu(rows), g)), P)
    Y = rrs.w4a4_gemm(X, to_gpu(a), to_gpu(s), to_gpu(tile_wq(rows) if tiled else rows),
                      to_gpu(b), g, flags=fl)
    _check(to_np(Y), P, a, s, b, K, path)


@pytest.mark.parametrize("M,N,g", [(17, 6144, 64), (32, 6160, 128), (25, 10224, 256),
                                   (32, 10256, 64), (17, 12304, 128), (32, 28672, 256)])
def test_eighths_of_k_are_the_streams_bits(M, N, g):
    # With the tiled layout the mid-size kernel, in the order of the weight stream.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    K = 8192
    print(f"[case] eighths M={M} N={N} g={g}", flush=True)
    assert rrs.gemm_path(M, N, K, g) == "stream"
    assert rrs.gemm_path(M, N, K, g, rrs.WEIGHT_TILED) == "mid_eighths"
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=gen, device="cuda").half()
    X[:, ::97] *= 40
    W = (0.02 * torch.randn((K, N), generator=gen, device="cuda")).half()
    Xq, a, s = rrs.rotate_smooth_quant(X, g)
    Y = [rrs.w4a4_gemm(Xq, a, s, *rrs.prepare_weight(W, None, f), g, flags=f)
         for f in (0, rrs.WEIGHT_TILED)]
    assert torch.equal(*Y)


@pytest.mark.parametrize("M,K,N,paths", [
    (663, 1024, 4336, ("main", "mid")), (757, 2048, 5264, ("fp6_teams", "main")),
    (788, 1024, 12912, ("fp6_small", "main"))])
def test_per_channel_bits_on_any_kernel(M, K, N, paths):
    # One exact sum and one rounding: the kernel, which here depends on the layout, does not.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    print(f"[case] per-channel bits M={M} K={K} N={N}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M)
    Xq = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    a = torch.rand(M, device="cuda", generator=gen) * 1e-2
    W = (0.02 * torch.randn((K, N), generator=gen, device="cuda")).half()
    Y = []
    for flags, path in zip((0, rrs.WEIGHT_TILED), paths):
        assert rrs.gemm_path(M, N, K, 128, flags, per_channel=True) == path
        Y.append(rrs.w4a4_gemm_per_channel(Xq, a, *rrs.prepare_weight(W, None, flags), flags=flags))
    assert torch.equal(*Y)
