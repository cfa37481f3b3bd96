"""The many-token GEMM on scratch memory (6-bit operands) against the entry points
without scratch (int8 operands): the partials of both are exact and each is
added with one FMA in the same order, so Y must be the same bits. (Where two teams
share a tile, or the halves of the last round's tiles, the order differs; the second test holds those to the binary64 sum,
with the bound of the mid-size kernel's test.) Codes are all
sixteen nibbles, at the edges of the tiles: ragged rows (a last block of 32 rows
partly or wholly past M) and columns, both tile shapes, every group size (64 at K =
16384: more groups than one register of scales), both weight layouts, the
runtime reorder's table and the per-channel scheme. -0 and rounding cannot hide
anything: the comparison is on the bits."""
import numpy as np
import pytest

from tests._gpu_util import tile_wq, to_gpu, to_np
from tests.test_gemm_mid_gpu import _case, _check, _pack, _partials

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    rrs.lib()


def _st():
    return torch.cuda.current_stream().cuda_stream


CASES = [  # 128 x 128 tiles, then 256 x 128
    (500, 512, 6208, 128, False), (777, 1024, 4160, 64, True), (500, 16384, 12304, 64, False),
    (500, 1024, 17008, 512, True),
    (1030, 1024, 5200, 128, True), (1057, 512, 5136, 64, False), (1300, 1024, 6160, 256, False),
    (2049, 1024, 4624, 512, False),
]


@pytest.mark.parametrize("M,K,N,g,tiled", CASES)
def test_scratch_gemm_same_bits(M, K, N, g, tiled):
    import paper_2409_20361_amd as rrs
    lib = rrs.lib()
    print(f"[case] scratch GEMM M={M} K={K} N={N} g={g} tiled={tiled}", flush=True)
    need = lib.rrs_gemm_scratch_bytes(M, N, K)
    assert need > 0
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    Xq = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    Wq = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    Xq[M // 2] = 0x88                                   # a row of -8 ...
    Wq[:16] = 0x88                                      # ... against columns of -8
    a = torch.rand(M, device="cuda", generator=gen) * 1e-2
    s = torch.exp(6 * torch.rand(K // g, device="cuda", generator=gen) - 3)
    w = torch.rand(N, device="cuda", generator=gen) * 1e-2
    order = torch.randperm(K // 32, device="cuda", generator=gen).to(torch.int32)
    fl = rrs.WEIGHT_TILED if tiled else 0
    p = [t.data_ptr() for t in (Xq, a, s, Wq, w)]
    for form in ("plain", "reorder", "per_channel"):
        Y = [torch.full((M, N), 7.0, dtype=torch.float16, device="cuda") for _ in range(2)]
        y = Y[0].data_ptr()
        if form == "plain":
            code = lib.rrs_w4a4_gemm_ex(*p, M, N, K, g, fl, y, _st())
            rrs.w4a4_gemm(Xq, a, s, Wq, w, g, out=Y[1], flags=fl)
        elif form == "reorder":
            code = lib.rrs_w4a4_gemm_reorder(*p, order.data_ptr(), M, N, K, g, fl, y, _st())
            rrs.w4a4_gemm_reorder(Xq, a, s, Wq, w, order, g, out=Y[1], flags=fl)
        else:
            code = lib.rrs_w4a4_gemm_per_channel(p[0], p[1], p[3], p[4], M, N, K, fl, y, _st())
            rrs.w4a4_gemm_per_channel(Xq, a, Wq, w, out=Y[1], flags=fl)
        assert code == 0
        torch.cuda.synchronize()
        bits = [t.view(torch.int16) for t in Y]
        assert torch.equal(*bits), f"{form}: {int((bits[0] != bits[1]).sum())} outputs differ"


# Two teams: from 513 tiles of 64 x 64 to 256 of 128 x 128, K from 2048.
TEAMS = [(520, 2048, 4112, 128, False), (577, 2048, 3600, 64, True), (70, 2048, 16400, 512, True),
         (1000, 4096, 2064, 256, False), (1024, 2048, 4096, 128, True)]
# The last tiles of 256 x 128 as halves with two teams: 294 and 266 tiles, 265 with a last
# half past M, 384 (the most halves), 520 (two full rounds).
TEAMS += [(1300, 2048, 6160, 256, False), (500, 2048, 17008, 512, True),
          (1070, 2048, 6736, 128, True), (1024, 2048, 12288, 512, False),
          (1250, 4096, 13312, 512, False)]


@pytest.mark.parametrize("M,K,N,g,tiled", TEAMS)
def test_two_teams(M, K, N, g, tiled):
    import paper_2409_20361_amd as rrs
    print(f"[case] two teams M={M} K={K} N={N} g={g} tiled={tiled}", flush=True)
    assert rrs.lib().rrs_gemm_scratch_bytes(M, N, K) > 0
    qx, qw, a, s, b = _case(M, K, N, g, M + K + N)
    qx[M // 2] = -8
    qw[:16] = -8
    dX, dA, dS, dB = to_gpu(_pack(qx)), to_gpu(a), to_gpu(s), to_gpu(b)
    dW = to_gpu(tile_wq(_pack(qw)) if tiled else _pack(qw))
    fl = rrs.WEIGHT_TILED if tiled else 0
    _check(to_np(rrs.w4a4_gemm(dX, dA, dS, dW, dB, g, flags=fl)), _partials(qx, qw, g), a, s, b, K,
           "plain")
    order = np.random.default_rng(M).permutation(K // 32).astype(np.int32)
    qr = qw.reshape(N, K // 32, 32)[:, order].reshape(N, K)
    _check(to_np(rrs.w4a4_gemm_reorder(dX, dA, dS, dW, dB, to_gpu(order), g, flags=fl)),
           _partials(qx, qr, g), a, s, b, K, "reorder")


def test_scratch_buffer_is_optional():
    import paper_2409_20361_amd as rrs
    lib = rrs.lib()
    M, K, N, g = 500, 512, 6208, 128
    need = lib.rrs_gemm_scratch_bytes(M, N, K)
    X = torch.randn(M, K, device="cuda").half()
    Wq, w = rrs.prepare_weight((0.02 * torch.randn(K, N, device="cuda")).half())
    ws = torch.zeros(rrs.linear_workspace_bytes(M, K, g), dtype=torch.uint8, device="cuda")
    buf = torch.full((need + 64,), 0xA5, dtype=torch.uint8, device="cuda")

    def call(scratch, nbytes):
        Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        code = lib.rrs_linear_scratch(X.data_ptr(), Wq.data_ptr(), w.data_ptr(), M, N, K, g, None,
                                      0, Y.data_ptr(), ws.data_ptr(), ws.numel(), scratch, nbytes,
                                      _st())
        torch.cuda.synchronize()
        return code, Y

    code, ref = call(None, 0)
    assert code == 0
    for nbytes in (need, need - 1):                     # just enough; too small: the plain path
        code, Y = call(buf.data_ptr(), nbytes)
        assert code == 0 and torch.equal(Y, ref)
    assert bool((buf[need:] == 0xA5).all())             # nothing written past it
    assert call(buf.data_ptr() + 8, need)[0] == -4      # not 16-byte aligned
    assert lib.rrs_gemm_scratch_bytes(16, N, K) == 0    # few tokens use none


def test_scratch_of_the_python_calls(monkeypatch):
    # The caller's buffer is the one that is used; without it one of the call's own, or none
    # where the memory is not to be had. One team of waves: Y is the same bits in each case.
    import paper_2409_20361_amd as rrs
    M, K, N, g = 257, 512, 19696, 256
    for form in ({}, {"reorder": True}, {"per_channel": True}):
        assert rrs.gemm_path(M, N, K, g, **form) == "fp6_small"
        assert rrs.gemm_path(M, N, K, g, scratch=False, **form) == "main"
    gen = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((M, K), device="cuda", generator=gen).half()
    Wq, w = rrs.prepare_weight((0.02 * torch.randn((K, N), device="cuda", generator=gen)).half())
    ws = torch.zeros(rrs.linear_reorder_workspace_bytes(M, K, g), dtype=torch.uint8, device="cuda")
    need = rrs.gemm_scratch_bytes(M, N, K)
    Xq, a, s = rrs.rotate_smooth_quant(X, g)
    order = torch.arange(K // 32, dtype=torch.int32, device="cuda").flip(0).contiguous()
    calls = [lambda **k: rrs.linear(X, Wq, w, g, workspace=ws, **k),
             lambda **k: rrs.linear_reorder(X, Wq, w, g, workspace=ws, **k),
             lambda **k: rrs.w4a4_gemm(Xq, a, s, Wq, w, g, **k),
             lambda **k: rrs.w4a4_gemm_reorder(Xq, a, s, Wq, w, order, g, **k),
             lambda **k: rrs.w4a4_gemm_per_channel(Xq, a, Wq, w, **k)]
    empty = torch.empty
    for i, call in enumerate(calls):
        print(f"[case] scratch of call {i}", flush=True)
        Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        ref = call(out=torch.empty_like(Y))
        sizes = []

        def counted(size, **k):
            sizes.append(size)
            return empty(size, **k)

        def refused(size, **k):
            raise torch.OutOfMemoryError("full card")

        buf = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
        with monkeypatch.context() as m:                # given: nothing is allocated
            m.setattr(torch, "empty", counted)
            call(out=Y, scratch=buf)
        torch.cuda.synchronize()
        assert not sizes and torch.equal(Y, ref) and not bool((buf == 0xA5).all())
        small = torch.full((need - 16,), 0xA5, dtype=torch.uint8, device="cuda")
        assert torch.equal(call(out=Y, scratch=small), ref) and bool((small == 0xA5).all())
        with monkeypatch.context() as m:                # a full card: the plain path
            m.setattr(torch, "empty", refused)
            call(out=Y.zero_())
        assert torch.equal(Y, ref)
        with pytest.raises(ValueError):
            call(out=Y, scratch=torch.empty(need, dtype=torch.uint8))


def test_scratch_under_capture(monkeypatch):
    import paper_2409_20361_amd as rrs
    from paper_2409_20361_amd import _binding
    M, K, N, g = 257, 512, 19696, 256
    dev = torch.device("cuda", torch.cuda.current_device())
    need = rrs.gemm_scratch_bytes(M, N, K)
    got = lambda: _binding._gemm_scratch(None, M, N, K, g, 0, dev)  # noqa: E731
    assert got()[2] == need
    with monkeypatch.context() as m:    # capturing, but the allocator has no pool for it
        m.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
        assert got() == (None, None, 0)
    x = torch.zeros(8, device=dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):       # torch's own capture
        x.add_(1)
        assert got()[2] == need
