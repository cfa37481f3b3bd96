"""The many-token GEMM on scratch memory (6-bit operands). Its forms with one team of waves
against the entry points without scratch, which take the int8 main kernel: the partials of
both are exact and each is added with one FMA in the same order, so Y must be the same bits.
Where two teams share a tile, or the halves of the last round's tiles, the order differs:
those are held to the binary64 sum of the exact partials, with the bound of the mid-size
kernel's test (the per-channel scheme's sum is exact: the same bits there too). Every case
names the kernel that each of its forms takes. Codes are all sixteen nibbles, at the edges of
the tiles: ragged rows (a last block of 32 rows partly or wholly past M) and columns, both
tile shapes, every group size (64 at K = 16384: more groups than one register of scales),
both weight layouts, the runtime reorder's table and the per-channel scheme. -0 and rounding
cannot hide anything: the comparison is on the bits."""
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


def _st():
    return torch.cuda.current_stream().cuda_stream


FORMS = ("plain", "reorder", "per_channel")
SMALL, LARGE, TEAMS, TAIL, MAIN, MID = ("fp6_small", "fp6_large", "fp6_teams", "fp6_tail", "main",
                                        "mid")


def _path(M, K, N, g, tiled, form, scratch=True):
    import paper_2409_20361_amd as rrs
    return rrs.gemm_path(M, N, K, g, rrs.WEIGHT_TILED if tiled else 0, scratch=scratch,
                         **({} if form == "plain" else {form: True}))


# The kernel of each form, in the order of FORMS.
CASES = [
    # 128 x 128 tiles: a last tile of one row, of three blocks of 32, ...
    (257, 512, 19696, 256, False, (SMALL, SMALL, SMALL)),
    (300, 512, 19696, 512, True, (SMALL, SMALL, SMALL)),
    (345, 512, 19696, 128, True, (SMALL, SMALL, SMALL)),
    (385, 512, 19712, 128, False, (SMALL, MAIN, MAIN)),
    (777, 1024, 4160, 64, True, (SMALL, SMALL, MAIN)),
    (1300, 1024, 6160, 256, False, (SMALL, MAIN, MAIN)),
    # 256 x 128
    (500, 16384, 12304, 64, False, (LARGE, LARGE, LARGE)),
    (257, 1024, 11184, 64, True, (LARGE, LARGE, MAIN)),
    (257, 2048, 11184, 128, True, (LARGE, LARGE, MAIN)),
    (513, 512, 26384, 128, False, (LARGE, LARGE, MAIN)),
    (1030, 2048, 16400, 256, True, (LARGE, LARGE, MAIN)),
    (1500, 512, 27296, 256, False, (LARGE, LARGE, LARGE)),
    (1281, 512, 23952, 512, False, (LARGE, MAIN, LARGE)),
    (1500, 512, 27296, 512, True, (LARGE, LARGE, LARGE)),
]


@pytest.mark.parametrize("M,K,N,g,tiled,paths", CASES)
def test_scratch_gemm_same_bits(M, K, N, g, tiled, paths):
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
    for form, path in zip(FORMS, paths):
        assert _path(M, K, N, g, tiled, form) == path
        assert _path(M, K, N, g, tiled, form, scratch=False) == MAIN
        if path == MAIN:
            continue
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


# Two teams, then the last tiles of 256 x 128 as halves with two teams.
TEAM_CASES = [
    (520, 2048, 4112, 128, False, (TEAMS, TEAMS, MID)),
    (577, 2048, 3600, 64, True, (TEAMS, TEAMS, MID)),
    (70, 2048, 16400, 512, True, (TEAMS, TEAMS, MID)),
    (1000, 4096, 2064, 256, False, (TEAMS, TEAMS, MID)),
    (1024, 2048, 4096, 128, True, (TEAMS, TEAMS, MAIN)),
    (577, 16384, 3600, 64, False, (TEAMS, TEAMS, MID)),   # 128 groups a team
    (257, 2048, 9968, 128, False, (TEAMS, TEAMS, TEAMS)),
    (257, 2048, 9968, 256, True, (TEAMS, TEAMS, TEAMS)),
    (777, 16384, 4096, 256, True, (TEAMS, TEAMS, TEAMS)),
    # 342 tiles: 11 of an XCD's 43 in halves, every second of them past M but for one row
    (257, 2048, 21824, 64, False, (TAIL, TAIL, TAIL)),
    (257, 2048, 21824, 128, True, (TAIL, TAIL, TAIL)),
    (257, 2048, 21824, 64, True, (TAIL, TAIL, TAIL)),
    (257, 2048, 21824, 128, False, (TAIL, TAIL, TAIL)),
    # the most halves, 16 of an XCD's 80
    (513, 2048, 27136, 128, False, (TAIL, TAIL, TAIL)),
    (769, 2048, 20480, 64, True, (TAIL, TAIL, TAIL)),
    (1300, 2048, 6160, 256, False, (TAIL, TAIL, TAIL)),
    (500, 2048, 17008, 512, True, (TAIL, TAIL, TAIL)),
    (1500, 4096, 12288, 128, False, (TAIL, TAIL, TAIL)),
    (1250, 4096, 13312, 512, False, (TAIL, TAIL, TAIL)),  # two full rounds
]


def _unpack(p):
    """Packed codes (rows x K/2, uint8, on the GPU) -> float64 codes."""
    lo = ((p & 15).to(torch.int8) ^ 8) - 8
    hi = ((p >> 4).to(torch.int8) ^ 8) - 8
    return torch.stack((lo, hi), -1).flatten(1).double()


def _check_sum(Y, qx, qw, a, s, w, K, g, label):
    """Y against the binary64 sum; the bound of _check in test_gemm_mid_gpu."""
    ref = torch.zeros(Y.shape, dtype=torch.float64, device="cuda")
    T = torch.zeros_like(ref)
    for b in range(K // g):
        P = s[b].double() * (qx[:, b * g:(b + 1) * g] @ qw[:, b * g:(b + 1) * g].t().contiguous())
        ref += P
        T += P.abs()
    sc = a.double()[:, None] * w.double()[None, :] / K
    ref, T = ref * sc, T * sc
    bound = (ref.abs() * 2.0 ** -11).clamp(min=2.0 ** -25) + (K // g + 3) * 2.0 ** -24 * T
    worst = ((Y.double() - ref).abs() / bound).max().item()
    assert worst <= 1.001, f"{label}: {worst} of the bound"


@pytest.mark.parametrize("M,K,N,g,tiled,paths", TEAM_CASES)
def test_two_teams(M, K, N, g, tiled, paths):
    import paper_2409_20361_amd as rrs
    print(f"[case] two teams M={M} K={K} N={N} g={g} tiled={tiled}", flush=True)
    for form, path in zip(FORMS, paths):
        assert _path(M, K, N, g, tiled, form) == path
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    Xq = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    rows = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    Xq[M // 2] = 0x88                                   # a row of -8 ...
    rows[:16] = 0x88                                    # ... against columns of -8
    a = 0.01 + 0.09 * torch.rand(M, device="cuda", generator=gen)
    s = torch.exp(6 * torch.rand(K // g, device="cuda", generator=gen) - 3)
    w = 1e-3 + 9e-3 * torch.rand(N, device="cuda", generator=gen)
    order = torch.randperm(K // 32, device="cuda", generator=gen).to(torch.int32)
    fl = rrs.WEIGHT_TILED if tiled else 0
    Wq = to_gpu(tile_wq(to_np(rows))) if tiled else rows
    qx, qw = _unpack(Xq), _unpack(rows)
    _check_sum(rrs.w4a4_gemm(Xq, a, s, Wq, w, g, flags=fl), qx, qw, a, s, w, K, g, "plain")
    qr = qw.view(N, K // 32, 32)[:, order.long()].reshape(N, K)
    _check_sum(rrs.w4a4_gemm_reorder(Xq, a, s, Wq, w, order, g, flags=fl), qx, qr, a, s, w, K, g,
               "reorder")
    Y = rrs.w4a4_gemm_per_channel(Xq, a, Wq, w, flags=fl)
    _check_sum(Y, qx, qw, a, torch.ones(1, device="cuda"), w, K, K, "per-channel")
    plain = torch.empty_like(Y)
    code = rrs.lib().rrs_w4a4_gemm_per_channel(Xq.data_ptr(), a.data_ptr(), Wq.data_ptr(),
                                               w.data_ptr(), M, N, K, fl, plain.data_ptr(), _st())
    assert code == 0 and torch.equal(Y, plain)


def test_scratch_buffer_is_optional():
    import paper_2409_20361_amd as rrs
    lib = rrs.lib()
    M, K, N, g = 300, 512, 19696, 512
    assert _path(M, K, N, g, False, "plain") == SMALL
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
    for form in FORMS:
        assert _path(M, K, N, g, False, form) == SMALL
        assert _path(M, K, N, g, False, form, scratch=False) == MAIN
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
