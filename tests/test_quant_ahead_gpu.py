"""The layer calls of up to 16 tokens, whose quantizer launch also reads the first weights of
the GEMM behind it: fewer column blocks than reading workgroups, one more than those, more than
are read ahead (512 blocks at K = 4096), the largest K, Ks below the rule. The outputs are the
bits of the separate quantizer and GEMM calls (which read nothing ahead), also over consecutive
calls on one workspace, and the rows' exchange reports no failed wait."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("reorder", [False, True])
@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("M,K,N,g", [(3, 4096, 16, 64), (16, 4096, 16 * 161, 128),
                                     (5, 4096, 16 * 600, 512), (16, 2048, 16 * 77, 128),
                                     (8, 8192, 16 * 9, 128), (16, 16384, 16 * 170, 64),
                                     (2, 16384, 48, 512), (4, 1024, 16 * 33, 128)])
def test_layer_reading_ahead(M, K, N, g, tiled, reorder):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    gen = torch.Generator(device="cuda").manual_seed(M * K + N)
    X = torch.randn((M, K), generator=gen, device="cuda").half()
    X[:, ::97] *= 40
    W = (0.02 * torch.randn((K, N), generator=gen, device="cuda")).half()
    flags = rrs.WEIGHT_TILED if tiled else 0
    Wq, w = rrs.prepare_weight(W, None, flags=flags)
    if reorder:
        nbytes = rrs.linear_reorder_workspace_bytes(M, K, g)
        Xq, a, s, order = rrs.rotate_smooth_quant_reorder(X, g)
        want = rrs.w4a4_gemm_reorder(Xq, a, s, Wq, w, order, g, flags=flags)
        layer = rrs.linear_reorder
    else:
        nbytes = rrs.linear_workspace_bytes(M, K, g)
        Xq, a, s = rrs.rotate_smooth_quant(X, g)
        want = rrs.w4a4_gemm(Xq, a, s, Wq, w, g, flags=flags)
        layer = rrs.linear
    ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    for _ in range(3):
        assert torch.equal(layer(X, Wq, w, g, workspace=ws, flags=flags), want)
    assert ws[4:8].view(torch.int32).item() == 0
