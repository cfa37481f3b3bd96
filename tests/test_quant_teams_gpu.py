"""The two-pass quantizer from K = 8192 (one, two or four row teams per workgroup,
512 threads per row at K = 16384) against the oracle bit for bit, at the row counts
where the number of teams changes (256 and 512 rows) and with ragged last
workgroups, with and without the static reorder and each ablation."""
import numpy as np
import pytest

import synth
from oracle import rrs_oracle as O
from tests._gpu_util import check_codes, to_gpu, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_20361_amd as rrs
    rrs.lib()


@pytest.mark.parametrize("M,K,g,perm,flags", [
    (70, 8192, 128, True, 0), (513, 8192, 256, False, 0), (515, 8192, 64, True, 0),
    (300, 8192, 512, False, 1), (520, 8192, 128, False, 2),
    (3, 16384, 128, True, 0), (255, 16384, 64, False, 0), (257, 16384, 256, True, 0),
    (261, 16384, 512, False, 1), (5, 16384, 128, False, 2), (517, 16384, 256, False, 0),
])
def test_row_teams(M, K, g, perm, flags):
    import paper_2409_20361_amd as rrs
    print(f"[case] quant teams M={M} K={K} g={g} perm={perm} flags={flags}", flush=True)
    w = synth.custom("qt", M, K, 16, g, M + K, n_chan=K // 100, chan_factor=(20, 100),
                     n_spike=max(1, M * K // 10000), spike_mag=(100, 500))
    X = synth.activations(w)
    p = synth.permutation(K, M) if perm else None
    Xq, a, s = rrs.rotate_smooth_quant(to_gpu(X), g, to_gpu(p) if perm else None, flags=flags)
    act = O.rotate_smooth_quant(X, g, perm=p, rotate=not flags & rrs.SKIP_ROTATION,
                                smooth=not flags & rrs.SKIP_SMOOTHING)
    check_codes(to_np(Xq), act, "quant teams")
    assert np.array_equal(to_np(a), act.alpha)
    assert np.array_equal(to_np(s), act.s)
