"""GPU: sizes at which a kernel changes the way it works (edges of tiles, of register-
resident runs, of the ranges of a launch rule), through the C ABI against the fp64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_progress import say as _say              # noqa: E402
from test_gpu_parity import _select_case          # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [63, 64, 65, 1023, 1025, 16383, 16384, 16385, 17408])
def test_select_around_the_register_resident_size(S):
    """Up to 16384 candidates are read once and kept in registers, 1024 candidates are one per
    thread; whole and partial batches of sixteen groups take different loops."""
    _say(f"select sizes S={S}")
    rng = np.random.default_rng(S)
    a = np.exp(rng.standard_normal((2, S)) * 2).astype(np.float32)
    b = (np.round(rng.random((2, S)) ** 4 * 64) / 64).astype(np.float32)      # ties and exact zeros
    for alpha in (0.3, 0.95, 0.9999):
        _select_case(a, b, alpha, alpha)


def test_sparse_attn_bitmap_in_several_segments():
    """Above 1M tokens a head's bitmaps are built in segments of 2^20 bits and the tile
    diagonals are listed by a launch of their own: strips on both sides of the cut, checked on
    the rows that meet them (bf16 probabilities against their fp64 softmax, as elsewhere)."""
    import paper_2406_15486_amd as sa
    S, w, cut = (1 << 20) + 3000, 64, 1 << 20
    _say(f"bitmap segments S={S}")
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, 1, S, 128, generator=g, device="cuda", dtype=torch.float32).bfloat16() for _ in range(3))
    off_max = (S + 255) // 256 * 256 - 1
    Ic = np.array([0, 31, 32, cut - 1, cut, cut + 1, S - 1])
    Is = np.array([100, off_max - cut - 1, off_max - cut, off_max - cut + 1, cut - 1, cut, S - 1])
    ci, si = (torch.zeros(1, S, dtype=torch.int32, device="cuda") for _ in range(2))
    ci[0, :len(Ic)] = torch.from_numpy(Ic.astype(np.int32))
    si[0, :len(Is)] = torch.from_numpy(Is.astype(np.int32))
    cc, sc = (torch.tensor([len(x)], dtype=torch.int32, device="cuda") for x in (Ic, Is))
    out, lse, _ = sa.sa_sparse_attn(q, k, v, ci, cc, si, sc, w, out_dtype=sa.SA_OUT_F32, want_lse=True)
    torch.cuda.synchronize()
    for i in (0, 63, 64, 2000, off_max - cut, off_max - cut + 500, cut - 1, cut, cut + 1, cut + 999, S - 257, S - 1):
        keys = np.unique(np.concatenate([Ic[Ic <= i], i - Is[Is <= i], np.arange(max(0, i - w + 1), i + 1)]))
        kk, vv = (t[0, 0, torch.from_numpy(keys).cuda()].double().cpu() for t in (k, v))
        s = kk @ q[0, 0, i].double().cpu() / np.sqrt(128.0)
        assert abs(float(torch.logsumexp(s, 0)) - float(lse[0, i])) < 2e-3, i
        assert (torch.softmax(s, 0) @ vv - out[0, 0, i].double().cpu()).abs().max() < 2e-2, i
