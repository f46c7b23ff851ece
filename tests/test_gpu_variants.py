"""Kernel variants chosen by size, at the sizes where they can go wrong.

Every case is checked bit for bit against the CPU FP64 oracle, so no
tolerance is involved.
"""
import numpy as np
import pytest

import oracle as orc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _rm():
    import paper_2504_13445_amd as rm
    return rm


def _g(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(_dev())


def _say(*a):
    print("[case]", *a, flush=True)


# FP32 screening: FP32 steps below 32 dimensions, split FP16 rows from there
# on (a row is padded to 16 values, a half row is 1 to 16 chunk pairs); rows
# whose values span 12 decades lose the small ones' low parts to the bound
@pytest.mark.parametrize("d", [31, 32, 33, 48, 49, 100, 127, 128, 129, 200, 224, 225, 255, 256])
@pytest.mark.parametrize("wide", [False, True])
def test_split_rows(d, wide):
    _say("split rows", d, wide)
    rng = np.random.default_rng(d)
    n, m, k = 259, 193, 9
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.6)
    if wide:
        U = (U * 10.0 ** rng.uniform(-9, 3, (n, d))).astype(np.float32)
        P = (P * 10.0 ** rng.uniform(-9, 3, (m, d))).astype(np.float32)
    rm = _rm()
    t, j, tk = orc.kmips_c(U, P, k)
    tau, tid, topk = rm.thresholds(_g(U), _g(P), k, with_topk=True)
    assert np.array_equal(tau.cpu().numpy().view(np.uint64), t.view(np.uint64))
    assert np.array_equal(tid.cpu().numpy(), j) and np.array_equal(topk.cpu().numpy(), tk)
    sc = orc.histogram_scores(tk, m)
    got = rm.scores(_g(U), tau, tid, _g(P), torch.arange(m, dtype=torch.int32, device=_dev()))
    assert np.array_equal(got.cpu().numpy(), sc)
    ids, s, _ = rm.topn(_g(U), _g(P), k, 20)
    ri, rs = orc.topn_from_scores(sc, 20)
    assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()
