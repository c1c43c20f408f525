"""GPU tests of the contrastive losses' arithmetic beyond the parity bars: the
order of a logit's sum, and what a NaN input does."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00690_amd import vl
    vl.lib()
    return vl


@pytest.mark.parametrize("n", [1, 33, 512, 513, 600])
@pytest.mark.parametrize("big,one,minus", [(0, 1, 2), (0, 4, 32), (3, 17, 63)])
def test_logit_is_one_ascending_chain_at_every_batch_size(V, n, big, one, minus):
    """Every logit is one chain of fused multiply-adds over ascending k,
    whatever the number of pairs, so a pair's logit has the same bits in every
    batch (a training step amplifies a last-bit change of dL/d(embedding) to
    some 1e-4 of its BF16 weight gradients).  2^24 + 1 - 2^24 is 0 in that
    order and 1 where the three terms fall into separate sums: with all logits
    0 the sigmoid loss is n ln 2 and dL/dbias n / 2 - 1 (terms of one size, so
    FP32 sums of n^2 of them are well within 1e-4)."""
    e = torch.zeros(n, 64)
    e[:, big], e[:, one], e[:, minus] = 2.0 ** 24, 1.0, -(2.0 ** 24)
    loss, _, _, dsb = V.vl_contrastive_loss(e.cuda(), torch.ones(n, 64).cuda(), "sigmoid", 1.0,
                                            0.0)
    assert float(loss.cpu()[0]) == pytest.approx(n * math.log(2.0), rel=1e-4)
    assert float(dsb.cpu()[1]) == pytest.approx(0.5 * n - 1.0, abs=1e-4 * n)


@pytest.mark.parametrize("n,row", [(1, 0), (64, 63), (65, 64), (65, 3), (130, 129), (1025, 1024)])
@pytest.mark.parametrize("where", ["emb", "texts"])
def test_softmax_nan_reaches_every_gradient(V, n, row, where):
    """A NaN embedding or text is in every log-sum-exp of the other side (and
    makes its own NaN), so the softmax loss and all gradients are NaN; also
    where its logits are the only ones of their 64 x 64 tile's rows (the last
    text of 65)."""
    g = torch.Generator().manual_seed(7 * n + row)
    e, t = (torch.nn.functional.normalize(torch.randn(n, 32, generator=g), dim=1)
            for _ in range(2))
    (e if where == "emb" else t)[row, 5] = float("nan")
    loss, de, dt, dsb = V.vl_contrastive_loss(e.cuda(), t.cuda(), "softmax", 10.0, 0.0)
    for x in (loss, de, dt, dsb[:1]):
        assert bool(torch.isnan(x).all())


@pytest.mark.parametrize("n", [65, 130])
def test_sigmoid_nan_stays_in_its_column(V, n):
    """Sigmoid head: a NaN text makes the loss, every dL/d(embedding) and its
    own gradient NaN; the other texts' gradients do not depend on it."""
    g = torch.Generator().manual_seed(n)
    e, t = (torch.nn.functional.normalize(torch.randn(n, 32, generator=g), dim=1)
            for _ in range(2))
    ref = V.vl_contrastive_loss(e.cuda(), t.cuda(), "sigmoid", 10.0, -10.0)[2].cpu().numpy()
    t[n - 1] = float("nan")
    loss, de, dt, _ = V.vl_contrastive_loss(e.cuda(), t.cuda(), "sigmoid", 10.0, -10.0)
    assert bool(torch.isnan(loss).all()) and bool(torch.isnan(de).all())
    assert bool(torch.isnan(dt[n - 1]).all())
    assert np.array_equal(dt[:n - 1].cpu().numpy(), ref[:n - 1])
