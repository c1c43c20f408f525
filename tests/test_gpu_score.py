"""GPU tests of the score GEMM's tile rule: a few images against many texts."""
import numpy as np
import pytest

from oracle import vit64 as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00690_amd import vl
    vl.lib()
    return vl


@pytest.mark.parametrize("rows", [1, 7, 16, 17])
@pytest.mark.parametrize("texts", [4096, 4100, 4116, 8196])
@pytest.mark.parametrize("dim", [16, 256, 272, 784])
def test_few_images_many_texts(V, rows, texts, dim):
    """Up to 16 images against more than 4096 texts run in 16 x 16 tiles, two
    workgroups to a CU; 17 images in 32 x 32 tiles, 4096 texts in one round.
    Each form against FP64 and, row by row, bitwise against the others: the
    sigmoid's derivative is at most 1/4, so a logit of |scale| times dim
    products, each rounded once, plus the exponential's own error bound the
    difference."""
    rng = np.random.Generator(np.random.PCG64(1000 * rows + texts + dim))
    e, t = rng.standard_normal((17, dim)), rng.standard_normal((texts, dim))
    e, t = (x / np.linalg.norm(x, axis=1, keepdims=True) for x in (e, t))
    e, t = e.astype(np.float32), t.astype(np.float32)
    ed, td = torch.from_numpy(e).cuda(), torch.from_numpy(t).cuda()

    def score(a, b):
        sc = torch.empty(a.shape[0], b.shape[0], device="cuda")
        top = torch.empty(a.shape[0], dtype=torch.int32, device="cuda")
        V.vl_score(a, b, "sigmoid", 10.0, -1.0, sc, top)
        torch.cuda.synchronize()
        return sc, top

    got, top = score(ed[:rows].contiguous(), td)
    ref, _ = O.score(e[:rows], t, "sigmoid", 10.0, -1.0)
    bar = (0.25 * 11 * (dim + 8) + 16) * 2.0 ** -24
    assert np.abs(got.cpu().numpy() - ref).max() <= bar
    full, _ = score(ed, td)
    assert torch.equal(got, full[:rows])
    part, _ = score(ed[:rows].contiguous(), td[-40:].contiguous())
    assert torch.equal(part, got[:, -40:])
    assert torch.equal(top.cpu(), got.argmax(1).to(torch.int32).cpu())
