"""GPU tests of the K/V-resident attention kernel against the streaming one,
bitwise, in every place that launches it: forced by VL_OPT_ATTN_RESIDENT 1 over
ragged batches and capacity-bucketed graphs, and by the default rule (equal
images of 7 .. 10 key tiles, 224 .. 256 (image, head) pairs)."""
import pytest

import synth
from helpers import pack

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00690_amd import vl
    vl.lib()
    return vl


B16_2 = synth.ModelConfig("b16_2block", patch=16, width=768, layers=2, heads=12, mlp=3072,
                          proj_dim=512, base_grid=14)
L14_1 = synth.ModelConfig("l14_1block", patch=14, width=1024, layers=1, heads=16, mlp=4096,
                          proj_dim=768, base_grid=24)


def _blob(c, seed=90):
    return torch.from_numpy(synth.params_to_blob(c, synth.make_params(c, seed, std=0.02))).cuda()


def _pixels(sizes, seed=91):
    return torch.from_numpy(pack(synth.make_images(sizes, seed))).cuda()


def _option(V, m, value):
    V.vl_model_set_option(m.handle, V.VL_OPT_ATTN_RESIDENT, value)


# Largest resident image of 4, 6, 8 (442 tokens: 7) and 10 key tiles: each
# instance of the kernel, with shorter resident ones, a streamed one of 65
# tokens and (but for the first) one of 785.
RAGGED = {4: [(224, 224), (192, 192), (176, 208)], 6: [(288, 288), (224, 224)],
          8: [(336, 336), (224, 224), (336, 320)], 10: [(400, 400), (336, 336), (384, 400)]}


@pytest.mark.parametrize("precision", ["bf16", "fp8w", "mxfp8"])
@pytest.mark.parametrize("tiles", [4, 6, 8, 10])
def test_forced_resident_batches_bitwise(V, precision, tiles):
    """Option 1 takes every image of 129 .. 640 tokens, in a ragged batch too:
    the plan lists them instead of their query blocks (less workspace), and
    the embeddings are those of the streamed batch (0) and of the default (2),
    which streams unequal images."""
    sizes = RAGGED[tiles] * 14 + [(128, 128)] + ([(448, 448)] if tiles > 4 else [])
    pix = _pixels(sizes)
    enc = V.Encoder(B16_2, _blob(B16_2), precision)
    out, need = {}, {}
    for value in (2, 0, 1, 2):
        _option(V, enc, value)
        e, w = enc.encode(pix, sizes).clone(), enc.workspace_bytes(sizes)
        torch.cuda.synchronize()
        assert value not in out or (torch.equal(out[value], e) and need[value] == w)
        out[value], need[value] = e, w
    enc.close()
    assert need[2] == need[0] > need[1]
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


def test_forced_resident_bucketed_graph_bitwise(V):
    """Option 1 with a capacity-bucketed graph: the resident launch is sized for
    the bucket and reads its image count on the device.  Batches with four,
    three and no resident images replay one graph."""
    blob = _blob(B16_2)
    eager = V.Encoder(B16_2, blob, "bf16")
    genc = V.Encoder(B16_2, blob, "bf16", graphs=True)
    _option(V, eager, 0)
    _option(V, genc, 1)
    # 541, 529 and 579 tokens (capacity 640); 4, 4 and 3 images, at most 128
    # tokens each in some of them
    batches = [[(224, 224), (160, 160), (256, 192), (112, 112)],
               [(224, 208), (208, 208), (176, 160), (128, 128)],
               [(224, 224), (224, 224), (208, 224)],
               [(176, 176)] * 4]
    for k, sizes in enumerate([batches[0], batches[1], batches[0], batches[2], batches[3],
                               batches[1]]):
        pix = _pixels(sizes, 100 + k)
        ref = eager.encode(pix, sizes).clone()
        got = genc.encode(pix, sizes).clone()
        torch.cuda.synchronize()
        assert torch.equal(got, ref), k
    eager.close()
    genc.close()


@pytest.mark.parametrize("precision", ["bf16", "mxfp8"])
@pytest.mark.parametrize("n", [13, 14, 16, 17])
def test_default_rule_l14_336_bitwise(V, precision, n):
    """Around the default rule at 16 heads: 14 .. 16 images of 577 tokens (ten
    key tiles) run resident, 13 and 17 stream."""
    sizes = [(336, 336)] * n
    pix = _pixels(sizes)
    enc = V.Encoder(L14_1, _blob(L14_1), precision, split=False)
    a, wa = enc.encode(pix, sizes).clone(), enc.workspace_bytes(sizes)
    _option(V, enc, 0)
    b, wb = enc.encode(pix, sizes).clone(), enc.workspace_bytes(sizes)
    torch.cuda.synchronize()
    enc.close()
    assert torch.equal(a, b)
    assert (wa < wb) == (14 <= n <= 16)


@pytest.mark.parametrize("n,split", [(14, False), (16, False), (28, True), (32, True)])
def test_training_on_resident_attention_bitwise(V, n, split):
    """The training forward's resident attention keeps the log-sum-exp that
    the backward reads: 14 and 16 images of 577 tokens in one pass, and 28 and
    32 in two halves, fall under the default rule; embeddings and every
    gradient are those of the streamed run."""
    sizes = [(336, 336)] * n
    pix = _pixels(sizes)
    de = torch.from_numpy(synth.make_texts(n, L14_1.proj_dim, 92)).cuda() * 0.1
    out = []
    for value in (2, 0):
        tr = V.Trainer(L14_1, _blob(L14_1), "bf16", split=split)
        _option(V, tr, value)
        need = tr.train_workspace_bytes(sizes)
        emb = tr.forward(pix, sizes).clone()
        grads = tr.backward(pix, sizes, de).clone()
        torch.cuda.synchronize()
        tr.close()
        out.append((emb, grads, need))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][2] < out[1][2]          # the resident form was planned


@pytest.mark.parametrize("n,split", [(5, False), (24, True)])
def test_training_forced_resident_bitwise(V, n, split):
    """Option 1 in training, where the default streams: images of 197 tokens
    (four key tiles), one pass and two halves."""
    sizes = [(224, 224)] * n
    pix = _pixels(sizes)
    de = torch.from_numpy(synth.make_texts(n, B16_2.proj_dim, 93)).cuda() * 0.1
    out = []
    for value in (1, 0):
        tr = V.Trainer(B16_2, _blob(B16_2), "bf16", split=split)
        _option(V, tr, value)
        emb = tr.forward(pix, sizes).clone()
        grads = tr.backward(pix, sizes, de).clone()
        torch.cuda.synchronize()
        tr.close()
        out.append((emb, grads))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
