"""The separate calls (quantiser over all rows, sum with the reconstruction, and
with several scales the index pass) at model sizes, every code width, one scale
and several, with codes left to the cache and stored nontemporally (more than
512 MB), and past 2^31 coordinates: every code, sum and output equals the
one-call step's, whose results other tests compare with the oracle."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import synth  # noqa: E402
from paper_2109_12497_amd.step import Step  # noqa: E402

DEV = torch.device("cuda:0")
RESNET50, VGG16 = 25_557_032, 138_357_544
TOP = {8: 127.0, 4: 7.0, 2: 1.0}


def gradients(d, M, seed):
    g = torch.empty((M, synth.round_up(d, 64)), dtype=torch.float32, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    for m in range(M):
        for n, c in enumerate(range(0, d, 1 << 26)):
            g[m, c:c + (1 << 26)].normal_(0.0, 10.0 ** -(2 + n % 4), generator=gen)
    g[:, 5::1009] *= 50.0  # outliers, so that every scale is in use
    return g


def compare(g, d, M, scales, bits, seed):
    a = Step(d, M, scales, device=DEV, bits=bits)
    assert a.one_call
    a.run(g, seed)
    b = Step(d, M, scales, device=DEV, bits=bits, **({"index_in_pass": False} if len(scales) > 1 else {}))
    b.shared_scale(g)
    # the index pass's norm is summed in another order: W to one ulp
    ulp = abs(int(a.w[:1].view(torch.int32)) - int(b.w[:1].view(torch.int32)))
    assert ulp <= (0 if len(scales) == 1 else 1)
    if ulp:
        b.w.copy_(a.w)
        b.idx.copy_(a.idx)
    b.quantize(g, seed)
    n = (d * bits + 7) // 8
    for m in range(M):
        for c in range(0, n, 1 << 28):
            assert torch.equal(a.codes[m, c:min(n, c + (1 << 28))], b.codes[m, c:min(n, c + (1 << 28))]), (m, c)
    a.codes = None
    b.sum_dequantize()
    if b.idx is not None:
        assert torch.equal(a.idx[:d], b.idx[:d])
        assert len(torch.unique(a.idx[:min(d, 1 << 26)])) > 1
    assert torch.equal(a.sum[:d], b.sum[:d])
    assert torch.equal(a.out[:d].view(torch.int32), b.out[:d].view(torch.int32))
    b.out.zero_()
    b.dequantize()
    assert torch.equal(a.out[:d].view(torch.int32), b.out[:d].view(torch.int32))
    del a, b
    torch.cuda.empty_cache()


@pytest.mark.parametrize("bits", [8, 4, 2])
@pytest.mark.parametrize("K", [1, 4])
@pytest.mark.parametrize("d,M", [(RESNET50, 8), (VGG16, 16)], ids=["resnet50", "vgg16"])
def test_model_sizes(d, M, K, bits):
    assert (M * ((d * bits + 7) // 8) > 512 << 20) == (d == VGG16)
    g = gradients(d, M, seed=bits + K)
    compare(g, d, M, [TOP[bits] * 16 ** k for k in range(K)], bits, seed=40 + bits)


@pytest.mark.parametrize("K,bits", [(1, 8), (4, 8), (1, 4), (4, 2)])
def test_rows_longer_than_2_pow_31(K, bits):
    """M * d past 2^32: the quantiser's grid is several launches."""
    d, M = (1 << 31) + 777, 2
    g = gradients(d, M, seed=31)
    compare(g, d, M, [TOP[bits] * 16 ** k for k in range(K)], bits, seed=50 + bits)
    del g
    torch.cuda.empty_cache()
