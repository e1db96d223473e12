"""uq_aggregate (a whole step in one call) against the separate calls and the
oracle, bit for bit, at the sizes where its routes and tiles change (SIZES),
256-coordinate tiles with a partial last one, and each number of row pairs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import synth  # noqa: E402
from oracle import oracle as O  # noqa: E402
import paper_2109_12497_amd as uq  # noqa: E402
from paper_2109_12497_amd.step import Step  # noqa: E402

DEV = torch.device("cuda:0")
# (d, M): tile and route edges: one block up to 4096 coordinates of 8 rows and
# 2048 of more; W formed by the rows pass (its partials reduced by every wave,
# two a lane from 65 a row on) up to 128 partials a row and 1024 in all; a
# tile's rows split over four waves from 11 rows on
SIZES = [(1, 1), (3, 2), (255, 3), (256, 5), (257, 8), (1000, 8), (2049, 16), (4095, 9), (4096, 4), (4097, 16),
         (8193, 7), (65_537, 13), (100_003, 6), (64 * 8192, 16), (64 * 8192 + 5, 16), (300_001, 1),
         (2048, 11), (4096, 9), (20_001, 11), (64 * 8192 + 1, 4), (65 * 8192, 15), (128 * 8192, 8), (128 * 8192, 1),
         (128 * 8192 + 1, 3), (128 * 8192, 13)]
SCALES = {"s127": [127.0], "K4": synth.scales_for(8, 4), "crowded": [1.0, 2.0, 3.0, 127.0]}


def separate(step, g, seed):
    """The same step through its separate calls."""
    step.shared_scale(g, w_only=True)
    if step.K > 1 and step.quant_sum:
        step.index_quantize_sum(g, seed)
    elif step.K > 1:
        step.index_quantize(g, seed)
        step.sum_dequantize()
    elif step.quant_sum:
        step.quantize_sum(g, seed)
    else:
        step.quantize(g, seed)
        step.sum_dequantize()


@pytest.mark.parametrize("d,M", SIZES)
@pytest.mark.parametrize("name,bits", [("s127", 0), ("s127", 8), ("K4", 0), ("K4", 8), ("crowded", 4), ("crowded", 2)])
def test_one_call_equals_the_separate_calls(d, M, name, bits):
    scales = SCALES[name]
    host = synth.mixed_rows(M, d, seed=d + M, ldg=synth.round_up(d, 64))
    if d > 300:  # non-finite padding past d is never read into a result
        host[:, d:] = np.nan
    g = torch.from_numpy(host).to(DEV)
    kw = dict(quant_sum=bits == 0, bits=bits or 8)
    a, b = Step(d, M, scales, device=DEV, **kw), Step(d, M, scales, device=DEV, **kw)
    assert a.one_call
    a.run(g, 99)
    separate(b, g, 99)
    torch.cuda.synchronize()
    assert torch.equal(a.w[:1].view(torch.int32), b.w[:1].view(torch.int32))
    for x, y in ((a.sum, b.sum), (a.out.view(torch.int32), b.out.view(torch.int32)), (a.idx, b.idx), (a.codes, b.codes)):
        assert (x is None and y is None) or torch.equal(x, y)
    if M * d < 300_000:
        W = np.float32(a.w[0].item())
        ref = O.pipeline(np.ascontiguousarray(host), scales, seed=99, d=d, W=W)
        assert np.array_equal(a.sum[:d].cpu().numpy(), ref["sum"])
        assert np.array_equal(a.out[:d].cpu().numpy().view(np.int32), ref["out"].view(np.int32))
        if len(scales) > 1:
            assert np.array_equal(a.index_host(), ref["idx"])
        if a.codes is not None and bits == 8:
            assert np.array_equal(a.codes[:, :d].cpu().numpy(), ref["codes"])


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("d", [700, 20_000])
def test_non_finite_rows_take_the_zero_path(value, d):
    M = 5
    host = synth.gaussian_rows(M, d, seed=3, ldg=synth.round_up(d, 64))
    host[2, d // 3] = value
    g = torch.from_numpy(host).to(DEV)
    for scales in (SCALES["s127"], SCALES["K4"]):
        st = Step(d, M, scales, device=DEV)
        st.codes.fill_(9)
        st.run(g, 1)
        torch.cuda.synchronize()
        assert not np.isfinite(st.w[0].item())
        assert not st.codes[:, :d].any() and not st.sum[:d].any() and not st.out[:d].any()
        assert st.idx is None or bool((st.idx[:d] == len(scales) - 1).all())


@pytest.mark.parametrize("cap", [8, 24])
def test_capped_grids(cap):
    """Several launches per pass (the grid capped far below one tile per block)."""
    d, M = 40_003, 6
    host = synth.mixed_rows(M, d, seed=cap, ldg=synth.round_up(d, 64))
    g = torch.from_numpy(host).to(DEV)
    for name, bits in (("s127", 8), ("K4", 0)):
        a = Step(d, M, SCALES[name], device=DEV, quant_sum=bits == 0)
        uq.uq_set_grid_cap(cap)
        try:
            a.run(g, 5)
            torch.cuda.synchronize()
        finally:
            uq.uq_set_grid_cap(0)
        ref = O.pipeline(host, SCALES[name], seed=5, d=d, W=np.float32(a.w[0].item()))
        assert np.array_equal(a.out[:d].cpu().numpy().view(np.int32), ref["out"].view(np.int32))


def test_invalid_calls_are_refused():
    d, M = 512, 4
    g = torch.zeros((17, 512), device=DEV)
    st = Step(d, M, [7.0], device=DEV)

    def call(M=M, scales=(7.0,), bits=8, idx=None, codes=st.codes, ws_bytes=st.ws_bytes):
        uq.uq_aggregate(g, d, M, 512, list(scales), len(scales), 1, bits, st.w, idx, codes, st.ldc, st.sum, st.out,
                        st.ws, ws_bytes)

    call()
    for kw in (dict(M=17), dict(bits=3), dict(bits=2), dict(scales=(7.0, 112.0)), dict(idx=st.sum), dict(codes=None),
               dict(ws_bytes=16), dict(scales=(0.5,))):
        with pytest.raises(uq.UQError):
            call(**kw)


@pytest.mark.parametrize("bits", [8, 4])
def test_codes_go_to_the_buffer_the_step_holds(bits):
    """A wider codes buffer put in the step's place (one allocation for several
    layers): its own row stride counts, not the one the step was made with."""
    d, M = 5000, 6
    host = synth.mixed_rows(M, d, seed=8, ldg=synth.round_up(d, 64))
    g = torch.from_numpy(host).to(DEV)
    scales = [127.0 if bits == 8 else 7.0]
    a, b = (Step(d, M, scales, device=DEV, bits=bits) for _ in range(2))
    b.codes = torch.zeros((M, a.ldc + 512), dtype=torch.int8, device=DEV)
    a.run(g, 4)
    b.run(g, 4)
    n = (d * bits + 7) // 8
    assert torch.equal(a.codes[:, :n], b.codes[:, :n])
    assert not b.codes[:, a.ldc:].any()


@pytest.mark.parametrize("d,M", [(1 << 21, 11), ((1 << 21) + 1, 11), (1 << 21, 16), ((1 << 21) + 1, 16),
                                 (1 << 22, 8), ((1 << 22) + 1, 8), ((1 << 22) + 255, 8), (12_058_624, 8),
                                 (12_058_625, 8)])
def test_rows_split_over_waves_at_its_edges(d, M):
    """One scale: a tile's rows are split over four waves with 11 to 16 rows of
    up to 8192 tiles, and with 8 rows beyond 16384 tiles up to 46 MB of
    outputs; otherwise one wave holds them all."""
    g = torch.empty((M, synth.round_up(d, 64)), device=DEV)
    g.normal_(0.0, 1e-3, generator=torch.Generator(device=DEV).manual_seed(d + M))
    a, b = (Step(d, M, [127.0], device=DEV, quant_sum=True) for _ in range(2))
    a.run(g, 21)
    b.shared_scale(g, w_only=True)
    for m in range(M):
        b.quantize_sum(g[m:m + 1], 21, rows=1, worker0=m, accumulate=int(m > 0), reconstruct=m == M - 1)
    assert torch.equal(a.w[:1].view(torch.int32), b.w[:1].view(torch.int32))
    assert torch.equal(a.sum, b.sum) and torch.equal(a.out.view(torch.int32), b.out.view(torch.int32))
    g[1, d - 1] = float("nan")  # under the same W, in the last tile
    g[M - 1, 5] = float("inf")
    a.quantize_sum(g, 21)
    for m in range(M):
        b.quantize_sum(g[m:m + 1], 21, rows=1, worker0=m, accumulate=int(m > 0), reconstruct=m == M - 1)
    assert torch.equal(a.sum, b.sum) and torch.equal(a.out.view(torch.int32), b.out.view(torch.int32))


# W given, not formed from the rows: the codes of finite values stay, and
# infinite or NaN ones are 0 and do not raise a coordinate's index
@pytest.mark.parametrize("W", [1.0, 1e-33])
@pytest.mark.parametrize("d,M", [(700, 2), (5003, 5), (5003, 8), (20_001, 11), (20_001, 16)])
@pytest.mark.parametrize("call", ["index_quantize", "index_quantize4", "index_quantize_sum", "quantize_sum"])
def test_non_finite_values_under_a_finite_scale(call, d, M, W):
    scales = [127.0] if call == "quantize_sum" else [7.0, 112.0, 1792.0]
    host = synth.mixed_rows(M, d, seed=d * M, ldg=synth.round_up(d, 64))
    host[:, :d] *= np.float32(0.3 * W) / np.abs(host[:, :d]).max()
    rng = np.random.default_rng(d)
    for value in (np.inf, -np.inf, np.nan):  # alone, in both rows of a pair, and in the last, ragged tile
        for m, i in [(0, int(rng.integers(d))), (M - 1, int(rng.integers(d))), (M - 1, d - 1), (M // 2, d - 2),
                     (min(1, M - 1), d - 1)]:
            host[m, i] = value
    host[:, d // 2] = np.nan  # no usable value in the coordinate
    g = torch.from_numpy(host).to(DEV)
    bits = 4 if call.endswith("4") else 8
    st = Step(d, M, scales, device=DEV, bits=bits, quant_sum=call.endswith("sum"))
    st.w[0] = W
    getattr(st, call.rstrip("4"))(g, 31)
    torch.cuda.synchronize()
    ref = O.pipeline(host, scales, seed=31, d=d, W=np.float32(W))
    assert np.abs(ref["codes"]).max() > 0
    if len(scales) > 1:
        assert np.array_equal(st.index_host(), ref["idx"])
        assert len(np.unique(ref["idx"])) > 1
    if call.endswith("sum"):
        assert np.array_equal(st.sum[:d].cpu().numpy(), ref["sum"])
        assert np.array_equal(st.out[:d].cpu().numpy().view(np.int32), ref["out"].view(np.int32))
    else:
        codes = st.codes.cpu().numpy()
        got = codes[:, :d] if bits == 8 else np.stack([O.unpack_codes(codes[m].view(np.uint8)[:(d + 1) // 2], d, 4)
                                                       for m in range(M)])
        assert np.array_equal(got, ref["codes"])
