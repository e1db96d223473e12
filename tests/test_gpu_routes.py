"""Which kernels a step launches, at the sizes where the choice changes (read
from a HIP graph the step is captured into; results are compared elsewhere)."""
import re

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from launches import captured  # noqa: E402
from paper_2109_12497_amd.step import Step  # noqa: E402

DEV = torch.device("cuda:0")


def kernels(d, M, scales, **kw):
    """[(kernel, template arguments, grid)] of one step."""
    st = Step(d, M, scales, device=DEV, **kw)
    g = torch.zeros((M, -(-d // 64) * 64), device=DEV)
    return launched(lambda: st.run(g, 1))


def launched(fn):
    out = []
    for name, grid in captured(fn):
        m = re.match(r"_ZN2uq(\d+)", name)
        start = m.end()
        end = start + int(m.group(1))
        args = re.match(r"I((?:L[a-z]-?\d+E)+)E", name[end:])
        out.append((name[start:end], tuple(int(x) for x in re.findall(r"L[a-z](-?\d+)E", args.group(1))) if args else (),
                    grid))
    return out


def names(*args, **kw):
    return [k[0] for k in kernels(*args, **kw)]


# One block up to 4096 coordinates of 8 rows, 2048 of 16: 16 rows of 4096 took
# 18.6 us in one block, 12.3 as norm and rows pass.
@pytest.mark.parametrize("d,M,one_block", [(4096, 1, True), (4096, 8, True), (4097, 8, False), (2048, 9, True),
                                           (2048, 16, True), (2049, 9, False), (4096, 16, False)])
@pytest.mark.parametrize("bits", [0, 8])
def test_small_steps_in_one_block(d, M, one_block, bits):
    for scales in ([127.0], [127.0, 2032.0]):
        ks = names(d, M, scales, quant_sum=bits == 0)
        assert (ks == ["k_step_small"]) == one_block
        assert len(ks) == (1 if one_block else 2)


def test_one_row_takes_the_one_row_kernel():
    """The rows pass codes rows in pairs: with one row every second Philox
    block would be drawn for nothing (25.6 M coordinates: 72.9 us, 60.5 here)."""
    assert names(1_200_000, 1, [127.0], quant_sum=True) == ["k_sumsq", "k_finish", "k_quant_sum"]
    assert names(1 << 20, 1, [127.0], quant_sum=True) == ["k_sumsq", "k_quant_sum_split"]  # W formed in it


# k_quantise<several scales, bits, nontemporal>: codes up to 512 MB are left to
# the Infinity Cache, where their sum follows at once.
@pytest.mark.parametrize("rows,nontemporal", [(10, 0), (15, 0), (16, 0), (17, 1)])
def test_stored_codes_leave_nontemporally_beyond_512_mb(rows, nontemporal):
    d = 32_000_000
    st = Step(256, 1, [127.0], device=DEV)  # its W; the rows below are only captured, never run
    g = torch.empty((1, 64), device=DEV)
    codes = torch.empty((1, 64), dtype=torch.int8, device=DEV)
    import paper_2109_12497_amd as uq

    ks = launched(lambda: uq.uq_quantize_single(g, d, rows, d, 0, st.w, 127, 1, codes, d))
    assert [(k, a) for k, a, _ in ks] == [("k_quantise", (0, 8, nontemporal))]


# One quad a lane with one scale (256 coordinates a block), two with several.
@pytest.mark.parametrize("d", [1, 255, 256, 257, 511, 512, 513, 1025, 100_003])
def test_reconstruction_blocks(d):
    import numpy as np

    for scales, tile in (([127.0], 256), ([127.0, 2032.0], 512)):
        st = Step(d, 3, scales, device=DEV, fused=False, **({"index_in_pass": False} if len(scales) > 1 else {}))
        (k, a, grid), = launched(lambda: st.dequantize())
        assert k == "k_dequant" and a == (len(scales) > 1, 0) and grid[0] == -(-d // tile)
        rng = np.random.default_rng(d)
        s = rng.integers(-381, 382, size=d).astype(np.int32)
        idx = rng.integers(0, len(scales), size=d)
        st.sum[:d] = torch.from_numpy(s).to(DEV)
        if st.idx is not None:
            st.idx[:d] = torch.from_numpy(idx.astype(np.uint8)).to(DEV)
        W = np.float32(0.37)
        st.w[0] = float(W)
        st.out.fill_(-1.0)
        st.dequantize()
        deq = np.array([W / np.float32(3 * x) for x in scales], dtype=np.float32)
        assert np.array_equal(st.out[:d].cpu().numpy(), s.astype(np.float32) * deq[idx])
        assert bool((st.out[d:] == -1.0).all())


# k_quant_sum_split<rows, stores, W from partials>: stores 0 through, 3 the
# sums through and the outputs nontemporally, 1 both nontemporally, 2 both hints.
@pytest.mark.parametrize("d,stores", [(11_173_962, 0), (12_058_624, 0), (12_058_625, 3), (16_000_001, 3),
                                      (23_068_672, 3), (23_068_673, 1), (67_108_864, 1), (67_108_865, 2)])
def test_stores_of_the_one_scale_rows_pass(d, stores):
    import paper_2109_12497_amd as uq

    st = Step(256, 6, [127.0], device=DEV)  # buffers of a small step: captured only, never run
    ks = launched(lambda: uq.uq_quantize_sum(st.out, d, 6, -(-d // 64) * 64, 0, st.w, [127.0], 1, None, 1, 0, st.sum,
                                             6, st.out, None))
    assert [(k, a) for k, a, _ in ks] == [("k_quant_sum_split", (6, stores, 0))]


# A tile's rows split over four waves (one scale): 11 to 16 rows up to 8192
# tiles, 8 rows beyond 16384 tiles up to 46 MB of outputs.
@pytest.mark.parametrize("d,M,kernel", [(100_003, 10, "k_quant_sum_split"), (100_003, 11, "k_quant_sum_waves"),
                                        (1 << 21, 16, "k_quant_sum_waves"), ((1 << 21) + 1, 16, "k_quant_sum_split"),
                                        (1 << 22, 8, "k_quant_sum_split"), ((1 << 22) + 1, 8, "k_quant_sum_waves"),
                                        ((1 << 22) + 1, 7, "k_quant_sum_split"), (11_173_962, 8, "k_quant_sum_waves"),
                                        (12_058_624, 8, "k_quant_sum_waves"), (12_058_625, 8, "k_quant_sum_split")])
def test_many_rows_split_over_waves(d, M, kernel):
    assert names(d, M, [127.0], quant_sum=True)[-1] == kernel


# Stored codes of one scale: quantiser and sum apart, or summed as they are stored.
@pytest.mark.parametrize("d,M,ks", [
    (1 << 19, 16, ["k_sumsq", "k_index_quantise"]),                        # 1024 partials: W formed in the pass
    ((1 << 19) + 1, 16, ["k_sumsq", "k_finish", "k_quantise", "k_sum"]),
    (1 << 20, 13, ["k_sumsq", "k_finish", "k_quantise", "k_sum"]),
    (1 << 20, 12, ["k_sumsq", "k_finish", "k_index_quantise"]),
    ((1 << 20) + 1, 4, ["k_sumsq", "k_finish", "k_quantise", "k_sum"]),    # more than 128 partials a row
])
def test_stored_codes_of_one_scale(d, M, ks):
    assert names(d, M, [127.0]) == ks
