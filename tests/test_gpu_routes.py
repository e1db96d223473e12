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
