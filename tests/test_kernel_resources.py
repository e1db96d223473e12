"""Vector registers of the built kernels: what a wave holds decides how many
waves a SIMD runs."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2109_12497_amd as uq

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: vector registers} of libuq.so."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    blob = open(uq.LIB_PATH, "rb").read()
    out, tmp = {}, tmp_path_factory.mktemp("co")
    for n, m in enumerate(re.finditer(b"\x7fELF", blob)):
        at = m.start()
        if int.from_bytes(blob[at + 18:at + 20], "little") != 224:  # EM_AMDGPU
            continue
        f = tmp / f"{n}.co"
        f.write_bytes(blob[at:])
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block).group(1)
            out[name] = int(block.split()[0]) + int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1))
    assert out, "no gfx950 kernels found in libuq.so"
    return out


# One scale, mangled as <rows, stores, W from partials>.
@pytest.mark.parametrize("rows,at_most", [(4, 80), (6, 88), (8, 96)])
def test_one_scale_rows_pass_holds_only_its_rows(kernels, rows, at_most):
    """Where W is read from memory the registers of the partials' reduction,
    which such a call does not take, are not held beside the rows: 5 rows of
    5.0 M coordinates took 43.7 us with them, 42.7 without."""
    plain = {n: r for n, r in kernels.items() if re.search(rf"k_quant_sum_splitILi{rows}ELi\dELb0E", n)}
    assert len(plain) >= 3
    assert all(r <= at_most for r in plain.values()), plain


@pytest.mark.parametrize("rows,at_most", [(2, 66), (4, 90)])
def test_few_rows_of_stored_codes_hold_only_their_rows(kernels, rows, at_most):
    """The same for up to 4 rows of stored codes (mangled as <rows, several
    scales, bits, nontemporal, W from partials>): one row of 25.6 M
    coordinates 46.3 us with the reduction's registers, 44.9 without."""
    plain = {n: r for n, r in kernels.items() if re.search(rf"k_index_quantiseILi{rows}ELb\dELi\dELb\dELb0E", n)}
    assert len(plain) == 12
    assert all(r <= at_most for r in plain.values()), plain
