"""GPU parity for GlobalRandK (Sec. 3.3-3.4): the selected index list
bit-exact against the oracle, gather/scatter exact, and the whole step
(selection, Algorithm 1/2 on the sampled coordinates, scatter) bit-exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import synth  # noqa: E402
from oracle import oracle as O  # noqa: E402
import paper_2109_12497_amd as uq  # noqa: E402
from paper_2109_12497_amd.step import RandKStep  # noqa: E402

DEV = torch.device("cuda:0")


def gpu_select(d, K, seed):
    st = RandKStep(d, 1, K, [127.0], device=DEV)
    st.select(seed)
    torch.cuda.synchronize()
    return st.sel[:K].cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("d,K,seed", [
    (1, 1, 0), (2, 1, 5), (5, 5, 1), (7, 3, 2), (100, 99, 3), (1000, 1, 4), (4097, 4096, 5),
    (65_539, 10_000, 6), (1 << 20, 32_768, 7), (1 << 20, 10_000, (1 << 63) + 12345), (300_000, 250_000, 10),
    (3_000_001, 10_000, 8), (11_173_962, 10_000, 9),
    # both sides of the largest K that one block sorts
    (100_000, 16_384, 11), (100_000, 16_385, 12),
])
@pytest.mark.parametrize("mode", [1, 0, 2, 3, 4], ids=["bracket", "histograms", "bracket-missed",
                                                     "histograms-refined", "bracket-missed-refined"])
def test_selection_matches_oracle(d, K, seed, mode):
    """Each way of finding the subset (for K <= 16384: the bracket of the K-th
    key, the histogram passes, and the bracket made to miss so that the
    selection block's exact fallback runs; and both of the last two with no
    boundary candidates kept, so that the exact refinement by the K-th key's
    whole 32-bit high word runs, as it does when more candidates arrive than
    the lists keep) against the oracle."""
    uq.uq_set_randk_mode(mode)
    try:
        got = gpu_select(d, K, seed)
    finally:
        uq.uq_set_randk_mode(1)
    want = O.randk_select(d, K, seed)
    assert np.array_equal(got, want)


def test_selection_repeatable_and_seeded():
    a = gpu_select(500_000, 2000, 1)
    b = gpu_select(500_000, 2000, 1)
    c = gpu_select(500_000, 2000, 2)
    assert np.array_equal(a, b) and not np.array_equal(a, c)


def test_gather_scatter_exact():
    d, M, K = 100_003, 3, 777
    host = synth.mixed_rows(M, d, seed=1, ldg=synth.round_up(d, 64))
    g = torch.from_numpy(host).to(DEV)
    st = RandKStep(d, M, K, [127.0], device=DEV)
    st.select(3)
    st.gather(g)
    st.inner.out[:K].copy_(torch.arange(K, dtype=torch.float32, device=DEV) + 0.5)
    st.out.fill_(7.0)
    st.scatter()
    torch.cuda.synchronize()
    sel = st.sel[:K].cpu().numpy().view(np.uint32).astype(np.int64)
    assert np.array_equal(st.sub[:, :K].cpu().numpy().view(np.int32), host[:, sel].view(np.int32))
    full = np.zeros(d, dtype=np.float32)
    full[sel] = np.arange(K, dtype=np.float32) + 0.5
    assert np.array_equal(st.out[:d].cpu().numpy(), full)


@pytest.mark.parametrize("scales", [[127.0], synth.scales_for(8, 2), synth.scales_for(4, 4)],
                         ids=["single", "two-scale", "K4"])
def test_randk_step_matches_oracle(scales):
    d, M, K = 1_000_003, 4, 10_000
    host = synth.mixed_rows(M, d, seed=7, ldg=synth.round_up(d, 64))
    g = torch.from_numpy(host).to(DEV)
    st = RandKStep(d, M, K, scales, device=DEV)
    out = st.run(g, seed=42)
    torch.cuda.synchronize()
    W = np.float32(st.inner.w[0].item())
    ref = O.randk_pipeline(host, K, scales, seed=42, d=d, W=W)
    assert abs(int(W.view(np.int32)) - int(ref["W_oracle"].view(np.int32))) <= 1
    assert np.array_equal(st.sel[:K].cpu().numpy().view(np.uint32), ref["sel"])
    assert np.array_equal(st.inner.codes[:, :K].cpu().numpy(), ref["codes"])
    assert np.array_equal(st.inner.sum[:K].cpu().numpy(), ref["sum"])
    assert np.array_equal(out.cpu().numpy().view(np.int32), ref["full"].view(np.int32))


def test_randk_workload_full_size():
    """The ResNet-18-shaped workload with the paper's K = 10000."""
    g, cfg = synth.make_gradients("resnet18", device=DEV)
    d, M = cfg["d"], cfg["M"]
    st = RandKStep(d, M, 10_000, [127.0], device=DEV)
    out = st.run(g, seed=2)
    torch.cuda.synchronize()
    sel = O.randk_select(d, 10_000, 2)
    assert np.array_equal(st.sel[:10_000].cpu().numpy().view(np.uint32), sel)
    host_sub = g[:, torch.from_numpy(sel.astype(np.int64)).to(DEV)].cpu().numpy()
    W = np.float32(st.inner.w[0].item())
    ref = O.pipeline(host_sub, [127.0], 2, W=W)
    full = np.zeros(d, dtype=np.float32)
    full[sel.astype(np.int64)] = ref["out"]
    assert np.array_equal(out.cpu().numpy().view(np.int32), full.view(np.int32))


def _key(hi, lo, i):
    return (int(hi) << 64) | (int(lo) << 32) | int(i)


@pytest.mark.parametrize("d,K", [(2 ** 32 - 1, 10_000), (3_000_000_007, 16_385)])
def test_selection_at_the_largest_d(d, K):
    """d up to 2^32 - 1 (about 4096 boundary candidates, uint32 indices near
    their limit), on both selection paths.  The oracle cannot sort 4e9 keys,
    so the rule is checked exactly inside windows: a coordinate there is
    selected iff its (hi, lo, i) is at most the largest selected one."""
    import paper_2109_12497_amd as uq

    seed = 21
    sel = torch.zeros(K + 64, dtype=torch.int32, device=DEV)
    wsb = uq.uq_randk_workspace_bytes(d, K)
    ws = torch.zeros(wsb // 4 + 64, dtype=torch.int32, device=DEV)
    uq.uq_randk_select(d, K, seed, sel, ws, wsb)
    torch.cuda.synchronize()
    got = sel[:K].cpu().numpy().view(np.uint32).astype(np.int64)
    assert np.all(np.diff(got) > 0) and got[0] >= 0 and got[-1] < d
    keys = [O.randk_keys(seed, int(i), 1) for i in got]
    top = max(_key(h[0], l[0], i) for (h, l), i in zip(keys, got))
    chosen = set(got.tolist())
    n = 1 << 20
    for i0 in (0, (1 << 31) - n // 2, d - n):
        hi, lo = O.randk_keys(seed, i0, n)
        # candidates by the high word first (cheap), then the exact rule
        near = np.nonzero(hi.astype(np.uint64) <= (top >> 64))[0]
        below = {i0 + int(j) for j in near if _key(hi[j], lo[j], i0 + int(j)) <= top}
        inside = {i for i in chosen if i0 <= i < i0 + n}
        assert below == inside, (i0, len(below), len(inside))


def _random_selections(n=18, seed=3344):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        d = int(rng.choice([int(rng.integers(1, 2000)), int(rng.integers(2000, 200_000)),
                            int(rng.integers(200_000, 1_500_000))]))
        K = int(rng.choice([1, int(rng.integers(1, d + 1)), min(d, int(rng.integers(1, 20_000)))]))
        out.append((d, K, int(rng.integers(0, 2 ** 64, dtype=np.uint64)), i % 5))
    return out


@pytest.mark.parametrize("d,K,seed,mode", _random_selections())
def test_random_selections(d, K, seed, mode):
    """Seeded random (d, K, seed) in every selection mode, against the oracle."""
    uq.uq_set_randk_mode([1, 0, 2, 3, 4][mode])
    try:
        got = gpu_select(d, K, seed)
    finally:
        uq.uq_set_randk_mode(1)
    assert np.array_equal(got, O.randk_select(d, K, seed))


@pytest.mark.parametrize("mode", [1, 0, 2], ids=["bracket", "histograms", "bracket-missed"])
@pytest.mark.parametrize("d,K,M", [(1, 1, 1), (6, 2, 3), (4096, 100, 2), (4097, 4000, 5), (16_384, 16_384, 1),
                                   (20_483, 9000, 4), (512 * 4096 - 3, 16_384, 2), (512 * 4096 + 1, 1000, 3),
                                   (2048 * 4096 + 5, 3000, 2), (100_001, 20_000, 2), (70_000, 10_000, 17)])
def test_select_gather_and_scatter_into(d, K, M, mode):
    """Selection, gather and the output's zeroing in one call, from one list
    of the key pass to the most and past one iteration of each; nothing past
    d or K is touched."""
    if mode == 2 and d > 100_000:
        pytest.skip("the slow fallback, covered at small sizes")
    host = synth.gaussian_rows(M, d, seed=d, ldg=synth.round_up(d, 64))
    g = torch.from_numpy(host).to(DEV)
    st = RandKStep(d, M, K, [127.0], device=DEV)
    out = torch.full((d + 64,), 3.0, device=DEV)
    sub = torch.full_like(st.sub, 5.0)
    vals = torch.arange(1, K + 1, dtype=torch.float32, device=DEV)
    uq.uq_set_randk_mode(mode)
    try:
        uq.uq_randk_select_gather(g, d, M, g.stride(0), K, 31, st.sel, sub, sub.stride(0), out, st.rk_ws,
                                  st.rk_ws_bytes)
        assert not out[:d].any() and bool((out[d:] == 3.0).all())
        out.fill_(2.0)
        uq.uq_randk_select_gather(g, d, M, g.stride(0), K, 31, st.sel, sub, sub.stride(0), None, st.rk_ws,
                                  st.rk_ws_bytes)
        assert bool((out == 2.0).all())
        uq.uq_scatter_into(vals, st.sel, K, out, d)
        torch.cuda.synchronize()
    finally:
        uq.uq_set_randk_mode(1)
    sel = O.randk_select(d, K, 31)
    assert np.array_equal(st.sel[:K].cpu().numpy().view(np.uint32), sel)
    at = sel.astype(np.int64)
    assert np.array_equal(sub[:, :K].cpu().numpy().view(np.int32), host[:, at].view(np.int32))
    assert bool((sub[:, K:] == 5.0).all())
    full = np.full(d, 2.0, dtype=np.float32)
    full[at] = np.arange(1, K + 1, dtype=np.float32)
    assert np.array_equal(out[:d].cpu().numpy(), full)


def test_gradients_in_the_steps_own_output():
    d, K = 50_003, 2000
    host = synth.gaussian_rows(1, d, seed=5, ldg=synth.round_up(d, 64))
    a, b = RandKStep(d, 1, K, [127.0], device=DEV), RandKStep(d, 1, K, [127.0], device=DEV)
    a.out[:d].copy_(torch.from_numpy(host[0, :d]))
    got = a.run(a.out.unsqueeze(0), 4)
    want = b.run(torch.from_numpy(host).to(DEV), 4)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))


def test_gradients_inside_the_output_under_another_storage():
    """The output may not be zeroed before the gather where the gradients lie
    in its memory, also when they come through an exchange that gives the same
    memory a storage of its own."""
    from paper_2109_12497_amd.step import RandKStep

    d, M, k, ldg = 30_000, 4, 500, 30_016
    host = synth.gaussian_rows(M, d, seed=12, ldg=ldg)
    want = RandKStep(d, M, k, [127.0], device=DEV)
    ref = want.run(torch.from_numpy(host).to(DEV), 9).clone()
    st = RandKStep(d, M, k, [127.0], device=DEV)
    st.out = torch.zeros(64 + M * ldg, dtype=torch.float32, device=DEV)
    g = torch.from_dlpack(st.out[64:]).view(M, ldg)
    assert g.untyped_storage().data_ptr() != st.out.untyped_storage().data_ptr()
    g.copy_(torch.from_numpy(host))
    assert torch.equal(st.run(g, 9), ref)
