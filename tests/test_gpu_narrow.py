"""BF16 inference of networks with d <= 64 runs on rows of 64 channels.  The same network padded to 128 channels is what
the persistent forward (model flags bit 3) runs, and a forward with ReadoutChEst on such a model runs its layers on 128
channels one by one: every product that differs has a zero operand and every sum keeps its order, so LLRs and channel
estimates are equal bit for bit.  Var-IO, which the persistent forward does not take, is held to the FP32 model at the
BF16 bar of 2e-2."""
import pytest

from nrx_cases import log

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
L = pytest.importorskip("paper_2409_02912_amd.libnrx")
from paper_2409_02912_amd import synth  # noqa: E402

BATCHES = {"one": [(1, 4, 1, [2])], "rows-44352": [(132, 4, 2, [4, 4])], "rows-71232": [(106, 4, 4, [4] * 4)],
           "mixed": [(9, 4, 3, [4, 2, 4]), (1, 2, 4, [2, 4, 4, 2]), (30, 4, 1, [4]), (17, 3, 2, [4, 2]), (23, 4, 3, [4] * 3)]}


def _run(d, flags, prec, shapes, n_ant, chest, C=3, R=2):
    m = L.nrx_model_create(n_ant, d, C, R, 4, prec, flags)
    try:
        lay = [(n, s) for n, _, s in L.weight_layout(m)]
        w = torch.from_numpy(synth.he_weights(lay, 11, perturb=True)).cuda()
        slots, sz = L.make_slots([dict(n_prb=p, n_ant=a, n_ue=u, bits=b) for p, a, u, b in shapes], 4)
        g = torch.Generator(device="cuda").manual_seed(12)
        y = torch.randn(2 * sz["y"], generator=g, device="cuda")
        ws = torch.empty(L.nrx_workspace_bytes(m, slots), dtype=torch.uint8, device="cuda")
        llr = torch.full((sz["llr"],), float("nan"), device="cuda")
        h = torch.full((2 * sz["h"],), float("nan"), device="cuda") if chest else None
        if chest:
            L.nrx_forward_chest(m, w, slots, y, llr, h, ws)
        else:
            L.nrx_forward(m, w, slots, y, llr, ws)
        torch.cuda.synchronize()
        return llr, h
    finally:
        L.nrx_model_destroy(m)


@pytest.mark.parametrize("chest", [False, True])
@pytest.mark.parametrize("d", [8, 32, 56, 64])
@pytest.mark.parametrize("name", list(BATCHES))
def test_64_channels_equal_128(name, d, chest):
    log(f"64-channel rows: {name}, d {d}, ReadoutChEst {chest}")
    fl = 2 if chest else 0
    a, ha = _run(d, fl, L.NRX_BF16, BATCHES[name], 4, chest)
    b, hb = _run(d, fl | 8, L.NRX_BF16, BATCHES[name], 4, chest)
    assert torch.isfinite(a).all()
    assert torch.equal(a, b)
    if chest:
        assert torch.isfinite(ha).all() and torch.equal(ha, hb)


def test_64_channels_16_antennas_and_one_iteration():
    shapes = [(5, 16, 2, [4, 4]), (4, 8, 4, [2] * 4)]
    for C, R in ((1, 0), (2, 2)):
        log(f"64-channel rows: 16 antennas, {C} blocks, {R} rounds")
        assert torch.equal(_run(40, 0, L.NRX_BF16, shapes, 16, False, C, R)[0], _run(40, 8, L.NRX_BF16, shapes, 16, False, C, R)[0])


def test_64_channels_var_io():
    log("64-channel rows: Var-IO")
    a, _ = _run(56, 4, L.NRX_BF16, BATCHES["mixed"], 4, False)
    b, _ = _run(56, 4, L.NRX_FP32, BATCHES["mixed"], 4, False)
    assert ((a - b).norm() / b.norm()).item() < 2e-2
