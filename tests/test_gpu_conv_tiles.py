"""The default convolution picks its tile (128 to 512 rows) by the number of rows of a launch.  Whatever the tile, an
output is the same products accumulated in the same order: BF16 LLRs equal those of a fixed-tile variant bit for bit.
FP32 models run their block convolutions on three BF16 parts per operand there, exact products with fewer roundings than
the FP32 variant: the two agree to 1e-5 (each is about 1e-6 from 64 bits after two blocks).
The training epilogues add their LayerNorm gradients up per tile, so a batch of n copies of one slot must give n times
that slot's gradient up to the rounding of the sums: fp32 partial sums of at most 512 rows x a few hundred workgroups,
each addition 6e-8 relative, random in sign, far below 1e-5 of the gradient's norm."""
import numpy as np
import pytest

from nrx_cases import log

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
L = pytest.importorskip("paper_2409_02912_amd.libnrx")
from paper_2409_02912_amd import synth  # noqa: E402

FIXED, DEFAULT = 7, 14


def _model(prec, n_ant=4):
    m = L.nrx_model_create(n_ant, 128, 2, 1, 4, prec)
    lay = [(n, s) for n, _, s in L.weight_layout(m)]
    return m, torch.from_numpy(synth.he_weights(lay, 3, perturb=True)).cuda()


# rows per batch: one tile or less, 128-row tiles, 256, 384, 512, two rounds of 384, and slots of different UE counts
SIZES = {"one-prb": [(1, 1)], "rows-30240": [(180, 1)], "rows-44352": [(132, 2)], "rows-71232": [(106, 4)],
         "rows-120960": [(180, 4)], "rows-183456": [(273, 4)], "mixed": [(37, 3), (5, 1), (61, 4), (2, 2), (90, 3)]}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("size", list(SIZES))
def test_tile_rule_keeps_every_bit(size, prec):
    log(f"conv tiles: {size}, precision {prec}")
    m, w = _model(prec)
    try:
        slots, sz = L.make_slots([dict(n_prb=p, n_ant=4, n_ue=u, bits=[4] * u) for p, u in SIZES[size]], 4)
        g = torch.Generator(device="cuda").manual_seed(5)
        y = torch.randn(2 * sz["y"], generator=g, device="cuda")
        ws = torch.empty(L.nrx_workspace_bytes(m, slots), dtype=torch.uint8, device="cuda")
        out = []
        for v in (FIXED, DEFAULT):
            L.set_all_conv_variants(m, v)
            llr = torch.full((sz["llr"],), float("nan"), device="cuda")
            L.nrx_forward(m, w, slots, y, llr, ws)
            torch.cuda.synchronize()
            out.append(llr)
        assert torch.isfinite(out[0]).all()
        if prec == 1:
            assert torch.equal(out[0], out[1])
        else:
            assert ((out[0] - out[1]).double().norm() / out[0].double().norm()).item() < 1e-5
    finally:
        L.nrx_model_destroy(m)


@pytest.mark.parametrize("prec", [0, 1])
def test_gradient_of_copies(prec):
    log(f"conv tiles: gradients of copies of one slot, precision {prec}")
    m, w = _model(prec)
    try:
        ref = None
        for n in (1, 6, 10, 25):
            slots, sz = L.make_slots([dict(n_prb=11, n_ant=4, n_ue=4, bits=[4] * 4, slot_number=0)] * n, 4)
            g = torch.Generator(device="cuda").manual_seed(5)
            y = torch.randn(2 * sz["y"] // n, generator=g, device="cuda").repeat(n)
            dl = torch.randn(sz["llr"] // n, generator=g, device="cuda").repeat(n)
            ws = torch.empty(L.nrx_workspace_bytes(m, slots, save_acts=True), dtype=torch.uint8, device="cuda")
            llr = torch.empty(sz["llr"], device="cuda")
            dw = torch.full_like(w, float("nan"))
            L.nrx_forward(m, w, slots, y, llr, ws, save_acts=True)
            L.nrx_backward(m, w, slots, dl, dw, ws)
            torch.cuda.synchronize()
            got = dw.double().cpu().numpy() / n
            assert np.all(np.isfinite(got))
            if ref is None:
                ref = got
            for name, off, shape in L.weight_layout(m):
                a, b = got[off:off + int(np.prod(shape))], ref[off:off + int(np.prod(shape))]
                assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), (n, name)
    finally:
        L.nrx_model_destroy(m)


@pytest.mark.parametrize("shapes", [[(1, 3), (2, 4)], [(7, 2), (1, 4), (3, 1), (5, 3)], [(1, 1)] * 9])
@pytest.mark.parametrize("prec", [0, 1])
def test_gradient_of_a_batch_is_the_sum_over_its_slots(shapes, prec):
    """Batches of remainders (tiles shorter than a step, partitions without rows, every UE count side by side): no slot's
    layers see another's, so the gradient of the batch is the sum of the slots' own up to the rounding of fp32 sums over
    at most a few thousand rows, 1e-5 of the norm as above."""
    log(f"conv tiles: gradient of a batch {shapes}, precision {prec}")
    m, w = _model(prec)

    def gradient(batch, y, dl):
        slots, sz = L.make_slots(batch, 4)
        ws = torch.empty(L.nrx_workspace_bytes(m, slots, save_acts=True), dtype=torch.uint8, device="cuda")
        llr = torch.empty(sz["llr"], device="cuda")
        dw = torch.full_like(w, float("nan"))
        L.nrx_forward(m, w, slots, y, llr, ws, save_acts=True)
        L.nrx_backward(m, w, slots, dl, dw, ws)
        torch.cuda.synchronize()
        return dw.double().cpu().numpy()
    try:
        batch = [dict(n_prb=p, n_ant=4, n_ue=u, bits=[4] * u, slot_number=i) for i, (p, u) in enumerate(shapes)]
        g = torch.Generator(device="cuda").manual_seed(9)
        ys = [torch.randn(2 * 12 * p * 14 * 4, generator=g, device="cuda") for p, _ in shapes]
        ds = [torch.randn(u * 14 * 12 * p * 4, generator=g, device="cuda") for p, u in shapes]
        got = gradient(batch, torch.cat(ys), torch.cat(ds))
        ref = sum(gradient([b], y, d) for b, y, d in zip(batch, ys, ds))
        for name, off, shape in L.weight_layout(m):
            a, b = (x[off:off + int(np.prod(shape))] for x in (got, ref))
            assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), name
    finally:
        L.nrx_model_destroy(m)
