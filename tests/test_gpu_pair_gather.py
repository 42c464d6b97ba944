"""Corner gathers shared by neighbouring lanes (gather_pairs): odd query counts (the last
lane's partner has no query of its own), every row width, tables of an odd number of rows
(the wide form reads the last row with the one before it) and tables the wide form cannot
read, against the oracle."""
import numpy as np
import pytest

from oracle import hash4d_oracle as O
from paper_2507_19141_amd import _lib, synth
from tests.util import RTOL_F32, RTOL_GRAD, needs_gpu, scaled_close

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _table(table, dt, shift):
    """(device tensor kept alive, address): the table `shift` rows into an allocation."""
    import torch
    rows, F = table.shape
    host = O.bf16_bits(table).reshape(rows, F).view(np.int16) if dt == _lib.BF16 else table
    buf = torch.zeros(((rows + shift) * F,), dtype=torch.int16 if dt == _lib.BF16 else torch.float32, device="cuda")
    buf[shift * F:] = _dev(host).reshape(-1)
    return buf, buf.data_ptr() + shift * F * buf.element_size()


@pytest.mark.parametrize("n", [1, 2, 65, 1023])
@pytest.mark.parametrize("dt", [_lib.F32, _lib.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("F,shift", [(1, 0), (1, 1), (2, 0), (2, 1), (4, 0), (8, 0)])
def test_every_row_width(F, shift, dt, n):
    needs_gpu()
    import torch
    rs, rt, T = [2, 12, 200], [2, 6, 20], 1031          # 81 + 1031 + 1031 rows; a prime T: no pair need be adjacent
    L = len(rs)
    og, lg = O.make_grid(L, F, rs, rt, T), _lib.h4d_grid_init(L, F, rs, rt, T)
    assert og.E % 2 == 1
    rng, x = synth.small_inputs(n + 10 * F + shift, n)
    x[-1] = 1.0
    table = synth.table_init(og.E, F, rng)
    ref_t = O.bf16_value(O.bf16_bits(table)).reshape(table.shape) if dt == _lib.BF16 else table
    keep, addr = _table(table, dt, shift)
    feat = torch.full((n, L * F), float("nan"), device="cuda")
    _lib.hash4d_encode(lg, dt, addr, _dev(x), n, feat)
    ref, scale = O.encode(x, ref_t, og), O.encode(x, np.abs(ref_t), og)
    torch.cuda.synchronize()
    scaled_close(feat.cpu().numpy(), ref, scale, RTOL_F32, "encode")
    # the smoothness pass and the input gradient gather the same way
    eps = synth.perturbation(n, rng, 2e-2)
    loss = torch.zeros(1, device="cuda")
    _lib.smoothness_reg(lg, dt, addr, _dev(x), _dev(eps), n, 1.0, loss, None)
    xp = O.perturbed(x, eps)
    d = np.abs(ref - O.encode(xp, ref_t, og))
    want = float(np.sum(d * d)) / n
    bound = float(np.sum(2 * d * (scale + O.encode(xp, np.abs(ref_t), og)))) / n
    assert abs(float(loss.cpu()[0]) - want) <= RTOL_F32 * (want + bound)
    gf = synth.upstream(n, L * F, rng)
    d_x = torch.zeros((n, 4), device="cuda")
    wb = _lib.hash4d_encode_backward_input_workspace_bytes(lg, dt, n)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    _lib.hash4d_encode_backward_input(lg, dt, addr, _dev(x), n, _dev(gf), 1.0, d_x, _lib.QUERY_MAJOR, ws, wb)
    torch.cuda.synchronize()
    rows, _ = O.corners(x, og)
    dw = np.abs(O.corner_weight_derivatives(x, og))
    mag = np.zeros((n, 4))
    for l in range(L):
        tg = np.abs(ref_t[rows[:, l]] * gf[:, None, l * F:(l + 1) * F]).sum(-1)
        mag += (dw[:, l] * tg[:, :, None]).sum(1)
    scaled_close(d_x.cpu().numpy(), O.encode_backward_input(x, ref_t, og, gf), mag, RTOL_GRAD, "input gradient")


@pytest.mark.parametrize("n", [1, 129])
@pytest.mark.parametrize("stride", [3, 4])
@pytest.mark.parametrize("F,dt", [(1, _lib.F32), (2, _lib.F32), (2, _lib.BF16), (4, _lib.BF16), (8, _lib.F32)])
def test_encode3_pairs(F, dt, stride, n):
    needs_gpu()
    import torch
    res, T = [2, 9, 300], 515
    og, lg = O.make_grid3(3, F, res, T), _lib.h4d_grid3_init(3, F, res, T)
    rng, x = synth.small_inputs(n + F, n)
    x = np.ascontiguousarray(x[:, :stride])
    table = synth.table_init(og.E, F, rng)
    ref_t = O.bf16_value(O.bf16_bits(table)).reshape(table.shape) if dt == _lib.BF16 else table
    keep, addr = _table(table, dt, 0)
    feat = torch.full((n, 3 * F), float("nan"), device="cuda")
    _lib.hash3d_encode(lg, dt, addr, _dev(x), stride, n, feat)
    torch.cuda.synchronize()
    scaled_close(feat.cpu().numpy(), O.encode3(x[:, :3], ref_t, og), O.encode3(x[:, :3], np.abs(ref_t), og), RTOL_F32,
                 "encode3")
