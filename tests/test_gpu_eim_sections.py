"""Effective-index fields at the edges of the column kernels' tiles: columns in
groups of 16 and 64, rows in groups of 16, the permittivities in LDS up to 1024
rows and from memory beyond, the line solve in groups of 64 rows."""
import numpy as np
import pytest

import workloads as W
from oracle import eim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(9, 8), (16, 9), (17, 15), (63, 16), (64, 257), (65, 1024),
                                   (33, 1025), (129, 1031), (193, 40)])
def test_random_permittivity_matches_oracle(nx, ny):
    """The field is FP64 rounded to complex64: an error of 2^-24 of each value.
    The line equation amplifies the modes' rounding (2^-53 times the rows) by
    its condition, which stays below 1e6 here."""
    import torch
    from paper_1902_00090_amd import FdfdOp, eim_field
    rng = np.random.default_rng(nx * 10000 + ny)
    eps = (2.085 + 10.165 * rng.random((ny, nx))).astype(np.float32)
    inst = W.Instance(eps, W.random_complex(rng, nx * ny), nx, ny, 0.025, 1.30, 3)
    op = FdfdOp.from_instance(inst)
    (F,) = eim_field([op], [torch.tensor(inst.b, device="cuda")])
    want = eim.eim_instance(inst)
    tol = 2.0 ** -24 * np.abs(want) + 1e6 * ny * 2.0 ** -53 * np.abs(want).max()
    assert (np.abs(F.cpu().numpy() - want) <= tol).all()


@pytest.mark.parametrize("entry", ["eim_field", "eim_field_noalloc"])
@pytest.mark.parametrize("over", [(0, 1, 2), (1, 0, 2)])
def test_outputs_in_the_memory_of_right_hand_sides(entry, over):
    """A field may be written over its own right-hand side, or over another
    problem's: every right-hand side is read before an output is written."""
    import torch
    from paper_1902_00090_amd import FdfdOp, _lib, eim_field
    insts = [W.grating(1020, nx=97, ny=43, npml=7), W.grating(1021, nx=97, ny=43, npml=7),
             W.grating(1022, nx=65, ny=30, npml=7)]
    ops = [FdfdOp.from_instance(i) for i in insts]
    want = eim_field(ops, [torch.tensor(i.b, device="cuda") for i in insts])
    # the right-hand sides behind each other in one buffer, field p in the place of
    # right-hand side over[p]
    buf = torch.cat([torch.tensor(i.b, device="cuda") for i in insts])
    at = [0, insts[0].D, insts[0].D + insts[1].D]
    F = [buf.view(torch.complex64)[2 * at[o]:2 * at[o] + i.D] for o, i in zip(over, insts)]
    _lib.check(getattr(_lib.lib(), entry)(
        _lib.ptr_array([op.handle for op in ops]), 3,
        _lib.ptr_array([buf[a:].data_ptr() for a in at]),
        _lib.ptr_array([f.data_ptr() for f in F]), torch.cuda.current_stream().cuda_stream), entry)
    for p in range(3):
        assert torch.equal(F[p], want[p]), p


@pytest.mark.parametrize("e", [-100, -60, 60, 100])
def test_unit_of_length(e):
    """The same problem in a unit of length of 2^e micrometres, its source scaled with
    the operator: the same field, to the rounding that scaling a mode on the way may
    change (tolerances as above)."""
    import torch
    from paper_1902_00090_amd import FdfdOp, eim_field
    inst = W.grating(1030, nx=65, ny=40, npml=7)
    u = 2.0 ** e
    op = FdfdOp(inst.eps, inst.omega / u, inst.dx * u, inst.npml)
    (F,) = eim_field([op], [torch.tensor(inst.b / (u * u), device="cuda")])
    want = eim.eim_instance(inst)
    tol = 2.0 ** -24 * np.abs(want) + 1e6 * inst.ny * 2.0 ** -53 * np.abs(want).max()
    assert (np.abs(F.cpu().numpy() - want) <= tol).all()


def test_core_at_the_edge_of_a_long_column():
    """A guiding core in the first rows and 2000 rows of cladding: below the eigenvalue
    the minors rise to the core and fall with the mode through the cladding, 0.3 in
    the exponent a row, until rounding brings the growing solution back."""
    import torch
    from paper_1902_00090_amd import FdfdOp, eim_field
    rng = np.random.default_rng(5)
    nx, ny = 17, 2050
    eps = (2.085 + 0.05 * rng.random((ny, nx))).astype(np.float32)
    eps[3:15] = 12.25
    inst = W.Instance(eps, W.random_complex(rng, nx * ny), nx, ny, 0.025, 1.30, 3)
    op = FdfdOp.from_instance(inst)
    (F,) = eim_field([op], [torch.tensor(inst.b, device="cuda")])
    want = eim.eim_instance(inst)
    tol = 2.0 ** -24 * np.abs(want) + 1e6 * ny * 2.0 ** -53 * np.abs(want).max()
    assert (np.abs(F.cpu().numpy() - want) <= tol).all()
