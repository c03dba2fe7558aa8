"""dlma_apply_dw on fields that overlap in part: the numbers of separate fields, in place refused."""
import ctypes

import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dims,n", [((4, 2, 4, 6), 3), ((8, 4, 8, 8), 10)])  # four lanes per site, 64 sites per wave
@pytest.mark.parametrize("shift", [7, -7, 12 * 192, -12 * 192])  # complex numbers from in to out
def test_partial_overlap(dims, n, shift):
    from paper_2201_09729_amd import dlma as D
    print("overlap", dims, n, shift, flush=True)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.3, 4)).cuda(), 0.121, 1.2)
    x = torch.from_numpy(synth.random_spinor(dims, n, 8)).cuda()
    ref = D.dlma_apply_dw(g, x).view(-1)
    m, s = x.numel(), abs(shift)
    buf = torch.zeros(m + s, dtype=torch.complex128, device="cuda")
    i, o = (0, s) if shift > 0 else (s, 0)
    buf[i:i + m] = x.view(-1)
    lib = D.load_library()
    p = lambda k: ctypes.c_void_p(buf.data_ptr() + 16 * k)  # noqa: E731
    assert lib.dlma_apply_dw(g.h, p(i), p(o), n, 0, D._stream()) == D.DLMA_OK
    assert torch.equal(buf[o:o + m], ref)
    assert lib.dlma_apply_dw(g.h, p(i), p(i), n, 0, D._stream()) == D.DLMA_EINVAL
