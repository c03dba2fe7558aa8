"""Block lengths of the BF16 tile kernels: long stencil blocks (with a shorter last strip, and
with short vector blocks beside them), long vector blocks with a remainder.

The operator sums nothing over sites, so the columns of a long-block call are, bit for bit,
those of calls of sixteen, whose blocks are short (which test_gpu_tiles.py holds against the
oracle).  Solves: the true residual in FP64."""
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_09729_amd import dlma
    return dlma


def setup(D, dims, n, seed):
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.25, 11)).cuda(), 0.120, 1.2)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return g, torch.randn((n,) + dims + (4, 3), dtype=torch.complex128, device="cuda", generator=gen)


# tile sites (per parity, times tiles) 22400, 71680, 68040, 23040; strips of 3 3 3 1, 3 3 3 1,
# 5 5 4 and, of one row longer than a block, 1 1
@pytest.mark.parametrize("dims,n", [((8, 4, 10, 28), 80), ((8, 8, 10, 28), 128), ((6, 6, 14, 18), 240), ((4, 4, 2, 120), 384)])
def test_long_blocks_give_the_numbers_of_short_ones(D, dims, n):
    print("tile blocks", dims, n, flush=True)
    g, x = setup(D, dims, n, 3)
    y = D.dlma_apply_schur(g, x, prec="mix_bf16")
    for i in range(0, n, 16):
        assert torch.equal(y[i:i + 16], D.dlma_apply_schur(g, x[i:i + 16], prec="mix_bf16")), i


@pytest.mark.parametrize("dims,n", [((8, 4, 10, 28), 80), ((6, 6, 14, 18), 240)])
def test_solves_with_long_blocks(D, dims, n):
    print("tile block solve", dims, n, flush=True)
    g, b = setup(D, dims, n, 4)
    (x,), st = D.dlma_solve([g], [b], opts=D.default_opts(tol=1e-10, prec="mix_bf16"))
    assert all(s["converged"] for s in st)
    r = (D.dlma_apply_dw(g, x) - b).reshape(n, -1)
    assert (torch.linalg.vector_norm(r, dim=1) / torch.linalg.vector_norm(b.reshape(n, -1), dim=1)).max().item() <= 1.001e-10
