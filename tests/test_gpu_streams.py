"""The sizes from which kernels go past the caches: same values on both sides of each line, written where they belong and nowhere else."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd

from test_gpu_brick import shifted

pytestmark = pytest.mark.gpu


def tree(lmax, radius):
    return octfd.Tree.build(3, lmax, sd.seed_points("rand", 1), np.array([int(radius * sd.Q)] * (lmax - 3), dtype=np.uint32))


@pytest.mark.parametrize("by", [0, 1])
@pytest.mark.parametrize("nvar", [1, 15, 16, 17])
def test_zip_on_both_sides_of_8192_blocks(dev, nvar, by):
    t = tree(3, 0.0)
    assert t.n == 512
    g = torch.Generator(device=dev).manual_seed(nvar)
    padded = shifted(torch.randn((nvar, t.n, 14, 14, 14), generator=g, dtype=torch.float64, device=dev), by)
    room = torch.full((nvar * t.n * 512 + 4,), -7.5, dtype=torch.float64, device=dev)
    z = room[2 + by:2 + by + nvar * t.n * 512]
    t.zip(padded, z.view(nvar, t.n, 8, 8, 8))
    assert torch.equal(z.view(nvar, t.n, 8, 8, 8), padded[:, :, 3:11, 3:11, 3:11])
    assert (room[:2 + by] == -7.5).all() and (room[2 + by + z.numel():] == -7.5).all()


@pytest.mark.parametrize("kind,lmax,radius,above", [("DERIVS", 5, 0.11, False), ("DERIVS", 6, 0.07, True), ("WAVE", 5, 0.11, False), ("WAVE", 6, 0.07, True),
                                                    ("BURGERS", 6, 0.09, False), ("BURGERS", 6, 0.12, True)])
def test_padded_evaluation_on_both_sides_of_256_mib(dev, kind, lmax, radius, above):
    k = octfd.KINDS[kind]
    t = tree(lmax, radius)
    vi, vo = octfd.nvar_in(k), octfd.nvar_out(k)
    print(kind, t.n, "blocks", flush=True)
    assert ((vi + vo) * t.n * 2744 * 8 > 256 << 20) == above
    g = torch.Generator(device=dev).manual_seed(5)
    u = torch.randn((vi, t.n, 8, 8, 8), generator=g, dtype=torch.float64, device=dev)
    sigma = 0.0 if kind == "DERIVS" else 0.3
    want = torch.empty((vo, t.n, 8, 8, 8), dtype=torch.float64, device=dev)
    t.rhs_eval_zipped(k, u, want, sigma=sigma)
    padded = torch.empty((vi, t.n, 14, 14, 14), dtype=torch.float64, device=dev)
    t.unzip(u, padded)
    out = torch.full((vo, t.n, 14, 14, 14), -7.5, dtype=torch.float64, device=dev)
    t.rhs_eval(k, padded, out, sigma=sigma)
    inner = out[:, :, 3:11, 3:11, 3:11]
    assert torch.equal(inner, want)
    inner.fill_(-7.5)
    assert (out == -7.5).all()


@pytest.mark.parametrize("nvar", [8, 9])
@pytest.mark.parametrize("centred", [False, True])
def test_fill_of_a_large_input_is_that_of_its_variables(dev, nvar, centred):
    """8 and 9 variables of 9,213 blocks are more than 256 MiB, one is not"""
    t = tree(6, 0.12)
    assert t.n * 4096 <= 256 << 20 < nvar * t.n * 4096
    g = torch.Generator(device=dev).manual_seed(7)
    u = torch.randn((nvar, t.n, 8, 8, 8), generator=g, dtype=torch.float64, device=dev)
    unzip = t.unzip_centred if centred else t.unzip
    out = torch.empty((nvar, t.n, 14, 14, 14), dtype=torch.float64, device=dev)
    one = torch.empty((1, t.n, 14, 14, 14), dtype=torch.float64, device=dev)
    unzip(u, out)
    for v in range(nvar):
        unzip(u[v:v + 1].contiguous(), one)
        assert torch.equal(out[v], one[0]), v
