"""DD 13/7 on the four-tap register tile kernels (calls that name no kernel
configuration and no scheme): the fused steps bit for bit the LDS-plane kernel's
results, whose parity with the oracle tests/test_gpu_lds.py holds, at the ends of
the kernels' tiles, for every storage type and direction; the factored ones (the
default of 16-bit storage) within an ulp of them; several levels bit for bit the
levels one by one; the smallest images against the oracle itself."""
import numpy as np
import pytest

import workloads
from oracle import lifting

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402

TOL = 1e-5                     # FP32, of the largest coefficient (as the LDS-plane kernel's tests)
LDS_CONFIG = 8


def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def one_by_one(direction, x, levels):
    """The transform of several levels as one call for each."""
    sizes = [x.shape[-2:]]
    for _ in range(levels - 1):
        sizes.append(tuple((n + 1) // 2 for n in sizes[-1]))
    y = x.clone()
    for h, w in sizes if direction is d.fwd else sizes[::-1]:
        y[..., :h, :w] = direction(y[..., :h, :w].contiguous(), "dd137", 1)
    return y


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("h,w,levels", [(20, 240, 1), (21, 241, 1), (27, 247, 2), (58, 486, 1), (111, 495, 2),
                                        (104, 480, 3), (200, 1000, 5), (2900, 2050, 2), (1, 1, 0)])
def test_equals_lds_plane_kernel(tdt, h, w, levels):
    # tiles are 240 pixels wide and 20 high, or 28 beyond 1024 tiles (2900 x 2050)
    if levels == 0:            # one image with interior tiles, ragged ends, and every plane of a stack
        n, h, w, levels = 3, 333, 1211, 4
    else:
        n = 1
    x = torch.from_numpy(workloads.planes(n, h, w, seed=91)).to(dev()).to(tdt)
    for direction in (d.fwd, d.inv):
        print("taps4", tdt, (n, h, w), levels, direction.__name__, flush=True)
        fused = direction(x, "dd137", levels, fused=True)
        assert torch.equal(fused, direction(x, "dd137", levels, config=LDS_CONFIG))
        if tdt == torch.float32:
            assert torch.equal(direction(x, "dd137", levels), fused)
            continue
        # one level: the same FP32 value up to its own rounding (1e-6 of the
        # largest), rounded once: neighbours in the storage type at most
        y, z = direction(x, "dd137", 1).float(), direction(x, "dd137", 1, fused=True).float()
        ulp = 2.0 ** (-7 if tdt == torch.bfloat16 else -10)
        assert bool(((y - z).abs() <= ulp * z.abs() + 1e-6 * z.abs().max()).all())
        assert torch.equal(direction(x, "dd137", levels), one_by_one(direction, x, levels))


@pytest.mark.parametrize("h", [2, 3, 4, 6, 7, 8, 9])
def test_small_images(h):
    for w in (2, 3, 5, 7, 8, 11, 241):
        x = workloads.uniform(h, w, seed=h * 300 + w)
        lv = lifting.max_levels(h, w)
        print("taps4 small", (h, w), lv, flush=True)
        ref = lifting.fwd(x, "dd137", lv)
        y = d.fwd(torch.from_numpy(x).to(dev()), "dd137", lv).cpu().numpy()
        assert np.abs(y - ref).max() <= TOL * np.abs(ref).max(), w
        c = ref.astype(np.float32)
        want = lifting.inv(c, "dd137", lv)
        r = d.inv(torch.from_numpy(c).to(dev()), "dd137", lv).cpu().numpy()
        assert np.abs(r - want).max() <= TOL * np.abs(want).max(), w


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,h,w,levels", [(1, 55, 215, 2), (1, 56, 216, 2), (2, 57, 217, 3), (1, 112, 432, 2),
                                          (3, 115, 650, 4), (3, 7, 9, 2), (1, 2030, 2050, 3), (260, 88, 216, 2),
                                          (130, 88, 217, 2), (1, 2801, 2799, 2)])
def test_two_levels_in_one_launch(tdt, n, h, w, levels):
    # tiles of both levels are 216 pixels wide and 56 high; 88 (16-bit storage, forward) beyond 512 of those
    x = torch.from_numpy(workloads.planes(n, h, w, seed=92)).to(dev()).to(tdt)
    for direction in (d.fwd, d.inv):
        print("taps4 pair", tdt, (n, h, w), levels, direction.__name__, flush=True)
        assert torch.equal(direction(x, "dd137", levels), one_by_one(direction, x, levels))
