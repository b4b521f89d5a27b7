"""Two levels in one launch, and the last three of small images (calls that name
no scheme and no kernel configuration), against one launch per level
(configuration 0): bit for bit the same, for every wavelet, storage type and
direction, at the ends of their tiles (224 pixels wide, 40 or 72 high; three
levels 192 wide, 32 high), on the smallest images, over odd pitches and plane
strides, and with an odd and an even number of levels."""
import pytest

import workloads
from oracle import lifting

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402

TYPES = [("cdf97", torch.float32), ("cdf97", torch.bfloat16), ("cdf97", torch.float16), ("cdf53", torch.int32),
         ("cdf53f", torch.float32), ("cdf53f", torch.bfloat16), ("cdf53f", torch.float16)]


def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def image(n, h, w, tdt, seed):
    x = torch.from_numpy(workloads.planes(n, h, w, seed=seed)).to(dev())
    return (x * 255).round().to(tdt) if tdt == torch.int32 else x.to(tdt)


def check(x, wavelet, levels):
    print("pair", wavelet, x.dtype, tuple(x.shape), levels, flush=True)
    y = d.fwd(x, wavelet, levels, config=0)
    assert torch.equal(d.fwd(x, wavelet, levels), y)
    assert torch.equal(d.inv(y, wavelet, levels), d.inv(y, wavelet, levels, config=0))
    if wavelet == "cdf97":
        assert torch.equal(d.adj(y, levels), d.adj(y, levels, config=0))


@pytest.mark.parametrize("wavelet,tdt", TYPES)
def test_tile_ends(wavelet, tdt):
    for n, h, w, levels in ((1, 39, 223, 2), (1, 40, 224, 3), (2, 41, 225, 2), (1, 44, 226, 4), (1, 81, 449, 2),
                            (3, 83, 460, 5), (1, 120, 672, 3), (1, 200, 1000, 4), (1, 31, 191, 3), (2, 32, 192, 3),
                            (1, 33, 193, 3), (1, 64, 384, 3), (3, 66, 387, 3), (40, 96, 200, 3)):
        check(image(n, h, w, tdt, 101), wavelet, levels)


@pytest.mark.parametrize("wavelet,tdt", TYPES)
def test_small_images(wavelet, tdt):
    for h in (3, 4, 5, 7, 8, 9, 14):
        for w in (3, 4, 6, 7, 9, 15, 225):
            check(image(1, h, w, tdt, 102), wavelet, lifting.max_levels(h, w))


@pytest.mark.parametrize("wavelet,tdt", TYPES[:4])
@pytest.mark.parametrize("n,h,w,levels", [(3, 1079, 2017, 3), (3, 1080, 2016, 2), (3, 1083, 2050, 5),
                                          (1, 4099, 8201, 3), (1, 8192, 4096, 2)])
def test_larger_levels(wavelet, tdt, n, h, w, levels):
    check(image(n, h, w, tdt, 103), wavelet, levels)


@pytest.mark.parametrize("wavelet,tdt", TYPES[:4])
@pytest.mark.parametrize("levels", [3, 4])
def test_strides(wavelet, tdt, levels):
    """Raw calls with offset buffers, odd pitches and gaps between planes."""
    n, h, w = 3, 85, 451
    x = image(n, h, w, tdt, 104)
    dt = d.dtype_code(x)
    ws = d.workspace(h, w, levels, dt, dev(), n)

    def strided(v, off, pitch, gap):
        ps = (h - 1) * pitch + w + gap
        buf = torch.zeros(off + n * ps + pitch, dtype=v.dtype, device=dev())
        s = buf[off:].as_strided(v.shape, (ps, pitch, 1))
        s.copy_(v)
        return s

    names = ["dwt2_fwd_planes", "dwt2_inv_planes"] + (["dwt2_adj_planes"] if wavelet == "cdf97" else [])
    ref = d.fwd(x, wavelet, levels, config=0)
    want = {"dwt2_fwd_planes": (x, ref), "dwt2_inv_planes": (ref, d.inv(ref, wavelet, levels, config=0))}
    if wavelet == "cdf97":
        want["dwt2_adj_planes"] = (ref, d.adj(ref, levels, config=0))
    for name in names:
        src0, out = want[name]
        src, dst = strided(src0, 3, w + 2, 5), strided(torch.zeros_like(x), 1, w + 1, 2)
        st = getattr(d.lib(), name)(src.data_ptr(), dst.data_ptr(), n, src.stride(0), dst.stride(0), h, w,
                                    src.stride(1), dst.stride(1), dt, d.WAVELETS[wavelet], levels, 0, 0,
                                    ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert st == 0, st
        assert torch.equal(dst, out), name


@pytest.mark.parametrize("wavelet,tdt", TYPES)
@pytest.mark.parametrize("n,h,w", [(130, 63, 190), (130, 64, 192), (64, 66, 193), (86, 65, 194), (1, 1501, 1499)])
def test_three_levels_tall_tiles(wavelet, tdt, n, h, w):
    """Three levels in tiles 64 high: more than 256 of the tiles 32 high, at
    most 256 (forward 384) of these."""
    check(image(n, h, w, tdt, 105), wavelet, 3)
