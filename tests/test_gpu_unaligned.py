"""Buffers at any sample-aligned address, with any pitch and plane stride,
give the coefficients and images of contiguous buffers bit for bit, and images
smaller than a border tile's reach match the oracle.

The tile kernel's vector accesses carry the alignment of one sample, so a
call's route does not depend on alignment; sizes below put rows and columns at
the ends of tiles (256 / 512 pixels wide, 24 ... 56 high) and one block
either side of them.
"""
import ctypes

import numpy as np
import pytest

import workloads
from oracle import lifting

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402

TILE_CONFIGS = range(5)
TOL = 1e-5                     # FP32, of the largest coefficient (as the parity tests)


def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def strided(x, off, pitch, gap):
    """x [n, h, w] copied to a buffer that starts `off` elements into an
    allocation, with that row pitch and `gap` elements between planes."""
    n, h, w = x.shape
    ps = (h - 1) * pitch + w + gap
    buf = torch.zeros(off + n * ps + pitch, dtype=x.dtype, device=x.device)
    v = buf[off:].as_strided(x.shape, (ps, pitch, 1))
    v.copy_(x)
    return v


def call(name, src, dst, wavelet, levels, flags):
    n, h, w = src.shape
    dt = d.dtype_code(src)
    ws = d.workspace(h, w, levels, dt, dev(), n)
    st = getattr(d.lib(), name)(src.data_ptr(), dst.data_ptr(), n, src.stride(0), dst.stride(0), h, w,
                                src.stride(1), dst.stride(1), dt, d.WAVELETS[wavelet], levels, 0, flags,
                                ws.data_ptr() if ws is not None else None, ws.numel() if ws is not None else 0,
                                torch.cuda.current_stream().cuda_stream)
    assert st == 0, st


@pytest.mark.parametrize("wavelet,tdt", [("cdf97", torch.float32), ("cdf97", torch.bfloat16),
                                         ("cdf97", torch.float16), ("cdf53", torch.int32), ("dd137", torch.float32),
                                         ("dd137", torch.bfloat16)])
@pytest.mark.parametrize("h,w,levels", [(61, 1037, 1), (128, 1030, 2), (50, 258, 3)])
def test_any_alignment_bit_identical(wavelet, tdt, h, w, levels):
    n = 2
    x = torch.from_numpy(workloads.planes(n, h, w, seed=81)).to(dev())
    x = (x * 255).round().to(tdt) if tdt == torch.int32 else x.to(tdt)
    names = ["dwt2_fwd_planes", "dwt2_inv_planes"] + (["dwt2_adj_planes"] if wavelet == "cdf97" else [])
    for cfg in TILE_CONFIGS if wavelet != "dd137" else [None]:
        flags = 0 if cfg is None else d.DWT2_FLAG_KERNEL(cfg)
        for name in names:
            ref = torch.empty_like(x)
            call(name, x, ref, wavelet, levels, flags)
            for off, ps, pd, gap in ((1, w, w, 0), (3, w + 1, w + 3, 5), (0, w + 2, w + 1, 2)):
                print("alignment", wavelet, tdt, (h, w), levels, cfg, name, off, ps, pd, gap, flush=True)
                src = strided(x, off, ps, gap)
                dst = strided(torch.zeros_like(x), off + 2, pd, gap + 1)
                call(name, src, dst, wavelet, levels, flags)
                assert torch.equal(dst, ref), (cfg, name, off, ps, pd, gap)


@pytest.mark.parametrize("h", [2, 3, 4, 5, 7, 8, 9])
def test_images_smaller_than_a_tiles_reach(h):
    """Heights and widths around the reach of a border tile (positions up to
    5 samples past an end, folded four times for a side of 2)."""
    for w in (2, 3, 5, 6, 7, 8, 9, 255, 257, 259):
        x = workloads.uniform(h, w, seed=h * 100 + w)
        xi = workloads.pixels_u8(h, w, seed=h * 100 + w)
        lv = lifting.max_levels(h, w)
        print("small", (h, w), lv, flush=True)
        for cfg in TILE_CONFIGS:
            for wav in ("cdf97", "cdf53f"):
                ref = lifting.fwd(x, wav, lv)
                y = d.fwd(torch.from_numpy(x).to(dev()), wav, lv, config=cfg)
                assert np.abs(y.cpu().numpy() - ref).max() <= TOL * np.abs(ref).max(), (wav, cfg, w)
                c = ref.astype(np.float32)
                r = d.inv(torch.from_numpy(c).to(dev()), wav, lv, config=cfg).cpu().numpy()
                want = lifting.inv(c, wav, lv)
                assert np.abs(r - want).max() <= TOL * np.abs(want).max(), (wav, cfg, w)
            yi = d.fwd(torch.from_numpy(xi).to(dev()), "cdf53", lv, config=cfg)
            assert np.array_equal(yi.cpu().numpy(), lifting.fwd(xi, "cdf53", lv)), (cfg, w)
            assert np.array_equal(d.inv(yi, "cdf53", lv, config=cfg).cpu().numpy(), xi), (cfg, w)
