"""GPU checks of the row rotation's split products where their forms meet: result rows
that allow no 16-byte stores, few rows, and components too small to be split exactly
in every product."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08734_amd import api as a
    a.lib()
    return a


def rotate(api, x, rot):
    return api.rotate_rows(torch.from_numpy(x).cuda(), torch.from_numpy(rot).cuda()).cpu().numpy()


def worst(out, x, rot):
    """Largest |out - exact| / sum |rot x| (0 where that is 0)."""
    x, rot = x.astype(np.float64), rot.astype(np.float64)
    mag = np.abs(x) @ np.abs(rot).T
    return (np.abs(out.astype(np.float64) - x @ rot.T) / np.where(mag > 0, mag, 1.0)).max()


# result rows in quads, in columns and in blocks; tiles and rows with remainders; rows
# that fill the chip and rows whose outputs are shared out
@pytest.mark.parametrize("n,d,dout", [
    (65_535, 64, 57), (65_536, 64, 57), (65_551, 33, 63), (70_007, 24, 17), (66_000, 32, 1),
    (100_003, 48, 41), (16_384, 128, 121), (16_391, 100, 77), (66_001, 64, 65), (65_600, 30, 64),
    (16_400, 128, 128), (131_075, 96, 24), (20_000, 128, 500), (20_000, 40, 333)])
def test_rotate_forms(api, n, d, dout):
    print(f"rotate n={n} d={d} dout={dout}", flush=True)
    rng = np.random.default_rng(n + d + dout)
    x = (rng.standard_normal((n, d)) * np.exp(3 * rng.standard_normal((n, 1)))).astype(np.float32)
    rot = rng.standard_normal((dout, d)).astype(np.float32)
    assert worst(rotate(api, x, rot), x, rot) <= (d + 2) * 2.0 ** -24  # of an FP32 sum


# small components in rot, in rows, in both (their products the smallest numbers that
# are held exactly, and below), in outputs that consist of them alone
@pytest.mark.parametrize("d,dout", [(128, 128), (64, 57), (48, 30), (31, 16)])
@pytest.mark.parametrize("in_rot,in_x", [(1e-17, 1.0), (1.0, 1e-17), (1e-12, 1e-19), (1e-17, 1e-17),
                                         (1e-31, 1.0), (1.0, 1e-33), (1e-38, 1.0)])
def test_rotate_small_components(api, d, dout, in_rot, in_x):
    print(f"rotate small d={d} dout={dout} {in_rot} {in_x}", flush=True)
    rng = np.random.default_rng(d)
    n = 66_000
    x = rng.standard_normal((n, d)).astype(np.float32)
    rot = rng.standard_normal((dout, d)).astype(np.float32)
    x[::40, 3] *= np.float32(in_x)
    x[7, :] *= np.float32(in_x)
    rot[1, 5] *= np.float32(in_rot)
    rot[dout - 1] = 0.0
    rot[dout - 1, 3] = np.float32(in_rot)  # this output is a small component alone
    out = rotate(api, x, rot)
    exact = x.astype(np.float64) @ rot.astype(np.float64).T
    mag = np.abs(x).astype(np.float64) @ np.abs(rot).astype(np.float64).T
    # (products below 2^-100 may lose 2^-126 each: FP32's smallest normal number)
    assert (np.abs(out - exact) <= (d + 2) * 2.0 ** -24 * mag + d * 2.0 ** -126).all()
