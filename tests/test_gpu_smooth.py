"""GPU parity on images without noise: few levels, long runs, large zones and
many equal neighbours, where the counting of the map kernels takes other
paths than in noise (lists of runs that fill up, equal pairs counted
together, dependences of every size)."""
import numpy as np
import pytest

from helpers import format_report, parity_report, to_dev
from oracle import oracle as O
from paper_2609_19190_amd import synth

pytestmark = pytest.mark.gpu
ALL = 63


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_19190_amd import binding
    binding.lib()
    return binding


def image(kind, shape):
    rng = np.random.default_rng(7)
    z, y, x = np.indices(shape)
    return {
        "constant": lambda: np.full(shape, 3),
        "rare": lambda: (rng.random(shape) < 0.02) * 5,
        "halves": lambda: (x >= shape[2] // 2) * 2,
        "blocks": lambda: x // 4 + 2 * (y // 5) + 5 * (z // 3),
        "stripes": lambda: (x + y) % 2,
        "binary": lambda: rng.random(shape) < 0.5,
        "gradient": lambda: x + 2 * y + 3 * z,
        "three": lambda: rng.integers(0, 3, shape),
        "ten": lambda: rng.integers(0, 10, shape),
        "mostly": lambda: np.where(rng.random(shape) < 0.7, 4, rng.integers(0, 40, shape)),
    }[kind]().astype(np.int16)


@pytest.mark.parametrize("radius", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("kind", ["constant", "rare", "halves", "blocks", "stripes", "binary", "gradient", "three", "ten",
                                  "mostly"])
@pytest.mark.parametrize("fill", [1.0, 0.9])
def test_smooth_images_against_the_oracle(B, kind, radius, fill):
    shape = (9, 12, 13) if radius < 4 else (9, 10, 11)
    vol = image(kind, shape)
    mask = (np.random.default_rng(3).random(shape) < fill).astype(np.uint8)
    mask[0, 0, 0] = 1
    case = synth.Case(kind, vol, mask, (1.0, 1.0, 2.0), O.FBW, 1.0, float("nan"), radius, ALL)
    v, m = to_dev(case)
    variants = [{}, dict(gldm_alpha=1), dict(glcm_distance=2, gldm_alpha=2)]
    if radius in (2, 3):
        variants.append(dict(averaged=True))
    for o in variants:
        opt = B.map_options(o.get("glcm_distance", 1), o.get("gldm_alpha", 0),
                            B.FR_AVERAGED if o.get("averaged") else B.FR_MERGED) if o else None
        gpu = B.fr_map(v, m, case.spacing, case.mode, case.value, case.lower, radius, ALL, case.n_mask, options=opt)
        B.fr_map_check()
        ok, rows = parity_report(gpu.cpu().numpy(), O.spatial_map(case, **o), O.map_names(ALL))
        assert ok, f"{o}\n" + format_report(rows, only_bad=True)
