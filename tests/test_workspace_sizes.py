"""Workspace a context asks for: programs size their memory and their
checkpoint plans by it, so that it must not grow."""
import pytest

from paper_2306_15678_amd.march import checkpoint_plan, make_desc, workspace_bytes


def _beams(n, count=1, n_screens=0):
    return [make_desc(n, 0.06, 0.1, wavelength=8e-7, n2=3.2e-23, terms=31 if n_screens else 15,
                      mpa_order=8, beta_k=1.6e-122, cn2=1e-14, screen_dz=1.0,
                      n_screens=n_screens, seed=1)] * count


BATCHES = {str(n): _beams(n) for n in (128, 256, 512, 768, 1024, 2048, 4096)}
BATCHES.update({"1024s3": _beams(1024, n_screens=3), "4096s3": _beams(4096, n_screens=3),
                "20x256": _beams(256, 20), "64x1024": _beams(1024, 64),
                "64mix": [b for n in (256, 512, 768, 1024) for b in _beams(n, n_screens=20)] * 16,
                "1000x128": _beams(128, 1000)})

# bytes that held each batch while the power partials were one per workgroup:
# complex64, then complex128, for (max_steps, ckpt_every, stored_segments) of
RECORDS = ((0, 1, 0), (100, 100, 0), (500, 23, 2))
BYTES = {
    "128": (630784, 13868288, 15179008, 899072, 27374848, 29996288),
    "256": (2245888, 55198208, 60441088, 3306752, 109212160, 119697920),
    "512": (9099520, 220911104, 241882624, 13318400, 436942336, 478885376),
    "768": (19263744, 495840768, 543026688, 28737792, 981892608, 1076264448),
    "1024": (34898176, 882146816, 966032896, 51724544, 1746222592, 1913994752),
    "2048": (136823040, 3525819904, 3861364224, 204030208, 6982024704, 7653113344),
    "4096": (541999360, 14097989120, 15440166400, 810631424, 27922611712, 30606966272),
    "1024s3": (47615744, 894864384, 978750464, 77025024, 1771523072, 1939295232),
    "4096s3": (743853824, 14299843584, 15642020864, 1213812480, 28325792768, 31010147328),
    "20x256": (24617472, 1083678464, 1188536064, 45795840, 2163918592, 2373633792),
    "64x1024": (1174494720, 55398456064, 60767165184, 2250866176, 110698789632, 121436207872),
    "64mix": (3084678656, 28502160128, 31018742528, 6106236416, 56941200128, 61974364928),
    "1000x128": (351143168, 13589414400, 14900134400, 618408192, 27094951424, 29716391424),
}


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("name", BYTES)
def test_workspace_does_not_grow(name, precision):
    for k, record in enumerate(RECORDS):
        held = BYTES[name][k + (3 if precision == 64 else 0)]
        assert workspace_bytes(BATCHES[name], precision, *record) <= held, record


@pytest.mark.parametrize("name", ["256", "4096", "64x1024"])
def test_budgets_hold_their_plans(name):
    """A budget that held all of a march's fields still does."""
    assert checkpoint_plan(BATCHES[name], 32, 100, BYTES[name][1]) == (100, 0, 0)
