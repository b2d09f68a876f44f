"""The Python list forms of profile fit and mass placement refuse tensors of another type,
shape, layout or place than the library reads, before any pointer is handed on."""
import pytest

torch = pytest.importorskip("torch")
from paper_1211_6932_amd import lbmp as B  # noqa: E402

PLACE = (32.0, 32.0, 10.0)


def fit_args(**kw):
    a = dict(rhos=[torch.ones(64, 64)] * 2, places=[PLACE] * 2, out=torch.zeros(2, 128),
             scratch=torch.zeros(2 * B.lbml_profile_scratch_bytes(64), dtype=torch.uint8))
    a.update(kw)
    return a


@pytest.mark.parametrize("bad,match", [
    (dict(out=torch.zeros(2, 128, dtype=torch.float64)), "out"), (dict(out=torch.zeros(3, 128)), "out"),
    (dict(out=torch.zeros(2, 127)), "out"), (dict(places=[PLACE]), "places"), (dict(), "GPU")])
def test_fits(bad, match):
    with pytest.raises(ValueError, match=match):
        B.profiles_extract(**fit_args(**bad))


@pytest.mark.parametrize("logrho,match", [
    (torch.zeros(2, 64), "logrho"), (torch.zeros(2, 256), "logrho"), (torch.zeros(2, 128, dtype=torch.float64), "logrho"),
    (torch.zeros(2, 128, dtype=torch.bfloat16), "logrho"), (torch.zeros(128), "logrho"), (torch.zeros(2, 128), "GPU")])
def test_placements(logrho, match):
    with pytest.raises(ValueError, match=match):
        B.profiles_to_rho0_mass(logrho, [(10.0, 32.0, 32.0, 64, 64, 100.0)] * 2)


@pytest.mark.gpu
def test_on_the_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    good = {k: [t.cuda() for t in v] if k == "rhos" else v.cuda() if torch.is_tensor(v) else v for k, v in fit_args().items()}
    for bad in (dict(rhos=[good["rhos"][0].double()] * 2), dict(rhos=[torch.ones(64, 64)] * 2),
                dict(rhos=[good["rhos"][0].t()[:, :60]] * 2), dict(scratch=good["scratch"][:-8]),
                dict(scratch=good["scratch"][::2]), dict(scratch=torch.zeros_like(good["scratch"], device="cpu"))):
        with pytest.raises(ValueError):
            B.profiles_extract(**{**good, **bad})
    print("[gpu-case] list wrappers", flush=True)
    assert B.profiles_extract(**good) is good["out"]
    wide = torch.zeros(2, 256, device="cuda")[:, :128]  # rows of a wider tensor
    fields, shifts = B.profiles_to_rho0_mass(wide - 2.0, [(10.0, 32.0, 32.0, 64, 64, 100.0)] * 2)
    assert len(fields) == 2 and shifts.shape == (2, 2)
    assert B.profiles_to_rho0_mass(wide[:0], [])[0] == []
    torch.cuda.synchronize()
