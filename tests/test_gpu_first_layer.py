"""First convolution layers of 1 to 3 channels with output channels that do not fill a block of 32, on few and
on many pixels (64 to 512 of them a workgroup, ragged last ones), in both arithmetic modes, with and
without normalisation, held to the oracle's groups as the other convolutions are."""
import pytest

torch = pytest.importorskip("torch")
import test_gpu_plane_products as planes  # noqa: E402

pytestmark = pytest.mark.gpu

NETS = {
    "3 to 16": dict(dims=(3, 16, 8, 10), side=(8, 8), batch=5),
    "1 to 24, ragged": dict(dims=(1, 24, 16, 10), side=(7, 9), batch=13),
    "2 to 40": dict(dims=(2, 40, 10), side=(16, 16), batch=17),
    "3 to 72, pool": dict(dims=(3, 72, 16, 10), side=(16, 32), batch=9, pool=0b01),
    "3 to 104, no normalisation": dict(dims=(3, 104, 10), side=(12, 12), batch=7, bn=0),
    "1 to 248": dict(dims=(1, 248, 10), side=(8, 8), batch=9),
    "3 to 64, many pixels": dict(dims=(3, 64, 8, 10), side=(32, 32), batch=70),
    "3 to 8, many pixels": dict(dims=(3, 8, 8, 10), side=(32, 32), batch=131),
}


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_against_the_oracle(name, bf16, monkeypatch):
    monkeypatch.setitem(planes.NETS, name, NETS[name])
    planes.test_plane_products_match_oracle(name, bf16)
