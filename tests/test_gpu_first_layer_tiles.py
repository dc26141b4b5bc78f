"""First convolution layers whose workgroups take several tiles of 32 pixels a wavefront, the last ones ragged, on image rows
that do and do not hold whole runs of 8 pixels, and whose output gradient is formed where the weight gradient reads it or,
where a shortcut hands it on, by the normalisation; held to the oracle's groups as the other convolutions are."""
import pytest

torch = pytest.importorskip("torch")
import test_gpu_plane_products as planes  # noqa: E402

pytestmark = pytest.mark.gpu

NETS = {
    "four tiles, rows of 36": dict(dims=(3, 8, 10), side=(30, 36), batch=245),
    "two tiles, rows of 40": dict(dims=(2, 40, 10), side=(27, 40), batch=121),
    "one tile, rows of 6": dict(dims=(1, 64, 10), side=(11, 6), batch=31),
    "a shortcut's sum": dict(dims=(3, 32, 32, 32, 10), side=(16, 16), batch=33, skip=0b100, preact=1),
    "a shortcut's input": dict(dims=(3, 32, 32, 32, 10), side=(16, 24), batch=23, skip=0b100),
}


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_against_the_oracle(name, bf16, monkeypatch):
    monkeypatch.setitem(planes.NETS, name, NETS[name])
    planes.test_plane_products_match_oracle(name, bf16)
