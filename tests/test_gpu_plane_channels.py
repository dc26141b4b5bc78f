"""Convolutions of any multiple of 8 channels on plane tensors by address: k-steps that cross taps at every
unit, channel blocks of the weight-gradient patches that are not full, filters whose classes of a stride-2
input gradient begin inside a k-step, projections; both arithmetic modes, held to the oracle's groups as
the multiples of 32 are."""
import pytest

torch = pytest.importorskip("torch")
import test_gpu_plane_products as planes  # noqa: E402

pytestmark = pytest.mark.gpu

NETS = {
    "24 and 40": dict(dims=(3, 24, 40, 24, 10), side=(32, 32), batch=16),
    "72 and 8": dict(dims=(8, 72, 8, 72, 10), side=(16, 32), batch=33),
    "56 and 104, ragged": dict(dims=(16, 56, 104, 10), side=(9, 11), batch=43),
    "48, stride and projection": dict(dims=(3, 24, 48, 48, 10), side=(32, 32), batch=16, stride=0b010, skip=0b100, proj=0b100),
    "40, stride and parameter-free shortcut": dict(dims=(3, 40, 80, 80, 10), side=(16, 16), batch=33, stride=0b010, skip=0b100),
    "24, pre-activation": dict(dims=(3, 24, 48, 48, 48, 48, 10), side=(16, 32), batch=17, stride=0b00010, skip=0b10100,
                               proj=0b00100, preact=1),
    "48 and 80, patches": dict(dims=(3, 48, 80, 48, 10), side=(16, 16), batch=40),
    "152, few pixels": dict(dims=(8, 152, 88, 10), side=(4, 4), batch=131),
    # stride 2, three planes: dX in classes with a column tile of 8 and one of 64, and (136) through a stored gradient
    "72, stride in classes": dict(dims=(3, 72, 104, 10), side=(32, 32), batch=33, stride=0b010),
    # (its second stride, on 2240 pixels, goes to the fp32-storage product)
    "128, stride in classes": dict(dims=(8, 128, 160, 64, 10), side=(16, 32), batch=35, stride=0b0110),
    "160, stride in classes": dict(dims=(8, 160, 64, 10), side=(16, 16), batch=90, stride=0b010),
    "104 to 320 on few pixels, stride through a stored gradient": dict(dims=(8, 104, 320, 10), side=(16, 16), batch=16, stride=0b010),
    "136, stride through a stored gradient": dict(dims=(8, 136, 64, 10), side=(16, 16), batch=90, stride=0b010),
    # last columns on half tiles of the three-plane patches: of 256 and (64 wide) of 128 pixels; 160 between one and two rounds
    "96 and 160, last columns on half tiles": dict(dims=(3, 96, 160, 80, 10), side=(16, 16), batch=23),
    "80 and 96, 64 wide": dict(dims=(3, 32, 80, 96, 10), side=(8, 64), batch=9),
    "160, whole tiles": dict(dims=(3, 32, 160, 10), side=(16, 16), batch=100),
    "88, pools": dict(dims=(3, 88, 56, 10), side=(16, 16), batch=33, pool=0b011),
}


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("name", sorted(NETS))
def test_against_the_oracle(name, bf16, monkeypatch):
    monkeypatch.setitem(planes.NETS, name, NETS[name])
    planes.test_plane_products_match_oracle(name, bf16)


def test_tall_images(monkeypatch):
    """192000 pixels in images of 16000 rows: the weight gradient's patches divide numbers whose product with the divisor
    is past 2^32."""
    monkeypatch.setitem(planes.NETS, "tall", dict(dims=(3, 32, 32, 10), side=(16000, 4), batch=3, K=1))
    planes.test_plane_products_match_oracle("tall", 0)
