"""Weight gradients of convolutions leave their partial sums to one launch at the end of a pass; more of them than its list
holds are added up at once, as before."""
import pytest

import launches


def reduces(model):
    names = launches.names(model)
    return names.count("reduce_list_kernel"), sum(n.startswith("conv_wgrad_kernel<") for n in names), \
        sum(n.startswith("splitk_reduce_kernel<") for n in names)


@pytest.mark.parametrize("bf16", [0, 1])
def test_one_launch_a_pass(bf16):
    model = dict(K=2, dims=(3, 32, 32, 48, 10), batch=64, n_conv=3, img_h=16, img_w=16, bn_mask=7, global_avg_pool=1, gemm_dtype=bf16)
    assert reduces(model) == (2, 4, 0)


def test_more_than_the_list_holds():
    """39 convolutions of 16 channels in 19 blocks, each closed by a projection: 57 weight gradients above the first layer's."""
    closing = sum(1 << l for l in range(2, 39, 2))
    model = dict(K=1, dims=(3,) + (16,) * 39 + (10,), batch=64, n_conv=39, img_h=16, img_w=16, bn_mask=(1 << 39) - 1,
                 skip_mask=closing, proj_mask=closing, global_avg_pool=1)
    lists, _, others = reduces(model)
    assert lists == 2 and others == 2 * (38 + 19 - 40)
