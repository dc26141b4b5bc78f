"""Weight gradients of convolutions leave their partial sums to one launch at the end of a pass; more of them than its list
holds are added up at once, as before."""
import pytest

import launches
import workloads
from paper_2509_03110_amd import lsam


def reduces(model):
    names = launches.names(model)
    return names.count("reduce_list_kernel"), sum(n.startswith("conv_wgrad_kernel<") for n in names), \
        sum(n.startswith("splitk_reduce_kernel<") for n in names)


@pytest.mark.parametrize("bf16", [0, 1])
def test_one_launch_a_pass(bf16):
    model = dict(K=2, dims=(3, 32, 32, 48, 10), batch=64, n_conv=3, img_h=16, img_w=16, bn_mask=7, global_avg_pool=1, gemm_dtype=bf16)
    assert reduces(model) == (2, 4, 0)


def blocks(n, channels=16, batch=64):
    """A first layer and n blocks of two convolutions, each closed by a projection: 3 n weight gradients above the first layer's."""
    convs = 2 * n + 1
    closing = sum(1 << l for l in range(2, convs, 2))
    return dict(K=1, dims=(3,) + (channels,) * convs + (10,), batch=batch, n_conv=convs, img_h=16, img_w=16,
                bn_mask=(1 << convs) - 1, skip_mask=closing, proj_mask=closing, global_avg_pool=1)


def test_more_than_the_list_holds():
    lists, _, others = reduces(blocks(19))
    assert lists == 2 and others == 2 * (3 * 19 - 40)


@pytest.mark.parametrize("K,channels,batch,side,bf16,listed", [
    (2, 112, 40, (28, 20), 1, False),      # 28 MiB a layer
    (2, 304, 18, (12, 12), 0, False),      # 19 MiB, 1624 workgroups
    (4, 64, 128, (8, 8), 0, True),         # 18 MiB, 144 workgroups
    (4, 144, 8, (16, 4), 0, True)])        # 6 MiB
def test_large_partial_sums_are_added_up_at_once(K, channels, batch, side, bf16, listed):
    model = dict(K=K, dims=(5, channels, channels, channels, 10), batch=batch, n_conv=3, img_h=side[0], img_w=side[1], bn_mask=7,
                 global_avg_pool=1, gemm_dtype=bf16)
    assert reduces(model)[0] == (2 if listed else 0)


def test_only_listed_products_have_a_place_of_their_own():
    """A block of three listed products takes their partial sums' room beside everything else; one past the list does not.
    (64 pieces of 64 x 576 sums for each 3x3 layer of 64 channels.)"""
    def room(n):
        return lsam.lsam_workspace_bytes(lsam.config_from_workload(workloads.Workload("p", tau=(1,), **blocks(n, 64)))[0])
    assert room(6) - room(5) >= room(19) - room(18) + 2 * 64 * 64 * 576 * 4
