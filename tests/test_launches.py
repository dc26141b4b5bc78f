"""What a step launches, seen without a GPU (launches.py)."""
import numpy as np
import pytest

import launches

# one process, in this order: every kernel that serves the dense gradients, the small tiles first
DENSE = [
    dict(K=2, dims=(784, 128, 10), batch=32),                                      # 64x64 tiles
    dict(K=4, dims=(3072, 1024, 1024, 10), batch=128),                             # 128x128
    dict(K=2, dims=(3, 8, 64, 10), batch=64, n_conv=1, img_h=16, img_w=16, gemm_dtype=1),      # rounded operands
    dict(K=8, dims=(3, 8, 640, 640, 10), batch=64, n_conv=1, img_h=16, img_w=16, gemm_dtype=1),
]


def test_kernels_with_much_lds_have_their_limit_raised():
    """A kernel that takes more than 64 KiB of dynamic LDS has to be allowed to, each kernel for itself, whatever
    ran before it in the process."""
    seen = set()
    for model, r in zip(DENSE, launches.record(*DENSE)):
        assert r["rc"] == 0, (model, r["error"])
        for l in r["launches"]:
            if l["name"].startswith("dense_gradients_kernel"):
                seen.add(l["name"])
            assert l["lds"] <= max(l["limit"], 64 << 10), (model, l)
    assert seen == {"dense_gradients_kernel<%d,2,%s>" % (t, r) for t in (64, 128) for r in ("false", "true")}


def test_long_batches_of_narrow_bf16_layers_are_accepted():
    """Four million rows of 32 columns, 256 MB an operand: within the 32-bit offsets of every product."""
    r = launches.record(dict(K=1, dims=(32, 32, 32), batch=4_000_000, gemm_dtype=1))[0]
    assert r["rc"] == 0, r["error"]


def dense_products(model):
    """(tile side of the first pass's launch of all gradients, its products, products of their own by name)"""
    got = [l for l in launches.record(model)[0]["launches"]]
    first = got[:next(i for i, l in enumerate(got) if l["name"].startswith("dense_gradients_kernel")) + 1]
    own = [l["name"] for l in first if l["name"].startswith("gemm_kernel<float,float") and ",false,false," in l["name"]]
    return int(first[-1]["name"].split("<")[1].split(",")[0]), own


@pytest.mark.parametrize("model,tile,own", [
    # long batches with few tiles are cut over workgroups, each product for itself
    (dict(K=1, dims=(784, 128, 10), batch=2048), 64, 2),
    (dict(K=1, dims=(784, 128, 10), batch=512), 64, 0),
    (dict(K=2, dims=(64, 64, 64, 10), batch=4096), 64, 3),
    (dict(K=8, dims=(256, 200, 100, 50), batch=4096), 64, 0),       # 208 tiles
    # a product too narrow for 128x128 tiles, where the others fill whole rounds of the compute units
    (dict(K=1, dims=(3072, 1024, 1024, 10), batch=1024), 128, 1),
    (dict(K=4, dims=(3072, 1024, 1024, 10), batch=1024), 128, 1),
    (dict(K=4, dims=(3072, 1024, 1024, 24), batch=512), 128, 1),
    (dict(K=4, dims=(3072, 1024, 1024, 24), batch=256), 128, 0),
    (dict(K=3, dims=(1000, 1500, 777, 37), batch=1024), 128, 0),
    # rounded operands
    (dict(K=1, dims=(3, 8, 64, 10), batch=4096, n_conv=1, img_h=16, img_w=16, gemm_dtype=1), 64, 2),
    (dict(K=8, dims=(3, 8, 640, 640, 10), batch=128, n_conv=1, img_h=16, img_w=16, gemm_dtype=1), 128, 0)])
def test_which_dense_gradients_share_a_launch(model, tile, own):
    got_tile, got_own = dense_products(model)
    assert got_tile == tile and len(got_own) == own, (got_tile, got_own)


@pytest.mark.parametrize("model,together", [
    (dict(K=3, dims=(1000, 1500, 777, 37), batch=100), True),
    (dict(K=1, dims=(3072, 4096, 1000), batch=1024), True), (dict(K=1, dims=(3072, 4096, 1000), batch=2048), False),
    (dict(K=4, dims=(3072, 1024, 1024, 10), batch=2048), True), (dict(K=4, dims=(3072, 1024, 1024, 10), batch=4096), False),
    (dict(K=1, dims=(2048,) * 5, batch=8192), False),
    (dict(K=16, dims=(512,) * 4, batch=8192), True),               # large work on layers of one group of tiles
    (dict(K=8, dims=(3072, 1024, 1024, 10), batch=64), False)])    # past the caches
def test_which_bf16_layers_step_together(model, together):
    names = launches.names(dict(model, gemm_dtype=1))
    joined = [n for n in names if n.startswith("fused_group_kernel")]
    assert len(joined) == (2 if together else 0), names
    if not together:
        # the step and the ascent of every layer; wide ones on large tiles
        for kind in (1, 3):
            mine = [n for n in names if n.startswith("gemm_bf16_kernel<float") and n.endswith(",%d>" % kind)]
            assert len(mine) == len(model["dims"]) - 1 and any(",64,64," not in n for n in mine), names


@pytest.mark.parametrize("side,batch,patches", [((16000, 4), 3, True), ((4000, 32), 7, True), ((32, 32), 128, True),
                                                ((30000, 4), 12, True)])
def test_weight_gradients_of_tall_images_come_from_patches(side, batch, patches):
    names = launches.names(dict(K=1, dims=(3, 32, 32, 10), batch=batch, n_conv=2, img_h=side[0], img_w=side[1], bn_mask=3,
                                global_avg_pool=1))
    assert any(n.startswith("conv_wgrad_kernel<3,") for n in names) == patches, names


def test_divisions_by_high_multiplies_are_exact():
    """The kernels' n / d = (n magic >> 32) >> shift against n / d, for every d up to 5000 and some beyond, at multiples
    of d up to 2^31 and beside them."""
    rng = np.random.default_rng(1)
    for d in list(range(2, 5000)) + [16002, 30002, 65535, 65536, 65537, (1 << 24) - 1]:
        log = max(1, (d - 1).bit_length())
        magic, shift = -(-(1 << (31 + log)) // d), log - 1
        assert magic < 1 << 32
        top = ((1 << 31) - 1) // d
        n = np.concatenate([rng.integers(0, top + 1, 200), np.arange(3), top - np.arange(min(3, top))]) * d
        n = np.concatenate([n, n + d - 1, [(1 << 31) - 1]])
        n = n[(n >= 0) & (n < 1 << 31)].astype(np.uint64)
        assert np.array_equal(n * np.uint64(magic) >> np.uint64(32 + shift), n // np.uint64(d)), d


def conv_net(channels, side, batch, bf16=0, K=1):
    return dict(K=K, dims=(channels, channels, channels, 10), batch=batch, n_conv=2, img_h=side, img_w=side, bn_mask=3,
                global_avg_pool=1, gemm_dtype=bf16)


@pytest.mark.parametrize("model,planes,patches", [
    (conv_net(48, 16, 26), True, False), (conv_net(48, 16, 64), True, True),           # 26 and 64 tiles
    (conv_net(112, 16, 30), True, False), (conv_net(112, 16, 34), True, True),         # 60 and 68
    (conv_net(56, 16, 16), False, False), (conv_net(56, 16, 26), True, False),         # 1.2e8 multiply-adds on 4096 pixels, 1.9e8
    (conv_net(48, 14, 27, bf16=1), False, False), (conv_net(56, 16, 16, bf16=1), True, False)])
def test_which_small_convolutions_take_planes_and_patches(model, planes, patches):
    names = launches.names(model)
    assert any(n.startswith("conv_gemm_kernel<") or "_patch_kernel<" in n for n in names) == planes, names
    assert any(n.startswith("conv_split_patch_kernel<") for n in names) == patches, names


@pytest.mark.parametrize("channels,side,batch,planes", [
    ((8, 184), 32, 64, False), ((16, 184), 32, 64, False), ((8, 88), 32, 64, True), ((8, 128), 32, 64, True), ((184, 8), 32, 64, True),
    ((24, 184), 16, 16, False), ((184, 24), 16, 16, True), ((40, 184), 16, 16, True), ((16, 184), 20, 42, True), ((8, 184), 20, 42, False),
    ((152, 16), 16, 18, True), ((64, 56), 16, 16, False)])
def test_which_widening_convolutions_take_planes(channels, side, batch, planes):
    names = launches.names(dict(K=1, dims=(3,) + channels + (10,), batch=batch, n_conv=2, img_h=side, img_w=side, bn_mask=3,
                                global_avg_pool=1))
    assert any(n.startswith("filters_kernel<3>") for n in names) == planes, names


@pytest.mark.parametrize("channels,batch,bf16,planes", [
    ((32, 48), 29, 0, False), ((32, 48), 88, 0, True), ((16, 24), 29, 0, False), ((16, 24), 64, 0, True), ((16, 24), 29, 1, False),
    ((24, 24), 36, 0, True), ((40, 48), 29, 0, True), ((8, 160), 36, 0, False), ((32, 16), 29, 0, False), ((32, 16), 49, 0, True),
    ((32, 16), 29, 1, True), ((32, 16), 49, 1, True), ((32, 40), 52, 0, False), ((32, 40), 64, 0, True), ((32, 40), 52, 1, True),
    ((32, 72), 29, 0, False), ((32, 72), 39, 0, True), ((128, 16), 29, 0, True), ((32, 16), 20, 1, False), ((8, 24), 47, 0, True),
    ((8, 184), 64, 0, True)])
def test_which_convolutions_on_the_data_take_planes(channels, batch, bf16, planes):
    names = launches.names(dict(K=1, dims=channels + (10,), batch=batch, n_conv=1, img_h=16, img_w=16, bn_mask=1,
                                global_avg_pool=1, gemm_dtype=bf16))
    assert any(n.startswith("filters_kernel<") for n in names) == planes, names


@pytest.mark.parametrize("channels,batch,gathers", [(104, 32, True), (104, 64, False), (184, 16, True), (184, 32, False),
                                                    (88, 48, True), (64, 240, True), (160, 240, True)])
def test_which_first_layers_with_bf16_products_gather_the_image(channels, batch, gathers):
    names = launches.names(dict(K=4, dims=(3, channels, 10), batch=batch, n_conv=1, img_h=16, img_w=16, bn_mask=1,
                                global_avg_pool=1, gemm_dtype=1))
    assert any(n.startswith("first_conv_forward_kernel<") for n in names) == gathers, names


@pytest.mark.parametrize("K,mb,streams", [(8, 90, False), (13, 110, False), (8, 120, False), (1, 100, True), (8, 130, True)])
def test_when_the_joined_ascent_and_descent_stream(K, mb, streams):
    names = launches.names(dict(K=K, d_raw=mb * (1 << 18) // K))
    assert any(n.startswith("descent_kernel<") and n.split(",")[2] == ("true" if streams else "false") for n in names), names


B16, F32 = "gemm_bf16_kernel<%s>", "gemm_kernel<float,float,%s>"


@pytest.mark.parametrize("model,kernels", [
    # test_large_tiles_with_remainders: forward products, input gradients, steps, ascents
    (dict(K=8, dims=(1000, 1400, 1500, 1100, 100), batch=300, gemm_dtype=1),
     [B16 % "__bf16,128,128,4,true,true,2,0", B16 % "__bf16,128,128,4,true,false,2,0", B16 % "float,128,128,4,false,false,2,1",
      B16 % "float,256,128,3,false,false,2,3", "gram_norm_kernel<64,8,2>"]),
    (dict(K=8, dims=(1000, 1400, 1500, 1100, 100), batch=600, gemm_dtype=1),
     [B16 % "__bf16,256,128,3,true,true,2,0", B16 % "__bf16,256,128,3,true,false,2,0", B16 % "float,256,128,3,false,false,2,2"]),
    # test_ragged_tiles_past_the_caches
    (dict(K=8, dims=(1000, 2500, 2300, 300), batch=300, gemm_dtype=1),
     [B16 % "float,256,128,3,false,false,2,3", B16 % "float,128,128,4,false,false,2,1"]),
    # test_bf16_ring_kernel_ragged_tiles_and_short_contractions and the wide layers with long Gram products
    (dict(K=2, dims=(352, 288, 288, 160), batch=160, gemm_dtype=1),
     [B16 % "__bf16,64,64,8,true,true,2,0", "fused_group_kernel<4>", "fused_group_kernel<5>"]),
    (dict(K=2, dims=(1040, 1536, 2048, 24), batch=32, gemm_dtype=1), ["gram_norm_kernel<64,8,2>"]),
    # test_fp32_large_tile_variants_one_replica
    (dict(K=16, dims=(256, 2048, 2048, 24), batch=512),
     [F32 % "256,128,4,true,true,2,0,false", F32 % "128,128,8,true,false,2,0,false", "dense_gradients_kernel<128,2,false>"]),
    # test_gpu_plane_channels.py
    (dict(K=2, dims=(3, 48, 80, 48, 10), batch=40, n_conv=3, img_h=16, img_w=16, bn_mask=7, global_avg_pool=1),
     ["conv_split_patch_kernel<2,2,11>", "conv_wgrad_kernel<3,2,64,9>"]),
    (dict(K=2, dims=(3, 24, 48, 48, 10), batch=16, n_conv=3, img_h=32, img_w=32, bn_mask=7, stride_mask=2, skip_mask=4,
          proj_mask=4, global_avg_pool=1), ["conv_gemm_kernel<3,1,128,64,2,2,2>", "conv_wgrad_kernel<3,2,64,9>"]),
    # test_gpu_dense_gradients.py
    (dict(K=4, dims=(520, 900, 900, 12), batch=100), ["dense_gradients_kernel<128,2,false>"]),
    (dict(K=4, dims=(1024, 1024, 10), batch=520), ["dense_gradients_kernel<128,2,false>", F32 % "64,64,8,false,false,2,0,false"]),
    (dict(K=8, dims=(3, 8, 650, 700, 10), n_conv=1, img_h=16, img_w=16, pool_mask=1, batch=40, gemm_dtype=1),
     ["dense_gradients_kernel<128,2,true>"])])
def test_gpu_tests_reach_the_kernels_they_name(model, kernels):
    names = launches.names(model)
    assert set(kernels) <= set(names), sorted(set(names))
