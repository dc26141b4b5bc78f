"""Which kernels serve the nets of the GPU tests that are named for them, and the edges of the rules that choose, seen without a
GPU (launches.py)."""
import pytest

pytest.importorskip("torch")
import bench  # noqa: E402
import launches  # noqa: E402
import test_gpu_plane_channels as channels  # noqa: E402
import test_gpu_relu_bits as bits  # noqa: E402

FIELDS = ("K", "dims", "batch", "n_conv", "img_h", "img_w", "bn_mask", "stride_mask", "skip_mask", "proj_mask", "preact",
          "pool_mask", "global_avg_pool", "gemm_dtype")


def names(net):
    w = bits.net(**net)
    return launches.names({f: getattr(w, f) for f in FIELDS})


@pytest.mark.parametrize("name,rows", [("96 and 160, last columns on half tiles", 256), ("80 and 96, 64 wide", 128),
                                       ("160, whole tiles", 0)])
def test_last_columns_on_half_tiles(name, rows):
    got = {n for n in names(channels.NETS[name]) if n.startswith("conv_split_patch_narrow_last_kernel<")}
    want = {256: "conv_split_patch_narrow_last_kernel<2,2,11", 128: "conv_split_patch_narrow_last_kernel<1,2,10"}
    assert (bool(got) and all(n.startswith(want[rows]) for n in got)) if rows else not got, got


@pytest.mark.parametrize("side,batch,depth", [((8, 8), 64, 1), ((16, 32), 64, 4), ((32, 32), 128, 16)])
def test_statistics_are_finished_as_deep_as_there_are_chunks(side, batch, depth):
    assert "bn_stats_finish_kernel<%d>" % depth in names(dict(dims=(3, 40, 10), side=side, batch=batch))


@pytest.mark.parametrize("bf16,cut", [(0, "conv_split_patch_kernel<1,2,10>"), (1, "conv_patch_kernel<26>")])
def test_pieces_of_a_cut_product_are_written_plainly(bf16, cut):
    got = names(dict(bits.NETS["chain, products cut over workgroups"], bf16=bf16))
    assert cut in got and cut.replace(">", ",true>") not in got
    whole = names(dict(bits.NETS["chain"], bf16=bf16))
    assert any(n in whole for n in ("conv_split_patch_kernel<2,2,11,true>", "conv_patch_kernel<22,true>"))


def stored(net):
    return "fold3x3_kernel" in names(net)


@pytest.mark.parametrize("name,fold", [("72, stride in classes", False), ("160, stride in classes", False),
                                       ("136, stride through a stored gradient", True),
                                       ("104 to 320 on few pixels, stride through a stored gradient", True)])
def test_input_gradients_of_strides(name, fold):
    assert stored(channels.NETS[name]) == fold


@pytest.mark.parametrize("cin,cout,batch,K,fold", [(72, 320, 28, 1, True), (72, 160, 24, 2, False), (112, 224, 28, 1, True),
                                                   (112, 224, 24, 2, False), (112, 448, 24, 2, True), (112, 448, 80, 2, False),
                                                   (64, 448, 28, 1, False)])
def test_classes_on_few_pixels(cin, cout, batch, K, fold):
    assert stored(dict(dims=(3, cin, cout, 10), side=(16, 16), batch=batch, K=K, stride=0b010)) == fold


@pytest.mark.parametrize("channels,side,images,skip,joined", [
    (64, 8, 4, 0, True), (64, 16, 48, 0, False), (64, 16, 100, 0, True), (64, 32, 48, 0, False), (64, 32, 100, 0, True),
    (64, 4, 4, 0b100, True), (16, 8, 48, 0b100, False), (64, 16, 192, 0b100, False), (64, 16, 512, 0b100, True),
    (64, 32, 512, 0b100, False)])
def test_joined_averages(channels, side, images, skip, joined):
    dims = (3,) + (channels,) * (3 if skip else 2) + (10,)
    net = dict(dims=dims, side=(side, side), batch=images // 4, K=4, skip=skip)
    got = names(net)
    assert ("bn_avgpool_kernel" in got) == joined and ("avgpool_kernel" in got) != joined
    w = bits.net(**net)        # (what the benchmark counts the bytes of)
    assert bench.joined_average(w, w.batch * side * side, channels, bool(skip)) == joined


@pytest.mark.parametrize("name,joined", [("average behind a shortcut", False), ("average of few positions behind a shortcut", True),
                                         ("average of few positions behind a projection", True), ("chain", False),
                                         ("chain, products cut over workgroups", True)])
def test_averages_of_the_gpu_tests(name, joined):
    assert ("bn_avgpool_kernel" in names(bits.NETS[name])) == joined
