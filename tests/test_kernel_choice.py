"""Which kernel, and which instance of it, the automatic choice takes for single layers (no GPU needed: a
dry run of a one-level network that has the layer in it)."""
import ctypes

import pytest

import bench
from paper_2601_11660_amd import binding as B


def choice(convs, n, h, w, step, up=None, base=32):
    d = B.UNetDesc()
    layers = (B.ConvLayer * len(convs))()
    for c, (cin, cout) in zip(layers, convs):
        c.cin, c.cout, c.packed_w, c.thresh = cin, cout, 0x10000, 0x20000
    d.levels, d.base, d.in_channels, d.n_classes, d.convs, d.fuse = 1, base, 3, 19, layers, 1
    if up:
        d.up_convs = (B.ConvLayer * 1)(B.ConvLayer(0x10000, 0x20000, up[0], up[1], 0))
    name = ctypes.c_char_p()
    assert B.lib().mbu_unet_step_kernel(ctypes.byref(d), n, h, w, step, ctypes.byref(name)) == 0, B.last_error()
    return B.last_kernel()


def layer(h, w, cin, cout, n=1):
    """Second encoder layer, with the pooled output."""
    return choice([(32, cin), (cin, cout), (cout, 32), (32, 32), (cout + 32, 32), (32, 32)], n, h, w, 2)


def up_sampled(h, w, ca, cb, cout, n=1):
    """Decoder layer over [skip | 2x up-sampled feature]."""
    return choice([(32, ca), (ca, ca), (ca, cb), (cb, cb), (ca + cb, cout), (cout, 32)], n, h, w, 7)


def concat(h, w, ca, cb, cout, n=1):
    """Decoder layer over [skip | feature of the transposed layer]."""
    return choice([(32, ca), (ca, ca), (ca, ca), (ca, ca), (ca + cb, cout), (cout, 32)], n, h, w, 8, (ca, cb))


SPLIT, BLOCK = "conv_mfma_split_kernel", "conv_mfma_block_kernel"


@pytest.mark.parametrize("h, w, cin, cout, kernel", [
    (64, 64, 512, 512, SPLIT + "<4, 32, true, false>"),      # 2048 groups x channel tiles
    (64, 66, 512, 512, BLOCK + "<2, 1, 4, true, false, true>"),
    (112, 128, 256, 256, BLOCK + "<2, 1, 4, true, false, true>"),
    (128, 128, 256, 256, BLOCK + "<2, 1, 4, true, false, true>"),
    (128, 64, 256, 256, SPLIT + "<2, 16, true, false>"),
    (36, 112, 1024, 512, SPLIT + "<2, 16, true, false>"),    # 576 blocks of four groups: not resident at once
    (112, 24, 256, 768, BLOCK + "<2, 1, 4, true, false, true>"),     # 2016 in the frame, 2688 with two 16-wide tiles
    (40, 96, 1024, 512, SPLIT + "<4, 32, true, false>"),
    (112, 64, 128, 256, SPLIT + "<1, 16, true, false>"),     # two steps: 1792
    (114, 64, 128, 256, BLOCK + "<2, 1, 4, true, false, true>"),
    (4, 6, 1024, 1024, SPLIT + "<1, 8, true, false>"),
])
def test_small_layers_up_to_the_line(h, w, cin, cout, kernel):
    assert layer(h, w, cin, cout) == kernel


@pytest.mark.parametrize("h, w, cin, cout, rows", [
    (210, 96, 128, 512, 4), (159, 128, 192, 512, 4), (127, 128, 192, 768, 4),    # 257 to 384 blocks, several channel groups
    (320, 128, 192, 256, 2), (240, 320, 192, 128, 2), (500, 300, 192, 64, 2),    # one group
    (66, 64, 512, 512, 2),                                                       # at most 256 blocks of two rows
])
def test_rows_per_wave_of_the_block_kernel(h, w, cin, cout, rows):
    assert layer(h, w, cin, cout).startswith(f"{BLOCK}<{rows}, ")


@pytest.mark.parametrize("h, w, ca, cb, cout, kernel", [
    (64, 96, 32, 64, 32, SPLIT + "<1, 32, false, true>"),    # not for the low-resolution kernel: 32 channels
    (75, 131, 64, 128, 64, SPLIT + "<1, 8, true, true>"),    # odd frame
    (13, 21, 32, 32, 64, SPLIT + "<1, 8, false, true>"),     # one step
    (101, 151, 96, 192, 96, SPLIT + "<2, 16, false, true>"),
    (151, 263, 96, 192, 96, BLOCK + "<4, 2, 2, false, true, false>"),
    (75, 131, 256, 512, 256, BLOCK + "<2, 1, 4, true, true, false>"),
    (64, 96, 64, 128, 64, "conv_mfma_upcat_split_kernel<1, 8>"),
])
def test_small_up_sampled_layers(h, w, ca, cb, cout, kernel):
    assert up_sampled(h, w, ca, cb, cout) == kernel


@pytest.mark.parametrize("cin, kernel", [(64 * k, f"tconv_res_kernel<{k}, {rows}>") for k, rows in
                                         ((1, 4), (2, 4), (3, 4), (4, 4), (5, 4), (6, 2), (8, 2), (10, 2), (12, 1), (16, 1))]
                         + [(448, "tconv_bits_kernel<4>"), (1088, "tconv_bits_kernel<4>"), (32, "tconv_mfma_kernel<false>")])
def test_transposed_layers(cin, kernel):
    """Weights resident for every width up to 1024 channels whose groups divide evenly over a block."""
    assert choice([(32, 32), (32, 32), (32, cin), (cin, cin), (64, 32), (32, 32)], 1, 40, 60, 6, (cin, 32)) == kernel


@pytest.mark.parametrize("n, h, w, cin, cout, kernel", [
    (1, 64, 1280, 256, 128, "tconv_wave_kernel<4, 2, 12, true>"),      # 2560 units of two rows
    (1, 62, 1280, 256, 128, "tconv_res_kernel<4, 4>"),
    (8, 62, 1024, 256, 128, "tconv_wave_kernel<4, 2, 12, true>"),      # 15872
    (8, 64, 1024, 256, 128, "tconv_wave_kernel<4, 4, 8, true>"),      # 16384
    (1, 128, 512, 512, 256, "tconv_wave_kernel<8, 2, 8, true>"),       # 4096
    (1, 126, 512, 512, 256, "tconv_res_kernel<8, 2>"),
    (8, 126, 1024, 64, 32, "tconv_wave_kernel<1, 2, 12, false>"),
    (8, 80, 119, 640, 320, "tconv_res_kernel<10, 2>"),
    (32, 40, 59, 1024, 512, "tconv_res_kernel<16, 1>"),
    (8, 128, 1024, 96, 64, "tconv_bits_kernel<4>"),
])
def test_large_transposed_layers(n, h, w, cin, cout, kernel):
    convs = [(32, 32), (32, 32), (32, cin), (cin, cin), (32 + cout, 32), (32, 32)]
    assert choice(convs, n, 2 * h, 2 * w, 6, (cin, cout)) == kernel


@pytest.mark.parametrize("h, w, ca, cout, kernel", [
    (128, 192, 64, 64, "conv_mfma_upcat_split_kernel<1, 8>"),       # 384 tiles, 3 steps
    (128, 256, 64, 64, "conv_mfma_upcat_rows2_kernel"),             # 512
    (64, 128, 256, 256, "conv_mfma_upcat_split_kernel<4, 8>"),      # 512 tiles, 12 steps
    (128, 128, 256, 256, "conv_mfma_upcat_rows2_kernel"),           # 256 blocks of two rows
    (256, 512, 64, 64, "conv_mfma_upcat_rows2_kernel"),             # 512
    (260, 512, 64, 64, "conv_mfma_upcat_kernel"),
    (64, 96, 512, 512, "conv_mfma_upcat_split_kernel<4, 8>"),       # 768 tiles, 24 steps
    (64, 128, 512, 512, "conv_mfma_upcat_rows2_kernel"),            # 256 blocks
    (68, 128, 512, 512, "conv_mfma_upcat_kernel"),
    (512, 1024, 64, 64, "conv_mfma_upcat_kernel"),
])
def test_rows_per_wave_of_the_up_sampled_layers(h, w, ca, cout, kernel):
    assert up_sampled(h, w, ca, 2 * ca, cout) == kernel


@pytest.mark.parametrize("n, h, w, co, blocks", [
    (1, 512, 512, 64, 512),      # segments of 4 rows at three waves per SIMD: three waves
    (2, 186, 334, 128, 518),     # 4
    (2, 120, 1146, 128, 720),    # 6
    (1, 540, 1280, 64, 450),     # 8: two
    (1, 720, 1280, 64, 450),     # 10
    (1, 720, 1280, 32, 720),     # 32 channels: three
    (1, 1024, 2048, 64, 512),    # 22
    (1, 1024, 2048, 128, 768),   # 44 in two chunks of channels: three
    (8, 480, 640, 64, 480),      # 26
    (2, 720, 2048, 64, 512),     # 30
    (2, 768, 2048, 64, 768),     # 32: three waves
    (2, 1024, 2048, 64, 768),    # 44
    (16, 480, 640, 64, 720),     # 54
])
def test_waves_of_the_first_layer(n, h, w, co, blocks):
    assert choice([(co, co)] * 4 + [(2 * co, co), (co, co)], n, h, w, 0, base=co) == "stem_rows_kernel"
    assert B.last_blocks() == blocks


@pytest.mark.parametrize("n, h, w, cin, cout, blocks", [
    (1, 256, 320, 64, 128, 256),          # 2560 units of two rows: fewer than the 3072 wave slots
    (1, 272, 320, 256, 128, 256),         # 2720
    (1, 64, 1280, 256, 192, 255),         # three channel tiles of 85 blocks
    (8, 160, 239, 256, 128, 256),
])
def test_large_transposed_layers_use_every_compute_unit(n, h, w, cin, cout, blocks):
    convs = [(32, 32), (32, 32), (32, cin), (cin, cin), (32 + cout, 32), (32, 32)]
    assert choice(convs, n, 2 * h, 2 * w, 6, (cin, cout)).startswith("tconv_wave_kernel<")
    assert B.last_blocks() == blocks


def test_bound_that_the_benchmark_names_for_transposed_layers():
    assert bench.tconv_bound("tconv_wave_kernel").startswith("mfma")
    assert bench.tconv_bound("tconv_res_kernel").startswith("alu")
