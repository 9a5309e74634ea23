"""Host rules that choose a product's kernel, without a GPU: a small host program links the
library, stands in for the HIP runtime and looks at the kernels that its passes launch.
"""
import os
import subprocess

import pytest

from paper_2412_09584_amd import build as BUILD

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_rules.cpp")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    from paper_2412_09584_amd import binding as B
    B.lib()                                              # built, or built now
    exe = str(tmp_path_factory.mktemp("rules") / "host_rules")
    lib = os.path.dirname(BUILD.OUT)
    r = subprocess.run([BUILD.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-I", BUILD.CSRC,
                        "-I", os.path.join(BUILD.ROOT, "include"), SRC, "-o", exe, "-L", lib, "-lbound",
                        f"-Wl,-rpath,{lib}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(name):
        r = subprocess.run([exe, name], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


def test_dense_products_are_one_geometry_with_one_pixel_and_tap(rules):
    """Only those may take the kernels whose row m is img m: a stride-2 layer onto one pixel has
    several phases with one source pixel and tap, a padded 1x1 layer several result pixels."""
    rules("dense")


def test_bf16_tile_needs_packed_weights(rules):
    """A 1x1 convolution on one pixel is dense but has no bf16 weights: neither the automatic
    rule nor the tuner's list may give it that tile, and its launcher refuses it."""
    rules("split_weights")


def test_direct_dma_option_chooses_the_staging(rules):
    """BOUND_OPT_DIRECT_DMA stages the automatic direct convolutions by LDS DMA, as it is
    declared, in saving and other passes."""
    rules("direct_dma")


def test_tuned_saving_passes_keep_fp32_kernels(rules):
    """Autotuning a SAVE_FOR_GRAD pass chooses among FP32 kernels that keep an order of the
    general ones, and its plans are not those of passes that save nothing."""
    rules("tuning")


def test_passes_larger_than_a_launch(rules):
    """HIP refuses launches of 2^32 threads and more: full CROWN's first pass and the tables'
    launch, which used to work in chunks of the workspace or on their own, take any size still."""
    rules("large")


def test_window_indices_stay_in_range(rules):
    """The window epilogues multiply in 24 bits; passes over layers whose pixel indices exceed
    that may not run on windows."""
    rules("window_index")


def test_large_window_passes_reach_their_configurations(rules):
    """The GPU test of large window passes runs blocks of several groups and 16-pixel windows."""
    rules("window_loops")


def test_debug_checks_cover_windows(rules):
    """BOUND_OPT_CHECK looks at the products that run without it, window passes included."""
    rules("debug_windows")


def test_one_block_picks_where_it_is_faster(rules):
    """Pick-outs that the device-wide sort does in less time keep it."""
    rules("picks")


def test_dense_kernels_by_measured_lines(rules):
    """Dense products of passes that save nothing: the kernel on either side of each line."""
    rules("dense_lines")
