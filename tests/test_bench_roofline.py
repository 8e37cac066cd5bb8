"""The benchmark's roofline line names the kernel that ran (no GPU)."""

import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def _bin(rows, multi, bits, pairs):
    return {"rows_per_lane": rows, "multi_strip": multi, "bits": bits, "pairs": pairs, "cells": 10 ** 9, "ms": 1.0}


def _name(bins, intra=0):
    import bench

    return bench.roofline({"sw_bins": bins}, 1.0, intra)["kernel"]


def test_kernel_of_the_dominant_bin():
    assert _name([_bin(6, 0, 16, 5)]) == "sw16_kernel<false, 3>"
    assert _name([_bin(9, 1, 16, 5)]) == "sw16_kernel<false, 3>"
    assert _name([_bin(6, 0, 32, 5)]) == "sw_pass1_kernel<5, 8, false>"
    # pairs of several strips in 32-bit lanes: by the number of them all and the knob
    few = [_bin(9, 1, 32, 1000), _bin(16, 1, 32, 1048), _bin(9, 1, 16, 5000)]
    many = [_bin(9, 1, 32, 1000), _bin(16, 1, 32, 1049), _bin(9, 1, 16, 5000)]
    for intra in (0, 1):
        assert _name(few, intra) == "sw_long_kernel<false>"
    assert _name(many) == "sw_pass1_kernel<9, 16, true>"
    assert _name(many, 1) == "sw_intra_pass1_kernel<9, 16>"
