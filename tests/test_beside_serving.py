"""CPU test of the kernels' resources: the ones that calls launch while the
serving executor is resident start beside it.  The executor holds two blocks of
256 threads on every CU until it has been idle for a while."""
import json
import os

import pytest

from paper_1505_01120_amd import build as libbuild

REGISTERS, WAVES = 512, 8  # of a SIMD, per lane
# Half a CU's LDS: blocks of 77 KiB start beside the executor's two, and one of
# 96 KiB was seen to wait until they left.
LDS = 80 << 10


@pytest.fixture(scope="module")
def isa():
    if not os.path.exists(libbuild.ISA_JSON):
        libbuild.build()
    with open(libbuild.ISA_JSON) as f:
        return json.load(f)


@pytest.mark.parametrize("kernel,threads", [
    ("k_task", 256), ("k_batch", 256), ("k_batch_mc", 256), ("k_map", 256), ("k_chain", 256),
    ("k_tree", 256), ("k_tree_flat", 1024), ("k_wordcount", 512), ("k_wl_scan", 512),
    ("k_wc_merge", 1024), ("k_wc_compact", 1024)])
def test_block_fits(isa, kernel, threads):
    def registers(k):  # of a wave, as allocated
        return -(-isa[k]["vgpr"] // 8) * 8
    waves = -(-threads // 256)  # a SIMD's, of four
    assert waves * registers(kernel) + 2 * registers("k_serve") <= REGISTERS
    assert isa[kernel]["lds_bytes"] + 2 * isa["k_serve"]["lds_bytes"] <= LDS
    assert waves + 2 <= WAVES
    assert isa[kernel]["private_segment_bytes"] == 0
