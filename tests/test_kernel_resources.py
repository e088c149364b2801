"""What the compiler says about the kernels of the last build (hipcc's kernel-resource-usage
remarks, kept by the build beside the objects): no attention kernel touches scratch memory, and
the selection kernels that are planned for several workgroups per compute unit fit their
register budget. Host-only: reads a text file the build wrote."""
import os
import subprocess

import pytest

from paper_2605_15508_amd import build


@pytest.fixture(scope="module")
def resources():
    if not os.path.exists(build.RESOURCES) or build.needs_build():
        build.build(force=True)
    return build.kernel_resources()


def demangle(sym):
    try:
        return subprocess.run(["c++filt", sym], capture_output=True, text=True, check=True).stdout.strip()
    except (OSError, subprocess.CalledProcessError):
        return sym


def test_every_attention_kernel_runs_without_scratch(resources):
    attn = {k: v for k, v in resources.items() if "attn_split_kernel" in k or "attn_combine_kernel" in k
            or "attn_probsum_kernel" in k}
    assert len(attn) >= 20                      # the instantiated variants are all there
    bad = {demangle(k): v["ScratchSize"] for k, v in attn.items() if v["ScratchSize"] != 0}
    assert not bad, bad


def test_the_logits_dump_at_head_size_128_has_no_four_tile_form(resources):
    # planned with two query tiles at most: its four-tile form would spill about a hundred registers
    assert not [k for k in resources if "attn_split_kernelILi128ELi4ELb0ELb1E" in k]


def test_selection_kernels_fit_the_occupancy_they_are_planned_for(resources):
    for k, v in resources.items():
        if "select_rowpass_kernelILi256" in k:
            assert v["VGPRs"] <= 96 and v["ScratchSize"] == 0, demangle(k)        # five workgroups per CU or more
        if "select_write_kernel" in k:
            assert v["VGPRs"] <= 128 and v["ScratchSize"] == 0, demangle(k)       # four workgroups per CU


def test_the_sampled_and_the_row_selection_fit_their_registers(resources):
    sampled = {k: v for k, v in resources.items() if "select_sampled_kernel" in k}
    row = {k: v for k, v in resources.items() if "select_row_kernel" in k}
    assert len(sampled) == 8 and len(row) == 8
    for k, v in {**sampled, **row}.items():
        assert v["VGPRs"] <= 128, demangle(k)                                         # 16 waves per compute unit
        # (512 threads hold 64 keys each in 128 registers: one loop-invariant word is spilled and reloaded three times)
        assert v["ScratchSize"] <= (8 if "ILi512ELi16E" in k else 0), demangle(k)
    for v in sampled.values():
        assert v["LDS Size"] <= 160 * 1024


# the row kernels of other names, and how many forms each has: rows whose scores are added up first, the longest rows of one score, rows
# of one bf16 score
@pytest.mark.parametrize("name,forms", [("select_row_scores_kernel", 5), ("short_select_row_scores_kernel", 3), ("select_row_long_kernel", 2), ("select_row16_kernel", 5)])
def test_every_form_of_the_row_selection_fits_its_registers(resources, name, forms):
    row = {k: v for k, v in resources.items() if f"{len(name)}{name}I" in k}        # (as the symbol has it: the whole name)
    assert len(row) == forms
    for k, v in row.items():
        assert v["VGPRs"] <= 128 and v["AGPRs"] == 0 and v["ScratchSize"] == 0, demangle(k)


def test_the_ranking_of_block_sums_leaves_room_for_others(resources):
    small = {k: v for k, v in resources.items() if "select_small_kernel" in k}
    blocks = {k: v for k, v in resources.items() if "select_blocks_kernel" in k}
    assert len(small) == 2 and len(blocks) == 8
    for k, v in {**small, **blocks}.items():
        assert v["LDS Size"] <= 40 * 1024, demangle(k)                                # several workgroups per CU
        assert v["VGPRs"] <= 128 and v["ScratchSize"] <= (8 if "ILi512ELi16E" in k else 0), demangle(k)
