"""What the compiler made of the kernels (no GPU needed: hipcc cross-compiles for gfx950 and
reports each kernel's registers, LDS and scratch).  The row-copy kernels must keep the chunks a
lane has in flight in registers: a local array of them was once promoted to LDS, 16 KB per
workgroup, which cost the hit gather a fifth of its rate; and no kernel may spill to scratch."""
import os
import re
import subprocess
import tempfile

import pytest


def resource_usage(source):
    from paper_2112_08541_amd import buildlib
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    with tempfile.TemporaryDirectory() as tmp:
        cmd = [hipcc, *buildlib.HIPCC_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
               os.path.join(buildlib.CSRC, source), "-o", os.path.join(tmp, "x.o")]
        p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert p.returncode == 0, p.stdout[-2000:]
    kernels, name = {}, None
    for line in p.stdout.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            kernels[name] = {}
            continue
        m = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", line)
        if m and name:
            kernels[name][m.group(1).strip()] = int(m.group(2))
    return kernels


def test_row_copy_kernels_keep_their_chunks_in_registers():
    kernels = resource_usage("bgl_cache.hip")
    copies = {k: v for k, v in kernels.items()
              if re.search(r"k_gather_hits|k_fetch_miss|k_fetch_link|k_fetch_ring|k_fetch_rows|k_insert_rows|k_assemble_rows|"
                        r"k_list_and_hits|k_insert_both|k_fetch_slots", k)}
    # four row widths of each variant; k_fetch_link, k_fetch_ring and k_fetch_slots take any
    assert len(copies) >= 4 * (1 + 2 + 4 + 1 + 2 + 1 + 1) + 4 + 1
    assert sum("k_fetch_link" in k for k in copies) == sum("k_fetch_ring" in k for k in copies) == 2
    for name, use in copies.items():
        # (k_list_and_hits: its list workgroups' scan; k_fetch_slots: its queues are sized at the launch)
        assert use["LDS Size"] <= (20 if "k_list_and_hits" in name else 0), (name, use)
        # (k_fetch_link's at most 64 workgroups leave every CU room: two rounds of positions and ids may cost it a wavefront)
        assert use["Occupancy"] >= (7 if "k_fetch_link" in name else 8), (name, use)
    for name, use in kernels.items():
        assert use["ScratchSize"] == 0, (name, use)
        if "k_assemble_pre" in name:                 # its per-wavefront lists of (position, slot): 4 x 64 x 8 bytes
            assert use["LDS Size"] == 2048, (name, use)
            continue
        assert use["LDS Size"] <= 1024, (name, use)  # scan scratch only; the sampler's hash table lives in bgl_sample.hip


def test_sampling_kernels_use_the_lds_they_declare():
    kernels = resource_usage("bgl_sample.hip")
    for name, use in kernels.items():
        assert use["ScratchSize"] == 0, (name, use)
        if "k_sample_insert" in name:
            # dedup table 2 x 512 x 8 B + its 2 x 512 x 4 B of entry indices + scan scratch
            assert use["LDS Size"] == 8192 + 4096 + 32, (name, use)
        if "k_sample_direct" in name:
            # table of first occurrences 2 x 512 x 4 B + the workgroup's ids 512 x 4 B + scan scratch
            assert use["LDS Size"] == 4096 + 2048 + 32, (name, use)
    assert sum("k_sample_direct" in k for k in kernels) == sum("k_sample_insert" in k for k in kernels) == 10


def test_ordering_kernels_keep_to_registers():
    kernels = resource_usage("bgl_order.hip")
    for kernel in ("k_expand", "k_count", "k_append"):
        assert sum(kernel in k for k in kernels) == 2, kernel
    for name, use in kernels.items():
        assert use["ScratchSize"] == 0, (name, use)
        if "k_expand" in name:                       # a byte per edge of each wavefront's tile
            assert use["LDS Size"] == 1024 and use["Occupancy"] == 8, (name, use)
