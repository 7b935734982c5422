"""The hash that ties the committed counter summaries to the kernels covers the
files that the summary says it covers, which are the sources of every product
(no GPU)."""
import hashlib
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1012_2270_amd", "csrc")


def test_hash_covers_the_named_sources():
    with open(os.path.join(bench.ROOT, "profiles", "rgcsr_spmv_hbm_counters.md")) as f:
        names = re.search(r"Kernel source hash \(([^)]*)\)", f.read())[1].split(", ")
    # conversion and the conjugate-gradient vectors have no counters
    products = {n for n in os.listdir(CSRC) if n.endswith(".hip")} - {"convert.hip", "cg.hip"}
    assert products <= set(names)
    h = hashlib.sha256()
    for n in names:
        with open(os.path.join(CSRC, n), "rb") as f:
            h.update(f.read())
    assert h.hexdigest()[:16] == bench.kernel_source_hash()
