"""A launch may ask for 64 KiB of LDS, static and dynamic together, unless the kernel's limit was raised.
The top-k kernel's dynamic LDS reaches 65536 bytes at the largest budgets (16 bytes per pick and
wave), in the layer with the small-batch dispatch behind it as well: it can have no static LDS."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2510_19366_amd import build as hip_build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_the_topk_kernels_have_no_static_lds(tmp_path):
    out = tmp_path / "route.s"
    subprocess.run(["hipcc", *hip_build.FLAGS, "--offload-device-only", "-S", os.path.join(hip_build.CSRC, "route.hip"),
                    "-o", str(out)], check=True, capture_output=True)
    sizes = re.findall(r"\.amdhsa_kernel (\S*topk_kernel\S*)\s+\.amdhsa_group_segment_fixed_size (\d+)", out.read_text())
    assert len(sizes) >= 2 and all(n == "0" for _, n in sizes), sizes


@pytest.mark.gpu
@pytest.mark.parametrize("T,E,k_max", [(40, 1100, 1024), (64, 3838, 1021), (200, 1030, 1024)])
def test_largest_budgets_of_a_small_batch(T, E, k_max):
    from gpu_util import max_rel, run_layer, to_np
    from oracle import oracle as O
    from paper_2510_19366_amd import binding as B
    from paper_2510_19366_amd import workloads as W
    k = np.random.default_rng(T).integers(k_max - 3, k_max + 1, size=T).astype(np.int32)
    wl = W.make_workload("budget", dtype="bf16", d=64, n_experts=E // 2, n_sub=2, inter_sub=32, req_tokens=[1] * T,
                         req_k=k, k_max=k_max, seed=T, bias_std=1.0, w_std=0.1)
    out, dev, ws = run_layer(wl)
    ref = O.layer_of(wl, return_all=True)
    im = B.layer_intermediates(dev["shape"], ws)
    assert np.array_equal(to_np(im["topk_ids"]), ref["ids"])
    for key, name in (("cnt", "group_count"), ("off", "group_offset"), ("sorted_pair", "sorted_pair"),
                      ("slot_of_pair", "slot_of_pair")):
        assert np.array_equal(to_np(im[name]), ref[key]), name
    assert max_rel(to_np(out), ref["out"]) <= 2e-2
