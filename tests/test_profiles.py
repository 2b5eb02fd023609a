"""The committed counter summaries (profiles/*_traffic.json) describe the kernels of this tree: the
benchmark reports a kernel's HBM traffic only while the hash of its sources is the one the counters were
taken on, so an edit to a source without a new profile takes the figure out of the report."""
import glob
import json
import os

import pytest

import bench
from paper_2609_29499_amd import profile_summary as P

SUMMARIES = sorted(glob.glob(os.path.join(bench.ROOT, "profiles", "*_traffic.json")))


@pytest.mark.parametrize("path", SUMMARIES, ids=[os.path.basename(p) for p in SUMMARIES])
def test_counters_belong_to_the_present_source(path):
    with open(path) as f:
        t = json.load(f)
    name = os.path.basename(path)[:-len("_traffic.json")]
    kernel = next(k for k in bench.KERNEL_SOURCES if name.startswith(k + "_"))
    assert t["kernel_source_hash"] == bench.source_hash(bench.KERNEL_SOURCES[kernel])
    assert bench.load_traffic(kernel, name[len(kernel) + 1:]) == t["bytes_per_launch"]


def test_projection_names_of_a_step():
    """O and down launches share a kernel and are told apart by their place in a step: decode, batched
    decode (operand preparation first) and prefill (operand preparation before every projection)."""
    def names(*kernels):
        return [n for n in P._named([P.kind_of(k) for k in kernels]) if n != "operand_prep"]

    assert names("gemv_kernel<1, 0, 8>", "attn_mfma_kernel<128>", "gemv_kernel<1, 1, 8>", "gemv_kernel<1, 2, 8>",
                 "gemv_kernel<1, 1, 8>", "gemv_kernel<1, 3, 8>") == \
        ["qkv_gemv", "attention", "o_gemv", "gateup_gemv", "down_gemv", "lmhead_gemv"]
    assert names("mfma_prep_kernel", "mfma_gemv_kernel<0, 8, 1, 0>", "attn_mfma_kernel<128>", "mfma_gemv_kernel<1, 4, 1, 0>",
                 "mfma_gemv_kernel<2, 4, 2, 0>", "mfma_gemv_kernel<1, 4, 1, 0>") == \
        ["qkv_mfma", "attention", "o_mfma", "gateup_mfma", "down_mfma"]
    layer = ["pf_i8_kernel<0, 2>", "pf_rope_kernel", "pf_attn_kernel<128>", "pf_quant_kernel<256>", "pf_i8_kernel<1, 2>",
             "pf_quant_kernel<256>", "pf_i8_kernel<2, 4>", "pf_quant_kernel<1024>", "pf_i8_kernel<1, 2>"]
    want = ["qkv_gemm", "rope_append", "prefill_attention", "o_gemm", "gateup_gemm", "down_gemm"]
    assert names("pf_quant_kernel<256>", *layer, "pf_quant_kernel<256>", *layer, "pf_i8_reduce_kernel") == \
        want + want + ["down_reduce"]
