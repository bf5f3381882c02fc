"""Register budgets of the hot kernels, read from the compiler's own resource report (no GPU needed).

The verify attention runs two workgroups per compute unit, i.e. 256 registers per wavefront, and its streaming loop
uses every one of them: a change anywhere in the kernel that makes the register allocator spill puts scratch
accesses into that loop (measured: 2-3 % of a launch).  The GEMM's hot instances likewise must not touch scratch.
"""
import os
import re
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

import pytest

import paper_2508_18588_amd as hs

CSRC = os.path.join(os.path.dirname(os.path.abspath(hs.__file__)), "csrc")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(hs.__file__)))


def resource_report(source):
    """{mangled kernel name: {field: int}} from -Rpass-analysis=kernel-resource-usage (device code only)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in hs.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory(prefix="hs_res_") as tmp:
        p = subprocess.run([hipcc] + flags + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only",
                                              "-c", os.path.join(CSRC, source), "-o", os.path.join(tmp, "dev.o"),
                                              "-Rpass-analysis=kernel-resource-usage"],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-2000:]
    report, cur = {}, None
    for line in p.stdout.splitlines():
        m = re.search(r"remark:\s+Function Name: (\S+)", line)
        if m:
            cur = report.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+([A-Za-z /\[\]]+?):\s+(\d+)\s+\[-Rpass", line)
        if m and cur is not None:
            cur[m.group(1).strip()] = int(m.group(2))
    return report


@pytest.fixture(scope="module")
def reports():
    """The sources' reports, compiled side by side (a GEMM source takes minutes)."""
    names = ("hs_gemm_stream.hip", "hs_gemm_wide.hip", "hs_gemm_folded.hip", "hs_accept.hip", "hs_attention.hip", "hs_elementwise.hip")
    with ThreadPoolExecutor(len(names)) as ex:
        return dict(zip(names, ex.map(resource_report, names)))


def test_verify_attention_keeps_two_workgroups_per_compute_unit_without_scratch(reports):
    rep = reports["hs_attention.hip"]
    kernels = {k: v for k, v in rep.items() if "attn_verify_mfma" in k}
    assert len(kernels) == 2, sorted(rep)                      # head_dim 128 and 64
    for name, r in kernels.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)
        assert r["Occupancy [waves/SIMD]"] >= 2, (name, r)
        assert r["LDS Size [bytes/block]"] <= 80 * 1024, (name, r)


def test_hot_gemm_instances_use_no_scratch(reports):
    rep = reports["hs_gemm_stream.hip"]
    # <EPI, PARTIAL, NU, MT, SA, SW> of a 7B-shape speculative step: gate/up, down, QKV and O, LM head (row maximum);
    # and the same at 128 rows (the one-token steps); three and four units at up to 160 rows, the operands fetched apart (other
    # shapes' gate/up, down, heads); then the passes of 64 rows: gate/up, O and down where K is not split, a head that keeps logits,
    # the row maximum
    hot = ["ILi2ELb0ELi5ELi3ELi2ELi3EE", "ILi0ELb1ELi4ELi3ELi2ELi4EE", "ILi0ELb1ELi2ELi3ELi2ELi6EE",
           "ILi3ELb0ELi5ELi3ELi2ELi3EE", "ILi2ELb0ELi5ELi2ELi2ELi4EE", "ILi0ELb1ELi4ELi2ELi3ELi4EE",
           "ILi0ELb1ELi2ELi2ELi2ELi8EE", "ILi3ELb0ELi5ELi2ELi2ELi4EE",
           "ILi2ELb0ELi3ELi2ELi3ELi5EE", "ILi2ELb0ELi4ELi2ELi3ELi4EE", "ILi0ELb1ELi3ELi2ELi3ELi5EE", "ILi1ELb0ELi3ELi2ELi3ELi5EE",
           "ILi1ELb0ELi4ELi2ELi3ELi4EE", "ILi0ELb0ELi3ELi2ELi3ELi5EE", "ILi0ELb0ELi4ELi2ELi3ELi4EE", "ILi3ELb0ELi4ELi2ELi3ELi4EE",
           "ILi2ELb0ELi3ELi0ELi4ELi5EE", "ILi2ELb0ELi4ELi0ELi3ELi4EE", "ILi1ELb0ELi3ELi0ELi4ELi5EE", "ILi1ELb0ELi4ELi0ELi3ELi4EE",
           "ILi0ELb0ELi3ELi0ELi4ELi5EE", "ILi0ELb0ELi4ELi0ELi3ELi4EE", "ILi3ELb0ELi4ELi0ELi3ELi4EE"]
    for tag in hot:
        names = [k for k in rep if "hs_gemm_stream" + tag in k]
        assert len(names) == 1, (tag, sorted(rep))
        r = rep[names[0]]
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (names[0], r)


def test_the_gemm_for_many_rows_uses_no_scratch(reports):
    """Four wavefronts with 256 accumulator registers and some 150 others each: one per SIMD, of 512."""
    rep = {k: v for k, v in reports["hs_gemm_wide.hip"].items() if "hs_gemm_wide" in k}
    assert len(rep) == 4, sorted(rep)                          # gate/up, split K, added, stored
    for name, r in rep.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)
        assert r["VGPRs"] + r["AGPRs"] <= 512 and r["AGPRs"] == 256, (name, r)


def test_folded_gemm_uses_no_scratch(reports):
    """Two sets of up to 64 accumulators in wavefronts of 256 registers."""
    rep = {k: v for k, v in reports["hs_gemm_folded.hip"].items() if "hs_gemm_folded" in k}
    assert len(rep) == 6, sorted(rep)                          # stored and added, 2 to 4 units
    for name, r in rep.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)


def test_greedy_acceptance_and_commit_fill_a_compute_unit(reports):
    """hs_accept_commit of a thousand sequences is one workgroup each: seven or eight of them per compute unit, not the one
    that the sampler's registers would leave."""
    rep = reports["hs_accept.hip"]
    kernels = {k: v for k, v in rep.items() if "accept_commit_kernel" in k and "Lb0E" in k}
    assert len(kernels) == 2, sorted(rep)                      # bf16 and float caches
    for name, r in kernels.items():
        assert r["VGPRs"] <= 72 and r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)
        assert r["Occupancy [waves/SIMD]"] >= 7, (name, r)
    sampler = {k: v for k, v in rep.items() if "reject_stats_kernel" in k or ("accept_commit_kernel" in k and "Lb1E" in k)}
    assert len(sampler) == 3, sorted(rep)                      # the sums, and the walk for either cache
    for name, r in sampler.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)


def test_row_kernels_for_many_rows_let_two_workgroups_share_a_compute_unit(reports):
    """hs_row_grid deals rows to 2048 threads per compute unit: eight wavefronts per SIMD, or a launch whose workgroups have 1024
    threads runs in two rounds.  (The instances for a few rows, EARLY, trade that for more loads in flight.)"""
    rep = reports["hs_elementwise.hip"]
    many = [k for k in rep if re.search(r"rmsnorm_kernelI[tf]Li[12]ELb0E|rope_kv_kernelI[tf]Lb0E|argmax_kernel", k)]
    assert len(many) >= 7, sorted(rep)
    for name in many:
        assert rep[name]["VGPRs"] <= 64 and rep[name]["Occupancy [waves/SIMD]"] == 8, (name, rep[name])
    for name, r in rep.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)
