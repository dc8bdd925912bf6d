"""Host-side checks of bench.py: the multi-GPU refusal and the thread-pool
form of the oracle used for the parallel CPU baseline."""

import json
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2409_04202_amd import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


@pytest.mark.parametrize("name,N", [("ring_n4_f32", None), ("ring_n4_i32", None),
                                    ("tree8x8_n64_f32", 4096 + 64),
                                    ("tree8x8x8_n512_bf16", 2048 + 512),
                                    ("cdc384_gentree_f32", 384 * 3 + 1)])
def test_parallel_oracle_equals_oracle(name, N):
    c = workloads.CONFIGS[name]
    N = c["N"] if N is None else N
    if c["kind"] == "gentree":
        plan = oracle.gentree_plan(oracle.from_preorder(c["fanin"]), N)
    else:
        plan = oracle.make_plan(c["kind"], c["n"], N, c["fanin"])
    xs = workloads.inputs(name, N=N)
    want = oracle.execute(plan, [x.copy() for x in xs], c["dtype"])
    with ThreadPoolExecutor(max_workers=4) as pool:
        got = bench.parallel_execute(plan, [x.copy() for x in xs], c["dtype"], pool)
    for q in range(len(xs)):
        assert np.array_equal(got[q], want[q])


def test_kernel_source_hash_ignores_comments_only():
    # the hash that ties the committed traffic counters to the kernel code
    # changes with code, not with comments or layout
    a = "int f(int x) {  // twice\n    return 2 * x; /* doubled */\n}\n"
    b = "// header\nint f(int x) {\n  return 2 * x;\n}\n"
    c = "int f(int x) {\n    return 3 * x;\n}\n"
    assert bench._code_only(a) == bench._code_only(b)
    assert bench._code_only(a) != bench._code_only(c)
    # the stripping assumes no string literal holds a comment marker
    csrc = os.path.join(ROOT, "paper_2409_04202_amd", "csrc")
    # (every file of the executor but the test hooks; the plan library, which
    # decides the steps and not their launches, is not among them)
    assert set(bench.KERNEL_SOURCES) == {f for f in os.listdir(csrc)
                                         if f.endswith((".hpp", ".hip", ".cpp"))} - {
        "debug.cpp", "capi.cpp", "genmodel.cpp", "internal.hpp", "plan.cpp", "plan.hpp"}
    for f in bench.KERNEL_SOURCES:
        for line in open(os.path.join(csrc, f)):
            code = line.split("//")[0]
            for lit in code.split('"')[1::2]:
                assert "//" not in lit and "/*" not in lit, (f, line)


def test_line_stays_short():
    # the printed line with every workload in it, from results of the largest
    # plausible width: a log's tail has to hold it
    form = {"ms_per_step": 12.34567, "timed_steps": 4000, "algbw_gbs": 12345.67,
            "plan_gbs": 12345.6, "kernel_ms_per_step": 12.34567, "reduce_launches": 6,
            "reduce_bytes": 1 << 40, "reduce_ms": 12.34567, "reduce_gbs": 12345.6,
            "reduce_frac": 0.1234, "copy_gbs": 12345.6,
            "kernels": ["phase_kernel", "sliced_kernel", "split_kernel"],
            "launches": [{"phase": 5, "k": 16, "max_dst": 64, "steps": 4032, "bytes": 1 << 40,
                          "ms": 12.34567, "gbs": 12345.6}] * 6,
            "_plan_bytes": (1 << 40, 1 << 40), "_red": [(0, 2, 1 << 40, 1.0)] * 3}
    base = {"value": 12.3456, "unit": "GB/s", "cores": 1, "kind": "oracle", "sample": "x" * 90,
            "cpu": "x" * 40, "seconds": 12.345}
    res = [{"workload": name, "plan": c["kind"], "n": c["n"], "N": c["N"], "dtype": c["dtype"],
            "fanin": None, "default": form, "as_written": form, "cpu_baseline": base,
            "cpu_parallel": base, "step_ms": {"median": 12.34567, "min": 12.34567}}
           for name, c in workloads.CONFIGS.items()]
    out = bench.headline_line(res[0], 20, 5, bench.HEADLINE)
    out["configs_fields"] = bench.CONFIGS_FIELDS
    out["configs"] = [bench.config_short(r) for r in res]
    out["ceiling"] = {"copy_gbs": 12345.6, "copy_lib_gbs": 12345.6, "fold2_gbs": 12345.6}
    assert len(json.dumps(out)) < 10000
    assert [e["workload"] for e in out["configs"]] == list(workloads.CONFIGS)
    assert all("launches" in bench.config_entry(r)["default"] for r in res)
