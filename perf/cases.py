"""The work that this framework is used for, as cases that can be measured.

A case is one AllReduce plan over ``n`` processors' buffers of ``N`` elements,
executed through the public binding (``paper_2409_04202_amd.arplan``) on the
current stream, in place.  ``prepare`` makes what a program holds before the
call (the buffers, the plan, the pointer array), ``run`` is one execution and
returns every buffer.

Buffers come in two layouts.  ``rows``: one allocation a processor, as a
program with a tensor per processor has them, so each starts on a 16-byte
boundary.  ``dense``: the rows of one contiguous (n, N) matrix, passed as a
base and a stride, so that an odd N leaves the rows off 16-byte alignment.

Sizes are those of the paper's workloads in ``workloads.CONFIGS``, of the
tests, and generic odd lengths: a vector's length is whatever its model gives
it and is seldom a multiple of the number of processors.
"""

import json
import math

import torch

from paper_2409_04202_amd import arplan, workloads

TORCH = {"f32": torch.float32, "i32": torch.int32, "bf16": torch.bfloat16}
ESIZE = workloads.ESIZE


def _case(name, kind, n, N, dtype, fan="", layout="rows", entry="execute", form="default",
          dist="uniform"):
    c = {"kind": kind, "n": n, "N": N, "dtype": dtype, "fan": fan, "layout": layout,
         "entry": entry, "form": form, "dist": dist}
    if name:
        c["name"] = name
    return c


def listed():
    c = workloads.CONFIGS
    return [
        # The smallest call: a handful of short vectors in a tight loop that
        # may not allocate.  Launch and call overhead.
        _case("ring4_64k_i32", "ring", 4, c["ring_n4_i32"]["N"], "i32", entry="noalloc",
              dist="int1000"),
        # Small messages between many processors, where the rounds of the
        # plan count and not its bytes.
        _case("ring64_4k_bf16", "ring", 64, workloads.SWEEP_N[0], "bf16"),
        _case("tree64_64k_f32", "tree", 64, workloads.SWEEP_N[1], "f32", fan="8,8"),
        # A vector whose length the processors do not divide: no block of the
        # plan starts on a 16-byte boundary.
        _case("ring64_odd64k_f32", "ring", 64, (1 << 16) + 5, "f32"),
        # A number of processors that is no power of two, an odd length, bf16.
        _case("rhd12_odd1m_bf16", "rhd", 12, 1000003, "bf16"),
        # The rows of one dense matrix of odd width.
        _case("cps16_dense_f32", "cps", 16, (1 << 20) + 7, "f32", layout="dense",
              entry="strided", dist="normal"),
        # Ordinary sizes: a hierarchy over an odd length, Ring at the end of
        # the message-size sweep.
        _case("tree64_odd1m_f32", "tree", 64, (1 << 20) + 5, "f32", fan="8,8"),
        _case("ring64_1m_f32", "ring", 64, workloads.SWEEP_N[2], "f32"),
        # The plan as it is written, a launch a phase, as a fit of the cost
        # model times it: 4 MiB a processor, a fan-in of 12.
        _case("written_cps12_1m_f32", "cps", 12, 1 << 20, "f32", form="written"),
        # Many processors: the three-level tree and the asymmetric data
        # centre.
        _case("tree512_256k_bf16", "tree", 512, c["tree8x8x8_n512_bf16"]["N"], "bf16", fan="8,8,8"),
        _case("asy384_768k_f32", "gentree", 384, c["asy384_gentree_f32"]["N"], "f32",
              fan=json.dumps(workloads.ASY384)),
        # The largest: 2 GiB, the headline configuration.
        _case("rhd8_64m_f32", "rhd", 8, c["rhd_n8_f32"]["N"], "f32"),
    ]


# Of the listed cases the largest holds 2 GiB; a drawn one at most this.
_MOST = 1 << 30


def draw(rng):
    """One more case: plan kind, processors, dtype, layout and length over the
    range of the listed ones (512 KiB to 1 GiB in all, 1K elements and more a
    processor), half of the lengths whatever the draw gives."""
    kind = rng.choice(("ring", "ring", "rhd", "rhd", "cps", "cps", "tree", "tree", "tree",
                       "gentree", "rb"))
    fan = ""
    if kind == "tree":
        levels = rng.choice((2, 2, 3))
        f = [rng.choice((2, 3, 4, 6, 8, 12, 16) if levels == 2 else (2, 4, 6, 8))
             for _ in range(levels)]
        n, fan = math.prod(f), ",".join(map(str, f))
    elif kind == "gentree":
        # middle switches of unequal size under one root
        spec = []
        for _ in range(rng.randint(2, 4)):
            servers = rng.choice((2, 4, 8))
            spec += [[servers] * rng.choice((1, 2, 4))] * rng.randint(1, 4)
        n, fan = sum(map(sum, spec)), json.dumps(spec)
    else:
        n = int(round(math.exp(rng.uniform(math.log(3), math.log(64 if kind != "rb" else 16)))))
    dtype = rng.choice(("f32", "f32", "bf16", "i32"))
    total = math.exp(rng.uniform(math.log(1 << 19), math.log(_MOST)))
    N = max(1024, int(total / (n * ESIZE[dtype])))
    if rng.random() < 0.5:  # a round length, as a power of two a processor's block
        N = n * max(16, 1 << int(math.log2(max(1, N // n))))
    layout = "dense" if rng.random() < 0.25 else "rows"
    entry = "strided" if layout == "dense" else "execute"
    form = "written" if rng.random() < 0.15 and kind != "ring" else "default"
    dist = "int1000" if dtype == "i32" else rng.choice(("uniform", "normal"))
    return _case("", kind, n, N, dtype, fan, layout, entry, form, dist)


# ---------------------------------------------------------------- inputs

def _stride(case):
    """Elements from one row to the next: rows of their own start on 512-byte
    boundaries, as allocations do."""
    if case["layout"] == "dense":
        return case["N"]
    unit = 512 // ESIZE[case["dtype"]]
    return -(-case["N"] // unit) * unit


def _inputs(case, seed):
    n, N, dtype = case["n"], case["N"], TORCH[case["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.zeros((n, _stride(case)), dtype=dtype, device="cuda")
    for p in range(n):  # a row at a time: no second copy of everything
        if case["dist"] == "int1000":
            r = torch.randint(-1000, 1001, (N,), generator=g, device="cuda", dtype=torch.int32)
        elif case["dist"] == "normal":
            r = torch.randn(N, generator=g, device="cuda")
        else:
            r = torch.rand(N, generator=g, device="cuda") * 2 - 1
        x[p, :N] = r.to(dtype)
    return x


class State:
    pass


def prepare(case, seed):
    s = State()
    s.x = _inputs(case, seed)
    s.out = s.x[:, :case["N"]]
    s.stride = _stride(case) * ESIZE[case["dtype"]]
    if case["kind"] == "gentree":
        fan = workloads.preorder(json.loads(case["fan"]))
    else:
        fan = [int(f) for f in case["fan"].split(",")] if case["fan"] else None
    s.plan = arplan.Plan(case["n"], case["N"], case["dtype"], case["kind"], fan)
    if case["form"] == "written":  # every step as listed, a launch a phase
        s.plan.set_option(arplan.AR_OPT_FUSE, 0)
        s.plan.set_option(arplan.AR_OPT_SLICE, 0)
    s.bufs = arplan.pointers(list(s.out))
    s.entry = case["entry"]
    return s


def run(s):
    stream = torch.cuda.current_stream()
    if s.entry == "strided":
        s.plan.execute_strided(s.x, s.stride, stream)
    elif s.entry == "noalloc":
        s.plan.execute_noalloc(s.bufs, stream)
    else:
        s.plan.execute(s.bufs, stream)
    return s.out


def work(case):
    n, N = case["n"], case["N"]
    return {"bytes": 2.0 * n * N * ESIZE[case["dtype"]], "flops": float(n - 1) * N}


def tolerance(case):
    # The interface fixes the arithmetic of every step (its source order, fp32
    # accumulation and one rounding a step for bf16, wrap-around for int32),
    # so a plan has one result.
    return "exact"


def exact(case, seed):
    x = _inputs(case, seed)[:, :case["N"]]
    if case["dtype"] == "i32":
        s = torch.zeros(case["N"], dtype=torch.int64, device="cuda")
        for p in range(case["n"]):
            s += x[p]
        s = s.to(torch.int32)
    else:
        s = torch.zeros(case["N"], dtype=torch.float64, device="cuda")
        for p in range(case["n"]):
            s += x[p]
    return s.expand(case["n"], case["N"])
