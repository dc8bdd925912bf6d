"""The one-pass launch (csrc/onepass.hpp): a whole AllReduce as one launch with
its values in registers, the form that plans whose steps do not lie on 16-byte
boundaries and buffers that do not take by default.

On the host, the library's check runs every segment's leaves on terms against
the executed steps and walks the tiles of every kernel instance.  On the GPU,
results equal the oracle's bit for bit at the sizes where the tiling changes.
"""

import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2409_04202_amd import workloads

from checklib import arplan as check, set_onepass
from test_capi_host import _check_tiling

if torch.cuda.is_available():
    from gpu_helpers import run_plan, say, to_device, to_host
    from paper_2409_04202_amd import arplan

ASY = workloads.preorder([[4, 4], [4, 2], 3, [2]])  # uneven switches, 19 servers

PLANS = [("ring", 2, None), ("ring", 5, None), ("ring", 64, None), ("ring", 70, None),
         ("rhd", 8, None), ("rhd", 12, None), ("rhd", 96, None), ("cps", 3, None),
         ("cps", 70, None), ("rb", 6, None), ("tree", 12, (3, 4)), ("tree", 24, (2, 3, 4)),
         ("tree", 96, (8, 12)), ("gentree", 19, tuple(ASY))]


@pytest.mark.parametrize("kind,n,fan", PLANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32"])
def test_program_and_tiles(kind, n, fan, dtype):
    # N off the processors and the vectors; around a tile of 64 4-byte lanes;
    # where the instance changes (64, 200, 512, 3072 and 7168 tiles of 1 KiB)
    es = 2 if dtype == "bf16" else 4
    kib = 1024 // es
    for N in (16 // es + 1, 67, max(n + 1, 16 // es), 64 * 4 // es + 1, 5 * n + 3, 64 * kib + 1,
              200 * kib - 1, 513 * kib - 1, 3072 * kib + 3,
              4608 * kib + 1, 7168 * kib + 5):
        with check.Plan(n, N, dtype, kind, fan) as p:
            L = p.launches()
            if n <= 512 and (N % n if kind != "rb" else N * es % 16):
                # a step boundary off 16 bytes: one launch moving each byte once
                assert [x[0] for x in L] == [-4] and L[0][4] == 2 * n * N * es, (N, L)
                assert p.launch_kernels() == ["onepass_kernel"]
            for fuse in (1, 0):
                p.set_option(check.AR_OPT_FUSE, fuse)
                for vecok in (1, 0):
                    st, msg = _check_tiling(p.handle, vecok)
                    assert st == check.AR_OK, (N, msg)
            # not without resident launches, nor without sliced ones
            p.set_option(check.AR_OPT_RESIDENT, 0)
            assert all(x[0] >= -1 for x in p.launches())
            p.set_option(check.AR_OPT_RESIDENT, 1)
            set_onepass(p.handle, 0)
            assert "onepass_kernel" not in p.launch_kernels()


@pytest.mark.parametrize("kind,n,N,dtype,kernel", [
    # over two buffers a sliced launch is as fast up to 12 MiB a buffer, and
    # where both hardly fit the caches; four-wave teams are not where predicted
    # at over 0.95 of the resident launch's time
    ("ring", 2, 1 << 21, "f32", "sliced_kernel"), ("rhd", 2, 3633184, "bf16", "sliced_kernel"),
    ("ring", 2, 11010048, "f32", "sliced_kernel"), ("ring", 2, 1 << 22, "f32", "onepass_kernel"),
    ("ring", 2, 1 << 24, "f32", "onepass_kernel"), ("ring", 28, 28224, "f32", "resident_kernel"),
    ("ring", 64, 1 << 15, "f32", "onepass_kernel"), ("rhd", 28, 28224, "f32", "onepass_kernel")])
def test_where_one_pass_takes_the_place_of_a_launch(kind, n, N, dtype, kernel):
    with check.Plan(n, N, dtype, kind) as p:
        assert p.launch_kernels() == [kernel]


def test_plans_that_have_no_one_pass_form():
    # buffers that end with different values, positions no step covers, a
    # plain copy (its bits are not to pass through an addition)
    N = 1001
    for n, steps in ((3, [(0, "reduce", 0, [0, 1], 0, N), (0, "copy", 2, [1], 0, N)]),
                     (2, [(0, "reduce", 0, [0, 1], 0, 500), (1, "copy", 1, [0], 0, 500)]),
                     (2, [(0, "copy", 1, [0], 0, N)])):
        h = check.ar_plan_create_custom(n, N, "f32", steps)
        try:
            L = [check.ar_plan_launch_info(h, i) for i in range(check.ar_plan_num_launches(h))]
            assert all(x[0] >= 0 for x in L), L
            for vecok in (1, 0):
                st, msg = _check_tiling(h, vecok)
                assert st == check.AR_OK, msg
        finally:
            check.ar_plan_destroy(h)


@pytest.mark.parametrize("swap", [False, True])
def test_a_long_chain_has_no_one_pass_form(swap):
    # 300000 phases, each folding the one before: far more folds than buffers,
    # found without descending them all (in a process of its own: a descent
    # that deep runs out of stack)
    code = """
import sys
sys.path.insert(0, %r)
from checklib import arplan as check
N, P, srcs = 1023, 300000, %r
steps = [(q, "reduce", 0, srcs, 0, N) for q in range(P)] + [(P, "copy", 1, [0], 0, N)]
h = check.ar_plan_create_custom(2, N, "f32", steps)
print("launches", check.ar_plan_num_launches(h))
""" % (os.path.dirname(os.path.abspath(__file__)), [1, 0] if swap else [0, 1])
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    assert int(r.stdout.split()[-1]) >= 300000, r.stdout


# (kind, n, N, dtype, fan): every instance, with a partial last vector
GPU = [("ring", 5, 67, "f32", None), ("rhd", 5, 4099, "f32", None), ("rhd", 7, 4099, "bf16", None),
       ("tree", 15, 4099, "f32", (3, 5)), ("tree", 35, 4099, "bf16", (5, 7)), ("ring", 64, 8195, "bf16", None), ("rhd", 12, 4099, "bf16", None),
       ("tree", 24, 20011, "i32", (2, 3, 4)), ("cps", 70, 1003, "bf16", None),
       ("gentree", 19, 30011, "bf16", tuple(ASY)), ("rhd", 96, 5003, "f32", None),
       ("cps", 3, 513 * 256 + 1, "f32", None), ("rhd", 6, 513 * 512 + 3, "bf16", None),
       ("tree", 12, 600 * 256 + 7, "f32", (3, 4)), ("ring", 17, 600 * 512 + 9, "bf16", None),
       ("rhd", 4, 3072 * 256 + 5, "f32", None), ("tree", 6, 3072 * 512 + 5, "bf16", (3, 2)),
       ("cps", 3, 7168 * 256 + 3, "i32", None), ("rhd", 4, 7168 * 512 + 7, "bf16", None),
       # teams of 16 and of 4 waves, several chunks, either side of their limits
       ("tree", 20, 64 * 256 - 1, "f32", (4, 5)), ("ring", 129, 96 * 512 + 1, "bf16", None),
       ("tree", 130, 97 * 256 + 1, "f32", (10, 13)), ("rhd", 66, 200 * 512 - 3, "bf16", None),
       ("cps", 21, 200 * 256 + 3, "i32", None), ("rhd", 300, 4099, "f32", None),
       ("rhd", 4, 7168 * 1024 + 3, "f32", None), ("cps", 2, 2049 * 16 * 512 + 5, "bf16", None),
       # U 4, 8 and 16 (from 12 buffers on), tile after tile beyond 32768 tiles
       ("cps", 12, 3072 * 256 + 5, "f32", None), ("tree", 12, 4608 * 256 + 3, "i32", (4, 3)),
       ("rhd", 12, 7168 * 256 + 9, "f32", None), ("tree", 12, 3100 * 512 + 1, "bf16", (4, 3)),
       ("ring", 13, 4608 * 512 + 7, "bf16", None), ("cps", 12, 7373 * 512 + 3, "bf16", None),
       ("rhd", 3, 32769 * 256 + 5, "f32", None),
       # tile after tile on aligned buffers alone: cached, and from 16384 tiles on
       ("cps", 6, 14000 * 256, "f32", None), ("rhd", 5, 5 * 4096 * 1024, "bf16", None),
       ("ring", 7, 7 * 2500 * 256, "i32", None)]


def _oracle_plan(kind, n, N, fan):
    if kind == "gentree":
        return oracle.gentree_plan(oracle.from_preorder(fan), N)
    return oracle.make_plan(kind, n, N, fan)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,n,N,dtype,fan", GPU)
def test_bit_exact(kind, n, N, dtype, fan):
    dist = "int1000" if dtype == "i32" else "uniform"
    xs0 = workloads.draw(n, N, dtype, dist, N % 89)
    want = oracle.execute(_oracle_plan(kind, n, N, fan), [x.copy() for x in xs0], dtype)
    # aligned buffers, and buffers each a few elements off 16 bytes
    for pad in (0, 1, 3):
        say("case: one-pass %s n=%d N=%d %s pad=%d" % (kind, n, N, dtype, pad))
        ts = to_device(xs0, dtype, pad)
        with arplan.Plan(n, N, dtype, kind, fan) as p:
            run_plan(p, ts)
        got = to_host(ts, dtype)
        for q in range(n):
            assert np.array_equal(got[q], want[q]), (pad, q)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32"])
def test_dense_rows_leave_their_surroundings_alone(dtype):
    # rows of one matrix of odd width (each row at another alignment), with
    # guard elements around it, through the strided and the no-allocation
    # entry points; special values among the inputs
    n, N = 9, 4101
    t = {"f32": torch.float32, "i32": torch.int32, "bf16": torch.bfloat16}[dtype]
    rng = np.random.default_rng(5)
    x = rng.integers(-100, 101, size=(n, N)).astype(np.float32)
    if dtype != "i32":
        x[rng.integers(0, n, 300), rng.integers(0, N, 300)] = np.inf
        x[rng.integers(0, n, 300), rng.integers(0, N, 300)] = -0.0
        x[:, :50] = -0.0
        x[:, 50:90] *= 1e-40  # denormal
        x[0, 100:120] = np.nan
    for kind in ("ring", "cps", "tree"):
        for entry in ("strided", "noalloc"):
            say("case: one-pass dense %s %s %s" % (kind, entry, dtype))
            outs = []
            for res in (1, 0):  # against the phase launches
                g = torch.full((n * N + 64,), 7, dtype=t, device="cuda")
                m = g[33:33 + n * N].view(n, N)
                m.copy_(torch.from_numpy(x).to(t))
                with arplan.Plan(n, N, dtype, kind, (3, 3) if kind == "tree" else None) as p:
                    p.set_option(arplan.AR_OPT_RESIDENT, res)
                    s = torch.cuda.current_stream()
                    if entry == "strided":
                        p.execute_strided(m, N * m.element_size(), s)
                    else:
                        p.execute_noalloc(list(m), s)
                    torch.cuda.synchronize()
                assert bool((g[:33] == 7).all()) and bool((g[33 + n * N:] == 7).all())
                outs.append(m.cpu())
            a, b = outs
            if dtype == "i32":
                assert torch.equal(a, b)
            else:
                nan = torch.isnan(b)
                assert torch.equal(torch.isnan(a), nan)
                bits = torch.int32 if dtype == "f32" else torch.int16
                assert torch.equal(a.view(bits)[~nan], b.view(bits)[~nan])


@pytest.mark.gpu
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("n,N,slice_", [(8, 8 * 4096, 2), (12, 4099, 2), (12, 4099, 0)])
def test_timer_records_one_launch_or_one_a_phase(n, N, slice_, pad):
    # one record an execution where it runs one-pass: on buffers off 16 bytes,
    # and wherever a step boundary is; one a phase launch without
    xs0 = workloads.draw(n, N, "f32", "uniform", 9)
    want = oracle.execute(oracle.rhd(n, N), [x.copy() for x in xs0], "f32")
    t = arplan.ar_timer_create(64)
    try:
        with arplan.Plan(n, N, "f32", "rhd") as p:
            p.set_option(arplan.AR_OPT_SLICE, slice_)
            L = p.launches()
            one = slice_ == 2 and (pad or p.launch_kernels() == ["onepass_kernel"])
            say("case: timed rhd n=%d N=%d slice=%d pad=%d" % (n, N, slice_, pad))
            for rep in range(2):
                ts = to_device(xs0, "f32", pad)
                p.execute_timed(ts, torch.cuda.current_stream(), t)
                torch.cuda.synchronize()
                got = to_host(ts, "f32")
                assert all(np.array_equal(got[q], want[q]) for q in range(n))
            recs = arplan.ar_timer_read(t, 64)
            assert [li for li, _ in recs] == (list(range(1 if one else len(L))) * 2)
            assert all(ms > 0 for _, ms in recs)
    finally:
        arplan.ar_timer_destroy(t)


@pytest.mark.gpu
def test_many_plans_share_the_no_allocation_array():
    # 20 plans of 2 MiB of records each (Ring over 128 buffers as written)
    # in turn: their images go round the 32 MiB array; a graph of the first
    # one replays after an uncaptured call has put its tables back
    n, N = 128, 1024
    xs0 = workloads.draw(n, N, "i32", "int1000", 3)
    ref, got = to_device(xs0, "i32"), to_device(xs0, "i32")
    s = torch.cuda.current_stream()
    plans = [arplan.Plan(n, N, "i32", "ring") for _ in range(20)]
    for p in plans:
        p.set_option(arplan.AR_OPT_FUSE, 0)
        p.set_option(arplan.AR_OPT_SLICE, 0)
    plans[0].execute_noalloc(got, s)
    plans[0].execute(ref, s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plans[0].execute_noalloc(got, torch.cuda.current_stream())
    for rnd in range(2):
        for i, p in enumerate(plans):
            say("case: noalloc round %d plan %d" % (rnd, i))
            p.execute_noalloc(got, s)
            p.execute(ref, s)
        plans[0].execute_noalloc(got, s)
        plans[0].execute(ref, s)
        torch.cuda.synchronize()
        g.replay()
        plans[0].execute(ref, s)
        torch.cuda.synchronize()
        assert all(np.array_equal(a, b) for a, b in zip(to_host(got, "i32"), to_host(ref, "i32"))), rnd
    for p in plans:
        p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1024, 1027])
def test_captured_copy_into_the_no_allocation_array(N):
    # a call captured when another plan was the last one records its copy,
    # which has not run when the next uncaptured call needs the tables
    n = 4
    xs0 = workloads.draw(n, N, "i32", "int1000", 5)
    ref, got = to_device(xs0, "i32"), to_device(xs0, "i32")
    s = torch.cuda.current_stream()
    with arplan.Plan(n, N, "i32", "ring") as p, arplan.Plan(n, N, "i32", "cps") as q:
        for r in (p, q):
            r.execute_noalloc(got, s)
            r.execute(ref, s)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        say("case: noalloc capture N=%d" % N)
        with torch.cuda.graph(g):
            p.execute_noalloc(got, torch.cuda.current_stream())
        for rnd in range(3):
            p.execute_noalloc(got, s)
            p.execute(ref, s)
            torch.cuda.synchronize()
            g.replay()
            p.execute(ref, s)
            torch.cuda.synchronize()
            for x, y in zip(to_host(got, "i32"), to_host(ref, "i32")):
                assert np.array_equal(x, y), rnd


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 8, 12, 16])
def test_phase_launches_on_element_aligned_buffers(n, dtype):
    # every source count's kernel, on rows each at another alignment, as
    # written (co-located PS: an n-way fold and copies, n ragged blocks) and
    # with the rewrites (many destinations); around a pass of 64 lanes x 2 or 4
    # vectors and a tile
    vec = 8 if dtype == "bf16" else 4
    # and about the steps of up to 64 elements with a remainder
    for N in (n + 1, 64 * vec * 2 * n + 1, 64 * vec * 4 * n - 1, 1024 * vec * n + 5,
              49 * n, 61 * n + 1, 64 * n - 1, 65 * n):
        xs0 = workloads.draw(n, N, dtype, "int1000" if dtype == "i32" else "uniform", N % 97)
        want = oracle.execute(oracle.make_plan("cps", n, N, None), [x.copy() for x in xs0], dtype)
        for fuse in (0, 1):
            say("case: element-aligned phases cps n=%d N=%d %s fuse=%d" % (n, N, dtype, fuse))
            ts = [to_device([x], dtype, 1 + q % (vec - 1))[0] for q, x in enumerate(xs0)]
            with arplan.Plan(n, N, dtype, "cps") as p:
                p.set_option(arplan.AR_OPT_FUSE, fuse)
                p.set_option(arplan.AR_OPT_SLICE, 0)
                run_plan(p, ts)
            got = to_host(ts, dtype)
            for q in range(n):
                assert np.array_equal(got[q], want[q]), (N, fuse, q)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32"])
@pytest.mark.parametrize("n", [7, 9, 12, 17, 31])
def test_narrow_passes_of_small_launches(n, dtype):
    # runtime source counts on both sides of the narrow pass's first one, and
    # copies, as written: around a fold pass of 64 lanes x 2 vectors, a copy
    # pass of 64 x 4 and a tile (blocks of 16-byte aligned length and not)
    vec = 8 if dtype == "bf16" else 4
    for blk in (vec, 64 * vec * 2, 64 * vec * 2 + vec, 64 * vec * 4 - vec, 1024 * vec + vec):
        for N in (n * blk, n * blk - 3):
            xs0 = workloads.draw(n, N, dtype, "int1000" if dtype == "i32" else "uniform", N % 97)
            want = oracle.execute(oracle.make_plan("cps", n, N, None),
                                  [x.copy() for x in xs0], dtype)
            say("case: narrow passes cps n=%d N=%d %s" % (n, N, dtype))
            ts = to_device(xs0, dtype)
            with arplan.Plan(n, N, dtype, "cps") as p:
                p.set_option(arplan.AR_OPT_FUSE, 0)
                p.set_option(arplan.AR_OPT_SLICE, 0)
                run_plan(p, ts)
            got = to_host(ts, dtype)
            for q in range(n):
                assert np.array_equal(got[q], want[q]), (N, q)
