"""Schedules as queue packets: streams that share a lane, buffers exchanged between runs, passes longer than a queue,
several contexts at once.  Every output is compared bit for bit with the sequential schedule's."""
import os
import shutil
import subprocess
import sys
import threading

import numpy as np
import pytest

from paper_2111_14255_amd import binding as B
from synth import GraphBuilder, zoo
from gpu_harness import Mix

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(np.array_equal(x.view(np.uint32), y.view(np.uint32)) for x, y in zip(a, b))


def chain(n_ops, batch=1):
    g = GraphBuilder("chain", "f16", batch, 4, 4, 16)
    t = 0
    for _ in range(n_ops):
        t = g.conv(t, 16, 1, bn=True)
    return g.done()


@pytest.mark.parametrize("n", [1, 4, 5, 7, 16])
def test_more_streams_than_lanes_keep_the_bits(n):
    # chains of different length: on a shared lane the shorter one ends while the longer one goes on
    names = ["tinyA", "tinyC", "tinyD", "tinyB"]
    mix = Mix([zoo.BUILDERS[names[i % 4]]("f16", 1 + i % 3) for i in range(n)], 31, "uniform")
    try:
        ref, _ = mix.run(mix.ctx.sequential())
        for stages in (1, 3):
            rho = [[-(-k * (j + 1) // stages) for j in range(stages - 1)] for k in mix.ctx.lens()]
            for flags in (0, B.MT_SCHED_PARALLEL_ISSUE | B.MT_SCHED_HOST_BARRIER, B.MT_SCHED_TIME_TENANTS):
                s = mix.ctx.schedule(rho, stages, flags=flags)
                for _ in range(2):
                    got, tm = mix.run(s)                     # other output buffers every time
                    assert same(got, ref) and tm["n_launches"] == sum(mix.ctx.lens())
                    assert abs(sum(tm["stage_ms"]) - tm["makespan_ms"]) < 1e-3
                if flags & B.MT_SCHED_TIME_TENANTS:
                    assert all(0 < d <= tm["makespan_ms"] + 1e-3 for d in tm["tenant_done_ms"])
    finally:
        mix.close()


def test_a_pass_of_more_packets_than_a_queue_holds():
    mix = Mix([chain(300) for _ in range(15)], 32)            # 4500 packets on one queue of 4096
    try:
        ref, _ = mix.run(mix.ctx.all_concurrent())
        got, _ = mix.run(mix.ctx.sequential())
        assert same(got, ref)
    finally:
        mix.close()


def test_equal_shares_and_shares_per_stage_get_their_own_queues():
    mix = Mix([zoo.BUILDERS["tinyC"]("f16", 2) for _ in range(3)], 33, "uniform")
    try:
        ref, _ = mix.run(mix.ctx.sequential())
        rho = [[3], [4], [5]]
        for share in ([128, 128, 128], [[64, 0, 64], [64, 32, 0]]):
            s = mix.ctx.schedule(rho, 2, cu_share=share)
            again = mix.ctx.schedule(rho, 2, cu_share=share)  # the same set of queues
            for k in (s, again, s):
                assert same(mix.run(k)[0], ref)
            s.close()
            again.close()
        mix.ctx.release_idle_streams()
        assert same(mix.run(mix.ctx.all_concurrent())[0], ref)
    finally:
        mix.close()


def test_two_contexts_on_two_threads_share_the_lanes():
    mixes = [Mix([zoo.BUILDERS[n]("f16", 2) for n in ("tinyA", "tinyC", "tinyD", "tinyB", "tinyA")], 34 + k, "uniform") for k in range(2)]
    refs = [m.run(m.ctx.sequential())[0] for m in mixes]
    bad = []

    def work(k):
        m = mixes[k]
        rho = [[-(-n // 2)] for n in m.ctx.lens()]
        scheds = [m.ctx.schedule(rho, 2), m.ctx.all_concurrent()]
        for i in range(40):
            if not same(m.run(scheds[i % 2])[0], refs[k]):
                bad.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not bad and not any(t.is_alive() for t in threads)
    for m in mixes:
        m.close()


@pytest.mark.parametrize("static", [False, True])
def test_a_pass_beside_a_capture_and_after_work_on_the_default_stream(static):
    import torch
    mix = Mix([zoo.BUILDERS["tinyC"]("f16", 2), zoo.BUILDERS["tinyA"]("f16", 1)], 36, "uniform")
    try:
        ref, _ = mix.run(mix.ctx.sequential())
        run = mix.ctx.run_static_scratch if static else mix.ctx.run
        sched = mix.ctx.all_concurrent()
        outs = [mix.ctx.make_output(t) for t in range(2)]
        # the caller captures work of its own: the pass neither joins the graph nor breaks the capture
        a = torch.arange(64, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            torch.mul(a, 2.0, out=b)
            run(sched, mix.inputs, outs)
        assert same([mix.ctx.output_to_numpy(t, o) for t, o in enumerate(outs)], ref)
        for k in range(3):
            a.add_(1.0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(b, 2.0 * a)
        # the inputs arrive behind a long fill on the default stream, the outputs are poisoned there
        big = torch.empty(1 << 28, dtype=torch.float32, device="cuda")
        late = [torch.zeros_like(x) for x in mix.inputs]
        run(sched, late, outs)
        for k in range(4):
            big.fill_(float(k))
        for x, y in zip(late, mix.inputs):
            x.copy_(y)
        for o in outs:
            o.fill_(float("nan"))
        run(sched, late, outs)
        assert same([mix.ctx.output_to_numpy(t, o) for t, o in enumerate(outs)], ref)
    finally:
        mix.close()


def test_library_whose_file_is_gone_since_it_was_loaded(tmp_path):
    """The kernels named in packets come from the loaded library, not from its file: an installation may be replaced under a
    running program."""
    lib = str(tmp_path / "libmtsched_copy.so")
    shutil.copy(B._build.lib_path(), lib)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    prog = """
import os, sys
sys.path[:0] = [%r, %r]
import torch
from paper_2111_14255_amd import binding as B
B.load()
os.unlink(%r)
from synth import zoo
from gpu_harness import Mix, assert_close
mix = Mix([zoo.BUILDERS["tinyC"]("f16", 1)], seed=3)
got, _ = mix.run(mix.ctx.sequential())
assert_close(got[0], mix.oracle()[0], "f16")
mix.close()
print("ran without the file")
""" % (root, os.path.join(root, "tests"), lib)
    r = subprocess.run([sys.executable, "-c", prog], env=dict(os.environ, MTSCHED_LIB=lib), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "ran without the file" in r.stdout, r.stdout + r.stderr
