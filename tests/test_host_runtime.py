"""The runtime's host side where several streams, processes, contexts or threads meet.  CPU only."""
import os
import shutil
import signal
import subprocess
import sys
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_08490_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")


def _compile(tmp_path, name, sources=("api.cpp", "host_build.cpp", "sampler.cpp")):
    """tests/sanitize/<name>.cpp with the host runtime and the launcher stand-ins, without device code."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / name)
    srcs = [os.path.join(CSRC, f) for f in sources] + [os.path.join(SAN, f) for f in ("launch_stubs.cpp", name + ".cpp")]
    cmd = [gxx, "-std=c++20", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, "-w", "-o", exe] + srcs + \
          ["-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return exe


def test_every_call_waits_for_an_upload_that_is_not_known_to_have_finished(tmp_path):
    """Two calls with one stream handle while the upload is under way: both wait (the handle of the per-thread stream, or of
    a stream made where another one was destroyed, is another stream the second time).  Once the upload has finished
    none waits, whatever the handle."""
    run = subprocess.run([_compile(tmp_path, "upload_wait")], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "upload wait ok" in run.stdout, run.stdout + run.stderr


FORK = '''
import os, sys
import numpy as np
sys.path.insert(0, %r)
from paper_2408_08490_amd import binding as B
from workloads import make_config, build_graph, sample_minibatch
cfg = make_config(0, scale=0.2, batch=8)
g = build_graph(cfg)
mb = sample_minibatch(cfg, g)

def build():
    ctx = B.Context(g.schema.rel_src, g.schema.rel_dst, g.schema.num_types, device=-1, host_threads=4)
    gr = ctx.hgnn_build_semantic_csr(mb.blocks)
    v = gr.host_view(0)
    gr.release()
    return ctx, v

parent, want = build()
pid = os.fork()
if pid == 0:
    ctx, got = build()
    ctx.close()
    parent.close()     # inherited: its threads are the parent's
    os._exit(0 if all(np.array_equal(got[k], want[k]) for k in ("rowptr", "colidx", "cptr", "crow")) else 3)
status = os.waitpid(pid, 0)[1]
again = build()        # the parent's own threads are as they were
print("fork ok" if status == 0 else "child: %%d" %% status)
'''


def test_a_forked_child_builds_with_threads_of_its_own():
    """A loader worker forked while the parent holds a context: its own host-only context builds, and the inherited one can
    be closed."""
    run = subprocess.Popen([sys.executable, "-c", FORK % ROOT], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                           start_new_session=True)
    try:
        out = run.communicate(timeout=60)[0]
    except subprocess.TimeoutExpired:
        os.killpg(run.pid, signal.SIGKILL)      # the child too
        pytest.fail("the child's build does not end")
    assert run.returncode == 0 and "fork ok" in out, out


def test_short_phases_do_not_wait_for_another_callers_long_ones(tmp_path):
    """A caller whose phase is over leaves at once, also when another caller's phase of 60 ms follows in the same place."""
    run = subprocess.run([_compile(tmp_path, "crew_phases")], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "crew phases ok" in run.stdout, run.stdout + run.stderr


def _contexts():
    """(context(threads, builders) of a small graph family, queue(context, n) = n builds of one mini-batch)"""
    from paper_2408_08490_amd import binding as B
    from workloads import build_graph, make_config, sample_minibatch
    cfg = make_config(2, scale=0.02, batch=64)
    g = build_graph(cfg)
    mb = sample_minibatch(cfg, g)

    def context(threads, builders):
        return B.Context(g.schema.rel_src, g.schema.rel_dst, g.schema.num_types, device=-1, host_threads=threads, concurrent_builds=builders)
    return context, lambda ctx, n: [ctx.hgnn_build_semantic_csr(mb.blocks) for _ in range(n)]


def test_a_context_does_not_wait_for_another_ones_queue():
    """Two builders' threads, 400 graphs queued by one context, one by another: that one is built between them."""
    context, queue = _contexts()
    a, b = context(2, 2), context(2, 2)
    graphs = queue(a, 400)
    t0 = time.perf_counter()
    one = queue(b, 1)
    one[0].wait()
    t_one = time.perf_counter() - t0
    graphs[-1].wait()
    t_all = time.perf_counter() - t0
    for g in graphs + one:
        g.release()
    a.close()
    b.close()
    assert t_one < t_all / 3, (t_one, t_all)


def test_closing_a_context_does_not_wait_for_another_ones_queue():
    """The crew gives back the threads that only the closed context asked for between two graphs of the other one's."""
    context, queue = _contexts()
    wide, b = context(8, 8), context(2, 2)
    own = queue(wide, 40)          # all eight threads have work, so that any of them may be the next to take some
    graphs = queue(b, 400)
    for g in own:
        g.release()
    t0 = time.perf_counter()
    wide.close()
    t_close = time.perf_counter() - t0
    graphs[-1].wait()
    t_all = time.perf_counter() - t0
    for g in graphs:
        g.release()
    b.close()
    assert t_close < t_all / 3, (t_close, t_all)


def test_of_several_bad_layers_the_first_is_reported():
    import numpy as np
    from paper_2408_08490_amd import binding as B
    from workloads import build_graph, make_config, sample_minibatch
    cfg = make_config(2, scale=0.02, batch=64)
    g = build_graph(cfg)
    mb = sample_minibatch(cfg, g)
    for b in mb.blocks:
        b.edge_type = np.array(b.edge_type)
    mb.blocks[0].edge_type[-1] = mb.blocks[1].edge_type[0] = 99     # the larger first layer's is found last
    ctx = B.Context(g.schema.rel_src, g.schema.rel_dst, g.schema.num_types, device=-1, host_threads=6)
    for _ in range(50):
        gr = ctx.hgnn_build_semantic_csr(mb.blocks, use_edge_id=False)
        with pytest.raises(B.HgnnError, match="layer 0: edge %d has type 99" % (len(mb.blocks[0].edge_type) - 1)):
            gr.wait()
        gr.release()
    ctx.close()


SPARSE = '''
import re, resource, sys
import numpy as np
sys.path.insert(0, %r)
from paper_2408_08490_amd import binding as B
R, N, E = 32, 65536, 3000
rng = np.random.default_rng(5)
indptr, nbr = [], []
for r in range(R):
    dst = np.sort(rng.integers(0, N, E))
    indptr.append(np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=N))]).astype(np.int64))
    nbr.append(rng.integers(0, N, E).astype(np.int32))
off = np.arange(R + 1, dtype=np.int64) * E

def sample(threads, targets):
    ctx = B.Context([0] * R, [0] * R, 1, device=-1, host_threads=threads)
    s = ctx.hgnn_sampler_create([N], indptr, nbr, off)
    gr = ctx.hgnn_sample_and_build(s, 0, targets, [64], 9, None)
    gr.wait()
    res = [gr.ids()[1][0], gr.host_view(0)["rowptr"], gr.host_view(0)["colidx"], gr.minibatch_view(0)["edge_id"]]
    gr.release()
    s.close()
    ctx.close()
    return res

sample(6, np.arange(64))
targets = np.arange(N)
want = sample(1, targets)
data = int(re.search(r"VmData:\\s+(\\d+) kB", open("/proc/self/status").read()).group(1)) << 10
resource.setrlimit(resource.RLIMIT_DATA, (data + (600 << 20),) * 2)     # 2.1 million merged rows of at most 64 edges, 96,000 edges
got = sample(6, targets)
print("sparse ok" if all(np.array_equal(a, b) for a, b in zip(got, want)) else "different")
'''


def test_sampling_on_several_threads_takes_room_for_the_edges_that_are_kept():
    """Many relations with an edge for few of their destinations, at the largest fan-out: as the one-thread path, the
    sampler's scratch goes with the edges and not with destinations times fan-out (1.6 GB here)."""
    run = subprocess.run([sys.executable, "-c", SPARSE % ROOT], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "sparse ok" in run.stdout, run.stdout + run.stderr


def test_a_failed_allocation_on_a_host_thread_is_an_error_of_that_graph(tmp_path):
    """Scratch that cannot grow, on one thread and on several, sampled or from lists: HGNN_ENOMEM, and the context goes on."""
    run = subprocess.run([_compile(tmp_path, "out_of_memory")], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "out of memory ok" in run.stdout, run.stdout + run.stderr


def test_the_crew_sleeps_between_builds():
    """A loop of a small build and 0.4 ms of something else keeps the crew's seven threads busy while it builds, not for
    good."""
    context, queue = _contexts()
    ctx = context(8, 1)

    def step():
        g = queue(ctx, 1)[0]
        g.wait()
        g.release()
        time.sleep(4e-4)
    for _ in range(20):
        step()
    t, c = time.perf_counter(), time.process_time()
    for _ in range(500):
        step()
    busy = (time.process_time() - c) / (time.perf_counter() - t)
    ctx.close()
    assert busy < 4.5, busy
