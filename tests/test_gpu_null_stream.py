"""The workspace that the null stream keeps between calls of sgemm_cube and
sgemm_cube_hgemm: calls queued back to back with sizes that grow and shrink
(nothing waits between them), and from several host threads at once, each give
the bits of sgemm_cube_ws with a workspace of its own.  In child processes
(tests/kept_workspace_child.py): what calls on other streams do to it when
memory has run out, and when another thread has a capture open."""
import os
import subprocess
import sys
import threading

import pytest

import workloads
from tests.gpu_util import log, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(300, 200, 1000), (33, 17, 64), (700, 900, 1100), (129, 130, 65), (1500, 1400, 300)]


def _operands():
    out = []
    for i, (M, N, K) in enumerate(SHAPES):
        A, B = workloads.make_operands(M, N, K, 60 + i, "normal")
        out.append((to_dev(A), to_dev(B)))
    return out


def test_queued_calls_of_changing_sizes(gpu):
    import torch

    from paper_2507_23387_amd import binding

    ops = _operands()
    want = [binding.matmul(a, b, workspace=binding.workspace(a.shape[0], b.shape[1], a.shape[1]))
            for a, b in ops]
    torch.cuda.synchronize()
    log("null stream: queued calls")
    assert torch.cuda.current_stream().cuda_stream == 0
    order = [0, 1, 2, 3, 4, 4, 3, 2, 1, 0, 2, 1, 4]
    got = []
    for i in order:
        got.append(binding.matmul(*ops[i]))
        binding.hgemm(*ops[i])
    torch.cuda.synchronize()
    for i, c in zip(order, got):
        assert torch.equal(c.view(torch.int32), want[i].view(torch.int32)), SHAPES[i]


def test_threads_on_the_null_stream(gpu):
    import torch

    from paper_2507_23387_amd import binding

    ops = _operands()
    want = [binding.matmul(a, b, workspace=binding.workspace(a.shape[0], b.shape[1], a.shape[1]))
            for a, b in ops]
    torch.cuda.synchronize()
    log("null stream: five host threads")
    got = [[] for _ in ops]

    def work(i):
        torch.cuda.set_device(0)
        for _ in range(20):
            got[i].append(binding.matmul(*ops[i]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(ops))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i, cs in enumerate(got):
        assert len(cs) == 20
        for c in cs:
            assert torch.equal(c.view(torch.int32), want[i].view(torch.int32)), SHAPES[i]


@pytest.mark.parametrize("scenario", ["memory", "capture", "capture_blocking"])
def test_kept_workspace_and_other_streams(gpu, scenario):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    log(f"kept workspace: {scenario} (child process)")
    r = subprocess.run([sys.executable, "-u", os.path.join(root, "tests", "kept_workspace_child.py"),
                        scenario], capture_output=True, text=True, timeout=100, cwd=root)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert r.stdout.strip().endswith("ok")
