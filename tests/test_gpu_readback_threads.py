"""Reading fields back keeps to the OpenMP threads that the caller allows, and
many threads may read at once."""
import os
import subprocess
import sys

import numpy as np
import pytest

from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import os, sys
sys.path.insert(0, {root!r})
import numpy as np
from paper_2605_25403_amd import ipcs as I
m, s = I.Mesh.unit_square(384), I.Mesh.unit_square(16)
r, q = I.Run(m), I.Run(s)
for x in (r, q):
    x.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))
q.velocity()
count = lambda: len(os.listdir("/proc/self/task"))
a = count()
r.velocity()
print("threads", a, count())
"""


def test_one_allowed_thread_reads_alone():
    require_gpu()
    print("read back with OMP_NUM_THREADS=1", flush=True)
    c = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT)], capture_output=True,
                       text=True, timeout=100, env=dict(os.environ, OMP_NUM_THREADS="1"))
    print(c.stdout, flush=True)
    assert c.returncode == 0, c.stderr[-2000:]
    a, b = [w for w in c.stdout.split() if w.isdigit()]
    assert a == b


def test_more_readers_at_once_than_pinned_buffers():
    """Nine threads read fields of several chunks from runs on streams of their
    own, again and again; every value is the one that was set."""
    torch, I = require_gpu()
    import threading
    print("read back by nine threads", flush=True)
    m = I.Mesh.unit_square(400)
    runs, sets = [], []
    for k in range(9):
        r = I.Run(m, I.ipcs_params_default(), stream=torch.cuda.Stream())
        rng = np.random.default_rng(k)
        u, p = rng.standard_normal((2, r.n2)), rng.standard_normal(r.n1)
        r.set_state(u, p, 0.0)
        runs.append(r)
        sets.append((u, p))
    wrong, go = [], threading.Barrier(len(runs))

    def read(k):
        try:
            go.wait(60)
            for _ in range(5):
                if not (np.array_equal(runs[k].velocity(), sets[k][0]) and
                        np.array_equal(runs[k].pressure(), sets[k][1])):
                    wrong.append(k)
        except Exception as e:   # noqa: BLE001 (reported below)
            wrong.append((k, e))

    ts = [threading.Thread(target=read, args=(k,)) for k in range(len(runs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not wrong, wrong
