"""The suites of the streaming legs, of the forms a cycle takes by its sizes, and of the lexicographic fronts against the
LDS-poison build (see test_gpu_lds_poison.py): LDS read before it is written turns a result into NaN."""

import os
import subprocess
import sys

import pytest

from gpu_util import note
from test_gpu_lds_poison import POISON_LIB, ROOT

pytestmark = pytest.mark.gpu

SUITES = ["tests/test_gpu_stream.py", "tests/test_gpu_cycle_forms.py"]


def test_cycle_forms_pass_with_poisoned_lds():
    note("lds poison build: cycle forms in a child process")
    assert os.path.exists(POISON_LIB), f"{POISON_LIB} is missing: build it with __graft_entry__.build()"
    cmd = [sys.executable, "-u", "-m", "pytest", "-x", "-q", "-m", "gpu", "-p", "no:cacheprovider", "--timeout", "300",
           "--timeout-method", "thread", *SUITES]
    r = subprocess.run(cmd, cwd=ROOT, env=dict(os.environ, SGBT_LIBRARY=POISON_LIB), capture_output=True, text=True,
                       timeout=900)
    tail = "\n".join((r.stdout + r.stderr).splitlines()[-30:])
    print(tail, flush=True)
    assert r.returncode == 0, tail
    assert " passed" in r.stdout and "failed" not in r.stdout, tail
