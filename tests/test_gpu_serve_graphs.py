"""A server's captured graphs stay when the kernel's form changes with the systems that iterate."""

import os
import subprocess
import sys

import pytest

from paper_2105_06176_amd import ppcg
from test_gpu_serve_budget import HERE, counter, runtime  # noqa: F401 (counter: a fixture)

pytestmark = pytest.mark.gpu


def test_systems_with_runs_come_and_go(counter):  # noqa: F811
    """Twelve visits to a running system: two lengths of chunk in two forms, captured anew at most once when the table
    first grows (a capture per visit and one after it would be 24)."""
    ppcg.lib()
    r = subprocess.run([sys.executable, os.path.join(HERE, "serve_graphs_run.py"), counter, runtime()],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert int(r.stdout.split("GRAPHS")[1]) <= 8
