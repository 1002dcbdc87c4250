"""A program that uses the package without importing torch itself."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import numpy as np
import paper_1612_09368_amd as cm
with cm.Graph() as g:
    g.load(3, np.array([0, 1], np.int32), np.array([1, 2], np.int32))
    s, d = g.export_edges()
    assert sorted(zip(s.tolist(), d.tolist())) == [(0, 1), (1, 2)]
print("import order: ok")
"""


def test_a_graph_without_an_import_of_torch():
    out = subprocess.run([sys.executable, "-c", CHILD], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                         capture_output=True, text=True, timeout=110)
    assert out.returncode == 0, (out.stdout[-1000:], out.stderr[-2000:])
    assert "import order: ok" in out.stdout
