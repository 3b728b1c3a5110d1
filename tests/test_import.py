"""Importing the package takes neither torch nor the built library (python -m paper_2505_03254_amd.build has neither)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_import_without_torch():
    code = ("import sys; sys.modules['torch'] = None\n"
            "import paper_2505_03254_amd as P, paper_2505_03254_amd.build\n"
            "print(P.library_path())")
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    assert p.stdout.strip().endswith("libprom.so")
