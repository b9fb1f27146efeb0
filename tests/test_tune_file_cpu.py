"""A saved tuning file: entries behind its format line are used as they are; of a
file without one, those chosen among fewer forms are left out, unless tuning is
off and nothing would replace them."""
import os
import subprocess
import sys

import pytest

from paper_2307_00391_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

OLD = ["batchform/c64/4.8x16 1", "fused/c64/25/0123456789abcdef 13 4 4", "fused/c64/26/0123456789abcdef 13 4",
       "cgemm/c64/1024/256/256/0 1", "eigpipe/c64/8/9 6 256 6 512 5 256"]
KEPT = ["batchform/c64/5.9x16 0", "fused/c64/25/00000000000000aa 13 4 1", "fused/c64/25/00000000000000bb 13 4 4 1",
        "cgemm/c64/512/256/256/0 3", "eigpipe/c64/8/10 6 256 6 512 0 0"]


def _loaded(path, **env):
    code = ("from paper_2307_00391_amd import binding as B\n"
            "B.sv_tune_set('probe/x', [1])\n"
            "print(B.sv_tune_report())\n")
    e = dict(os.environ, SV_TUNE_CACHE=str(path), **env)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=e, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return set(ln for ln in r.stdout.splitlines() if ln and not ln.startswith("probe/"))


@pytest.mark.parametrize("head,env,want", [("", {}, KEPT), ("", {"SV_AUTOTUNE": "0"}, OLD + KEPT), ("format 2\n", {}, OLD + KEPT)])
def test_entries_of_a_file(tmp_path, head, env, want):
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("libsv.so not built")
    f = tmp_path / "tune.txt"
    f.write_text(head + "\n".join(OLD + KEPT) + "\n")
    assert _loaded(f, **env) == set(want)


@pytest.mark.gpu
def test_written_file_carries_the_line_and_is_read_back(tmp_path):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = tmp_path / "tune.txt"
    code = ("import torch\n"
            "from paper_2307_00391_amd import binding as B\n"
            "s = B.State(12, 'c64')\n"
            "B.sv_init_basis(s.h, 0)\n"
            "B.sv_apply_ctrl_unitary(s.h, torch.eye(16, dtype=torch.complex64, device='cuda'), 0, 4, 11)\n"
            "print(B.sv_tune_report())\n")
    e = dict(os.environ, SV_TUNE_CACHE=str(f))
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=e, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    lines = f.read_text().splitlines()
    assert lines[0] == "format 2"
    assert set(lines[1:]) == set(ln for ln in r.stdout.splitlines() if ln.startswith("cgemm/")) == _loaded(f)
