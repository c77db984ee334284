"""Registers of the initial-score kernels: compiled for gfx950, none of them spills to
scratch memory (a spill in the chunk pass costs every tile of every chunk)."""
import re
import subprocess

from paper_2608_05326_amd import build as b


def test_initial_score_kernels_do_not_spill(tmp_path):
    cmd = [b._hipcc(), "-c", "-x", "hip", f"{b.CSRC}/prefill_scores.hip", "-o", str(tmp_path / "ps.o"),
           "--offload-device-only", "-Rpass-analysis=kernel-resource-usage"] + b.FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(scratch) and sum("k_obs_chunks" in n for n in names) == 4
    assert not {n: x for n, x in zip(names, scratch) if x}
