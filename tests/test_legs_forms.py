"""The forms of the fused legs that the library holds are those that it can launch (no GPU)."""
import re
import subprocess

from paper_2001_02327_amd import _lib


def _symbols():
    return subprocess.run(["nm", "-C", _lib.LIB_PATH], capture_output=True, text=True, check=True).stdout


def test_no_form_without_a_caller():
    """FP32 has legs for coarse levels (boundary rule) in every form, and for multigrid level 0 streamed ones with a
    single post-smoothing sweep: no launcher takes another combination, no kernel exists for one."""
    syms = _symbols()
    for name in ("launch_level_down", "launch_level_up", "launch_stream_down", "launch_stream_up", "launch_tile2_down",
                 "launch_tile2_up"):
        sig = re.findall(r"np::%s<float>\((.*)\)" % name, syms)
        assert sig and not any("bool" in s for s in sig), name  # (which one of the two it is, is no argument)
    assert not re.search(r"k_tile_(down|up)3<float, \d, false", syms)
    assert not re.search(r"k_tile2<float, \d, false", syms)
    up = set(re.findall(r"k_leg3<float, (\d), (\d), true", syms))
    assert up == {("1", "0"), ("2", "0"), ("1", "1")}  # sweeps; boundary rule or level 0
