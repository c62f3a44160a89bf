"""A pd_video_push that fails part of the way leaves its slot free; what it had
enqueued must be over before the slot is used again.  The host code runs against
a pretended HIP runtime in which each call of a push fails in turn (no GPU)."""
import os
import subprocess

from paper_1611_01642_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_failed_push_leaves_nothing_running(tmp_path):
    objs = []
    for src in (os.path.join(build.CSRC, "video.hip"), os.path.join(HERE, "failed_push.cpp")):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fPIC",
                        "-I", build.CSRC, "-c", src, "-o", obj], check=True, capture_output=True, timeout=300)
        objs.append(obj)
    exe = str(tmp_path / "failed_push")
    subprocess.run(["g++", *objs, "-o", exe], check=True, capture_output=True, timeout=120)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
