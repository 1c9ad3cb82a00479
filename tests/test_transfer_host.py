"""Field transfers on the host alone: csrc/transfer.hip built against HIP calls
that fail on demand (transfer_host.cpp); every failure must be reported."""
import os
import subprocess

from paper_2308_08085_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_failure_is_reported(tmp_path):
    objs = []
    for src in (os.path.join(build.CSRC, "transfer.hip"), os.path.join(HERE, "transfer_host.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIE", "-I", build.CSRC,
                        "-c", src, "-o", objs[-1]], check=True, capture_output=True)
    exe = str(tmp_path / "transfer_host")
    subprocess.run(["g++", "-o", exe] + objs + ["-pthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-1000:]
