"""Which kernel a convolution call launches (route_probe.cpp): no GPU needed."""
import functools
import os
import re
import subprocess
import tempfile

from conftest import ROOT

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import build

_TYPES = {"rtoss::f16_t": "f16", "rtoss::bf16_t": "bf16", "float": "f32"}


@functools.lru_cache(None)
def _probe():
    exe = os.path.join(tempfile.mkdtemp(prefix="rtoss_routes_"), "route_probe")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-isystem", os.path.join(rocm, "include"),
                           "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "route_probe.cpp"), "-o", exe, "-rdynamic", build.LIB,
                           "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-ldl", "-Wl,-rpath," + build.HERE, "-Wl,-rpath," + os.path.join(rocm, "lib")])
    names = {}
    for line in subprocess.check_output(["nm", "-C", build.LIB], text=True).splitlines():
        m = re.match(r"([0-9a-f]+) . void rtoss::(?:\(anonymous namespace\)::)?(?!__device_stub__)(\w+)_kernel<(.*?)>\(", line)
        if m:
            args = [_TYPES.get(a, a) for a in m.group(3).split(", ")]
            names[int(m.group(1), 16)] = "%s<%s>" % (m.group(2), ",".join(args))
    return exe, names


def launches(calls):
    """calls: tuples (dt, N, Ci, Co, H, W, ksize, stride, k, rule, out_dt, fused, coherent).  Returns for each (kernel, dynamic LDS bytes,
    their limit), the kernel as 'conv3x3_strip<bf16,f32,3,0,true>' or the status of a call that was refused."""
    exe, names = _probe()
    text = "".join("%d %d %d %d %d %d %d  %d %d %d %d %d  %d\n" % (coherent, Co, Ci, ks, k, rule, dt, N, H, W, stride, out_dt, fused)
                   for dt, N, Ci, Co, H, W, ks, stride, k, rule, out_dt, fused, coherent in calls)
    out = []
    for line in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines():
        status, at, lds, limit = line.split()
        out.append((names[int(at, 16)] if int(status) == B.OK else int(status), int(lds), int(limit)))
    assert len(out) == len(calls)
    return out


def kernels(calls):
    return [kernel for kernel, lds, limit in launches(calls)]


def library_kernels(prefix):
    return [name for name in _probe()[1].values() if name.startswith(prefix)]
