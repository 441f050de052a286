"""The library's host code on a machine without a GPU: libplbm built for the
host only and linked against a HIP runtime that records launches instead of
making them (recorder/hip_recorder.cpp)."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

from paper_1402_5487_amd import _plbm, build

HERE = os.path.dirname(os.path.abspath(__file__))


class Launch:
    def __init__(self, lib, i):
        grid, block, lds = ctypes.c_uint(), ctypes.c_uint(), ctypes.c_size_t()
        src, dst, extra = ctypes.c_void_p(), ctypes.c_void_p(), (ctypes.c_int * 7)()
        lib.rec_launch(i, *map(ctypes.byref, (grid, block, lds, src, dst)), extra)
        self.name = lib.rec_name(i).decode()
        # the kernel's own name out of the mangled one: _ZN12_GLOBAL__N_16k_tile..
        m = re.search(r"\d(k_[a-z0-9_]+?)(?=I|E|P|$)", self.name)
        self.kernel = m.group(1) if m else self.name
        self.grid, self.block, self.lds = grid.value, block.value, lds.value
        self.src, self.dst, self.extra = src.value, dst.value, list(extra)


class Recorder:
    def __init__(self, path):
        self.lib = lib = ctypes.CDLL(path)
        lib.rec_name.restype = ctypes.c_char_p
        lib.rec_bytes.restype = ctypes.c_longlong
        lib.rec_allow_mallocs.argtypes = [ctypes.c_longlong]
        P, vp, D = ctypes.POINTER(_plbm.PlbmDesc), ctypes.c_void_p, ctypes.POINTER(ctypes.c_double)
        for f in (lib.plbm_step, lib.plbm_advance, lib.plbm_step_noalloc):
            f.argtypes = [P, vp, vp, ctypes.c_int, D, vp]
        lib.plbm_step_fields.argtypes = [P, vp, vp, ctypes.c_int, vp, vp, vp, vp, vp]
        _plbm._setup_batch(lib)

    def launches(self):
        out = [Launch(self.lib, i) for i in range(self.lib.rec_count())]
        self.lib.rec_clear()
        return out

    def step(self, d, n, entry="plbm_step", sums=False):
        """The launches of n steps from buffer 0x1000 to 0x2000 and on."""
        self.lib.rec_clear()
        s = (ctypes.c_double * 5)() if sums else None
        rc = getattr(self.lib, entry)(ctypes.byref(d), 0x1000, 0x2000, n, s, None)
        assert rc == _plbm.PLBM_OK, (entry, rc)
        return self.launches()


def build_recorder(folder):
    if not (shutil.which(build.HIPCC) or os.path.exists(build.HIPCC)):
        pytest.skip("hipcc not available")
    flags = ["-O1", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip",
             "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC]
    srcs = [os.path.join(build.CSRC, s) for s in build.SOURCES] + [os.path.join(HERE, "recorder", "hip_recorder.cpp")]
    objs = [os.path.join(folder, os.path.basename(s) + ".o") for s in srcs]
    procs = [subprocess.Popen([build.HIPCC, *flags, "-c", s, "-o", o], stderr=subprocess.PIPE) for s, o in zip(srcs, objs)]
    for p in procs:
        err = p.communicate()[1]
        assert p.returncode == 0, err.decode()[-2000:]
    # the device code that a host-only build leaves out
    syms = subprocess.run(["nm", *objs], capture_output=True, text=True, check=True).stdout
    fat = sorted(set(re.findall(r"U (__hip_fatbin_\w+)", syms)))
    out = os.path.join(folder, "librecord.so")
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *[f"-Wl,--defsym={f}=0" for f in fat], *objs, "-o", out,
                    "-lpthread"], check=True)
    return Recorder(out)


@pytest.fixture(scope="session")
def recorder(tmp_path_factory):
    return build_recorder(str(tmp_path_factory.mktemp("recorder")))
