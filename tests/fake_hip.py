"""libdz's host side on a HIP runtime without a GPU (fake_hip.cpp): which kernels a call launches, with what memory.
Has to be used in a process of its own that has loaded no other HIP library: see `run`."""
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIBDZ = os.path.join(os.path.dirname(HERE), "paper_2312_05215_amd", "libdz.so")
SPLIT_K, WIDE_TILE, REUSE_SEGMENTS = 1, 5, 6        # option keys of include/dz.h
STREAM = ctypes.c_void_p(0x30000)                  # (the default stream cannot be captured)


def run(test_file, scenario, tmp_path, data=None):
    """Call function `scenario` of `test_file` in a new process, with the fake runtime built under `tmp_path`."""
    so = os.path.join(str(tmp_path), "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.cpp")], check=True)
    p = subprocess.run([sys.executable, test_file, scenario], env=dict(os.environ, FAKE_HIP=so, FAKE_HIP_DATA=json.dumps(data)), text=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=120)
    assert p.returncode == 0, p.stdout


def data():
    return json.loads(os.environ["FAKE_HIP_DATA"])


def static_lds(kernel):
    """LDS bytes that the compiler gave kernels of this name in libdz.so, from the metadata of their code objects."""
    import msgpack
    data, at, found = open(LIBDZ, "rb").read(), 0, set()
    while (at := data.find(b"AMDGPU\0\0", at + 1)) >= 0:      # ELF note: name size, size, type 32, name, contents
        if data[at - 12:at - 8] == (7).to_bytes(4, "little") and data[at - 4:at] == (32).to_bytes(4, "little"):
            size = int.from_bytes(data[at - 8:at - 4], "little")
            for k in msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"]:
                if kernel in k[".name"]:
                    found.add(k[".group_segment_fixed_size"])
    assert found, kernel
    return max(found)


class Sim:
    """One context on the fake runtime.  Addresses are made up: nothing is ever read through them."""

    def __init__(self, libdz=None):
        self.fake = ctypes.CDLL(os.environ["FAKE_HIP"], mode=ctypes.RTLD_GLOBAL)
        self.fake.fake_name.restype = ctypes.c_char_p
        for f in ("fake_room", "fake_capture"):
            getattr(self.fake, f).argtypes = [ctypes.c_uint64]
        for f in ("fake_lds", "fake_live_bytes"):
            getattr(self.fake, f).restype = ctypes.c_size_t
        self.dz = ctypes.CDLL(libdz or LIBDZ)
        self.dz.dz_last_hip_error.restype = ctypes.c_char_p
        self.ctx = ctypes.c_void_p()
        assert self.dz.dz_create(ctypes.byref(self.ctx), 0) == 0

    def option(self, key, value):
        assert self.dz.dz_set_option(self.ctx, key, value) == 0

    def capture(self, ident):
        self.fake.fake_capture(ident)

    def room(self, more):
        """From now on `more` bytes can be allocated."""
        self.fake.fake_room(self.fake.fake_live_bytes() + more)

    def launches(self):
        """[(kernel, workgroups, dynamic LDS, watched argument)] since the last time, and forget them."""
        out = []
        for i in range(self.fake.fake_launches()):
            name = self.fake.fake_name(i).decode()
            short = next(k for k in ("segment_kernel", "fused_list_kernel", "fused_kernel", "prefill_kernel", "tile_kernel", "stream_kernel", "shrink", "expand",
                                     "clear", "") if k in name)
            out.append((short or name, self.fake.fake_grid(i), self.fake.fake_lds(i), self.fake.fake_watched(i)))
        self.fake.fake_clear()
        return out

    def kernels(self):
        return [l[0] for l in self.launches()]

    def segment(self, T, D):
        return self.dz.dz_segment(self.ctx, ctypes.c_void_p(0x10000), T, D, None, None, None, STREAM)

    def linear(self, Ns, K, D, T, bits=4, group=128, ids=0x10000):
        P = len(Ns)
        W = (ctypes.c_void_p * P)(*[0x1000000 * (p + 1) for p in range(P)])
        out = (ctypes.c_void_p * P)(*[0x9000000 + 0x1000000 * p for p in range(P)])
        deltas = (ctypes.c_void_p * max(P * D, 1))(*[0x100000000 + 0x1000000 * m for m in range(P * D)])
        return self.dz.dz_linear_group(self.ctx, ctypes.c_void_p(0x20000), P, W, deltas, D, ctypes.c_void_p(ids), out,
                                       (ctypes.c_int * P)(*Ns), T, K, bits, group, STREAM)

    def lora(self, T, rank=8):
        one = (ctypes.c_void_p * 1)(0x40000)
        return self.dz.dz_lora_sbmm(self.ctx, ctypes.c_void_p(0x20000), one, one, 1, rank, ctypes.c_void_p(0x10000),
                                    ctypes.c_void_p(0x50000), T, 16, 256, 0, STREAM)
