"""The host runtime on the CPU, over a stand-in for the HIP runtime: what it
allocates, captures, launches and refuses (tests/runtime_check.cpp).  And the
binding's objects over a stand-in for the library: what keeps what alive."""
import ctypes
import gc
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2008_10596_amd import ckpt as K

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_10596_amd", "csrc")
HIP = "/opt/rocm/include"


@pytest.fixture(scope="module")
def runtime_check(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP, "hip")):
        pytest.skip("no g++ or no HIP headers")
    exe = str(tmp_path_factory.mktemp("runtime") / "runtime_check")
    sources = [os.path.join(ROOT, "tests", "runtime_check.cpp")]
    sources += [os.path.join(CSRC, f) for f in ("runtime.cpp", "noalloc.cpp", "server.cpp", "crc_tables.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-D__align__(x)=__attribute__((aligned(x)))", "-DHIP_SYMBOL(x)=((const void*)&(x))",
                    "-I", HIP, "-I", os.path.join(ROOT, "include"), "-I", CSRC, *sources,
                    "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("what", ["dense", "graph", "link", "capture", "server"])
def test_host_runtime(runtime_check, what):
    r = subprocess.run([runtime_check, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "all checks held" in r.stdout, r.stdout + r.stderr


class StandIn:
    """Counts what is open; an image's sections lie in memory of its own."""

    def __init__(self):
        self.open, self.made, self.memory = set(), 0, {}

    def __getattr__(self, name):
        raise AssertionError("unexpected call: " + name)

    def _new(self, out):
        self.made += 1
        self.open.add(self.made)
        out._obj.value = self.made
        return 0

    def ckpt_init(self, cfg, out):
        return self._new(out)

    def ckpt_checkpoint(self, ctx, stream, mode, base, out):
        return self._new(out)

    def ckpt_checkpoint_batch(self, ctxs, n, stream, outs):
        for i in range(n):
            self.made += 1
            self.open.add(self.made)
            outs[i] = self.made
        return 0

    def ckpt_destroy(self, h):
        self.open.remove(h)

    def ckpt_image_free(self, h):
        self.open.remove(h)

    def ckpt_image_view(self, h, section, p, n):
        buf = self.memory.setdefault((h, section), ctypes.create_string_buffer(64))
        p._obj.value, n._obj.value = ctypes.addressof(buf), 64
        return 0


@pytest.fixture
def stand_in(monkeypatch):
    s = StandIn()
    monkeypatch.setattr(K, "_lib", s)
    yield s
    gc.collect()


def test_snapshots_keep_their_context(stand_in):
    """A snapshot's dense image lies in its context's memory: the image keeps
    the context.  The address that it gives out keeps neither."""
    ctx = K.Context(flags=K.CKPT_NO_DRAIN)
    img = ctx.checkpoint()
    del ctx
    gc.collect()
    assert stand_in.open == {1, 2}
    ptr, n = img.dense_ptr
    assert type(ptr) is int and ptr == ctypes.addressof(stand_in.memory[2, K.CKPT_SEC_DENSE]) and n == 64
    raw = dict(data=(ptr, False))        # as an array interface holds it
    del img
    assert stand_in.open == set() and raw


def test_host_views_keep_their_image(stand_in):
    """A section's array, and what is made of it, keeps the image that holds
    its memory."""
    ctx = K.Context()
    crc = ctx.checkpoint().crc
    part = crc[4:8].view(np.uint8)
    del crc
    gc.collect()
    assert stand_in.open == {1, 2} and part.base is not None
    del part
    gc.collect()
    assert stand_in.open == {1}
    ctx.close()


def test_batch_images_keep_the_first_context(stand_in):
    ctxs = [K.Context(flags=K.CKPT_NO_DRAIN), K.Context(flags=K.CKPT_NO_DRAIN)]
    a, b = K.checkpoint_batch(ctxs)
    del ctxs
    gc.collect()
    assert stand_in.open == {1, 3, 4}
    a.close()
    assert stand_in.open == {1, 4}
    del a, b
    gc.collect()
    assert stand_in.open == set()


def test_drained_images_do_not_keep_their_context(stand_in):
    img = K.Context().checkpoint()
    gc.collect()
    assert stand_in.open == {2}
    img.close()
    assert stand_in.open == set()
