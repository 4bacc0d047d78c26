"""Builds and loads tests/lds_fill.hip (see there)."""
import ctypes as C
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "lds_fill.hip")
LIB = os.path.join(HERE, "liblds_fill.so")


def build(force: bool = False) -> str:
    if force or not os.path.exists(LIB):
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                        "-o", LIB, SRC], check=True, stderr=subprocess.DEVNULL)
    return LIB


def load():
    """fill(word): every LDS word of the current GPU holds `word` afterwards (on the current torch stream)."""
    import torch
    fn = C.CDLL(build()).lds_fill
    fn.argtypes = [C.c_uint, C.c_void_p]

    def fill(word: int):
        assert fn(word, torch.cuda.current_stream().cuda_stream) == 0
    return fill
