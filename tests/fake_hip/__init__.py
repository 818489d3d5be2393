"""Runs code against the library's host side with a stand-in for the HIP runtime (no GPU, no kernel runs)."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

PRELUDE = """
import ctypes, sys
sys.path.insert(0, %r)
fake = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)   # in front of the real runtime for what is loaded from here on
fake.fake_launches.restype, fake.fake_launches.argtypes = ctypes.c_int64, [ctypes.c_char_p, ctypes.c_void_p]
fake.fake_blocks.restype, fake.fake_blocks.argtypes = ctypes.c_uint64, [ctypes.c_char_p]
fake.fake_calls.restype, fake.fake_calls.argtypes = ctypes.c_int64, [ctypes.c_char_p]
fake.fake_new_limit.argtypes = [ctypes.c_int64]
fake.fake_host_bytes.restype = fake.fake_mallocs_on.restype = fake.fake_races.restype = ctypes.c_int64
import numpy as np
import paper_1610_02496_amd as pk

def launches(name):
    '''launches so far of kernels whose name contains `name`, their workgroups, threads of the largest of them'''
    most = ctypes.c_uint64()
    n = fake.fake_launches(name.encode(), ctypes.addressof(most))
    return n, fake.fake_blocks(name.encode()), most.value

def races():
    '''accesses to the buffers of streamed chunks so far that nothing puts in order, and the first one'''
    first = ctypes.create_string_buffer(200)
    return fake.fake_races(first, ctypes.c_int64(200)), first.value.decode()

def code_of(call):
    '''status code of a call of the binding'''
    try:
        call()
    except pk.SaberError as e:
        return e.code
    return 0
"""


def build(folder):
    lib = os.path.join(str(folder), "libfake_hip.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "fake_hip.cpp")])
    return lib


def run(lib, code, timeout=300):
    """Runs `code` in a process of its own (the stand-in is process-wide); its failed assertion fails the test."""
    p = subprocess.run([sys.executable, "-c", PRELUDE % (ROOT, lib) + textwrap.dedent(code)], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=timeout, cwd=ROOT)
    assert p.returncode == 0, p.stdout[-4000:]
