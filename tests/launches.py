"""The launches of a call on a machine without a GPU: the library in a process of its own, with launch_recorder.c in the place of the HIP
runtime's launch functions.  No pointer of the call is followed."""
import ctypes
import json
import os
import subprocess
import sys

from paper_2509_18467_amd import lawcat

_SOURCE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_recorder.c")
_CHILD = """
import ctypes, json, sys
recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the library: its calls find these functions first
library = ctypes.CDLL(sys.argv[2])
recorded = (ctypes.c_uint * 320).in_dll(recorder, "launches")
count = ctypes.c_int.in_dll(recorder, "n_launches")
out = []
for name, args in json.load(sys.stdin):
    values = []
    for kind, v in args:
        values.append(ctypes.create_string_buffer(bytes.fromhex(v)) if kind == "bytes" else ctypes.c_size_t(v) if kind == "size" else ctypes.c_void_p(v))
    count.value = 0
    status = getattr(library, name)(*values)
    out.append([status, [[recorded[5 * i], recorded[5 * i + 1], recorded[5 * i + 2], recorded[5 * i + 3]] for i in range(count.value)]])
print(json.dumps(out))
"""

AT = ("pointer", 0x10000)
NULL = ("pointer", None)


def desc(d):
    return "bytes", bytes(d).hex()


def offsets(starts):
    return "bytes", bytes((ctypes.c_int32 * len(starts))(*starts)).hex()


def size(n):
    return "size", n


def prefill(d, workspace, room, state=NULL):
    """Arguments of lawcat_layer_prefill"""
    return "lawcat_layer_prefill", [desc(d), AT, AT, AT, AT, AT, AT, state, state, NULL, NULL, AT, NULL, ("pointer", 0x20000), ("pointer", 0x30000), NULL, NULL,
                                    workspace, size(room), NULL]


def static(d):
    return "lawcat_layer_prefill_static", [desc(d), AT, AT, AT, AT, AT, AT, NULL, NULL, NULL, NULL, AT, NULL, AT, AT, NULL, NULL, NULL]


def packed(d, starts, workspace, room, one_launch=True):
    return "lawcat_layer_prefill_varlen", [desc(d), offsets(starts), AT if one_launch else NULL, AT, AT, AT, AT, AT, AT, NULL, NULL, NULL, NULL, AT, NULL, AT, AT,
                                           NULL, NULL, workspace, size(room), NULL]


def conv_adjoint(d, heads, workspace, room):
    """Arguments of lawcat_conv1d_backward"""
    return "lawcat_conv1d_backward", [desc(d), ("pointer", heads), AT, AT, NULL, AT, AT, AT, NULL, workspace, size(room), NULL]


def run(calls, directory):
    """[(status, [(grid x, grid y, grid z, threads)])] of the calls"""
    recorder = os.path.join(directory, "launch_recorder.so")
    if not os.path.exists(recorder):
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", _SOURCE, "-o", recorder], check=True)
    done = subprocess.run([sys.executable, "-c", _CHILD, recorder, lawcat.LIB_PATH], input=json.dumps(calls), capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    return [(status, [tuple(x) for x in launches]) for status, launches in json.loads(done.stdout)]
