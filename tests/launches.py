"""What the library launches for given arguments, without a GPU: in a process of its own, launches.c stands in for the HIP
runtime, so the entry points check their arguments, choose a kernel and its grid, and nothing runs."""
import functools
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2412_04964_amd", "libfc.so")

_CHILD = """
import ctypes, json, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
for name, args in json.load(sys.stdin):
    f = getattr(L, name)
    print("R", f(*[ctypes.c_int64(a) for a in args]), flush=True)
"""


@functools.lru_cache(None)
def _stand_in():
    folder = tempfile.mkdtemp()
    lib = os.path.join(folder, "launches.so")
    subprocess.run([os.environ.get("CC", "gcc"), "-shared", "-fPIC", "-O1", "-o", lib, os.path.join(HERE, "launches.c")], check=True)
    return lib


def launches(calls):
    """calls: (entry point, integer arguments; pointers as addresses).  For each: (return code, [(kernel, workgroups, threads per
    workgroup, bytes of LDS asked for at the launch)]), the kernel as name<template arguments>, e.g. k_quantize<4,8,0,16,128>."""
    r = subprocess.run([sys.executable, "-c", _CHILD, _stand_in(), LIB], input=json.dumps(calls), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, seen = [], []
    for line in r.stdout.splitlines():
        if line.startswith("L "):
            _, name, grid, block, lds = line.split()
            seen.append((_readable(name), int(grid), int(block), int(lds)))
        elif line.startswith("R "):
            out.append((int(line[2:]), seen))
            seen = []
    assert len(out) == len(calls)
    return out


def _readable(mangled):
    m = re.match(r"_ZN?(?:K?2fc)?(?:12_GLOBAL__N_1)?(\d+)", mangled)
    at = m.end()
    name, rest = mangled[at:at + int(m.group(1))], mangled[at + int(m.group(1)):]
    args = re.match(r"I((?:L[ib]n?\d+E)+)E", rest)
    return name + ("<%s>" % ",".join(re.findall(r"L[ib](n?\d+)E", args.group(1))) if args else "")


# the calls by quantizer, with addresses that are aligned and never followed
P = 1 << 20
SUFFIX = {"asym": "", "sym": "_sym", "fp8": "_fp8", "cmeta": "_cmeta"}


def _meta(quantizer, copies=1):
    return (P, P) if quantizer == "asym" else (P,)


def quantize(quantizer, elems, group, bits=8):
    return "fc_quantize" + SUFFIX[quantizer], [P, elems // group, group, group, *(() if quantizer == "fp8" else (bits,)), P, *_meta(quantizer), 0]


def dequantize(quantizer, elems, group, bits=8):
    return "fc_dequantize" + SUFFIX[quantizer], [P, *_meta(quantizer), elems // group, group, group, *(() if quantizer == "fp8" else (bits,)), P, 0]


def fused(quantizer, n_src, elems, group, bits_in=8, bits_out=8):
    bits = () if quantizer == "fp8" else (bits_in, bits_out)
    return ("fc_dequant_reduce_requant" + SUFFIX[quantizer],
            [P, elems * bits_in // 8, P, *([P] if quantizer == "asym" else []), elems // group, n_src, elems // group, group, group, *bits, P,
             *_meta(quantizer), 0])


def allreduce(quantizer, n_src, elems, group, bits_rs=8, bits_ag=8):
    bits = () if quantizer == "fp8" else (bits_rs, bits_ag)
    return "fc_allreduce_sim" + SUFFIX[quantizer], [P, n_src, elems // group, group, group, *bits, P, P, 1 << 44, 0]


QUANTIZER = {"asym": 0, "sym": 1, "fp8": 2}


def quantize_rot(quantizer, elems, hidden, group, bits=8):
    return "fc_quantize_rot", [P, elems // hidden, hidden, group, bits, QUANTIZER[quantizer], P, P, P, 0]


def dequantize_rot(quantizer, elems, hidden, group, bits=8):
    return "fc_dequantize_rot", [P, P, P, elems // hidden, hidden, group, bits, QUANTIZER[quantizer], P, 0]


def allreduce_rot(quantizer, n_src, elems, hidden, group, bits_rs=8, bits_ag=8):
    return "fc_allreduce_sim_rot", [P, n_src, elems // hidden, hidden, group, bits_rs, bits_ag, QUANTIZER[quantizer], P, P, 1 << 44, 0]
