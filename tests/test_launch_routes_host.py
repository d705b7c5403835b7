"""Which kernels the library's calls launch, read off its host code on a machine without a GPU: a child process loads the
built library above a stand-in for the HIP runtime (launch_recorder.c) that notes every launch and runs nothing.  A size that
one of the rules takes to a path, and one that it leaves, are stated here as such; what the paths compute is tested on the GPU."""
import json
import os
import re
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2604_26881_amd", "libmoe_hip.so")
SHAPE = -2

CHILD = """
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.recorder_take.restype = ctypes.c_char_p
lib = ctypes.CDLL(sys.argv[2])
kinds = dict(p=ctypes.c_void_p, i=ctypes.c_int, z=ctypes.c_size_t, f=ctypes.c_float)
for name, args in json.load(sys.stdin):
    rc = getattr(lib, name)(*[kinds[k](v) for k, v in args])
    print(json.dumps([rc, rec.recorder_take().decode().splitlines()]), flush=True)
"""


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    so = str(tmp_path_factory.mktemp("rec") / "recorder.so")
    r = subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.c"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(calls):
        """(status, launches) of each call"""
        r = subprocess.run([sys.executable, "-c", CHILD, so, LIB], input=json.dumps(calls), capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, f"the process ended with {r.returncode} after {len(r.stdout.splitlines())} of {len(calls)} calls\n{r.stderr}"
        out = []
        for line in r.stdout.splitlines():
            rc, launches = json.loads(line)
            out.append((rc, [short(l.split()[0]) for l in launches]))
        return out
    return run


def short(mangled):
    """expert_tile_kernel<160,256,1,4,1,3,1,1,1,0> of a mangled name"""
    at, name = mangled.index("N") + 1, None
    while mangled[at].isdigit():       # length-prefixed names: namespaces, then the kernel's
        n = re.match(r"\d+", mangled[at:]).group(0)
        at += len(n)
        name, at = mangled[at:at + int(n)], at + int(n)
    args = re.match(r"I((?:L(?:[a-z]|N[^E]*E)n?\d+E)*)E", mangled[at:])
    return f"{name}<{','.join(re.findall(r'[a-zE](n?[0-9]+)E', args.group(1))) if args else ''}>"


def layer(T, H, E, K, I, Is, gather=False, lo=0, hi=None, policy=0, shared_policy=0, wgate=True, **memory):
    """moe_layer_forward on memory of its own for every operand (terabytes apart), but for what `memory` says: name ->
    (name of another operand, byte offset in it) or a size"""
    names = ["x", "Wr", "bias", "Wg", "Wu", "Wd", "Wsg", "Wsu", "Wsd", "wgate", "topk_ids", "topk_w", "expert_offsets", "src_of_row",
             "row_of_pair", "Xp", "Yp", "S", "sg", "out", "permute_workspace", "workspace", "shared_workspace", "next"]
    at = {n: (i + 1) << 40 for i, n in enumerate(names)}
    at["bias"] = at["next"] = None
    if gather:
        at["Xp"] = None
    if Is == 0:
        for n in ("Wsg", "Wsu", "Wsd", "wgate", "S", "sg", "shared_workspace"):
            at[n] = None
    if not wgate:
        at["wgate"] = None
    size = {n: 1 << 38 for n in ("permute_workspace", "workspace", "shared_workspace")}
    for n, v in memory.items():
        if isinstance(v, tuple):
            at[n] = at[v[0]] + v[1]
        else:
            size[n] = v
    p = lambda *ns: [["p", at[n]] for n in ns]
    i = lambda *vs: [["i", v] for v in vs]
    room = lambda n: p(n) + [["z", size[n]]]
    return ["moe_layer_forward",
            p("x", "Wr", "bias") + [["p", None]] + i(0) + p("Wg", "Wu", "Wd", "Wsg", "Wsu", "Wsd", "wgate") +
            i(T, H, E, K, I, Is, 1, lo, E if hi is None else hi, policy, shared_policy) +
            p("topk_ids", "topk_w", "expert_offsets", "src_of_row", "row_of_pair", "Xp", "Yp", "S", "sg", "out") +
            room("permute_workspace") + room("workspace") + room("shared_workspace") + [["f", 0.0]] + p("next") + [["p", None]]]


def named(launches, kernel):
    return [l for l in launches if l.startswith(kernel)]


@pytest.mark.parametrize("T", [5, 640])        # a batch sorted beside its experts, one sorted in a launch of its own
@pytest.mark.parametrize("I", [0, -64, 100])
def test_experts_without_columns_are_refused_behind_the_sort(record, T, I):
    (rc, launches), = record([layer(T, 64, 8, 2, I, 64)])
    assert rc == SHAPE
    assert named(launches, "route") and named(launches, "permute") and not named(launches, "expert")
