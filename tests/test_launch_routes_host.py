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
    (name of another operand, byte offset in it), None (NULL) or a workspace's size"""
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
        if v is None:
            at[n] = None
        elif isinstance(v, tuple):
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


def gate_up(launches):
    """The tile kernels' gate/up launches: their sixth argument says which projection"""
    return [l for l in named(launches, "expert_tile_kernel") if l.split("<")[1].split(",")[4] == "1"]


# one (T, Is, hosted) each, for 60 experts of H 128, I 1152, top 4 (tiles of 128, 160 and 256 rows): whole sets of I columns, a
# narrower last set that covers all column tiles of a set or fewer, one set narrower than I; too many sets.  What the path computes is compared at the same sizes in test_gpu_kernel_edges.py.
SHARED_BESIDE = [(640, 2304, True), (640, 2240, True), (640, 1216, True), (640, 64, True), (640, 10432, False),
                 (2100, 2304, True), (2100, 2240, True), (2100, 1088, True), (2100, 1216, True), (2100, 64, True), (2100, 10432, False),
                 (3000, 2304, True), (3000, 2240, True), (3000, 1088, True), (3000, 1216, True), (3000, 64, True), (3000, 10432, False)]
# the benchmark's layer at every tile height; layers whose shared tiles are mostly empty, or fill more rounds beside the
# routed ones than alone; too few tokens
OTHERS = [(777, 2048, 60, 4, 1408, 5632, True), (2048, 2048, 60, 4, 1408, 5632, True), (3000, 2048, 60, 4, 1408, 5632, True),
          (2000, 1024, 200, 8, 512, 1728, True), (2100, 2048, 60, 4, 1152, 1216, True), (6000, 1024, 32, 4, 960, 1984, False),
          (4513, 1024, 16, 1, 4096, 192, False), (9015, 1024, 48, 1, 4032, 512, False), (1449, 1024, 24, 2, 3840, 26880, False),
          (4007, 1024, 32, 1, 2048, 8192, False), (700, 1536, 64, 6, 1024, 2048, False), (256, 2048, 8, 4, 1408, 5632, False)]


@pytest.mark.parametrize("T,H,E,K,I,Is,hosted", [(T, 128, 60, 4, 1152, Is, hosted) for T, Is, hosted in SHARED_BESIDE] + OTHERS)
@pytest.mark.parametrize("gather", [False, True])
def test_shared_gate_up_joins_the_routed_launch_where_its_tiles_cost_no_more_there(record, T, H, E, K, I, Is, hosted, gather):
    (rc, launches), = record([layer(T, H, E, K, I, Is, gather)])
    assert rc == 0
    assert len(gate_up(launches)) == (1 if hosted else 2), launches


def test_a_call_on_a_few_experts_keeps_its_narrower_tiles_for_itself(record):
    (rc, whole), (rc_few, few) = record([layer(2048, 2048, 60, 4, 1408, 5632), layer(2048, 2048, 60, 4, 1408, 5632, lo=7, hi=14)])
    assert rc == rc_few == 0
    assert len(gate_up(whole)) == 1 and "<160,256," in gate_up(whole)[0]
    assert len(gate_up(few)) == 2 and "<160,128," in gate_up(few)[0]


@pytest.mark.parametrize("H,Is", [(2048, 5632), (1024, 8192), (2560, 4096)])
def test_shared_expert_beside_small_kernels_keeps_off_the_tiles_that_hold_them_up(record, H, Is):
    p = [["p", 1 << 40]]
    call = lambda T, policy: ["moe_shared_forward_ex", p * 5 + [["i", T], ["i", H], ["i", Is]] + p * 3 + [["z", 1 << 38], ["i", policy], ["p", None]]]
    sizes = list(range(64, 16385, 160))
    alone, beside = record([call(T, 0) for T in sizes]), record([call(T, 0x400) for T in sizes])
    assert any("<192,256," in gate_up(l)[0] for _, l in alone if gate_up(l))
    for T, (rc, launches) in zip(sizes, beside):
        assert rc == 0 and len(gate_up(launches)) == 1, T
        assert "<192,256," not in launches[0], T
        if "<160,256," in launches[0]:
            assert -(-T // 160) * -(-Is // 128) <= 512, T
    assert any("<256,256," in l[0] for _, l in beside)


# T, K, E of a layer of H 64, I 64, and whether its pairs are sorted beside gate/up: up to 128 of them, also where the
# streaming kernel takes two token tiles per pass (a mean above 10).  test_gpu_kernel_edges.py computes them.
SORT_BESIDE = [(63, 1, 12, True), (64, 1, 256, True), (65, 1, 256, True), (127, 1, 200, True), (64, 2, 33, True), (128, 1, 64, True),
               (48, 2, 8, True), (64, 2, 8, True), (62, 2, 4, True), (129, 1, 64, False), (65, 2, 8, False)]


def sorted_beside(launches):
    """Whether the pairs were sorted in the narrow streaming kernel's gate/up launch (its last argument), or by the sort's own"""
    beside = [l for l in launches if l.startswith("expert_stream_lds_kernel") and l.endswith(",1>")]
    assert len(beside) + min(1, len(named(launches, "permute"))) == 1
    return beside


@pytest.mark.parametrize("T,K,E,beside", SORT_BESIDE)
@pytest.mark.parametrize("gather", [False, True])
def test_pairs_are_sorted_beside_gate_up(record, T, K, E, beside, gather):
    (rc, launches), = record([layer(T, 64, E, K, 64, 0, gather)])
    assert rc == 0
    assert len(sorted_beside(launches)) == beside
    if beside:
        tiles = 2 if T * K / E > 10 else 1
        assert sorted_beside(launches)[0].startswith(f"expert_stream_lds_kernel<{tiles},1,4,0,"), launches


def test_pairs_are_sorted_beside_gate_up_and_a_riding_shared_expert(record):
    for T, K, E, gather in [(1, 2, 8, False), (24, 2, 8, True), (32, 4, 60, False), (32, 4, 22, True)]:
        (rc, launches), = record([layer(T, 64, E, K, 128, 512, gather)])
        assert rc == 0
        assert [l.split("<")[1] for l in sorted_beside(launches)] == ["1,1,4,1,0,1>"], (T, launches)
    # a wide contraction of more than 6 rows per expert is the wide kernel's
    (rc, launches), = record([layer(60, 320, 8, 1, 320, 0)])
    assert rc == 0 and not sorted_beside(launches) and named(launches, "expert_stream_wide")


# T, K, E, H, I on either side of the two lines in the number of the launch's waves
@pytest.mark.parametrize("T,K,E,H,I,beside", [
    (1, 4, 60, 2048, 1408, True), (1, 1, 60, 2048, 3264, True), (1, 1, 60, 2048, 3328, False), (1, 8, 256, 2048, 960, True),
    (1, 8, 256, 2048, 1024, False), (2, 8, 256, 1024, 4096, False), (4, 8, 256, 2048, 2048, True), (1, 4, 64, 1024, 4096, False),
    (32, 4, 60, 2048, 1408, True), (16, 8, 256, 1024, 256, True), (16, 8, 256, 1024, 512, False), (9, 8, 256, 1024, 512, True),
    (16, 8, 256, 2048, 768, False), (12, 8, 256, 2048, 768, False), (8, 8, 256, 2048, 768, True), (8, 8, 256, 1024, 4096, False)])
def test_pairs_are_sorted_apart_beside_many_waves(record, T, K, E, H, I, beside):
    (rc, launches), = record([layer(T, H, E, K, I, 0)])
    assert rc == 0 and len(sorted_beside(launches)) == beside


H_, I_, P_ = 64, 64, 16        # T 8, K 2, E 8: bytes of the operands
SORT_IN_USE = [dict(topk_ids=("workspace", 0)), dict(topk_ids=("workspace", P_ * I_ * 2 - 4)), dict(expert_offsets=("workspace", 8)),
               dict(src_of_row=("workspace", 64)), dict(row_of_pair=("workspace", 128)), dict(x=("workspace", P_ * I_ * 2 - 16)),
               dict(Xp=("workspace", 0)), dict(Xp=("x", 16)), dict(topk_ids=("row_of_pair", 0)), dict(topk_ids=("src_of_row", 4)),
               dict(topk_ids=("expert_offsets", 32))]
SORT_FREE = [dict(topk_ids=("workspace", P_ * I_ * 2)), dict(x=("workspace", P_ * I_ * 2)), dict(Xp=("x", 8 * H_ * 2)),
             dict(topk_ids=("row_of_pair", P_ * 4)), dict(topk_ids=("expert_offsets", 36)), dict(permute_workspace=("workspace", 0))]


@pytest.mark.parametrize("beside,memory", [(False, m) for m in SORT_IN_USE] + [(True, m) for m in SORT_FREE])
def test_memory_that_gate_up_writes_keeps_the_sort_in_its_own_launch(record, beside, memory):
    (rc, launches), = record([layer(8, H_, 8, 2, I_, 0, **memory)])
    assert rc == 0 and len(sorted_beside(launches)) == beside


# T 640, H 128, E 60, K 4, I 1152, Is 2304: the shared hidden rows are written while the routed experts' launches run
HOST_ROWS, HOST_H = 640 * 4, 640 * 2304 * 2
HOST_IN_USE = [(False, dict(shared_workspace=("workspace", 0))), (False, dict(shared_workspace=("workspace", HOST_ROWS * 1152 * 2 - 256))),
               (False, dict(workspace=("shared_workspace", HOST_H - 256))), (False, dict(shared_workspace=("Xp", 0))),
               (False, dict(shared_workspace=("Yp", 256))), (True, dict(src_of_row=("shared_workspace", 512))),
               (False, dict(expert_offsets=("shared_workspace", 0))), (False, dict(x=("shared_workspace", HOST_H - 256))),
               (False, dict(x=("workspace", 0))), (False, dict(Yp=("x", 256)))]
HOST_FREE = [(False, dict(shared_workspace=("workspace", HOST_ROWS * 1152 * 2))), (False, dict(workspace=("shared_workspace", HOST_H))),
             (False, dict(out=("shared_workspace", 0))), (False, dict(permute_workspace=("shared_workspace", 0)))]


@pytest.mark.parametrize("hosted,gather,memory", [(False, *m) for m in HOST_IN_USE] + [(True, *m) for m in HOST_FREE])
def test_memory_that_the_routed_experts_use_keeps_the_shared_gate_up_in_its_own_launch(record, hosted, gather, memory):
    (rc, launches), = record([layer(640, 128, 60, 4, 1152, 2304, gather, **memory)])
    assert rc == 0 and len(gate_up(launches)) == (1 if hosted else 2)


@pytest.mark.parametrize("change,status", [(dict(shared_workspace=640 * 2304 * 2 - 1), -3), (dict(S=None), -1), (dict(sg=None), -1),
                                           (dict(Wsd=None), -1), (dict(shared_policy=10), 0), (dict(policy=5), 0), (dict(wgate=False), 0)])
def test_what_the_shared_call_refuses_is_left_to_it(record, change, status):
    call = lambda gather: layer(640, 128, 60, 4, 1152, 2304, gather, **change)
    for rc, launches in record([call(False), call(True)]):
        assert rc == status
        assert len(gate_up(launches)) == (1 if status or "wgate" in change else 2)
        if status:     # the routed experts have been enqueued, the shared one has not
            assert len(named(launches, "expert_tile_kernel")) == 2 and not named(launches, "combine")


# mean rows of 60 experts and the height of the layer's tiles; H, I of which one projection is full width in the uncut call.
# test_gpu_kernel_edges.py compares the bits at these sizes.
@pytest.mark.parametrize("mean,bm", [(60, 128), (140, 160), (232, 256)])
@pytest.mark.parametrize("H,I,down", [(256, 1152, False), (448, 1152, False), (2304, 64, True), (2304, 448, True)])
def test_calls_on_a_few_experts_take_narrower_tiles(record, mean, bm, H, I, down):
    p, P = lambda n: [["p", (i + 1) << 40] for i in range(n)], 60 * mean
    call = lambda lo, hi: ["moe_expert_group_forward", [["i", lo], ["i", hi]] + p(5) + [["i", v] for v in (P, H, 60, I)] + p(2) +
                           [["z", 1 << 38], ["p", None]]]
    shapes = []
    for rc, launches in record([call(0, 60), call(3, 10)]):
        assert rc == 0 and len(launches) == 2
        shapes.append(tuple(launches[down].split("<")[1].split(",")[:2]))
    assert shapes[0] == (str(bm), "256") and shapes[1] in [(str(bm), "128"), (str(bm), "64")], shapes
