"""What the library's host code launches and allocates, on a HIP runtime without a GPU
(host/fake_hip.cpp): nothing is computed here."""
import json
import os
import re
import shutil
import subprocess
import sys

import pytest

import paper_2307_06554_amd as pm
from paper_2307_06554_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")

# made-up device addresses, far enough apart for the largest calls here
A, B, C, W = (k << 44 for k in (1, 2, 3, 4))
Q30, EVEN = 1068236801, 1 << 20
GOLDILOCKS = (1 << 64) - (1 << 32) + 1


@pytest.fixture(scope="module")
def drive(tmp_path_factory):
    fake = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(HERE, "host", "fake_hip.cpp"), "-o", fake],
                   check=True, capture_output=True, text=True)

    def run(calls):
        res = subprocess.run([sys.executable, os.path.join(HERE, "host_routes.py"), fake, pm.lib_path(), binding.__file__,
                              json.dumps(calls)], capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stdout + res.stderr
        return [json.loads(line) for line in res.stdout.splitlines()]

    return run


def kernels(result):
    """Names of the launched kernels, without namespace and template arguments."""
    return [re.sub(r"^_ZN?(2pm|12_GLOBAL__N_1)?\d*", "", launch[0]) for launch in result["launches"]]


def call(fn, *args, **more):
    return dict(fn=fn, args=list(args), **more)


# ------------------------------------------------------------ direct calls with a workspace
def outer_words_used(result, word):
    """Words from the start of the workspace to the end of b's points, as the outer launch has them:
    a, b, c, a's points, b's points."""
    a, b, c, sa, sb = (int(v) for v in result["launches"][0][5:10])
    return sa, (sb - sa) // word * 2


@pytest.mark.parametrize("n,products", [(16384, 48), (32768, 5), (65536, 16)])
def test_workspace_is_what_the_transform_uses(drive, n, products):
    size = binding.polymul_workspace_size(n, products, 4)
    got = drive([call("polymul_negacyclic_rns_workspace", A, B, C, n, {"u32": [Q30]}, 1, products, W, size, None)])[0]
    assert got["status"] == 0
    assert [k for k in kernels(got) if "outer" in k] and "pt_outer_forward" in got["launches"][0][0]
    assert outer_words_used(got, 4) == (W, size // 4)
    size = binding.polymul_workspace_size(n, products, 8)
    got = drive([call("polymul_negacyclic_u64_workspace", A, B, C, n, GOLDILOCKS, products, W, size, None)])[0]
    assert got["status"] == 0 and outer_words_used(got, 8) == (W, size // 8)
    assert size == 4 * n * products * 8


def test_karatsuba_table_has_no_part_in_the_workspace_calls(drive):
    n, products = 65536, 16
    calls = []
    for depth in (0, 1, 3, binding.KARATSUBA_BUILTIN):
        for word, fn, mod in ((8, "polymul_negacyclic_u64_workspace", [GOLDILOCKS]),
                              (4, "polymul_negacyclic_rns_workspace", [{"u32": [Q30]}, 1])):
            size = 4 * n * products * word
            calls += [call("polymul_tune_set_karatsuba", n, products, word, depth),
                      call(fn, A, B, C, n, *mod, products, W, size, None)]
    for got in drive(calls)[1::2]:
        assert got["status"] == 0
        assert ["pt_outer_forward" in got["launches"][0][0], "pt_outer_inverse" in got["launches"][2][0],
                len(got["launches"])] == [True, True, 3]


def test_workspace_arguments(drive):
    EINVAL, EALIAS = 1, 2
    n, need = 16384, 4 * 16384 * 2 * 4
    rns = lambda ws, size, q=Q30, L=1, n=n, a=A, c=C: call(
        "polymul_negacyclic_rns_workspace", a, B, c, n, {"u32": [q] * L}, L, 2 // L, ws, size, None)
    u64 = lambda ws, size, q=GOLDILOCKS: call("polymul_negacyclic_u64_workspace", A, B, C, 8192, q, 4, ws, size, None)
    cases = [
        (rns(W, need), 0), (rns(W, need, L=2), 0), (rns(W, need - 1), EINVAL), (rns(W + 8, need), EINVAL),
        (rns(None, need), EINVAL), (rns(A + 16, need), EALIAS), (rns(C - 16, need), EALIAS), (rns(W, need, a=C + 16), EALIAS),
        (rns(W, need, q=1), EINVAL), (rns(W, need, n=10000), EINVAL),
        (rns(None, 0, q=EVEN), 0), (rns(None, 0, n=8192), 0),  # no workspace in use
        (u64(W, 4 * 8192 * 4 * 8), 0), (u64(W, 4 * 8192 * 4 * 8 - 1), EINVAL), (u64(B, 4 * 8192 * 4 * 8), EALIAS),
        (u64(None, 0, q=1 << 40), 0), (u64(None, 0, q=0), EINVAL),
        (call("polymul_workspace_size", 100, 1, 4, {"out": 64}), EINVAL),
        (call("polymul_workspace_size", 16384, 1, 2, {"out": 64}), EINVAL),
        (call("polymul_workspace_size", 16384, 1 << 41, 4, {"out": 64}), EINVAL),
    ]
    for (c, want), got in zip(cases, drive([c for c, _ in cases])):
        assert got["status"] == want, c
    for n in (4096, 8192):
        assert binding.polymul_workspace_size(n, 7, 4) == 0
    assert binding.polymul_workspace_size(4096, 7, 8) == 0 and binding.polymul_workspace_size(8192, 7, 8) == 4 * 8192 * 7 * 8


# ------------------------------------------------------------------ launches the hardware holds
BIG = [  # entry point, its arguments after a, b, c, degree, words per product's group, products
    ("polymul_negacyclic_shared", [4096, Q30], 1, (1 << 23) + 100),
    ("polymul_negacyclic_shared", [8192, Q30], 1, (1 << 22) + 3),
    ("polymul_negacyclic_shared", [1024, Q30], 1, (1 << 25) + 5),
    ("polymul_negacyclic_rns_shared", [2048, {"u32": [Q30, 12289, 65537]}, 3], 3, (1 << 24) // 3 + 7),
    ("polymul_cyclic", [4096, Q30], 1, (1 << 23) + 1),
    ("polymul_cyclic", [8192, Q30], 1, (1 << 22) + 1),
]


@pytest.mark.parametrize("fn,args,channels,batch", BIG, ids=[f"{f[8:]}-{a[0]}" for f, a, _, _ in BIG])
def test_arrays_beyond_one_grid(drive, fn, args, channels, batch):
    """Arrays of more than 128 GiB (a and c, or one operand squared, fit the memory): more
    work-items than a launch holds, so several launches over consecutive products."""
    n = args[0]
    b = A if fn == "polymul_cyclic" else B
    got = drive([call(fn, A, b, C, *args, batch, None)])[0]
    assert got["status"] == 0
    at = 0
    for launch in got["launches"]:
        assert "ptrans" in launch[0]
        grid, block = int(launch[1]), int(launch[3])
        a, bb, c, nprod = (int(v) for v in launch[5:9])
        assert grid * block < 1 << 32
        assert (a, c) == (A + 4 * n * at, C + 4 * n * at) and bb == (b if b == B else a)
        assert nprod % channels == 0 and grid * max(1, 4096 // n) >= nprod > 0
        at += nprod
    assert at == batch * channels and len(got["launches"]) == 2


# ------------------------------------------------------------------------------------- plans
MIB = 1 << 20


def test_plan_buffer_is_bounded_over_all_groups(drive):
    # each group's sub-products would take 234 MiB
    got = drive([dict(plan=[[8192, Q30, 5000]] * 3)])[0]
    assert got["status"] == 0 and got["leaked"] == 0
    assert got["held"] < 258 * MIB
    assert [k for k in kernels(got) if "grouped" in k] and sum("kara_combine" in k for k in kernels(got)) == 1


@pytest.mark.parametrize("room", [4 * MIB, 0.01 * MIB], ids=["no room for sub-products", "no room at all"])
def test_plan_without_room_for_sub_products(drive, room):
    """A group of n = 8192 that needs a buffer on the transform and none on tiles takes those where
    the buffer finds no room; the allocation that failed is not reported by the launches after it."""
    plan = [[8192, Q30, 300], [1024, Q30, 64]]
    got = drive([dict(plan=plan), dict(plan=plan, limit=int(room)), dict(plan=[[256, Q30, 1]])])
    assert got[0]["held"] > 14 * MIB and sum("kara_combine" in k for k in kernels(got[0])) == 1
    assert got[1]["status"] == (0 if room > MIB else 4)
    assert not any("kara_combine" in k for k in kernels(got[1]))
    assert [g["status"] for g in got[::2]] == [0, 0] and not any(g["leaked"] for g in got)


@pytest.mark.parametrize("plan,transform", [
    # n = 1024 alone or beside smaller degrees: tiles up to three quarters of the CUs
    ([[1024, Q30, 1]], False), ([[1024, Q30, 768]], False), ([[1024, Q30, 769]], True),
    ([[1024, Q30, 600], [1024, Q30 + 2, 600]], True), ([[1024, Q30, 8], [256, Q30, 100]], False),
    ([[1024, Q30, 8], [2048, Q30, 1]], True), ([[1024, Q30, 8], [2048, 12289, 1]], False),
    # n = 4096 and 8192: runs of whole products on tiles that fill at most every CU once
    ([[8192, Q30, 1]], True), ([[8192, Q30, 3]], False), ([[8192, Q30, 5]], True), ([[8192, Q30, 8]], False),
    ([[8192, Q30, 12]], False), ([[8192, Q30, 16]], True), ([[4096, Q30, 8]], True), ([[4096, Q30, 14]], False),
    ([[4096, Q30, 30]], False), ([[4096, Q30, 45]], True), ([[8192, Q30, 6], [4096, Q30, 6]], False),
    ([[8192, Q30, 8], [256, Q30, 1]], True), ([[8192, Q30, 7], [256, Q30, 100]], False),
    ([[8192, Q30, 3], [256, Q30, 100]], True), ([[4096, Q30, 14], [256, Q30, 1]], True),
    ([[8192, Q30, 7], [512, Q30, 10]], True), ([[8192, EVEN, 4], [8192, Q30, 4]], True),
    ([[2048, Q30, 1]], True), ([[8192, Q30, 2], [1024, Q30, 1]], True),
])
def test_light_plans(drive, plan, transform):
    got = drive([dict(plan=plan)])[0]
    assert got["status"] == 0
    assert ("grouped_kernelILb1" in got["launches"][0][0]) == transform


# ------------------------------------------------------------------ depth 0 of the Karatsuba calls
@pytest.mark.parametrize("n,q,products,levels", [
    (8192, Q30, 1, True), (8192, Q30, 56, True), (8192, Q30, 57, False), (8192, 4194301, 56, True),
    (8192, 4194301, 57, False), (8192, 3329, 44, True), (8192, 3329, 45, False), (1024, Q30, 1, False),
    (1024, 4194301, 8, False), (2048, Q30, 1, False),
    (4096, Q30, 1, False), (16384, Q30, 1, False),
])
def test_depth_0_with_few_products(drive, n, q, products, levels):
    size = pm.polymul_karatsuba_workspace_size(n, 1, products, 0)
    args = [A, B, C, n, {"u32": [q]}, 1, products, 0]
    got = drive([call("polymul_negacyclic_rns_karatsuba", *args, W, size, None),
                 call("polymul_negacyclic_rns_karatsuba_noalloc", *args, None)])
    for g in got:
        assert g["status"] == 0
        assert any("kara_split" in launch[0] for launch in g["launches"]) == levels


# ---------------------------------------------------------------------------- one shared operand
@pytest.mark.parametrize("q,channels,batch,tiles", [
    (4194301, 1, 8, True), (4194301, 1, 511, True), (4194301, 1, 512, False), (4194301, 4, 127, True),
    (4194301, 4, 128, False), (Q30, 1, 1, False),
])
def test_shared_operand_at_n_1024(drive, q, channels, batch, tiles):
    got = drive([call("polymul_negacyclic_rns_shared", A, B, C, 1024, {"u32": [q] * channels}, channels, batch, None)])[0]
    assert got["status"] == 0 and ("mfma32_shared" in got["launches"][0][0]) == tiles


# -------------------------------------------------- the kernels that test_gpu_routes.py is about
def launched(drive, calls):
    got = drive(calls)
    assert not any(g["status"] for g in got)
    return [[launch[0] for launch in g["launches"]] for g in got]


@pytest.mark.parametrize("n", [8192, 16384, 32768])
def test_direct_64_bit_calls_stream(drive, n):
    fns = ("polymul_negacyclic_u64", "polymul_cyclic_u64", "polymul_negacyclic_u64_shared")
    for names in launched(drive, [call(fn, A, B, C, n, GOLDILOCKS, 2, None) for fn in fns]):
        assert len(names) == 1 and "stream8_kernel" in names[0]


def test_ten_channels_stream_in_two_launches(drive):
    names, = launched(drive, [call("polymul_negacyclic_rns", A, B, C, 16384, {"u32": [Q30] * 10}, 10, 2, None)])
    assert len(names) == 2 and all("stream_kernel" in k for k in names)


@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_tiles_beside_the_transform(drive, n):
    for q in (3330, 1 << 20, Q30 - 1, (1 << 32) - 5):
        shared, direct, cyclic = launched(drive, [call(fn, A, B, C, n, q, 5, None) for fn in (
            "polymul_negacyclic_shared", "polymul_negacyclic", "polymul_cyclic")])
        assert ["mfma32_shared_kernel" in shared[0], "mfma32_group_kernel" in direct[0],
                "mfma32_group_kernel" in cyclic[0]] == [True] * 3


def test_karatsuba_sub_products_and_library_scratch(drive):
    qs = {"u32": [Q30 - 1, (1 << 32) - 5, 3329]}
    calls = [call("polymul_negacyclic_rns_karatsuba", A, B, C, n, qs, 3, 3, depth, W, 1 << 30, None)
             for n, depth in ((2048, 1), (4096, 1), (8192, 1), (4096, 2), (8192, 3))]
    for names in launched(drive, calls):
        assert "mfma32_group_kernel" in names[1]
    small, outer = launched(drive, [call("polymul_negacyclic_rns_karatsuba_noalloc", A, B, C, n, {"u32": [Q30, 12289]}, 2, 3, 0, None)
                                    for n in (4096, 16384)])
    assert "ptrans_kernel" in small[0] and ["pt_outer_forward" in outer[0], "ptrans_kernel" in outer[1],
                                            "pt_outer_inverse" in outer[2]] == [True] * 3
