"""The C-ABI library loads and exports every entry point of include/arbor.h
(host-only checks; no kernel is launched)."""
import ctypes
import os
import random
import re

import pytest

from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    src = open(os.path.join(ROOT, "include", "arbor.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(arbor_[a-z_]+)\s*\(", src)))


def test_header_matches_binding():
    assert declared_functions() == sorted(L.exported_symbols())


def test_library_exports_every_symbol():
    lib = L.load()
    for name in declared_functions():
        assert hasattr(lib, name), name


STRUCTS = {"Geom": "arbor_geom_t", "TreeS": "arbor_tree_t", "PoolS": "arbor_pool_t",
           "Params": "arbor_params_t", "Sizes": "arbor_sizes_t",
           "DecodeCredit": "arbor_decode_credit_t", "Timing": "arbor_timing_t",
           "Walk": "arbor_walk_t"}


def test_struct_layouts(tmp_path):
    """Every binding struct has the C compiler's size and field offsets for
    the header's struct (a host C program built with gcc prints them)."""
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "arbor.h"', "int main(void) {"]
    for py, c in STRUCTS.items():
        lines.append(f'  printf("{py} size %zu\\n", sizeof({c}));')
        for name, _ in getattr(L, py)._fields_:
            lines.append(f'  printf("{py} {name} %zu\\n", offsetof({c}, {name}));')
    lines.append("  return 0; }")
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines) + "\n")
    exe = tmp_path / "layout"
    import subprocess
    subprocess.run(["gcc", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                    "-I", "/opt/rocm/include", str(src), "-o", str(exe)], check=True)
    got = {}
    for line in subprocess.run([str(exe)], check=True, capture_output=True,
                               text=True).stdout.splitlines():
        py, name, val = line.split()
        got[(py, name)] = int(val)
    for py in STRUCTS:
        cls = getattr(L, py)
        assert got[(py, "size")] == ctypes.sizeof(cls), py
        for name, _ in cls._fields_:
            assert got[(py, name)] == getattr(cls, name).offset, (py, name)


def test_strerror_and_workspace_size_are_host_only():
    assert L.arbor_strerror(L.ENOPAGES) == "not enough free pages"
    assert L.arbor_strerror(12345) == "unknown status"
    lib = L.load()
    g = L.Geom(32, 8, 4, 128, 16, L.BF16, 1408)
    sz = L.Sizes(85, 22528, 1792, 85, 32, 2, 4, 32)
    n = lib.arbor_workspace_size(ctypes.byref(g), ctypes.byref(sz))
    assert n > 22528 * 16


def test_product_path_refuses_cpu_tensors():
    import torch
    with pytest.raises(ValueError):
        L._dev(torch.zeros(3), "x")


def test_timing_request_is_validated_on_the_host():
    """A per-call timing request names a known kernel and both events; a bad
    one is refused before anything is enqueued (the geometry is checked
    first, so no tree or pool is needed)."""
    lib = L.load()
    e = ctypes.c_void_p(1)
    for bad in (L.Timing(L.KERNEL_COUNT, e, e),
                L.Timing(-1, e, e), L.Timing(L.KERNEL_SELECT, e, None),
                L.Timing(L.KERNEL_SELECT, None, e)):
        g = L.Geom(32, 8, 4, 128, 16, L.BF16, 1408)
        g.timing = ctypes.pointer(bad)
        assert lib.arbor_select(ctypes.byref(g), None, None, None, None, None, None, None,
                                None) == L.EINVAL


def test_library_keeps_no_timing_state():
    """No entry point other than those of the header is exported: in
    particular no process-wide setter of timing events."""
    lib = L.load()
    assert not hasattr(lib, "arbor_set_kernel_events")


def test_uncertainty_workspace_sizes_on_the_host():
    # the chunked forms need per-chunk partials and, for top-K, K <= 256
    # candidates per chunk: the size grows with the rows and covers them
    small = L.arbor_uncertainty_workspace_size(8, 128256, L.BF16)
    large = L.arbor_uncertainty_workspace_size(85, 128256, L.BF16)
    assert 0 < small < large
    assert large >= 85 * (16 + 4 * 256 + 4)
    assert L.arbor_uncertainty_workspace_size(0, 128256, L.BF16) > 0
    with pytest.raises(ValueError):
        import torch
        L.arbor_uncertainty(torch.zeros(4), 0, None, None, None)


def test_decode_workspace_covers_the_credit_lse():
    # the scored decode keeps a log2 LSE per (leaf, layer, query head) in the
    # shared workspace: more leaves or layers need more bytes
    lib = L.load()
    g = L.Geom(32, 8, 4, 128, 16, L.BF16, 1408)
    a = L.Sizes(85, 22528, 1792, 1, 32, 2, 4, 32)
    b = L.Sizes(85, 22528, 1792, 1, 32, 2, 64, 32)
    na = lib.arbor_workspace_size(ctypes.byref(g), ctypes.byref(a))
    nb = lib.arbor_workspace_size(ctypes.byref(g), ctypes.byref(b))
    assert nb - na >= (64 - 4) * 32 * 32 * 4


@pytest.mark.parametrize("dtype", [L.BF16, L.F32])
def test_a_workspace_also_fits_every_smaller_call(dtype):
    """Fewer observers, slice layers, leaves or layers, or a shorter window, than a
    workspace was sized for may take another launch shape, which may not need more of it."""
    lib, rng = L.load(), random.Random(7)
    for _ in range(20000):
        g = L.Geom(32, rng.choice([1, 2, 4, 8]), rng.choice([1, 4, 8]), 128, 16, dtype, 4096)
        big = [rng.choice([1, 2, 8, 20, 85, 341]), rng.randint(1, 64), rng.randint(1, 8),
               rng.randint(1, 32), rng.randint(1, 32)]
        small = [rng.randint(1, x) if rng.random() < 0.7 else x for x in big]
        nb, ns = (lib.arbor_workspace_size(ctypes.byref(g), ctypes.byref(
            L.Sizes(341, 40000, 5120, *x))) for x in (big, small))
        assert ns <= nb, (big, small)


@pytest.mark.parametrize("nodes", [1, 13, 512, 513, 20000])
def test_allocate_refuses_a_small_workspace(nodes):
    """Before anything is enqueued, also where the kernel keeps its state in LDS."""
    lib, any_ptr = L.load(), 256
    t = L.TreeS(nodes, 40 * nodes, *([any_ptr] * 6))
    p = L.params_struct(dict(synth.DEFAULT_PARAMS))
    for ws, size in ((None, 0), (any_ptr, 8 * nodes)):
        assert lib.arbor_allocate(ctypes.byref(t), any_ptr, 1, 100, any_ptr, ctypes.byref(p),
                                  any_ptr, any_ptr, any_ptr, any_ptr, ws, size,
                                  None) == L.EWORKSPACE


def _decode_need(parent, n, leaves, L_, H, G, D, dtype, n_slice):
    """Bytes that the tree decode's plan takes of the workspace: the carved arrays, then
    units, lists, partials and kept products (chunk sizes by the waves' even share)."""
    maxd, up256 = 64, lambda x: (x + 255) // 256 * 256
    below = {}
    for leaf in leaves:
        x = leaf
        while x >= 0:
            below[x] = below.get(x, 0) + 1
            x = parent[x]
    blocks = lambda x: (below[x] * G + 15) // 16
    planes, bf = L_ * H, dtype == L.BF16
    waves = 3072 if bf and D == 64 else 2048
    work = planes * sum(n[x] * blocks(x) for x in below)
    least = min((n[x] for x in below if n[x]), default=1 << 30)
    C = 64
    for c in ([1024, 512, 256, 128] if bf else [256, 128]):
        if 4 * work >= c * waves * (5 if least < c else 4):
            C = c
            break
    chunks = lambda x: -(-n[x] // C)
    units = sum(chunks(x) * blocks(x) for x in below)
    rows = sum(chunks(x) * below[x] * G for x in below)
    chain = lambda x: [] if x < 0 else [x] + chain(parent[x])
    max_np = max(sum(chunks(x) for x in chain(leaf)) for leaf in leaves)
    nb, pieces = len(leaves), sum(-(-n[x] // 64) for x in below)
    floats = 12 * units + nb * max_np + pieces + 8 + rows * planes * (2 + D)
    floats += n_slice * H * 64 * sum(below[x] * G * -(-n[x] // 64) for x in below)
    carve = up256(64) + 3 * up256(4 * nb * maxd) + 2 * up256(4 * nb)
    if nb > 64:
        carve += 7 * up256(4 * nb * maxd) + up256(8 * nb * maxd)
    return carve + 4 * floats + 256


@pytest.mark.parametrize("dtype,D", [(L.BF16, 128), (L.BF16, 64), (L.F32, 128)])
def test_the_workspace_covers_the_decode_plan(dtype, D):
    """Trees from one leaf to wide frontiers, short and long blocks, one layer to 80."""
    lib, rng = L.load(), random.Random(D + dtype)
    for _ in range(1500):
        V = rng.choice([1, 2, 5, 30, 200])
        parent = [-1] + [rng.randint(max(0, i - rng.choice([1, 4, V])), i - 1) for i in range(1, V)]
        depth = [0] * V
        for i in range(1, V):
            if depth[parent[i]] >= 62:
                parent[i] = 0
            depth[i] = depth[parent[i]] + 1
        top = rng.choice([1, 40, 300, 3000])
        n = [rng.randint(0, top) for _ in range(V)]
        n[0] = rng.choice([0, 64, 5000, 70000])
        leaves = [rng.randrange(V) for _ in range(rng.choice([1, 3, 16, 64, 65, 150]))]
        L_, H, G, S = rng.choice([1, 4, 32, 80]), rng.choice([1, 4, 8]), rng.choice([1, 4, 8]), \
            rng.choice([0, 1, 2])
        total = [0] * V
        for i in range(V):
            total[i] = n[i] + (total[parent[i]] if i else 0)
        g = L.Geom(L_, H, G, D, 16, dtype, 1 << 20)
        sz = L.Sizes(V, sum(n), max(total[x] for x in leaves), 0, 1, S, len(leaves), L_)
        size = lib.arbor_workspace_size(ctypes.byref(g), ctypes.byref(sz))
        need = _decode_need(parent, n, leaves, L_, H, G, D, dtype, S)
        assert need <= size, (V, len(leaves), L_, H, G, S, need, size)
