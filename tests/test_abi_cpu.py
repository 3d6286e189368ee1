"""CPU-only checks of the C ABI: the library loads, exports what include/floe.h declares, and rejects
bad arguments before touching the device (no compute call is made here)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2505_05950_amd import binding
    if not os.path.exists(binding.lib_path()):
        from paper_2505_05950_amd import build
        build.build()
    return binding.load()


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "floe.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(floe_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared_functions()
    assert {"floe_quantize_expert", "floe_expert_ffn_sparse", "floe_moe_layer_decode", "floe_stage_channels"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_status_strings_and_version(lib):
    assert lib.floe_abi_version() >= 1
    seen = {lib.floe_status_string(s) for s in range(0, -7, -1)}
    assert len(seen) == 7 and all(seen)


def test_argument_validation_happens_before_any_device_work(lib):
    from paper_2505_05950_amd.binding import _Expert, _Shape
    fake = C.c_void_p(4096)            # never dereferenced: every call below must fail validation first

    def q(d, f, bits, group):
        s = _Shape(d, f, bits, group)
        return lib.floe_quantize_expert(C.byref(s), fake, fake, fake, fake, None)

    assert q(4096, 16, 5, 64) == -3            # bits
    assert q(4096, 16, 2, 48) == -3            # group not a power of two in range
    assert q(4096 + 64, 16, 2, 128) == -2      # d % group
    assert q(4096 + 64, 16, 2, 64) == -2       # d % 512
    assert q(16384, 16, 2, 64) == -3           # d too large
    assert q(4096, 0, 2, 64) == -1
    s = _Shape(4096, 16, 2, 64)
    assert lib.floe_quantize_expert(C.byref(s), None, fake, fake, fake, None) == -1
    assert lib.floe_up_gemv(C.byref(s), fake, fake, fake, fake, -1, fake, None) == -1
    assert lib.floe_up_gemv(C.byref(s), fake, fake, fake, C.c_void_p(4098), 1, fake, None) == -1   # misaligned x
    assert lib.floe_select_channels(fake, 0, 1, fake, fake, fake, None) == -1
    e = _Expert(s, 4096, 4096, 4096, 4096, 0, 16)
    ws = C.c_void_p(1 << 20)
    need = lib.floe_expert_workspace_bytes(C.byref(s), 1)
    assert need > 0
    assert lib.floe_expert_ffn_sparse(C.byref(e), fake, 1, fake, None, fake, fake, fake, ws, need - 1, None) == -4
    e_bad = _Expert(s, 4096, 4096, 4096, 4096, 0, 15)                                   # gd_rows != f
    assert lib.floe_expert_ffn_sparse(C.byref(e_bad), fake, 1, fake, None, fake, fake, fake, ws, need, None) == -1
    assert lib.floe_stage_channels(None, 4096, 16, fake, fake, 4, fake, None, None, None) == -1
    assert lib.floe_expert_workspace_bytes(C.byref(_Shape(4096, 16, 7, 64)), 1) == 0


def test_tuning_switch_validates_its_arguments(lib):
    bad = [(1, 4), (1, -1), (2, 4097), (2, -1), (3, 3), (3, -1), (4, 257), (4, -1), (0, 0), (9, 0)]
    for key, value in bad:
        assert lib.floe_tuning(key, value) == -1, (key, value)
    try:
        for key, values in ((1, (1, 2, 3)), (2, (1, 32, 4096)), (3, (1, 2)), (4, (1, 16, 256))):
            for v in values:
                assert lib.floe_tuning(key, v) == 0, (key, v)
    finally:
        for key in (1, 2, 3, 4):
            assert lib.floe_tuning(key, 0) == 0


def test_layer_workspace_query_for_every_path_the_dispatch_can_take(lib):
    """The workspace plan (host logic only) for the two layer shapes of the benchmark at batch sizes on both sides of
    every dispatch boundary, under every tuning: a size is returned, it holds at least the partial results of one block
    per (token, slot), and it is the same when asked twice (the decode call sizes its pointers with the same routine)."""
    from paper_2505_05950_amd.binding import _Layer, _Shape
    lib.floe_layer_workspace_bytes.restype = C.c_size_t
    fake = C.c_void_p(4096)
    shapes = [(4096, 14336, 2, 64, 8, 2, 0), (2048, 1408, 3, 32, 64, 6, 2), (1024, 300, 4, 128, 3, 1, 1),
              (1536, 700, 8, 64, 100, 4, 0)]
    try:
        for fused_tasks in (0, 16, 256):
            for grouped in (0, 1, 2):
                for union in (0, 1, 2, 3):
                    lib.floe_tuning(4, fused_tasks), lib.floe_tuning(3, grouped), lib.floe_tuning(1, union)
                    for d, f, bits, group, n, top_k, n_shared in shapes:
                        L = _Layer(n, top_k, n_shared, 1, _Shape(d, f, bits, group), 4096, None, 4096, 0, 4096, 0)
                        slots = top_k + n_shared
                        for T in (1, 2, 3, 4, 8, 9, 16, 17, 32, 33, 64, 128, 500, 4096):
                            need = lib.floe_layer_workspace_bytes(C.byref(L), T)
                            assert need >= T * slots * d * 4, (d, f, bits, n, T, fused_tasks, grouped, union)
                            assert need == lib.floe_layer_workspace_bytes(C.byref(L), T)
                            assert need < (64 << 30)
                        assert lib.floe_layer_workspace_bytes(C.byref(L), -1) == 0
                        assert lib.floe_moe_layer_decode(C.byref(L), fake, 1, fake, None, fake, 16, None) == -4
    finally:
        for key in (1, 3, 4):
            lib.floe_tuning(key, 0)


@pytest.mark.parametrize("d,f,bits,group,n,top_k,n_shared", [
    (4096, 14336, 2, 64, 8, 2, 0), (2048, 1408, 3, 32, 64, 6, 2), (1024, 3584, 2, 64, 8, 2, 0), (2560, 6911, 4, 128, 6, 2, 0),
    (512, 300, 8, 64, 34, 1, 1),
])
def test_a_workspace_sized_for_the_largest_batch_serves_the_smaller_ones(lib, d, f, bits, group, n, top_k, n_shared):
    """The plans for tokens that share rows jump up and down with the batch size; what the queries ask for does not, and holds
    each of them (forced here, so that no call falls back to a plan that needs less)."""
    import torch
    from paper_2505_05950_amd.binding import _Expert, _Layer, _Shape
    if torch.cuda.is_available():
        pytest.skip("the pointers below are made up: without a device the calls end at their first HIP call")
    lib.floe_layer_workspace_bytes.restype = lib.floe_expert_workspace_bytes.restype = C.c_size_t
    fake, ws = C.c_void_p(4096), C.c_void_p(1 << 20)
    s = _Shape(d, f, bits, group)
    L = _Layer(n, top_k, n_shared, 1, s, 4096, None, 4096, 0, 4096, 0)
    e = _Expert(s, 4096, 4096, 4096, 4096, 0, f)

    def sizes(T, mode):
        lib.floe_tuning(1, mode)
        return lib.floe_layer_workspace_bytes(C.byref(L), T), lib.floe_expert_workspace_bytes(C.byref(s), T)

    try:
        lib.floe_tuning(4, 1)
        last = (0, 0)
        for T in list(range(17, 340)) + [511, 512, 513, 1025, 4096]:
            one_token, now = sizes(T, 3), sizes(T, 1)
            assert all(a >= max(b, c) for a, b, c in zip(now, last, one_token)), (T, last, now, one_token)
            last = now
        for top in (81, 145, 160, 161, 257, 339):
            layer_bytes, expert_bytes = (C.c_size_t(b) for b in sizes(top, 1))
            for T in range(17, top + 1):
                assert lib.floe_moe_layer_decode(C.byref(L), fake, T, fake, None, ws, layer_bytes, None) == -5, (T, top)
                assert lib.floe_expert_ffn_sparse(C.byref(e), fake, T, fake, None, fake, None, None, ws, expert_bytes, None) == -5, (T, top)
    finally:
        lib.floe_tuning(1, 0), lib.floe_tuning(4, 0)


@pytest.mark.parametrize("d,f,bits,group,n,top_k,n_shared,T", [
    (3072, 14784, 4, 64, 32, 4, 0, 19), (2560, 6911, 4, 128, 6, 2, 0, 3), (1536, 64, 2, 32, 8, 2, 0, 1), (3072, 60000, 3, 64, 8, 2, 0, 2),
])
def test_one_kernel_between_the_powers_of_two_is_not_a_condition(lib, d, f, bits, group, n, top_k, n_shared, T):
    """A workspace that holds the separate kernels serves a call that would rather run the fused one, a list-driven call among them."""
    import torch
    from paper_2505_05950_amd.binding import _Expert, _Layer, _Shape
    if torch.cuda.is_available():
        pytest.skip("the pointers below are made up: without a device the calls end at their first HIP call")
    lib.floe_layer_workspace_bytes.restype = lib.floe_expert_workspace_bytes.restype = C.c_size_t
    p, ws = C.c_void_p(4096), C.c_void_p(1 << 20)
    s = _Shape(d, f, bits, group)
    L, e = _Layer(n, top_k, n_shared, 1, s, 4096, None, 4096, 0, 4096, 0), _Expert(s, 4096, 4096, 4096, 4096, 0, f)
    Te = min(T, 16)

    def sizes():
        return lib.floe_layer_workspace_bytes(C.byref(L), T), lib.floe_expert_workspace_bytes(C.byref(s), Te)

    def tuned(key, value):  # no layer call small enough to be fused; one expert's tokens sharing rows
        lib.floe_tuning(key, value)
        try:
            return sizes()
        finally:
            lib.floe_tuning(key, 0)

    for layer_bytes, expert_bytes in ((tuned(4, 1)[0], tuned(1, 2)[1]), sizes()):
        assert lib.floe_moe_layer_decode(C.byref(L), p, T, p, None, ws, C.c_size_t(layer_bytes), None) == -5
        assert lib.floe_expert_ffn_sparse(C.byref(e), p, Te, p, None, p, None, None, ws, C.c_size_t(expert_bytes), None) == -5
        assert lib.floe_gate_down_sparse(C.byref(e), p, Te, p, p, p, None, p, ws, C.c_size_t(expert_bytes), None) == -5


@pytest.mark.parametrize("shape,layer,one_token,wide", [
    ((1024, 3584, 2, 64), None, (17, 128, 160), (256, 320)),             # batches at which each way measured clearly faster
    ((2048, 5632, 4, 64), None, (17, 48), (96, 200)),
    ((2048, 8000, 4, 64), None, (17, 32), (36, 64)),
    ((4096, 4096, 2, 64), None, (17, 32), (48, 128)),
    ((4096, 14336, 2, 64), None, (), (17, 24, 64)),
    ((2048, 1408, 3, 32), None, (17, 200, 256), ()),
    ((5120, 4000, 2, 64), None, (8, 20), (28, 64)),
    ((5120, 1408, 2, 64), None, (40, 128), (200,)),
    ((2560, 14336, 3, 64), None, (3, 10), (17, 64)),                     # (small ones: the fused kernel, which either choice leaves in place)
    ((3072, 14336, 2, 64), None, (4, 6), (16, 24)),
    ((2048, 8000, 2, 128), None, (17, 64, 128), (200, 320)),
    ((1024, 14336, 2, 32), None, (17, 96), (200, 320)),
    ((4096, 14336, 4, 128), None, (), (17, 64)),
    ((1536, 3000, 8, 64), None, (64, 200), ()),
    ((2560, 6911, 2, 64), None, (17,), (48, 200)),
    ((1024, 3584, 2, 64), (8, 2, 0), (64, 96, 128), (200, 512)),
    ((4096, 14336, 2, 64), (8, 2, 0), (), (40, 64, 512)),
    ((2048, 1408, 3, 32), (64, 6, 2), (33,), (82, 132, 512)),
    ((1024, 2048, 2, 64), (64, 8, 0), (48, 64), (128, 256)),
    ((2048, 3000, 2, 32), (8, 2, 0), (40, 64), (96, 128)),
    ((2048, 5632, 4, 64), (8, 2, 0), (32, 40), (64, 128)),
    ((1536, 2048, 4, 64), (24, 4, 1), (25,), (60, 160)),
    ((3072, 4000, 2, 64), (8, 2, 0), (12,), (40, 128)),
    ((4096, 4000, 3, 64), (8, 2, 0), (), (17, 40)),
    ((4096, 1200, 4, 64), (8, 2, 0), (24, 40), (136,)),
    ((1024, 4000, 4, 32), (4, 2, 0), (), (40, 68)),
    ((2048, 1408, 3, 32), (128, 6, 2), (40,), (100,)),                   # (40: 2.5 tasks per expert, no grouped kernel: the packed one is more accurate)
    ((2560, 8000, 4, 64), (8, 2, 0), (6, 9, 24), (32, 64)),
    ((2560, 2048, 2, 64), (48, 6, 2), (4, 8, 18), (40,)),                # (18: the fused launch would be uneven)
])
def test_each_batch_runs_the_way_that_measured_faster(lib, shape, layer, one_token, wide):
    """Seen by the workspace that is asked for: the same as with the one-token kernels forced, or not."""
    from paper_2505_05950_amd.binding import _Layer, _Shape
    lib.floe_layer_workspace_bytes.restype = lib.floe_expert_workspace_bytes.restype = C.c_size_t
    s = _Shape(*shape)

    def size(T, mode):
        lib.floe_tuning(1, mode)
        if layer is None:
            return lib.floe_expert_workspace_bytes(C.byref(s), T)
        n, top_k, n_shared = layer
        return lib.floe_layer_workspace_bytes(C.byref(_Layer(n, top_k, n_shared, 1, s, 4096, None, 4096, 0, 4096, 0)), T)

    try:
        for T in one_token:
            assert size(T, 0) == size(T, 3), T
        for T in wide:
            assert size(T, 0) == size(T, 1), T
    finally:
        lib.floe_tuning(1, 0)
