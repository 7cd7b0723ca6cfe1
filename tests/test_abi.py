"""Host-only checks of the C ABI: the library loads without a GPU, exports every entry point the
header declares, and rejects bad shapes before anything could be launched."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "moehot.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(moe_[a-z_0-9]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    from paper_2411_10003_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2411_10003_amd import build
        build.build(verbose=False)
    return binding.load()


def test_every_declared_symbol_is_exported(lib):
    from paper_2411_10003_amd import binding
    names = _declared()
    assert len(names) >= 15
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(binding.EXPORTS) == names


def test_create_validates_shapes(lib):
    from paper_2411_10003_amd.binding import _Shape
    good = dict(T=64, d=64, h=128, E=8, k=2, P=4, self=0, G=2, dtype=1, act=0, renorm=1)

    def create(**kw):
        f = dict(good)
        f.update(kw)
        s = _Shape(*(f[n] for n, _ in _Shape._fields_))
        h = ctypes.c_void_p()
        rc = lib.moe_create(ctypes.byref(h), ctypes.byref(s))
        if rc == 0:
            n = ctypes.c_size_t()
            assert lib.moe_workspace_bytes(h, ctypes.byref(n)) == 0 and n.value % 256 == 0 and n.value > 0
            assert lib.moe_destroy(h) == 0
        return rc

    assert create() == 0
    assert create(dtype=0, d=36) == 0
    assert create(k=0) == -2 and create(k=9) == -2 and create(E=1) == -2
    assert create(d=100) == -2 and create(h=100) == -2            # bf16 needs multiples of 64
    assert create(dtype=0, d=34) == -2
    assert create(P=9) == -2 and create(self=4) == -2 and create(G=0) == -2 and create(G=9) == -2
    assert create(E=128, G=64) == 0 and create(E=128, G=65) == -2    # bf16: at most 64 hosted groups
    assert create(dtype=0, E=128, G=65) == 0
    assert create(d=64, h=1 << 22) == -2 and create(d=1 << 22, h=64) == -2   # bf16: a 256-row tile is addressed in 32 bits
    assert create(dtype=7) == -5 and create(act=3) == -2 and create(renorm=2) == -2
    assert create(T=0) == -2
    assert lib.moe_create(None, None) == -1
    assert lib.moe_status_string(-3).decode() == "expert placement out of range"


def test_plan_validates_arguments(lib):
    """moe_plan checks its arguments on the host before anything is launched (no GPU needed here)."""
    from paper_2411_10003_amd.binding import _PlanOut, _Planner
    good = dict(D=4, E=8, n=1, overlap=0, alpha=1.0, size_input=8.0, size_params=16.0, size_grads=16.0, B=1.0, t=1.0,
                T_FNEC=0.0, T_BNEC=0.0)
    out = _PlanOut(*([0x1000] * 7))                       # never dereferenced: every call below fails validation

    def call(**kw):
        f = dict(good)
        f.update(kw)
        c = _Planner(*(f[n] for n, _ in _Planner._fields_))
        return lib.moe_plan(ctypes.byref(c), ctypes.c_void_p(0x1000), ctypes.byref(out), None)

    assert lib.moe_plan(None, None, None, None) == -1
    assert call(D=0) == -2 and call(D=65, E=65) == -2 and call(E=6) == -2 and call(E=2048, D=64) == -2
    assert call(n=-1) == -2 and call(n=4) == -2 and call(overlap=2) == -2
    assert call(B=0.0) == -2 and call(t=-1.0) == -2 and call(alpha=float("nan")) == -2 and call(size_params=float("inf")) == -2
    missing = _PlanOut(0x1000, 0, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000)
    c = _Planner(*(good[n] for n, _ in _Planner._fields_))
    assert lib.moe_plan(ctypes.byref(c), ctypes.c_void_p(0x1000), ctypes.byref(missing), None) == -1


def test_trans_validates_arguments(lib):
    """moe_trans checks tensor counts, sizes and alignment on the host (no GPU needed: every call fails early)."""
    from paper_2411_10003_amd.binding import _Shape
    shp = _Shape(64, 64, 128, 8, 2, 4, 0, 2, 1, 0, 1)
    h = ctypes.c_void_p()
    assert lib.moe_create(ctypes.byref(h), ctypes.byref(shp)) == 0
    vp = ctypes.c_void_p
    pools = (vp * 2)(0x1000, 0x2000)
    groups = (vp * 2)(0x3000, 0x4000)
    sizes = (ctypes.c_size_t * 2)(4096, 4096)
    dest, slots, pver, sver = vp(0x5000), vp(0x6000), vp(0x7000), vp(0x8000)
    assert lib.moe_trans(h, None, pver, slots, sver, 2, pools, groups, sizes, None) == -1
    assert lib.moe_trans(h, dest, pver, slots, None, 2, pools, groups, sizes, None) == -1      # versions: both or neither
    assert lib.moe_trans(h, dest, None, slots, sver, 2, pools, groups, sizes, None) == -1
    assert lib.moe_trans(h, dest, pver, slots, sver, 0, pools, groups, sizes, None) == -2
    assert lib.moe_trans(h, dest, pver, slots, sver, 9, pools, groups, sizes, None) == -2
    bad_sizes = (ctypes.c_size_t * 2)(4096, 4100)                   # not a multiple of 16
    assert lib.moe_trans(h, dest, pver, slots, sver, 2, pools, groups, bad_sizes, None) == -2
    bad_pools = (vp * 2)(0x1000, 0x2004)                            # misaligned
    assert lib.moe_trans(h, dest, None, slots, None, 2, bad_pools, groups, sizes, None) == -2
    missing = (vp * 2)(0x1000, 0)
    assert lib.moe_trans(h, dest, pver, slots, sver, 2, missing, groups, sizes, None) == -1
    assert lib.moe_destroy(h) == 0


def test_static_counts_and_settings_validate_arguments(lib):
    """The entry point without a workspace rejects inputs beyond its built-in array before anything is launched;
    moe_set_act_saved takes 0 or 1."""
    from paper_2411_10003_amd.binding import _Shape
    vp = ctypes.c_void_p
    big = _Shape(1 << 22, 64, 128, 1024, 1, 4, 0, 2, 1, 0, 0)       # 16384 chunks x 1024 experts = 2^24 words
    h = ctypes.c_void_p()
    assert lib.moe_create(ctypes.byref(h), ctypes.byref(big)) == 0
    assert lib.moe_expert_counts_static(h, vp(0x1000), vp(0x2000), None) == -8
    assert lib.moe_expert_counts_static(h, None, vp(0x2000), None) == -1
    assert lib.moe_expert_counts_static(None, vp(0x1000), vp(0x2000), None) == -1
    assert b"scratch" in lib.moe_status_string(-8)
    assert lib.moe_set_act_saved(h, 2) == -2 and lib.moe_set_act_saved(h, 1) == 0 and lib.moe_set_act_saved(h, 0) == 0
    assert lib.moe_set_act_saved(None, 1) == -1
    assert lib.moe_destroy(h) == 0


@pytest.mark.parametrize("missing", ["_raw_stream", "_current_device"])
def test_stream_without_the_raw_handle(monkeypatch, missing):
    """Either of torch's two private names may be missing: the stream then comes from its public interface."""
    import torch
    from paper_2411_10003_amd import binding

    class Stream:
        cuda_stream = 4711

    monkeypatch.setattr(binding, "_raw_stream", lambda device: 42)
    monkeypatch.setattr(binding, "_current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream())
    assert binding._stream() == 42
    monkeypatch.setattr(binding, missing, None)
    assert binding._stream() == 4711
