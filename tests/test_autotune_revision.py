"""The variant search leaves out what a context does not use and keeps no setting past a
change of the kernels (CPU: the timing and the device are stand-ins)."""
import json

import pytest

from paper_2503_22227_amd import autotune as A
from paper_2503_22227_amd.fhe import Context


class Ctx:
    scheme, log_n, alpha, device = "ckks", 15, 8, 0
    q, p = [97, 193], [257]

    def __init__(self, fused):
        self.fused_modup = fused
        self.levels = {}

    def get_tuning(self, nl):
        return dict(self.levels.get(nl, A.DEFAULT_LEVEL))

    def set_tuning(self, nl, setting):
        self.levels[nl] = dict(setting)


def _setup(tmp_path, monkeypatch):
    monkeypatch.setenv("RF_AUTOTUNE_CACHE", str(tmp_path / "cache.json"))
    monkeypatch.setattr(A, "device_key", lambda device=None: "fake")


@pytest.mark.parametrize("fused", [False, True])
def test_modup_chunk_is_searched_only_where_a_launch_reads_it(fused, tmp_path, monkeypatch):
    _setup(tmp_path, monkeypatch)
    ctx = Ctx(fused)
    seen = set()

    def fake_time(fn, reps, repeats=3):
        t = ctx.levels[2]
        seen.add(t["modup_chunk"])
        return 1.0 - 0.1 * (t["modup_chunk"] == 4)

    monkeypatch.setattr(A, "time_fn", fake_time)
    res = A.tune_level(ctx, 2, lambda: None)
    assert res["setting"]["modup_chunk"] == (8 if fused else 4)
    assert seen == ({8} if fused else {4, 8, 16})


def test_a_new_kernel_revision_searches_again(tmp_path, monkeypatch):
    _setup(tmp_path, monkeypatch)
    ctx = Ctx(True)
    monkeypatch.setattr(A, "time_fn", lambda fn, reps, repeats=3: 1.0)
    assert not A.tune_level(ctx, 2, lambda: None)["cached"]
    assert A.tune_level(ctx, 2, lambda: None)["cached"]
    shape = A.shape_key([(14, 3)])
    monkeypatch.setattr(A, "KERNEL_REVISION", A.KERNEL_REVISION + 1)
    assert not A.tune_level(ctx, 2, lambda: None)["cached"]
    assert A.shape_key([(14, 3)]) != shape
    assert len(json.load(open(tmp_path / "cache.json"))["fake"]) == 2


NARROW, WIDE = [(1 << 45) + 1], [(1 << 50) + 1]


@pytest.mark.parametrize("scheme,log_n,alpha,q,fused", [
    ("ckks", 12, 4, WIDE, True), ("ckks", 13, 4, WIDE, False), ("ckks", 13, 1, WIDE, True),
    ("ckks", 16, 4, NARROW, True), ("bgv", 15, 2, NARROW, True), ("bfv", 15, 2, NARROW, False),
    ("ckks", 13, 4, [1 << 46], False), ("bfv", 15, 1, WIDE, True)])
def test_which_contexts_launch_a_conversion(scheme, log_n, alpha, q, fused):
    ctx = object.__new__(Context)
    ctx.scheme, ctx.log_n, ctx.alpha, ctx.q, ctx.p, ctx._h = scheme, log_n, alpha, q, WIDE, None
    assert ctx.fused_modup is fused
