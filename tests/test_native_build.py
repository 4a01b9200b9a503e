"""The native call path's build: what makes it stale, that a failed build leaves what was there, and that Plan.forward does without."""
import os
import subprocess

import pytest

import workloads as W
from paper_2506_06095_amd import binding, build


def test_the_native_module_is_stale_with_another_header_source_or_torch(monkeypatch, tmp_path):
    import torch
    binding._load_native()
    assert build.extension_current()
    for name in ("ABI_HEADER", "EXT_SOURCE"):
        with monkeypatch.context() as m:
            changed = tmp_path / name
            changed.write_bytes(open(getattr(build, name), "rb").read() + b"\n")
            m.setattr(build, name, str(changed))
            assert not build.extension_current()
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "0.0")
        assert not build.extension_current()
    with monkeypatch.context() as m:
        m.setattr(build, "EXT", str(tmp_path / "none.so"))
        assert not build.extension_current()


def test_a_failed_build_of_the_native_module_leaves_the_old_one(monkeypatch, tmp_path):
    old = tmp_path / "_smha_torch.so"
    old.write_bytes(b"old")
    monkeypatch.setattr(build, "EXT", str(old))
    monkeypatch.setenv("CXX", "false")
    with pytest.raises(subprocess.CalledProcessError):
        build.build_extension()
    assert old.read_bytes() == b"old" and os.listdir(tmp_path) == ["_smha_torch.so"]


def hide_native_module(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(build, "EXT", str(tmp_path / "_smha_torch.so"))
    monkeypatch.setenv("CXX", "false")


def test_without_the_native_module_calls_go_the_general_way(monkeypatch, tmp_path):
    import torch
    hide_native_module(monkeypatch, tmp_path)
    x = torch.zeros(1, 1, 64, 64, dtype=torch.float16)
    with binding.Plan.from_desc(W.MaskSpec(flags=W.CAUSAL), 1, 1, 64, device_id=-2) as plan:
        with pytest.warns(RuntimeWarning, match="native call path"), pytest.raises(ValueError, match="on the GPU"):
            plan.forward(x, x, x)
        with pytest.raises(ValueError, match="on the GPU"):  # (no second warning: they are errors here)
            import warnings
            with warnings.catch_warnings():
                warnings.simplefilter("error")
                plan.forward(x, x, x)


@pytest.mark.gpu
def test_without_the_native_module_results_are_the_same(monkeypatch, tmp_path):
    import torch
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(2, 3, 130, 64, device="cuda", generator=g).half() for _ in range(3))
    with binding.Plan.from_desc(W.MaskSpec(flags=W.WINDOW, window_left=20, window_right=3), 2, 3, 130, head_dim=64) as plan:
        want = plan.forward(q, k, v)
        hide_native_module(monkeypatch, tmp_path)
        with pytest.warns(RuntimeWarning, match="native call path"):
            assert torch.equal(plan.forward(q, k, v), want)
