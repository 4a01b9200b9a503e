"""The entry point that allocates nothing (smha_forward_static) against smha_forward, through the C ABI."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def test_static_workspace_entry_point_matches_forward_on_two_calls_in_a_row():
    """Two calls in a row through the library's own workspace array, the second with a smaller input (a quarter of the
    heads, half the head size): each output equals smha_forward's bit for bit (the merge of
    split 128-row groups runs in a fixed order) and matches the oracle; an unprepared shape is refused."""
    import torch
    import paper_2506_06095_amd as smha
    assert torch.cuda.is_available(), "this test needs the GPU"
    gen = torch.Generator(device="cuda").manual_seed(21)
    cases = [
        (W.MaskSpec(flags=W.BIGBIRD, block=64, n_window_blocks=3, n_global_blocks=2, n_random_blocks=2, seed=4), 1, 8, 4096, 128),
        (W.MaskSpec(flags=W.WINDOW | W.GLOBAL, window_left=32, window_right=32, n_global=70), 1, 2, 4096, 64),
        # the wave form's own workspace: parts of 32 rows, one counter a group
        (W.MaskSpec(flags=W.WINDOW | W.GLOBAL, window_left=20, window_right=20, n_global=40), 1, 9, 6000, 64),
        (W.MaskSpec(flags=W.WINDOW | W.GLOBAL, window_left=20, window_right=20, n_global=5), 1, 3, 6000, 128),
    ]
    for spec, B, H, S, d in cases:
        form = 1 if (S, d) == (4096, 64) else 0                 # (left to the library it takes the wave form, which cuts nothing here)
        with smha.Plan.from_desc(spec, B, H, S, head_dim=d, force=smha.SMHA_KERNEL_BLOCK, block_form=form) as plan:
            assert plan.info()["n_split_rows"] > 0              # the call really uses the workspace and its counters
            if S == 6000:
                assert smha.smha_call_kernel_name(plan.handle, B, H, d, smha.SMHA_F16) == "smha_wave_fwd"
                assert (plan.export("wave_items").reshape(-1, 8)[:, 3] >= 0).any()
            q, k, v = (torch.randn(B, H, S, d, device="cuda", generator=gen).half() for _ in range(3))
            out = torch.full_like(q, float("nan"))
            with pytest.raises(smha.SmhaError):                 # nothing prepared yet: the entry point may not allocate
                plan.forward_static(q, k, v, out)
            plan.prepare(B, H, d)
            for rep in range(2):                                # (the second call finds the counters as the first left them)
                out.fill_(float("nan"))
                plan.forward_static(q, k, v, out)
                torch.cuda.synchronize()
                want = plan.forward(q, k, v)
                torch.cuda.synchronize()
                assert torch.equal(out, want), (S, rep)
            masks = W.dense_mask(spec, B, H, S)
            Qb, Kb, Vb = (x.cpu().numpy().view(np.uint16) for x in (q, k, v))
            h = H - 1
            ref = oracle.masked_attention(*(np.ascontiguousarray(x[:1, h:h + 1]) for x in (Qb, Kb, Vb)), "f16", masks)
            got = out[:1, h:h + 1].float().cpu().numpy().astype(np.float64)
            assert np.abs(got - ref).max() <= 5e-3
            assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-3


@pytest.mark.parametrize("H,S", [(2, 512), (16, 4096)])
def test_a_call_shape_that_ran_with_one_type_serves_the_other(H, S):
    """At 64 columns both input types run the same form, so a float16 forward prepares the bfloat16 call too."""
    import torch
    import paper_2506_06095_amd as smha
    spec = W.MaskSpec(flags=W.WINDOW | W.GLOBAL, window_left=32, window_right=32, n_global=8)
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, H, S, 64, device="cuda", generator=g) for _ in range(3))
    with smha.Plan.from_desc(spec, 1, H, S, head_dim=64, force=smha.SMHA_KERNEL_BLOCK) as plan:
        plan.forward(q.half(), k.half(), v.half())
        args = [x.bfloat16() for x in (q, k, v)]
        out = torch.full_like(args[0], float("nan"))
        plan.forward_static(*args, out)
        assert torch.equal(out, plan.forward(*args))


@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_a_plan_destroyed_on_another_thread_leaves_a_capture_alone(mode):
    """A capture that only binds its own thread survives the end of another thread's plan (a finaliser, say), also of a
    plan whose launches have to be waited for."""
    import threading

    import torch
    import paper_2506_06095_amd as smha
    spec = W.MaskSpec(flags=W.WINDOW | W.GLOBAL, window_left=40, window_right=9, n_global=8)
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, 4, 512, 64, device="cuda", generator=g).half() for _ in range(3))
    out = torch.empty_like(q)
    with smha.Plan.from_desc(spec, 1, 4, 512, head_dim=64, force=smha.SMHA_KERNEL_BLOCK) as plan:
        plan.prepare(1, 4, 64)
        eager = plan.forward(q, k, v)
        torch.cuda.synchronize()
        other = smha.Plan.from_desc(spec, 1, 4, 512, head_dim=64, force=smha.SMHA_KERNEL_BLOCK)
        elsewhere, side, graph = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
        kept = other.forward(q, k, v, stream=elsewhere)  # noqa: F841 (its memory is held until it has run)
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side, capture_error_mode=mode):
            closer = threading.Thread(target=other.close)
            closer.start()
            closer.join()
            plan.forward(q, k, v, out=out)
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager)


SPLIT_SPEC = W.MaskSpec(flags=W.WINDOW | W.GLOBAL, window_left=32, window_right=32, n_global=8)  # (1000 keys: whole lists; 6000: cut ones)


def smha_width(d):
    return next(w for w in (32, 64, 96, 128, 160, 256) if d <= w)


def widths_of_kernels_run(torch, call):
    """The kernel widths of the attention kernels that the call launches."""
    import re
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [int(m[1]) for m in (re.search(r"smha_\w*fwd\w*<(\d+)", e.key) for e in prof.key_averages()) if m]


@pytest.mark.parametrize("S", [1000, 6000])
@pytest.mark.parametrize("prepared,d", [(64, 24), (128, 80), (256, 136), (24, 64), (80, 128), (136, 256)])
def test_what_one_head_size_prepared_serves_the_others_of_its_64_128_or_256_columns(prepared, d, S):
    """... where nothing may be allocated (smha_forward_static, a forward that is captured): at the wider width, both results
    against the oracle; with nothing prepared, or another batch size, the entry point refuses."""
    import torch
    import paper_2506_06095_amd as smha
    B, H = 2, 4
    g = torch.Generator(device="cuda").manual_seed(d)
    q, k, v = (torch.randn(B, H, S, d, device="cuda", generator=g).half() for _ in range(3))
    ref = oracle.masked_attention(*(np.ascontiguousarray(x[1:, 3:].cpu().numpy().view(np.uint16)) for x in (q, k, v)), "f16",
                                  W.dense_mask(SPLIT_SPEC, B, H, S)[-1:, -1:])

    def check(out):
        got = out[1:, 3:].double().cpu().numpy()
        assert np.abs(got - ref).max() <= 5e-3 and np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-3
    for form in (0, 1):
        with smha.Plan.from_desc(SPLIT_SPEC, B, H, S, head_dim=d, force=smha.SMHA_KERNEL_BLOCK, block_form=form) as plan:
            if form == 0:
                assert smha.smha_call_kernel_name(plan.handle, B, H, d, smha.SMHA_F16) == "smha_wave_fwd"
                assert (plan.export("wave_items").reshape(-1, 8)[:, 3] >= 0).any() == (S == 6000)
            assert S == 1000 or plan.info()["n_split_rows"] > 0
            out = torch.full_like(q, float("nan"))
            with pytest.raises(smha.SmhaError):
                plan.forward_static(q, k, v, out)
            plan.prepare(B, H, prepared)
            with pytest.raises(smha.SmhaError):
                plan.forward_static(q[:1], k[:1], v[:1], out[:1])
            for _ in range(2):
                plan.forward_static(q, k, v, out.fill_(float("nan")))
                check(out)
            assert widths_of_kernels_run(torch, lambda: plan.forward_static(q, k, v, out)) == [smha_width(max(prepared, d))]
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                plan.forward(q, k, v, out=out)
            for _ in range(3):
                out.fill_(float("nan"))
                graph.replay()
                check(out)
            plan.prepare(B, H, d)
            plan.forward_static(q, k, v, out.fill_(float("nan")))
            check(out)
            assert torch.equal(out, plan.forward(q, k, v))
            assert widths_of_kernels_run(torch, lambda: plan.forward_static(q, k, v, out)) == [smha_width(d)]


@pytest.mark.parametrize("before,d", [(64, 32), (128, 96), (256, 160), (96, 128)])
def test_a_forward_runs_at_its_own_width_whatever_ran_before(before, d):
    import torch
    import paper_2506_06095_amd as smha
    g = torch.Generator(device="cuda").manual_seed(d)
    q, k, v = (torch.randn(2, 4, 1000, d, device="cuda", generator=g).half() for _ in range(3))
    x = torch.randn(2, 4, 1000, before, device="cuda", generator=g).half()
    make = lambda: smha.Plan.from_desc(SPLIT_SPEC, 2, 4, 1000, head_dim=d, force=smha.SMHA_KERNEL_BLOCK)  # noqa: E731
    with make() as plan, make() as other:
        other.forward(x, x, x)
        assert torch.equal(other.forward(q, k, v), plan.forward(q, k, v))
        name = smha.smha_call_kernel_name(other.handle, 2, 4, d, smha.SMHA_F16)
        assert name == smha.smha_call_kernel_name(plan.handle, 2, 4, d, smha.SMHA_F16)
        assert widths_of_kernels_run(torch, lambda: other.forward(q, k, v)) == [d]
