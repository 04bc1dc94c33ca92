"""How alt_conv2d_multi issues lists of convolutions (host only): what is planned is kept, and what goes out together."""
import pytest

import paper_2210_12415_amd as alt
from test_gpu_group import MORE, SETS, describe


def call(i, N, C, H, K, R, dtype=alt.BF16, layout="NHWC", ws=1 << 26, W=None, pad=None, **more):
    """The i-th call of a list, on buffers of its own that nothing reads."""
    pad = R // 2 if pad is None else pad
    d = alt.conv_desc(N, C, H, W or H, K, R, R, pad=pad, in_dtype=dtype, out_dtype=dtype, x_layout="NCHW->" + layout,
                      w_layout="OIHW->" + ("OHWI" if layout == "NHWC" else "OIHW"), y_layout="NCHW->" + layout, **more)
    at = (i + 1) << 40
    return dict(d=d, x=at, w=at + (1 << 36), y=at + (2 << 36), workspace=at + (3 << 36) if ws else None, ws_bytes=ws, stream=0)


def stages(n, batch, width, size, **kw):
    return [call(i, batch, width << i, max(size >> i, 1), width << i, 3, **kw) for i in range(n)]


def test_lists_are_planned_once():
    """Fifty lists that go out as one launch and a hundred that do not, in turn: each is planned on its first pass alone."""
    h = alt.Handle()
    together = [stages(2 + i % 3, 1 + i // 3, 32 + 8 * (i % 5), 28) for i in range(50)]
    # (large layers, calls of two types, and a layout that no kernel of several problems takes)
    apart = ([stages(3, 256, 64, 56 + i) for i in range(10)] + [[call(0, 1 + i, 64, 14, 64, 3), call(1, 1 + i, 64, 14, 64, 3, dtype=alt.F32)] for i in range(45)] +
             [[call(j, 1 + i, 64, 14, 64, 3, layout="NCHW16c", ) for j in range(2)] for i in range(45)])
    for again in (0, 1, 1):
        for i in range(100):
            plans = [h.conv2d_multi_plan(apart[i])] + ([h.conv2d_multi_plan(together[i])] if i < 50 else [])
            assert all(p.kept == again for plan in plans for p in plan), (again, i)
            assert [p.launch for p in plans[0]] == list(range(len(apart[i]))) and all((p.family, p.body, p.slices) == (0, -1, 0) for p in plans[0])
            for p in plans[1:]:
                assert all(q.launch == 0 and q.family == 2 and q.body >= 0 and q.slices >= 1 for q in p)


def test_kept_lists_are_told_apart():
    """By sizes, layouts, alignment, workspaces and the flags of every call, the last one's too."""
    h = alt.Handle()
    base = lambda: stages(3, 1, 64, 28)
    assert [p.kept for p in h.conv2d_multi_plan(base()) + h.conv2d_multi_plan(base())] == [0] * 3 + [1] * 3

    def changed(i, **more):
        calls = base()
        calls[i] = dict(call(i, 1, 64 << i, 28 >> i, 64 << i, 3, **{k: v for k, v in more.items() if k not in calls[i]}),
                        **{k: v for k, v in more.items() if k in calls[i]})
        return calls

    other = [changed(i, **m) for i in range(3) for m in (dict(y=((i + 1) << 40) + (2 << 36) + 8), dict(ws_bytes=1 << 20), dict(epilogue=alt.EPI_RELU),
                                                         dict(layout="NCHW"), dict(dil=2, pad=2), dict(dtype=alt.F32), dict(W=29))]
    other += [base()[:2], base() + base()[:1]]
    for calls in other:
        assert not any(p.kept for p in h.conv2d_multi_plan(calls))
        assert all(p.kept for p in h.conv2d_multi_plan(calls))


def test_windows_streams_and_buffers():
    h = alt.Handle()
    nine = [call(i, 1, 16 + 8 * i, 10, 24, 3) for i in range(9)]
    assert [p.launch for p in h.conv2d_multi_plan(nine)] == [0] * 8 + [1]
    for c in nine[4:]:
        c["stream"] = 64
    assert [p.launch for p in h.conv2d_multi_plan(nine)] == [0] * 4 + [1] * 5
    # one reads what another writes
    two = nine[:2]
    assert [p.launch for p in h.conv2d_multi_plan(two)] == [0, 0]
    two[1] = dict(two[1], x=two[0]["y"] + 64)
    assert [(p.launch, p.family) for p in h.conv2d_multi_plan(two)] == [(0, 0), (1, 0)]
    two[1] = dict(two[1], x=nine[1]["x"], d=call(1, 1, 24, 10, 24, 3, variant=0)["d"])
    assert [(p.launch, p.kept) for p in h.conv2d_multi_plan(two)] == [(0, 1), (1, 1)]
    assert h.conv2d_multi_plan([]) == []


@pytest.mark.parametrize("kind,family,bodies", [(("f32", "NHWC"), 1, 6), (("bf16", "NHWC"), 2, 9), (("bf16", "NCHW"), 3, 8)])
def test_the_lists_run_on_the_gpu_reach_every_body(kind, family, bodies):
    """.. and sums in slices, of one tap and of nine (channel-planar kernels take none)."""
    h = alt.Handle()
    dtype, layout = kind
    reached, sliced = set(), set()
    for problems in [SETS[kind]] + MORE[kind]:
        calls = []
        for i, problem in enumerate(problems):
            d, ws_elems = describe(dtype, layout, problem, alt.F32 if dtype == "f32" or problems is SETS[kind] else alt.BF16)
            at = (i + 1) << 40
            calls.append(dict(d=d, x=at, w=at + (1 << 36), y=at + (2 << 36), bias=at + (5 << 36) if problem[7] else None, workspace=at + (3 << 36),
                              ws_bytes=4 * ws_elems, stream=0))
        plan = h.conv2d_multi_plan(calls)
        assert all((p.launch, p.family) == (0, family) for p in plan)
        reached |= {p.body for p in plan}
        sliced |= {problem[5] for p, problem in zip(plan, problems) if p.slices > 1}
    assert reached == set(range(bodies))
    assert sliced == {"f32": {1, 3}, "bf16": {1} if layout == "NHWC" else set()}[dtype]
