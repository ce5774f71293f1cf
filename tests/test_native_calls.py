"""_hmcall: what it takes, and what it leaves to the binding's Python code."""
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2508_09591_amd import binding as B

NAMES = [n[3:] for n in B._NATIVE]


def test_every_entry_point_is_handed_over_in_order():
    B.lib()
    assert all(callable(getattr(B._native, n)) for n in NAMES)
    with pytest.raises(TypeError):
        B._native.bind(1, 2)


@pytest.mark.parametrize("name", NAMES)
def test_anything_out_of_the_ordinary_is_left_to_python(name):
    B.lib()
    f = getattr(B._native, name)
    cpu = torch.zeros((4, 8), dtype=torch.bfloat16)
    for n in range(18):
        for arg in (None, 1, 1.5, "x", [1, 2], cpu, torch.zeros((4, 8), dtype=torch.float32, device="meta")):
            assert f(*[arg] * n) is None


def test_a_refused_call_changes_nothing():
    """The plan's table is only adopted by a call that is made."""
    B.lib()
    c = B.hm_plan_out()
    e = lambda *shape, dtype=torch.int32: torch.zeros(shape, dtype=dtype)
    plan = B.Plan(T=4, K=2, level=1, num_dest=4, row_capacity=8, dest_count=e(4), dest_offset=e(5), row_token=e(8), slot_row=e(8),
                  slot_keep=e(8, dtype=torch.uint8), row_weight=e(8, dtype=torch.float32), rank_mask=None, node_mask=None, status=e(1),
                  workspace=e(64), c=c)
    assert B._native.plan(e(2, 2), e(2, 2, dtype=torch.float32), e(8), 2, 2, 1, plan) is None
    assert (plan.T, plan.K, plan.num_dest) == (4, 2, 4)
    with pytest.raises(TypeError):
        B.hm_plan(e(2, 2), e(2, 2, dtype=torch.float32), e(8), 2, 2, 1, plan=plan)


def test_the_library_works_without_the_native_half():
    """A binding that cannot load _hmcall says so and has every entry point all the same."""
    code = ("import sys, warnings; sys.modules['paper_2508_09591_amd._hmcall'] = None\n"
            "from paper_2508_09591_amd import binding as B\n"
            "with warnings.catch_warnings(record=True) as w:\n"
            "    warnings.simplefilter('always'); L = B.lib(); B.lib()\n"
            "assert [x.category for x in w] == [RuntimeWarning] and '_hmcall' in str(w[0].message), w\n"
            "assert all(hasattr(L, n) for n in B.EXPORTS) and B.status_string(-2) == 'bad shape'\n"
            "assert B.hm_plan_workspace_bytes(8192, 8, 256, 4, 8, 2) > 0 and B._native.plan(1, 2) is None\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=B.os.path.dirname(B.os.path.dirname(B.__file__)))
    assert r.returncode == 0, r.stderr


# ---- on the GPU: each call by each way into the library -------------------------------------------------
class _Recorder:
    """_hmcall with a note of each call: its name and whether it was taken."""
    def __init__(self, native):
        self.native, self.calls = native, []

    def __getattr__(self, name):
        def call(*args):
            rc = getattr(self.native, name)(*args)
            self.calls.append((name, rc is not None))
            return rc
        return call


def _world():
    """name -> (call(stream), outputs); every call on tensors of its own, small and ragged."""
    T, K, E, nodes, rpn, H = 701, 6, 48, 3, 4, 264
    G, rng = nodes * rpn, np.random.default_rng(12)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    full = lambda *shape, dtype=torch.int32: torch.full(shape, 55, dtype=dtype, device="cuda")
    bf16, f32, f64 = torch.bfloat16, torch.float32, torch.float64
    ids = rng.integers(0, E, (T, K), dtype=np.int32)
    ids[rng.random((T, K)) < 0.1] = -1
    ids, w, e2r = dev(ids), dev(rng.random((T, K), dtype=np.float32)), dev((np.arange(E) * G // E).astype(np.int32))
    rows = lambda n, dtype: dev(rng.standard_normal((n, H), dtype=np.float32)).to(dtype)
    plan = B.hm_plan(ids, w, e2r, nodes, rpn, B.HM_DEDUP_GPU)
    n = B.hm_plan_status(plan)[1]
    table = torch.where(e2r < rpn, e2r, torch.full_like(e2r, -1))
    world = {}

    def fields(p):
        return [t for t in (p.dest_count, p.dest_offset, p.row_token, p.slot_row, p.slot_keep, p.row_weight, p.rank_mask, p.node_mask, p.status,
                            p.load_expert, p.load_rank, p.load_node) if t is not None]

    p1 = B.alloc_plan(T, K, E, nodes, rpn, B.HM_DEDUP_NODE, loads=True)
    world["plan"] = (lambda s: B.hm_plan(ids, w, e2r, nodes, rpn, B.HM_DEDUP_NODE, plan=p1, stream=s), fields(p1))
    p2 = B.alloc_plan(T, K, E, 1, 1, B.HM_DEDUP_GPU, num_dest=rpn)
    world["plan_mapped"] = (lambda s: B.hm_plan_mapped(ids, w, table, rpn, True, plan=p2, stream=s), fields(p2))
    x, y, yf, xf = rows(T, bf16), rows(n, bf16), rows(n, f32), rows(T, f32)
    for name, fn, t, out in (("dispatch_pack", B.hm_dispatch_pack, x, full(n, H, dtype=bf16)), ("combine_transpose", B.hm_combine_transpose, xf, full(n, H, dtype=f32)),
                             ("combine_transpose_bf16", B.hm_combine_transpose_bf16, x, full(n, H, dtype=bf16))):
        world[name] = (lambda s, fn=fn, t=t, out=out: fn(t, plan, out, stream=s), [out])
    for name, fn, t, dtype in (("combine", B.hm_combine, y, bf16), ("combine_f32", B.hm_combine_f32, yf, f32), ("combine_mix", B.hm_combine_mix, y, bf16)):
        a, b = full(T, H, dtype=dtype), full(T, H, dtype=dtype)
        world[name] = (lambda s, fn=fn, t=t, a=a, b=b: (fn(t, w, plan, a, stream=s), fn(t, None, plan, b, stream=s)), [a, b])
    load, own, st = [full(E), full(G), full(nodes)], full(3, 64), [full(1) for _ in range(3)]
    world["expert_load"] = (lambda s: B.hm_expert_load(ids, e2r, nodes, rpn, *load, status=st[0], stream=s), load + st[:1])
    world["group_counts"] = (lambda s: B.hm_group_counts(ids, e2r, G, (G, nodes, 1), own, status=st[1], stream=s), [own, st[1]])
    pi, times, best = dev(rng.integers(0, 999, (2, 64), dtype=np.int32)), full(4, dtype=f64), full(1)
    world["alltoall_times"] = (lambda s: B.hm_alltoall_times([1, nodes], G, 264, 2.0, pi, pi, [0.0, 0.3], [0.0, 1e-7], [0.7, 0.1], [5e-7, 1e-7], times, best,
                                                             stream=s), [times, best])
    Z = [full(E, E, nodes), full(E, E, G)]
    ws = full(int(B.lib().hm_swap_multi_workspace_bytes(T, K, E, G, 2, (B.ctypes.c_int32 * 2)(nodes, G))) // 4 + 1)
    world["swap_counts_multi"] = (lambda s: B.hm_swap_counts_multi(ids, e2r, G, [nodes, G], Z, status=st[2], workspace=ws, stream=s), Z + st[2:])
    zi, za = dev(rng.integers(1, 99, (E, E, nodes), dtype=np.int32)), dev(rng.integers(1, 99, (E, E, G), dtype=np.int32))
    Q, pair, time = full(E, E, dtype=f64), full(2), full(1, dtype=f64)
    ws2 = full(int(B.lib().hm_swap_select_workspace_bytes(E)) // 8 + 1, dtype=f64)
    world["swap_select"] = (lambda s: B.hm_swap_select([1, nodes], G, 264.0, 2, [None, zi], za, [0.0, 1.0], 3, [0.0, 0.3], [0.0, 1e-7], 0.1, 1e-7, 10.0, Q, pair, time,
                                                       workspace=ws2, stream=s), [Q, pair, time])
    placed, chosen = e2r.clone(), dev(np.array([1, E - 2], dtype=np.int32))
    world["swap_apply"] = (lambda s: B.hm_swap_apply(placed, chosen, stream=s), [placed])
    torch.cuda.synchronize()
    return world, e2r


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_every_way_into_the_library_gives_the_same(name, monkeypatch):
    """Through _hmcall, on the default stream, on the current stream of a context and into a graph; through ctypes on a given stream and where
    _hmcall is absent: the same bits, and each way the one that was meant."""
    B.lib()
    world, e2r = _world()
    call, outputs = world[name]
    native, fill = B._native, lambda: [o.copy_(e2r) if name == "swap_apply" else o.fill_(77) for o in outputs]
    want = {"combine": 2, "combine_f32": 2, "combine_mix": 2}.get(name, 1)

    def run(way, taken, do):
        rec = _Recorder(native)
        monkeypatch.setattr(B, "_native", rec)
        fill()
        torch.cuda.synchronize()
        do()
        torch.cuda.synchronize()
        monkeypatch.setattr(B, "_native", native)
        assert rec.calls == [(name, True)] * taken, (name, way, rec.calls)
        return [o.clone() for o in outputs]

    ref = run("current", want, lambda: call(None))
    assert any(bool((o != (e2r if name == "swap_apply" else 77)).any()) for o in ref), name
    same = lambda got: all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(ref, got))
    side = torch.cuda.Stream()

    def inside():
        with torch.cuda.stream(side):
            call(None)
    assert same(run("context", want, inside)), name
    assert same(run("given stream", 0, lambda: call(side))), name
    graph = torch.cuda.CUDAGraph()

    def capture():
        with torch.cuda.graph(graph):      # a launch on any other stream would not be recorded
            call(None)
    run("capture", want, capture)
    for _ in range(3):
        assert same(run("replay", 0, graph.replay)), name
        assert same(run("between replays", want, lambda: call(None))), name
    monkeypatch.setattr(B, "_native", B._Absent("not here"))
    fill()
    call(None)
    torch.cuda.synchronize()
    assert same([o.clone() for o in outputs]), name


@pytest.mark.gpu
def test_what_does_not_fit_is_refused_before_any_launch(monkeypatch):
    """GPU tensors of the wrong size, type or layout: _hmcall leaves them to the Python code, which raises; the plan describes the
    table it did before."""
    B.lib()
    T, K, E, H = 64, 4, 16, 32
    e = lambda *shape, dtype=torch.int32: torch.zeros(shape, dtype=dtype, device="cuda")
    bf16, f32, f16 = torch.bfloat16, torch.float32, torch.float16
    ids, w, e2r = e(T, K), e(T, K, dtype=f32), e(E)
    plan = B.hm_plan(ids, w, e2r, 1, 4, B.HM_DEDUP_GPU)
    few_masks = B.alloc_plan(T, K, E, 1, 4, B.HM_DEDUP_GPU)
    x, rows, out = e(T, H, dtype=bf16), e(T * K, H, dtype=bf16), e(T, H, dtype=bf16)
    rec = _Recorder(B._native)
    monkeypatch.setattr(B, "_native", rec)
    level = B.HM_DEDUP_GPU
    twice = e(2 * T, 2 * H, dtype=bf16)
    cases = [
        (ValueError, lambda: B.hm_plan(e(T + 1, K), e(T + 1, K, dtype=f32), e2r, 1, 4, level, plan=plan)),           # more slots than the plan has room for
        (ValueError, lambda: B.hm_plan(e(T, K + 1), e(T, K + 1, dtype=f32), e2r, 1, 4, level, plan=plan)),
        (ValueError, lambda: B.hm_plan(e(2 * T, K // 2), e(2 * T, K // 2, dtype=f32), e2r, 1, 4, level, plan=few_masks)),   # as many slots, more tokens
        (ValueError, lambda: B.hm_plan(ids, e(T, K - 1, dtype=f32), e2r, 1, 4, level, plan=plan)),
        (ValueError, lambda: B.hm_plan_mapped(ids, e(T + 1, K, dtype=f32), e2r, 4, True, plan=plan)),
        (TypeError, lambda: B.hm_plan(ids.long(), w, e2r, 1, 4, level, plan=plan)),
        (TypeError, lambda: B.hm_plan(ids, w.to(f16), e2r, 1, 4, level, plan=plan)),
        (TypeError, lambda: B.hm_plan(e(K, T).t(), w, e2r, 1, 4, level, plan=plan)),
        (TypeError, lambda: B.hm_plan_mapped(ids, w, e2r.cpu(), 4, True, plan=plan)),
        (ValueError, lambda: B.hm_dispatch_pack(e(T + 1, H, dtype=bf16), plan, rows)),
        (ValueError, lambda: B.hm_dispatch_pack(x[:-1], plan, rows)),
        (TypeError, lambda: B.hm_dispatch_pack(x.to(f16), plan, rows)),
        (TypeError, lambda: B.hm_dispatch_pack(twice[::2, :H], plan, rows)),
        (TypeError, lambda: B.hm_dispatch_pack(x, plan, e(T * K, 2 * H, dtype=bf16)[:, ::2])),
        (ValueError, lambda: B.hm_combine_transpose(e(T + 1, H, dtype=f32), plan, e(T * K, H, dtype=f32))),
        (TypeError, lambda: B.hm_combine_transpose(x, plan, e(T * K, H, dtype=f32))),
        (ValueError, lambda: B.hm_combine_transpose_bf16(e(T + 1, H, dtype=bf16), plan, rows)),
        (ValueError, lambda: B.hm_combine(rows, None, plan, e(T + 1, H, dtype=bf16))),
        (ValueError, lambda: B.hm_combine(rows, e(T, K + 1, dtype=f32), plan, out)),
        (TypeError, lambda: B.hm_combine(rows, w.double(), plan, out)),
        (TypeError, lambda: B.hm_combine(rows, w, plan, twice[:T, :H])),
        (ValueError, lambda: B.hm_combine_mix(rows, e(T - 1, K, dtype=f32), plan, out)),
        (ValueError, lambda: B.hm_combine_f32(rows.float(), None, plan, e(T - 1, H, dtype=f32))),
        (TypeError, lambda: B.hm_expert_load(ids, e2r, 1, 4, e(E), e(4), e(1, dtype=f32))),
        (TypeError, lambda: B.hm_group_counts(ids, e2r, 4, [4], e(1, 64, dtype=torch.int64))),
        (ValueError, lambda: B.hm_swap_counts_multi(ids, e2r, 4, [4, 2], [e(E, E, 4)], workspace=e(100000))),
        (TypeError, lambda: B.hm_swap_counts_multi(ids, e2r, 4, [4], [e(E, 4, E).transpose(1, 2)], workspace=e(100000))),
        (TypeError, lambda: B.hm_swap_apply(e2r, e(2, dtype=torch.int64))),
    ]
    few_masks.rank_mask = few_masks.rank_mask[:T]
    for i, (error, call) in enumerate(cases):
        with pytest.raises(error):
            call()
        assert (plan.T, plan.K, few_masks.T, few_masks.K) == (T, K, T, K) or error is TypeError, i
        plan.T, plan.K = T, K                       # the Python code adopts a table before it looks at its types
    assert len(rec.calls) == len(cases) and not any(taken for _, taken in rec.calls), rec.calls
    torch.cuda.synchronize()
