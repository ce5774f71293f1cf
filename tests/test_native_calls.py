"""_hmcall: what it takes, and what it leaves to the binding's Python code."""
import subprocess
import sys

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
