"""The extension's codegemm_gemm and codegemm_gemm_grouped against their ctypes forms: the same arguments reach the library in every form of a
call that these take, and the same exceptions leave it."""
import ctypes
import os
import subprocess
import sys

import pytest

import paper_2512_17970_amd as cg
from paper_2512_17970_amd import binding

vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        if isinstance(self.at, Exception):
            raise self.at
        return self.at


class Index:
    def __int__(self):
        return 0x1230


@pytest.fixture()
def calls():
    """Both forms with the library's functions replaced by ones that note what they are given and return `status`."""
    lib, seen, status = binding.load(), [], [0]

    def gemm(desc, plan, *rest):
        seen.append((bytes(desc[0]), bytes(plan[0]) if plan else None, *rest))
        return status[0]

    def grouped(desc, plan, x, group, count, *rest):
        members = [bytes(group[k]) for k in range(count)]
        seen.append((bytes(desc[0]), bytes(plan[0]) if plan else None, x, members, *rest))
        return status[0]

    dp, pp = ctypes.POINTER(cg.Desc), ctypes.POINTER(cg.Plan)
    one = ctypes.CFUNCTYPE(ctypes.c_int, dp, pp, vp, vp, vp, vp, vp, vp, sz, vp)(gemm)
    group = ctypes.CFUNCTYPE(ctypes.c_int, dp, pp, vp, ctypes.POINTER(cg.GroupMember), i32, vp, sz, vp)(grouped)
    real = lib.codegemm_gemm, lib.codegemm_gemm_grouped
    address = lambda f: ctypes.cast(f, vp).value
    lib.codegemm_gemm, lib.codegemm_gemm_grouped = one, group
    binding._calls.use(address(one), address(group))
    yield seen, status
    lib.codegemm_gemm, lib.codegemm_gemm_grouped = real
    binding._calls.use(address(real[0]), address(real[1]))


def outcome(f, seen, *args, **kwargs):
    del seen[:]
    try:
        got = f(*args, **kwargs)
    except Exception as e:
        got = (type(e), str(e))
    return got, list(seen)


DESC, PLAN = cg.Desc.make(4, 512, 256, 8, 2, g=128), cg.Plan.make(8, 1, 2, 4, 0, 0, 32, 2)


def test_the_module_exports_the_extension():
    assert cg.codegemm_gemm is binding._calls.codegemm_gemm and cg.codegemm_gemm_grouped is binding._calls.codegemm_gemm_grouped


@pytest.mark.parametrize("status", [0, -1, -3])
def test_gemm(calls, status):
    seen, result = calls
    result[0] = status
    t = [Tensor(0x1000 * k) for k in range(1, 7)]
    forms = [(DESC, PLAN, *t, 4096, 77), (DESC, None, *t, 4096), (DESC, PLAN, 1, 2, 3, 4, 5, 2**63 + 8, 2**40, 2**64 - 16), (DESC, PLAN, None, *t[1:], 0, 0),
             (DESC, PLAN, Tensor(0), *t[1:], 5, 0), (DESC, PLAN, Index(), *t[1:], 5, 0), (DESC, PLAN, -8, *t[1:], 5, 0), (DESC, PLAN, True, *t[1:], 5, 0),
             (DESC, PLAN, *t, 4096, None), (DESC, PLAN, *t, -1, 3), (DESC, PLAN, *t, 4.0, 3), (DESC, PLAN, *t, 4096, 3.0), (DESC, PLAN, *t, 4096, vp(9)),
             (DESC, PLAN, *t[:5], "x", 4096), (DESC, PLAN, Tensor(RuntimeError("no storage")), *t[1:], 1), (DESC, PLAN, Tensor([]), *t[1:], 1),
             (PLAN, PLAN, *t, 4096), (DESC, DESC, *t, 4096), (None, PLAN, *t, 4096), (DESC, 7, *t, 4096), (DESC, PLAN, *t), (DESC, PLAN, *t, 1, 2, 3), (),
             (DESC, PLAN, 2**70, *t[1:], 1), (DESC, PLAN, *t, 2**70)]
    for args in forms:
        assert outcome(cg.codegemm_gemm, seen, *args) == outcome(binding._gemm, seen, *args), args
    names = dict(zip(("x", "packed_codes", "codebooks", "scales", "y", "workspace", "workspace_bytes"), (*t, 64)))
    for kwargs in (names, dict(names, stream=5), dict(names, stray=1)):
        assert outcome(cg.codegemm_gemm, seen, DESC, PLAN, **kwargs) == outcome(binding._gemm, seen, DESC, PLAN, **kwargs)


@pytest.mark.parametrize("status", [0, -2])
def test_gemm_grouped(calls, status):
    seen, result = calls
    result[0] = status
    t = [Tensor(0x1000 * k) for k in range(1, 6)]
    member = (128, *t[1:])
    forms = [(DESC, PLAN, t[0], [member] * k, 9, 4096, 3) for k in range(6)] + [
             (DESC, None, t[0], (member, (64, 1, 2, None, 2**64 - 4)), t[1], 4096), (DESC, PLAN, 5, [list(member)], 9, 4096), (DESC, PLAN, 5, iter([member]), 9, 4096),
             (DESC, PLAN, 5, [member[:4]], 9, 4096), (DESC, PLAN, 5, [(2**31, *t[1:])], 9, 4096), (DESC, PLAN, 5, [(-1, *t[1:])], 9, 4096),
             (DESC, PLAN, 5, [("n", *t[1:])], 9, 4096), (DESC, PLAN, 5, [(1, *t[1:4], "y")], 9, 4096), (DESC, PLAN, 5, 6, 9, 4096), (DESC, PLAN, 5, [member], 9, "b"),
             (DESC, PLAN, 5, [member], 9, 4096, None), (DESC, PLAN, 5, [member]), (PLAN, PLAN, 5, [member], 9, 4096)]
    for args in forms:
        assert outcome(cg.codegemm_gemm_grouped, seen, *args) == outcome(binding._gemm_grouped, seen, *args), args
    kwargs = dict(x=t[0], members=[member], workspace=1, workspace_bytes=2, stream=3)
    assert outcome(cg.codegemm_gemm_grouped, seen, DESC, PLAN, **kwargs) == outcome(binding._gemm_grouped, seen, DESC, PLAN, **kwargs)


def test_a_list_that_shrinks_while_it_is_read(calls):
    """data_ptr() is any Python: members that are gone by then are not read."""
    seen, _ = calls
    members = [(1, None, 2, 3, 4), (2, 5, 6, 7, 8), (3, 5, 6, 7, 8)]

    class Clearing:
        def data_ptr(self):
            del members[1:]
            return 0x40

    members[0] = (1, Clearing(), 2, 3, 4)
    cg.codegemm_gemm_grouped(DESC, PLAN, 1, members, 9, 4096)
    assert [len(s[3]) for s in seen] == [1]


@pytest.mark.parametrize("error", [KeyboardInterrupt, SystemExit, MemoryError, RuntimeError, OverflowError])
def test_what_a_data_ptr_raises_once(calls, error):
    """An interrupt in data_ptr() is not lost, and no data_ptr() that raised is called again."""
    seen, _ = calls

    class Once:
        asked = 0

        def data_ptr(self):
            self.asked += 1
            if self.asked == 1:
                raise error("once")
            return 0x40

    for at in range(6):
        for call in (cg.codegemm_gemm, binding._gemm):
            once, args = Once(), [1, 2, 3, 4, 5, 6]
            args[at] = once
            with pytest.raises(error):
                call(DESC, PLAN, *args, 4096, 0)
            assert once.asked == 1 and not seen
    for at in range(6):
        for call in (cg.codegemm_gemm_grouped, binding._gemm_grouped):
            once, args = Once(), [1, 2, 3, 4, 5, 6]
            args[at] = once
            with pytest.raises(error):
                call(DESC, PLAN, args[0], [(1, 2, 3, 4, 5), (1, *args[1:5])], args[5], 4096)
            assert once.asked == 1 and not seen


def test_which_of_two_errors_is_raised(calls):
    """Members are looked at before x."""
    x, y = Tensor(KeyError("x")), Tensor(ValueError("y"))
    for call in (cg.codegemm_gemm_grouped, binding._gemm_grouped):
        with pytest.raises(ValueError):
            call(DESC, PLAN, x, [(1, 2, 3, 4, y)], 6, 4096)


WITHOUT = """
import ctypes, sys
sys.modules["paper_2512_17970_amd._calls"] = None          # what an import finds where the extension has not been built
import paper_2512_17970_amd as cg
from paper_2512_17970_amd import binding
assert binding._calls is None and cg.codegemm_gemm is binding._gemm and cg.codegemm_gemm_grouped is binding._gemm_grouped
desc = cg.Desc.make(1, 512, 512, 8, 1)
for call in (lambda: cg.codegemm_gemm(desc, None, 16, 16, 16, 16, 16, None, 0), lambda: cg.codegemm_gemm_grouped(desc, None, None, [(512, 16, 16, 16, 16)], 16, 0)):
    try:
        call()
    except cg.CodegemmError as e:
        assert e.status == -1, e
    else:
        raise AssertionError("no error")
print(cg.codegemm_workspace_bytes(desc))
"""


def test_the_library_without_the_extension():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", WITHOUT], cwd=root, capture_output=True, text=True)
    assert out.returncode == 0 and int(out.stdout) == cg.codegemm_workspace_bytes(cg.Desc.make(1, 512, 512, 8, 1)), out.stderr


def test_a_build_without_a_compiler_or_headers(monkeypatch, tmp_path, capsys):
    from paper_2512_17970_amd import build
    monkeypatch.setattr(build.subprocess, "run", lambda *a, **k: pytest.fail("nothing to run"))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_calls() == "" and "Python.h" in capsys.readouterr().out
