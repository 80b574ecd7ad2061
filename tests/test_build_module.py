"""How the argument marshalling module is built and what happens without it."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_1908_04207_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def elsewhere(monkeypatch, tmp_path):
    """The build's outputs in an empty folder, compilers replaced by a recorder that writes them."""
    for name in ("LIB", "STAMP", "MARSHAL", "MARSHAL_STAMP"):
        monkeypatch.setattr(build, name, str(tmp_path / os.path.basename(getattr(build, name))))
    monkeypatch.setattr(build, "OBJDIR", str(tmp_path / "obj"))
    monkeypatch.setenv("CXX", "the-host-compiler")
    commands = []

    def run(cmd):
        commands.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()

    monkeypatch.setattr(build, "_run", run)
    return commands


def test_module_belongs_to_one_interpreter(elsewhere):
    """Its name carries the interpreter's tag, an untagged one (which any interpreter would load) goes,
    and a module of another interpreter or of other sources does not count as built."""
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.basename(build.MARSHAL) == "_marshal" + suffix and suffix != ".so"
    untagged = os.path.join(os.path.dirname(build.MARSHAL), "_marshal.so")
    open(untagged, "w").close()
    assert build.build() == build.LIB
    assert os.path.exists(build.MARSHAL) and not os.path.exists(untagged) and build.is_current()
    os.remove(build.MARSHAL)
    assert not build.is_current()
    open(build.MARSHAL, "w").close()
    with open(build.MARSHAL_STAMP, "w") as f:
        f.write("0123456789abcdef\n")
    assert not build.is_current()


def test_library_is_built_without_a_host_compiler(elsewhere, monkeypatch):
    run = build._run

    def no_host_compiler(cmd):
        if cmd[0] == "the-host-compiler":
            raise FileNotFoundError(cmd[0])
        run(cmd)

    monkeypatch.setattr(build, "_run", no_host_compiler)
    with pytest.warns(UserWarning, match="not built"):
        assert build.build() == build.LIB
    assert os.path.exists(build.LIB) and not os.path.exists(build.MARSHAL)
    assert build.is_current()                        # nothing more can be built here


def test_binding_without_the_module():
    """ctypes takes every call: same plan, same refusals."""
    program = """
import sys, warnings
blocked = sys.argv[1] == "blocked"
if blocked:
    sys.modules["paper_1908_04207_amd._marshal"] = None
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_1908_04207_amd import binding as eb
assert blocked == any("ctypes" in str(w.message) for w in seen)
print(bytes(eb.eager_plan_participation(eb.SOLO, [3.0, 1.0], 1, 0)).hex())
print(bytes(eb.eager_plan_quorum([3.0, 1.0], 2, 0)).hex())
ctx = eb.Context(2, [0], [4])
for call in (lambda: ctx.eager_partial_allreduce(eb.make_plan(eb.SOLO, 2, 0, 1), [16, 32], [48, 64], recv=4, stream=0),
             lambda: ctx.eager_sgd_step(8, (16, 32, 0.1, 0.9), stream=0),
             lambda: ctx.eager_stash(7, 16, 32, stream=0), lambda: ctx.eager_average_views([16, 16], stream=0)):
    try:
        call()
    except eb.EagerError as e:
        print(e)
ctx.close()
"""
    out = [subprocess.run([sys.executable, "-c", program, how], cwd=ROOT, capture_output=True, text=True, check=True).stdout
           for how in ("blocked", "there")]
    assert out[0] == out[1] and out[0].count("EAGER_EINVAL") == 4
