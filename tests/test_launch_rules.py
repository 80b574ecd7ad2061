"""The launch rules of csrc/eager_rules.h on the CPU, and on the GPU the largest run a call accepts."""
import os
import subprocess

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rules_on_the_host(tmp_path):
    exe = tmp_path / "launch_rules_host"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-static-libasan", "-Wall", "-Wextra", "-Werror",
                           "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "c", "launch_rules_host.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.stdout[-500:], r.stderr[-2000:])


def test_chunk_lists_on_the_host(tmp_path):
    """The list that chunk_kernel takes, worked through as the kernel does, against the slots it was made of."""
    exe = tmp_path / "chunk_list_host"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-static-libasan", "-ffp-contract=off", "-Wall", "-Wextra",
                           "-Werror", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "c", "chunk_list_host.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.stdout[-500:], r.stderr[-2000:])


def test_short_lists_on_the_host(tmp_path):
    """The list that short_kernel takes, in the same way."""
    exe = tmp_path / "short_list_host"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-static-libasan", "-ffp-contract=off", "-Wall", "-Wextra",
                           "-Werror", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "c", "short_list_host.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.stdout[-500:], r.stderr[-2000:])


@pytest.mark.parametrize("wrong", [0, 1, 2, 3])
def test_launches_take_a_kernel_with_arguments_of_its_own_types(wrong):
    from paper_1908_04207_amd import build
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "--offload-host-only",
                        "-fsyntax-only", f"-DWRONG={wrong}", "-x", "hip",
                        os.path.join(ROOT, "tests", "c", "launch_types.hip")], capture_output=True, text=True)
    if wrong:
        assert r.returncode != 0 and "no matching function for call to 'launch" in r.stderr, r.stderr[-2000:]
    else:
        assert r.returncode == 0, r.stderr[-2000:]


def test_hints_of_streams_and_of_the_state_are_independent():
    """"nt_state" concerns w, v and the receive buffer: chunk_kernel exists with every combination of their hint
    (fourth parameter) and the streams' (third), for every type, order, kind and length of list."""
    import itertools
    import re
    from paper_1908_04207_amd import build
    names = subprocess.check_output(["nm", "-C", build.LIB], text=True)
    kernels = {tuple(m.split(", ")) for m in re.findall(r"chunk_kernel<((?:\w+, ){7})", names)}
    kernels = {k[:6] + (k[6].strip(" ,"),) for k in kernels}
    flags = ("false", "true")
    assert kernels == set(itertools.product(flags, flags, flags, flags, flags, flags, ("8", "16")))


@pytest.mark.gpu
def test_a_run_just_below_the_largest():
    """2^33 - 1 elements: every tile but the last is full and three elements are left over.  One process
    on time, so the result is its gradient."""
    from paper_1908_04207_amd import binding as eb
    n = (1 << 33) - 1
    if torch.cuda.mem_get_info()[0] < 9 * n:
        pytest.skip("needs 77 GB of free device memory")
    dev = torch.device("cuda:0")
    grad = torch.empty(n + 1, device=dev)
    step = 1 << 28
    for k in range(0, n + 1, step):
        grad[k:k + step] = torch.arange(k % 1009, k % 1009 + step, device=dev, dtype=torch.int32).remainder(997)
    recv = torch.full((n + 1,), -1.0, device=dev)
    unread = torch.zeros(4, device=dev)              # an on-time process's empty send buffer
    ctx = eb.Context(1, [0], [n])
    ctx.eager_partial_allreduce_solo(eb.make_plan(eb.SOLO, 1, 0, 1), [grad], [unread], recv=recv)
    torch.cuda.synchronize()
    for k in range(0, n, step):
        e = min(k + step, n)
        assert torch.equal(recv[k:e], grad[k:e]), k
    assert recv[n].item() == -1.0
    ctx.close()


@pytest.mark.gpu
def test_an_error_of_another_call_is_not_a_launch_s():
    """The runtime keeps the last error of a thread until somebody asks.  One that an unrelated call has left there
    (a device that does not exist) is not reported by any launch of the library as its own, nor taken away."""
    import ctypes
    from paper_1908_04207_amd import binding as eb
    dev, n, P = torch.device("cuda:0"), 1000, 2
    torch.cuda.synchronize()
    hip = ctypes.CDLL(eb.LIB_PATH)                  # the runtime that the library is linked with
    t = lambda: torch.zeros(n, device=dev)          # noqa: E731
    G, R, w, v, u = [t(), t()], [t(), t()], t(), t(), t()
    ctx, plain = eb.Context(P, [0], [n]), eb.Context(P, [0], [n])
    stats = torch.zeros(32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    workspace, sink = torch.empty(need, dtype=torch.uint8, device=dev), t()
    ctx.eager_stats_attach(stats, workspace, need)
    opt, s = (w, v, 0.1, 0.9), torch.cuda.current_stream().cuda_stream
    step = iter(range(100))
    plan = lambda mask: eb.make_plan(eb.MAJORITY, P, next(step), mask)      # noqa: E731
    calls = {
        "round": lambda: plain.eager_partial_allreduce(plan(0b01), G, R, opt=opt, stream=s),
        "round with norms": lambda: ctx.eager_partial_allreduce(plan(0b11), G, R, recv=u, stream=s),
        "step": lambda: plain.eager_sgd_step(u, opt, stream=s),
        "layer-wise step": lambda: ctx.eager_sgd_step_lars(u, opt, 0.02, 1e-9, stream=s),
        "layer-wise step, own scratch": lambda: plain.eager_sgd_step_lars_static(u, opt, 0.02, stats, 1e-9, stream=s),
        "stash": lambda: plain.eager_stash(1, G[1], R[1], stream=s),
        "flush": lambda: plain.eager_flush(R, opt=opt, stream=s),
        "views": lambda: plain.eager_sgd_step_views(u, [w], [v], 0.1, 0.9, stream=s),
        "average": lambda: plain.eager_average_views([w, v], stream=s),
        "copy": lambda: eb.eager_calib_copy(R[0], G[0], 4 * n, stream=s),
        "read": lambda: eb.eager_calib_read(G[0], 4 * n, sink, stream=s),
        "mix": lambda: eb.eager_calib_mix(G, R, n // 4, sink=sink, stream=s)}
    for name, call in calls.items():
        left = hip.hipSetDevice(1 << 20)
        assert left != 0
        try:
            call()
        finally:
            assert hip.hipGetLastError() == left, name
            assert hip.hipGetLastError() == 0
    torch.cuda.synchronize()
    ctx.close(), plain.close()
