"""Operators that follow one another in the memory of destroyed ones: other
sizes, several alive at once, other contexts; every result is that of a plain
sum over the stencils."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def problem(N, n, seed):
    """Caller stencils, weights and a state on the GPU, and L u from them."""
    rng = np.random.default_rng(seed)
    off = np.stack([1 + rng.choice(min(N - 1, 150), n - 1, replace=False) for _ in range(1)])[0]
    idx = np.concatenate([np.arange(N)[:, None], (np.arange(N)[:, None] + off[None]) % N], axis=1).astype(np.int32)
    w = rng.standard_normal((N, n))
    w[:, 0] = -w[:, 1:].sum(1)
    u = rng.standard_normal(N)
    return [torch.as_tensor(a).cuda() for a in (idx, w, u)] + [(w * u[idx]).sum(1), (np.abs(w) * np.abs(u[idx])).sum(1)]


def check(op, p):
    got = op.apply(p[2]).cpu().numpy()
    assert np.all(np.abs(got - p[3]) <= 2 * p[0].shape[1] * 2.0 ** -53 * p[4])


def test_sizes_in_turn(lib):
    """Equal, smaller, much smaller (not served by the kept memory) and larger operators, one after another."""
    ctx = lib.Context()
    for q, (N, n) in enumerate([(3000, 31), (3000, 31), (2000, 31), (200, 9), (9000, 50), (9000, 33), (64, 2), (70000, 60),
                                (65, 64)]):
        p = problem(N, n, q)
        op = lib.Operator(p[0], p[1], ctx=ctx)
        check(op, p)
        op.close()
    ctx.close()


def test_several_alive(lib):
    ctx = lib.Context()
    ps = [problem(N, 31, N) for N in (2000, 2000, 2500)]
    ops = []
    for turn in range(3):
        ops += [lib.Operator(p[0], p[1], ctx=ctx) for p in ps]
        for op, p in zip(ops, ps):
            check(op, p)
        ops.pop(turn).close()
        ps = ps[:turn] + ps[turn + 1:] + [ps[turn]]
        for op, p in zip(ops, ps[:2]):
            check(op, p)
        for op in ops:
            op.close()
        ops = []
    ctx.close()


def test_on_another_context(lib):
    """An operator applied on a second context's stream, destroyed and followed
    by one in its memory while that stream may still be busy."""
    a, b = lib.Context(), lib.Context()
    p, q = problem(200000, 31, 1), problem(200000, 31, 2)
    for turn in range(3):
        op = lib.Operator(p[0], p[1], ctx=a)
        op.ctx = b
        outs = [op.apply(p[2]) for _ in range(20)]
        op.close()
        op = lib.Operator(q[0], q[1], ctx=a)
        check(op, q)
        assert all(torch.equal(o, outs[0]) for o in outs)
        assert np.all(np.abs(outs[0].cpu().numpy() - p[3]) <= 62 * 2.0 ** -53 * p[4])
        op.close()
    a.close()
    b.close()


def test_recorded_application_outlives_nothing(lib):
    """A graph of applications launched on a stream the library does not know:
    destroying the operator waits for it before the memory serves another."""
    ctx = lib.Context()
    p, q = problem(200000, 31, 3), problem(200000, 31, 4)
    side = torch.cuda.Stream()
    for turn in range(3):
        op = lib.Operator(p[0], p[1], ctx=ctx)
        out = torch.zeros_like(p[2])
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=ctx.stream):
            for _ in range(60):
                rc = ctx.lib.rbffd_apply_noalloc(ctx.h, op.h, 0, ctypes.c_void_p(p[2].data_ptr()),
                                                 ctypes.c_void_p(out.data_ptr()))
                assert rc == 0
        with torch.cuda.stream(side):
            g.replay()
        op.close()
        op = lib.Operator(q[0], q[1], ctx=ctx)
        check(op, q)
        torch.cuda.synchronize()
        assert np.all(np.abs(out.cpu().numpy() - p[3]) <= 62 * 2.0 ** -53 * p[4])
        op.close()
    ctx.close()


def test_no_workspace_before_it_is_needed(lib):
    """80 bytes a row of state workspace: not taken by an operator that is built
    and only applied without allocation, taken once by one that is applied or stepped."""
    ctx = lib.Context()
    N = 1 << 20
    p = problem(N, 2, 5)

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    lib.Operator(p[0], p[1], ctx=ctx)  # scratch, code objects
    out = torch.empty_like(p[2])
    ctx.lib.rbffd_destroy(ctx.h)  # gives everything back
    ctx.h = None
    ctx = lib.Context()
    before = free()
    op = lib.Operator(p[0], p[1], ctx=ctx)
    built = before - free()
    assert ctx.lib.rbffd_apply_noalloc(ctx.h, op.h, 0, ctypes.c_void_p(p[2].data_ptr()),
                                       ctypes.c_void_p(out.data_ptr())) == 0
    assert before - free() == built
    assert built < 140 * N  # slots 18, diagonal 8, halo lists 40, order 4 bytes a row; scratch 5: not 80 more
    ctx.enter(p[2])
    rc = ctx.lib.rbffd_apply(ctx.h, op.h, 0, ctypes.c_void_p(p[2].data_ptr()), ctypes.c_void_p(out.data_ptr()))
    ctx.leave()
    assert rc == 0
    first = before - free()
    assert first - built >= 80 * N
    check(op, p)
    op.step(p[2], 1e-6, 2)
    ctx.stream.synchronize()
    op.close()
    ctx.close()
