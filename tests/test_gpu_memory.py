"""Contexts whose device memory is limited: a caller's allocator that returns NULL beyond
a limit.  What is optional (private copies of accumulated outputs, permuted operand
copies) and what the eight-contraction form of the residual takes beyond the
nine-contraction one never fails a call that fits without it.  Results agree with an
unlimited context's to the difference of the summation orders: the sweeps stop at
1e-13 of the amplitudes, 1e-11 of the largest element is allowed."""
import numpy as np
import pytest

import ftcc_inputs as fi

pytestmark = pytest.mark.gpu

NO_COPIES = 1 << 40   # a cap that binds nothing: a capped context takes no optional copies


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_01729_amd import ftcc
    return ftcc


class Pool:
    """Device memory from torch's caching allocator up to `limit` bytes."""

    def __init__(self):
        self.limit, self.held, self.size = None, 0, {}

    def alloc(self, nbytes):
        import torch
        if self.limit is not None and self.held + nbytes > self.limit:
            return 0
        p = torch.cuda.caching_allocator_alloc(nbytes, 0)
        self.size[p] = nbytes
        self.held += nbytes
        return p

    def free(self, p):
        import torch
        self.held -= self.size.pop(p)
        torch.cuda.caching_allocator_delete(p)


def _system(kind):
    """(h, eri, eps, mu, beta, labels or None)"""
    if kind.startswith("ring"):   # a label per orbital
        s = fi.hubbard_config(L=int(kind[4:]), U=2.0, T=1.0)
        return s.h, s.eri, s.eps, s.mu, s.beta, s.momentum
    n = int(kind.lstrip("dense").lstrip("pair"))
    h, eri, eps = fi.random_hamiltonian(n, seed=n, scale=0.2 / n)
    if kind.startswith("dense"):
        return h, eri, eps, 0.1, 0.5, None
    lab = np.arange(n) % 2      # two labels: dense storage, blocked contractions
    h = h * ((lab[:, None] + lab) % 2 == 0)
    eri = eri * ((lab[:, None, None, None] + lab[:, None, None] + lab[:, None] + lab) % 2 == 0)
    return h, eri, eps, 0.1, 0.5, (lab, [2])


def _context(F, s, pool, **opt):
    h, eri, eps, mu, beta, labels = s
    ctx = F.Context(1, n_tau=4, nodes_per_panel=2, tol=1e-13, **opt)
    ctx.set_allocator(pool.alloc, pool.free)
    if labels is not None:
        ctx.set_momentum(0, *labels)
    ctx.set_hamiltonian(0, h, eri, eps)
    return ctx


def _step(ctx, s):
    ctx.solve(s[3], s[4])
    out = [ctx.grand_potential()[0], *ctx.amplitudes(0, 1)]
    ctx.lam()
    r = ctx.response(want_mu=True, want_beta=True, want_h=True, want_eps=True)
    return out + [r["mu"], r["beta"], *r["h"], *r["eps"]]


def _close(out, ref, tol=1e-11):
    for a, b in zip(out, ref):
        a, b = np.asarray(a), np.asarray(b)
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1e-3)


def _run(F, kind, limit=None, after_solve=False, **opt):
    """A step with at most `limit` bytes; after_solve: no more than the solve took."""
    s, pool = _system(kind), Pool()
    pool.limit = limit
    print(f"[memory] {kind} limit={limit} after_solve={after_solve} {opt}", flush=True)
    ctx = _context(F, s, pool, **opt)
    try:
        if after_solve:
            ctx.solve(s[3], s[4])
            pool.limit = pool.held
        out = _step(ctx, s)
        held = pool.held
    finally:
        ctx.close()
    assert pool.held == 0
    return out, held


@pytest.mark.parametrize("kind", ["ring6", "pair10", "dense10", "dense41"])
def test_step_without_room_for_optional_copies(F, kind):
    ref, held = _run(F, kind, mem_cap_bytes=NO_COPIES)
    out, _ = _run(F, kind, limit=held)
    _close(out, ref)


@pytest.mark.parametrize("kind", ["ring6", "pair10", "dense10", "dense41"])
def test_step_with_less_room_than_the_eight_contraction_form(F, kind):
    """One byte less than the form with eight contractions takes."""
    ref, held = _run(F, kind, mem_cap_bytes=NO_COPIES)
    out, less = _run(F, kind, limit=held - 1)
    _close(out, ref)
    assert less < held


@pytest.mark.parametrize("kind", ["ring6", "pair10", "dense10"])
def test_response_without_room_after_the_solve(F, kind):
    ref, _ = _run(F, kind)
    out, _ = _run(F, kind, after_solve=True)
    _close(out, ref)


def _density(F, kind, room=None, monkeypatch=None, **opt):
    """The density with `room` bytes beyond what solve, lambda and response hold."""
    s, pool = _system(kind), Pool()
    print(f"[memory] density {kind} room={room} {opt}", flush=True)
    ctx = _context(F, s, pool, **opt)
    try:
        _step(ctx, s)
        held = pool.held
        if room is not None:
            pool.limit = held + room
        gam = ctx.two_body_density()
        took = pool.held - held
    finally:
        ctx.close()
    return gam, took


@pytest.mark.parametrize("less", [0, 1])
@pytest.mark.parametrize("kind", ["ring6", "pair10", "dense10"])
def test_density_without_room_for_optional_copies(F, kind, less):
    """Room for the density's own buffers only, and one byte less than that (the
    executors' nine-contraction form makes up for it)."""
    ref, took = _density(F, kind, mem_cap_bytes=NO_COPIES)
    gam, _ = _density(F, kind, room=took - less)
    _close(gam, ref)


def test_density_takes_no_more_with_packed_states(F, monkeypatch):
    """Labels all distinct: the density's executor works on the packed node states, so it
    allocates what it does over dense ones (FTCC_PACK=0), and not a state per slot more."""
    took = []
    for pack in ("1", "0"):
        monkeypatch.setenv("FTCC_PACK", pack)
        took.append(_density(F, "ring6", mem_cap_bytes=NO_COPIES)[1])
    assert took[0] <= took[1]


# the least that solve, Lambda, the response (mu, beta, h, eps) and the density (but
# propagator 5) ran in before the node states were packed
LEAST = [("ring10", 0, 0, 144829184), ("ring10", 2, 0, 142078976), ("ring10", 4, 0, 144284160),
         ("ring10", 5, 0, 139591680), ("ring10", 0, 4, 146124544), ("pair14", 0, 0, 186715136),
         ("pair14", 4, 0, 178135296), ("dense12", 0, 0, 181944576)]


@pytest.mark.parametrize("kind,propagator,diis,limit", LEAST)
def test_runs_in_the_memory_it_ran_in(F, kind, propagator, diis, limit):
    s, pool = _system(kind), Pool()
    pool.limit = limit
    print(f"[memory] {kind} propagator={propagator} diis={diis} limit={limit}", flush=True)
    ctx = _context(F, s, pool, propagator=propagator, diis_depth=diis)
    try:
        _step(ctx, s)
        if propagator != 5:
            ctx.two_body_density()
    finally:
        ctx.close()


def test_descriptors_of_a_small_context_are_small(F):
    """What a context of a 4-site ring takes beside the caller's allocator.  Descriptor
    chunks of fixed sizes (1 MiB, and 4 MiB per executor) took at least 9 MiB; the plan
    itself is below 1 MiB, and the stream and the graphs took 2.25 beside those chunks."""
    import torch
    s, pools = _system("ring4"), []
    warm = torch.empty(1 << 32, dtype=torch.uint8, device="cuda")   # the pools' memory: held by torch
    del warm

    def one():
        pools.append(Pool())
        ctx = _context(F, s, pools[-1])
        _step(ctx, s)
        return ctx
    ctxs = [one()]
    torch.cuda.synchronize()
    free, reserved = torch.cuda.mem_get_info()[0], torch.cuda.memory_reserved()
    ctxs += [one() for _ in range(8)]
    torch.cuda.synchronize()
    own = free - torch.cuda.mem_get_info()[0] - (torch.cuda.memory_reserved() - reserved)
    for c in ctxs:
        c.close()
    assert own / 8 < 6 << 20


def test_a_context_goes_on_after_a_solve_without_memory(F):
    """A solve that finds no memory leaves a context that solves once there is some: with the
    same labels, with labels set in between, and a Hamiltonian that breaks them is refused."""
    h, eri, eps, mu, beta, momentum = _system("ring6")

    def omega(labels, late=False, limit=None):
        pool = Pool()
        print(f"[memory] labels={labels} late={late} limit={limit}", flush=True)
        ctx = _context(F, (h, eri, eps, mu, beta, None if late else momentum if labels else None), pool)
        if limit is not None:
            pool.limit = limit
            with pytest.raises(F.FTCCError) as e:
                ctx.solve(mu, beta)
            assert e.value.code == F.ENOMEM
            pool.limit = None
        if late:
            ctx.set_momentum(0, *momentum)
        if limit is not None and labels and not late:
            bad = eri.copy()
            bad[0, 0, 0, 1] = 1.0
            with pytest.raises(F.FTCCError):   # at once where the labels are laid out, else by the solve
                ctx.set_hamiltonian(0, h, bad, eps)
                ctx.solve(mu, beta)
            with pytest.raises(F.FTCCError):
                ctx.set_hamiltonian(0, h[:5, :5], eri[:5, :5, :5, :5], eps[:5])
            ctx.set_hamiltonian(0, h, eri, eps)
        ctx.solve(mu, beta)
        out = [ctx.grand_potential()[0], *ctx.amplitudes(0, 1)]
        ctx.close()
        return out

    for labels in (True, False):
        ref = omega(labels)
        # 128 MiB of what a context holds are one workspace: limits before it, and among what
        # comes after it, the executors' buffers last
        for limit in (1 << 20, 134_800_000, 135_050_000 if labels else 135_300_000):
            for late in ((False, True) if labels else (False,)):
                _close(omega(labels, late, limit), ref)
