"""The device memory kept for later plans: bounded, given back, and the same
plans whichever block they land in."""
import numpy as np
import pytest

import graphgen
from gpu_helpers import _dev, _plan, _spmm_check, assert_plan_matches_oracle

torch = pytest.importorskip("torch")
import paper_2308_11825_amd as agcn  # noqa: E402

pytestmark = pytest.mark.gpu


def _graph(n, d, seed):
    rng = np.random.default_rng(seed)
    return graphgen.random_csr(n, n, rng.integers(0, 2 * d, size=n), seed=seed)


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_small_plans_after_a_large_one_reuse_their_blocks():
    """Six sizes in turn, the largest first: at most four blocks stay cached,
    every plan is right, and release gives all of it back."""
    agcn.agcn_release_cached_memory()
    gs = [_graph(n, d, 7 + n) for n, d in [(60000, 40), (3000, 8), (3100, 8), (20000, 12), (500, 3),
                                           (30000, 30)]]
    sizes = []
    for g in gs:
        p = _plan(g)
        sizes.append(p.stats.device_bytes)
        _spmm_check(p, g, 8)      # whatever torch and the runtime load once is loaded now
        p.destroy()
    agcn.agcn_release_cached_memory()
    torch.cuda.empty_cache()
    before = _free()
    for _ in range(3):
        for g in gs:
            p = _plan(g)
            assert_plan_matches_oracle(p, g)
            _spmm_check(p, g, 8)
            p.destroy()
    torch.cuda.empty_cache()
    held = before - _free()
    assert held <= sum(sorted(sizes)[-4:]) + (16 << 20), (held, sizes)
    agcn.agcn_release_cached_memory()
    torch.cuda.empty_cache()
    assert before - _free() <= (8 << 20)


def test_alternating_sizes_allocate_nothing_new():
    """A large and two small graphs in turn: after the first round the free
    memory stays where it is."""
    agcn.agcn_release_cached_memory()
    gs = [_graph(60000, 40, 1), _graph(3000, 8, 2), _graph(2990, 8, 3)]
    csr = [(_dev(g.rowptr), _dev(g.colidx), _dev(g.vals)) for g in gs]
    seen = []
    for _ in range(4):
        for c in csr:
            agcn.Plan(*c).destroy()
        seen.append(_free())
    assert len(set(seen[1:])) == 1, seen
    agcn.agcn_release_cached_memory()


def test_a_plan_of_over_4_gib_keeps_its_block_between_small_ones():
    """The largest block stays whatever the others sum to: after the first round
    neither plan of an alternation allocates."""
    agcn.agcn_release_cached_memory()
    n, d = 1_000_000, 600
    rowptr = torch.arange(n + 1, dtype=torch.int32, device="cuda:0") * d
    cols = torch.randint(0, n, (n * d,), dtype=torch.int32, device="cuda:0")
    big = (rowptr, cols, torch.ones(n * d, device="cuda:0"))
    g = _graph(3000, 8, 2)
    small = (_dev(g.rowptr), _dev(g.colidx), _dev(g.vals))
    for k in range(3):
        for csr in (big, small):
            before = _free()
            p = agcn.Plan(*csr)
            if csr is big:
                assert p.stats.device_bytes > 4 << 30
            if k > 0:
                assert _free() == before, k
            p.destroy()
    agcn.agcn_release_cached_memory()


def test_calls_with_another_current_device_context_and_stream():
    """Executes inside a stream context run on that stream, as before."""
    g = _graph(2000, 6, 5)
    p = _plan(g)
    X = torch.randn((g.n_cols, 16), device="cuda:0")
    Y = p.spmm(X)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        assert agcn._stream_handle(X.device) == s.cuda_stream
        Z = p.spmm(X)
        H = agcn.linear(X, torch.eye(16, device="cuda:0"))
    s.synchronize()
    assert torch.equal(Y, Z) and torch.equal(H, X)
    p.destroy()
    with pytest.raises(RuntimeError):
        p.workspace(16)
    with pytest.raises(RuntimeError):
        p.spmm(X)
