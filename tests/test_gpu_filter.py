"""The hooks that test the entries against a bitmap in LDS, at the edges of the
sizes they are chosen for: labels bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
from gpu_helpers import assert_same_labels, log, to_dev, to_host_u32

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_2507_03695_amd")

LDS_MAX_N = 36864 * 32


@pytest.fixture(scope="module")
def ctx():
    c = cc.Context(zroot_samples=4096)
    yield c
    c.close()


def by_steps(ctx, ed, n, flags=0):
    """The zero-root path through its steps, the entries in two hooks (the second
    finds marks that are not in P)."""
    P = torch.empty(n, dtype=torch.int32, device="cuda")
    h = ed.shape[0] // 2
    ctx.init(n, P)
    ctx.zroot(ed, n)
    ctx.push(ed, n, P)
    ctx.hook(ed[:h], n, P, flags=cc.F_ZROOT | flags)
    ctx.hook(ed[h:], n, P, flags=cc.F_ZROOT | flags)
    ctx.compress(n, P, flags=cc.F_ZROOT)
    ctx.canon(n, P)
    return P


def graph(kind, n, m, seed):
    if kind == "er":
        return graphgen.er(n, m, seed)
    if kind == "rmat":
        e = graphgen.rmat(max(1, (n - 1).bit_length()), m, seed).astype(np.int64)
        return np.ascontiguousarray((e % n).astype(np.uint32))
    if kind == "paths":                        # no giant component: paths of 16 vertices, twice
        a = np.arange(n - 1, dtype=np.uint32)
        e = np.stack([a, a + 1], 1)[a % 16 != 15]
        e = np.concatenate([e[::-1], e[:, ::-1], e])
        return np.ascontiguousarray(e[np.arange(m) % len(e)])
    # "rows": sorted by first endpoint, as a CSR graph written out
    e = graphgen.er(n, m, seed)
    return np.ascontiguousarray(e[np.argsort(e[:, 0], kind="stable")])


@pytest.mark.parametrize("kind", ["er", "rmat", "paths", "rows"])
@pytest.mark.parametrize("n,m", [(1, 1 << 18), (33, 1 << 18), (65536, (1 << 18) - 1), (65537, 1 << 18),
                                 (131071, 262145), (131071, 262142), (479_999, 4_200_001),
                                 (LDS_MAX_N, 3_000_000), (LDS_MAX_N + 1, 3_000_000)])
def test_whole_bitmap_in_lds(ctx, kind, n, m):
    if kind != "er" and n < 100:
        pytest.skip("er covers it")
    e = graph(kind, n, m, n + m)
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    log(f"{kind} n={n} m={m}")
    for name, fl in [("plain", 0), ("zroot", cc.F_ZROOT)]:
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"{kind} n={n} m={m} [{name}]")
    assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"{kind} n={n} m={m} [steps]")
    L = torch.empty(n, dtype=torch.int32, device="cuda")
    cc.solve_noalloc(ed, n, L)
    assert_same_labels(to_host_u32(L), want, f"{kind} n={n} m={m} [no allocation]")


def test_whole_bitmap_symmetric_range_and_zroot(ctx):
    n, m = 300_001, 1_200_000
    e = graphgen.er(n, m // 2, 9)
    sym = np.concatenate([e, e[:, ::-1]])
    want = oracle.cc_labels(n, e)
    for fl in (cc.F_SYMMETRIC, cc.F_SYMMETRIC | cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve(to_dev(sym), n, flags=fl)), want, f"symmetric {fl}")
    # the zero root reported is the sampled one's, also after a plain solve
    ctx.solve(to_dev(e), n, flags=cc.F_ZROOT)
    z = ctx.get_zroot()
    assert z == oracle.zroot(n, e, 4096)
    ctx.solve(to_dev(e), n)
    assert ctx.get_zroot() == z
    # an endpoint out of range in the last entry, on either side
    for bad in ([n, 0], [0, 0xFFFFFFFF]):
        b = np.concatenate([e, np.array([bad], np.uint32)])
        for fl in (0, cc.F_ZROOT):
            L = torch.empty(n, dtype=torch.int32, device="cuda")
            ctx.solve_async(to_dev(b), n, L, flags=fl)
            assert ctx.sync() == cc.CC_ERANGE
