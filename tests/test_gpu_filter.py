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


SLICE = 1 << 19


@pytest.mark.parametrize("kind", ["er", "rmat", "paths", "rows"])
@pytest.mark.parametrize("n,m", [(LDS_MAX_N + 33, 1 << 20), (LDS_MAX_N + 33, (1 << 20) - 1),
                                 (3 * SLICE, 6_000_001), (3 * SLICE + 1, 3 * SLICE + 1),
                                 (3 * SLICE + 1, 3 * SLICE), (8 * SLICE + 40, 12_000_000),
                                 (22 * SLICE, 12_000_003), (22 * SLICE + 5, (1 << 24) + 77),
                                 (22 * SLICE + 5, (1 << 24) - 1)])
def test_tiles(ctx, kind, n, m):
    """One partition pass up to 22 slices of 2^19 vertices, two beyond; a last slice
    of few vertices; graphs with and without a giant component."""
    e = graph(kind, n, m, n + m)
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    log(f"{kind} n={n} m={m}")
    for name, fl in [("plain", 0), ("zroot", cc.F_ZROOT)]:
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"{kind} n={n} m={m} [{name}]")
    assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"{kind} n={n} m={m} [steps]")


def test_tiles_symmetric_range_and_few_tiles(ctx):
    n, m = 5 * SLICE + 11, 8_000_000
    e = graphgen.er(n, m // 2, 3)
    sym = np.concatenate([e, e[:, ::-1]])
    want = oracle.cc_labels(n, e)
    for fl in (cc.F_SYMMETRIC, cc.F_SYMMETRIC | cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve(to_dev(sym), n, flags=fl)), want, f"symmetric {fl}")
    # every first endpoint in the last slice (11 vertices) or in one slice: few tiles hold entries
    for lo, hi in ((5 * SLICE, n), (2 * SLICE, 3 * SLICE)):
        f = e.copy()
        f[:, 0] = lo + f[:, 0] % (hi - lo)
        want = oracle.cc_labels(n, f)
        for fl in (0, cc.F_ZROOT):
            assert_same_labels(to_host_u32(ctx.solve(to_dev(f), n, flags=fl)), want, f"first in {lo} {fl}")
    for bad in ([n, 0], [0, 0xFFFFFFFF]):
        b = np.concatenate([e, np.array([bad], np.uint32)])
        for fl in (0, cc.F_ZROOT):
            L = torch.empty(n, dtype=torch.int32, device="cuda")
            ctx.solve_async(to_dev(b), n, L, flags=fl)
            assert ctx.sync() == cc.CC_ERANGE


def test_scratch_that_cannot_grow(ctx):
    """Under capture the filter's scratch cannot grow, nor can a server's block past
    its budget: those solves take the direct hook."""
    n, m = 3 * SLICE, 2 * SLICE * 3
    e = graphgen.er(n, m, 12)
    want = oracle.cc_labels(n, e)
    c = cc.Context(zroot_samples=4096)
    ed, L = to_dev(e), torch.empty(n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.solve_async(ed, n, L)
    for _ in range(3):
        L.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert_same_labels(to_host_u32(L), want, "captured")
    del g
    c.close()
    # room for the entries and the labels, not for the filter's tiles
    need = 8 * m + 4 * n
    s = cc.Server(ctx, streams=1, hbm_budget=(need + (4 << 20)) * 4 // 3)
    try:
        out = np.empty(n, np.uint32)
        t = s.submit(e, n, out)
        assert s.wait(t)[0] == cc.CC_OK
        assert_same_labels(out, want, "served")
    finally:
        s.close()


@pytest.mark.parametrize("kind,n,m", [("rmat", 65537, 1 << 18), ("er", 65537, (1 << 18) - 1),
                                      ("er", LDS_MAX_N, 3_000_000), ("paths", 3 * SLICE + 1, 3_000_000),
                                      ("rmat", 8 * SLICE + 40, 12_000_000),
                                      ("er", 22 * SLICE + 5, (1 << 24) + 77)])
def test_wide_ids(ctx, kind, n, m):
    """64-bit IDs through the filters: labels, IDs beyond 32 bits reported, and the
    zero root of a solve by steps untouched by one in between."""
    e = graph(kind, n, m, n + m)
    want = oracle.cc_labels(n, e)
    w = torch.from_numpy(e.astype(np.int64)).cuda()
    log(f"wide {kind} n={n} m={m}")
    assert_same_labels(ctx.solve_u64(w, n).cpu().numpy().astype(np.uint32), want, f"wide {kind} n={n}")
    bad = w.clone()
    bad[m // 2, 1] += 1 << 32
    L = torch.empty(n, dtype=torch.int64, device="cuda")
    ctx.solve_u64_async(bad, n, L)
    assert ctx.sync() == cc.CC_ERANGE
    ed = to_dev(e)
    P = torch.empty(n, dtype=torch.int32, device="cuda")
    ctx.init(n, P)
    ctx.zroot(ed, n, flags=cc.F_ZROOT | cc.F_ZROOT_HINT, zroot_hint=n - 1)
    ctx.solve_u64_async(w, n, L)
    ctx.hook(ed, n, P, flags=cc.F_ZROOT)
    ctx.compress(n, P, flags=cc.F_ZROOT)
    ctx.canon(n, P)
    assert_same_labels(to_host_u32(P), want, f"steps around a wide solve {kind} n={n}")


def test_tiles_beyond_256_slices(ctx):
    """512 second-endpoint slices: a share of R-MAT scale 28 (n = 2^28 global)."""
    ed, n = graphgen.rmat_share_dev(28, 18, graphgen.config_seed(5), 16, 0)
    assert ed.shape[0] >= n
    log(f"share28 generated: m={ed.shape[0]}")
    want = oracle.cc_labels(n, ed.cpu().numpy().view(np.uint32))
    log("share28 oracle done")
    for fl in (0, cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"share28 flags={fl}")


@pytest.mark.parametrize("n,m", [(1, 0), (1, 5), (2, 1), (65, 64), (1023, 4096), (16384, 65536), (16385, 65536),
                                 (32768, 65536), (32769, 65536), (32768, 65537), (16384, 65535)])
def test_small_in_one_launch(n, m):
    """Small whole solves by one workgroup: labels, the zero root and what later steps
    read of it, symmetric lists, endpoints out of range."""
    c = cc.Context()
    e = graph("rmat", n, m, 5 * n + m) if n > 100 else graphgen.er(n, m, 5 * n + m)
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    for fl in (0, cc.F_ZROOT, cc.F_ZROOT | cc.F_ZROOT_EXACT):
        assert_same_labels(to_host_u32(c.solve(ed, n, flags=fl)), want, f"n={n} m={m} flags={fl}")
    if m <= 65536:
        assert c.get_zroot() == oracle.zroot(n, e, 65536)
    L = c.solve(ed, n, flags=cc.F_ZROOT | cc.F_ZROOT_HINT, zroot_hint=n - 1)
    assert_same_labels(to_host_u32(L), want, f"n={n} m={m} hint")
    assert c.get_zroot() == n - 1
    sym = np.concatenate([e[:m // 2], e[:m // 2, ::-1]])
    for fl in (cc.F_SYMMETRIC, cc.F_SYMMETRIC | cc.F_ZROOT):
        assert_same_labels(to_host_u32(c.solve(to_dev(sym), n, flags=fl)), oracle.cc_labels(n, sym), f"sym {fl}")
    one_way = sym[sym[:, 0] > sym[:, 1]]           # on such a list no entry is hooked
    assert_same_labels(to_host_u32(c.solve(to_dev(one_way), n, flags=cc.F_SYMMETRIC)), np.arange(n), "one way")
    if m:
        b = e.copy()
        b[-1] = [0, n]
        for fl in (0, cc.F_ZROOT):
            c.solve_async(to_dev(b), n, L, flags=fl)
            assert c.sync() == cc.CC_ERANGE
    c.close()


@pytest.mark.parametrize("kind,n,m", [("rmat", 65537, 1 << 18), ("er", LDS_MAX_N, 3_000_000),
                                      ("paths", 300_001, 1_000_003), ("paths", 3 * SLICE + 1, 3_000_000),
                                      ("rmat", 8 * SLICE + 40, 12_000_000), ("er", 8 * SLICE + 40, 12_000_000)])
def test_rows(ctx, kind, n, m):
    """CSR graphs read as entries by the zero-root filters: empty rows, symmetric rows,
    offsets that are no row index."""
    e = graph(kind, n, m, n + m).astype(np.int64)
    e[:, 0] -= e[:, 0] % 3                         # two rows in three are empty
    e = e[np.argsort(e[:, 0], kind="stable")]
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(e[:, 0], minlength=n), out=off[1:])
    adj = to_dev(np.stack([e[:, 1], e[:, 1]], 1).astype(np.uint32))[:, 0].contiguous()
    offd = torch.from_numpy(off).cuda()
    want = oracle.cc_labels(n, e.astype(np.uint32))
    log(f"rows {kind} n={n} m={m}")
    for fl in (0, cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve_csr(offd, adj, n, flags=fl)), want, f"rows {kind} n={n} {fl}")
    assert ctx.get_zroot() == oracle.zroot_csr(off.astype(np.uint64))
    both = np.concatenate([e, e[:, ::-1]])         # a list in both orders, as the flag says
    both = both[np.argsort(both[:, 0], kind="stable")]
    off2 = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(both[:, 0], minlength=n), out=off2[1:])
    adj2 = to_dev(np.stack([both[:, 1], both[:, 1]], 1).astype(np.uint32))[:, 0].contiguous()
    got = ctx.solve_csr(torch.from_numpy(off2).cuda(), adj2, n, flags=cc.F_ZROOT | cc.F_SYMMETRIC)
    assert_same_labels(to_host_u32(got), want, f"rows {kind} n={n} symmetric")
    L = torch.empty(n, dtype=torch.int32, device="cuda")
    bad = offd.clone()
    bad[n // 2] = m + 5
    ctx.solve_csr_async(bad, adj, n, L, flags=cc.F_ZROOT)
    assert ctx.sync() == cc.CC_EINVAL


@pytest.mark.parametrize("kind", ["er", "rmat", "paths", "rows"])
@pytest.mark.parametrize("n,m", [(36 * SLICE + 7, (1 << 24) + 77), (13_421_861, (1 << 24) + 77),
                                 (13_421_834, (1 << 24) + 77), (22 * SLICE + 5, 28_835_853),
                                 (22 * SLICE + 5, 28_835_852)])
def test_two_passes_by_entries_per_vertex(ctx, kind, n, m):
    """Fewer entries than vertices, each side of 5/4 (zero root) and of 5/2 (plain)."""
    e = graph(kind, n, m, n + m)
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    log(f"{kind} n={n} m={m}")
    for name, fl in [("plain", 0), ("zroot", cc.F_ZROOT)]:
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"{kind} n={n} m={m} [{name}]")
    assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"{kind} n={n} m={m} [steps]")


def rows_of(e, n):
    """(offsets, adj) on the device of the rows (u, v) of a list."""
    e = e[np.argsort(e[:, 0], kind="stable")]
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(e[:, 0], minlength=n), out=off[1:])
    return torch.from_numpy(off).cuda(), to_dev(np.stack([e[:, 1], e[:, 1]], 1))[:, 0].contiguous()


@pytest.mark.parametrize("n,m", [(3 * SLICE + 5, 3_000_000), (8 * SLICE + 40, 12_000_000),
                                 (23 * SLICE, (1 << 24) + 8192)])
def test_chunks_without_an_entry(n, m):
    """The first chunks of 8192 entries (and some later ones) hold none that is kept:
    self-loops, or u > v on a symmetric list. Their slots in the tiles are whatever the
    scratch held before, here another list's entries."""
    c = cc.Context(zroot_samples=4096)
    c.solve(to_dev(graphgen.er(n, m + 70_000, 31)), n)
    e = graphgen.er(n, m, 32)
    loops = e.copy()
    loops[:20_000] = 0                             # row 0 of the rows begins with them too
    for a in (0, 8192, 40 * 8192, m // 8192 * 8192):
        loops[a:a + 8192, 1] = loops[a:a + 8192, 0]
    half = np.sort(e[:m // 2], axis=1)
    sym = np.ascontiguousarray(np.concatenate([half[:, ::-1], half]))   # every u > v first
    for name, x, fl in (("loops", loops, 0), ("symmetric", sym, cc.F_SYMMETRIC)):
        want = oracle.cc_labels(n, x)
        ed = to_dev(x)
        off, adj = rows_of(x, n)
        for zr in (0, cc.F_ZROOT):
            log(f"{name} n={n} m={m} zr={zr}")
            assert_same_labels(to_host_u32(c.solve(ed, n, flags=fl | zr)), want, f"{name} n={n} {zr}")
            assert_same_labels(to_host_u32(c.solve_csr(off, adj, n, flags=fl | zr)), want, f"{name} rows n={n} {zr}")
        assert_same_labels(to_host_u32(by_steps(c, ed, n, flags=fl)), want, f"{name} n={n} steps")
    c.close()


@pytest.mark.parametrize("n,m", [(900, 4000), (16_384, 60_000), (40_000, 300_000), (400_000, 900_000)])
def test_entries_rewritten_by_the_kernel_before(n, m):
    """Solves queued one after another on one buffer that a kernel rewrites in between,
    with no wait: each reads the entries written last (every path reads them only after
    a coherence point, also the small one-launch solve and the zero root's sample)."""
    c = cc.Context()
    lists = [graphgen.er(n, m, 50 + k) for k in range(4)]
    lists[2][:, 1] = lists[2][:, 0]                # nothing joined: any old entry would show
    wants = [oracle.cc_labels(n, x) for x in lists]
    devs = [to_dev(x) for x in lists]
    buf = torch.empty_like(devs[0])
    out = torch.empty((40, n), dtype=torch.int32, device="cuda")
    for fl in (0, cc.F_ZROOT):
        for i in range(len(out)):
            buf.copy_(devs[i % 4])
            c.solve_async(buf, n, out[i], flags=fl)
        assert c.sync() == cc.CC_OK
        for i in range(len(out)):
            assert_same_labels(to_host_u32(out[i]), wants[i % 4], f"n={n} m={m} flags={fl} call {i}")
    c.close()


def test_captured_solves_keep_their_scratch():
    """A solve captured on a warm context holds pointers into its scratch: larger solves
    that outgrow the scratch (and the bitmap) leave the old blocks to it until the
    context is destroyed. Replayed between eager solves."""
    n, m = 3 * SLICE, 24_000_000
    e = graphgen.er(n, m, 61)
    want = oracle.cc_labels(n, e)
    big_n, big_m = 5 * SLICE, 40_000_000
    big = to_dev(graphgen.er(big_n, big_m, 62))
    ed = to_dev(e)
    c = cc.Context(zroot_samples=4096)
    for fl in (0, cc.F_ZROOT):
        c.solve(ed, n, flags=fl)
    L = torch.empty(n, dtype=torch.int32, device="cuda")
    Lz = torch.empty(n, dtype=torch.int32, device="cuda")
    Lb = torch.empty(big_n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.solve_async(ed, n, L)
        c.solve_async(ed, n, Lz, flags=cc.F_ZROOT)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    c.solve_async(big, big_n, Lb)
    c.solve_async(big, big_n, Lb, flags=cc.F_ZROOT)
    assert c.sync() == cc.CC_OK
    # the outgrown block is still there: all of the larger list's 5 bytes per entry are
    # new, not only what they exceed the captured list's by (the runtime's own buffers
    # come and go by a few MB, hence halfway between)
    assert free - torch.cuda.mem_get_info()[0] >= 5 * big_m - 5 * m // 2, "the captured scratch was given back"
    for rep in range(3):
        L.fill_(-1)
        Lz.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert_same_labels(to_host_u32(L), want, f"replay {rep}")
        assert_same_labels(to_host_u32(Lz), want, f"replay {rep} [zroot]")
        c.solve_async(big, big_n, Lb, flags=cc.F_ZROOT if rep else 0)
    assert c.sync() == cc.CC_OK
    del g
    c.close()


def test_capture_that_would_grow_the_scratch():
    """At the sizes of the regrouped hooks a capture on a cold context takes the direct
    hook, plain and with a zero root (whose bitmap is there), and the steps too."""
    n, m = 8 * SLICE, (1 << 24) + 5
    e = graphgen.er(n, m, 63)
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    L = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)]
    c = cc.Context(zroot_samples=4096)
    c.solve(ed[:1000], n, flags=cc.F_ZROOT)         # the bitmap, no tiles
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.solve_async(ed, n, L[0])
        c.solve_async(ed, n, L[1], flags=cc.F_ZROOT)
        c.init(n, L[2])
        c.hook(ed, n, L[2])
        c.compress(n, L[2])
    for rep in range(3):
        for x in L:
            x.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        for k, x in enumerate(L):
            assert_same_labels(to_host_u32(x), want, f"replay {rep} [{k}]")
    del g
    c.close()
    cold = cc.Context()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cold.solve_async(ed, n, L[0])
        with pytest.raises(cc.CCError):              # no bitmap to capture with
            cold.solve_async(ed, n, L[1], flags=cc.F_ZROOT)
    g.replay()
    torch.cuda.synchronize()
    assert_same_labels(to_host_u32(L[0]), want, "after a refused call")
    del g
    cold.close()


def test_a_call_that_succeeds_leaves_no_failure_text():
    """A solve that goes on by another hook where its scratch cannot grow returns CC_OK
    and leaves the thread's last failure as it was."""
    n, m = 3 * SLICE, 6 * SLICE
    ed = to_dev(graphgen.er(n, m, 64))
    L = torch.empty(n, dtype=torch.int32, device="cuda")
    c = cc.Context()
    lib = cc.load()
    assert lib.cc_solve(5, 0, None, None) == cc.CC_EINVAL
    text = lib.cc_last_error_detail()
    assert text
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.solve_async(ed, n, L)
    assert lib.cc_last_error_detail() == text
    del g
    c.close()


@pytest.mark.parametrize("down", [False, True])
@pytest.mark.parametrize("n,m,path", [(1_000_000, 3_000_000, 1 << 18), (4_000_000, 8_000_000, 1 << 21)])
def test_a_long_path_beside_a_giant_component(ctx, n, m, path, down):
    """A uniform graph's component and one path of many vertices listed in order, up and
    down: the filter runs, and the path's entries all go to P, whose walks have to be
    shortened as they go."""
    h = n - path
    p = np.arange(h, n - 1, dtype=np.uint32)
    p = p[::-1] if down else p
    e = np.ascontiguousarray(np.concatenate([graphgen.er(h, m, 71), np.stack([p, p + 1], 1)]))
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    off, adj = rows_of(e, n)
    log(f"path n={n} down={down}")
    for fl in (0, cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"n={n} down={down} {fl}")
    assert_same_labels(to_host_u32(ctx.solve_csr(off, adj, n, flags=cc.F_ZROOT)), want, f"rows n={n} down={down}")
    assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"steps n={n} down={down}")
    w = ctx.solve_u64(torch.from_numpy(e.astype(np.int64)).cuda(), n)
    assert_same_labels(w.cpu().numpy().astype(np.uint32), want, f"wide n={n} down={down}")


def parts(n, m, k, side, seed):
    """k equal uniform components: side by side in the IDs, or dealt over them."""
    r = np.random.RandomState(seed)
    size = n // k
    c, a, b = r.randint(0, k, m), r.randint(0, size, m), r.randint(0, size, m)
    e = np.stack([c * size + a, c * size + b] if side else [a * k + c, b * k + c], 1)
    return np.ascontiguousarray(e.astype(np.uint32))


@pytest.mark.parametrize("side", [False, True])
@pytest.mark.parametrize("n,m,k", [(300_000, 1_200_000, 20), (100_000, 1_600_000, 20), (4 * SLICE, 1 << 24, 12),
                                   (4 * SLICE, (1 << 24) - 1, 12), (3 * SLICE + 1, 1 << 24, 12),
                                   (8 * SLICE + 40, (1 << 24) + 8191, 31), (22 * SLICE, (1 << 24) + 77, 12),
                                   (23 * SLICE, 40_000_000, 20)])
def test_components_of_equal_size(ctx, n, m, k, side):
    """Dense lists without a giant component, each side of the sizes at which their
    regrouped entries are hooked: lists, symmetric lists, steps, rows, 64-bit IDs, an
    endpoint out of range."""
    e = parts(n, m, k, side, n + m)
    want = oracle.cc_labels(n, e)
    ed = to_dev(e)
    off, adj = rows_of(e, n)
    log(f"parts n={n} m={m} side={side}")
    for fl in (0, cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"n={n} m={m} {fl}")
    assert_same_labels(to_host_u32(ctx.solve_csr(off, adj, n, flags=cc.F_ZROOT)), want, f"rows n={n} m={m}")
    assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"n={n} m={m} steps")
    w = ctx.solve_u64(ed.to(torch.int64), n)
    assert_same_labels(w.cpu().numpy().astype(np.uint32), want, f"wide n={n} m={m}")
    del w
    both = torch.cat([ed, ed.flip(1)])
    for fl in (cc.F_SYMMETRIC, cc.F_SYMMETRIC | cc.F_ZROOT):
        assert_same_labels(to_host_u32(ctx.solve(both, n, flags=fl)), want, f"symmetric n={n} m={m} {fl}")
    ed[m // 2, 1] = n
    L = torch.empty(n, dtype=torch.int32, device="cuda")
    for fl in (0, cc.F_ZROOT):
        ctx.solve_async(ed, n, L, flags=fl)
        assert ctx.sync() == cc.CC_ERANGE


def test_few_tiles_without_a_giant_component(ctx):
    """First endpoints in one slice or in a last slice of few vertices: nearly all tiles
    are empty, and parts of the tile hook's index space hold several or none."""
    n = 5 * SLICE + 11
    i = np.arange(1 << 24, dtype=np.int64)
    for lo, size in ((2 * SLICE, SLICE), (5 * SLICE, 11), (0, 3)):
        u = lo + i * 7919 % size
        v = (u % 11 + 11 * (i * 104729 % (n // 11))) % n    # a vertex's residue mod 11 is its part's
        e = np.ascontiguousarray(np.stack([u, v], 1).astype(np.uint32))
        want = oracle.cc_labels(n, e)
        ed = to_dev(e)
        log(f"few tiles at {lo}")
        for fl in (0, cc.F_ZROOT):
            assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=fl)), want, f"first in {lo} {fl}")
        assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"first in {lo} steps")


@pytest.mark.parametrize("n,m", [(60 * SLICE, (1 << 24) + 1), (36 * SLICE + 7, 23_035_903), (36 * SLICE + 7, 23_035_904),
                                 (22 * SLICE + 5, 18_087_935), (22 * SLICE + 5, 18_087_936)])
def test_few_entries_to_a_workgroup(ctx, n, m):
    """Two passes with few entries to a workgroup of the filter, and each side of 32,768
    (37 slices: 37 * 19 workgroups) and of twice that (23 slices: 23 * 12) on average:
    nearly all entries are kept, or a skewed list's marks settle most; a share's first
    endpoints lie in few slices, whose workgroups have many."""
    for kind in ("er", "rmat", "paths", "share"):
        e = graph("rmat" if kind == "share" else kind, n, m, n + m)
        if kind == "share":
            e[:, 0] %= 2 * SLICE + 77
        want = oracle.cc_labels(n, e)
        ed = to_dev(e)
        off, adj = rows_of(e, n)
        log(f"{kind} n={n} m={m}")
        assert_same_labels(to_host_u32(ctx.solve(ed, n, flags=cc.F_ZROOT)), want, f"{kind} n={n} m={m}")
        assert_same_labels(to_host_u32(ctx.solve_csr(off, adj, n, flags=cc.F_ZROOT)), want, f"rows {kind} n={n}")
        assert_same_labels(to_host_u32(by_steps(ctx, ed, n)), want, f"{kind} n={n} m={m} steps")


@pytest.mark.parametrize("kind", ["er", "rmat", "star"])
@pytest.mark.parametrize("n", [11 * SLICE, 11 * SLICE + 1])
def test_rows_by_their_longest(n, kind):
    """Rows of skewed graphs take the two-pass hook from 12 slices on, others the one-pass
    tiles; a hint leaves the longest row unknown. The zero root is the longest row's."""
    m = (1 << 24) + 9
    e = graph("er" if kind == "star" else kind, n, m, n)
    if kind == "star":                             # one long row is enough to be skewed
        e[: 1 << 12, 0] = n - 5
    want = oracle.cc_labels(n, e)
    off, adj = rows_of(e, n)
    log(f"rows {kind} n={n}")
    c = cc.Context()
    for fl in (cc.F_ZROOT, 0):
        assert_same_labels(to_host_u32(c.solve_csr(off, adj, n, flags=fl)), want, f"{kind} n={n} {fl}")
        assert c.get_zroot() == oracle.zroot_csr(off.cpu().numpy().astype(np.uint64))
    L = torch.empty(n, dtype=torch.int32, device="cuda")
    c.solve_csr_async(off, adj, n, L, flags=cc.F_ZROOT | cc.F_ZROOT_HINT, zroot_hint=n - 1)
    assert c.sync() == cc.CC_OK
    assert_same_labels(to_host_u32(L), want, f"{kind} n={n} hint")
    assert c.get_zroot() == n - 1
    c.close()


def test_served_requests_share_a_tight_arena():
    """Two requests that fit the arena together without the filter's scratch are in
    flight together; with room to spare a request has it."""
    n, m = 3 * SLICE, 6_000_000
    es = [graphgen.er(n, m, 81 + k) for k in range(2)]
    wants = [oracle.cc_labels(n, e) for e in es]
    ctx = cc.Context()
    both = 2 * (8 * m + 4 * n) + (4 << 20)
    for arena in (both, 8 * both):
        s = cc.Server(ctx, streams=2, hbm_budget=arena * 4 // 3)
        try:
            outs = [np.empty(n, np.uint32) for _ in es]
            ts = [s.submit(e, n, o) for e, o in zip(es, outs)]
            stats = [s.wait(t) for t in ts]
            assert [rc for rc, _ in stats] == [cc.CC_OK] * 2
            for o, w in zip(outs, wants):
                assert_same_labels(o, w, f"served, arena {arena}")
            a, b = stats[0][1], stats[1][1]
            assert b.t_admit_ns < a.t_done_ns, "the second request waited for the first one's room"
        finally:
            s.close()
    ctx.close()
