"""The device's check of an uploaded pool: it accepts and lays out what the host
check accepts, and refuses the rest with the host's code and message, the old
pool staying."""
import numpy as np
import pytest

from canvasgen import LEAF, LEAF_DTYPE, LEAF_F64, LEAF_RGBA8_F16, Canvas, make_view, trees

from test_gpu_links import check_records

pytestmark = pytest.mark.gpu

FREE = 0xFFFFFFFF


@pytest.fixture(scope="module")
def sess():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    s = Session(0)
    yield s
    s.close()


def _with_gaps(cv, seed):
    """The same tree with its groups moved to random places of a larger pool,
    garbage in the groups between them, leaves shared and in another order."""
    rng = np.random.Generator(np.random.PCG64(seed))
    roots = (cv.R ** 3 + 7) // 8 * 8
    n = (len(cv.nodes) - roots) // 8
    place = rng.permutation(2 * n + 3)[:n]
    old = cv.nodes.astype(np.int64)
    new = rng.integers(0, 2 ** 32, (roots + 8 * (2 * n + 3), 2)).astype(np.uint32)
    ids = np.concatenate([np.arange(roots),
                          (roots + 8 * place[:, None] + np.arange(8)).reshape(-1)])
    child, parent = old[:, 0].copy(), old[:, 1].copy()
    inner = child < LEAF
    inner[cv.R ** 3:roots] = False
    child[inner] = ids[child[inner]]
    li = rng.integers(0, max(len(cv.leaves) // 2, 1), (~inner).sum())
    child[~inner] = LEAF | li
    has = parent != FREE
    has[:roots] = False
    parent[has] = ids[parent[has]]
    new[ids, 0], new[ids, 1] = child, parent
    return Canvas(R=cv.R, max_depth=cv.max_depth, origin=cv.origin, root_edge=cv.root_edge,
                  leaf_format=cv.leaf_format, nodes=new, leaves=cv.leaves)


def _walk(cv):
    """Record words and leaf indices by node id, from the roots down."""
    x = np.full(len(cv.nodes), FREE, np.uint32)
    leaf = np.full(len(cv.nodes), -1, np.int64)
    level, d = np.arange(cv.R ** 3), 0
    while len(level):
        c = cv.nodes[level, 0]
        inner = c < LEAF
        x[level] = np.where(inner, c, 1 | d << 1)
        leaf[level[~inner]] = c[~inner] & (LEAF - 1)
        level = (c[inner, None].astype(np.int64) + np.arange(8)).reshape(-1)
        d += 1
    return x, leaf


def _pools():
    for fmt in (LEAF_RGBA8_F16, LEAF_F64):
        yield "one root", trees.single_cell((0.2, 0.4, 0.6), 0.5, fmt)
        for R, depth, p, n in ((1, 1, 0.5, 9), (1, 8, 0.6, 6000), (2, 6, 0.5, 4000),
                               (3, 5, 0.3, 3000), (7, 3, 0.2, 4000)):
            cv = trees.random_tree(R, depth, seed=R + n, p_split=p, max_nodes=n, leaf_format=fmt)
            yield "R=%d" % R, cv
            yield "R=%d, gaps" % R, _with_gaps(cv, n)
        yield "depth 30", trees.deep_path_tree(30, seed=9, leaf_format=fmt)
    # more refined nodes on a level (68,921) than one pass of a launch takes (65,536)
    R = 41
    first = (R ** 3 + 7) // 8 * 8
    nodes = np.full((first + 8 * R ** 3, 2), FREE, np.uint32)
    nodes[:R ** 3, 0] = first + 8 * np.arange(R ** 3)
    nodes[first:, 0] = LEAF | np.arange(8 * R ** 3)
    nodes[first:, 1] = np.arange(8 * R ** 3) // 8
    leaves = np.zeros(8 * R ** 3, LEAF_DTYPE[LEAF_RGBA8_F16])
    leaves["r"] = np.arange(8 * R ** 3) % 251
    yield "wide", Canvas(R=R, max_depth=1, origin=(0.0, 0.0, 0.0), root_edge=1.0,
                         leaf_format=LEAF_RGBA8_F16, nodes=nodes, leaves=leaves)


def test_upload_lays_out_what_the_host_check_accepts(sess):
    from paper_1704_02724_amd import cvx
    for name, cv in _pools():
        print(name, cv.leaf_format, len(cv.nodes), flush=True)
        for depth in (cv.max_depth, min(cv.max_depth + 2, 30 - (cv.R - 1).bit_length())):
            cv.max_depth = depth
            sess.upload(0, cv)
            rec = cvx.cvx_read_records(sess.ctx, 0)
            x, leaf = _walk(cv)
            np.testing.assert_array_equal(rec[:, 0], x)
            assert (rec[x == FREE] == FREE).all()
            pay = cvx.cvx_read_payloads(sess.ctx, 0, LEAF_DTYPE[cv.leaf_format])
            want = np.zeros(len(x), cv.leaves.dtype)
            want[leaf >= 0] = cv.leaves[leaf[leaf >= 0]]
            assert pay.tobytes() == want.tobytes()
        if len(x) < 20000:
            check_records(rec, cv.R)


def _faults(cv, rng):
    """Pools with one fault (or none: some words may take any value)."""
    n = cv.nodes
    inner = np.nonzero(n[:, 0] < LEAF)[0]
    leaf = np.nonzero(n[:, 0] >= LEAF)[0]
    leaf = leaf[(leaf < cv.R ** 3) | (leaf >= (cv.R ** 3 + 7) // 8 * 8)]
    groups = np.unique(n[inner, 0])

    def put(node, word, value):
        a = n.copy()
        a[node, word] = value
        return a, cv.leaves

    a, b = rng.choice(inner, 2, replace=False)
    yield put(a, 0, n[b, 0])                                # a group shared
    up = int(inner[-1])
    yield put(up, 0, n[0, 0] if n[0, 0] < LEAF else groups[0])  # a cycle, or shared
    m = n.copy()                                            # two leaves claim one group
    p, q = rng.choice(leaf, 2, replace=False)
    m = np.concatenate([m, np.full((8, 2), LEAF, np.uint32)])
    m[[p, q], 0] = len(n)
    m[len(n):, 1] = q
    yield m, cv.leaves
    yield put(p, 0, len(n))                                 # past the end
    yield put(p, 0, len(n) - 4)
    yield put(p, 0, 0x7FFFFFF8)
    yield put(a, 0, n[a, 0] + 4)
    yield put(a, 0, 0)
    yield put(p, 0, LEAF | len(cv.leaves))
    yield put(p, 0, 0xFFFFFFFF)
    yield put(int(n[a, 0]) + rng.integers(8), 1, a ^ 1)
    yield put(cv.R ** 3 - 1, 1, 0)
    for i in rng.integers(0, len(n), 12):                   # any word, any value near
        w = int(rng.integers(2))
        yield put(i, w, rng.choice([0, 8, n[i, w] ^ 1, n[i, w] ^ 8, n[i, w] ^ LEAF, FREE]))
    bad = [0x8001, 0xBC00, 0x7C00, 0x7E00, 0xFC00] if cv.leaf_format == LEAF_RGBA8_F16 else \
        [np.nan, np.inf, -np.inf, -1e-300]
    for v in bad + [0x8000 if cv.leaf_format == LEAF_RGBA8_F16 else -0.0]:  # minus zero is taken
        lv = cv.leaves.copy()
        lv["kappa"][rng.integers(len(lv))] = v
        yield n, lv
    if cv.leaf_format == LEAF_F64:
        lv = cv.leaves.copy()
        lv["g"][-1] = np.nan
        yield n, lv


@pytest.mark.parametrize("fmt", [LEAF_RGBA8_F16, LEAF_F64])
@pytest.mark.parametrize("R,depth", [(1, 7), (2, 5), (3, 4)])
def test_upload_refuses_what_the_host_check_refuses(sess, fmt, R, depth):
    from paper_1704_02724_amd import cvx
    rng = np.random.Generator(np.random.PCG64(10 * R + depth))
    cv = trees.random_tree(R, depth, seed=R, max_nodes=2500, leaf_format=fmt)
    view = [make_view((0.5, 0.5, -1.0), (0.0, 0.0, 1.0), 0.5, 16, 16, canvas_id=0)]
    variant = "fp32_rebased" if fmt == LEAF_RGBA8_F16 else "fp64_plain"
    sess.upload(0, cv)
    ref = sess.render(view, variant).cpu().numpy()
    refused = 0
    for k, (nodes, leaves) in enumerate(_faults(cv, rng)):
        print(k, flush=True)
        for limit in (depth, depth - 1) if k == 0 else (depth,):
            d = cvx.make_desc(cv.origin, cv.root_edge, R, limit, fmt)
            rc, msg = cvx.cvx_validate_pool(d, nodes, leaves)
            if rc == 0:
                cvx.cvx_upload_pool(sess.ctx, 1, d, nodes, leaves)
                continue
            refused += 1
            with pytest.raises(cvx.CvxError) as e:
                cvx.cvx_upload_pool(sess.ctx, 0, d, nodes, leaves)
            assert e.value.code == rc and msg in str(e.value)
    assert refused >= 12
    np.testing.assert_array_equal(sess.render(view, variant).cpu().numpy(), ref)


@pytest.mark.parametrize("name", ["R=2, gaps", "depth 30", "wide"])
def test_first_edit_after_an_upload(sess, name):
    """The first edit counts the leaves per depth on the device (the wide pool
    has more nodes than one pass of that launch): one refined leaf gives the
    records of a fresh upload, and merged again those of the first."""
    from paper_1704_02724_amd import cvx
    cv = dict((n, c) for n, c in _pools() if c.leaf_format == LEAF_RGBA8_F16)[name]
    sess.upload(0, cv)
    before = cvx.cvx_read_records(sess.ctx, 0)
    x, _ = _walk(cv)
    leaves = np.nonzero((x != FREE) & (x & 1 == 1) & (x >> 1 < cv.max_depth))[0]
    if name == "wide":  # its leaves are at its max_depth: one more
        cv.max_depth = 2
        sess.upload(0, cv)
        leaves = np.nonzero(x & 1)[0]
    i, g = int(leaves[len(leaves) // 2]), (len(x) + 7) // 8 * 8
    first = sess.edit(0, [(1, i, 0)], np.repeat(cv.leaves[:1], 8))
    assert first[0] == g
    edited = cvx.cvx_read_records(sess.ctx, 0)
    nodes = np.concatenate([cv.nodes, np.full((g + 8 - len(x), 2), FREE, np.uint32)])
    nodes[i, 0], nodes[g:, 0], nodes[g:, 1] = g, LEAF, i
    cv.nodes = nodes
    sess.upload(1, cv)
    np.testing.assert_array_equal(edited, cvx.cvx_read_records(sess.ctx, 1))
    sess.edit(0, [(2, i, 0)], cv.leaves[:1])
    np.testing.assert_array_equal(cvx.cvx_read_records(sess.ctx, 0)[:len(x)], before)
