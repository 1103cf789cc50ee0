"""The number-theoretic transform at the default geometries, on the GPU
against the CPU oracle.

Untuned calls take the carry-less forms wherever those are faster, so the row
and column kernels compiled for the default geometries' shapes run only where
they are not, in flat batches, or under a geometry of the caller's.  A geometry
that differs from the default in nothing but a fixed row workgroup size (the
one the default would use) selects the transform on the same shapes; here each
shape runs so on the plain, plan and batched paths, and the library's launch
record shows that it did.
"""
import contextlib

import numpy as np
import pytest

import oracle
import paper_1809_07592_amd as pa
from paper_1809_07592_amd import workloads as wl
from test_gpu_fixed_shapes import SHAPES, block_for, dev, extreme_blocks, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()


@contextlib.contextmanager
def transform_only(L, blocks):
    """The default geometry of L with its row workgroup size fixed; on the
    way out checks that the row passes of all `blocks` blocks were the
    transform's, which move 12 L bytes each."""
    d = pa.plan_info(L)
    try:
        for cls in (0, 1):
            pa.tune_set(L, cls, 0, 0, 0, d["row_threads"])
            got = pa.tune_get_geometry(L, cls)
            assert (1 << got["log2_rows"], got["tile_width"]) == (d["rows"], d["tile_width"])
        pa.profile_enable(True)
        pa.profile_collect()
        yield
        torch.cuda.synchronize()
        prof = pa.profile_collect()
        assert "direct" not in prof
        assert prof["rowconv"]["alg_bytes"] >= 12 * L * blocks
    finally:
        pa.profile_enable(False)
        for cls in (0, 1):
            pa.tune_set(L, cls, 0, 0)


def check(L, n, m, tag, plan=True):
    key, seed = wl.key_and_seed(tag, n, m, 0)
    want = oracle.toeplitz_hash(key, n, seed, m)
    dk, ds = dev(key), dev(seed)
    with transform_only(L, 6 if plan else 5):
        assert np.array_equal(host(pa.toeplitz_hash(dk, n, ds, m), m), want), ("plain", n)
        if plan:
            with pa.Plan(ds, n + m - 1, transform_len=L) as p:
                assert np.array_equal(host(p.hash(dk, n, m), m), want), ("plan", n)
        outs = [torch.zeros(wl.words(m), dtype=torch.int64, device="cuda") for _ in range(2)]
        seeds = (ds, ds.clone())
        pa.toeplitz_hash_batched([(dk, n, s, m, o) for s, o in zip(seeds, outs)])
        for o in outs:
            assert np.array_equal(host(o, m), want), ("batched", n)
        outs = [torch.zeros(wl.words(m), dtype=torch.int64, device="cuda") for _ in range(2)]
        pa.toeplitz_hash_batched([(dk, n, ds, m, o) for o in outs])
        for o in outs:
            assert np.array_equal(host(o, m), want), ("shared seed", n)


IDS = [f"L{L}_row{r}_col{c}" for L, r, c in SHAPES]


@pytest.mark.parametrize("L,sh,cs", SHAPES, ids=IDS)
def test_every_default_shape(L, sh, cs):
    n, m = block_for(L)
    check(L, n, m, 160 + sh)


@pytest.mark.parametrize("L,sh,cs", SHAPES, ids=IDS)
def test_ends_of_each_length(L, sh, cs):
    for n in extreme_blocks(L, 1_037):
        check(L, n, 1_037, 180 + sh, plan=False)


@pytest.mark.parametrize("L", [393216, 1572864])
def test_many_blocks_on_wide_forward_tiles(L):
    # at least 1024 forward tiles of 64 columns
    d = pa.plan_info(L)
    assert d["tile_width"] == 16 and pa.plan_info(L, 0, 64)["col_shape"] != 0
    count, n, m = -(-1024 // (2 * d["cols"] // 64)), int(L * 0.9), 20_037
    assert pa.transform_len(n, m) == L
    pair = [wl.key_and_seed(195, n, m, i) for i in range(2)]
    wants = [oracle.toeplitz_hash(k, n, s, m) for k, s in pair]
    sent = [(dev(k), dev(s)) for k, s in pair]
    out = torch.zeros(count, wl.words(m), dtype=torch.int64, device="cuda")
    blocks = [(sent[i % 2][0], n, sent[i % 2][1].clone(), m, out[i]) for i in range(count)]
    with transform_only(L, count):
        pa.toeplitz_hash_batched(blocks)
    got = out.cpu().numpy().view(np.uint64)
    assert all(np.array_equal(got[i], wants[i % 2]) for i in range(count))
