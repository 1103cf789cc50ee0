"""Every size of the split form at the ends of its range, on the GPU against
the CPU oracle.

Single blocks and plans take a direct product up to 1.75 10^10 key bits times
outputs, so they never run the smallest split sizes; batches whose blocks have
about as many outputs as key bits do, and served requests always.  The launch
record says which size ran: the operations of its product pass differ for all
of them.
"""
import numpy as np
import pytest

import oracle
import paper_1809_07592_amd as pa
from paper_1809_07592_amd import workloads as wl
from test_gpu_gf2_routes import check_windows, dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (T, g, log3 of the half point count): chunks of (T / 3) g words
SIZES = [(81, 1, 1), (81, 2, 1), (81, 3, 1), (243, 1, 2), (243, 2, 2), (243, 3, 2), (243, 4, 2), (243, 5, 2), (729, 1, 2)]


def capacity(k):
    T, g, _ = SIZES[k]
    return 32 * T * (T // 3) * g


def product_ops(k):
    """Binary multiply-adds of a block's product pass."""
    T, g, a = SIZES[k]
    M = T // 3 * g
    leaf = 64 * M // 3**a
    return 2.0 * T * 2 * 3**a * leaf * leaf


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()
    yield


def run(call, blocks, k):
    """The call, recorded; every block must have run at size k (None: none)."""
    torch.cuda.synchronize()
    pa.profile_enable(True)
    try:
        pa.profile_collect()
        call()
        torch.cuda.synchronize()
        prof = pa.profile_collect()
    finally:
        pa.profile_enable(False)
    ops = prof["rowconv"]["alg_ops"]
    assert "direct" not in prof
    if k is None:
        assert "rowspec" in prof and all(ops != pytest.approx(blocks * product_ops(i), rel=1e-9) for i in range(len(SIZES)))
    else:
        assert ops == pytest.approx(blocks * product_ops(k), rel=1e-9)


def data(n, m, seed_bits, i):
    key = wl.random_bits(n, wl.rng(120 + i, wl.ROLE_KEY, n), garbage_tail=True)
    seed = wl.random_bits(seed_bits, wl.rng(120 + i, wl.ROLE_SEED, n), garbage_tail=True)
    return key, seed, torch.full((wl.words(m),), -1, dtype=torch.int64, device="cuda")


@pytest.mark.parametrize("modified", [False, True])
@pytest.mark.parametrize("k", range(len(SIZES)))
def test_batches_at_the_ends_of_a_size(k, modified):
    top = capacity(k) // 64 * 64
    ends = [top] if k in (0, 1) else [capacity(k - 1) // 64 * 64 + 64, top]  # (below: direct)
    for need in ends:
        # required length 64 (ceil((n - 1) / 64) + ceil(m / 64)); a modified
        # block's hashed part may start 63 bits into its first word
        wm = need // 128
        m, n = 64 * wm - 27, need - 64 * wm + 1 - (63 if modified else 0)
        print(SIZES[k], need, n, m, flush=True)
        n += m if modified else 0
        sets = [data(n, m, n - 1 if modified else n + m - 1, i) for i in range(3)]
        blocks = [(dev(key), n, dev(seed), m, out) for key, seed, out in sets]
        run(lambda: (pa.modified_toeplitz_hash_batched if modified else pa.toeplitz_hash_batched)(blocks), 3, k)
        for key, seed, out in sets:
            check_windows(out.cpu().numpy().view(np.uint64), key, n, seed, m, modified)


@pytest.mark.parametrize("k,total", [(None, 2_000), (0, 14_000), (0, capacity(0) - 126), (1, capacity(0) - 125), (1, capacity(1) - 126)])
@pytest.mark.parametrize("part", [2, 7])
def test_served_requests_at_the_smallest_sizes(k, total, part):
    # the registered seed's length picks the size; a request's area, 4 L
    # bytes, holds the smallest size's 13,122 words from L = 13,824 on, and
    # shorter requests take the transform
    m = total // part
    n = total + 1 - m
    sets = [data(n, m, total, i) for i in range(2)]
    seed = dev(sets[0][1])
    keys = [dev(s[0]) for s in sets]
    torch.cuda.synchronize()
    with pa.Server(1 << 30) as server:
        sid = server.register_seed(seed, total)

        def serve():
            for dk, (_, _, out) in zip(keys, sets):
                server.submit(sid, dk, n, m, out)
            server.drain()

        run(serve, 2, k)
    for key, _, out in sets:
        check_windows(out.cpu().numpy().view(np.uint64), key, n, sets[0][1], m)
