"""Which form a call takes, and that the choice changes nothing else, on the
GPU against the CPU oracle."""
import numpy as np
import pytest

import oracle
import paper_1809_07592_amd as pa
from paper_1809_07592_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def host(t, m):
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)[: wl.words(m)]


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()
    yield


@pytest.mark.parametrize("form", ["plain", "modified", "plan"])
def test_blocks_of_one_length_share_a_workspace(form):
    # a call captured after another one of its transform length, whatever the
    # forms that the two take: nothing may be allocated then
    L, sizes = 3_145_728, [(3_000_000, 2_000), (3_000_001, 20_003)]  # direct, split
    mod = form == "modified"
    hash_, want = ((pa.modified_toeplitz_hash, oracle.modified_toeplitz_hash) if mod else
                   (pa.toeplitz_hash, oracle.toeplitz_hash))
    seed_bits = sum(sizes[1])
    seed = wl.random_bits(seed_bits, wl.rng(98, wl.ROLE_SEED, 0))
    ds, data = dev(seed), []
    for i, (n, m) in enumerate(sizes):
        assert pa.transform_len(n, m) == L
        n += m if mod else 0
        key = wl.random_bits(n, wl.rng(98, wl.ROLE_KEY, i))
        data.append((key, dev(key), n, m, torch.zeros(wl.words(m), dtype=torch.int64, device="cuda")))
    plan = pa.Plan(ds, seed_bits, transform_len=L) if form == "plan" else None

    def call(i):
        _, dk, n, m, out = data[i]
        plan.hash(dk, n, m, out) if plan else hash_(dk, n, ds, m, out)

    call(1)  # its kernels are loaded, on another stream
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call(1)
    for i in (1, 0, 1):
        for d in data:
            d[4].fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        if i == 0:
            call(0)  # eager work between the replays
        key, _, n, m, out = data[1]
        assert np.array_equal(host(out, m), want(key, n, seed, m)), form
    key, _, n, m, out = data[0]
    call(0)
    assert np.array_equal(host(out, m), want(key, n, seed, m)), form
