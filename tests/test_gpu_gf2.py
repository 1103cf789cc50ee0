"""The carry-less forms of the hash on the GPU, bit for bit against the CPU
oracle: direct binary products (every alignment of the key's end, sizes
around the tile and unit edges, one launch and several slices of the key) and
split cyclic products (each transform size at its smallest and largest block),
through the plain, modified, plan, batched and graph calls."""
import numpy as np
import pytest

import oracle
import paper_1809_07592_amd as pa
from paper_1809_07592_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build()
    yield


def inputs(n, m, modified=False, tag=0, ones=False):
    sb = n - 1 if modified else n + m - 1
    if ones:
        return (np.full(wl.words(n), 2**64 - 1, np.uint64), np.full(wl.words(sb), 2**64 - 1, np.uint64))
    # words past the last bit hold garbage, as a caller's buffers may
    return (wl.random_bits(n, wl.rng(95, wl.ROLE_KEY, tag), garbage_tail=True),
            wl.random_bits(sb, wl.rng(95, wl.ROLE_SEED, tag), garbage_tail=True))


def want(key, n, seed, m, modified):
    return (oracle.modified_toeplitz_hash if modified else oracle.toeplitz_hash)(key, n, seed, m)


def check_one(n, m, modified=False, ones=False):
    key, seed = inputs(n, m, modified, ones=ones)
    out = torch.full((wl.words(m) + 2,), -1, dtype=torch.int64, device="cuda")
    (pa.modified_toeplitz_hash if modified else pa.toeplitz_hash)(dev(key), n, dev(seed), m, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint64)
    w = want(key, n, seed, m, modified)
    assert np.array_equal(got[: w.size], w), (n, m, modified)
    assert (got[w.size:] == 2**64 - 1).all(), "wrote past the output"


def check_batch(shapes, modified=False, graph=False):
    data = [(*inputs(n, m, modified, tag=i), n, m) for i, (n, m) in enumerate(shapes)]
    blocks = [(dev(k), n, dev(s), m, torch.full((wl.words(m),), -1, dtype=torch.int64, device="cuda"))
              for k, s, n, m in data]
    if graph:
        with pa.BatchGraph(blocks, modified=modified) as g:
            for _ in range(2):
                for b in blocks:
                    b[4].fill_(-1)
                g.launch()
                torch.cuda.synchronize()
    else:
        (pa.modified_toeplitz_hash_batched if modified else pa.toeplitz_hash_batched)(blocks)
    torch.cuda.synchronize()
    for (k, s, n, m), b in zip(data, blocks):
        assert np.array_equal(b[4].cpu().numpy().view(np.uint64), want(k, n, s, m, modified)), (n, m, modified)


@pytest.mark.parametrize("modified", [False, True])
def test_direct_every_alignment(modified):
    # key ends at every bit of a word, lengths below one unit of steps, at
    # its edges and over several (1024 bits a unit), odd output lengths
    shapes = [(n, max(1, min(n - 1, 1 + (37 * n) % 700))) for n in range(2, 66)]
    for base in (128 - 16, 1024 - 16, 2048 - 16, 8192 - 16, 13568 - 16, 16384 - 16):
        shapes += [(base + d, 1 + (53 * (base + d)) % 1100) for d in range(0, 64, 3)]
    check_batch([(n, min(m, n - 1)) for n, m in shapes], modified=modified)


@pytest.mark.parametrize("n,m", [(1, 1), (64, 64), (4097, 4097), (70_001, 1), (65_000, 255), (65_001, 256), (65_002, 257),
                                 (99_991, 1023), (99_999, 1025), (200_017, 30_011), (131_090, 65_535), (100_003, 70_001)])
def test_direct_one_block(n, m):
    check_one(n, m)
    if m < n:
        check_one(n, m, modified=True)


def test_direct_all_ones():
    # every count at its largest: n ones
    check_one(4097, 4097, ones=True)
    check_one(200_000, 50_000, ones=True)


# cyclic lengths of the split sizes: 32 T M bits, M = (T / 3) g words
SIZES = [(81, 1), (81, 2), (81, 3), (243, 1), (243, 2), (243, 3), (243, 4), (243, 5), (729, 1)]


@pytest.mark.parametrize("k", range(len(SIZES)))
@pytest.mark.parametrize("modified", [False, True])
def test_split_smallest_and_largest(k, modified):
    # plans always split: the seed's length picks the size
    def cap(i):
        T, g = SIZES[i]
        return 32 * T * (T // 3) * g

    lo = cap(k - 1) - 100 if k else 2_000
    hi = cap(k) - 130
    for total in (lo, hi):
        m = min(total // 5, 40_000) + 3
        n = total - m + 1
        if modified:
            check_one(n, min(m, n // 2), modified=True)
            continue
        key, seed = inputs(n, m, tag=total % 97)
        with pa.Plan(dev(seed), n + m - 1, transform_len=pa.transform_len(n, m)) as plan:
            got = plan.hash(dev(key), n, m)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy().view(np.uint64)[: wl.words(m)], want(key, n, seed, m, False))
        check_one(n, m)


def test_split_largest_size():
    # T = 729 with the widest chunks, just above the size below it
    check_one(5_600_011, 70_003)


def test_split_all_ones_and_full_output():
    check_one(1_000_000, 250_000, ones=True)
    check_one(300_007, 300_007)


def test_plan_with_a_longer_seed_and_many_sizes():
    # the seed is longer than the blocks need, and longer than the transform
    for seed_bits, L in ((400_000, 0), (900_000, 589_824), (1_000_000, 1_048_576)):
        seed = wl.random_bits(seed_bits, wl.rng(96, wl.ROLE_SEED, L), garbage_tail=True)
        with pa.Plan(dev(seed), seed_bits, transform_len=L) as plan:
            for n, m in ((200_000, 100_001), (150_007, 1), (99_999, 99_999), (333_333, 66_000), (5_000, 77)):
                if n + m - 1 > seed_bits or 64 * ((n + 62) // 64 + (m + 63) // 64) > plan.transform_len:
                    continue
                key = wl.random_bits(n, wl.rng(96, wl.ROLE_KEY, n))
                got = plan.hash(dev(key), n, m)
                torch.cuda.synchronize()
                assert np.array_equal(got.cpu().numpy().view(np.uint64)[: wl.words(m)],
                                      oracle.toeplitz_hash(key, n, seed, m)), (seed_bits, L, n, m)


@pytest.mark.parametrize("modified", [False, True])
@pytest.mark.parametrize("graph", [False, True])
def test_batches_of_both_forms(modified, graph):
    g = np.random.default_rng(97)
    shapes = []
    for _ in range(24):
        n = int(round(2.0 ** g.uniform(9, 20)))
        shapes.append((n, max(1, min(n - 1, int(round(n * g.uniform(0.05, 0.5)))))))
    check_batch(shapes, modified=modified, graph=graph)


def test_graph_update_to_other_sizes_of_the_same_lengths():
    # blocks of one transform length, captured small and updated to the
    # largest key and the largest output that the length takes
    L = 98_304
    for first, second in (((60_000, 20_000), (97_000, 1_200)), ((97_000, 1_200), (49_000, 49_000))):
        for n, m in (first, second):
            assert pa.transform_len(n, m) == L
        data = [[(*inputs(n, m, tag=7 * i + j), n, m) for j in range(3)] for i, (n, m) in enumerate((first, second))]
        sets = [[(dev(k), n, dev(s), m, torch.full((wl.words(m),), -1, dtype=torch.int64, device="cuda"))
                 for k, s, n, m in d] for d in data]
        with pa.BatchGraph(sets[0]) as graph:
            for blocks, d in ((sets[0], data[0]), (sets[1], data[1]), (sets[0], data[0])):
                graph.update(blocks)
                for b in blocks:
                    b[4].fill_(-1)
                graph.launch()
                torch.cuda.synchronize()
                for (k, s, n, m), b in zip(d, blocks):
                    assert np.array_equal(b[4].cpu().numpy().view(np.uint64), oracle.toeplitz_hash(k, n, s, m)), (n, m)


def check_many(n, m, jobs, modified=False):
    """`jobs` blocks, two different ones in turn, each in buffers of its own."""
    pair = [(*inputs(n, m, modified, tag=t),) for t in range(2)]
    wants = [want(k, n, s, m, modified) for k, s in pair]
    sent = [(dev(k), dev(s)) for k, s in pair]
    out = torch.full((jobs, wl.words(m)), -1, dtype=torch.int64, device="cuda")
    blocks = [(sent[i % 2][0].clone(), n, sent[i % 2][1].clone(), m, out[i]) for i in range(jobs)]
    (pa.modified_toeplitz_hash_batched if modified else pa.toeplitz_hash_batched)(blocks)
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint64)
    bad = [i for i in range(jobs) if not np.array_equal(got[i], wants[i % 2])]
    assert not bad, (n, m, jobs, modified, bad[:5])


@pytest.mark.parametrize("n,m,jobs", [(20_003, 2_001, 40), (9_001, 2_300, 100), (150_001, 3_001, 8)])
def test_direct_many_blocks(n, m, jobs):
    # two and four tiles a workgroup, and slices of the key
    check_many(n, m, jobs)


@pytest.mark.parametrize("wide", [1, 2, 4])
@pytest.mark.parametrize("g", [1, 2, 3, 4, 5])
def test_split_many_blocks(g, wide):
    # enough blocks for the inverse pass that stages products, at each of its
    # widths: ranges of 1024 words (2048 with even g) times 1, 2 and 4
    half = 16 * 243 * 81 * g - 100
    cover = 1024 * wide * (2 if g % 2 == 0 else 1) - 2
    ranges = -(-(-(-half // 64) * 2 + 1) // cover)
    check_many(half + 37, half - 30, -(-256 // ranges))


@pytest.mark.parametrize("n,m,jobs", [(36_001, 33_003, 6), (70_001, 66_003, 6), (104_001, 100_003, 6),
                                      (3_600_001, 20_003, 5), (5_800_001, 20_003, 5)])
def test_split_some_blocks(n, m, jobs):
    check_many(n, m, jobs)


@pytest.mark.parametrize("m", [64_000, 64_001, 64_031, 64_032, 64_033, 64_063])
def test_split_key_inside_its_buffer(m):
    # every kind of start of the hashed part within its 64-bit word, odd and
    # even word units, few and many blocks, and a cyclic length that only
    # the block without those bits would fit
    for n in (400_001, 900_001):
        check_one(n, m, modified=True)
        check_many(n, m, 6, modified=True)
    total = 32 * 243 * 81
    check_one(total - 63, m, modified=True)
    check_many(total - 40, m, 70, modified=True)
