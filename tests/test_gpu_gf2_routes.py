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


def bits_from(words, at, count):
    """Bits at .. at + count - 1 of packed words, packed."""
    w = np.concatenate([words[at // 64:], np.zeros(1, np.uint64)])[: wl.words(count) + 1]
    s = np.uint64(at % 64)
    return w[:-1] if s == 0 else (w[:-1] >> s) | (w[1:] << (np.uint64(64) - s))


def check_windows(got, key, n, seed, m, modified=False):
    """Three windows of an output, its ends and its middle, against the
    oracle: outputs from i on are those of the seed's bits from i on."""
    kn, x = (n - m, bits_from(key, m, n - m)) if modified else (n, key)
    for i in sorted({0, m // 128 * 64, max(0, (m - 1) // 64 * 64 - 192)}):
        w = min(256, m - i)
        want = oracle.toeplitz_hash(x, kn, bits_from(seed, i, kn + w - 1), w)
        if modified:
            head = bits_from(key, i, w)
            if w % 64:
                head[-1] &= np.uint64((1 << (w % 64)) - 1)
            want = want ^ head
        assert np.array_equal(got[i // 64: i // 64 + wl.words(w)], want), (n, m, i)


def form_of(prof, L, jobs):
    """The form that the recorded launches took: a row pass of the transform
    moves 12 L bytes a block, the split form's far less."""
    if "rowconv" not in prof:
        return "direct"
    return "transform" if prof["rowconv"]["alg_bytes"] >= 12 * L * jobs else "split"


def run_use(use, n, m, jobs, L):
    """jobs blocks of n to m, two different ones in turn, as `use` has them
    done; checks the outputs and returns the form."""
    mod = use == "modified"
    sb = n - 1 if mod else n + m - 1
    keys = [wl.random_bits(n, wl.rng(99, wl.ROLE_KEY, i), garbage_tail=True) for i in range(min(2, jobs))]
    seeds = [wl.random_bits(sb, wl.rng(99, wl.ROLE_SEED, i), garbage_tail=True)
             for i in range(min(2, jobs) if use == "batch" else 1)]
    dk, ds = [dev(k) for k in keys], [dev(s) for s in seeds]
    out = torch.full((jobs, wl.words(m)), -1, dtype=torch.int64, device="cuda")
    blocks = [(dk[i % 2], n, ds[i % 2].clone() if use == "batch" else ds[0], m, out[i]) for i in range(jobs)]
    torch.cuda.synchronize()
    plan = pa.Plan(ds[0], sb, transform_len=L) if use == "plan" else None
    server = pa.Server(2 << 30) if use == "serve" else None
    sid = server.register_seed(ds[0], sb) if server else None
    pa.profile_enable(True)
    try:
        pa.profile_collect()
        if use in ("batch", "shared"):
            pa.toeplitz_hash_batched(blocks)
        elif server:
            for k, _, _, _, o in blocks:
                server.submit(sid, k, n, m, o)
            server.drain()
        elif plan:
            plan.hash(dk[0], n, m, out[0])
        else:
            (pa.modified_toeplitz_hash if mod else pa.toeplitz_hash)(dk[0], n, ds[0], m, out[0])
        torch.cuda.synchronize()
        prof = pa.profile_collect()
    finally:
        pa.profile_enable(False)
        if server:
            server.close()
        if plan:
            plan.destroy()
    got = out.cpu().numpy().view(np.uint64)
    for i in range(min(2, jobs)):
        check_windows(got[i], keys[i], n, seeds[i % len(seeds)], m, mod)
        assert (got[i::2] == got[i]).all(), (use, n, m, i)
    return form_of(prof, L, jobs)


def fill(L, m):
    """The longest key whose block of m outputs has transform length L."""
    return L - 64 * wl.words(m) + 1


def length(n, m):
    need = 64 * ((n + 62) // 64 + wl.words(m))
    return next(x for x in pa.supported_lengths() if x >= need)


A, B, C, D, E = 3_538_944, 4_718_592, 7_077_888, 9_437_184, 14_155_776


# the form at both sides of each line between the forms: lengths just above a
# split size run at the transform, beyond a number of outputs or of blocks
@pytest.mark.parametrize("use,L,m,jobs,form", [
    ("plain", A, A // 4, 1, "split"), ("plain", A, A // 4 + 1, 1, "transform"), ("plain", B, 20_003, 1, "split"),
    ("plain", C, 20_003, 1, "transform"), ("plain", C, C // 2 - 300, 1, "transform"),
    ("plain", D, D // 16 * 6, 1, "split"), ("plain", D, D // 16 * 6 + 1, 1, "transform"),
    ("plain", E, 20_003, 1, "split"), ("plan", A, 20_003, 1, "transform"), ("plan", A, 4_001, 1, "direct"),
    ("plan", B, B // 2 - 300, 1, "split"),
    ("plan", C, 20_003, 1, "transform"), ("plan", D, D // 8, 1, "split"), ("plan", D, D // 8 + 1, 1, "transform"),
    ("plan", E, E // 2 - 300, 1, "split"),
    ("serve", 221_184, 20_003, 3, "transform"), ("serve", 294_912, 20_003, 3, "split"),
    ("serve", 131_072, 20_003, 3, "split"), ("serve", 147_456, 20_003, 3, "transform"),
    ("serve", A, A // 8, 3, "split"), ("serve", A, A // 8 + 1, 3, "transform"), ("serve", C, 20_003, 3, "transform"),
    ("serve", D, D // 8, 2, "split"), ("serve", D, D // 8 + 1, 2, "transform"),
    ("batch", 221_184, 50_003, 11, "split"), ("batch", 221_184, 50_003, 12, "transform"),
    ("batch", 221_184, 50_003, 136, "split"), ("batch", 262_144, 60_003, 12, "transform"),
    ("batch", A, A // 16 * 7, 2, "split"), ("batch", A, A // 16 * 7 + 1, 2, "transform"),
    ("batch", A, A // 16 * 7 + 1, 3, "split"), ("batch", C, 20_003, 2, "transform"), ("batch", C, 2_003, 2, "transform"),
    ("batch", D, D // 16 * 5, 2, "split"), ("batch", D, D // 16 * 5 + 1, 2, "transform"), ("batch", E, 20_003, 2, "split"),
    ("shared", 221_184, 50_003, 5, "split"), ("shared", 221_184, 50_003, 6, "transform"),
    ("shared", 3_145_728, 20_003, 9, "split"), ("shared", 3_145_728, 20_003, 10, "transform"),
    ("shared", 3_145_728, 20_003, 22, "split"), ("shared", A, A // 16 * 3 + 1, 3, "transform"),
    ("shared", A, A // 16 * 6, 8, "split"), ("shared", D, D // 8, 3, "split"), ("shared", D, D // 8 + 1, 3, "transform"),
])
def test_lines_between_split_form_and_transform(use, L, m, jobs, form):
    print(use, L, m, jobs, flush=True)
    n = fill(L, m)
    assert length(n, m) == L
    assert run_use(use, n, m, jobs, L) == form


@pytest.mark.parametrize("kn,m,form", [(100_000, 140_000, "split"), (80_000, 160_000, "direct"),
                                       (120_000, 131_072, "direct"), (fill(E, E // 16 * 12), E // 16 * 12, "split"),
                                       (fill(E, E // 16 * 12 + 1), E // 16 * 12 + 1, "transform")])
def test_lines_of_long_outputs(kn, m, form):
    assert run_use("modified", kn + m, m, 1, length(kn, m)) == form


def test_one_plan_serves_both_spectra():
    # a plan at a length where the outputs decide: both forms in turn, the
    # transform's spectrum as the diagnostics have it, and a short block
    L = D
    seed = wl.random_bits(L, wl.rng(100, wl.ROLE_SEED, 0))
    ds = dev(seed)
    with pa.Plan(ds, L, transform_len=L) as plan:
        for m in (L // 8, L // 4, L // 8 - 64, 1_000, L // 4 + 77):
            n = fill(L, m) if m > 1_000 else 1_000_000
            key = wl.random_bits(n, wl.rng(100, wl.ROLE_KEY, m))
            check_windows(host(plan.hash(dev(key), n, m), m), key, n, seed, m)
        spec = plan.spectrum()
        torch.cuda.synchronize()
    try:
        for cls in (0, 1):
            pa.tune_set(L, cls, 0, 0, 0, pa.plan_info(L)["row_threads"])
        with pa.Plan(ds, L, transform_len=L) as plan:
            assert torch.equal(spec, plan.spectrum())
    finally:
        for cls in (0, 1):
            pa.tune_set(L, cls, 0, 0)


@pytest.mark.parametrize("L,jobs,outputs", [(221_184, 12, (50_003, 101_009, 3_001)), (110_592, 2, (2_601, 49_999, 1)),
                                            (98_304, 2, (1, 2_601, 48_000))])
def test_graph_updated_within_its_form(L, jobs, outputs):
    # blocks that take the transform, or a sliced or unsliced direct product,
    # replayed, then updated to other sizes of their length
    sets = []
    for m in outputs:
        n = fill(L, m)
        keys = [wl.random_bits(n, wl.rng(101, wl.ROLE_KEY, i + m)) for i in range(jobs)]
        seeds = [wl.random_bits(n + m - 1, wl.rng(101, wl.ROLE_SEED, i + m)) for i in range(jobs)]
        sets.append((n, m, keys, seeds, [(dev(k), n, dev(s), m, torch.full((wl.words(m),), -1, dtype=torch.int64,
                                                                           device="cuda")) for k, s in zip(keys, seeds)]))
    with pa.BatchGraph(sets[0][4]) as g:
        for n, m, keys, seeds, blocks in sets + sets[:1]:
            g.update(blocks)
            for _ in range(2):
                for b in blocks:
                    b[4].fill_(-1)
                g.launch()
                torch.cuda.synchronize()
                for k, s, b in zip(keys, seeds, blocks):
                    check_windows(host(b[4], m), k, n, s, m)


@pytest.mark.parametrize("modified", [False, True])
def test_graph_memory_is_bounded_by_its_lengths(modified):
    # a graph keeps room for the most outputs of its blocks' lengths; sliced
    # direct products of few outputs must not multiply that by their slices
    L, m = 9_437_184, 60
    n = fill(L, m)
    key, seed = dev(wl.random_bits(n + m, wl.rng(102, wl.ROLE_KEY, 0))), dev(wl.random_bits(n + m, wl.rng(102, wl.ROLE_SEED, 0)))
    out = torch.zeros(1, dtype=torch.int64, device="cuda")
    blocks = [(key, n + (m if modified else 0), seed, m, out)]
    with pa.BatchGraph([(key, 5_000, seed, m, out)], modified=modified) as g:  # (what a first graph allocates)
        g.launch()
        torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    with pa.BatchGraph(blocks, modified=modified) as g:
        used = before - torch.cuda.mem_get_info()[0]
        for _ in range(2):
            g.launch()
            torch.cuda.synchronize()
    assert used <= 8 * L + (32 << 20), used
    k, s = key.cpu().numpy().view(np.uint64), seed.cpu().numpy().view(np.uint64)
    check_windows(host(out, m), k, blocks[0][1], s, m, modified)
