"""The performance cases of the Toeplitz-hash library: what a key-distillation
program has it do, through the public entry points of paper_1809_07592_amd.

A case is a form of the call and its sizes (n key bits to m output bits):

  plain     one block, toeplitz_hash
  modified  one block of the (I, V) matrix, modified_toeplitz_hash
  plan      one key against a plan that keeps the seed's spectrum
  batch     `count` blocks in one toeplitz_hash_batched call; n and m of
            every block, or (n_lo, n_hi, mix) for blocks of mixed sizes
  shared    a batch whose blocks all use one seed
  graph     a batch captured once in a BatchGraph and replayed
  serve     `count` requests of mixed sizes against four registered seeds,
            submitted to a Server and waited for

Outputs are the packed key bits themselves, whole numbers with one right
value each, so there is no rounding to compare and no exact().
"""
import math
import random

import torch

import paper_1809_07592_amd as pa

# The longest block and the most key bits a case may hold.
N_MIN, N_MAX = 1 << 10, 12_800_000
TOTAL_MAX = 256_000_000


def listed():
    return [
        # one short block: launch latency, as in a link that distils key in
        # small frames or authenticates short messages
        {"name": "plain_4k", "form": "plain", "n": 4097, "m": 1025},
        # an ordinary odd-sized block below the finite-size regime
        {"name": "plain_100k", "form": "plain", "n": 100_003, "m": 25_001},
        # the small configuration of the benchmark
        {"name": "plain_262k", "form": "plain", "n": 262_144, "m": 65_536},
        # the benchmark's headline: a finite-size block of 10^6 bits
        {"name": "plain_1m", "form": "plain", "n": 1_000_000, "m": 250_000},
        # the benchmark's large block, high loss (ratio 0.1)
        {"name": "plain_12m8", "form": "plain", "n": 12_800_000, "m": 1_280_000},
        # the paper's own matrix (I, V), half the seed length
        {"name": "modified_1m", "form": "modified", "n": 1_000_000, "m": 250_000},
        # one seed kept for many keys: the seed's spectrum stays resident
        {"name": "plan_1m", "form": "plan", "n": 1_000_000, "m": 250_000},
        # a fixed set of short blocks replayed, as a steady link does
        {"name": "graph_32x100k", "form": "graph", "n": 100_000, "m": 20_000, "count": 32},
        # bulk distillation: 256 finite-size blocks, each with its own seed
        {"name": "batch_256x1m", "form": "batch", "n": 1_000_000, "m": 250_000, "count": 256},
        # the benchmark's uneven batch: blocks between 2^18 and 2^22 bits
        {"name": "batch_64_uneven", "form": "batch", "n_lo": 1 << 18, "n_hi": 1 << 22, "mix": 4, "count": 64},
        # one public seed for every key of a batch
        {"name": "shared_64x1m", "form": "shared", "n": 1_000_000, "m": 250_000, "count": 64},
        # a burst of requests at the serving loop, 10^5 to 10^7 bits
        {"name": "serve_48", "form": "serve", "n_lo": 100_000, "n_hi": 10_000_000, "mix": 5, "count": 48},
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _ratio(rng, n):
    return max(1, min(n - 1, int(round(n * rng.uniform(0.05, 0.5)))))


def draw(rng):
    """One more case: a form, n log-uniform (odd sizes included) and m/n
    uniform in [0.05, 0.5]; batches as large as TOTAL_MAX key bits."""
    form = rng.choice(["plain", "plain", "plain", "modified", "plan", "batch", "shared", "graph", "serve"])
    if form in ("plain", "modified", "plan"):
        n = _log_uniform(rng, N_MIN, N_MAX)
        return {"form": form, "n": n, "m": _ratio(rng, n)}
    if form == "serve":
        lo = _log_uniform(rng, 50_000, 300_000)
        return {"form": form, "n_lo": lo, "n_hi": lo * rng.randint(4, 32), "mix": rng.randrange(1 << 20),
                "count": rng.randint(8, 48)}
    n = _log_uniform(rng, 1 << 14, 4_000_000)
    count = _log_uniform(rng, 2, max(2, min(256, TOTAL_MAX // (2 * n))))
    if form == "batch" and rng.random() < 0.5:
        return {"form": form, "n_lo": n // 4, "n_hi": n, "mix": rng.randrange(1 << 20), "count": count}
    return {"form": form, "n": n, "m": _ratio(rng, n), "count": count}


def _shapes(case):
    """(n, m) of every block."""
    count = case.get("count", 1)
    if "n_lo" not in case:
        return [(case["n"], case["m"])] * count
    g = random.Random(case["mix"])
    shapes = []
    for _ in range(count):
        n = _log_uniform(g, case["n_lo"], case["n_hi"])
        m = _ratio(g, n)
        shapes.append((n, m))
    return shapes


def _seed_bits(case, n, m):
    return n - 1 if case["form"] == "modified" else n + m - 1


class _Serving:
    """A server with its registered seeds, closed with the state."""

    def __init__(self, seeds, bits):
        self.server = pa.Server(4 << 30, max_inflight=256)
        self.seed_ids = [self.server.register_seed(s, bits) for s in seeds]

    def __del__(self):
        self.server.close()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def bits(k):
        return torch.randint(-(1 << 63), (1 << 63) - 1, (pa.words(k),), dtype=torch.int64, device="cuda", generator=gen)

    form = case["form"]
    shapes = _shapes(case)
    # the outputs of a call lie one after the other in one buffer
    out = torch.zeros(sum(pa.words(m) for _, m in shapes), dtype=torch.int64, device="cuda")
    outs = list(out.split([pa.words(m) for _, m in shapes]))
    state = {"form": form, "out": out}
    keys = [bits(n) for n, _ in shapes]
    if form == "serve":
        longest = max(_seed_bits(case, n, m) for n, m in shapes)
        state["seeds"] = [bits(longest) for _ in range(4)]
        torch.cuda.synchronize()  # the server's streams are not ordered after torch's
        state["serving"] = _Serving(state["seeds"], longest)
        state["requests"] = [(state["serving"].seed_ids[i % 4], k, n, m, o)
                             for i, (k, (n, m), o) in enumerate(zip(keys, shapes, outs))]
        return state
    if form == "shared":
        one = bits(_seed_bits(case, *shapes[0]))
        seeds = [one] * len(shapes)
    else:
        seeds = [bits(_seed_bits(case, n, m)) for n, m in shapes]
    state["blocks"] = [(k, n, s, m, o) for k, (n, m), s, o in zip(keys, shapes, seeds, outs)]
    if form == "plan":
        n, m = shapes[0]
        state["plan"] = pa.Plan(seeds[0], n + m - 1, transform_len=pa.transform_len(n, m))
    elif form == "graph":
        state["graph"] = pa.BatchGraph(state["blocks"])
    return state


def run(state):
    form = state["form"]
    if form == "serve":
        server = state["serving"].server
        for request in state["requests"]:
            server.submit(*request)
        server.drain()
    elif form == "graph":
        state["graph"].launch()
    elif form in ("batch", "shared"):
        pa.toeplitz_hash_batched(state["blocks"])
    else:
        key, n, seed, m, out = state["blocks"][0]
        if form == "plain":
            pa.toeplitz_hash(key, n, seed, m, out)
        elif form == "modified":
            pa.modified_toeplitz_hash(key, n, seed, m, out)
        else:
            state["plan"].hash(key, n, m, out)
    return state["out"]


def work(case):
    """Bytes: every key, seed and output once.  Operations: a convolution of
    N = n + m - 1 bits through three transforms, one operation per bit and
    level (no transform is known to do with fewer)."""
    shapes = _shapes(case)
    form = case["form"]
    nbytes, flops, seeds = 0, 0.0, {}
    for i, (n, m) in enumerate(shapes):
        sb = _seed_bits(case, n, m)
        nbytes += (n + m) / 8
        key = 0 if form == "shared" else (i % 4 if form == "serve" else i)
        seeds[key] = max(seeds.get(key, 0), sb)
        flops += 3.0 * sb * math.log2(max(sb, 2))
    return {"bytes": nbytes + sum(seeds.values()) / 8, "flops": flops}
