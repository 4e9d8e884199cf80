"""Performance cases: the work a user of the library has it do, through its public entry points.

A case is a dict: "op" names the entry point, "gen" and "dtype" the generator and
the output type, the rest are sizes.

    generate   rng_generate           n_streams x n samples, states advanced
    split      rng_generate_split     one sequence of `total` samples over `threads`
    leapfrog   rng_generate_leapfrog  the same sequence, leapfrogged
    batch      rng_batch_set + rng_batch_launch   `requests` slices of uneven length
    pi         rng_fused_pi           every sample consumed in the kernel
    seed_skip  rng_seed + rng_skip    states of a job's share of the streams, moved to its part

listed() is the fixed list, draw() gives more of the same ranges, prepare() makes
what a program holds before the call, run() is one pass, work() the bytes and
integer operations it cannot do without, and exact() the outputs computed from
the recurrences in 64-bit integer arithmetic.
"""
import math

import numpy as np
import torch

import paper_1101_1846_amd as R
from paper_1101_1846_amd import workloads

GENS = ("MWC32", "XS256", "XS32", "KISS", "MWC1616")
DTYPES = ("u32", "f32")
WORDS = {"MWC32": 2, "XS256": 8, "XS32": 1, "KISS": 6, "MWC1616": 4}
# integer operations per number (shifts, logical operations, additions and multiplications of the recurrences)
OPS = {"MWC32": 3, "XS256": 18, "XS32": 6, "KISS": 20, "MWC1616": 10}
PI_OPS = 4  # per number: a shift, half of two squares, an addition and a comparison


def listed():
    return [
        # the smallest bulk call: a simulation step that draws 1024 numbers for each of 4096 walkers; latency counts
        {"name": "small", "op": "generate", "gen": "MWC32", "dtype": "u32", "n_streams": 4096, "n": 1024},
        # the bulk workload, integers: a pool of 2^20 streams x 256
        {"name": "bulk_xs256", "op": "generate", "gen": "XS256", "dtype": "u32", "n_streams": 1 << 20, "n": 256},
        # the bulk workload, uniforms, the generator with the largest arithmetic
        {"name": "bulk_kiss_f32", "op": "generate", "gen": "KISS", "dtype": "f32", "n_streams": 1 << 20, "n": 256},
        # round decimal sizes and a stream count that fills no last group: 1000 uniforms for each of 300007 histories
        {"name": "ragged_xs256_f32", "op": "generate", "gen": "XS256", "dtype": "f32", "n_streams": 300007, "n": 1000},
        # one stream, one long array: the plain "give me 10^8 uniforms" call
        {"name": "one_stream_kiss_f32", "op": "generate", "gen": "KISS", "dtype": "f32", "n_streams": 1, "n": 10 ** 8},
        # one reproducible sequence split over the device
        {"name": "split_xs256", "op": "split", "gen": "XS256", "dtype": "u32", "total": 1 << 30, "threads": 1 << 20},
        # the same with sizes that divide nothing evenly (1001 samples a thread, the last thread short)
        {"name": "split_ragged_f32", "op": "split", "gen": "MWC1616", "dtype": "f32", "total": 10 ** 8, "threads": 99991},
        # the other way to share one sequence
        {"name": "leapfrog_xs256", "op": "leapfrog", "gen": "XS256", "dtype": "u32", "total": 1 << 30,
         "threads": 1 << 20},
        # the batched workload: 10^4 requests of 2^8 to 2^22 samples over three generators and both types
        {"name": "batch_10k", "op": "batch", "requests": 10000, "lo": 8, "hi": 22, "wide": 0, "table": 4},
        # what a server launches under light load: a few requests, planned and launched at once; latency counts
        {"name": "batch_small", "op": "batch", "requests": 16, "lo": 10, "hi": 18, "wide": 0, "table": 4},
        # Monte Carlo inside the kernel: no number is stored
        {"name": "pi_kiss", "op": "pi", "gen": "KISS", "n_streams": 1 << 20, "n": 4096},
        # a job that takes its share of the streams and moves them to its part of the sequences
        {"name": "seed_skip_xs256", "op": "seed_skip", "gen": "XS256", "n_streams": 1 << 20, "skip": 274877907944},
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm; a third of them round ones."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    kind = rng.randrange(3)
    if kind == 0:  # a power of two
        return int(min(hi, max(lo, 2 ** round(math.log2(x)))))
    if kind == 1:  # two decimal digits
        e = 10 ** max(0, int(math.log10(x)) - 1)
        return int(min(hi, max(lo, round(x / e) * e)))
    return int(x)


def draw(rng):
    op = rng.choice(("generate", "generate", "generate", "split", "leapfrog", "batch", "pi", "seed_skip"))
    gen, dtype = rng.choice(GENS), rng.choice(DTYPES)
    if op == "generate":
        total = math.exp(rng.uniform(math.log(1 << 18), math.log(3 << 27)))
        streams = min(_log_int(rng, 1, 1 << 20), int(total) // 64)
        return {"op": op, "gen": gen, "dtype": dtype, "n_streams": streams, "n": _log_int(rng, 64, max(64, int(total / streams)))}
    if op in ("split", "leapfrog"):
        total = _log_int(rng, 1 << 20, 1 << 29)
        return {"op": op, "gen": gen, "dtype": dtype, "total": total,
                "threads": _log_int(rng, 1 << 10, min(1 << 20, total // 64))}
    if op == "batch":
        hi = rng.randint(14, 22)
        return {"op": op, "requests": _log_int(rng, 1, 4000), "lo": rng.randint(6, hi - 3), "hi": hi, "wide": rng.randrange(2),
                "table": rng.randrange(1 << 16)}
    if op == "pi":
        total = math.exp(rng.uniform(math.log(1 << 22), math.log(1 << 32)))
        streams = _log_int(rng, 1, 1 << 20)
        return {"op": op, "gen": gen, "n_streams": streams, "n": max(2, int(total / streams))}
    return {"op": op, "gen": gen, "n_streams": _log_int(rng, 1 << 10, 1 << 20), "skip": _log_int(rng, 1, 1 << 40)}


# ---------------------------------------------------------------- prepare and run
class Batch:
    """A batch handle that is destroyed with its owner."""

    def __init__(self, requests, samples):
        self.h = R.rng_batch_create(requests, samples)

    def __del__(self):
        R.rng_batch_destroy(self.h)


def _out(n, dtype):
    return torch.zeros(n, dtype=torch.float32 if dtype == "f32" else torch.int32, device="cuda")


def _seeded(gen, seed, n):
    st = torch.empty((WORDS[gen], n), dtype=torch.int32, device="cuda")
    R.rng_seed(R.GENERATORS[gen], seed, 0, n, st)
    return st


def _batch_table(case):
    gens = GENS if case["wide"] else workloads.BATCH_GENERATORS
    return workloads.batch_table(case["requests"], case["table"], gens, case["lo"], case["hi"])


def prepare(case, seed):
    R.rng_init()
    op = case["op"]
    s = {"case": dict(case), "op": op, "seed": seed}
    if op == "batch":
        t = _batch_table(case)
        offs, words = workloads.layout_outputs(t["length"])
        s["pools"] = [_seeded(g, seed + 1 + k, case["requests"]) for k, g in enumerate(t["generators"])]
        s["out"] = _out(words, "u32")
        reqs = []
        for i in range(case["requests"]):
            k = int(t["gen"][i])
            reqs.append((R.GENERATORS[t["generators"][k]], int(t["dtype"][i]), s["pools"][k].data_ptr() + 4 * i,
                         case["requests"], 0, int(t["length"][i]), s["out"].data_ptr() + 4 * int(offs[i])))
        s["reqs"] = R.make_requests(reqs)
        s["batch"] = Batch(case["requests"], int(t["length"].sum()))
        return s
    s["g"] = R.GENERATORS[case["gen"]]
    if op == "seed_skip":
        s["state"] = torch.zeros((WORDS[case["gen"]], case["n_streams"]), dtype=torch.int32, device="cuda")
        return s
    if op in ("split", "leapfrog"):
        s["t"] = R.DTYPES[case["dtype"]]
        s["state"] = _seeded(case["gen"], seed, 1)
        s["final"] = torch.zeros_like(s["state"])
        s["out"] = _out(case["total"], case["dtype"])
        size = R.rng_split_workspace_bytes if op == "split" else R.rng_leapfrog_workspace_bytes
        s["ws_bytes"] = size(s["g"], case["threads"])
        s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device="cuda")
        return s
    s["state"] = _seeded(case["gen"], seed, case["n_streams"])
    if op == "pi":
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    else:
        s["t"] = R.DTYPES[case["dtype"]]
        s["out"] = _out(case["n_streams"] * case["n"], case["dtype"])
    return s


def run(s):
    c, op = s["case"], s["op"]
    if op == "generate":
        R.rng_generate(s["g"], s["state"], c["n_streams"], c["n"], s["t"], s["out"])
        return {"out": s["out"], "state": s["state"]}
    if op in ("split", "leapfrog"):
        f = R.rng_generate_split if op == "split" else R.rng_generate_leapfrog
        f(s["g"], s["state"], c["total"], c["threads"], s["t"], s["out"], s["final"], s["ws"], s["ws_bytes"])
        return {"out": s["out"], "final": s["final"]}
    if op == "batch":
        R.rng_batch_set(s["batch"].h, s["reqs"])
        R.rng_batch_launch(s["batch"].h)
        return {"out": s["out"], "pools": s["pools"]}
    if op == "pi":
        s["count"].zero_()
        R.rng_fused_pi(s["g"], s["state"], c["n_streams"], c["n"], s["count"])
        return {"count": s["count"], "state": s["state"]}
    R.rng_seed(s["g"], s["seed"], 0, c["n_streams"], s["state"])
    R.rng_skip(s["g"], s["state"], c["n_streams"], c["skip"])
    return {"state": s["state"]}


def work(case):
    op = case["op"]
    if op == "batch":
        t = _batch_table(case)
        w = [WORDS[t["generators"][k]] for k in t["gen"]]
        ops = [OPS[t["generators"][k]] for k in t["gen"]]
        return {"bytes": 4 * int(t["length"].sum()) + 8 * sum(w), "flops": int(np.dot(t["length"], ops))}
    w, ops = WORDS[case["gen"]], OPS[case["gen"]]
    if op in ("split", "leapfrog"):
        return {"bytes": 4 * case["total"] + 8 * w, "flops": ops * case["total"]}
    if op == "seed_skip":
        return {"bytes": 4 * w * case["n_streams"], "flops": ops * case["n_streams"]}
    total = case["n_streams"] * case["n"]
    if op == "pi":
        return {"bytes": 8 * w * case["n_streams"] + 8, "flops": (ops + PI_OPS) * total}
    return {"bytes": 4 * total + 8 * w * case["n_streams"], "flops": ops * total}


# ---------------------------------------------------------------- exact
# The recurrences on int64 tensors that hold 32-bit values: many streams at
# once, one step at a time; far starts by the k-th power of the step.
M32 = 0xFFFFFFFF
MWC32_A = 65274
MWC32_M = MWC32_A * 2 ** 32 - 1


def _multipliers():
    """The a < 2^16 with a 2^16 - 1 and a 2^15 - 1 prime, ascending."""
    sieve = np.ones(1 << 16, dtype=bool)
    sieve[:2] = False
    for p in range(2, 256):
        if sieve[p]:
            sieve[p * p::p] = False
    a = np.arange(2, 1 << 16, dtype=np.int64)
    m, h = a * 65536 - 1, a * 32768 - 1
    for p in np.flatnonzero(sieve):
        keep = ((m % p != 0) | (m == p)) & ((h % p != 0) | (h == p))
        a, m, h = a[keep], m[keep], h[keep]
    return a


def _shr(x, k):
    """Logical right shift of int64 bit patterns."""
    return (x >> k) & ((1 << (64 - k)) - 1)


def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _draws(seed, n, per, device):
    """SplitMix64 outputs 0 .. n * per - 1 as (low, high) 32-bit halves, [per][n]."""
    i = torch.arange(1, n * per + 1, dtype=torch.int64, device=device)
    z = i * _signed(0x9E3779B97F4A7C15) + _signed(seed % (1 << 64))
    z = (z ^ _shr(z, 30)) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _signed(0x94D049BB133111EB)
    z = (z ^ _shr(z, 31)).reshape(n, per).T
    return z & M32, _shr(z, 32)


def _exact_seed(gen, seed, n, device):
    """State words [words][n] of streams 0 .. n - 1."""
    per = {"MWC32": 1, "XS32": 1, "MWC1616": 2, "KISS": 3, "XS256": 4}[gen]
    lo, hi = _draws(seed, n, per, device)
    if gen == "MWC32":
        z = hi[0] % MWC32_A * 2 ** 32 + lo[0]
        z = torch.where(z == 0, 1, z)
        z = torch.where(z == MWC32_M, MWC32_M - 1, z)
        return torch.stack([z & M32, z >> 32])
    if gen == "XS32":
        return torch.where(lo == 0, 1, lo)
    if gen == "XS256":
        v = torch.stack([lo, hi], 1).reshape(8, n)
        v[7] = torch.where((v == 0).all(0), 1, v[7])
        return v
    t = torch.from_numpy(_multipliers()).to(device)
    i = lo[0] % len(t)
    j = (i + 1 + hi[0] % (len(t) - 1)) % len(t)
    words = []
    for a, h in ((t[i], lo[1]), (t[j], hi[1])):
        z = ((h >> 16) % a) * 65536 + (h & 0xFFFF)
        z = torch.where(z == 0, 1, z)
        m = a * 65536 - 1
        words.append((torch.where(z == m, m - 1, z), a))
    if gen == "MWC1616":
        return torch.stack([words[0][0], words[1][0], words[0][1], words[1][1]])
    return torch.stack([words[0][0], words[1][0], torch.where(lo[2] == 0, 1, lo[2]), hi[2], words[0][1], words[1][1]])


def _xs32(y):
    y = y ^ (y << 13) & M32
    y = y ^ (y >> 17)
    return y ^ (y << 5) & M32


def _step(gen, st):
    """One step of every stream: (the new words as a list, the output)."""
    if gen == "MWC32":
        t = MWC32_A * st[0] + st[1]
        return [t & M32, t >> 32], t & M32
    if gen == "XS32":
        y = _xs32(st[0])
        return [y], y
    if gen == "XS256":
        v0, v1, v3, v4, v7 = st[0], st[1], st[3], st[4], st[7]
        u = v7 ^ (v7 << 13)
        w = v0 ^ (v0 >> 7)
        n = (u ^ (u << 9) ^ v4 ^ (v4 << 7) ^ v3 ^ (v3 >> 3) ^ v1 ^ (v1 >> 10) ^ w ^ (w << 24)) & M32
        return list(st[1:]) + [n], n
    z = st[-2] * (st[0] & 0xFFFF) + (st[0] >> 16)
    w = st[-1] * (st[1] & 0xFFFF) + (st[1] >> 16)
    u = ((z << 16) + w) & M32
    if gen == "MWC1616":
        return [z, w, st[2], st[3]], u
    c = (69069 * st[3] + 1234567) & M32
    y = _xs32(st[2])
    return [z, w, y, c, st[4], st[5]], ((u ^ c) + y) & M32


def _mulmod(z, k, m, limb):
    """z k mod m by limbs of k (z < 2^(63 - limb))."""
    r = torch.zeros_like(z)
    for i in reversed(range(0, 48, limb)):
        r = (r * (1 << limb) + z * ((k >> i) & ((1 << limb) - 1))) % m
    return r


def _powmod(a, k, m):
    """a^k mod m of int64 tensors, m < 2^32."""
    r, b = torch.ones_like(a), a
    while k:
        if k & 1:
            r = _mulmod(r, b, m, 16)
        b = _mulmod(b, b, m, 16)
        k >>= 1
    return r


def _bits(words):
    """[n] words of 32 bits each as rows of bits, [32 n][streams]."""
    return torch.cat([(w >> torch.arange(32, device=w.device)[:, None]) & 1 for w in words])


def _unbits(b):
    return [sum(b[32 * i + j].to(torch.int64) << j for j in range(32)) for i in range(len(b) // 32)]


def _gf2_power(gen, k, device):
    """The k-th power of a xorshift step as a matrix of bits."""
    n = 256 if gen == "XS256" else 32
    unit = _unbits(torch.eye(n, dtype=torch.int64, device=device))
    b = _bits(_step(gen, unit)[0]).double()
    r = torch.eye(n, dtype=torch.float64, device=device)
    while k:
        if k & 1:
            r = (b @ r) % 2
        b = (b @ b) % 2
        k >>= 1
    return r


def _jump(gen, st, k):
    """Every stream of st moved k steps on."""
    dev = st[0].device
    if gen in ("XS32", "XS256"):
        return _unbits((_gf2_power(gen, k, dev) @ _bits(st).double()) % 2)
    if gen == "MWC32":
        z = _mulmod(st[1] * 2 ** 32 + st[0], pow(MWC32_A, k, MWC32_M), MWC32_M, 14)
        return [z & M32, z >> 32]
    st = list(st)
    for i in (0, 1):
        a = st[i - 2]
        st[i] = _mulmod(st[i], _powmod(a, k, a * 65536 - 1), a * 65536 - 1, 16)
    if gen == "KISS":
        st[2] = _jump("XS32", [st[2]], k)[0]
        a, c, pa, pc = 1, 0, 69069, 1234567
        while k:
            if k & 1:
                a, c = pa * a & M32, (pa * c + pc) & M32
            pa, pc = pa * pa & M32, (pa * pc + pc) & M32
            k >>= 1
        st[3] = (a * st[3] + c) & M32
    return st


def _numbers(gen, st, n):
    """n numbers of every stream, [streams][n], and the words after them."""
    st = list(st)
    out = torch.empty((n, len(st[0])), dtype=torch.int64, device=st[0].device)
    for k in range(n):
        st, out[k] = _step(gen, st)
    return out.T, st


def _sequence(gen, st, total):
    """`total` numbers of one stream ([words][1]) and the words after them: starts by doubling, then all at once."""
    rows = 1 << max(0, min(20, total.bit_length() // 2 + 3))
    per = -(-total // rows)
    starts, k = list(st), per
    while len(starts[0]) < rows:
        starts = [torch.cat(w) for w in zip(starts, _jump(gen, starts, k * len(starts[0])))]
    out = torch.empty(rows * per, dtype=torch.int32, device=starts[0].device).view(rows, per)
    w, end = starts, None
    last, left = (total - 1) // per, total - (total - 1) // per * per
    for i in range(per):
        w, u = _step(gen, w)
        out[:, i] = _int32(u)
        if i + 1 == left:
            end = [x[last:last + 1].clone() for x in w]
    return out.view(-1)[:total], end


def _int32(x):
    return torch.where(x >= 1 << 31, x - (1 << 32), x).to(torch.int32)


def _typed(x, dtype):
    """Outputs of their type from 32-bit values: int32 bit patterns, or (u >> 8) 2^-24 in 64 bits."""
    if dtype == "u32":
        return x if x.dtype == torch.int32 else _int32(x)
    if x.dtype == torch.int32:
        return ((x >> 8) & 0xFFFFFF).double() * 2.0 ** -24
    return (x >> 8).double() * 2.0 ** -24


def _state(st):
    return _int32(torch.stack(list(st)))


def exact(case, seed):
    dev, op = "cuda" if torch.cuda.is_available() else "cpu", case["op"]
    if op == "batch":
        if case["requests"] > 32:
            return None  # minutes: every request has its own start states
        t = _batch_table(case)
        offs, words = workloads.layout_outputs(t["length"])
        pools = [_exact_seed(g, seed + 1 + k, case["requests"], dev) for k, g in enumerate(t["generators"])]
        out = torch.zeros(words, dtype=torch.int32, device=dev)
        for i in range(case["requests"]):
            k, n = int(t["gen"][i]), int(t["length"][i])
            u, end = _sequence(t["generators"][k], [w[i:i + 1] for w in pools[k]], n)
            if int(t["dtype"][i]):
                u = _typed(u, "f32").float().view(torch.int32)
            out[int(offs[i]):int(offs[i]) + n] = u
            pools[k][:, i] = torch.cat(end)
        return {"out": out, "pools": [_int32(p) for p in pools]}
    gen = case["gen"]
    if op in ("split", "leapfrog"):
        u, end = _sequence(gen, _exact_seed(gen, seed, 1, dev), case["total"])
        return {"out": _typed(u, case["dtype"]), "final": _state(end)}
    st = _exact_seed(gen, seed, case["n_streams"], dev)
    if op == "seed_skip":
        return {"state": _state(_jump(gen, st, case["skip"]))}
    streams, n = case["n_streams"], case["n"]
    if n > 1 << 16:  # few long streams
        if streams > 16 or op == "pi":
            return None
        rows, ends = zip(*(_sequence(gen, [w[i:i + 1] for w in st], n) for i in range(streams)))
        return {"out": _typed(torch.cat(rows), case["dtype"]),
                "state": _state([torch.cat([e[k] for e in ends]) for k in range(len(ends[0]))])}
    if op == "pi":
        count, st = torch.zeros(1, dtype=torch.int64, device=dev), list(st)
        for _ in range(n // 2):
            st, x = _step(gen, st)
            st, y = _step(gen, st)
            count += ((x >> 8) ** 2 + (y >> 8) ** 2 < 1 << 48).sum()
        if n % 2:
            st, _ = _step(gen, st)
        return {"count": count, "state": _state(st)}
    u, st = _numbers(gen, st, n)
    return {"out": _typed(u.reshape(-1), case["dtype"]), "state": _state(st)}
