"""The work that a training program has the rehearsal buffer do, as measurable cases.

A case is one way of calling the buffer (`call`) at one shape:

  two_calls   rb_update, then rb_sample_augment: the mini-batch goes in, representatives come out
  step        rb_update_sample: the same as one call, what a training loop without a prefetching loader makes
  announced   rb_announce_next + rb_update_sample: the loader holds the next mini-batch's labels already
  many        rb_announce_next_many + rb_update_sample_many: the loader is `n` mini-batches ahead
  pipeline    rb_announce_next_many + Pipeline.step_many + Pipeline.drain: the same on a stream of its own, under training

Buffers are in the state of a training run that has been going for a while: every second class is full, the others
half full, so that candidates both append and replace.  Mini-batches come from a ring of resident ones.  Results are the
representatives with their labels, and the buffer's own contents afterwards.
"""
import math

import torch

import paper_2406_03285_amd as rb

RING = 8                      # resident mini-batches
FILL_BYTES = 256 << 20        # most bytes of the block of rows the buffer is filled from before the first pass
FILL_ROWS = 4096
LIB_SEED = 0x5EED0BADC0FFEE

POLICIES = {
    "uniform": (rb.RB_SELECT_EXACT, rb.RB_EVICT_UNIFORM),
    "fifo": (rb.RB_SELECT_EXACT, rb.RB_EVICT_FIFO),
    "reservoir": (rb.RB_SELECT_EXACT, rb.RB_EVICT_RESERVOIR),
    "bernoulli": (rb.RB_SELECT_BERNOULLI, rb.RB_EVICT_UNIFORM),
    "bernoulli_reservoir": (rb.RB_SELECT_BERNOULLI, rb.RB_EVICT_RESERVOIR),
}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "u8": torch.uint8}


def _case(name, call, K, S, elems, dtype, b, c, r, n=1, store=None, policy="uniform", labels="uniform"):
    return {"name": name, "call": call, "K": K, "S": S, "elems": elems, "dtype": dtype, "store": store or dtype,
            "b": b, "c": c, "r": r, "n": n, "policy": policy, "labels": labels}


def listed():
    return [
        # a toy run on 3x32x32 images: nothing but latency and launches
        _case("tiny_two_calls", "two_calls", 10, 20, 3072, "f32", 16, 4, 4),
        # 100 classes of 3x32x32 images, the README's minimal use
        _case("small_images_step", "step", 100, 500, 3072, "f32", 128, 16, 16),
        # the method's own setting (b, c, r = 56, 14, 7; 1000 classes of 3x224x224), one call per iteration
        _case("imagenet_step", "step", 1000, 8, 150528, "f32", 56, 14, 7),
        # the same images in groups of 32 iterations on the buffer's own stream, under the training computation
        _case("imagenet_pipeline", "pipeline", 1000, 8, 150528, "f32", 64, 8, 8, n=32),
        # bfloat16 images, large mini-batches, skewed labels: in two calls, in one, with the next labels known, 20 steps at once
        _case("large_two_calls", "two_calls", 1000, 32, 150528, "bf16", 512, 64, 64, labels="zipf"),
        _case("large_step", "step", 1000, 32, 150528, "bf16", 512, 64, 64, labels="zipf"),
        _case("large_announced", "announced", 1000, 32, 150528, "bf16", 512, 64, 64, labels="zipf"),
        _case("large_many", "many", 1000, 32, 150528, "bf16", 512, 64, 64, n=20, labels="zipf"),
        # latent replay of 2048 features, 10000 classes of which 50 occur in a step: large counts of short rows
        _case("features_step", "step", 10000, 100, 2048, "f32", 4096, 1024, 1024, labels="active50"),
        _case("features_many", "many", 10000, 100, 2048, "f32", 4096, 1024, 1024, n=16, labels="active50"),
        # 3x224x224 images kept in 8 bits per element
        _case("imagenet_u8_step", "step", 1000, 32, 150528, "f32", 64, 8, 8, store="u8"),
        # 200 classes of 3x64x64 images kept as bfloat16, a coin per sample, reservoir replacement, ragged counts
        _case("mid_images_variant_step", "step", 200, 250, 12288, "f32", 250, 90, 75, store="bf16", policy="bernoulli_reservoir"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["two_calls", "step", "step", "announced", "many", "pipeline"])
    dtype, store = rng.choice([("f32", "f32"), ("f32", "f32"), ("bf16", "bf16"), ("f32", "bf16"), ("f32", "u8")])
    K = _log_int(rng, 10, 10000)
    elems = 16 * _log_int(rng, 16, 9408)                       # 256 ... 150528 elements
    size = 4 if dtype == "f32" else 2
    b = _log_int(rng, 16, min(4096, max(32, (160 << 20) // (elems * size))))
    # at most what the largest listed single step moves: 64 + 64 rows of 3x224x224 in bfloat16
    most = max(1, min(1024, b, (20 << 20) // (elems * size)))
    c = _log_int(rng, min(4, most), most)
    r = max(1, min(most, round(c * 2 ** rng.uniform(-2, 2))))
    S = max(2, min(_log_int(rng, 8, 500), (4 << 30) // (K * elems * DTYPES[store].itemsize)))
    return {"call": call, "K": K, "S": S, "elems": elems, "dtype": dtype, "store": store, "b": b, "c": c, "r": r,
            "n": rng.randint(2, 20) if call in ("many", "pipeline") else 1, "policy": rng.choice(list(POLICIES)),
            "labels": rng.choice(["uniform", "zipf", "active50"])}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _make_labels(case, count, g):
    K, b = case["K"], case["b"]
    if case["labels"] == "uniform":
        return torch.randint(0, K, (count, b), generator=g, device="cuda")
    if case["labels"] == "zipf":                               # P(k) ~ (k + 1)^-1.1
        p = torch.arange(1, K + 1, device="cuda", dtype=torch.float64) ** -1.1
        u = torch.rand((count, b), generator=g, device="cuda", dtype=torch.float64) * p.sum()
        return torch.searchsorted(p.cumsum(0), u).clamp_(max=K - 1)
    active = torch.stack([torch.randperm(K, generator=g, device="cuda")[:50] for _ in range(count)])   # 50 classes per step
    return active.gather(1, torch.randint(0, active.shape[1], (count, b), generator=g, device="cuda"))


def _inputs(case, seed):
    """Ring of mini-batches, and the rows and labels the buffer is filled from."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1_000_003 + 17)
    dtype, K, S, elems = DTYPES[case["dtype"]], case["K"], case["S"], case["elems"]
    x = torch.rand((RING, case["b"], elems), generator=g, device="cuda", dtype=dtype)        # image values lie in [0, 1)
    y = _make_labels(case, RING, g)
    held = torch.tensor([S if k % 2 == 0 else S // 2 for k in range(K)], device="cuda")
    fill_y = torch.repeat_interleave(torch.arange(K, device="cuda"), held)
    fill_y = fill_y[torch.randperm(fill_y.numel(), generator=g, device="cuda")].contiguous()
    rows = max(1, min(FILL_ROWS, fill_y.numel(), FILL_BYTES // (elems * x.element_size())))
    fill_x = torch.rand((rows, elems), generator=g, device="cuda", dtype=dtype)
    return x, y, fill_x, fill_y


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case, s.call = case, case["call"]
    b, c, r, n, elems = case["b"], case["c"], case["r"], case["n"], case["elems"]
    dtype = DTYPES[case["dtype"]]
    s.x, s.y, fill_x, fill_y = _inputs(case, seed)
    s.stream = torch.cuda.Stream() if s.call == "pipeline" else None
    s.buf = rb.RehearsalBuffer(case["K"], case["S"], (elems,), dtype=dtype, store_dtype=DTYPES[case["store"]])
    s.buf.set_policy(*POLICIES[case["policy"]])
    s.buf.buf_x.zero_()
    s.t = 0
    for at in range(0, fill_y.numel(), fill_x.shape[0]):       # everything of a chunk goes in: c = b
        m = min(fill_x.shape[0], fill_y.numel() - at)
        s.buf.update(fill_x[:m], fill_y[at:at + m], m, LIB_SEED, s.t)
        s.t += 1
    # two sets of results: one is being written while the other is in use
    s.out_x = torch.zeros((2, n, r, elems), dtype=dtype, device="cuda")
    s.out_y = torch.full((2, n, r), -1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    if s.stream is not None:
        s.buf.set_stream(s.stream)
        s.pipe = rb.Pipeline(s.buf)
    s.results = [{"reps": s.out_x[q], "labels": s.out_y[q], "stored": s.buf.buf_x, "stored_labels": s.buf.buf_y} for q in range(2)]
    s.first = s.t
    s.bx, s.by = list(s.x), list(s.y)
    s.px, s.py = [x.data_ptr() for x in s.bx], [y.data_ptr() for y in s.by]
    s.ox = [[s.out_x[q, i].data_ptr() for i in range(n)] for q in range(2)]
    s.oy = [[s.out_y[q, i].data_ptr() for i in range(n)] for q in range(2)]
    s.passes = 0
    return s


def _ok(rc):
    if rc != rb.RB_OK:
        raise rb.RbError(rc, "rb")


def run(s):
    case, h = s.case, s.buf.handle
    b, c, r, n = case["b"], case["c"], case["r"], case["n"]
    at, q, t = s.t - s.first, s.passes & 1, s.t
    i = at % RING
    if s.call == "two_calls":
        _ok(rb.rb_update(h, s.px[i], s.py[i], b, c, LIB_SEED, t))
        _ok(rb.rb_sample_augment(h, r, LIB_SEED, t, s.ox[q][0], s.oy[q][0]))
    elif s.call == "step":
        _ok(rb.rb_update_sample(h, s.px[i], s.py[i], b, c, r, LIB_SEED, t, s.ox[q][0], s.oy[q][0]))
    elif s.call == "announced":
        _ok(rb.rb_announce_next(h, s.py[(i + 1) % RING]))
        _ok(rb.rb_update_sample(h, s.px[i], s.py[i], b, c, r, LIB_SEED, t, s.ox[q][0], s.oy[q][0]))
    else:
        now = [(at + k) % RING for k in range(n)]
        _ok(rb.rb_announce_next_many(h, n, [s.py[(at + n + k) % RING] for k in range(n)]))
        px, py = [s.px[k] for k in now], [s.py[k] for k in now]
        if s.call == "many":
            _ok(rb.rb_update_sample_many(h, n, px, py, b, c, r, LIB_SEED, t, s.ox[q], s.oy[q]))
        else:
            train = torch.cuda.current_stream()
            s.pipe.step_many([s.bx[k] for k in now], [s.by[k] for k in now], c, r, LIB_SEED, t, s.ox[q], s.oy[q], train)
            s.pipe.drain(train)
    s.t += n
    s.passes += 1
    return s.results[q]


def _row_bytes(case):
    return case["elems"] * DTYPES[case["dtype"]].itemsize, case["elems"] * DTYPES[case["store"]].itemsize


def work(case):
    """A candidate row is read from the mini-batch and stored, a representative read from the buffer and handed out; labels."""
    sample, stored = _row_bytes(case)
    return {"bytes": case["n"] * ((case["c"] + case["r"]) * (sample + stored) + 8 * (case["b"] + case["c"] + 2 * case["r"])), "flops": 0}


def tolerance(case):
    """Rows are moved, or converted by a rounding that is defined bit for bit."""
    return "exact"


# ---------------------------------------------------------------------------
# The method once more, sequentially and in plain Python, where rows are converted on the way (elsewhere the results are
# the very bytes that went in, and there is nothing to compute).
# ---------------------------------------------------------------------------
def _below(step, purpose, index, n):
    """Philox4x32-10, counter (index, purpose, step), key LIB_SEED; the high half of draw * n."""
    M = 0xFFFFFFFF
    x = [index, purpose, step & M, step >> 32]
    ka, kb = LIB_SEED & M, LIB_SEED >> 32
    for _ in range(10):
        pa, pb = 0xD2511F53 * x[0], 0xCD9E8D57 * x[2]
        x = [(pb >> 32) ^ x[1] ^ ka, pb & M, (pa >> 32) ^ x[3] ^ kb, pa & M]
        ka, kb = (ka + 0x9E3779B9) & M, (kb + 0xBB67AE85) & M
    return ((x[0] | x[1] << 32) * n) >> 64


def _floyd(step, purpose, m, n):
    got = {}
    for i in range(m):
        t = _below(step, purpose, i, n - m + i + 1)
        got[n - m + i if t in got else t] = i
    return list(got)


def exact(case, seed):
    if case["store"] == case["dtype"]:
        return None
    K, S, b, c, r, n = (case[k] for k in ("K", "S", "b", "c", "r", "n"))
    selection, eviction = POLICIES[case["policy"]]
    x, y, fill_x, fill_y = _inputs(case, seed)
    rows, labels = fill_x.shape[0], y.tolist()
    # slots[k][s]: number of the row held, in the ring's rows followed by the filling block's
    slots, offered, oldest = [[] for _ in range(K)], [0] * K, [0] * K
    for at, k in enumerate(fill_y.tolist()):
        slots[k].append(RING * b + at % rows)
        offered[k] += 1
    step = -(-fill_y.numel() // rows)
    reps, rep_labels = [], []
    for i in range(n):
        t = step + i
        if selection == rb.RB_SELECT_BERNOULLI:
            chosen = [p for p in range(b) if _below(t, 4, p, b) < c]
        else:
            chosen = sorted(_floyd(t, 1, c, b))
        for p in chosen:
            k = labels[i % RING][p]
            row, room = i % RING * b + p, slots[k]
            if len(room) < S:
                room.append(row)
            elif eviction == rb.RB_EVICT_FIFO:
                room[oldest[k]] = row
                oldest[k] = (oldest[k] + 1) % S
            else:
                at = _below(t, 2, p, offered[k] + 1 if eviction == rb.RB_EVICT_RESERVOIR else S)
                if at < S:
                    room[at] = row
            offered[k] += 1
        held = [(k, row) for k in range(K) for row in slots[k]]
        picked = [held[g] for g in _floyd(t, 3, min(r, len(held)), len(held))]
        reps.append([row for _, row in picked] + [-1] * (r - len(picked)))
        rep_labels.append([k for k, _ in picked] + [-1] * (r - len(picked)))
    every = torch.cat([x.reshape(RING * b, -1), fill_x])

    def gathered(ids, dtype, handed_out):
        """The rows `ids` as they are stored or handed out; an id of -1 is a row that was never written: zeros."""
        out = torch.zeros((len(ids), case["elems"]), dtype=dtype, device="cuda")
        for lo in range(0, len(ids), 1024):
            part = torch.tensor(ids[lo:lo + 1024], device="cuda")
            v = every[part.clamp(min=0)]
            if case["store"] == "bf16":
                v = v.to(torch.bfloat16).double()
            else:
                v = (v.double() * 255).round().clamp_(0, 255)
                v = v / 255 if handed_out else v
            out[lo:lo + 1024] = (v * (part >= 0)[:, None]).to(dtype)
        return out

    flat = [row for k in range(K) for row in slots[k] + [-1] * (S - len(slots[k]))]
    stored_labels = [k if at < len(slots[k]) else -1 for k in range(K) for at in range(S)]
    return {"reps": gathered([row for step_rows in reps for row in step_rows], torch.float64, True).reshape(n, r, -1),
            "labels": torch.tensor(rep_labels, device="cuda"),
            "stored": gathered(flat, torch.float64, False).reshape(K, S, -1) if case["store"] == "bf16" else None,
            "stored_labels": torch.tensor(stored_labels, device="cuda").reshape(K, S)}
