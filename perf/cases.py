"""The calls whose speed matters to a program that decodes with this package.

A case is a dict of plain values: the kind of call, the shape of the embedding matrix, the hash
hyper-parameters and the shape of the step.  Kinds:

  step      one decode step on the LSH candidate list, launched from the host;
  full      the same step with the candidate list forced to all of V (the plain softmax that the
            LSH step is compared with, and what a program runs where it wants no approximation);
  sentence  a whole sentence: `steps` decode steps chained through their scores, each followed by
            the beam bookkeeping (history, reorder of the four state arrays of a 2-layer LSTM), and
            the backtrace at the end.  With graph = True the steps are replayed as one HIP graph;
  build     tables over an embedding matrix that has changed, and the first step on them.

Inputs are drawn on the device: words scattered around cluster centres, so that bucket sizes are
skewed as those of trained embeddings are; hidden rows near the embedding of a Zipf-distributed
word, scaled so that the softmax is as peaked as a trained model's; a share `off` of the hidden rows
near no word at all.  The most frequent words are the lowest ids.
"""
import math

import torch

from paper_1806_00588_amd import binding

ZIPF_S = 1.1
H_SCALE = 16.0      # logits of the best words 10 to 15 above the bulk
CLUSTER = 40        # words per cluster
EOS = 2


def _case(name, kind, d, V, S, B, K=8, P=32, W=8, T=1000, t=1, bf16=False, off=0.0, steps=1, graph=False):
    return {"name": name, "kind": kind, "d": d, "V": V, "S": S, "B": B, "K": K, "P": P, "W": W, "T": T, "t": t,
            "bf16": bf16, "off": off, "steps": steps, "graph": graph}


def listed():
    return [
        # the smallest model anybody decodes with: nothing but latency, launches and host work
        _case("tiny step", "step", 64, 1000, 1, 4, P=16, W=4, T=50),
        # one sentence at a time, beam 12, launched from a decoder's host loop
        _case("one sentence, a step", "step", 1000, 40000, 1, 12),
        # the same model decoding a whole sentence, the loop captured once and replayed
        _case("one sentence, replayed", "sentence", 1000, 40000, 1, 12, steps=16, graph=True),
        # a server's small batch, beam 5, bf16 embeddings, every call launched from the host
        _case("small batch, launched", "sentence", 1024, 40000, 8, 5, bf16=True, steps=8),
        # batched translation
        _case("batch of 32, a step", "step", 1000, 40000, 32, 10),
        # wide beams: a search for many different outputs
        _case("wide beam, a step", "step", 1000, 100000, 4, 50, K=16, P=48, W=12, T=2000),
        # a large vocabulary in bf16 with a large batch
        _case("large vocabulary, a step", "step", 1024, 200000, 64, 10, P=64, W=16, T=2000, bf16=True, off=0.1),
        # fine banding with a hit threshold (many short codes, a word counts when it collides often)
        _case("500 bands, a step", "step", 1000, 40000, 1, 12, P=1500, W=500, t=5),
        # sizes that are multiples of nothing
        _case("odd sizes, a step", "step", 1001, 39989, 5, 17, P=28, W=7, T=777, off=0.1),
        # the exact softmax, for one sentence and for a batch
        _case("all words, one sentence", "full", 1000, 40000, 1, 12),
        _case("all words, batch of 32", "full", 1000, 40000, 32, 10),
        # the index rebuilt after the embeddings have changed
        _case("tables and first step", "build", 1000, 40000, 1, 12),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 5e12, w["flops"] / 1e14)


def draw(rng):
    limit = max(_cost(c) for c in listed())
    kind = rng.choice(["step"] * 6 + ["full"] * 2 + ["sentence"] * 2 + ["build"])
    while True:
        # three hidden sizes in four are multiples of 8, as models have them
        d = _log_int(rng, 64, 1536)
        if rng.random() < 0.75:
            d = (d + 7) // 8 * 8
        V = _log_int(rng, 1000, 200000)
        S, B = _log_int(rng, 1, 64), _log_int(rng, 1, 64)
        T = min(V, _log_int(rng, 50, 2000))
        bf16 = rng.random() < 0.35
        off = rng.choice([0.0, 0.0, 0.1])
        if kind == "step" and rng.random() < 0.2:       # the threshold on fine bands
            W, K, u, t = rng.randint(100, 500), 8, 3, rng.randint(3, 8)
            V, S = min(V, 100000), min(S, 4)
        else:
            W, K, u, t = rng.randint(4, 16), rng.choice([8, 8, 16]), 4, 1
        c = _case(None, kind, d, V, S, B, K, u * W, W, T, t, bf16, off,
                  rng.randint(4, 24) if kind == "sentence" else 1, kind == "sentence" and rng.random() < 0.5)
        del c["name"]
        if _cost(c) <= limit:
            return c


# ---- inputs -----------------------------------------------------------------------------------

def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(seed * 16 + stream)


def _embeddings(c, seed):
    g = _generator(seed, 1)
    V, d = c["V"], c["d"]
    n = max(8, V // CLUSTER)
    sd = 1.0 / math.sqrt(d)
    centres = torch.randn(n, d, device="cuda", generator=g) * sd
    E = torch.randn(V, d, device="cuda", generator=g).mul_(0.3 * sd)
    E += centres[torch.arange(V, device="cuda") % n]
    return E.bfloat16() if c["bf16"] else E


def _permutations(c, seed):
    g = _generator(seed, 2)
    return torch.rand(c["P"], c["d"], device="cuda", generator=g).topk(c["K"], dim=1).indices.int().contiguous()


def _hidden(c, E, seed, steps):
    g = _generator(seed, 3)
    V, d, n = c["V"], c["d"], steps * c["S"] * c["B"]
    rank = torch.arange(1, V + 1, device="cuda", dtype=torch.float64) ** -ZIPF_S
    cdf = rank.cumsum(0)
    u = torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * cdf[-1]
    w = torch.searchsorted(cdf, u).clamp_(max=V - 1)
    sd = 1.0 / math.sqrt(d)
    H = E[w].float() * 0.8 + torch.randn(n, d, device="cuda", generator=g) * (0.3 * sd)
    if c["off"] > 0:
        far = torch.rand(n, device="cuda", generator=g) < c["off"]
        H[far] = (torch.rand(int(far.sum()), d, device="cuda", generator=g) * 2 - 1) * (math.sqrt(3.0) * sd)
    return (H * H_SCALE).view(steps, c["S"] * c["B"], d).contiguous()


def _beam_scores(c, seed):
    """Accumulated log-probabilities some steps into a sentence: best first, a few tenths apart."""
    g = _generator(seed, 4)
    gaps = torch.rand(c["S"], c["B"], device="cuda", generator=g) * (6.0 / c["B"])
    return (-8.0 - gaps.cumsum(1)).reshape(-1).contiguous()


def prepare(case, seed):
    c = case
    R = c["S"] * c["B"]
    st = {"case": c, "E": _embeddings(c, seed), "perms": _permutations(c, seed), "seed": seed & 0xFFFF,
          "topfreq": torch.arange(c["T"], dtype=torch.int32, device="cuda"),
          "sp": binding.step_params(c["S"], c["B"], c["T"], c["t"], c["kind"] == "full")}
    st["H"] = _hidden(c, st["E"], seed, c["steps"])
    st["scores_in"] = _beam_scores(c, seed)
    st["beam"] = torch.empty(R, dtype=torch.int32, device="cuda")
    st["word"] = torch.empty(R, dtype=torch.int32, device="cuda")
    st["score"] = torch.empty(R, dtype=torch.float32, device="cuda")
    st["tables"] = None
    if c["kind"] == "build":
        return st
    st["tables"] = binding.build_tables(st["E"], st["perms"], c["K"], c["W"], seed=st["seed"])
    st["ws"] = torch.empty(binding.step_workspace_bytes(st["tables"], st["sp"]), dtype=torch.uint8, device="cuda")
    if c["kind"] == "sentence":
        g = _generator(seed, 5)
        st["hist"] = binding.BeamHistory(c["S"], c["B"], c["steps"], n_states=4, state_dim=c["d"], eos=EOS)
        st["states"] = [[torch.randn(R, c["d"], device="cuda", generator=g) for _ in range(4)] for _ in range(3)]
        st["next"] = torch.empty(R, dtype=torch.float32, device="cuda")
        if c["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _steps(st)
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            st["replay"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(st["replay"]):
                _steps(st)
    return st


# ---- one pass ---------------------------------------------------------------------------------

def _states_after(st, i):
    """State arrays after i steps: the initial ones stay, the others alternate."""
    return st["states"][0 if i == 0 else 1 + (i & 1)]


def _steps(st):
    for i in range(st["case"]["steps"]):
        binding.decode_step(st["tables"], st["H"][i], st["scores_in"] if i == 0 else st["next"], st["topfreq"], st["sp"],
                            st["ws"], st["beam"], st["word"], st["score"])
        binding.beam_advance(st["hist"], i, st["beam"], st["word"], st["score"], _states_after(st, i),
                             _states_after(st, i + 1), st["next"])


def run(state):
    st, c = state, state["case"]
    if c["kind"] == "sentence":
        if c["graph"]:
            st["replay"].replay()
        else:
            _steps(st)
        tokens, length, best = binding.beam_backtrace(st["hist"], c["steps"])
        h = st["hist"]
        return {"tokens": tokens, "length": length, "best": best, "backptr": h.backptr, "words": h.words, "scores": h.scores,
                "next": st["next"], "states": _states_after(st, c["steps"])}
    if c["kind"] == "build":
        if st["tables"] is not None:
            st["tables"].close()
        st["tables"] = binding.build_tables(st["E"], st["perms"], c["K"], c["W"], seed=st["seed"])
        st["ws"] = torch.empty(binding.step_workspace_bytes(st["tables"], st["sp"]), dtype=torch.uint8, device="cuda")
    binding.decode_step(st["tables"], st["H"][0], st["scores_in"], st["topfreq"], st["sp"], st["ws"], st["beam"], st["word"],
                        st["score"])
    return {"beam": st["beam"], "word": st["word"], "score": st["score"]}


# ---- what a pass cannot do without -------------------------------------------------------------

def _candidates(c, rows):
    """Expected size of the union of `rows` hidden rows' candidates and the top-frequent words
    (an estimate: the lists depend on the data)."""
    if c["t"] > 1:                                       # cluster members, and whoever collides often by chance
        m = 1.15 * c["W"] * float(c["K"]) ** -(c["P"] // c["W"])
        seldom = sum(math.exp(-m) * m ** i / math.factorial(i) for i in range(c["t"]))
        hit = min(1.0, 1.0 - seldom + CLUSTER / c["V"])
    else:
        near = min(1.0, 0.07 * c["W"]) * CLUSTER         # members of the row's own cluster
        hit = min(1.0, (near + c["W"] * c["V"] * float(c["K"]) ** -(c["P"] // c["W"])) / c["V"])
    return c["V"] * (1.0 - (1.0 - min(1.0, c["T"] / c["V"])) * (1.0 - hit) ** rows)


def work(case):
    c = case
    e = 2 if c["bf16"] else 4
    R = c["S"] * c["B"]
    row = c["d"] * e
    small = R * (c["d"] * 4 + 4 + 12)                    # hidden rows, scores, results
    if c["kind"] == "full":
        nbytes, flops = c["V"] * row + small, 2.0 * R * c["V"] * c["d"]
    else:
        lookups = R * c["W"] * 32 + c["P"] * c["K"] * 4 + c["T"] * 4
        if c["t"] > 1:
            lookups += R * c["W"] * c["V"] * 4.0 * c["K"] ** -(c["P"] // c["W"])
        nbytes = _candidates(c, R) * row + small + lookups
        flops = 2.0 * R * _candidates(c, c["B"]) * c["d"]
    if c["kind"] == "sentence":
        nbytes = c["steps"] * (nbytes + 2 * 4 * R * c["d"] * 4 + R * 16)
        flops *= c["steps"]
    if c["kind"] == "build":
        # the rows of E are read and their codes grouped: code and id of every (word, band)
        nbytes += c["V"] * (row + c["W"] * 8.0)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # fp32 sums of up to 1536 products, in any order; scores closer than that may change places
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
