"""The feed-forward work that programs built on this library have it do, as timed cases.

Every case goes through the public entry points with device tensors, the way bench.py and the tests call
them: selection of expert neurons from a prompt, selection together with the prompt's own output,
compaction of the selected neurons, and generated tokens through the pruned block, one row or many.
Shapes are those of the configurations in synth/ (a tiny fp32 block, Llama-2-7B-, Gemma-7B-,
Llama-2-13B- and Mistral-7B-shaped blocks) and, in draw(), generic ones around them.

A case is a dict of plain values:
  kind    select   griffin_prefill_select (+ griffin_index_sets_build: the membership words that
                   programs with more than one prompt decode from)
          phase    griffin_prompt_phase (selection and the prompt's output from one Z)
          onboard  griffin_prefill_select, then griffin_compact of the set it chose
          decode   griffin_ff_decode, `rows` rows through one compact block
          sets     griffin_ff_decode_indexed_sets, `rows` rows with their own sets in the full block
  d, n    model width and neurons held (D_ff of a full block, kept neurons of a compact one)
  k       neurons selected per sequence (select, phase, onboard, sets)
  tokens  lengths of the packed prompts, "a+b+c" (select, phase, onboard)
  rows    rows decoded in one call (decode, sets)
  act     "silu", "gelu" or "relu";  gated: Eq. 3 blocks, else Eq. 2;  bias: with bg, b1, b2
  dtype   "bf16" or "f32"
"""
import torch

import paper_2404_01365_amd as G

_ACT = {"silu": G.ACT_SILU, "gelu": G.ACT_GELU_TANH, "relu": G.ACT_RELU}

# sixteen prompts of 256 to 2048 tokens, 20600 in all: the batch of the Mistral-shaped configuration
_PACKED = "1789+466+1923+1270+814+1555+604+2031+1117+1398+381+1742+958+1486+1183+1883"


def _case(name, kind, d, n, *, k=0, tokens="", rows=0, act="silu", gated=True, bias=False, dtype="bf16"):
    c = dict(kind=kind, d=d, n=n, k=k, tokens=tokens, rows=rows, act=act, gated=gated, bias=bias, dtype=dtype)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: the tiny fp32 block of the smoke test, whole prompt phase; launches and latency count
        _case("phase_tiny_f32", "phase", 256, 688, k=344, tokens="64", dtype="f32"),
        # a chat turn of 40 tokens on a 7B-shaped layer: short prompts read all the weights for little arithmetic
        _case("select_7b_40", "select", 4096, 11008, k=5504, tokens="40"),
        # the 7B-shaped layer of bench.py with its 512-token prompt
        _case("select_7b_512", "select", 4096, 11008, k=5504, tokens="512"),
        # the Gemma-shaped layer (GEGLU) with a long prompt
        _case("select_gemma_2048", "select", 3072, 24576, k=12288, tokens="2048", act="gelu"),
        # a batch of sixteen prompts of ragged lengths on the Mistral-shaped layer, every prompt with its own set: the largest
        _case("select_mistral_packed16", "select", 4096, 14336, k=7168, tokens=_PACKED),
        # prompt phase of a 13B-shaped layer: selection and the full block's output for every prompt token
        _case("phase_13b_1024", "phase", 5120, 13824, k=6912, tokens="1024"),
        # what a program does with a new prompt before the first generated token: select, then compact (odd length)
        _case("onboard_13b_777", "onboard", 5120, 13824, k=6912, tokens="777"),
        # one generated token through the 7B-shaped compact block (half of the neurons): the commonest call
        _case("decode_7b_row1", "decode", 4096, 5504, rows=1),
        # a few rows through a full Eq. 2 block with biases (OPT-style ReLU)
        _case("decode_eq2_bias_rows3", "decode", 4096, 11008, rows=3, act="relu", gated=False, bias=True),
        # sixteen rows that share one set, 13B-shaped compact block
        _case("decode_13b_rows16", "decode", 5120, 6912, rows=16),
        # a larger serving batch that shares one set, Gemma-shaped compact block
        _case("decode_gemma_rows40", "decode", 3072, 12288, rows=40, act="gelu"),
        # sixteen sequences that keep their own halves of the Mistral-shaped block, one token each
        _case("sets_mistral_rows16", "sets", 4096, 14336, k=7168, rows=16),
    ]


def draw(rng):
    """One more case of the same ranges: widths 512 to 8192, 2.5 to 8 times as many neurons (at most ~420 MB of
    weights), 8 to 4096 prompt tokens in 1 to 8 prompts, 1 to 64 rows; one in six a small fp32 block."""
    kind = rng.choice(["select", "select", "phase", "onboard", "decode", "decode", "sets"])
    small = rng.random() < 1 / 6
    log = lambda lo, hi: lo * (hi / lo) ** rng.random()  # noqa: E731
    if small:
        d = 8 * int(log(8, 128))
        n = int(d * rng.uniform(2.0, 4.0))
        total = int(log(4, 256))
    else:
        d = 64 * int(log(8, 128) + 0.5)
        if rng.random() < 0.5:
            d = 512 * max(1, (d + 256) // 512)
        n = int(min(d * log(2.5, 8.0), 70e6 / d))
        n = n if rng.random() < 0.25 else (n + 15) // 16 * 16      # one in four takes an odd number
        total = int(log(8, 4096))
    rows = int(log(1, 64.999))
    act = rng.choice(["silu", "silu", "gelu", "relu"])
    # Eq. 2 blocks come with ReLU (opening the top-k margin scales rows, see _open_margin)
    gated = act != "relu" or rng.random() < 0.4
    bias = rng.random() < 0.3
    keep = rng.uniform(0.25, 0.75)
    dtype = "f32" if small else "bf16"
    kw = dict(act=act, gated=gated, bias=bias, dtype=dtype)
    if kind == "decode":
        return _case(None, kind, d, max(64, int(n * keep)), rows=rows, **kw)
    k = max(1, int(n * keep))
    if kind == "sets":
        return _case(None, kind, d, n, k=k, rows=rows, **kw)
    seqs = rng.randint(2, 8) if kind == "select" and total >= 64 and rng.random() < 0.5 else 1
    cuts = sorted(rng.sample(range(1, total), seqs - 1)) if seqs > 1 else []
    lens = [b - a for a, b in zip([0] + cuts, cuts + [total])]
    return _case(None, kind, d, n, k=k, tokens="+".join(str(v) for v in lens), **kw)


# ----------------------------------------------------------------------------------------------- inputs
def _lens(case):
    return [int(v) for v in case["tokens"].split("+")]


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _inputs(case, seed):
    """Weights N(0, 1/d) and N(0, 1/n), prompts and rows around one mean per sequence, RMS-normalised: the
    recipe of synth/, drawn on the device."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    t, d, n = _dtype(case), case["d"], case["n"]

    def normal(*shape, scale):
        return (torch.randn(*shape, generator=g, device="cuda") * scale).to(t)

    def rows(count):
        x = torch.randn(1, d, generator=g, device="cuda") + 0.5 * torch.randn(count, d, generator=g, device="cuda")
        return (x / x.square().mean(dim=1, keepdim=True).sqrt()).to(t)

    # one neuron's rows side by side, as bench.py lays a compact block out; full blocks as separate matrices
    if case["kind"] == "decode" and case["gated"]:
        blk = torch.empty(n, 3, d, dtype=t, device="cuda")
        blk[:, 0] = normal(n, d, scale=d ** -0.5)
        blk[:, 1] = normal(n, d, scale=d ** -0.5)
        blk[:, 2] = normal(n, d, scale=n ** -0.5)
        w = dict(Wg=blk[:, 0], W1=blk[:, 1], W2=blk[:, 2])
    else:
        w = dict(Wg=normal(n, d, scale=d ** -0.5) if case["gated"] else None, W1=normal(n, d, scale=d ** -0.5),
                 W2=normal(n, d, scale=n ** -0.5))
    w["bg"] = normal(n, scale=0.1) if case["bias"] and case["gated"] else None
    w["b1"] = normal(n, scale=0.1) if case["bias"] else None
    w["b2"] = normal(d, scale=0.1) if case["bias"] else None
    if case["kind"] in ("decode", "sets"):
        w["x"] = torch.cat([rows(1) for _ in range(case["rows"])])
    else:
        w["x"] = torch.cat([rows(v) for v in _lens(case)])
        if len(_lens(case)) == 1:
            _open_margin(case, w)
    if case["kind"] == "sets":
        score = torch.rand(case["rows"], n, generator=g, device="cuda")
        w["idx"] = score.topk(case["k"], dim=1).indices.sort(dim=1).values.to(torch.int32)
    return w


def _sigma(act, a):
    if act == "silu":
        return a * torch.sigmoid(a)
    if act == "gelu":
        return 0.5 * a * (1 + torch.tanh(0.7978845608028654 * (a + 0.044715 * a ** 3)))
    return a.clamp_min(0)


def _z64(case, w):
    """The activations FF_1(X) in 64 bits."""
    x = w["x"].double()
    u = x @ w["W1"].double().t()
    if w["b1"] is not None:
        u += w["b1"].double()
    if w["Wg"] is None:
        return _sigma(case["act"], u)
    a = x @ w["Wg"].double().t()
    if w["bg"] is not None:
        a += w["bg"].double()
    return _sigma(case["act"], a).mul_(u)


def _s64(case, z):
    """The statistic of every sequence in 64 bits."""
    r2 = z.square().sum(dim=1, keepdim=True)
    q = z.square().mul_(torch.where(r2 > 0, 1 / r2, torch.zeros_like(r2)))
    return torch.stack([p.sum(dim=0).sqrt() for p in q.split(_lens(case))])


def _open_margin(case, w):
    """Index sets are compared as they are, so the gap at the k-th score is opened as the tests do it: neurons
    within 0.4 % of it have their row of W1 scaled by 0.8 % away from it (s is linear in that scale)."""
    if case["k"] >= case["n"]:
        return
    s = _s64(case, _z64(case, w))[0]
    v = s.sort(descending=True).values
    t = 0.5 * (v[case["k"] - 1] + v[case["k"]])
    if not bool(t > 0):
        return
    near = (s / t - 1).abs() < 0.004
    f = torch.where(near, torch.where(s >= t, 1.008, 0.992), 1.0)
    w["W1"].copy_((w["W1"].float() * f[:, None]).to(w["W1"].dtype))
    if w["b1"] is not None:
        w["b1"].copy_((w["b1"].float() * f).to(w["b1"].dtype))


# ----------------------------------------------------------------------------------------------- the passes
def _bytes(size):
    return torch.empty(max(int(size), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    w = _inputs(case, seed)
    act, kind, d, n, k, t = _ACT[case["act"]], case["kind"], case["d"], case["n"], case["k"], _dtype(case)
    L = G.layer(w["W1"], w["W2"], w["Wg"], act=act, bg=w["bg"], b1=w["b1"], b2=w["b2"])
    st = dict(kind=kind, L=L, x=w["x"], k=k, rows=case["rows"])
    if kind in ("decode", "sets"):
        st["y"] = torch.zeros_like(w["x"])
        st["ws"] = _bytes(G.griffin_decode_workspace_bytes(d, n, case["rows"]))
        if kind == "sets":
            st["idx"] = w["idx"]
            st["sets"] = torch.zeros(G.griffin_index_sets_bytes(n, case["rows"]) // 4, dtype=torch.int32, device="cuda")
            G.griffin_index_sets_build(w["idx"], k, case["rows"], n, st["sets"])
        return st
    lens = _lens(case)
    cu = [0]
    for v in lens:
        cu.append(cu[-1] + v)
    st["cu"] = cu
    st["idx"] = torch.zeros(len(lens), k, dtype=torch.int32, device="cuda")
    st["s"] = torch.zeros(len(lens), n, dtype=torch.float32, device="cuda")
    if kind == "phase":
        st["W2p"] = w["W2"].t().contiguous()
        st["y"] = torch.zeros_like(w["x"])
        st["ws"] = _bytes(G.griffin_prompt_phase_workspace_bytes(L, cu[-1], len(lens)))
    else:
        st["ws"] = _bytes(G.griffin_prefill_workspace_bytes(L, cu[-1], len(lens), False))
    if len(lens) > 1:
        st["sets"] = torch.zeros(G.griffin_index_sets_bytes(n, len(lens)) // 4, dtype=torch.int32, device="cuda")
    if kind == "onboard":
        mats = 3 if case["gated"] else 2
        blk = torch.zeros(k, mats, d, dtype=t, device="cuda")
        vec = lambda v: None if v is None else torch.zeros(k, dtype=t, device="cuda")  # noqa: E731
        st["blk"], st["cbg"], st["cb1"] = blk, vec(w["bg"]), vec(w["b1"])
        st["C"] = G.layer(blk[:, mats - 2], blk[:, mats - 1], blk[:, 0] if case["gated"] else None, act=act,
                          bg=st["cbg"], b1=st["cb1"], b2=w["b2"])
    return st


def run(st):
    kind = st["kind"]
    if kind == "decode":
        G.griffin_ff_decode(st["L"], st["x"], st["y"], st["rows"], workspace=st["ws"])
        return {"y": st["y"]}
    if kind == "sets":
        G.griffin_ff_decode_indexed_sets(st["L"], st["idx"], st["k"], st["sets"], st["rows"], st["x"], st["y"],
                                         workspace=st["ws"])
        return {"y": st["y"]}
    if kind == "phase":
        G.griffin_prompt_phase(st["L"], st["W2p"], st["x"], st["cu"], st["k"], st["idx"], st["y"], s_out=st["s"],
                               workspace=st["ws"])
        return {"idx": st["idx"], "s": st["s"], "y": st["y"]}
    G.griffin_prefill_select(st["L"], st["x"], st["cu"], st["k"], st["idx"], s_out=st["s"], workspace=st["ws"])
    if kind == "onboard":
        G.griffin_compact(st["L"], st["idx"], st["k"], st["C"])
        out = {"idx": st["idx"], "s": st["s"], "blk": st["blk"]}
        if st["cb1"] is not None:
            out["b1"] = st["cb1"]
        if st["cbg"] is not None:
            out["bg"] = st["cbg"]
        return out
    if "sets" in st:
        # several prompts: their sets go on as membership words (one word per neuron, so that a near-tie at one
        # prompt's boundary changes two words and not the order of a whole list)
        G.griffin_index_sets_build(st["idx"], st["k"], len(st["cu"]) - 1, st["L"].n, st["sets"])
        return {"sets": st["sets"], "s": st["s"]}
    return {"idx": st["idx"], "s": st["s"]}


def work(case):
    es, d, n, mats = (2 if case["dtype"] == "bf16" else 4), case["d"], case["n"], (3 if case["gated"] else 2)
    if case["kind"] in ("decode", "sets"):
        m = case["rows"]
        return {"bytes": es * (mats * n * d + 2 * m * d),
                "flops": 2.0 * mats * (n if case["kind"] == "decode" else case["k"]) * d * m}
    lens = _lens(case)
    m = sum(lens)
    w = {"bytes": es * ((mats - 1) * n * d + m * d) + 4 * len(lens) * (n + case["k"]), "flops": 2.0 * (mats - 1) * m * n * d}
    if case["kind"] == "phase":
        w["bytes"] += es * (n * d + m * d)
        w["flops"] += 2.0 * m * n * d
    if case["kind"] == "onboard":
        w["bytes"] += es * 2 * mats * case["k"] * d
    return w


# Measured against exact(): the statistic is 0.6e-7 to 1.6e-7 off (2-norm; fp32 sums of up to 8192 products), bf16
# outputs 1.7e-3 (their own rounding), outputs of the prompt phase 2.4e-3 (Z is rounded to bf16 on its way into the
# second product), fp32 outputs 1.5e-7 (one block) and 6e-7 (prompt phase).
def tolerance(case):
    kind = case["kind"]
    if kind in ("decode", "sets", "phase"):
        if case["dtype"] == "f32":
            return {"rel": 3e-6}
        return {"rel": 7e-3 if kind != "phase" else 1e-2, "max": 0.05}
    # sets of several prompts: a few near-ties at the boundaries; single prompts have their margin opened
    return {"rel": 1e-6, "differ": 1e-3 if len(_lens(case)) > 1 else 0.0}


def exact(case, seed):
    w = _inputs(case, seed)
    if case["kind"] in ("decode", "sets"):
        z = _z64(case, w)
        if case["kind"] == "sets":
            keep = torch.zeros_like(z)
            keep.scatter_(1, w["idx"].long(), 1.0)
            z *= keep
        y = z @ w["W2"].double()
        return {"y": y if w["b2"] is None else y + w["b2"].double()}
    z = _z64(case, w)
    s = _s64(case, z)
    if case["kind"] == "phase":
        y = z @ w["W2"].double()
        return {"idx": None, "s": s, "y": y if w["b2"] is None else y + w["b2"].double()}
    if case["kind"] == "onboard":
        out = {"idx": None, "s": s, "blk": None}
        if w["b1"] is not None:
            out["b1"] = None
        if w["bg"] is not None:
            out["bg"] = None
        return out
    return {"sets" if len(_lens(case)) > 1 else "idx": None, "s": s}
