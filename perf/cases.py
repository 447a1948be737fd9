"""The calls that a user of the verifier makes, as cases to measure: one pass = one call (or the few calls that belong
together) through `paper_2511_15898_amd.binding`.

A case is a dict of plain values:
  path    "verify"  gr_solve_verify / gr_solve_logits_verify: a batch of decode positions with its drafts in hand
          "slice"   gr_solve, gr_verify and gr_policy_slice: the two steps apart, and the whole distribution pi(.|drafts)
          "sweep"   gr_accept_sweep: the acceptance over a grid of top-k sizes and draft counts
          "tree"    gr_tree_walk: multi-step verification of a tree of draft paths per sequence
  rows    "probs" or "logits": how the target and draft rows are given
  B, V    decode positions (tree: sequences) and vocabulary;  n, k  drafts per position (tree: paths) and top-k (0: none)
  tol     the error threshold tau of the truncated programs;  tail_mass  nucleus cut of the draft (0: none)
  t_lo, t_hi  the row's temperature, uniform between the two;  draft_t  the draft's own temperature (0: the row's)
  corr    draft logits = corr * target logits + N(0, 1);  near  share of rows whose draft is almost the target
  L       levels of the tree;  ks, ns  the grid of the sweep (k = 0: the whole vocabulary)

Rows stand in for language models' next-token distributions: heavy-tailed target logits with a correlated draft, the
recipe of `workloads.py`, drawn on the GPU."""
import math
import weakref

import torch

from paper_2511_15898_amd import binding as gr


def _verify(name, B, V, n, k, **more):
    case = {"name": name, "path": "verify", "rows": "probs", "B": B, "V": V, "n": n, "k": k, "tol": 1e-4, "tail_mass": 0.0,
            "t_lo": 1.0, "t_hi": 1.0, "draft_t": 0.0, "corr": 0.7, "near": 0.0}
    case.update(more)
    return case


def listed():
    return [
        # one sequence being decoded: nothing to fill the chip with, what counts is the chain from the call to the token
        _verify("one row", 1, 32000, 4, 64, corr=0.8, t_lo=0.7, t_hi=0.7),
        # a small vocabulary and few rows: launches and the host path weigh most
        _verify("small batch", 64, 1024, 4, 32, corr=0.8),
        # an ordinary serving batch
        _verify("serving batch", 256, 32000, 4, 64, corr=0.8),
        # the headline configuration: a large vocabulary, eight drafts
        _verify("large vocabulary", 256, 128256, 8, 128),
        # four times as many rows as the chip has compute units, mixed temperatures, some drafts almost the target
        _verify("stress batch", 1024, 128256, 8, 128, t_lo=0.5, t_hi=1.5, near=0.1),
        # as many drafts as the library takes, sizes that are multiples of nothing
        _verify("many drafts, odd sizes", 203, 50021, 16, 101, t_lo=0.5, t_hi=1.5),
        # the rows as the models leave them: logits and a temperature per row
        _verify("logits", 256, 128256, 8, 128, rows="logits", t_lo=0.7, t_hi=1.0),
        # top-p sampling of the draft, the two steps called apart and the whole distribution read out
        _verify("top-p, distribution", 64, 32000, 4, 0, path="slice", tail_mass=1e-3, corr=0.8),
        # no top-k at all on a large batch: supports of the whole vocabulary
        _verify("whole vocabulary", 1024, 128256, 8, 0, t_lo=0.5, t_hi=1.5, near=0.1),
        # the study of the acceptance over top-k sizes and draft counts
        _verify("acceptance grid", 256, 128256, 10, 256, path="sweep", ks="8,16,32,64,128,256", ns="1,2,3,4,5,6,7,8,9,10"),
        # the same with top-k sizes up to the whole vocabulary
        _verify("acceptance grid to V", 256, 128256, 10, 0, path="sweep", ks="10,100,1000,10000,100000,0", ns="1,2,3,4,5,6,7,8,9,10"),
        # several decoding steps at once: a tree of draft paths per sequence
        _verify("draft tree", 32, 32000, 4, 64, path="tree", L=5, corr=0.8),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["top-k", "top-k", "top-k", "logits", "logits", "slice", "whole", "sweep", "sweep to V", "tree"])
    case = _verify("", _log_between(rng, 1, 1024), _log_between(rng, 300, 128256), rng.randint(1, 16), _log_between(rng, 8, 256),
                   tol=rng.choice([1e-3, 1e-4]), t_lo=0.6, t_hi=1.4, corr=rng.choice([0.7, 0.8]), near=rng.choice([0.0, 0.1]))
    del case["name"]
    if rng.random() < 0.4:
        case["V"] = max(304, case["V"] // 8 * 8)                 # vocabularies are often padded
    if kind == "logits":
        case["rows"] = "logits"
        case["draft_t"] = rng.choice([0.0, 1.0])
    elif kind == "slice":
        case["path"] = "slice"
        case["B"] = min(case["B"], max(1, (1 << 25) // case["V"]))
        case["tail_mass"] = rng.choice([0.0, 0.0, 1e-3])
        if case["tail_mass"]:
            case["k"] = 0
    elif kind == "whole":
        case["k"] = 0 if rng.random() < 0.5 else _log_between(rng, 257, max(258, case["V"]))
        case["tail_mass"] = rng.choice([0.0, 0.0, 1e-8, 1e-3])
        case["rows"] = "probs" if case["tail_mass"] else rng.choice(["probs", "probs", "logits"])
    elif kind.startswith("sweep"):
        case["path"] = "sweep"
        case["B"] = min(case["B"], 256)
        top = case["V"] if kind == "sweep to V" else 256
        ks = sorted({_log_between(rng, 4, top) for _ in range(rng.randint(2, 8))})
        if kind == "sweep to V":
            ks[-1] = 0
        case["ks"] = ",".join(map(str, ks))
        case["ns"] = ",".join(map(str, sorted(rng.sample(range(1, 17), rng.randint(2, 12)))))
        case["k"] = 0 if kind == "sweep to V" else max(ks)
    elif kind == "tree":
        case["path"] = "tree"
        case["rows"] = rng.choice(["probs", "logits"])
        case["L"] = rng.randint(2, 8)
        case["n"] = rng.randint(2, 8)
        case["B"] = max(1, min(case["B"], (1 << 26) // (case["n"] * case["L"] * case["V"])))
        case["near"] = 0.0
    return case


class _State:
    pass


def _logits(case, gen, rows):
    """Target and draft logits of `rows` positions, [rows, V]."""
    V = case["V"]
    gumbel = torch.empty((rows, V), device="cuda").exponential_(generator=gen).clamp_(min=1e-9).log_().neg_()
    target = gumbel.mul_(4.0)
    draft = torch.randn((rows, V), device="cuda", generator=gen)
    near = torch.rand((rows, 1), device="cuda", generator=gen) < case["near"]
    draft.mul_(torch.where(near, 0.01, 1.0))
    draft.add_(target * torch.where(near, 1.0, case["corr"]))
    return target, draft


def _drafts(q, k, n, gen):
    """n independent draws per row from q cut to its k largest."""
    if 0 < k < q.shape[1]:
        mass, ids = torch.topk(q, k)
        return ids.gather(1, torch.multinomial(mass, n, replacement=True, generator=gen)).int()
    return torch.multinomial(q, n, replacement=True, generator=gen).int()


def _nucleus(q, tail_mass):
    """q cut to the fewest tokens that hold 1 - tail_mass of it."""
    mass, ids = torch.sort(q, dim=1, descending=True, stable=True)
    before = mass.double().cumsum(1) - mass.double()
    mass = mass * (before < 1.0 - tail_mass - 1e-6)              # a little inside the cut: every draft lies in the support
    return torch.zeros_like(q).scatter_(1, ids, mass)


def prepare(case, seed):
    """The rows, drafts and uniforms on the GPU, the buffers for the results, and the handle that a program creates once."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    B, V, n, k = case["B"], case["V"], case["n"], case["k"]
    s = _State()
    s.case = case
    temp = torch.empty((B, 1), device="cuda").uniform_(case["t_lo"], case["t_hi"], generator=gen)
    draft_temp = torch.full_like(temp, case["draft_t"]) if case["draft_t"] else temp
    s.temp, s.draft_temp = temp.view(-1), draft_temp.view(-1) if case["draft_t"] else None
    s.uniforms = torch.rand(B, device="cuda", generator=gen).clamp_(max=1.0 - 2.0 ** -24)
    s.handle = gr.gr_create(B, V, max_k=k, max_n=n, tail_mass=case["tail_mass"])
    weakref.finalize(s, gr.gr_destroy, s.handle)
    if case["path"] == "tree":
        return _prepare_tree(s, case, gen, temp)
    target, draft = _logits(case, gen, B)
    if case["rows"] == "logits":
        s.p, s.q = target, draft
        q = torch.softmax(draft / draft_temp, 1)
    else:
        s.p = torch.softmax(target.div_(temp), 1)
        s.q = q = torch.softmax(draft.div_(draft_temp), 1)
    if case["path"] == "sweep":
        s.ks, s.ns = ([int(x) for x in case[w].split(",")] for w in ("ks", "ns"))
        s.grid = torch.empty((B, len(s.ks), len(s.ns)), device="cuda")
    else:
        s.drafts = _drafts(_nucleus(q, case["tail_mass"]) if case["tail_mass"] else q, k, n, gen)
        s.accept_prob = torch.empty(B, device="cuda")
        s.token = torch.empty(B, dtype=torch.int32, device="cuda")
        s.accepted = torch.empty(B, dtype=torch.uint8, device="cuda")
    s.status = torch.empty(B, dtype=torch.int32, device="cuda")
    return s


def _prepare_tree(s, case, gen, temp):
    """Paths drawn token by token; paths with equal prefixes see equal rows."""
    S, K, L, V = case["B"], case["n"], case["L"], case["V"]
    s.p = torch.empty((S, K, L, V), device="cuda")
    s.q = torch.empty((S, K, L, V), device="cuda")
    paths = torch.zeros((S, K, L), dtype=torch.int32, device="cuda")
    for l in range(L):
        same = (paths[:, :, None, :l] == paths[:, None, :, :l]).all(-1)          # [S, K, K]
        first = same.int().argmax(-1)                                          # the first path with this prefix
        row = (torch.arange(S, device="cuda")[:, None] * K + first).view(-1)
        target, draft = _logits(case, gen, S * K)
        target, draft = target[row], draft[row]
        q = torch.softmax(draft / temp.repeat_interleave(K, 0), 1)
        if case["rows"] == "probs":
            target, draft = torch.softmax(target / temp.repeat_interleave(K, 0), 1), q
        s.p[:, :, l], s.q[:, :, l] = target.view(S, K, V), draft.view(S, K, V)
        paths[:, :, l] = _drafts(q, case["k"], 1, gen).view(S, K)
    s.paths = paths.cpu().numpy()
    s.uniforms = torch.rand((S, L), device="cuda", generator=gen).clamp_(max=1.0 - 2.0 ** -24).cpu().numpy()
    s.temp = s.temp.cpu().numpy() if case["rows"] == "logits" else None
    return s


def run(s):
    c = s.case
    n, k, tol = c["n"], c["k"], c["tol"]
    if c["path"] == "sweep":
        return gr.gr_accept_sweep(s.handle, s.p, s.q, s.ks, s.ns, s.grid, s.status)
    if c["path"] == "tree":
        return gr.gr_tree_walk(s.handle, s.p, s.q, s.paths, s.uniforms, k, tol, temperature=s.temp)
    if c["path"] == "slice":
        gr.gr_solve(s.handle, s.p, s.q, n, k, tol, s.accept_prob, s.status)
        gr.gr_verify(s.handle, s.drafts, s.uniforms, s.token, s.accepted)
        return (s.accept_prob, s.status, s.token, s.accepted) + gr.gr_policy_slice(s.handle, s.drafts, c["V"])
    if c["rows"] == "logits":
        return gr.gr_solve_logits_verify(s.handle, s.p, s.q, s.temp, n, k, tol, s.drafts, s.uniforms, s.accept_prob, s.status,
                                         s.token, s.accepted, draft_temperature=s.draft_temp)
    return gr.gr_solve_verify(s.handle, s.p, s.q, n, k, tol, s.drafts, s.uniforms, s.accept_prob, s.status, s.token, s.accepted)


def work(case):
    """Bytes: the rows once (of a tree: one node per sequence and level) and the outputs once.  Operations: one evaluation
    of the routed masses, which no solver does without (about 50 quadrature nodes, 4 n^2 per node and token of the program,
    at most 128 of them); of a sweep, a difference of two prefix masses for every token, top-k size and draft count."""
    B, V, n, k = case["B"], case["V"], case["n"], case["k"]
    if case["path"] == "sweep":
        nk, nn = case["ks"].count(",") + 1, case["ns"].count(",") + 1
        return {"bytes": 8 * B * V + 4 * B * nk * nn + 4 * B, "flops": 4 * B * (k or V) * nk * nn}
    rows = B * (case["L"] if case["path"] == "tree" else 1)
    bytes_ = rows * (8 * V + 4 * n + 4 + 13)
    if case["path"] == "slice":
        bytes_ += B * (4 * V + 4)
    return {"bytes": bytes_, "flops": rows * (50 * 4 * n * n * min(k or 128, 128) + 2 * V)}


def tolerance(case):
    """The acceptance and the distribution are float32 roundings of float64 results whose programs are solved to 1e-8.  A
    token differs only where the uniform falls within that of an edge of the distribution, a status only where a program
    stands at its cap."""
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.004}
