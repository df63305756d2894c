"""The work that a user of this library has it do, as cases that can be timed.

A speculative decode step of a video LLM calls the library in four places, and every case is one of them:

  attn    decode attention of all layers: the draft's single query over its pruned cache, the verifier's block of
          gamma + 1 queries over the full cache, a draft tree, a ragged batch of requests
  score   the language-to-video attention scores of the verifier's layers, once per request after the prefill
  prune   the retention set and the draft's cache made from it (optionally sized by score mass), once per request
  accept  which drafted tokens survive, once per step

Shapes are those of the workloads in ``paper_2508_16201_amd.synth`` (14 x 14 or 16 x 16 tokens a frame, head shapes
4/1, 14/2, 28/4, 40/8 and 64/8); values are drawn on the device from the recipe of that module: unit-variance
queries, keys and values, 2 % of the video keys planted as heavy, long-tailed scores, logits whose drafts are
right about four times in five.
"""
import math
import random

import torch

from paper_2508_16201_amd import binding as B
from paper_2508_16201_amd import synth

# (query heads, kv heads, head size) of the models that the workloads describe
HEADS = ((4, 1, 64), (14, 2, 64), (28, 4, 128), (40, 8, 128), (64, 8, 128))
VOCAB = 152064


# ------------------------------------------------------------------------------------------------- the cases
def attn(name, layers, q_len, kv_len, heads, **more):
    hq, hkv, d = heads
    case = {"name": name, "kind": "attn", "layers": layers, "batch": 1, "q_len": q_len, "kv_len": kv_len, "hq": hq,
            "hkv": hkv, "d": d, "token_major": False, "tree": False, "graph": True, "lse": False, "lens": 0}
    case.update(more)
    return case


def score(name, layers, n_text, n_video, heads, **more):
    hq, hkv, d = heads
    case = {"name": name, "kind": "score", "layers": layers, "batch": 1, "n_text": n_text, "n_video": n_video, "hq": hq,
            "hkv": hkv, "d": d, "token_major": False, "row_lse": False, "norm_mode": 0, "lens": 0}
    case.update(more)
    return case


def prune(name, layers, n_text, n_video, kv_heads, d, keep_percent, **more):
    case = {"name": name, "kind": "prune", "layers": layers, "batch": 1, "n_text": n_text, "n_video": n_video,
            "hkv": kv_heads, "d": d, "keep_percent": keep_percent, "token_major": False, "top_p": False, "lens": 0}
    case.update(more)
    return case


def accept(name, batch, gamma, vocab, sampling, tree=False):
    return {"name": name, "kind": "accept", "batch": batch, "gamma": gamma, "vocab": vocab, "sampling": sampling,
            "tree": tree}


def listed():
    return [
        # the draft's decode over its pruned cache: gamma of these stages make the drafted block of a step, so their
        # launches and latencies are what a step waits for
        attn("draft-decode", 24, 1, 1511, (14, 2, 64), token_major=True),
        # the verification of a chain block, all layers of the 72B shape: 4.2 GB of cache in one stage, the largest
        # part of a decode step
        attn("verify-72b", 80, 6, 12806, (64, 8, 128)),
        # the same at the long video (128 frames of 256 tokens): bandwidth, not latency
        attn("verify-long", 64, 6, 33030, (40, 8, 128)),
        # eight requests of very different lengths in one call of a serving loop, which makes its calls as it goes
        attn("verify-ragged", 1, 6, 32994, (64, 8, 128), batch=8, token_major=True, graph=False, lens=4),
        # the verification of a draft tree of 26 nodes: 208 query rows a kv head
        attn("verify-tree", 80, 26, 12826, (64, 8, 128), tree=True),
        # the scores of a request of the 72B shape, all layers in one call: most of what pruning costs
        score("score-72b", 80, 256, 12544, (64, 8, 128)),
        # self-speculation with the 7B shape; the prefill attention has saved the row normalisers
        score("score-lse-7b", 28, 256, 25088, (28, 4, 128), row_lse=True),
        # one layer of the smallest shape (8 frames), called as the layers go by
        score("score-small", 1, 64, 1568, (4, 1, 64)),
        # the retention set of a 72B-shaped request and its small draft's cache
        prune("prune-draft", 24, 256, 12544, 2, 64, 10, token_major=True),
        # self-speculation: the verifier's own cache is pruned, Stage I sized by score mass
        prune("prune-self", 80, 256, 12544, 8, 128, 10, top_p=True),
        # greedy acceptance of a chain, and rejection sampling at the longest chain that the workloads use
        accept("accept-greedy", 1, 5, VOCAB, False),
        accept("accept-sampling", 1, 7, VOCAB, True),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("attn", "attn", "attn", "score", "score", "prune", "prune", "accept"))
    heads = rng.choice(HEADS)
    hq, hkv, d = heads
    if kind == "attn":
        what = rng.choice(("draft", "verify", "ragged", "tree"))
        token_major, lse = rng.random() < 0.5, rng.random() < 0.25
        if what == "ragged":
            kv_len = log_int(rng, 700, 40000)
            case = attn("", 1, rng.randint(1, 64 // (hq // hkv)), kv_len, heads, batch=rng.randint(2, 12), graph=False,
                        lens=rng.randint(1, 1 << 20))
        elif what == "draft":
            case = attn("", 1, 1, log_int(rng, 200, 20000), heads)
        elif what == "verify":
            case = attn("", 1, rng.randint(2, 8), log_int(rng, 400, 131072), heads)
        else:
            case = attn("", 1, rng.randint(9, 64), log_int(rng, 400, 40000), heads, tree=True)
        case.update(token_major=token_major, lse=lse)
        # as many layers as a model of these heads has, within 4 GB of cache
        if what != "ragged":
            room = 4e9 / (4 * case["kv_len"] * hkv * d)
            case["layers"] = max(1, min(rng.choice((16, 24, 28, 64, 80)), int(room)))
            case["graph"] = rng.random() < 0.75
    elif kind == "score":
        n_video = log_int(rng, 800, 33000)
        case = score("", 1, log_int(rng, 16, 512), n_video, heads, token_major=rng.random() < 0.5,
                     norm_mode=int(rng.random() < 0.25), row_lse=rng.random() < 0.25)
        if rng.random() < 0.25:
            case.update(batch=rng.randint(2, 4), lens=rng.randint(1, 1 << 20))
        # within the logits of the 72B request (a text query's padding to 64 included)
        per_layer = case["batch"] * (case["n_text"] + 63) // 64 * 64 * hq * n_video
        case["layers"] = max(1, min(rng.choice((1, 1, 24, 28, 64, 80)), int(80 * 256 * 64 * 12544 / per_layer)))
        if case["row_lse"]:
            case["layers"] = min(case["layers"], 28)
    elif kind == "prune":
        n_video = log_int(rng, 800, 33000)
        case = prune("", rng.choice((24, 28, 64, 80)), log_int(rng, 16, 512), n_video, hkv, d,
                     rng.choice((10, 10, 25, 50)), token_major=rng.random() < 0.5, top_p=rng.random() < 0.5)
        if rng.random() < 0.25:
            case.update(batch=rng.randint(2, 8), lens=rng.randint(1, 1 << 20))
        rows = case["batch"] * (case["n_text"] + n_video)
        case["layers"] = max(1, min(case["layers"], int(4e9 / (4 * rows * hkv * d))))
    else:
        what = rng.choice(("greedy", "sampling", "tree"))
        case = accept("", rng.randint(1, 8), rng.randint(1, 8), rng.choice((1024, 32000, 65537, VOCAB)),
                      what == "sampling")
        if what == "tree":
            case.update(gamma=rng.randint(9, 40), tree=True)
    del case["name"]
    return case


# ------------------------------------------------------------------------------------- sizes, work, tolerances
def lengths(case, longest):
    """The requests' own lengths: all the same, or (lens: a seed) spread over an eighth of the longest and up."""
    if not case["lens"]:
        return [longest] * case["batch"]
    r = random.Random(case["lens"])
    return [longest] + [r.randint(max(1, longest // 8), longest) for _ in range(case["batch"] - 1)]


def budget(case, n_video):
    return (n_video * case["keep_percent"] + 50) // 100


def work(case):
    if case["kind"] == "attn":
        hq, hkv, d, q_len = case["hq"], case["hkv"], case["d"], case["q_len"]
        keys = sum(lengths(case, case["kv_len"]))
        one = 2 * 2 * keys * hkv * d + 2 * 2 * case["batch"] * q_len * hq * d + 4 * case["lse"] * case["batch"] * q_len * hq
        return {"bytes": case["layers"] * one, "flops": case["layers"] * 4 * keys * q_len * hq * d}
    if case["kind"] == "score":
        hq, hkv, d, n_text = case["hq"], case["hkv"], case["d"], case["n_text"]
        videos = sum(lengths(case, case["n_video"]))
        keys = videos + case["batch"] * n_text
        one = 2 * keys * hkv * d + 2 * case["batch"] * n_text * hq * d + 4 * case["row_lse"] * case["batch"] * n_text * hq
        # one evaluation of every logit
        return {"bytes": case["layers"] * one + 4 * videos, "flops": case["layers"] * 2 * keys * n_text * hq * d}
    if case["kind"] == "prune":
        videos = lengths(case, case["n_video"])
        kept = sum(budget(case, v) for v in videos)
        rows = kept + case["batch"] * case["n_text"]
        return {"bytes": 4 * sum(videos) + 5 * kept + 2 * 4 * case["layers"] * rows * case["hkv"] * case["d"], "flops": 0}
    rows = 2 * case["gamma"] + 1 if case["sampling"] else case["gamma"] + 1
    return {"bytes": 4 * case["batch"] * rows * case["vocab"], "flops": 0}


def tolerance(case):
    # (largest seen against the same sums in 64 bits, listed cases: attention 0.0029 and 0.013, whose output and
    # probabilities are bf16; scores 6e-7 and 1.1e-6, sums of up to 1.3 million 32-bit terms whose order is free)
    if case["kind"] == "attn":
        return {"rel": 1e-2, "max": 5e-2}
    if case["kind"] == "score":
        return {"rel": 4e-6, "max": 2e-5}
    return "exact"


# ------------------------------------------------------------------------------------------------------ inputs
def generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def offsets(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return torch.tensor(cu, dtype=torch.int32, device="cuda")


def normal(g, layers, tokens, heads, d, token_major):
    """bf16 [layers, tokens, heads, d], with tokens or heads outermost in memory."""
    if token_major:
        return torch.randn((layers, tokens, heads, d), generator=g, device="cuda", dtype=torch.bfloat16)
    return torch.randn((layers, heads, tokens, d), generator=g, device="cuda", dtype=torch.bfloat16).permute(0, 2, 1, 3)


def captured(state, stage):
    """A decode stage is a launch-bound chain of short kernels: captured once, replayed at every step."""
    stage(state)
    torch.cuda.synchronize()
    state["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(state["graph"]):
        stage(state)


def prepare(case, seed):
    return {"attn": prepare_attn, "score": prepare_score, "prune": prepare_prune, "accept": prepare_accept}[case["kind"]](
        case, seed)


def prepare_attn(case, seed):
    g = generator(seed)
    layers, batch, q_len, hq, hkv, d = (case[x] for x in ("layers", "batch", "q_len", "hq", "hkv", "d"))
    lens = lengths(case, case["kv_len"])
    lens = [max(n, q_len) for n in lens]
    s = {"case": case, "graph": None, "scale": 1.0 / math.sqrt(d)}
    s["k"] = normal(g, layers, sum(lens), hkv, d, case["token_major"])
    s["v"] = normal(g, layers, sum(lens), hkv, d, case["token_major"])
    s["q"] = normal(g, layers, batch * q_len, hq, d, True)
    s["out"] = torch.empty_like(s["q"])
    s["more"] = {"workspace": B.new_workspace(B.decode_attn_workspace_bytes(batch, q_len, max(lens), hq, hkv, d))}
    if case["lse"]:
        s["more"]["want_lse"] = True
    if batch > 1:
        s["more"].update(cu_q=offsets([q_len] * batch), cu_kv=offsets(lens), max_q_len=q_len, max_kv_len=max(lens))
    if case["tree"]:
        masks = synth.ancestor_masks(synth.make_tree(q_len, seed))
        s["more"]["ancestor_mask"] = torch.tensor(masks.view("int64"), device="cuda").repeat(batch)
    if case["graph"]:
        captured(s, attn_stage)
    return s


def attn_stage(s):
    lse = []
    for layer in range(s["case"]["layers"]):
        got = B.decode_attn(s["q"][layer], s["k"][layer], s["v"][layer], s["scale"], out=s["out"][layer], **s["more"])
        if s["case"]["lse"]:
            lse.append(got[1])
    s["lse"] = torch.stack(lse) if lse else None
    return s["out"], s["lse"]


def prepare_score(case, seed):
    g = generator(seed)
    layers, batch, n_text, hq, hkv, d = (case[x] for x in ("layers", "batch", "n_text", "hq", "hkv", "d"))
    videos = lengths(case, case["n_video"])
    keys = [v + n_text for v in videos]
    s = {"case": case, "scale": 1.0 / math.sqrt(d), "more": {}}
    s["q"] = normal(g, layers, batch * n_text, hq, d, True)
    s["k"] = normal(g, layers, sum(keys), hkv, d, case["token_major"])
    # 2 % of the video keys are heavy: each is the direction of one text query (the mean over the q heads of its
    # group) at a group-mean logit of 11
    first = 0
    for b, v in enumerate(videos):
        n = max(1, v // 50)
        at = first + torch.randperm(v, generator=g, device="cuda")[:n]
        who = b * n_text + torch.randint(n_text, (n,), generator=g, device="cuda")
        for layer in range(layers):
            mean = s["q"][layer, who].float().view(n, hkv, hq // hkv, d).mean(2)
            size = mean.norm(dim=-1, keepdim=True)
            s["k"][layer, at] = (mean * (11.0 / (s["scale"] * size * size))).to(torch.bfloat16)
        first += keys[b]
    if batch > 1:
        s["more"].update(cu_text=offsets([n_text] * batch), cu_keys=offsets(keys), cu_video=offsets(videos),
                         max_n_text=n_text, max_n_keys=max(keys), max_n_video=max(videos), total_video=sum(videos))
    if case["row_lse"]:
        s["row_lse"] = saved_normalisers(case, s, keys, videos)
    need = B.score_layers_workspace_bytes(layers, n_text, max(keys), max(videos), hq, hkv, d, case["row_lse"], batch=batch)
    s["more"].update(workspace=B.new_workspace(need), norm_mode=case["norm_mode"])
    return s


def saved_normalisers(case, s, keys, videos):
    """Natural-log softmax normalisers of the text queries, as the verifier's prefill attention leaves them."""
    n_text, hq, hkv = case["n_text"], case["hq"], case["hkv"]
    lse = torch.empty((case["layers"], case["batch"] * n_text, hq), dtype=torch.float32, device="cuda")
    first = 0
    for b, (n, v) in enumerate(zip(keys, videos)):
        hidden = torch.arange(n, device="cuda")[None, :] > (v + torch.arange(n_text, device="cuda"))[:, None]
        if case["norm_mode"]:
            hidden = hidden | (torch.arange(n, device="cuda") >= v)[None, :]
        for layer in range(case["layers"]):
            q = s["q"][layer, b * n_text:(b + 1) * n_text].float().permute(1, 0, 2).reshape(hkv, -1, case["d"]).contiguous()
            k = s["k"][layer, first:first + n].float().permute(1, 2, 0).contiguous()
            logits = (torch.bmm(q, k) * s["scale"]).view(hq, n_text, n).masked_fill_(hidden[None], float("-inf"))
            lse[layer, b * n_text:(b + 1) * n_text] = torch.logsumexp(logits, dim=-1).transpose(0, 1)
        first += n
    return lse


def prepare_prune(case, seed):
    g = generator(seed)
    layers, batch, n_text, hkv, d = (case[x] for x in ("layers", "batch", "n_text", "hkv", "d"))
    videos = lengths(case, case["n_video"])
    keep = [budget(case, v) for v in videos]
    rows = sum(videos) + batch * n_text
    s = {"case": case, "total_video": sum(videos), "total_keep": sum(keep)}
    # long-tailed scores: a flat background near 1/n, 2 % of the tokens 20 to 100 times heavier
    flat = (1.0 + 0.05 * torch.randn(sum(videos), generator=g, device="cuda")) / max(videos)
    heavy = torch.rand(sum(videos), generator=g, device="cuda") < 0.02
    s["scores"] = torch.where(heavy, flat * (20 + 80 * torch.rand(sum(videos), generator=g, device="cuda")), flat).abs()
    s["k"] = normal(g, layers, rows, hkv, d, case["token_major"])
    s["v"] = normal(g, layers, rows, hkv, d, case["token_major"])
    kept = rows - sum(videos) + sum(keep)
    shape = (layers, kept, hkv, d) if case["token_major"] else (layers, hkv, kept, d)
    s["k_dst"], s["v_dst"] = (torch.empty(shape, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    if not case["token_major"]:
        s["k_dst"], s["v_dst"] = s["k_dst"].permute(0, 2, 1, 3), s["v_dst"].permute(0, 2, 1, 3)
    s["budget"] = torch.tensor(keep, dtype=torch.int32, device="cuda")
    s["k_top"] = torch.tensor([n // 2 for n in keep], dtype=torch.int32, device="cuda")
    s["mass"], s["select"], s["gather"] = {}, {}, {}
    if batch > 1:
        cu_video, cu_keep = offsets(videos), offsets(keep)
        s["mass"] = {"cu_video": cu_video, "max_n_video": max(videos)}
        s["select"] = {"cu_video": cu_video, "cu_keep": cu_keep, "max_n_video": max(videos)}
        s["gather"] = {"cu_keys": offsets([v + n_text for v in videos]), "cu_video": cu_video, "cu_keep": cu_keep}
    return s


def prepare_accept(case, seed):
    g = generator(seed)
    batch, gamma, vocab = case["batch"], case["gamma"], case["vocab"]
    s = {"case": case}
    s["target"] = 3.0 * torch.randn((batch, gamma + 1, vocab), generator=g, device="cuda")
    draft = s["target"][:, :gamma] + 0.3 * torch.randn((batch, gamma, vocab), generator=g, device="cuda")
    if case["tree"]:
        parent = synth.make_tree(gamma + 1, seed)
        # every node drafts the most likely token after its parent, or the draft's own guess at it
        at = torch.tensor(parent, device="cuda").clamp(min=0).long()
        sure = torch.rand((batch, gamma + 1), generator=g, device="cuda") < 0.5
        best = s["target"].argmax(-1)
        guess = torch.cat([draft.argmax(-1), best[:, :1]], dim=1)
        s["tokens"] = torch.where(sure, best[:, at], guess[:, at]).to(torch.int32)
        s["parent"] = torch.tensor(parent, device="cuda")
        s["workspace"] = B.new_workspace(B.accept_workspace_bytes(batch, gamma, vocab, False))
        return s
    s["draft"] = s["uniforms"] = None
    if case["sampling"]:
        s["draft"] = draft
        s["uniforms"] = torch.rand((batch, gamma + 1), generator=g, device="cuda").clamp_(max=1.0 - 2.0 ** -24)
        draft = draft - torch.log(-torch.log(torch.rand(draft.shape, generator=g, device="cuda").clamp_(1e-7, 1.0 - 1e-7)))
    s["tokens"] = draft.argmax(-1).to(torch.int32)
    s["workspace"] = B.new_workspace(B.accept_workspace_bytes(batch, gamma, vocab, case["sampling"]))
    s["n_accepted"] = torch.empty(batch, dtype=torch.int32, device="cuda")
    s["out_tokens"] = torch.empty((batch, gamma + 1), dtype=torch.int32, device="cuda")
    return s


# ----------------------------------------------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    if case["kind"] == "attn":
        if s["graph"] is None:
            return attn_stage(s)
        s["graph"].replay()
        return s["out"], s["lse"]
    if case["kind"] == "score":
        if case["layers"] == 1:
            return B.score(s["q"][0], s["k"][0], 0, case["n_video"], -1, s["scale"],
                           row_lse=s["row_lse"][0] if case["row_lse"] else None, **s["more"])
        return B.score_layers(s["q"], s["k"], 0, case["n_video"], -1, s["scale"],
                              row_lse=s["row_lse"] if case["row_lse"] else None, **s["more"])
    if case["kind"] == "prune":
        k_top, count = s["k_top"], None
        if case["top_p"]:
            k_top = count = B.top_p_count(s["scores"], 0.4, max_count=s["budget"], **s["mass"])
        keep_idx, from_topk = B.select(s["scores"], k_top, s["budget"], s["total_keep"], **s["select"])
        B.gather_kv(s["k"], s["v"], 0, s["total_video"], keep_idx, k_dst=s["k_dst"], v_dst=s["v_dst"], **s["gather"])
        return keep_idx, from_topk, count, s["k_dst"], s["v_dst"]
    if case["tree"]:
        return B.accept_tree(s["target"], s["tokens"], s["parent"], workspace=s["workspace"])
    return B.accept(s["target"], s["tokens"], draft_logits=s["draft"], uniforms=s["uniforms"], workspace=s["workspace"],
                    n_accepted=s["n_accepted"], out_tokens=s["out_tokens"])
