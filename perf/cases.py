"""The work a user has this framework do, as measurable cases: likelihood queries, parameter flows and EM steps of compiled
circuits of the five structure families of `paper_2406_00766_amd.workloads`, from single-sample queries of a small HMM to
the training step of a 520 M-edge HMM.

A case is a dict of plain values:
  family   "hmm", "hclt", "pd", "rat" or "layer" (one wide block-sparse sum layer), with that family's own sizes
  K        node block size;  B  samples of the batch
  tree     seed of the random structure (the tree of an HCLT, the kept blocks of a PD or a layer, a RAT-SPN's permutations):
           part of the case, since a user compiles a structure once; parameters and data come from the seed of `prepare`
  mode     "forward"  log-likelihoods of a batch (evaluation, outlier scores, likelihood queries)
           "static"   the same through pc_forward_static (serving loops that allocate nothing)
           "flows"    forward + backward, the flows accumulated (full-batch EM over many batches)
           "em"       forward + backward + pc_em_step (mini-batch EM)
  masked   a share of the variables is marginalised, differently in every sample (conditional queries, missing data)
  scratch  the memory-saving mode: product values recomputed in the backward pass
"""
from __future__ import annotations

import functools

import numpy as np
import torch

from paper_2406_00766_amd import binding as pcb
from paper_2406_00766_amd import workloads as W

FLT_MIN = torch.finfo(torch.float32).tiny


def listed():
    return [
        # one sentence scored in a serving loop: a small HMM, one sample, some tokens unknown
        dict(name="hmm_16x32_static_b1", family="hmm", T=16, H=32, V=64, K=32, B=1, mode="static", masked=True),
        # the small HMM of the benchmark configurations, trained by mini-batch EM
        dict(name="hmm_16x32_em_b128", family="hmm", T=16, H=32, V=64, K=32, B=128, mode="em", masked=False),
        # a language-model HMM of moderate size, a batch that is no multiple of anything
        dict(name="hmm_32x512_flows_b77", family="hmm", T=32, H=512, V=50257, K=64, B=77, mode="flows", masked=False),
        # the large language-model HMM (the headline configuration)
        dict(name="hmm_32x4096_flows_b256", family="hmm", T=32, H=4096, V=50257, K=128, B=256, mode="flows", masked=False),
        # 28 x 28 images with missing pixels scored by a hidden Chow-Liu tree, ragged batch
        dict(name="hclt_784x128_forward_b100", family="hclt", D=784, M=128, K=64, B=100, tree=240600768, mode="forward", masked=True),
        # the same tree, one training batch of full-batch EM
        dict(name="hclt_784x128_flows_b512", family="hclt", D=784, M=128, K=64, B=512, tree=240600768, mode="flows", masked=False),
        # 32 x 32 x 3 images, mini-batch EM
        dict(name="hclt_3072x256_em_b256", family="hclt", D=3072, M=256, K=64, B=256, tree=240600769, mode="em", masked=False),
        # 32 x 32 pixels, Poon-Domingos structure with three quarters of its edge blocks pruned
        dict(name="pd_32x32_keep25_flows_b256", family="pd", grid=8, cell=4, M=256, K=32, keep=0.25, B=256, tree=240600771,
             mode="flows", masked=False, scratch=False),
        # a dense PD where memory is short: product values recomputed
        dict(name="pd_16x16_scratch_flows_b300", family="pd", grid=8, cell=2, M=64, K=32, keep=1.0, B=300, tree=240600771,
             mode="flows", masked=False, scratch=True),
        # the RAT-SPN of the batch-size table at its largest batch, mini-batch EM
        dict(name="rat_784_em_b512", family="rat", D=784, depth=4, R=4, S=256, K=32, B=512, tree=240600772, mode="em", masked=False),
        # the same structure asked for the likelihoods of a handful of images
        dict(name="rat_784_forward_b16", family="rat", D=784, depth=4, R=4, S=256, K=32, B=16, tree=240600772, mode="forward",
             masked=False),
        # a block-sparse sum layer in blocks of 16 (the vector kernels), odd batch
        dict(name="layer_28x1024_k16_flows_b333", family="layer", sets=28, M=1024, K=16, keep=0.3, B=333, tree=240600773,
             mode="flows", masked=False),
    ]


# ---- sizes ----
def _pd_blocks(c):
    """(sum block, child block) pairs before pruning, excluding the root's, and the root's child blocks."""
    g, nb, pairs, root = c["grid"], c["M"] // c["K"], 0, 0
    for w in range(1, g + 1):
        for h in range(1, g + 1):
            n = (g - w + 1) * (g - h + 1) * max(1, (w - 1) + (h - 1)) * nb
            if w == g and h == g:
                root = n
            else:
                pairs += n * nb
    return pairs, root


def _sizes(c):
    """(sum edges between nodes, parameter blocks, tables, categories, variables, input blocks per table)."""
    K, f = c["K"], c["family"]
    if f == "hmm":
        nb = c["H"] // K
        return (c["T"] - 1) * c["H"] ** 2 + c["H"], nb * nb + nb, nb, c["V"], c["T"], c["T"]
    if f == "hclt":
        nb = c["M"] // K
        return (c["D"] - 1) * c["M"] ** 2 + c["M"], (c["D"] - 1) * nb * nb + nb, c["D"] * nb, 256, c["D"], 1
    if f == "pd":
        pairs, root = _pd_blocks(c)
        n = int(pairs * c["keep"])
        D = (c["grid"] * c["cell"]) ** 2
        return n * K * K + int(root * c["keep"]) * K, n + int(root * c["keep"]), D * c["M"] // K, 256, D, 1
    if f == "rat":
        nb = c["S"] // K
        n = c["R"] * (2 ** c["depth"] - 2) * nb * nb * nb
        return n * K * K + c["R"] * nb * nb * K, n + c["R"] * nb * nb, c["R"] * c["D"] * nb, 256, c["D"], 1
    nb = c["M"] // K
    n = int(c["sets"] * nb * nb * c["keep"])
    return n * K * K + c["M"], n + nb, c["sets"] * nb, 256, c["sets"], 1


def work(case):
    """Inputs read once and outputs written once.  Of the tables a batch needs the rows of the categories that occur; the
    EM step reads and writes all parameters.  Two operations per edge and sample in the forward pass, four more in the
    backward pass (flows to the children and to the parameters)."""
    E, n_pb, n_tab, n_cats, D, uses = _sizes(case)
    K, B, mode = case["K"], case["B"], case["mode"]
    theta, tables = 4.0 * n_pb * K * K, 4.0 * n_tab * n_cats * K
    rows = 4.0 * n_tab * min(n_cats, B * uses) * K
    data = 4.0 * B * D + (B * D if case["masked"] else 0) + 4.0 * B
    if mode == "em":
        return {"bytes": 2 * (theta + tables) + data, "flops": 6.0 * E * B}
    if mode == "flows":
        return {"bytes": 3 * (theta + rows) + data, "flops": 6.0 * E * B}
    return {"bytes": theta + rows + data, "flops": 2.0 * E * B}


def tolerance(case):
    """fp32 values that went through a logarithm and an exponential per layer: an argument of some 20 nats is held to 1e-6,
    and the errors of the layers (up to a few hundred) add up like a random walk in the flows; a log-likelihood itself is
    large and relatively exact."""
    return {"rel": 1e-5} if case["mode"] in ("forward", "static") else {"rel": 1e-4, "max": 1e-3}


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        f = rng.choice(["hmm", "hmm", "hclt", "hclt", "pd", "rat", "layer"])
        c = dict(family=f, B=_log_int(rng, 1, 512), mode=rng.choice(["forward", "flows", "em"]), masked=rng.random() < 0.25)
        if f == "hmm":
            c["K"] = rng.choice([32, 64, 128])
            c.update(T=_log_int(rng, 8, 64), H=c["K"] * max(1, _log_int(rng, 32, 4096) // c["K"]), V=_log_int(rng, 64, 50257))
        elif f == "hclt":
            c["K"] = rng.choice([32, 64, 128])
            c.update(D=_log_int(rng, 24, 3072), M=c["K"] * max(1, _log_int(rng, 32, 256) // c["K"]))
        elif f == "pd":
            c["K"] = rng.choice([32, 32, 64])
            keep = rng.choice([0.25, 1.0])
            c.update(grid=rng.randint(3, 8), cell=rng.randint(2, 4), M=rng.choice([64, 128, 256] if keep < 1 else [64, 128]), keep=keep,
                     scratch=rng.random() < 0.2)
        elif f == "rat":
            c["K"] = rng.choice([32, 32, 64])
            c.update(D=_log_int(rng, 64, 784), depth=rng.randint(2, 4), R=rng.randint(1, 4), S=rng.choice([64, 128, 256]))
        else:
            c["K"] = rng.choice([8, 16, 32, 64])
            c.update(sets=_log_int(rng, 3, 200), M=rng.choice([128, 256, 512, 1024]), keep=rng.choice([0.1, 0.3, 1.0]))
        if f != "hmm":
            c["tree"] = rng.randrange(1 << 30)
        if _cost(c) <= most:
            return c


# ---- structures, parameters, data ----
@functools.lru_cache(maxsize=1)
def _structure(key):
    c = dict(key)
    K = c["K"]
    if c["family"] == "hmm":
        w = W.hmm(c["T"], c["H"], c["V"], K, 1, 0, draw=False)
    elif c["family"] == "hclt":
        w = W.hclt(c["D"], c["M"], K, 1, c["tree"], draw=False)
    elif c["family"] == "pd":
        w = W.pd(c["grid"], c["cell"], c["M"], K, 1, c["tree"], keep=c["keep"], draw=False)
    elif c["family"] == "rat":
        w = W.rat_spn(c["D"], c["depth"], c["R"], c["S"], K, 1, c["tree"], draw=False)
    else:
        w = W.sum_layer(c["sets"], c["M"], K, 1, c["tree"], keep=c["keep"], draw=False)
    return pcb.pc_order_for_scratch(w) if c.get("scratch") else w


def _random_rows(shape, alpha, gen):
    """Unnormalised Dirichlet(alpha) draws."""
    t = torch.empty(shape, dtype=torch.float32, device="cuda")
    return t.exponential_(generator=gen) if alpha == 1.0 else torch._standard_gamma(t.fill_(alpha), generator=gen)


def _fill_parameters(c, w, alpha, gen):
    """Every sum node's weights over all its children, and every input node's table over the categories, add up to one."""
    K = w.K
    sums = np.nonzero(w.type == W.SUM)[0]
    first = {}                                             # parameter-block list (by its first id) -> (length, real rows)
    for u in sums:
        e0, e1 = int(w.child_ptr[u]), int(w.child_ptr[u + 1])
        first.setdefault(int(w.param_blk[e0]), (e1 - e0, int(w.n_real[u])))
    starts = sorted(first)                                 # the lists are consecutive ids and cover all blocks
    lens = torch.tensor([first[s][0] for s in starts], device="cuda")
    real = torch.tensor([first[s][1] for s in starts], device="cuda")
    theta = c.theta.view(-1, K, K)
    raw = _random_rows(theta[1:].shape, alpha, gen)
    z = torch.segment_reduce(raw.sum(dim=2), "sum", lengths=lens, axis=0)
    of = torch.repeat_interleave(torch.arange(len(starts), device="cuda"), lens)
    raw /= z[of][:, :, None]
    raw.clamp_(min=FLT_MIN)
    raw *= (torch.arange(K, device="cuda")[None, :] < real[of][:, None])[:, :, None]
    theta[1:].copy_(raw)
    del raw
    tables = c.tables.view(w.n_tables, w.n_cats, K)
    raw = _random_rows(tables.shape, alpha, gen)
    raw /= raw.sum(dim=1, keepdim=True)
    torch.clamp(raw, min=FLT_MIN, out=tables)


def _data(case, w, gen):
    """Zipf tokens for the language models, per-variable Gaussian grey values for the image models, uniform ones elsewhere."""
    B, D, n = case["B"], w.n_vars, w.n_cats
    if case["family"] == "hmm" and n >= 1000:
        cdf = torch.cumsum((torch.arange(n, dtype=torch.float64) + 1.0) ** -1.1, 0)
        u = torch.rand((B, D), generator=gen, dtype=torch.float64) * cdf[-1]
        return torch.searchsorted(cdf, u, right=True).clamp_(max=n - 1)
    if case["family"] in ("hclt", "rat"):
        mu = torch.rand((1, D), generator=gen) * (n - 1)
        return (mu + torch.randn((B, D), generator=gen) * (40.0 * n / 256.0)).round_().clamp_(0, n - 1)
    return torch.randint(0, n, (B, D), generator=gen)


def prepare(case, seed):
    """A compiled circuit with its parameters, zeroed flows and one batch on the GPU."""
    w = _structure(tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "B", "mode", "masked"))))
    c = pcb.Circuit(w)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    host = torch.Generator().manual_seed(seed)
    _fill_parameters(c, w, 0.1 if case["family"] == "hmm" and case["V"] >= 1000 else 1.0, gen)
    x = _data(case, w, host).to(torch.int32).numpy()
    mask = (torch.rand(x.shape, generator=host) < 0.3).numpy().astype(np.uint8) if case["masked"] else None
    c.set_batch(x, mask)
    return {"circuit": c, "mode": case["mode"]}


def run(state):
    c, mode = state["circuit"], state["mode"]
    if mode == "static":
        pcb.pc_forward_static(c.handle, c.theta, c.tables, c.x, c.mask, c.B, c.ll)
        return {"ll": c.ll}
    ll = c.forward()
    if mode == "forward":
        return {"ll": ll}
    c.backward()
    if mode == "em":
        c.em_step(0.1, 0.01)
        return {"ll": ll, "theta": c.theta, "tables": c.tables, "theta_flow": c.theta_flow, "table_flow": c.table_flow}
    return {"ll": ll, "theta_flow": c.theta_flow, "table_flow": c.table_flow}
