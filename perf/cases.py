"""Performance cases of the PASA forward: what a video DiT (or the tools around it) calls, through the public
entry points of ``paper_2604_12219_amd``, from the tiny check to the 720p and long-video launches.

The cases come from the repository's workloads (``workloads.WORKLOADS``, the 50-step budget schedule) and its tests;
inputs are the synthetic video tensors of ``workloads.make_qkv`` (white noise plus a smooth field), drawn from the seed.

``path`` of a case:
  forward  pasa.forward with the buffers a denoising loop keeps                       -> out, idx
  single   pasa_forward: the whole path in one library call, one workspace            -> out, lse
  stages   the stage entry points with the covariance prior of the routing logit      -> out, lse, idx
  dense    pasa_attn_dense_ref, the steps before the sparse ones (dense prefix)       -> out, lse
  select   scoring and routing alone, as the selection studies run them               -> scores, idx, mask
  static   pasa_sparse_attn_fwd_static on a caller's index lists (no bitmap)          -> out, lse
  l1       pasa_l1_distance, the calibration signal of the budget                     -> scalar
"""
import ctypes
import math

import torch

import paper_2604_12219_amd as P
import workloads

AMP = 0.125  # routing noise of the benchmark, in logit units


def _case(path, frames, rows, cols, heads, d=128, block=64, group=32, keep=0.15, batch=1, noise=1.0, token_major=False,
          gumbel=False, dtype="bf16"):
    return {"path": path, "frames": frames, "rows": rows, "cols": cols, "heads": heads, "d": d, "block": block, "group": group,
            "keep": keep, "batch": batch, "noise": noise, "token_major": token_major, "gumbel": gumbel, "dtype": dtype}


def listed():
    cases = {
        # the tiny workload: what the smoke check and a first try run; launches and host work count here
        "tiny-forward": _case("forward", 4, 16, 16, 2, d=64, keep=0.25),
        # a short clip: two prompts (classifier-free guidance), head dimension 64, ragged everywhere, the dense steps
        "short-dense-d64": _case("dense", 5, 21, 13, 3, d=64, batch=2),
        # a caller with index lists of its own and no allocation allowed (graph capture), two-chunk groups
        "static-lists": _case("static", 9, 20, 23, 4, group=64, keep=0.15),
        # the first sparse steps of a Wan 2.1 1.3B 480p generation
        "wan1.3b-480p": _case("forward", 21, 30, 52, 12, keep=0.20),
        # late steps of its budget schedule: low density, smooth inputs
        "wan1.3b-480p-late": _case("single", 21, 30, 52, 12, keep=0.10, noise=0.2),
        # the dense prefix of the same generation (a fifth of the steps)
        "wan1.3b-480p-dense": _case("dense", 21, 30, 52, 12),
        # the selection studies (routing noise, histogram) run scoring and routing only
        "select-480p": _case("select", 21, 30, 52, 12, keep=0.20, gumbel=True),
        # the calibration signal between two velocity fields (64 values a token)
        "l1-480p": _case("l1", 21, 30, 52, 1, d=64),
        # one rank's share (40 heads on 8 GPUs) of Wan 2.1 14B 720p, token-major storage as a transformer hands it over,
        # full routing logit of Eq.8
        "wan14b-720p-rank": _case("stages", 21, 45, 80, 5, keep=0.15, token_major=True),
        # the headline: Wan 2.1 14B 720p on one GPU
        "wan14b-720p": _case("single", 21, 45, 80, 40, keep=0.15),
        # one rank's share (24 heads on 8 GPUs) of HunyuanVideo 13B 720p, 64 blocks per group
        "hunyuan13b-720p-rank": _case("forward", 33, 45, 80, 3, group=64, keep=0.15),
        # long video: coarse blocks, very sparse
        "long-video": _case("single", 41, 45, 80, 40, block=128, keep=0.05),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = work(next(c for c in listed() if c["name"] == "long-video"))["flops"]
    path = rng.choice(["forward", "single", "stages", "dense", "select", "static", "forward", "single", "stages", "dense", "l1"])
    while True:
        n = _log_uniform(rng, 256, 147600)
        frames = max(1, min(41, int(round(n ** (1 / 3) * rng.uniform(0.3, 0.9)))))
        rows = max(4, int(round(math.sqrt(n / frames) * rng.uniform(0.6, 1.0))))
        cols = max(4, n // (frames * rows))
        c = _case(path, frames, rows, cols, _log_uniform(rng, 1, 40), d=rng.choice([64, 128, 128]), block=rng.choice([64, 64, 128]),
                  group=rng.choice([32, 32, 32, 64, 16]), keep=round(math.exp(rng.uniform(math.log(0.05), math.log(0.40))), 3),
                  batch=rng.choice([1, 1, 2]), noise=round(rng.uniform(0.2, 1.0), 2), token_major=rng.random() < 0.4,
                  gumbel=path in ("stages", "select") and rng.random() < 0.4, dtype="f32" if path == "l1" and rng.random() < 0.5 else "bf16")
        c["token_major"] = c["token_major"] and path != "l1"
        nb = -(-_n(c) // c["block"])
        if work(c)["flops"] > limit or nb > 4096 or c["batch"] * c["heads"] > 48:
            continue
        if path == "static" and P.attn_workspace_bytes(_shape_of_case(c)) > P.STATIC_SCRATCH_BYTES:
            continue
        return c


def _n(c):
    return c["frames"] * c["rows"] * c["cols"]


def _shape_of_case(c):
    n, d = _n(c), c["d"]
    return P.Shape(c["batch"], c["heads"], n, d, c["block"], c["group"], c["heads"] * n * d, n * d, d)


def prepare(case, seed):
    c = case
    grid, dev = (c["frames"], c["rows"], c["cols"]), "cuda"
    if c["path"] == "l1":  # velocity fields of two consecutive steps, [batch, tokens, values]
        g = torch.Generator(device=dev)
        g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
        size = (c["batch"], _n(c), c["d"])
        a = torch.randn(size, generator=g, device=dev)
        b = a + 0.1 * torch.randn(size, generator=g, device=dev)
        dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        return {"case": c, "a": a.to(dtype), "b": b.to(dtype), "ws": torch.empty(1 << 14, dtype=torch.uint8, device=dev)}
    q, k, v = workloads.make_qkv(grid, c["heads"], c["d"], seed=int(seed), noise_amplitude=c["noise"], device=dev, batch=c["batch"])
    if c["token_major"]:  # [B, H, n, d] views of [B, n, H, d] storage
        q, k, v = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (q, k, v))
    shape = P.Shape.of(q, block=c["block"], group=c["group"])
    bh = shape.B * shape.H
    s = {"case": c, "q": q, "k": k, "v": v, "shape": shape, "seed": int(seed) & 0xFFFFFFFF}
    if c["path"] == "forward":
        s["buffers"] = {}
        return s
    nb = P.num_blocks(shape)
    k_sel = P.topk_count(nb, c["keep"])
    s["k_sel"] = k_sel
    if c["path"] != "select":
        s["out"] = torch.empty_like(q)
        s["lse"] = torch.empty((bh, shape.n), dtype=torch.float32, device=dev)
    if c["path"] == "single":
        size = int(P.load_library().pasa_forward_workspace_bytes(ctypes.byref(shape.c()), c["keep"]))
        s["ws"] = torch.empty(size, dtype=torch.uint8, device=dev)
    elif c["path"] in ("dense", "stages"):
        s["ws"] = torch.empty(P.attn_workspace_bytes(shape), dtype=torch.uint8, device=dev)
    if c["path"] in ("stages", "select"):
        s["scores"] = torch.empty((bh, nb, nb), dtype=torch.float32, device=dev)
        s["idx"] = torch.empty((bh, nb, k_sel), dtype=torch.int32, device=dev)
        s["mask"] = torch.empty((bh, nb, P.mask_words(nb)), dtype=torch.int32, device=dev)
        s["ws_score"] = torch.empty(P.score_workspace_bytes(shape), dtype=torch.uint8, device=dev)
        s["beta"] = torch.empty((bh, nb), dtype=torch.float32, device=dev)
    if c["path"] == "static":  # the caller's own selection
        s["idx"], _ = P.route(P.block_score(q, k, shape), k_sel, s["seed"], AMP)
    return s


def run(state):
    s, c = state, state["case"]
    path = c["path"]
    if path == "l1":
        return P.l1_distance(s["a"], s["b"], ws=s["ws"])
    q, k, v, shape = s["q"], s["k"], s["v"], s["shape"]
    if path == "forward":
        return P.forward(q, k, v, c["keep"], s["seed"], AMP, block=c["block"], group=c["group"], buffers=s["buffers"])
    if path == "single":
        return P.forward_single_call(q, k, v, shape, c["keep"], s["seed"], AMP, out=s["out"], lse=s["lse"], ws=s["ws"], want_lse=True)
    if path == "dense":
        return P.attn_dense_ref(q, k, v, shape, out=s["out"], lse=s["lse"], ws=s["ws"], want_lse=True)
    if path == "static":
        P.sparse_attn_fwd_static(q, k, v, shape, s["idx"], None, s["out"], lse=s["lse"])
        return s["out"], s["lse"]
    noise = "gumbel" if c["gumbel"] else "uniform"
    if path == "select":
        P.block_score(q, k, shape, scores=s["scores"], ws=s["ws_score"])
        idx, mask = P.route(s["scores"], s["k_sel"], s["seed"], AMP, idx=s["idx"], mask=s["mask"], noise=noise)
        return s["scores"], idx, mask
    P.kv_stats(k, v, shape, ws=s["ws"])
    P.key_prior(k, v, shape, s["ws"], beta=s["beta"])
    P.block_score(q, k, shape, key_bias=s["beta"], scores=s["scores"], ws=s["ws_score"], stats_ws=s["ws"])
    P.route(s["scores"], s["k_sel"], s["seed"], AMP, idx=s["idx"], mask=s["mask"], noise=noise)
    P.sparse_attn_fwd(q, k, v, shape, s["idx"], s["mask"], out=s["out"], lse=s["lse"], ws=s["ws"], want_lse=True, prepared=True)
    return s["out"], s["lse"], s["idx"]


def work(case):
    c, path = case, case["path"]
    n, d, b = _n(c), c["d"], c["block"]
    bh = c["batch"] * c["heads"]
    if path == "l1":
        return {"bytes": 2 * c["batch"] * n * d * (2 if c["dtype"] == "bf16" else 4), "flops": 3 * c["batch"] * n * d}
    tensor = bh * n * d * 2  # one of Q, K, V, O
    if path == "dense":
        return {"bytes": 4 * tensor + 4 * bh * n, "flops": 4 * bh * n * n * d}
    nb = -(-n // b)
    k = max(1, min(nb, int(c["keep"] * nb + 0.5)))
    selection = 4 * bh * nb * (k + -(-nb // 32))
    scoring = 2 * bh * nb * nb * d
    if path == "select":
        return {"bytes": 2 * tensor + 4 * bh * nb * nb + selection, "flops": scoring + 2 * bh * n * d}
    groups = -(-nb // c["group"])
    # exact tiles, zeroth order (mean keys, value sums), first order (one d x d matrix per group), statistics (K^T V)
    attention = bh * nb * (4 * k * b * b * d + 4 * b * nb * d + 2 * groups * b * d * d) + 2 * bh * n * d * d
    if path == "static":
        return {"bytes": 4 * tensor + 4 * bh * (n + nb * k), "flops": attention}
    if path == "stages":  # the prior needs the statistics of every block on its own
        return {"bytes": 4 * tensor + 4 * bh * n + 4 * bh * nb * nb + selection, "flops": attention + scoring + 3 * bh * nb * d * d}
    extra = 4 * bh * nb * k if path == "forward" else 4 * bh * n
    return {"bytes": 4 * tensor + extra, "flops": attention + scoring}


def _philox(ctr, key):
    """Philox4x32-10 of int64 tensors holding 32-bit words, ctr = 4 words, key = 2 ints -> 4 words"""
    low = 0xFFFFFFFF
    c, (k0, k1) = list(ctr), key
    for _ in range(10):
        # the 64-bit product of two 32-bit words from two 48-bit ones (int64 would overflow)
        hi, lo = [], []
        for m, x in ((0xD2511F53, c[0]), (0xCD9E8D57, c[2])):
            a, b = m * (x & 0xFFFF), m * (x >> 16)
            t = a + ((b & 0xFFFF) << 16)
            lo.append(t & low)
            hi.append((b >> 16) + (t >> 32))
        c = [hi[1] ^ c[1] ^ k0, lo[1], hi[0] ^ c[3] ^ k1, lo[0]]
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return c


def _select(scores, head, k_sel, seed, gumbel):
    """the k_sel largest of one head's logits plus the seeded bias -> ascending block numbers per row"""
    nb = scores.shape[0]
    i = torch.arange(nb, device=scores.device)[:, None].expand(nb, -(-nb // 4))
    j4 = torch.arange(-(-nb // 4), device=scores.device)[None, :].expand_as(i)
    words = _philox((j4, i, torch.full_like(i, head), torch.zeros_like(i)), (seed, 0))
    u = torch.stack(words, dim=-1).reshape(nb, -1)[:, :nb]
    if gumbel:
        bias = -torch.log(-torch.log(((u >> 9).double() + 0.5) * 2.0 ** -23))
    else:
        bias = ((torch.where(u >= 2 ** 31, u - 2 ** 32, u)) >> 8).double() * 2.0 ** -23
    top = torch.sort(scores + AMP * bias, dim=1, descending=True, stable=True).indices[:, :k_sel]
    return torch.sort(top, dim=1).values


def exact(case, seed):
    """What run() returns, in 64 bits, straight from the definition of the path (None where that takes too long)."""
    c, path = case, case["path"]
    if work(c)["flops"] > 8e12:
        return None
    s = prepare(c, seed)
    if path == "l1":
        return (s["a"].double() - s["b"].double()).abs().mean().reshape(1)
    q4, k4, v4 = s["q"], s["k"], s["v"]
    n, d, b, B, H = _n(c), c["d"], c["block"], c["batch"], c["heads"]
    nb, scale, dev = -(-n // b), c["d"] ** -0.5, q4.device
    pad = nb * b - n
    size = torch.full((nb,), b, dtype=torch.float64, device=dev)
    size[-1] = b - pad
    group = min(c["group"], nb)
    k_sel = max(1, min(nb, int(c["keep"] * nb + 0.5)))
    bits = 2 ** torch.arange(32, device=dev)
    outs, lses, all_scores, lists, masks = [], [], [], [], []
    for head in range(B * H):
        # [blocks, tokens of a block, d], zero beyond the last token
        q, k, v = (torch.nn.functional.pad(t[head // H, head % H].double(), (0, 0, 0, pad)).view(nb, b, d) for t in (q4, k4, v4))
        if path == "dense":
            o, l = [], []
            for r in range(0, n, 1024):
                z = q.view(-1, d)[r:min(r + 1024, n)] @ k.view(-1, d)[:n].T * scale
                l.append(torch.logsumexp(z, dim=1))
                o.append(torch.exp(z - l[-1][:, None]) @ v.view(-1, d)[:n])
            outs.append(torch.cat(o))
            lses.append(torch.cat(l))
            continue
        kbar, vsum = k.sum(1) / size[:, None], v.sum(1)
        scores = (q.sum(1) / size[:, None]) @ kbar.T * scale
        if path != "select":
            cov = k.transpose(1, 2) @ v - kbar[:, :, None] * vsum[:, None, :]
            of_group = torch.arange(nb, device=dev) // group
            n_groups = int(of_group[-1]) + 1
            member = torch.nn.functional.one_hot(of_group, n_groups).double()
            mean_cov = (member.T @ cov.reshape(nb, -1) / member.sum(0)[:, None]).view(n_groups, d, d)
            if path == "stages":
                scores = scores + torch.log((cov - mean_cov[of_group]).flatten(1).norm(dim=1) + 1e-6)
            del cov
        idx = s["idx"].view(B * H, nb, k_sel)[head].long() if path == "static" else _select(scores, head, k_sel, s["seed"], c["gumbel"])
        lists.append(idx)
        chosen = torch.zeros((nb, -(-nb // 32) * 32), dtype=torch.bool, device=dev)
        chosen.scatter_(1, idx, True)
        if path == "select":
            word = (chosen.view(nb, -1, 32) * bits).sum(-1)
            masks.append(torch.where(word >= 2 ** 31, word - 2 ** 32, word).to(torch.int32))
            all_scores.append(scores)
            continue
        ragged = torch.arange(nb * b, device=dev).view(nb, b) >= n
        o, l = [], []
        step = max(1, int(2 ** 26 / (k_sel * b * d)))
        for r in range(0, nb, step):
            rows, qr = idx[r:r + step], q[r:r + step] * scale
            m = rows.shape[0]
            z = qr @ k[rows].view(m, -1, d).transpose(1, 2)
            z = z.masked_fill(ragged[rows].view(m, 1, -1), -math.inf)
            za = (qr @ kbar.T).masked_fill(chosen[r:r + step, None, :nb], -math.inf)
            top = torch.maximum(z.amax(-1), za.amax(-1))[..., None]
            p, a = torch.exp(z - top), torch.exp(za - top)
            den = p.sum(-1) + a @ size
            num = p @ v[rows].view(m, -1, d) + a @ vsum
            weight = a @ member
            for g in range(n_groups):
                num += weight[..., g:g + 1] * (qr @ mean_cov[g])
            o.append(num / den[..., None])
            l.append(top[..., 0] + torch.log(den))
        outs.append(torch.cat(o).view(-1, d)[:n])
        lses.append(torch.cat(l).view(-1)[:n])
    if path == "select":
        return torch.stack(all_scores), torch.stack(lists).int(), torch.stack(masks)
    out = torch.stack(outs).view(B, H, n, d)
    if path == "forward":
        return out, torch.stack(lists).int()
    if path == "stages":
        return out, torch.stack(lses), torch.stack(lists).int()
    return out, torch.stack(lses)


def tolerance(case):
    """About four times what was measured: outputs against the fp64 oracle (2-norm 1.7e-3, largest 6e-3) and against the
    same path summed in another order (key-range slices: 6e-4, largest 8e-3); bf16 rounding of P and O sets both."""
    if case["path"] == "l1":
        return {"rel": 1e-6}  # fp32 partial sums, double in the last stage: 2e-8 seen against double throughout
    if case["path"] == "select":
        # key means summed on the vector unit or on the matrix cores: 2e-8, largest 4e-6; no selection differed
        return {"rel": 1e-6, "max": 5e-5, "differ": 1e-3}
    return {"rel": 8e-3, "max": 4e-2, "differ": 1e-3}
