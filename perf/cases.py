"""The work a user has this library do, as timed cases.

A case is one call sequence through the public entry points of
paper_2412_09764_amd at one size.  `do` names the sequence:

  infer            mem_search (or its variant) + the value bag, outputs and
                   workspace kept by the caller: a decode or prefill step
  train            search, value bag, and every backward of one memory layer:
                   value gradient, score gradient, queries, sub-keys (with the
                   gate's, the query normalisation's or the sink's when on)
  search           the product-key search on its own, outputs allocated by the call
  bag_backward     the value backward with touched rows only (large tables)
  search_backward  the gradients into queries and sub-keys on their own

Options: `gate` (Memory+), `qnorm` (query normalisation), `r` (extra pairs per
token and head), `sink` (a fixed pair per head), `query` (distribution of the
queries), `dtype`.  Sizes follow this library's own workloads: 4K to 64M keys,
value dims 64 to 2048, 1 to 8 heads, k 1 to 64.
"""
import math

import torch

import paper_2412_09764_amd as pk

GIB = 1 << 30
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, do, T, S, H, n, D, k, dtype="bf16", query="normal", gate=False, qnorm=False, r=0,
          sink=False):
    c = dict(do=do, T=T, S=S, H=H, n=n, D=D, k=k, dtype=dtype, query=query, gate=gate, qnorm=qnorm,
             r=r, sink=sink)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # one token of one sequence decoded: the smallest serving call, 1M keys
        _case("decode_t1", "infer", 1, 1024, 4, 512, 1024, 32),
        # a batch of 32 sequences decoded through a Memory+ layer, 4M keys x 2048
        _case("decode_t32_gated", "infer", 32, 2048, 4, 512, 2048, 32, gate=True),
        # one prompt of 2000 tokens (ragged) prefilled through the same layer
        _case("prefill_t2000_gated", "infer", 2000, 2048, 4, 512, 2048, 32, gate=True),
        # fp32 model, odd sizes, the largest k (64 of 300 per half)
        _case("infer_f32_t777_k64", "infer", 777, 300, 2, 96, 200, 64, dtype="f32"),
        # the forward of the 4M-key training workload: 8 sequences x 4096 tokens
        _case("forward_4m_t32768", "infer", 32768, 2048, 4, 512, 2048, 32),
        # the largest sub-key tables (64M keys), clustered queries
        _case("search_64m_t8192", "search", 8192, 8192, 4, 512, 256, 32, query="clusters"),
        # the small fp32 configuration, a whole training step
        _case("train_f32_t256", "train", 256, 64, 1, 64, 64, 8, dtype="f32"),
        # a micro-batch of 512 tokens, 256K values x 2048, Memory+ layer
        _case("train_t512_gated", "train", 512, 512, 4, 512, 2048, 32, gate=True),
        # odd sizes everywhere, extra pairs and the sink of the model ablations
        _case("train_t3001_sink", "train", 3001, 700, 3, 320, 640, 17, r=6, sink=True),
        # the 1M-key training workload: 16384 tokens, normalised queries, Memory+ layer
        _case("train_1m_t16384", "train", 16384, 1024, 4, 512, 1024, 32, gate=True, qnorm=True),
        # value gradient as touched rows of a 16 GiB table (its dense gradient is 32 GiB)
        _case("bag_bwd_4m_t4096", "bag_backward", 4096, 2048, 4, 512, 2048, 32),
        # key gradients of the 4M-key training workload
        _case("search_bwd_4m_t32768", "search_backward", 32768, 2048, 4, 512, 2048, 32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        do = rng.choice(["infer", "infer", "infer", "train", "train", "search", "bag_backward",
                         "search_backward"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        T = _log(rng, 1, 32768) if do in ("infer", "search") else _log(rng, 64, 32768)
        S = _log(rng, 64, 2400 if do != "search" else 8192)
        if rng.random() < 0.4:
            S = max(64, 1 << int(round(math.log2(S))))
        H = rng.choice([1, 2, 3, 4, 4, 8])
        if dtype == "bf16":
            d = rng.choice([32, 64, 96, 128, 160, 256, 256, 8 * rng.randint(4, 32)])
        else:
            d = rng.choice([16, 32, 48, 64, 4 * rng.randint(4, 16)])
        D = rng.choice([64, 128, 256, 512, 1024, 2048, 8 * rng.randint(8, 256)])
        k = rng.choice([8, 16, 32, 32, 32, 64, rng.randint(1, 48)])
        sink = do in ("infer", "train", "search") and rng.random() < 0.15
        r = rng.randint(1, 16) if do in ("infer", "train", "search") and rng.random() < 0.15 else 0
        qnorm = not sink and not r and do != "bag_backward" and rng.random() < 0.25
        gate = do in ("infer", "train") and rng.random() < 0.4
        query = rng.choice(["normal", "normal", "layernorm", "clusters"])
        if k + r + sink > 64:
            continue
        esz = 4 if dtype == "f32" else 2
        if D * esz > 8192:
            continue
        c = _case(None, do, T, S, H, 2 * d, D, k, dtype, query, gate, qnorm, r, sink)
        L = T * H * (k + r + sink)
        table = 0 if do in ("search", "search_backward") else (S * S + H) * D
        if table * esz > 16 * GIB or (do == "train" and table * 4 > 4 * GIB):
            continue
        # no larger than the listed ones: lookups x row bytes, scores, score products
        if L * D * esz * (1 if do == "infer" else 4 if do == "train" else 2) > 16 * GIB:
            continue
        if do != "infer" and L > 1 << 22 or T * H * S * d > 32768 * 4 * 2048 * 256:
            continue
        if dtype == "f32" and T * H * S * d > 8192 * 4 * 2048 * 64:
            continue
        if table and do != "train" and do != "infer" and L * D * 4 > 5 * GIB:
            continue
        return c


def _kk(c):
    return c["k"] + c["r"] + (1 if c["sink"] else 0)


def _touched(L, N):
    """Distinct rows that L uniform lookups into N rows take, on average."""
    return max(1, int(round(-N * math.expm1(-L / N))))


def _queries(c, g, dev):
    T, H, n = c["T"], c["H"], c["n"]
    x = torch.randn((T, H, n), generator=g, device=dev)
    if c["query"] == "layernorm":
        x = torch.nn.functional.layer_norm(x, (n,), eps=1e-5)
    elif c["query"] == "clusters":
        centres = torch.randn((64, H, n), generator=g, device=dev)
        ids = torch.randint(0, 64, (T,), generator=g, device=dev)
        x = centres[ids] + 0.1 * x
    if c["qnorm"]:
        x = 2.0 * x + 0.5  # not normalised by the caller: the search does it
    return x.to(DT[c["dtype"]]).contiguous()


def _select(q, K, k):
    """Product-key selection in plain torch: (idx [T,H,k], softmax weights)."""
    T, H, n = q.shape
    S, d = K.shape[2], K.shape[3]
    idx = torch.empty((T, H, k), dtype=torch.int64, device=q.device)
    w = torch.empty((T, H, k), dtype=torch.float32, device=q.device)
    for t0 in range(0, T, 8192):
        t1 = min(T, t0 + 8192)
        for h in range(H):
            s, i = [], []
            for p in range(2):
                z = q[t0:t1, h, p * d:(p + 1) * d].float() @ K[h, p].float().t().contiguous()
                v, j = torch.topk(z, k, dim=1)
                s.append(v)
                i.append(j)
            z = (s[0][:, :, None] + s[1][:, None, :]).reshape(t1 - t0, k * k)
            v, j = torch.topk(z, k, dim=1)
            idx[t0:t1, h] = torch.gather(i[0], 1, j // k) * S + torch.gather(i[1], 1, j % k)
            w[t0:t1, h] = torch.softmax(v, dim=1)
    return idx, w


def prepare(case, seed):
    c, dev = case, torch.device("cuda")
    T, S, H, n, D, k = (c[x] for x in ("T", "S", "H", "n", "D", "k"))
    dt, d, kk, do = DT[c["dtype"]], c["n"] // 2, _kk(c), c["do"]
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    st = {"case": dict(c)}
    q = st["q"] = _queries(c, g, dev)
    # scores of spread about one, as trained keys give
    std = 1.0 / math.sqrt(2 * d) if c["dtype"] == "bf16" else 1.0 / math.sqrt(d)
    K = st["K"] = (torch.randn((H, 2, S, d), generator=g, device=dev) * std).to(dt)
    if c["sink"]:
        st["sink_keys"] = (torch.randn((H, n), generator=g, device=dev) * std).to(dt)
    if c["r"]:
        st["extra"] = torch.randint(0, S * S, (T, H, c["r"]), generator=g, device=dev)
    if do in ("infer", "train", "bag_backward"):
        rows = S * S + (H if c["sink"] else 0)
        st["V"] = torch.empty((rows, D), dtype=dt, device=dev).normal_(0.0, 0.02, generator=g)
    if c["gate"]:
        st["gate"] = torch.randn((T, D), generator=g, device=dev).to(dt)
    if do in ("train", "bag_backward"):
        st["dy"] = torch.randn((T, D), generator=g, device=dev).to(dt)
    if do == "bag_backward":
        # U distinct rows (as many as L uniform lookups touch), each taken at
        # least once, the other lookups skewed towards some of them; in random order
        L, N = T * H * k, S * S
        U = min(L, _touched(L, N))
        pool = torch.randperm(N, generator=g, device=dev)[:U]
        more = pool[(U * torch.rand(L - U, generator=g, device=dev, dtype=torch.float64) ** 2).long()]
        order = torch.randperm(L, generator=g, device=dev)
        st["idx"] = torch.cat([pool, more])[order].reshape(T, H, k)
        st["w"] = torch.softmax(torch.randn((T, H, k), generator=g, device=dev), dim=-1)
    if do == "search_backward":
        qs = q
        if c["qnorm"]:
            qs = torch.nn.functional.layer_norm(q.float(), (n,), eps=1e-5).to(dt)
        st["idx"], st["w"] = _select(qs, K, k)
        st["gz"] = torch.randn((T, H, k), generator=g, device=dev) * st["w"]

    u8 = dict(dtype=torch.uint8, device=dev)
    if do in ("infer", "train", "search"):
        nb = pk.mem_search_workspace_size(T, H, S, k)
        plain = not (c["qnorm"] or c["r"] or c["sink"])
        st["noalloc"] = do == "infer" and plain and nb <= pk.NOALLOC_SCRATCH_BYTES
        if not st["noalloc"]:
            st["ws"] = torch.empty(nb, **u8)
    if do == "infer":
        st["idx"] = torch.empty((T, H, kk), dtype=torch.int64, device=dev)
        st["w"] = torch.empty((T, H, kk), dtype=torch.float32, device=dev)
        st["out"] = torch.empty((T, D), dtype=dt, device=dev)
    if do in ("train", "bag_backward"):
        mode = "auto" if do == "train" else "sorted"
        nb = pk.mem_bag_backward_workspace_size(T, H, kk, st["V"].shape[0], D, mode)
        st["bws"] = torch.empty(nb, **u8)
    if do in ("train", "search_backward"):
        L = pk.load()
        if c["sink"]:
            nb = int(L.mem_search_backward_sink_workspace_size(T, H, n, S, kk - 1))
        else:
            nb = int(L.mem_search_backward_workspace_size(T, H, S, kk))
        st["sws"] = torch.empty(nb, **u8)
        st["gK"] = torch.zeros((H, 2, S, d), dtype=torch.float32, device=dev)
    if do == "train":
        st["gV"] = torch.zeros((st["V"].shape[0], D), dtype=torch.float32, device=dev)
        if c["sink"]:
            st["gsink"] = torch.zeros((H, n), dtype=torch.float32, device=dev)
    return st


def _search(st, idx=None, w=None, want_score=False):
    c, k = st["case"], st["case"]["k"]
    q, K = st["q"], st["K"]
    o = dict(idx_out=idx, w_out=w, want_score=want_score)
    if st["noalloc"]:
        return pk.mem_search_noalloc(q, K, k, **o)
    o["workspace"] = st["ws"]
    if c["sink"]:
        return pk.mem_search_sink(q, K, k, st["sink_keys"], c["S"] * c["S"], st.get("extra"), **o)
    if c["r"]:
        return pk.mem_search_extra(q, K, k, st["extra"], **o)
    if c["qnorm"]:
        return pk.mem_search_qnorm(q, K, k, 1e-5, **o)
    return pk.mem_search(q, K, k, **o)


def run(st):
    c = st["case"]
    do = c["do"]
    if do == "infer":
        idx, w = _search(st, st["idx"], st["w"])[:2]
        if c["gate"]:
            out, _ = pk.mem_bag_forward_gated(st["V"], idx, w, st["gate"], want_y=False,
                                              out=st["out"])
        else:
            out = pk.mem_bag_forward(st["V"], idx, w, y_out=st["out"])
        return {"out": out, "w": w}
    if do == "search":
        idx, w, score = _search(st, want_score=True)[:3]
        return {"idx": idx, "w": w, "score": score}
    if do == "bag_backward":
        rows, grad_rows, _, gz = pk.mem_bag_backward_sparse(
            st["dy"], st["V"], st["idx"], st["w"], want_grad_w=False, workspace=st["bws"])
        return {"rows": rows, "grad_rows": grad_rows, "grad_scores": gz}
    if do == "search_backward":
        f = pk.mem_search_backward_qnorm if c["qnorm"] else pk.mem_search_backward
        gq, gK = f(st["q"], st["K"], st["idx"], st["gz"], grad_subkeys=st["gK"],
                   workspace=st["sws"])
        return {"grad_q": gq, "grad_subkeys": gK}
    # train: one memory layer forward and backward
    idx, w = _search(st)[:2]
    res = {}
    if c["gate"]:
        out, y = pk.mem_bag_forward_gated(st["V"], idx, w, st["gate"])
        dy, res["grad_gate"] = pk.mem_gate_backward(st["dy"], st["gate"], y)
    else:
        out, dy = pk.mem_bag_forward(st["V"], idx, w), st["dy"]
    gV, _, gz = pk.mem_bag_backward(dy, st["V"], idx, w, grad_values=st["gV"], want_grad_w=False,
                                    workspace=st["bws"])
    o = dict(grad_subkeys=st["gK"], workspace=st["sws"])
    if c["sink"]:
        gq, gK, res["grad_sink"] = pk.mem_search_backward_sink(
            st["q"], st["K"], idx, gz, st["sink_keys"], grad_sink=st["gsink"], **o)
    elif c["qnorm"]:
        gq, gK = pk.mem_search_backward_qnorm(st["q"], st["K"], idx, gz, 1e-5, **o)
    else:
        gq, gK = pk.mem_search_backward(st["q"], st["K"], idx, gz, **o)
    res.update(out=out, grad_values=gV, grad_q=gq, grad_subkeys=gK)
    return res


def work(case):
    c = case
    T, S, H, n, D, k, kk = *(c[x] for x in ("T", "S", "H", "n", "D", "k")), _kk(c)
    e, do, d = (4 if c["dtype"] == "f32" else 2), c["do"], c["n"] // 2
    L, N = T * H * kk, S * S
    U = _touched(L, N)
    keys = H * 2 * S * d
    b = f = 0.0
    if do in ("infer", "search", "train"):
        b += T * H * n * e + keys * e + 12 * L + 8 * T * H * c["r"] + (4 * L if do == "search" else 0)
        f += 2.0 * T * H * 2 * S * d + 2.0 * T * H * (c["r"] + c["sink"]) * n
    if do in ("infer", "train"):
        b += U * D * e + T * D * e * (1 + c["gate"])
        f += 2.0 * L * D
    if do == "train":
        b += T * D * e + U * D * 8 + U * D * e
        if c["gate"]:
            b += T * D * (3 * e + 4)
    if do == "bag_backward":
        b += T * D * e + U * D * (e + 4) + 16 * L
    if do in ("train", "bag_backward"):
        f += 4.0 * L * D
    if do in ("train", "search_backward"):
        b += T * H * n * (e + 4) + keys * (e + 8) + 12 * L
        f += 4.0 * L * n
    return {"bytes": b, "flops": f}


def tolerance(case):
    # fp32: sums in another order (and selections at a near-tie); bf16: one
    # rounding of the outputs, dy and y rounded once more on the way
    if case["do"] == "search":
        return {"rel": 2e-5, "max": 0.02, "differ": 2e-3}
    if case["do"] == "infer":
        return {"rel": 2e-5 if case["dtype"] == "f32" else 4e-3, "max": 0.1}
    if case["do"] in ("bag_backward", "search_backward"):
        # a normalised query may round to its other bf16 neighbour
        return {"rel": 1e-4 if case["qnorm"] else 1e-5, "max": 1e-2 if case["qnorm"] else 1e-3}
    return {"rel": 1e-4 if case["dtype"] == "f32" else 1e-2, "max": 0.3}


def _exact_search(st, chunk):
    """Yields (t0, t1, scored queries, idx, w, score) of the search in 64 bits."""
    c = st["case"]
    T, S, H, n, k = (c[x] for x in ("T", "S", "H", "n", "k"))
    d = n // 2
    K64 = st["K"].double()
    for t0 in range(0, T, chunk):
        t1 = min(T, t0 + chunk)
        q = st["q"][t0:t1].double()
        if c["qnorm"]:  # the scored query is stored in the query dtype
            q = torch.nn.functional.layer_norm(q, (n,), eps=1e-5).to(DT[c["dtype"]]).double()
        idx, z = [], []
        for h in range(H):
            s, i = [], []
            for p in range(2):
                a = q[:, h, p * d:(p + 1) * d].contiguous() @ K64[h, p].t().contiguous()
                v, j = torch.sort(a, dim=1, descending=True, stable=True)
                s.append(v[:, :k])
                i.append(j[:, :k])
            zz = (s[0][:, :, None] + s[1][:, None, :]).reshape(t1 - t0, -1)
            ii = (i[0][:, :, None] * S + i[1][:, None, :]).reshape(t1 - t0, -1)
            ii, o = torch.sort(ii, dim=1)  # equal sums: lower index first
            v, j = torch.sort(torch.gather(zz, 1, o), dim=1, descending=True, stable=True)
            ii, v = torch.gather(ii, 1, j[:, :k]), v[:, :k]
            if c["r"]:
                x = st["extra"][t0:t1, h]
                e1, e2 = K64[h, 0][x // S], K64[h, 1][x % S]
                ex = (q[:, h, None, :d] * e1).sum(-1) + (q[:, h, None, d:] * e2).sum(-1)
                ii, v = torch.cat([ii, x], 1), torch.cat([v, ex], 1)
            if c["sink"]:
                sk = (q[:, h] * st["sink_keys"][h].double()).sum(-1, keepdim=True)
                ii = torch.cat([ii, torch.full_like(ii[:, :1], S * S + h)], 1)
                v = torch.cat([v, sk], 1)
            idx.append(ii)
            z.append(v)
        z = torch.stack(z, 1)
        yield t0, t1, q, torch.stack(idx, 1), torch.softmax(z, -1), z


def _exact_search_backward(st, t0, t1, q, idx, gz, gK, gq, gsink):
    """Adds the chunk's gradients of the scores (q: as scored)."""
    c = st["case"]
    S, H, n = c["S"], c["H"], c["n"]
    d, kk = n // 2, idx.shape[2] - (1 if gsink is not None else 0)
    K64 = st["K"].double()
    out = torch.zeros_like(q)
    for h in range(H):
        g = gz[:, h, :kk]
        for p in range(2):
            i = (idx[:, h, :kk] // S, idx[:, h, :kk] % S)[p]
            G = torch.zeros((t1 - t0, S), dtype=torch.float64, device=q.device).scatter_add_(1, i, g)
            out[:, h, p * d:(p + 1) * d] = G @ K64[h, p].contiguous()
            gK[h, p] += G.t().contiguous() @ q[:, h, p * d:(p + 1) * d].contiguous()
        if gsink is not None:
            gs = gz[:, h, kk:]
            out[:, h] += gs * st["sink_keys"][h].double()
            gsink[h] += (gs * q[:, h]).sum(0)
    if c["qnorm"]:
        x = st["q"][t0:t1].double()
        mean = x.mean(-1, keepdim=True)
        rstd = 1.0 / torch.sqrt(x.var(-1, unbiased=False, keepdim=True) + 1e-5)
        xh = (x - mean) * rstd
        out = rstd * (out - out.mean(-1, keepdim=True) - xh * (out * xh).mean(-1, keepdim=True))
    gq[t0:t1] = out


def exact(case, seed):
    c = case
    T, S, H, n, D, k, kk = *(c[x] for x in ("T", "S", "H", "n", "D", "k")), _kk(c)
    do, d = c["do"], c["n"] // 2
    st = prepare(case, seed)
    f64 = dict(dtype=torch.float64, device="cuda")
    chunk = 1024 if do == "search" else 256
    if do == "search":
        got = [(i.clone(), w, z) for _, _, _, i, w, z in _exact_search(st, chunk)]
        return {name: torch.cat([x[j] for x in got]) for j, name in enumerate(("idx", "w", "score"))}
    if do == "infer":
        out = torch.empty((T, D), **f64)
        ws = torch.empty((T, H, kk), **f64)
        for t0, t1, _, i, w, _ in _exact_search(st, chunk):
            ws[t0:t1] = w
            for a in range(t0, t1, 64):
                b = min(t1, a + 64)
                v = st["V"][i[a - t0:b - t0].reshape(-1)].double().reshape(b - a, H * kk, D)
                out[a:b] = (v * w[a - t0:b - t0].reshape(b - a, H * kk, 1)).sum(1)
        if c["gate"]:
            g = st["gate"].double()
            out *= g * torch.sigmoid(g)
        return {"out": out, "w": ws}
    if do == "search_backward":
        gK = torch.zeros((H, 2, S, d), **f64)
        gq = torch.zeros((T, H, n), **f64)
        for t0 in range(0, T, 2048):
            t1 = min(T, t0 + 2048)
            q = st["q"][t0:t1].double()
            if c["qnorm"]:
                q = torch.nn.functional.layer_norm(q, (n,), eps=1e-5).to(DT[c["dtype"]]).double()
            _exact_search_backward(st, t0, t1, q, st["idx"][t0:t1], st["gz"][t0:t1].double(), gK,
                                   gq, None)
        return {"grad_q": gq, "grad_subkeys": gK}
    if do == "bag_backward":
        rows, inv = torch.unique(st["idx"].reshape(-1), return_inverse=True)
        inv = inv.reshape(T, H * k)
        gr = torch.zeros((rows.numel(), D), **f64)
        gz = torch.empty((T, H, k), **f64)
        for t0 in range(0, T, 64):
            t1 = min(T, t0 + 64)
            dy, w = st["dy"][t0:t1].double(), st["w"][t0:t1].double()
            v = st["V"][st["idx"][t0:t1].reshape(-1)].double().reshape(t1 - t0, H * k, D)
            gw = (v * dy[:, None]).sum(-1).reshape(t1 - t0, H, k)
            gz[t0:t1] = w * (gw - (w * gw).sum(-1, keepdim=True))
            con = w.reshape(t1 - t0, H * k, 1) * dy[:, None]
            gr.index_add_(0, inv[t0:t1].reshape(-1), con.reshape(-1, D))
        return {"rows": rows, "grad_rows": gr, "grad_scores": gz}
    # train
    gK = torch.zeros((H, 2, S, d), **f64)
    gq = torch.zeros((T, H, n), **f64)
    gsink = torch.zeros((H, n), **f64) if c["sink"] else None
    gV = torch.zeros((st["V"].shape[0], D), **f64)
    out = torch.empty((T, D), **f64)
    gg = torch.empty((T, D), **f64) if c["gate"] else None
    for t0, t1, q, idx, w, _ in _exact_search(st, chunk):
        gz = torch.empty((t1 - t0, H, kk), **f64)
        for a in range(t0, t1, 64):
            b = min(t1, a + 64)
            i, ww, m = idx[a - t0:b - t0], w[a - t0:b - t0], b - a
            v = st["V"][i.reshape(-1)].double().reshape(m, H * kk, D)
            y = (v * ww.reshape(m, H * kk, 1)).sum(1)
            dy = st["dy"][a:b].double()
            if c["gate"]:
                g = st["gate"][a:b].double()
                sig = torch.sigmoid(g)
                out[a:b] = y * g * sig
                gg[a:b] = dy * y * sig * (1 + g * (1 - sig))
                dy = dy * g * sig
            else:
                out[a:b] = y
            gw = (v * dy[:, None]).sum(-1).reshape(m, H, kk)
            gz[a - t0:b - t0] = ww * (gw - (ww * gw).sum(-1, keepdim=True))
            con = (ww.reshape(m, H * kk, 1) * dy[:, None]).reshape(-1, D)
            gV.index_add_(0, i.reshape(-1), con)
        _exact_search_backward(st, t0, t1, q, idx, gz, gK, gq, gsink)
    res = dict(out=out, grad_values=gV, grad_q=gq, grad_subkeys=gK)
    if c["gate"]:
        res["grad_gate"] = gg
    if c["sink"]:
        res["grad_sink"] = gsink
    return res
