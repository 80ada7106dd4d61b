"""Workloads timed on a GPU: whole decompositions through the public binding.

A case is one decomposition call (or one burst of served requests) at the sizes
of this repository's workloads, of the paper's experiments, or of the ranges
around them.  `listed()` gives fixed cases, `draw(rng)` more of the same
ranges; `prepare` makes the inputs on the GPU from a seed, `run` is one pass
through the entry points, `work` the bytes and flops the path cannot do
without, and `exact` the same outputs in float64 with plain torch operations.

Tensors are Tucker models (Gaussian core scaled by a geometric decay along each
mode, orthonormal factors) or tensor rings (Gaussian cores scaled along each
bond), plus Gaussian noise at a given SNR.  `tail` is the scale of the last of
a mode's R components relative to the first.
"""
import math

import numpy as np
import torch

import paper_2211_14828_amd as rb

DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}


def _ints(text):
    return [int(v) for v in str(text).split("x")]


def _text(values):
    return "x".join(str(int(v)) for v in values)


def _tucker(dims, ranks, p, q, dtype, precision="plain", tail=0.1, snr=10.0, **more):
    return dict(kind="tucker", dims=_text(dims), ranks=_text(ranks), p=p, q=q, dtype=dtype, precision=precision,
                tail=tail, snr=snr, **more)


def listed():
    return [
        # the smallest call: 64^3 in double precision, ranks 8, where launches
        # and their gaps are all of the time
        dict(_tucker([64] * 3, [8] * 3, 5, 2, "f64", snr=20.0), name="f64_64"),
        # the paper's own size and type for its synthetic tables: 200^3,
        # ranks 10, double precision
        dict(_tucker([200] * 3, [10] * 3, 5, 2, "f64", snr=5.0), name="f64_200"),
        # 400^3, ranks 20, in the plain float32 form ...
        dict(_tucker([400] * 3, [20] * 3, 10, 3, "f32"), name="f32_400"),
        # ... and in the bf16 form
        dict(_tucker([400] * 3, [20] * 3, 10, 3, "f32", "mixed_bf16"), name="bf16_400"),
        # the headline workload: 1000^3, ranks 50, block-scaled fp8 products
        dict(_tucker([1000] * 3, [50] * 3, 10, 4, "f32", "mixed_fp8", tail=0.08), name="fp8_1000"),
        # the same in the plain float32 form it is compared with
        dict(_tucker([1000] * 3, [50] * 3, 10, 4, "f32", tail=0.08), name="f32_1000"),
        # a colour video as an order-4 tensor, a thin mode of 3 and sketches
        # wider than 64 (the paper's video sizes and ranks)
        dict(_tucker([288, 352, 3, 250], [85, 90, 3, 50], 5, 2, "f32", tail=0.3, snr=20.0), name="video_f32"),
        # odd sizes, bf16 storage, sequential truncation (the ST-HOSVD form)
        dict(_tucker([301, 257, 190], [17, 12, 23], 5, 2, "bf16", truncation="sequential", snr=20.0),
             name="ragged_bf16_seq"),
        # q chosen by the Fit rule on the paper's 200^3
        dict(_tucker([200] * 3, [10] * 3, 5, 20, "f32", snr=5.0, adaptive=True), name="adaptive_200"),
        # tensor ring of a 64^5 tensor through 16^5 (order 5, the largest input)
        dict(kind="htr", dims=_text([64] * 5), ranks=_text([16] * 5), tr=_text([8] * 5), p=6, q=2, dtype="f32",
             precision="plain", bond=0.8, snr=15.0, name="ring_64x5"),
        # tensor ring of an image set (the paper's image sizes, compress sizes
        # min(5 R, I)): one mode far longer than the others together
        dict(kind="htr", dims="32x32x3x7200", ranks="30x30x3x30", tr="6x6x3x6", p=5, q=2, dtype="f32",
             precision="plain", bond=0.9, snr=20.0, name="images_htr"),
        # a burst of served requests: third-order bf16 tensors of mixed sizes
        dict(kind="serve", count=32, slots=8, mix=7, lo=32, hi=256, name="served_32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f64", "f32", "f32", "bf16", "fp8", "stored_bf16", "sequential", "sampled", "power", "adaptive",
                       "order4", "ring", "serve"])
    if kind == "serve":
        return dict(kind="serve", count=rng.randint(8, 48), slots=rng.randint(2, 16), mix=rng.randrange(1 << 16),
                    lo=32, hi=256)
    if kind == "ring":
        N = rng.choice([3, 4, 5])
        hi = {3: 320, 4: 96, 5: 40}[N]
        dims = [_log_int(rng, 20, hi) for _ in range(N)]
        r = rng.randint(3, 6)
        ranks = [min(d, rng.randint(10, 16)) for d in dims]
        return dict(kind="htr", dims=_text(dims), ranks=_text(ranks), tr=_text([r] * N), p=5, q=2, dtype="f32",
                    precision="plain", bond=0.85, snr=rng.choice([15.0, 20.0]))
    if kind == "order4":
        dims = [_log_int(rng, 24, 160) for _ in range(3)]
        dims.insert(rng.randint(0, 3), rng.choice([3, 4, 7, 10]))
    else:
        lo, hi = {"f64": (48, 320), "adaptive": (64, 320), "fp8": (200, 900), "bf16": (130, 700)}.get(kind, (64, 640))
        dims = [_log_int(rng, lo, hi) for _ in range(3)]
    r = _log_int(rng, 6, 36)
    ranks = [max(2, min(d // 4, int(r * rng.uniform(0.75, 1.33)))) if d > 12 else d for d in dims]
    ranks = [min(ranks[n], max(2, math.prod(ranks) // ranks[n] // 4)) for n in range(len(dims))]
    p, q = rng.choice([5, 8, 10]), rng.choice([1, 2, 3])
    snr = rng.choice([10.0, 15.0, 20.0])
    case = _tucker(dims, ranks, p, q, "f64" if kind == "f64" else "f32", snr=snr)
    if kind in ("bf16", "fp8"):
        case["precision"] = "mixed_" + kind
    elif kind == "stored_bf16":
        case["dtype"] = "bf16"
    elif kind == "sequential":
        case["truncation"] = "sequential"
    elif kind == "sampled":
        case.update(rate=rng.choice([0.25, 0.5]), precision=rng.choice(["plain", "mixed_bf16"]))
    elif kind == "power":
        case.update(variant="power", precision=rng.choice(["plain", "mixed_bf16", "mixed_fp8"]))
    elif kind == "adaptive":
        case.update(adaptive=True, q=20)
    return case


# ------------------------------------------------------------------ inputs


def _orthonormal(gen, n, r):
    return torch.linalg.qr(torch.randn((n, r), dtype=torch.float64, generator=gen))[0]


def _expand(G, factors):
    """G x_1 U_1 ... x_N U_N, one two-dimensional product per mode."""
    X = G
    for n, U in enumerate(factors):
        if n == 0:
            X = U @ X.reshape(X.shape[0], -1)
            shape = [U.shape[0]] + list(G.shape[1:])
        else:
            X = X.movedim(n, -1).contiguous()
            lead = list(X.shape[:-1])
            X = (X.reshape(-1, X.shape[-1]) @ U.T).reshape(lead + [U.shape[0]]).movedim(-1, n).contiguous()
            shape = list(X.shape)
        X = X.reshape(shape)
    return X.contiguous()


def _add_noise(X, snr, seed):
    gen = torch.Generator(device=X.device)
    gen.manual_seed(seed)
    flat, step = X.reshape(-1), 1 << 27
    scale = math.sqrt(float(torch.linalg.vector_norm(flat, dtype=torch.float64)) ** 2 / flat.numel()) / 10 ** (snr / 20)
    for s in range(0, flat.numel(), step):
        part = flat[s:s + step]
        part.add_(torch.randn(part.shape, dtype=X.dtype, device=X.device, generator=gen), alpha=scale)
    return X


def _tucker_tensor(dims, ranks, tail, snr, dtype, seed):
    gen = torch.Generator()
    gen.manual_seed(seed)
    G = torch.randn(ranks, dtype=torch.float64, generator=gen)
    for n, R in enumerate(ranks):
        d = tail ** (torch.arange(R, dtype=torch.float64) / max(R - 1, 1))
        G = G * d.reshape([-1 if k == n else 1 for k in range(len(ranks))])
    work = torch.float64 if dtype == torch.float64 else torch.float32
    factors = [_orthonormal(gen, I, R).to("cuda", work) for I, R in zip(dims, ranks)]
    return _add_noise(_expand(G.to("cuda", work), factors), snr, seed + 1).to(dtype)


def _ring_tensor(dims, r, bond, snr, dtype, seed):
    """trace(G_1[:, i_1, :] ... G_N[:, i_N, :]) + noise, the ring ranks r with
    the closing rank r_N; bond index b scaled by bond^b."""
    gen = torch.Generator()
    gen.manual_seed(seed)
    N, cores = len(dims), []
    for k, I in enumerate(dims):
        ra, rc = r[k - 1], r[k]
        C = torch.randn((ra, I, rc), dtype=torch.float64, generator=gen) / math.sqrt(ra)
        cores.append((C * bond ** torch.arange(rc, dtype=torch.float64)).to("cuda", torch.float32))
    X = torch.empty(dims, dtype=torch.float32, device="cuda")
    close = cores[-1].permute(2, 0, 1).contiguous().reshape(r[-1] * r[-2], dims[-1])
    for i in range(dims[0]):
        T = cores[0][:, i, :]
        for C in cores[1:-1]:
            T = (T.reshape(-1, C.shape[0]) @ C.reshape(C.shape[0], -1)).reshape(list(T.shape[:-1]) + list(C.shape[1:]))
        X[i] = (T.movedim(0, -2).contiguous().reshape(-1, r[-1] * r[-2]) @ close).reshape(dims[1:])
    return _add_noise(X, snr, seed + 1).to(dtype)


def _requests(case):
    """Recipes of a served mix: dims U{lo..hi}, ranks U{4..32} capped at dim/2
    and at what the other two ranks can carry, SNR U[10, 30] dB, q U{1, 2, 3}."""
    rng = np.random.default_rng(case["mix"])
    out = []
    for _ in range(case["count"]):
        dims = [int(v) for v in rng.integers(case["lo"], case["hi"] + 1, size=3)]
        r = [int(min(v, d // 2)) for v, d in zip(rng.integers(4, 33, size=3), dims)]
        ranks = [min(r[n], max(1, r[n - 1] * r[n - 2] // 4)) for n in range(3)]
        out.append((dims, ranks, float(rng.uniform(10.0, 30.0)), int(rng.integers(1, 4))))
    return out


def _inputs(case, seed):
    if case["kind"] == "serve":
        return [_tucker_tensor(d, r, 0.3, snr, torch.bfloat16, seed * 1000003 + 2 * i)
                for i, (d, r, snr, _) in enumerate(_requests(case))]
    dims, dtype = _ints(case["dims"]), DTYPES[case["dtype"]]
    if case["kind"] == "htr":
        return _ring_tensor(dims, _ints(case["tr"]), case["bond"], case["snr"], dtype, seed)
    return _tucker_tensor(dims, _ints(case["ranks"]), case["tail"], case["snr"], dtype, seed)


def prepare(case, seed):
    state = dict(case=case, X=_inputs(case, seed), seed=seed)
    if case["kind"] == "serve":
        state["requests"] = _requests(case)
        state["server"] = rb.Server(4 << 30, case["slots"])
    return state


def run(state):
    case, X = state["case"], state["X"]
    if case["kind"] == "serve":
        server = state["server"]
        tickets = [server.submit(x, ranks, p=5, q=q, seed=state["seed"] + i)
                   for i, (x, (_, ranks, _, q)) in enumerate(zip(X, state["requests"]))]
        done = [server.wait(t) for t in tickets]
        return {"cores": torch.cat([d[0].reshape(-1) for d in done]),
                "factors": torch.cat([u.reshape(-1) for d in done for u in d[1]]),
                "errors": torch.tensor([d[2] for d in done], dtype=torch.float32)}
    ranks = _ints(case["ranks"])
    opts = dict(p=case["p"], seed=state["seed"], precision=case["precision"])
    if case["kind"] == "htr":
        cores, err = rb.htr(X, ranks, _ints(case["tr"]), q=case["q"], **opts)
        return {"cores": cores, "err": err}
    if case.get("adaptive"):
        core, factors, err, q = rb.tucker_adaptive(X, ranks, max_q=case["q"], **opts)
        return {"core": core, "factors": factors, "err": err, "q": q}
    core, factors, err = rb.tucker(X, ranks, q=case["q"], variant=case.get("variant", "krylov"),
                                   sample_rate=case.get("rate", 1.0), truncation=case.get("truncation", "independent"),
                                   **opts)
    return {"core": core, "factors": factors, "err": err}


# ------------------------------------------------------------------ work


def _tucker_work(dims, ranks, p, q, esize, sequential=False):
    """Input and outputs once; per mode the cheaper of one Gram pass and
    q + 2 passes of products with the sketch, then the core and the error."""
    T, flops, cur = math.prod(dims), 0.0, list(dims)
    for n, R in enumerate(ranks):
        I, J = cur[n], math.prod(cur) // cur[n]
        S = min(R + p, I, J)
        flops += min(I * (I + 1.0) * J + 2.0 * I * J * S + 2.0 * I * I * S * (q + 1), 2.0 * I * J * S * (2 * q + 2))
        if sequential:
            flops += 2.0 * R * I * J
            cur[n] = R
    if not sequential:
        for n in sorted(range(len(dims)), key=lambda k: -dims[k] / ranks[k]):
            flops += 2.0 * ranks[n] * math.prod(cur)
            cur[n] = ranks[n]
    out = math.prod(ranks) + sum(I * R for I, R in zip(dims, ranks))
    flops += 2.0 * T * ranks[0]
    return T * esize + out * (8 if esize == 8 else 4), flops


def work(case):
    if case["kind"] == "serve":
        each = [_tucker_work(d, r, 5, q, 2) for d, r, _, q in _requests(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    esize = {"f64": 8, "f32": 4, "bf16": 2}[case["dtype"]]
    q = 2 if case.get("adaptive") else case["q"]
    b, f = _tucker_work(_ints(case["dims"]), _ints(case["ranks"]), case["p"], q, esize,
                        case.get("truncation") == "sequential")
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ float64


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    def mul(m, c):
        low = m * (c & 0xFFFF)
        high = m * (c >> 16) + (low >> 16)
        return high >> 16, ((high & 0xFFFF) << 16) | (low & 0xFFFF)
    for i in range(10):
        a = (k0 + i * 0x9E3779B9) & 0xFFFFFFFF
        b = (k1 + i * 0xBB67AE85) & 0xFFFFFFFF
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ a, l1, h0 ^ c3 ^ b, l0
    return c0, c1, c2, c3


def _omega(seed, mode, J, S):
    """The sketch's J x S Gaussians, transposed (S x J): linear index s J + j."""
    total = J * S
    out = torch.empty(total + 1, dtype=torch.float64, device="cuda")
    for m0 in range(0, (total + 1) // 2, 1 << 24):
        m = torch.arange(m0, min(m0 + (1 << 24), (total + 1) // 2), device="cuda")
        w = _philox(m & 0xFFFFFFFF, m >> 32, torch.full_like(m, mode), torch.zeros_like(m), seed & 0xFFFFFFFF, seed >> 32)
        u = [((w[k].double() * 2.0 ** 20 + (w[k + 1] >> 12).double()) + 0.5) * 2.0 ** -52 for k in (0, 2)]
        r = torch.sqrt(-2.0 * torch.log(u[0]))
        out[2 * m0:2 * (m0 + m.numel())] = torch.stack([r * torch.cos(2 * math.pi * u[1]),
                                                        r * torch.sin(2 * math.pi * u[1])], 1).reshape(-1)
    return out[:total].reshape(S, J)


def _sample(seed, mode, J, m):
    k = torch.arange(m, device="cuda")
    lo = k * J // m
    width = (k + 1) * J // m - lo
    w = _philox(k & 0xFFFFFFFF, k >> 32, torch.full_like(k, mode), torch.ones_like(k), seed & 0xFFFFFFFF, seed >> 32)[0]
    return lo + ((w * width) >> 32)


def _orth(Y):
    return torch.linalg.qr(Y.cpu())[0].cuda()


def _signs(U):
    top = torch.gather(U, 0, U.abs().argmax(0, keepdim=True))
    return U * torch.where(top < 0, -1.0, 1.0)


def _leading(Q, C, R):
    lam, V = torch.linalg.eigh((Q.T @ (C @ Q)).cpu())
    return _signs(Q @ V.flip(1)[:, :R].cuda())


def _mode_bases(X, n, R, p, q, seed, variant="krylov", rate=1.0):
    """C = X_(n) X_(n)^T and the orthonormal bases after 0, 1, ..., q steps."""
    I = X.shape[n]
    Xn = X.movedim(n, 0).reshape(I, -1)
    J = Xn.shape[1]
    m = max(1, min(J, int(math.floor(rate * J + 0.5)))) if rate < 1.0 else J
    Y = Xn[:, _sample(seed, n, J, m)] if m < J else Xn
    S = min(R + p, I, m)
    W = Y @ _omega(seed, n, m, S).T
    C = Xn @ Xn.T
    K = Y @ Y.T if m < J else C
    Q = last = _orth(W)
    bases = [Q]
    for _ in range(q):
        if variant == "power":
            Q = last = _orth(K @ last)
        elif Q.shape[1] + S >= I:
            Q = torch.eye(I, dtype=torch.float64, device="cuda")
            last = last[:, :0]
        else:
            Z = K @ last
            for _ in range(2):
                Z = Z - Q @ (Q.T @ Z)
            last = _orth(Z)
            Q = torch.cat([Q, last], 1)
        bases.append(Q)
        if Q.shape[1] >= I and variant != "power":
            bases += [Q] * (q + 1 - len(bases))
            break
    return C, bases


def _project(X, factors):
    for n, U in enumerate(factors):
        if U is not None:
            X = (X.movedim(n, -1).reshape(-1, U.shape[0]) @ U).reshape(
                [d for k, d in enumerate(X.shape) if k != n] + [U.shape[1]]).movedim(-1, n)
    return X.contiguous()


def _tucker_exact(X, ranks, p, q, seed, variant="krylov", rate=1.0, truncation="independent", fit_tol=None):
    X = X.double()
    n2 = float((X * X).sum())
    steps, factors, Y = q, [], X
    if fit_tol is not None:
        S = [min(R + p, I, X.numel() // I) for R, I in zip(ranks, X.shape)]
        steps = min([q, max(-(-I // s) for I, s in zip(X.shape, S))] + [1200 // s - 1 for s in S])
        modes = [_mode_bases(X, n, ranks[n], p, steps, seed) for n in range(X.dim())]
        before = None
        for t in range(steps + 1):
            factors = [_leading(B[t], C, R) for (C, B), R in zip(modes, ranks)]
            G = _project(X, factors)
            err = math.sqrt(max(0.0, 1 - float((G * G).sum()) / n2))
            if (t and abs(err - before) <= fit_tol) or t == steps:
                return G, factors, err, t
            before = err
    for n in range(X.dim()):
        C, B = _mode_bases(Y, n, ranks[n], p, q, seed, variant, rate)
        factors.append(_leading(B[-1], C, ranks[n]))
        if truncation == "sequential":
            Y = _project(Y, [factors[n] if k == n else None for k in range(X.dim())])
    G = Y if truncation == "sequential" else _project(X, factors)
    return G, factors, math.sqrt(max(0.0, 1 - float((G * G).sum()) / n2)), q


def _split(M, r):
    """The r leading singular triplets as U and S V^T, zero-padded, each left
    vector's largest entry positive."""
    lam, V = torch.linalg.eigh((M @ M.T).cpu())
    k = min(r, M.shape[0])
    U = _signs(V.flip(1)[:, :k].cuda())
    pad = torch.zeros((M.shape[0], r - k), dtype=M.dtype, device=M.device)
    return torch.cat([U, pad], 1), torch.cat([U, pad], 1).T @ M


def _ring_exact(G, tr):
    S, r = list(G.shape), [tr[-1]] + tr
    U, M = _split(G.reshape(S[0], -1), r[0] * r[1])
    cores = [U.reshape(S[0], r[0], r[1]).permute(1, 0, 2)]
    M = M.reshape([r[0], r[1]] + S[1:]).movedim(0, -1)
    for k in range(1, len(S) - 1):
        U, M = _split(M.reshape(r[k] * S[k], -1), r[k + 1])
        cores.append(U.reshape(r[k], S[k], r[k + 1]))
        M = M.reshape([r[k + 1]] + S[k + 1:] + [r[0]])
    cores.append(M.reshape(r[-2], S[-1], r[0]))
    T = cores[0].reshape(-1, r[1])
    for C in cores[1:]:
        T = T.reshape(-1, C.shape[0]) @ C.reshape(C.shape[0], -1)
    T = T.reshape([r[0]] + S + [r[0]]).diagonal(dim1=0, dim2=-1).sum(-1)
    return cores, float(((G - T) ** 2).sum())


def _flat(e):
    return torch.tensor(e, dtype=torch.float64)


def exact(case, seed):
    """The outputs in float64.  The mixed forms round the operands, which moves
    a factor by up to 1e-3 and so can turn a column's sign where its two
    largest entries are that close: for them only the error has such a value."""
    X = _inputs(case, seed)
    if case["kind"] == "serve":
        done = [_tucker_exact(x, r, 5, q, seed + i) for i, (x, (_, r, _, q)) in enumerate(zip(X, _requests(case)))]
        return {"cores": torch.cat([d[0].reshape(-1) for d in done]),
                "factors": torch.cat([u.reshape(-1) for d in done for u in d[1]]),
                "errors": torch.tensor([d[2] for d in done], dtype=torch.float64)}
    ranks = _ints(case["ranks"])
    G, factors, err, q = _tucker_exact(X, ranks, case["p"], case["q"], seed, case.get("variant", "krylov"),
                                       case.get("rate", 1.0), case.get("truncation", "independent"),
                                       1e-3 if case.get("adaptive") else None)
    if case["kind"] == "htr":
        n2 = float(X.double().square().sum())
        cores, gap = _ring_exact(G, _ints(case["tr"]))
        cores = [(U @ C.permute(1, 0, 2).reshape(C.shape[1], -1)).reshape(-1, C.shape[0], C.shape[2]).permute(1, 0, 2)
                 .contiguous() for C, U in zip(cores, factors)]
        return {"cores": cores, "err": _flat(math.sqrt(err ** 2 + gap / n2))}
    if case["precision"] != "plain":
        return {"core": None, "factors": None, "err": _flat(err)}
    if case.get("adaptive"):
        return {"core": G, "factors": factors, "err": _flat(err), "q": q}
    return {"core": G, "factors": factors, "err": _flat(err)}
