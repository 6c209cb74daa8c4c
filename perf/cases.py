"""The calls whose speed is measured: inputs, one pass, its work and its tolerance.

Each case is one call of the library through its Python entry points, with
the objects a program keeps between calls (weights, workspace, output
buffers) made beforehand.  Inputs are synthetic and drawn on the GPU from the
seed: visual tokens are a Gaussian mixture with exact copies (redundant image
patches), or frames that repeat the previous one with small changes (video);
question tokens are normal; predictor weights have the spread that gives a
peaked attention, as a trained predictor does; attention for the teacher
selection is a softmax with a middle-layer question field.

`draw` spreads the sizes over what the listed cases stand for: images from a
small thumbnail grid (144 tokens) to eight frames (4608), one image to a
serving batch of 16, feature widths of common models, both storage types.
"""
import math

import torch

import paper_2608_06411_amd as mp

DEV = "cuda"
TAU = 1e-2
WEIGHT_NAMES = ("w1_v", "b1_v", "w2_v", "b2_v", "w_k", "w1_t", "b1_t", "w2_t", "b2_t", "w_q")


def listed():
    return [
        # One LLaVA-1.5 image (576 tokens) pruned to 64 straight into the language model's input: the
        # smallest serving call, where launches and latency count.
        dict(name="prune_576_bf16", kind="prune", form="assemble", dtype="bf16", B=1, N=576, D=4096, D_h=1024, d_p=128,
             M_lo=32, M_hi=32, K=64, K0=32, clusters=64, dup=0.08, frames=1),
        # The same image with everything in float32: the option for checking a deployment's precision.
        dict(name="prune_576_f32", kind="prune", form="rows", dtype="f32", B=1, N=576, D=4096, D_h=1024, d_p=128,
             M_lo=32, M_hi=32, K=64, K0=32, clusters=64, dup=0.08, frames=1),
        # One LLaVA-NeXT image (2880 tokens) pruned to 160: the headline call.
        dict(name="prune_2880_bf16", kind="prune", form="rows", dtype="bf16", B=1, N=2880, D=4096, D_h=1024, d_p=128,
             M_lo=64, M_hi=64, K=160, K0=80, clusters=256, dup=0.08, frames=1),
        # A serving batch of 16 LLaVA-NeXT images with ragged questions at the usual budget.
        dict(name="prune_16x2880_bf16", kind="prune", form="assemble", dtype="bf16", B=16, N=2880, D=4096, D_h=1024,
             d_p=128, M_lo=16, M_hi=128, K=160, K0=80, clusters=256, dup=0.05, frames=1),
        # Eight clips of eight frames (4608 tokens, 3584 wide): long inputs with much repetition.
        dict(name="prune_8x4608_frames", kind="prune", form="rows", dtype="bf16", B=8, N=4608, D=3584, D_h=1024,
             d_p=128, M_lo=96, M_hi=96, K=256, K0=128, clusters=512, dup=0.0, frames=8),
        # Scores alone, for a caller with its own selection: three images of an odd token count.
        dict(name="score_3x1225_bf16", kind="score", dtype="bf16", B=3, N=1225, D=3584, D_h=1024, d_p=128, M_lo=16,
             M_hi=90, clusters=128, dup=0.05, frames=1),
        # The whole cosine matrix of two LLaVA-NeXT images, for a caller that studies redundancy.
        dict(name="similarity_2x2880_bf16", kind="similarity", dtype="bf16", B=2, N=2880, D=4096, clusters=256, dup=0.08),
        # Selection on given scores and similarity at the largest budget of the retention sweep.
        dict(name="select_4x2880_k640", kind="select", B=4, N=2880, D=1024, K=640, K0=320, clusters=256, dup=0.05),
        # Teacher selection over one sample's attention in all 32 layers of a 7B model.
        dict(name="teacher_32x32x2880", kind="teacher", dtype="bf16", B=1, L=32, H=32, N=2880, M_lo=64, M_hi=64, M_ref=8,
             n_top=1),
        # One training step of the predictor on two LLaVA-NeXT images: forward, loss, all gradients.
        dict(name="train_2x2880_bf16", kind="train", dtype="bf16", B=2, N=2880, D=4096, D_h=1024, d_p=128, M_lo=40,
             M_hi=72, clusters=256, dup=0.08, frames=1),
        # The language model's layer over one pruned image and its question (160 + 64 rows).
        dict(name="decoder_224", kind="decoder", d=4096, ff=11008, B=1, R_lo=224, R_hi=224),
        # The same layer over an unpruned image (2880 + 64 rows): the prefill that pruning avoids.
        dict(name="decoder_2944", kind="decoder", d=4096, ff=11008, B=1, R_lo=2944, R_hi=2944),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_features(rng, tokens):
    """Images, tokens and widths of a call over at most `tokens` visual tokens."""
    N = _log_int(rng, 144, 4608)
    B = max(1, min(16, _log_int(rng, 1, max(1, min(16, tokens // N)))))
    D = rng.choice((1024, 1152, 2048, 3584, 4096, 4096))
    D_h, d_p = rng.choice(((1024, 128), (1024, 128), (1024, 128), (512, 64)))
    lo = rng.randint(8, 64)
    return dict(B=B, N=N, D=D, D_h=D_h, d_p=d_p, M_lo=lo, M_hi=lo + rng.randint(0, 64), clusters=max(8, N // 11),
                dup=rng.choice((0.0, 0.05, 0.08)), frames=1)


def draw(rng):
    kind = rng.choice(("prune", "prune", "prune", "score", "similarity", "select", "teacher", "train", "decoder", "decoder"))
    if kind == "prune":
        c = dict(kind="prune", form=rng.choice(("rows", "assemble")), dtype=rng.choice(("bf16", "bf16", "bf16", "f32")))
        c.update(_draw_features(rng, 46080))
        if c["dtype"] == "f32":
            c["B"] = 1
        elif rng.random() < 0.25:
            per = _log_int(rng, 144, 576)
            c.update(frames=8, N=8 * per, B=max(1, min(c["B"], 46080 // (8 * per))), dup=0.0)
        c["K"] = min(640, max(16, int(c["N"] * math.exp(rng.uniform(math.log(1 / 24), math.log(1 / 4))))))
        c["K0"] = rng.choice((c["K"] // 2, c["K"] // 2, c["K"] // 4, c["K"]))
        return c
    if kind == "score":
        c = dict(kind="score", dtype=rng.choice(("bf16", "bf16", "f32")))
        c.update(_draw_features(rng, 46080 if c["dtype"] == "bf16" else 4608))
        return c
    if kind == "similarity":
        c = dict(kind="similarity", dtype=rng.choice(("bf16", "bf16", "f32")))
        f = _draw_features(rng, 11520 if c["dtype"] == "bf16" else 2880)
        if c["dtype"] == "f32":
            f["N"] = min(f["N"], 2880)
        c.update({k: f[k] for k in ("B", "N", "D", "clusters", "dup")})
        return c
    if kind == "select":
        f = _draw_features(rng, 11520)
        K = min(640, max(16, int(f["N"] * math.exp(rng.uniform(math.log(1 / 24), math.log(1 / 4))))))
        return dict(kind="select", B=f["B"], N=f["N"], D=1024, K=K, K0=rng.choice((K // 2, K // 4, 0)),
                    clusters=f["clusters"], dup=f["dup"])
    if kind == "teacher":
        lo = rng.randint(8, 48)
        N = 8 * _log_int(rng, 18, 360)
        L = rng.choice((12, 24, 32))
        return dict(kind="teacher", dtype=rng.choice(("bf16", "f32")), B=rng.randint(1, 2), L=L, H=rng.choice((16, 32)), N=N,
                    M_lo=lo, M_hi=lo + rng.randint(0, 16), M_ref=rng.randint(4, 16), n_top=rng.choice((1, 1, 3)))
    if kind == "train":
        c = dict(kind="train", dtype=rng.choice(("bf16", "bf16", "f32")))
        c.update(_draw_features(rng, 11520 if c["dtype"] == "bf16" else 1152))
        if c["dtype"] == "f32":
            c["N"] = min(c["N"], 1152)
        return c
    d, ff = rng.choice(((1024, 2816), (2048, 5632), (4096, 11008), (4096, 11008)))
    rows = _log_int(rng, 48, 2944)
    B = rng.randint(1, max(1, min(8, rows // 40)))
    lo = max(16, rows // B - rng.randint(0, rows // B // 3))
    return dict(kind="decoder", d=d, ff=ff, B=B, R_lo=lo, R_hi=max(lo, 2 * (rows // B) - lo))


# ---------------------------------------------------------------- inputs

def _dtype(case):
    return {"bf16": torch.bfloat16, "f32": torch.float32}[case["dtype"]]


def _lengths(B, lo, hi):
    """B lengths spread over [lo, hi], the same for every seed."""
    return [lo + (b * 37 + (17 if B > 1 else 0)) % (hi - lo + 1) for b in range(B)]


def _offsets(lengths):
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    return off


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _mixture(g, n, D, clusters, dup):
    centres = _normal(g, clusters, D)
    v = centres[torch.randint(clusters, (n,), generator=g, device=DEV)] + 0.3 * _normal(g, n, D)
    n_dup = int(dup * n)
    if n_dup:
        perm = torch.randperm(n, generator=g, device=DEV)
        slots, keep = perm[:n_dup], perm[n_dup:]
        v[slots] = v[keep[torch.randint(n - n_dup, (n_dup,), generator=g, device=DEV)]]
    return v


def _visual(case, g, dtype):
    B, N, D, frames = case["B"], case["N"], case["D"], case.get("frames", 1)
    V = torch.empty(B, N, D, dtype=dtype, device=DEV)
    per = N // frames
    for b in range(B):
        f = _mixture(g, per, D, case["clusters"], case["dup"])
        for t in range(frames):
            if t:
                moved = torch.randperm(per, generator=g, device=DEV)[:int(round(0.7 * per))]
                f[moved] += 0.1 * _normal(g, moved.numel(), D)
            V[b, t * per:(t + 1) * per] = f
    return V


def _features(case, seed):
    """Predictor weights and one call's inputs."""
    g, dtype = _gen(seed), _dtype(case)
    B, N, D, H, dp = case["B"], case["N"], case["D"], case["D_h"], case["d_p"]
    lens = _lengths(B, case["M_lo"], case["M_hi"])
    V = _visual(case, g, dtype)
    T = _normal(g, sum(lens), D).to(dtype)
    # standard deviation 0.03 at (4096, 1024): the same activations at other widths
    s1, s2 = 0.03 * math.sqrt(4096 / D), 0.03 * math.sqrt(1024 / H)
    shapes = dict(w1_v=(H, D), b1_v=(H,), w2_v=(H, H), b2_v=(H,), w_k=(dp, H),
                  w1_t=(H, D), b1_t=(H,), w2_t=(H, H), b2_t=(H,), w_q=(dp, H))
    w = {n: ((s1 if n.startswith("w1") else s2) * _normal(g, *shapes[n])).to(dtype) for n in WEIGHT_NAMES}
    pos_v = torch.arange(N, dtype=torch.int32, device=DEV).repeat(B, 1)
    pos_t = torch.cat([N + torch.arange(m, dtype=torch.int32, device=DEV) for m in lens])
    return dict(w=w, V=V, T=T, pos_v=pos_v, pos_t=pos_t, t_off=_offsets(lens))


def _peaked(g, B, N, alpha):
    """Peaked distributions over N tokens: Gamma(alpha) weights, normalised, as float32."""
    # Gamma(alpha) = Gamma(alpha + 1) * U^(1 / alpha); Gamma(1 + alpha) is near Exp(1) for a small alpha
    u = torch.rand(B, N, generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-300)
    e = torch.empty(B, N, device=DEV, dtype=torch.float64).exponential_(generator=g)
    p = (e * u ** (1 / alpha)).clamp_min(1e-12)
    return (p / p.sum(1, keepdim=True)).float()


def _select_inputs(case, seed):
    g = _gen(seed)
    V = _visual(case, g, torch.float32)
    norms = V.norm(dim=2)
    S = torch.empty(case["B"], case["N"], case["N"], device=DEV)
    for b in range(case["B"]):
        u = V[b] / norms[b][:, None]
        S[b] = u @ u.t()
    S = (0.5 * (S + S.transpose(1, 2))).contiguous()
    return _peaked(g, case["B"], case["N"], 0.1), S, norms


def _attention(case, seed):
    g, dtype = _gen(seed), _dtype(case)
    B, L, H, N = case["B"], case["L"], case["H"], case["N"]
    lens = _lengths(B, case["M_lo"], case["M_hi"])
    x = (torch.arange(L, device=DEV) + 0.5) / L
    beta = (2.5 * torch.exp(-((x - 0.45) / 0.2) ** 2)).reshape(L, 1, 1, 1)
    A = torch.empty(L * H * sum(lens) * N, dtype=dtype, device=DEV)
    ref = torch.empty(B, L, H, case["M_ref"], N, dtype=dtype, device=DEV)
    at = 0
    for m, b in zip(lens, range(B)):
        image, field = _normal(g, L, 1, 1, N), _normal(g, N)
        z = image + beta * field + 0.7 * _normal(g, L, H, m, N)
        A[at:at + z.numel()] = (0.5 * torch.softmax(z, 3)).to(dtype).reshape(-1)
        at += z.numel()
        ref[b] = (0.5 * torch.softmax(image + 0.7 * _normal(g, L, H, case["M_ref"], N), 3)).to(dtype)
    return A, ref, _offsets(lens)


def _decoder_inputs(case, seed):
    g, d, ff = _gen(seed), case["d"], case["ff"]
    off = _offsets(_lengths(case["B"], case["R_lo"], case["R_hi"]))

    def weight(*shape):
        return (0.02 * _normal(g, *shape)).to(torch.bfloat16)

    w = dict(attn_norm=(1 + 0.1 * _normal(g, d)).to(torch.bfloat16), w_qkv=weight(3 * d, d), w_o=weight(d, d),
             ffn_norm=(1 + 0.1 * _normal(g, d)).to(torch.bfloat16), w_gate_up=weight(2 * ff, d), w_down=weight(d, ff))
    X = _normal(g, off[-1], d).to(torch.bfloat16)
    # kept tokens carry the positions they had in the image: gaps of random length
    pos = torch.cumsum(torch.randint(1, 20, (off[-1],), generator=g, device=DEV), 0)
    pos = torch.cat([pos[a:b] - pos[a] for a, b in zip(off, off[1:])]).to(torch.int32)
    return w, X, pos, off


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("prune", "score", "train"):
        x = _features(case, seed)
        x["weights"] = mp.PredictorWeights(**x["w"])
        B, N, D, dev = case["B"], case["N"], case["D"], x["V"].device
        if kind == "prune":
            K = case["K"]
            x["workspace"] = mp.PruneWorkspace(x["weights"], x["V"], x["t_off"], K)
            out = dict(idx=torch.empty(B, K, dtype=torch.int32, device=dev), p=torch.empty(B, N, device=dev),
                       order=torch.empty(B, K, dtype=torch.int32, device=dev), gain=torch.empty(B, K, device=dev))
            if case["form"] == "assemble":
                rows = B * K + x["t_off"][-1]
                out.update(X=torch.empty(rows, D, dtype=_dtype(case), device=dev),
                           pos_x=torch.empty(rows, dtype=torch.int32, device=dev))
            else:
                out.update(V_out=torch.empty(B, K, D, dtype=_dtype(case), device=dev),
                           pos_out=torch.empty(B, K, dtype=torch.int32, device=dev))
            x["out"] = out
        elif kind == "score":
            x["p_out"] = torch.empty(B, N, device=dev)
        else:
            x["p_teacher"] = _peaked(_gen(seed + 7919), B, N, 1.0)
            x["workspace"] = mp.TrainWorkspace(x["weights"], x["V"], x["t_off"])
            x["grads"] = {n: torch.empty(x["w"][n].shape, device=dev) for n in WEIGHT_NAMES}
            x["p_out"] = torch.empty(B, N, device=dev)
        return dict(case=case, **x)
    if kind == "similarity":
        V = _visual(case, _gen(seed), _dtype(case))
        return dict(case=case, V=V, S=torch.empty(case["B"], case["N"], case["N"], device=DEV),
                    norms=torch.empty(case["B"], case["N"], device=DEV))
    if kind == "select":
        p, S, norms = _select_inputs(case, seed)
        B, K = case["B"], case["K"]
        return dict(case=case, p=p, S=S, norms=norms, idx=torch.empty(B, K, dtype=torch.int32, device=DEV),
                    order=torch.empty(B, K, dtype=torch.int32, device=DEV), gain=torch.empty(B, K, device=DEV))
    if kind == "teacher":
        A, ref, off = _attention(case, seed)
        return dict(case=case, A=A, ref=ref, off=off, out=None)
    w, X, pos, off = _decoder_inputs(case, seed)
    weights = mp.DecoderWeights(n_heads=case["d"] // 128, **w)
    return dict(case=case, weights=weights, X=X, pos=pos, off=off, out=torch.empty_like(X),
                workspace=mp.decoder_workspace(weights, off[-1], X.device))


# ---------------------------------------------------------------- one pass

def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "prune":
        call = mp.map_prune_assemble if c["form"] == "assemble" else mp.map_prune
        return call(state["weights"], state["V"], state["pos_v"], state["T"], state["pos_t"], state["t_off"], c["K"], c["K0"],
                    TAU, out=state["out"], workspace=state["workspace"])
    if kind == "score":
        return mp.map_score(state["weights"], state["V"], state["pos_v"], state["T"], state["pos_t"], state["t_off"],
                            p_out=state["p_out"])
    if kind == "similarity":
        return mp.map_similarity(state["V"], S_out=state["S"], norms_out=state["norms"])
    if kind == "select":
        return mp.map_select(state["p"], state["S"], state["norms"], c["K"], c["K0"], TAU, idx_out=state["idx"],
                             order_out=state["order"], gain_out=state["gain"])
    if kind == "teacher":
        out = mp.map_teacher(state["A"], state["ref"], state["off"], c["L"], c["H"], c["N"], c["M_ref"], c["n_top"],
                             out=state["out"])
        state["out"] = out
        return {n: out[n] for n in ("p", "p_ref", "js", "layers", "teacher")}
    if kind == "train":
        return mp.map_train_step(state["weights"], state["V"], state["pos_v"], state["T"], state["pos_t"], state["t_off"],
                                 state["p_teacher"], grads=state["grads"], p_out=state["p_out"], workspace=state["workspace"])
    return mp.map_decoder_layer(state["weights"], state["X"], state["pos"], state["off"], out=state["out"],
                                workspace=state["workspace"])


# ---------------------------------------------------------------- its work

def work(case):
    kind = case["kind"]
    e = 2 if case.get("dtype", "f32") == "bf16" else 4
    B, N = case["B"], case.get("N", 0)
    if kind in ("prune", "score", "train"):
        D, H, dp = case["D"], case["D_h"], case["d_p"]
        lens = _lengths(B, case["M_lo"], case["M_hi"])
        rows = B * N + sum(lens)
        params = 2 * (H * D + H + H * H + H + dp * H)
        # layer 1; W_K W_2 folded and applied (its last step is affine); the logits
        forward = 2 * rows * D * H + 2 * 2 * dp * H * H + 2 * rows * H * dp + 2 * N * sum(lens) * dp
        inputs = e * (rows * D + params) + 4 * rows
        if kind == "score":
            return dict(bytes=inputs + 4 * B * N, flops=forward)
        if kind == "train":
            # back through the logits and the folded product (dL/dh and its weights), dL/dW_1 and dL/dW_2
            backward = 2 * 2 * N * sum(lens) * dp + 2 * 2 * rows * H * dp + 2 * rows * D * H + 2 * 4 * dp * H * H
            return dict(bytes=inputs + 4 * B * N * 2 + 4 * B + 4 * params, flops=forward + backward)
        K = case["K"]
        out = e * B * K * D + 4 * B * (4 * K + N) + ((e * D + 4) * sum(lens) if case["form"] == "assemble" else 0)
        # the cosine rows of the kept tokens and the Gram-Schmidt updates over all tokens
        return dict(bytes=inputs + out, flops=forward + 2 * B * K * N * D + B * K * K * N)
    if kind == "similarity":
        return dict(bytes=e * B * N * case["D"] + 4 * B * N * (N + 1), flops=B * N * (N + 1) * case["D"])
    if kind == "select":
        K = case["K"]
        return dict(bytes=4 * B * (2 * N + K * N + 3 * K), flops=B * K * K * N)
    if kind == "teacher":
        lens = _lengths(B, case["M_lo"], case["M_hi"])
        read = (sum(lens) + B * case["M_ref"]) * case["L"] * case["H"] * N
        return dict(bytes=e * read + 4 * B * N * (2 * case["L"] + 1) + 8 * B * case["L"], flops=read)
    d, ff = case["d"], case["ff"]
    lens = _lengths(B, case["R_lo"], case["R_hi"])
    R = sum(lens)
    return dict(bytes=2 * (4 * d * d + 3 * d * ff + 2 * d) + 2 * 2 * R * d + 4 * R,
                flops=2 * R * (4 * d * d + 3 * d * ff) + sum(2 * 2 * d * n * (n + 1) // 2 for n in lens))


def tolerance(case):
    """About four times what each kind's error against 64 bits measures, over listed and drawn sizes."""
    kind = case["kind"]
    if kind == "similarity":
        return dict(rel=2e-6)
    if kind == "select":
        return dict(rel=1e-5, differ=0.01)
    if kind == "teacher":
        return dict(rel=1e-6)
    if kind == "decoder":
        return dict(rel=2e-2)
    if case["dtype"] == "f32":
        return dict(rel=1e-5, differ=0.01)
    if kind == "train":
        return dict(rel=2e-2)
    return dict(rel=1e-2, differ=0.01)


# ---------------------------------------------------------------- the same in 64 bits

def _rope(z, pos, theta=10000.0):
    half = z.shape[1] // 2
    ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=z.device) / z.shape[1])
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = z[:, :half], z[:, half:]
    return torch.cat([a * c - b * s, b * c + a * s], 1)


def _predict(x, w, case):
    """Eq. (3) in the weights' precision: p [B, N]."""
    def branch(v, pos, t):
        h = torch.nn.functional.gelu(v @ w["w1_" + t].t() + w["b1_" + t])
        return _rope((h @ w["w2_" + t].t() + w["b2_" + t]) @ w["w_k" if t == "v" else "w_q"].t(), pos)

    rows = []
    for b in range(case["B"]):
        k = branch(x["V"][b].double(), x["pos_v"][b], "v")
        at = slice(x["t_off"][b], x["t_off"][b + 1])
        q = branch(x["T"][at].double(), x["pos_t"][at], "t")
        rows.append(torch.softmax(q @ k.t() / math.sqrt(case["d_p"]), 1).mean(0))
    return torch.stack(rows)


def _greedy(p, S, norms, K, K0):
    """Gains of the greedy selection of Eq. (4) on given scores and similarity (all float64)."""
    B, N = p.shape
    at = torch.arange(B, device=p.device)
    C = torch.zeros(B, K, N, dtype=torch.float64, device=p.device)
    r2 = (norms > 0).double()
    taken = torch.zeros(B, N, dtype=torch.bool, device=p.device)
    first = torch.argsort(p, dim=1, descending=True, stable=True)
    gains = torch.zeros(B, K, dtype=torch.float64, device=p.device)
    for t in range(K):
        if t < K0:
            i = first[:, t]
            gains[:, t] = p[at, i]
        else:
            score = torch.where(r2 > TAU * TAU, p * norms * r2.clamp_min(0).sqrt(), 0.0)
            score = score.masked_fill(taken, -1.0)
            gains[:, t], i = score.max(1)
            none = gains[:, t] <= 0
            i = torch.where(none, p.masked_fill(taken, -1.0).argmax(1), i)
            gains[:, t].clamp_min_(0)
        taken[at, i] = True
        r = r2[at, i].clamp_min(0).sqrt()
        row = S[at, i] - (C[at, :t, i][:, :, None] * C[:, :t]).sum(1) if t else S[at, i]
        C[:, t] = torch.where((r > TAU)[:, None], row / r.clamp_min(TAU)[:, None], 0.0)
        r2 = r2 - C[:, t] ** 2
    return gains


def _cosine(V):
    """Similarity and norms of V [B, N, D] in float64."""
    norms = torch.stack([v.double().norm(dim=1) for v in V])
    S = []
    for v, n in zip(V, norms):
        u = v.double() * torch.where(n > 0, 1 / n, 0.0)[:, None]
        S.append(u @ u.t())
    return torch.stack(S), norms


def _exact_decoder(case, seed):
    w, X, pos, off = _decoder_inputs(case, seed)
    d = case["d"]
    x = X.double()

    def norm(v, g):
        return v * torch.rsqrt((v * v).mean(1, keepdim=True) + 1e-6) * g.double()

    def linear(v, m):  # in pieces: the weights in 64 bits a part at a time
        return torch.cat([v @ part.double().t() for part in m.split(2048)], 1)

    qkv = linear(norm(x, w["attn_norm"]), w["w_qkv"])
    o = torch.empty_like(x)
    for a, b in zip(off, off[1:]):
        mask = torch.ones(b - a, b - a, dtype=torch.bool, device=X.device).tril()
        for h in range(d // 128):
            q, k, v = (qkv[a:b, j * d + h * 128:j * d + (h + 1) * 128] for j in range(3))
            q, k = _rope(q, pos[a:b]), _rope(k, pos[a:b])
            s = (q @ k.t() / math.sqrt(128)).masked_fill(~mask, -math.inf)
            o[a:b, h * 128:(h + 1) * 128] = torch.softmax(s, 1) @ v
    x1 = x + linear(o, w["w_o"])
    gu = linear(norm(x1, w["ffn_norm"]), w["w_gate_up"])
    g, u = gu[:, :case["ff"]], gu[:, case["ff"]:]
    return x1 + linear(torch.nn.functional.silu(g) * u, w["w_down"])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("prune", "score", "train"):
        x = _features(case, seed)
        w = {n: t.double().requires_grad_(kind == "train") for n, t in x["w"].items()}
        if kind == "train":
            p = _predict(x, w, case)
            teacher = _peaked(_gen(seed + 7919), case["B"], case["N"], 1.0).double()
            loss = torch.where(teacher > 0, teacher * (teacher.clamp_min(1e-300) / p).log(), 0.0).sum(1)
            loss.mean().backward()
            return loss.detach(), p.detach(), {n: w[n].grad for n in WEIGHT_NAMES}
        with torch.no_grad():
            p = _predict(x, w, case)
            if kind == "score":
                return p
            # in bf16 the scores' rounding decides near ties, and the gains after one follow another order
            gain = _greedy(p, *_cosine(x["V"]), case["K"], case["K0"]) if case["dtype"] == "f32" else None
        rows = ("X", "pos_x") if case["form"] == "assemble" else ("V_out", "pos_out")
        return {"idx": None, rows[0]: None, rows[1]: None, "p": p, "order": None, "gain": gain}
    if kind == "similarity":
        return _cosine(_visual(case, _gen(seed), _dtype(case)))
    if kind == "select":
        p, S, norms = _select_inputs(case, seed)
        return None, None, _greedy(p.double(), S.double(), norms.double(), case["K"], case["K0"])
    if kind == "teacher":
        A, ref, off = _attention(case, seed)
        L, H, N = case["L"], case["H"], case["N"]

        def shares(a):
            s = torch.stack([part.reshape(-1, N).sum(0, dtype=torch.float64) for part in a.reshape(L, -1, N)])
            return s / s.sum(1, keepdim=True)

        p = torch.stack([shares(A[a * L * H * N:b * L * H * N]) for a, b in zip(off, off[1:])])
        p_ref = torch.stack([shares(r) for r in ref])
        m = 0.5 * (p + p_ref)
        js = 0.5 * (torch.xlogy(p, p / m) + torch.xlogy(p_ref, p_ref / m)).sum(2)
        top = torch.argsort(js, dim=1, descending=True, stable=True)[:, :case["n_top"]]
        teacher = torch.stack([p[b, top[b]].mean(0) for b in range(case["B"])])
        return {"p": p, "p_ref": p_ref, "js": js, "layers": None, "teacher": teacher}
    return _exact_decoder(case, seed)
