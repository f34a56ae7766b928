"""The calls this library is timed on, and the ranges they stand for.

A program that uses the library holds one `Stage` per pipeline stage (or a `Pipeline` of them) and makes three kinds of
calls: patch calls (`Stage.patch_forward`, one per patch and diffusion step: nearly all the time of a run), the warm-up
pass over the whole sequence (`Stage.kv_init`, once per run and stage) and whole sampling runs (`Pipeline.run`).  The
cases below are such calls at the sizes of `workloads.CONFIGS` (the four model families at the scale the paper runs
them, and the tiny fp32 stage), with the options those models use: text rows riding along, q/k RMSNorm, RoPE on the
two-stream block, the guidance pair in one call, odd patch and text lengths.

Weights, latents and conditioning are Gaussians of the distributions `workloads.py` documents, drawn on the GPU.
"""
from __future__ import annotations

import torch

from paper_2405_14430_amd import Stage
from paper_2405_14430_amd.pipeline import Pipeline

# model families: block kind, width of the stage and the conditioning scale of workloads.CONFIGS
FAMILIES = {
    "adaln": dict(kind=0, heads=6, head_dim=64, mlp=1536, cond_std=1.0),        # C1
    "pixart": dict(kind=1, heads=16, head_dim=72, mlp=4608, cond_std=1.0),      # C2, C5
    "sd3": dict(kind=2, heads=24, head_dim=64, mlp=6144, cond_std=0.5),         # C3
    "flux": dict(kind=3, heads=24, head_dim=128, mlp=12288, cond_std=0.25),     # C4
}


def _case(name, op, family, dtype, layers, grid_h, grid_w, patches, **kw):
    """One case: `op` is "patch" (a patch call), "warmup" (the full-sequence pass) or "sample" (a whole sampling run)."""
    c = dict(op=op, family=family, dtype=dtype, layers=layers, grid_h=grid_h, grid_w=grid_w, patches=patches, patch=1,
             text=0, batch=1, with_text=False, same_cond=True, qk_norm=0, joint_rope=0, stages=1, steps=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: 64 tokens of a tiny fp32 stage, all latency and launches (C1)
        _case("tiny_fp32_patch", "patch", "adaln", "f32", 1, 16, 16, 4),
        # an fp32 stage at a real width: what a user runs to judge the bf16 path against
        _case("pixart_fp32_patch", "patch", "pixart", "f32", 1, 64, 64, 8, text=120),
        # the ordinary call of a 1024 px PixArt run: 512 of 4096 tokens, every patch but the first of a step (C2)
        _case("pixart_patch", "patch", "pixart", "bf16", 4, 64, 64, 8, text=120),
        # conditional and unconditional image of a guided run in one call
        _case("pixart_pair_patch", "patch", "pixart", "bf16", 4, 64, 64, 8, text=120, batch=2),
        # SD3-scale image-only call that derives its modulation vectors (a new conditioning embedding) (C3)
        _case("sd3_patch", "patch", "sd3", "bf16", 3, 64, 64, 8, text=154, same_cond=False),
        # the first patch of an SD3 step: the text rows ride along
        _case("sd3_text_patch", "patch", "sd3", "bf16", 3, 64, 64, 8, text=154, patch=0, with_text=True, same_cond=False),
        # two-stream block with q/k norm and RoPE on an odd image size: 375-token patches, 77 text rows, joint call
        _case("sd3_ragged_norm_patch", "patch", "sd3", "bf16", 2, 45, 75, 9, text=77, patch=4, with_text=True, qk_norm=1,
              joint_rope=1),
        # the call of a 2048 px Flux run: 2048 of 16384 tokens, 7 blocks (C4)
        _case("flux_patch", "patch", "flux", "bf16", 7, 128, 128, 8, text=512),
        # Flux blocks as the model has them (q/k RMSNorm), first patch of a step with its 512 text rows
        _case("flux_norm_text_patch", "patch", "flux", "bf16", 2, 128, 128, 8, text=512, patch=0, with_text=True, qk_norm=1,
              same_cond=False),
        # the call of a 4096 px PixArt run: 4096 of 65536 tokens (C5)
        _case("pixart_long_patch", "patch", "pixart", "bf16", 4, 256, 256, 16, text=120),
        # the synchronous first step of a Flux run: the whole sequence through the stage
        _case("flux_warmup", "warmup", "flux", "bf16", 2, 128, 128, 8, text=512),
        # a short sampling run: two stages, one warm-up step and two pipelined steps with the update between them
        _case("pixart_sample", "sample", "pixart", "bf16", 2, 64, 64, 8, text=120, stages=2, steps=3),
    ]


def draw(rng):
    """One more case of the same ranges: family, options, patch of whole grid rows (64 to 4096 tokens), 2 to 16 patches."""
    biggest = max(work(c)["flops"] for c in listed())
    biggest_f32 = max(work(c)["flops"] for c in listed() if c["dtype"] == "f32")
    while True:
        family = rng.choice(["adaln", "pixart", "pixart", "sd3", "sd3", "flux", "flux"])
        dtype = "f32" if family == "adaln" or rng.random() < 0.15 else "bf16"
        joint = family in ("sd3", "flux")
        width = rng.choice([16, 24, 32, 40, 48, 50, 64, 75, 96, 100, 128])
        rows = max(1, round(2 ** rng.uniform(6.0, 12.0) / width))     # a patch is `rows` whole rows of the grid
        patches = rng.choice([2, 3, 4, 5, 7, 8, 8, 12, 16])
        op = rng.choice(["patch"] * 5 + ["warmup", "sample"])
        if not 64 <= rows * width <= 4096 or rows * patches > 256:
            continue
        with_text = joint and op == "patch" and rng.random() < 0.4
        c = _case(None, op, family, dtype, rng.choice([1, 2, 3]), rows * patches, width, patches,
                  patch=0 if with_text else rng.randrange(patches),
                  text=0 if family == "adaln" else rng.choice([19, 37, 77, 120, 154, 256, 300, 512]), with_text=with_text,
                  batch=2 if op == "patch" and rng.random() < 0.25 else 1, same_cond=rng.random() < 0.7,
                  qk_norm=int(joint and rng.random() < 0.4), joint_rope=int(family == "sd3" and rng.random() < 0.3),
                  stages=2 if op == "sample" else 1, steps=2 if op == "sample" else 0)
        if work(c)["flops"] <= (biggest_f32 if dtype == "f32" else biggest):
            return c


def _config(case):
    f = FAMILIES[case["family"]]
    d = f["heads"] * f["head_dim"]
    return dict(kind=f["kind"], dtype=case["dtype"], n_layers=case["layers"], hidden=d, n_heads=f["heads"],
                head_dim=f["head_dim"], mlp_dim=f["mlp"], seq_img=case["grid_h"] * case["grid_w"], grid_h=case["grid_h"],
                grid_w=case["grid_w"], n_patches=case["patches"], text_len=case["text"],
                cross_dim=d if f["kind"] == 1 else 0, batch=case["batch"], qk_norm=case["qk_norm"],
                joint_rope=case["joint_rope"])


def _layer(cfg, normal):
    """Weights of one layer of one stream, as host arrays in the form `Stage` takes them."""
    d, F, kind, dh = cfg["hidden"], cfg["mlp_dim"], cfg["kind"], cfg["head_dim"]
    fan_in = cfg["dtype"] == "f32"          # fp32 stages draw N(0, 1 / fan_in), bf16 stages N(0, 0.02): see workloads.py

    def mat(out_f, in_f):
        std = in_f ** -0.5 if fan_in else 0.02
        return normal(out_f, in_f, std=std).cpu().numpy(), normal(out_f, std=std).cpu().numpy()

    w = {}
    if kind == 1:
        w["w_mod"] = mat(6, d)[0]
        w["xattn_wq"], w["xattn_bq"] = mat(d, d)
        w["xattn_wkv"], w["xattn_bkv"] = mat(2 * d, cfg["cross_dim"])
        w["xattn_wo"], w["xattn_bo"] = mat(d, d)
    else:
        w["w_mod"], w["b_mod"] = mat((3 if kind == 3 else 6) * d, d)
    w["w_qkv"], w["b_qkv"] = mat(3 * d, d)
    if kind != 3:
        w["w_o"], w["b_o"] = mat(d, d)
    w["w_up"], w["b_up"] = mat(F, d)
    w["w_down"], w["b_down"] = mat(d, d + F if kind == 3 else F)
    if cfg["qk_norm"]:
        w["q_norm_w"] = (1.0 + normal(dh, std=0.25)).cpu().numpy()
        w["k_norm_w"] = (1.0 + normal(dh, std=0.25)).cpu().numpy()
    return w


def _inputs(case, seed):
    """(configuration, layers, latent, the previous step's latent, conditioning, text, conditioning of each step)."""
    cfg = _config(case)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std)

    kind, d, L, T, B = cfg["kind"], cfg["hidden"], cfg["seq_img"], cfg["text_len"], cfg["batch"]
    lead = (B,) if B > 1 else ()
    layers = []
    for _ in range(cfg["n_layers"] * case["stages"]):
        w = _layer(cfg, normal)
        if kind == 2:
            w["txt"] = _layer(cfg, normal)
        layers.append(w)
    x = normal(*lead, L, d)
    x_prev = x + 0.05 * normal(*lead, L, d)
    cond_std = FAMILIES[case["family"]]["cond_std"]
    if kind == 1:    # the model-global modulation vector: std of a projection of SiLU(embedding) (workloads.py)
        w_std = d ** -0.5 if cfg["dtype"] == "f32" else 0.02
        cond_shape, cond_std = (*lead, 6 * d), w_std * d ** 0.5 * 0.55 * cond_std
    else:
        cond_shape = (*lead, d)
    cond = normal(*cond_shape, std=cond_std)
    text = None
    if kind == 1:
        text = normal(*lead, T, cfg["cross_dim"]).to(torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32)
    elif kind in (2, 3):
        text = normal(*lead, T, d)
    conds = [cond + 0.1 * cond_std * normal(*cond_shape) for _ in range(case["steps"])]
    return cfg, layers, x, x_prev, cond, text, conds


def _dts(case):
    return [-0.2 / case["steps"]] * case["steps"]


def prepare(case, seed):
    cfg, layers, x, x_prev, cond, text, conds = _inputs(case, seed)
    state = dict(case=case, cond=cond, text=text)
    if case["op"] == "sample":
        per = cfg["n_layers"]
        state["pipe"] = Pipeline(cfg, [layers[i * per:(i + 1) * per] for i in range(case["stages"])])
        state["kv"] = [st.kv.view(st.dt) for st in state["pipe"].stages]
        state["x"], state["conds"], state["dts"] = x, conds, _dts(case)
        return state
    stage = Stage(cfg, layers)
    state["stage"] = stage
    state["kv"] = stage.kv.view(stage.dt)          # the K/V buffers every call updates
    if case["op"] == "warmup":
        state["x"] = x_prev
        return state
    stage.kv_init(x_prev, cond, text)              # the previous step's K/V: the rows of the other patches stay stale
    n, p = cfg["seq_img"] // case["patches"], case["patch"]
    state["x"] = x[..., p * n:(p + 1) * n, :].contiguous()
    return state


def run(state):
    case = state["case"]
    if case["op"] == "sample":
        x = state["pipe"].run(state["x"], state["conds"], state["dts"], warmup_steps=1, text=state["text"])
        return {"x": x, "eps": state["pipe"].eps, "kv": state["kv"]}
    stage = state["stage"]
    if case["op"] == "warmup":
        y, text_out = stage.kv_init(state["x"], state["cond"], state["text"], want_output=True)
    elif case["with_text"]:
        y, text_out = stage.patch_forward(state["x"], state["cond"], case["patch"], text=state["text"],
                                          same_cond=case["same_cond"])
    else:
        y, text_out = stage.patch_forward(state["x"], state["cond"], case["patch"], same_cond=case["same_cond"]), None
    out = {"y": y, "kv": state["kv"]}
    if text_out is not None:
        out["text"] = text_out
    return out


def _pass_work(cfg, img_rows, text_rows, derive):
    """(flops, bytes) of one pass of the stage over img_rows image rows and text_rows text rows of each image."""
    d, F, kind, B = cfg["hidden"], cfg["mlp_dim"], cfg["kind"], cfg["batch"]
    e = 2 if cfg["dtype"] == "bf16" else 4
    T = cfg["text_len"]
    joint = kind in (2, 3)
    kv_rows = cfg["seq_img"] + (T if joint else 0)
    rows = B * (img_rows + text_rows)
    linear = 3 * d * d + (d * (d + F) if kind == 3 else d * d + d * F) + d * F      # per row and stream
    flops = 2.0 * rows * linear + 4.0 * rows * kv_rows * d
    weights = linear * (2 if kind == 2 and text_rows else 1)
    if kind == 1:
        flops += 2.0 * rows * 2 * d * d + 4.0 * rows * T * d
        weights += 2 * d * d
    elif derive:
        mod = (3 if kind == 3 else 6) * d * d * (2 if kind == 2 and text_rows else 1)
        flops += 2.0 * B * mod
        weights += mod
    # K/V of the rows this pass does not produce are read once, its own rows are written once
    kv = 2.0 * B * kv_rows * d * e + (2.0 * B * T * d * e if kind == 1 else 0.0)
    return cfg["n_layers"] * flops, cfg["n_layers"] * (weights * e + kv) + 2.0 * rows * d * 4


def work(case):
    cfg = _config(case)
    L = cfg["seq_img"]
    n = L // case["patches"]
    T = case["text"] if cfg["kind"] in (2, 3) else 0
    if case["op"] == "patch":
        flops, nbytes = _pass_work(cfg, n, T if case["with_text"] else 0, not case["same_cond"])
    elif case["op"] == "warmup":
        flops, nbytes = _pass_work(cfg, L, T, True)
    else:
        f0, b0 = _pass_work(cfg, L, T, True)                        # warm-up step
        f1, b1 = _pass_work(cfg, n, T, True)                        # first patch of a step
        f2, b2 = _pass_work(cfg, n, 0, False)                       # the others
        later, M = case["steps"] - 1, case["patches"]
        flops = case["stages"] * (f0 + later * (f1 + (M - 1) * f2))
        nbytes = case["stages"] * (b0 + later * (b1 + (M - 1) * b2)) + case["steps"] * 3.0 * L * cfg["hidden"] * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16: the path against itself through its plain kernels (kernel_path = PF_PATH_SIMT: same storage formats, sums in
    # another order) over these cases: at most 2.6e-3 (2-norm) and 2.3e-2 (largest), both in the K/V buffers.  fp32: the
    # path against the float64 oracle: at most 6.6e-7 and 8.2e-6 on one layer, stages of up to three are drawn.
    return {"rel": 5e-6, "max": 6e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.1}


class _Exact:
    """One stage in float64 and plain torch: the block of each kind over a K/V buffer that keeps the stale rows."""

    def __init__(self, cfg, layers):
        self.c = cfg
        dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32      # the form in which a stage holds its weights

        def wide(w):
            return {k: wide(v) if isinstance(v, dict) else torch.from_numpy(v).to("cuda", dt).double() for k, v in w.items()}

        self.layers = [wide(w) for w in layers]
        B, H, dh, T = cfg["batch"], cfg["n_heads"], cfg["head_dim"], cfg["text_len"]
        self.joint = cfg["kind"] in (2, 3)
        self.rows = cfg["seq_img"] + (T if self.joint else 0)
        self.pad = -(-self.rows // 128) * 128
        self.tpad = -(-max(T, 1) // 128) * 128
        self.K = [torch.zeros(B, H, self.pad, dh, dtype=torch.float64, device="cuda") for _ in layers]
        self.V = [torch.zeros_like(k) for k in self.K]
        self.KC = [torch.zeros(B, H, self.tpad, dh, dtype=torch.float64, device="cuda") for _ in layers] if cfg["kind"] == 1 else []
        self.VC = [torch.zeros_like(k) for k in self.KC]

    def kv(self):
        """The buffers as the stage lays them out: K, V transposed, cross-attention K, V transposed, layer by layer."""
        parts = []
        for l in range(len(self.layers)):
            parts += [self.K[l], self.V[l].transpose(-1, -2)]
            if self.KC:
                parts += [self.KC[l], self.VC[l].transpose(-1, -2)]
        return torch.cat([t.reshape(-1) for t in parts])

    @staticmethod
    def _lin(x, w, name):
        return x @ w["w" + name].T + w["b" + name]

    def _ln(self, x, shift, scale):
        x = x - x.mean(-1, keepdim=True)
        return x / (x.square().mean(-1, keepdim=True) + 1e-6).sqrt() * (1.0 + scale) + shift

    @staticmethod
    def _gelu(x):
        return torch.nn.functional.gelu(x, approximate="tanh")

    def _heads(self, x):
        return x.unflatten(-1, (self.c["n_heads"], self.c["head_dim"])).transpose(-2, -3)

    def _attend(self, q, K, V):
        """q [B, H, n, dh] over K, V [B, H, rows, dh], a piece of the queries of one head at a time -> [B, n, H * dh]."""
        out = torch.empty_like(q)
        step = max(1, 2 ** 27 // K.shape[2])
        for b in range(q.shape[0]):
            for h in range(q.shape[1]):
                kt, v = (K[b, h].T * q.shape[-1] ** -0.5).contiguous(), V[b, h]
                for i in range(0, q.shape[2], step):
                    s = q[b, h, i:i + step] @ kt
                    s = s.sub_(s.amax(-1, keepdim=True)).exp_()
                    out[b, h, i:i + step] = (s @ v) / s.sum(-1, keepdim=True)
        return out.transpose(1, 2).flatten(2)

    def _rotate(self, t, first):
        """t [B, H, n, dh]: first half of a head's channel pairs turned by the grid row, second half by the column."""
        n, dh = t.shape[-2:]
        tok = torch.arange(first, first + n, device="cuda", dtype=torch.float64)
        freq = 1e4 ** (-4.0 * torch.arange(dh // 4, device="cuda", dtype=torch.float64) / dh)
        ang = torch.cat([(tok // self.c["grid_w"])[:, None] * freq, (tok % self.c["grid_w"])[:, None] * freq], 1)
        a, b = t[..., 0::2], t[..., 1::2]
        return torch.stack([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()], -1).flatten(-2)

    def _project(self, l, h, w, row0, first):
        """q of rows h, their k and v written to buffer rows from row0; first: image token of the first row, or None."""
        q, k, v = (self._heads(t) for t in self._lin(h, w, "_qkv").chunk(3, -1))
        if self.c["qk_norm"]:
            q, k = (t / (t.square().mean(-1, keepdim=True) + 1e-6).sqrt() * g
                    for t, g in ((q, w["q_norm_w"]), (k, w["k_norm_w"])))
        if first is not None and (self.c["kind"] == 3 or self.c["joint_rope"]):
            q, k = self._rotate(q, first), self._rotate(k, first)
        self.K[l][:, :, row0:row0 + h.shape[1]] = k
        self.V[l][:, :, row0:row0 + h.shape[1]] = v
        return q

    def run(self, x, first, cond, text=None):
        """x [B, n, d] at image token `first` (and text [B, T, d] of the joint kinds) through every layer."""
        kind, T = self.c["kind"], self.c["text_len"]
        x, cond, d = x.double(), cond.double(), self.c["hidden"]
        row0 = first + (T if self.joint else 0)
        xt = text.double() if self.joint and text is not None else None
        for l, w in enumerate(self.layers):
            K, V = self.K[l][:, :, :self.rows], self.V[l][:, :, :self.rows]

            def modulation(w):
                m = w["w_mod"].flatten() + cond if kind == 1 else self._lin(torch.nn.functional.silu(cond), w, "_mod")
                return [t[:, None, :] for t in m.view(x.shape[0], -1, d).unbind(1)]

            streams = [(xt, w.get("txt", w), 0, None)] if xt is not None else []
            streams.append((x, w, row0, first))
            mods = [modulation(s[1]) for s in streams]
            hs = [self._ln(s[0], m[0], m[1]) for s, m in zip(streams, mods)]
            q = torch.cat([self._project(l, h, s[1], s[2], s[3]) for s, h in zip(streams, hs)], 2)
            att = self._attend(q, K, V).split([s[0].shape[1] for s in streams], 1)
            new = []
            for (xs, ws, _, _), m, h, a in zip(streams, mods, hs, att):
                if kind == 3:
                    both = torch.cat([a, self._gelu(self._lin(h, ws, "_up"))], -1)
                    new.append(xs + m[2] * self._lin(both, ws, "_down"))
                    continue
                xs = xs + m[2] * self._lin(a, ws, "_o")
                if kind == 1:
                    qc = self._heads(xs @ ws["xattn_wq"].T + ws["xattn_bq"])
                    xs = xs + self._attend(qc, self.KC[l][:, :, :T], self.VC[l][:, :, :T]) @ ws["xattn_wo"].T + ws["xattn_bo"]
                u = self._gelu(self._lin(self._ln(xs, m[3], m[4]), ws, "_up"))
                new.append(xs + m[5] * self._lin(u, ws, "_down"))
            x, xt = new[-1], new[0] if len(new) == 2 else xt
        return x, xt

    def warm_up(self, x, cond, text):
        if self.c["kind"] == 1:
            T = text.shape[1]
            for l, w in enumerate(self.layers):
                k, v = (text.double() @ w["xattn_wkv"].T + w["xattn_bkv"]).chunk(2, -1)
                self.KC[l][:, :, :T], self.VC[l][:, :, :T] = self._heads(k), self._heads(v)
        return self.run(x, 0, cond, text)


def exact(case, seed):
    cfg, layers, x, x_prev, cond, text, conds = _inputs(case, seed)
    n, B = cfg["seq_img"] // case["patches"], cfg["batch"]

    def lead(t):      # every array with its image axis
        return t if B > 1 or t is None else t[None]

    def back(t):
        return t if B > 1 else t[0]

    if case["op"] == "sample":
        per, x = cfg["n_layers"], lead(x).double()
        stages = [_Exact(cfg, layers[i * per:(i + 1) * per]) for i in range(case["stages"])]
        for step, (c, dt) in enumerate(zip(conds, _dts(case))):
            eps = torch.empty_like(x)
            for p in range(1 if step == 0 else case["patches"]):
                rows = slice(0, None) if step == 0 else slice(p * n, (p + 1) * n)
                h, t = x[:, rows], lead(text)
                for st in stages:
                    if step == 0:
                        h, t = st.warm_up(h, lead(c), lead(text) if cfg["kind"] == 1 else t)
                    else:
                        h, t = st.run(h, p * n, lead(c), t if p == 0 else None)
                eps[:, rows] = h
            x = x + dt * eps
        return {"x": back(x), "eps": back(eps), "kv": [st.kv() for st in stages]}
    st = _Exact(cfg, layers)
    y, text_out = st.warm_up(lead(x_prev), lead(cond), lead(text))
    if case["op"] == "patch":
        p = case["patch"]
        y, text_out = st.run(lead(x)[:, p * n:(p + 1) * n], p * n, lead(cond), lead(text) if case["with_text"] else None)
    out = {"y": back(y), "kv": st.kv()}
    if st.joint and text_out is not None:
        out["text"] = back(text_out)
    return out
