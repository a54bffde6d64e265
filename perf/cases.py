"""The work that a user of this library has it do, as a list of timed cases.

Four kinds of case:

layer      one cached-activation convolution on an edited input: difference mask and block list, then the
           convolution on the active blocks, scattered into the cached output.  "how" names the calls a program
           makes: "fused" (reduction, fused convolution), "pair" (marking pass, 3x3 and 1x1 shortcut in the
           shared launch), "calls" (reduction, gather, convolution, scatter).  The arguments are marshalled once
           with api.record(), as a serving loop does.
attention  the edited tokens' queries against all cached keys and values (also recorded once).
unet       a denoising network: "step" is one sparse step of an edit, replayed from the HIP graph that a sampler
           captures once per edit; "precompute" is the dense pass on a new original image, called eagerly.
generator  an interactive label edit: the new label map is compared with the current one, the block lists are
           rebuilt (one readback each) and the active blocks of every layer are updated, called eagerly.

Everything is drawn on the GPU from the case's seed: activations N(0, 1), weights N(0, 1 / fan_in), edits made of
a few ellipses or a rectangle with fresh noise inside them.
"""
from __future__ import annotations

import math

import torch

from paper_2211_02048_amd import api, inputs
from paper_2211_02048_amd.layers import BlockList, SigeConv, Workspace
from paper_2211_02048_amd.spade import SigeSpade
from paper_2211_02048_amd.unet import SigeUNet

DEV = "cuda"
DDPM_CHANNELS = (128, 128, 256, 256, 512, 512)
LATENT_CHANNELS = (320, 640, 1280, 1280)
GENERATOR_CHANNELS = (1024, 1024, 1024, 512, 256, 128, 64)


def listed():
    return [
        # the smallest layer in use: 64x64x64, fp32, 6x6 blocks, one rectangle; two or three launches, all latency
        dict(name="layer_64_fp32", kind="layer", how="fused", dtype="f32", H=64, W=64, cin=64, cout=64, cs=0, block=6,
             gn=False, area=0.05),
        # a ResBlock entry at 256x256: GroupNorm + SiLU + 3x3 and the 1x1 shortcut, a 1 % edit
        dict(name="layer_256_pair", kind="layer", how="pair", dtype="f16", H=256, W=256, cin=128, cout=128, cs=256,
             block=16, gn=True, area=0.01),
        # the same resolution at the paper's 15.5 % edit, as the separate calls (gather, convolution, scatter)
        dict(name="layer_256_calls", kind="layer", how="calls", dtype="f16", H=256, W=256, cin=128, cout=128, cs=0,
             block=16, gn=True, area=0.155),
        # the largest: every block of a 1024x1024 image edited; memory and matrix cores, no latency
        dict(name="layer_1024_all", kind="layer", how="fused", dtype="f16", H=1024, W=1024, cin=128, cout=128, cs=0,
             block=16, gn=True, area=1.0),
        # the first self-attention of a latent-diffusion model on 512x512 images, a small edit (six 4x4 blocks)
        dict(name="attention_4096_96q", kind="attention", dtype="bf16", T=4096, heads=8, d=40, nq=96),
        # the paper's counting example: 64x128 tokens, 672 edited queries
        dict(name="attention_8192_672q", kind="attention", dtype="bf16", T=8192, heads=8, d=40, nq=672),
        # pixel-space denoiser: one step of a 1.2 % and of a 15.5 % edit, and the dense pass before them
        dict(name="ddpm_step_1pct", kind="unet", net="ddpm", run="step", dtype="f16", res=256, area=0.012),
        dict(name="ddpm_step_15pct", kind="unet", net="ddpm", run="step", dtype="f16", res=256, area=0.155),
        dict(name="ddpm_precompute", kind="unet", net="ddpm", run="precompute", dtype="f16", res=256, area=0.0),
        # latent-space denoiser with transformer blocks: one step of a 1 % and of a 20 % edit
        dict(name="latent_step_1pct", kind="unet", net="latent", run="step", dtype="bf16", res=64, area=0.01),
        dict(name="latent_step_20pct", kind="unet", net="latent", run="step", dtype="bf16", res=64, area=0.20),
        # a 1 % label edit of the conditional generator at 256x512
        dict(name="generator_edit", kind="generator", dtype="f16", h0=8, w0=16, area=0.01),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "attention", "attention", "unet", "unet", "unet", "generator"])
    if kind == "layer":
        how = rng.choice(["fused", "pair", "calls"])
        dtype = rng.choice(["f16", "f16", "bf16", "f32"])
        while True:
            H, W = int(_log(rng, 40, 1024)), int(_log(rng, 40, 1024))
            cin, cout = 16 * round(_log(rng, 2, 32)), 16 * round(_log(rng, 2, 32))
            area = _log(rng, 0.005, 1.0)
            s = 4 if dtype == "f32" else 2
            if H * W * max(cin, cout) * s <= 2 ** 28 and H * W * cin * cout * area * (16 if dtype == "f32" else 1) <= 2 ** 34:
                break
        cs = 16 * round(_log(rng, 2, 32)) if how == "pair" else 0
        return dict(kind="layer", how=how, dtype=dtype, H=H, W=W, cin=cin, cout=cout, cs=min(cs, 2 * cin),
                    block=rng.choice([6, 8, 16, 16]), gn=rng.random() < 0.7 and cin % 32 == 0, area=round(area, 4))
    if kind == "attention":
        dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
        T = int(_log(rng, 200, 4096 if dtype == "f32" else 9216))
        return dict(kind="attention", dtype=dtype, T=T, heads=rng.choice([1, 2, 4, 8]),
                    d=rng.choice([32, 40, 64, 80, 128, 160]), nq=max(24, int(T * _log(rng, 0.01, 1.0))))
    if kind == "unet":
        area = round(_log(rng, 0.005, 0.25), 4)
        if rng.random() < 0.5:
            run = "precompute" if rng.random() < 0.25 else "step"
            return dict(kind="unet", net="ddpm", run=run, dtype=rng.choice(["f16", "f16", "bf16"]),
                        res=32 * rng.randint(2, 8), area=0.0 if run == "precompute" else area)
        run = "precompute" if rng.random() < 0.2 else "step"
        return dict(kind="unet", net="latent", run=run, dtype=rng.choice(["bf16", "bf16", "f16"]),
                    res=32 if run == "precompute" else rng.choice([32, 64, 64]),
                    area=0.0 if run == "precompute" else min(area, 0.2))
    h0 = rng.choice([4, 6, 8])
    return dict(kind="generator", dtype="f16", h0=h0, w0=h0 * rng.choice([1, 2]), area=round(_log(rng, 0.004, 0.15), 4))


# ---- inputs ------------------------------------------------------------------------------------------------------

class _Draws:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device=DEV).manual_seed(seed)
        self.td = inputs.DTYPES[dtype]

    def normal(self, *shape, sigma=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * sigma

    def uniform(self, lo, hi, n):
        return (torch.rand(n, generator=self.g, device=DEV) * (hi - lo) + lo).tolist()

    def weight(self, cout, cin, k, gain=1.0):
        return self.normal(cout, cin, k, k, sigma=gain / math.sqrt(cin * k * k)).to(self.td)

    def bias(self, n, sigma=0.1):
        return self.normal(n, sigma=sigma)

    def norm(self, n):
        """gamma ~ N(1, 0.1), beta ~ N(0, 0.1) (variances)."""
        return 1.0 + self.normal(n, sigma=math.sqrt(0.1)), self.normal(n, sigma=math.sqrt(0.1))

    def edit_mask(self, H, W, area, rect=False):
        """u8 [H, W]: one rectangle, or the union of three ellipses scaled until it covers the area."""
        m = torch.zeros((H, W), dtype=torch.uint8, device=DEV)
        if area >= 1.0:
            return m.fill_(1)
        if rect:
            fy, uy, ux = self.uniform(0, 1, 3)
            h = min(H, max(1, int(H * (0.125 + 0.25 * fy))))
            w = max(1, min(W, round(area * H * W / h)))
            y0, x0 = int(uy * (H - h + 0.999)), int(ux * (W - w + 0.999))
            m[y0:y0 + h, x0:x0 + w] = 1
            return m
        n = 3
        cy, cx = self.uniform(0, H, n), self.uniform(0, W, n)
        a, b, th = self.uniform(5, 12, n), self.uniform(5, 12, n), self.uniform(0, math.pi, n)
        yy = torch.arange(H, device=DEV, dtype=torch.float64)[:, None]
        xx = torch.arange(W, device=DEV, dtype=torch.float64)[None, :]
        r2 = None
        for i in range(n):
            dy, dx = yy - cy[i], xx - cx[i]
            u = (dx * math.cos(th[i]) + dy * math.sin(th[i])) / a[i]
            v = (dy * math.cos(th[i]) - dx * math.sin(th[i])) / b[i]
            q = u * u + v * v
            r2 = q if r2 is None else torch.minimum(r2, q)
        # the union of the scaled ellipses is {r2 <= s^2}: the scale is a quantile of r2
        k = max(1, round(area * H * W))
        return (r2 <= torch.kthvalue(r2.flatten(), k).values).to(torch.uint8)


def _edited(dr, H, W, C, mask, sigma):
    a_o = dr.normal(H, W, C)
    a_e = (a_o + dr.normal(H, W, C, sigma=sigma)).to(dr.td)
    a_o = a_o.to(dr.td)
    return a_o, torch.where(mask.bool()[:, :, None], a_e, a_o).contiguous()


def _pow2(n):
    return 1 << max(0, (n - 1).bit_length())


def _prepare_layer(c, seed):
    dr = _Draws(seed, c["dtype"])
    H, W, cin, cout, cs, b = c["H"], c["W"], c["cin"], c["cout"], c["cs"], c["block"]
    a_o, a_e = _edited(dr, H, W, cin, dr.edit_mask(H, W, c["area"], rect=not c["gn"]), math.sqrt(0.5))
    main = SigeConv(dr.weight(cout, cin, 3), dr.bias(cout), H, W, b, 1, 1)
    short = SigeConv(dr.weight(cs, cin, 1), dr.bias(cs), H, W, b, 1, 0) if cs else None
    scale = shift = None
    act = api.ACT_NONE
    if c["gn"]:
        gamma, beta = dr.norm(cin)
        scale, shift = torch.zeros(cin, device=DEV), torch.zeros(cin, device=DEV)
        mean, var = torch.zeros(32, device=DEV), torch.zeros(32, device=DEV)
        api.sige_gn_stats(a_o, 32, mean, var, gamma=gamma, beta=beta, scale=scale, shift=shift)
        act = api.ACT_SILU
    # the cached outputs, from one pass with every block active on the original input
    ws = Workspace(DEV)
    y = torch.empty((H, W, cout), dtype=dr.td, device=DEV)
    main.forward(a_o, y, BlockList(main.g, DEV).all_active(), ws, scale=scale, shift=shift, act=act, fused=True)
    ys = None
    if short is not None:
        ys = torch.empty((H, W, cs), dtype=dr.td, device=DEV)
        short.forward(a_o, ys, BlockList(short.g, DEV).all_active(), ws, fused=True)
    mask = torch.zeros((H, W), dtype=torch.uint8, device=DEV)
    # launches sized for this edit (one readback), counts left on the device as in a captured step
    convs = [main] + ([short] if short is not None else [])
    lists = [BlockList(cv.g, DEV) for cv in convs]
    caps = []
    for bl in lists:
        bl.reduce(a_orig=a_o, a_edit=a_e, mask_out=mask)
        caps.append(max(8, _pow2(bl.sync_count())))
        bl.n_host = -1
    for bl in lists:
        bl.max_blocks = min(bl.g.grid_blocks, max(caps))
    st = dict(ws=ws, y=y, ys=ys, mask=mask, lists=lists, keep=(a_o, a_e, main, short, scale, shift))

    def body():
        if c["how"] == "pair":
            BlockList.mark_together(lists, a_orig=a_o, a_edit=a_e, mask_out=mask)
            first, _ = main.fused_call(a_e, y, lists[0], ws, scale=scale, shift=shift, act=act, tag="main")
            second, _ = short.fused_call(a_e, ys, lists[1], ws, tag="short")
            api.sige_fused_conv_pair_marked(first, second, [bl.desc() for bl in lists])
            st["keep_calls"] = (first, second)
        else:
            lists[0].reduce(a_orig=a_o, a_edit=a_e, mask_out=mask)
            main.forward(a_e, y, lists[0], ws, scale=scale, shift=shift, act=act, fused=c["how"] == "fused")

    with api.record() as calls:
        body()
    st["calls"] = calls
    st["out"] = dict(y=y, mask=mask, counts=[bl.count for bl in lists], lists=[bl.indices for bl in lists])
    if ys is not None:
        st["out"]["shortcut"] = ys
    return st


def _prepare_attention(c, seed):
    dr = _Draws(seed, c["dtype"])
    T, h, d, nq = c["T"], c["heads"], c["d"], c["nq"]
    q, k, v = (dr.normal(n, h, d).to(dr.td) for n in (nq, T, T))
    o = torch.zeros_like(q)
    nb = api.sige_sparse_attn_workspace_bytes(nq, T, h, d)
    ws = torch.empty(nb // 4, dtype=torch.float32, device=DEV) if nb else None
    with api.record() as calls:
        api.sige_sparse_attn(q, k, v, o, 1.0 / math.sqrt(d), workspace=ws)
    return dict(calls=calls, out=o, keep=(q, k, v, ws))


def _unet_params(dr, ops, in_ch):
    """inputs.unet_params' distributions, drawn on the GPU."""
    P = {}

    def linear(name, cout, cin, k=1):
        P[name + ".w"], P[name + ".b"] = dr.weight(cout, cin, k), dr.bias(cout)

    def norm(name, n):
        P[name + ".gamma"], P[name + ".beta"] = dr.norm(n)

    for op in ops:
        n, cin = op["name"], op["x"][2]
        if op["kind"] == "conv":
            y = op["y"] if op["y"] is not None else next(o["y"] for o in ops if o.get("shortcut") == n)
            linear(n, y[2], cin, op["k"])
            if n == "conv_in":
                P[n + ".w"][:, in_ch:] = 0
            if n == "conv_out":
                P[n + ".w"][in_ch:] = 0
                P[n + ".b"][in_ch:] = 0
            if op["gn"]:
                norm(n, cin)
            continue
        norm(n, cin)
        if op["kind"] == "attn":
            for part in "qkvo":
                linear(f"{n}.{part}", cin, cin)
            continue
        for ln in ("ln1", "ln2", "ln3"):
            norm(f"{n}.{ln}", cin)
        for part in ("in", "q1", "k1", "v1", "o1", "q2", "o2", "out"):
            linear(f"{n}.{part}", cin, cin)
        for part in ("k2", "v2"):
            linear(f"{n}.{part}", cin, op["d_ctx"])
        linear(n + ".ff1", 8 * cin, cin)
        linear(n + ".ff2", cin, 4 * cin)
        if "ctx" not in P:
            P["ctx"] = dr.normal(op["n_ctx"], op["d_ctx"]).to(dr.td)
    return P


def _unet_config(c):
    """(constructor arguments, image channels) of the case's network."""
    r = c["res"]
    if c["net"] == "ddpm":
        return dict(res=r, channels=DDPM_CHANNELS, attn_res=(r // 16,), heads=4, block=16,
                    min_sparse_res=r // 4), 3
    return dict(res=r, channels=LATENT_CHANNELS, attn_res=(r, r // 2, r // 4), heads=8, block=8,
                min_sparse_res=max(16, r // 4), in_ch=4, attn_kind="xfmr", ctx=(77, 768)), 4


def _unet_topology(cfg):
    return inputs.unet_topology(cfg["res"], cfg.get("in_ch", 3), cfg["channels"], cfg["attn_res"], cfg["heads"],
                                attn_kind=cfg.get("attn_kind", "attn"), ctx=cfg.get("ctx", (77, 768)))


def _prepare_unet(c, seed):
    dr = _Draws(seed, c["dtype"])
    cfg, in_ch = _unet_config(c)
    r = c["res"]
    net = SigeUNet(dtype=c["dtype"], device=DEV, params=_unet_params(dr, _unet_topology(cfg)[1], in_ch), **cfg)
    mask = dr.edit_mask(r, r, c["area"]) if c["area"] else torch.zeros((r, r), dtype=torch.uint8, device=DEV)
    pad = torch.zeros((r, r, 16 - in_ch), dtype=dr.td, device=DEV)
    a_o, a_e = (torch.cat([a, pad], 2).contiguous() for a in _edited(dr, r, r, in_ch, mask, 1.0))
    st = dict(net=net, image=a_o, out=dict(net.B))
    for n, L in net.layers.items():
        if L["op"]["kind"] == "xfmr":
            st["out"][n + ".qkv"] = L["qkv"]
    if c["run"] == "step":
        net.precompute(a_o)
        # transformer blocks size their calls by the counts; the others leave them on the device
        net.set_edit(mask, exact=c["net"] == "latent")
        st["graph"] = net.capture(a_e)
        st["image"] = a_e
    return st


def _generator_topology(c):
    h, w = c["h0"], c["w0"]
    return dict(out_hw=(32 * h, 32 * w), start_hw=(h, w), channels=GENERATOR_CHANNELS, stats_cached_above=(2 * h, 2 * w))


def _prepare_generator(c, seed):
    dr = _Draws(seed, c["dtype"])
    topo = _generator_topology(c)
    bufs, ops = inputs.spade_topology(**topo)
    P = {"z": dr.normal(*bufs["z"]).to(dr.td)}
    for op in ops:
        if op["kind"] != "conv":
            continue
        n = op["name"]
        gb = n.endswith(".gb")      # modulation convolutions: 1 + gamma stays near one
        P[n + ".w"] = dr.weight(op["cout"], op["cin"], op["k"], 0.25 if gb else 1.0)
        P[n + ".b"] = dr.bias(op["cout"], 0.0 if n.endswith(".short") else 0.025 if gb else 0.1)
    net = SigeSpade(topo=topo, dtype=c["dtype"], device=DEV, params=P, min_sparse=(c["h0"], c["w0"]))
    H, W = topo["out_hw"]
    # a label map of 40 regions (nearest seed) with random classes, and the same with three ellipses relabelled
    cy, cx = torch.tensor(dr.uniform(0, H, 40), device=DEV), torch.tensor(dr.uniform(0, W, 40), device=DEV)
    cls = torch.randint(0, 35, (40,), generator=dr.g, device=DEV)
    dist = ((torch.arange(H, device=DEV)[:, None, None] - cy) ** 2 + (torch.arange(W, device=DEV)[None, :, None] - cx) ** 2)
    lab = cls[dist.argmin(-1)]
    m = dr.edit_mask(H, W, c["area"]).bool()
    new = torch.where(m, (lab + torch.randint(1, 35, (1,), generator=dr.g, device=DEV)) % 35, lab)

    def pyramid(labels):
        out = {}
        for (h, w) in net.seg_sizes:
            oh = torch.zeros((h, w, 48), dtype=dr.td, device=DEV)
            out[(h, w)] = oh.scatter_(2, labels[::H // h, ::W // w].unsqueeze(-1), 1.0)
        return out

    maps = [pyramid(new), pyramid(lab)]
    net.precompute(maps[1])
    keep = {n: t for n, t in net.B.items() if n != "z" and not n.startswith("seg")}
    return dict(net=net, maps=maps, turn=0, out=keep)


def prepare(case, seed):
    return {"layer": _prepare_layer, "attention": _prepare_attention, "unet": _prepare_unet,
            "generator": _prepare_generator}[case["kind"]](case, seed)


def run(state):
    if "calls" in state:
        state["calls"].run()
    elif "graph" in state:
        state["graph"].replay()
    elif "maps" in state:        # the user edits the labels and takes the edit back, turn by turn
        state["net"].set_edit(state["maps"][state["turn"]])
        state["turn"] ^= 1
        state["net"].step()
    else:
        state["net"].precompute(state["image"])
    return state["out"]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------

def _size(dtype):
    return 4 if dtype == "f32" else 2


def work(case):
    c, s = case, _size(case["dtype"])
    if c["kind"] == "layer":
        px = c["H"] * c["W"]
        wide = c["cout"] + c["cs"]
        w = 9 * c["cin"] * c["cout"] + c["cin"] * c["cs"]
        # both activations compared, the mask written, the edited pixels' outputs written, the weights read
        return dict(bytes=2 * px * c["cin"] * s + px + c["area"] * px * wide * s + w * s, flops=2 * c["area"] * px * w)
    if c["kind"] == "attention":
        ch = c["heads"] * c["d"]
        return dict(bytes=(2 * c["T"] + 2 * c["nq"]) * ch * s, flops=4 * c["nq"] * c["T"] * ch)
    if c["kind"] == "unet":
        cfg, _ = _unet_config(c)
        bufs, ops = _unet_topology(cfg)
        dense = c["run"] == "precompute"
        nbytes = flops = 0.0
        for op in ops:
            r, cin = bufs[op["x"][0]][0], op["x"][2]
            f = 1.0 if dense or r < cfg["min_sparse_res"] else c["area"]
            tok = f * r * r
            if op["kind"] == "conv":
                y = op["y"] if op["y"] is not None else next(o["y"] for o in ops if o.get("shortcut") == op["name"])
                w = op["k"] ** 2 * cin * y[2]
                out = tok * 4 if op["up"] else tok / op["stride"] ** 2
                nbytes += (w + tok * cin + out * y[2]) * s
                flops += 2 * out * w
            elif op["kind"] == "attn":
                w = 4 * cin * cin
                nbytes += (w + 2 * tok * cin) * s
                flops += 2 * tok * w + 4 * tok * r * r * cin
            else:
                w = 20 * cin * cin
                kv = 2 * op["n_ctx"] * op["d_ctx"] * cin if dense else 0
                nbytes += (w + (2 * op["d_ctx"] * cin if dense else 0) + 2 * tok * cin + 2 * r * r * cin) * s
                flops += 2 * tok * w + 4 * tok * (r * r + op["n_ctx"]) * cin + 2 * kv
        return dict(bytes=nbytes, flops=flops)
    topo = _generator_topology(c)
    bufs, ops = inputs.spade_topology(**topo)
    nbytes = 2 * 32 * 32 * c["h0"] * c["w0"] * 48 * s      # the two label maps compared
    flops = 0.0
    for op in ops:
        h, w_ = op["hw"]
        px = h * w_ * (c["area"] if h > c["h0"] else 1.0)
        if op["kind"] != "conv":
            nbytes += px * 1.25 * op["cin"] * s
            continue
        w = op["k"] ** 2 * op["cin"] * op["cout"]
        nbytes += (w + px * (op["cin"] + op["cout"])) * s
        flops += 2 * px * w
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """About four times what the same pass with its sums in another order differs by (other shapes and splits of
    the products chosen through api.knobs; relative 2-norm and largest difference seen):
    layer      f32 7e-7 on the active part, 2.2e-6; f16 4e-5 (few values round the other way), 9.8e-4 (one unit of
               the last place); bf16 has eight times f16's unit
    attention  f16 2.5e-4 and 1e-3; bf16 9e-5 and 7.8e-3; f32 like the layers
    networks   f16 denoiser 1.6e-3 and 2.2e-2, f16 transformers 1.7e-3 and 1.2e-2, generator 1.3e-3 and 7.3e-3; a bf16
               chain differs from itself by 1.8e-2 and 0.13 (statistics of the dense pass are summed with atomics)
    """
    half = case["dtype"] == "f16"
    if case["kind"] == "layer":
        return {"f32": dict(rel=4e-6, max=2e-5), "f16": dict(rel=2e-4, max=4e-3),
                "bf16": dict(rel=1.5e-3, max=3e-2)}[case["dtype"]]
    if case["kind"] == "attention":
        return {"f32": dict(rel=4e-6, max=2e-5), "f16": dict(rel=1e-3, max=4e-3),
                "bf16": dict(rel=4e-4, max=3e-2)}[case["dtype"]]
    if case["kind"] == "generator":
        return dict(rel=5e-3, max=3e-2)
    return dict(rel=7e-3, max=9e-2) if half else dict(rel=3e-2, max=0.5)
