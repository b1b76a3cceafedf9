"""The work this library is asked to do, as cases that can be timed and compared.

A pass is one request to a program that keeps a loaded model: a noise latent and a text embedding go in, the denoised latent
comes out, after every step of the schedule (`AsyncDiff.reset`, then `AsyncDiff.step` until the schedule ends).  One kind of case
drives the components itself (`component_forward`, `precompute_text`, `ddim_update`), as a caller with a schedule of its own does,
and also returns what the components store.

listed()   the configurations of tests/configs.py with the runs they are used with, and two sizes that are not tuned for
draw(rng)  other sizes, batches, step counts, schedules and options of the same families
"""
import collections
import math

import numpy as np
import torch

import paper_2406_06911_amd as ad

DEVICE = "cuda:0"

# UNet families: channels per level, transformer depth per level and in the middle, what the text embedding looks like
SD = dict(channels="320,640,1280,1280", depth="1,1,1,0", mid=1, head_dim=64, groups=32, ctx_len=77, ctx_dim=1024, pooled=0)
SDXL = dict(channels="320,640,1280", depth="0,2,10", mid=10, head_dim=64, groups=32, ctx_len=77, ctx_dim=2048, pooled=1280)
SD_NARROW = dict(SD, channels="64,128,256,256")
SDXL_NARROW = dict(SDXL, channels="64,128,256", depth="0,1,2", mid=2, ctx_dim=256, pooled=128)
TINY = dict(channels="32,64", depth="0,0", mid=1, head_dim=16, groups=8, ctx_len=8, ctx_dim=32, pooled=0, layers=1)


def _case(family, height, width, batch, n, warmup, steps, **more):
    """family: a dict above; more: what differs from the plain run (stride 1, DDIM, bf16).  Guidance: both rows are computed and
    combined whatever the scale is.  With random weights the two predictions differ by noise, which a scale of 7.5 would multiply
    (two correct bf16 evaluations of the model then end 3-4 % apart); 1.5 keeps them within 0.7 %."""
    c = dict(kind="run", drive=0, layers=2, frames=0, heads_t=0, dtype="bf16", stride=1, wrap=False, euler=False, shift=False, graphs=True, edges=True)
    c.update(family)
    c.update(height=height, width=width, batch=batch, n=n, warmup=warmup, steps=steps, guidance=1.5 if batch == 2 and not c["frames"] else 1.0)
    c.update(more)
    return c


def listed():
    video = dict(frames=16, heads_t=8)
    cases = {
        # the smallest requests: a few dozen tiny fp32 launches per step, launched directly; latency and host work
        "tiny_f32": _case(TINY, 16, 16, 1, 2, 1, 10, dtype="f32", graphs=False, edges=False),
        # fp32 storage at a size where the arithmetic counts (reference-quality runs of a small model)
        "narrow_f32": _case(SD_NARROW, 24, 24, 2, 2, 1, 10, dtype="f32", graphs=False, edges=False),
        # small bf16 model, every launch near the floor, four components side by side
        "narrow": _case(SD_NARROW, 24, 24, 2, 4, 3, 50),
        # small model with stride denoising, Euler, pooled embedding
        "narrow_stride2": _case(SDXL_NARROW, 32, 32, 2, 4, 3, 50, stride=2, euler=True),
        # 512px model, two components, guidance: the ordinary request
        "sd_512": _case(SD, 64, 64, 2, 2, 1, 50),
        # no guidance, one component, one stream, an odd image format (576 x 320 px): plain sequential denoising, direct launches
        "sd_ragged_sequential": _case(SD, 72, 40, 1, 1, 0, 20, graphs=False, edges=False),
        # 768px model, four components, rounds without a barrier: the headline configuration
        "sd_768": _case(SD, 96, 96, 2, 4, 3, 50),
        # the same with the wrapped segmentation and a barrier around every round
        "sd_768_wrapped": _case(SD, 96, 96, 2, 4, 3, 20, wrap=True, edges=False),
        # the same model driven component by component by the caller on one stream: the first steps of a schedule
        "sd_768_components": _case(SD, 96, 96, 2, 4, 0, 20, kind="components", drive=4, graphs=False, edges=False),
        # deep transformers at 1024px, stride 2, Euler, pooled embedding: the most arithmetic per step
        "sdxl_1024": _case(SDXL, 128, 128, 2, 4, 3, 50, stride=2, euler=True),
        # sixteen frames with temporal attention: the largest activations
        "video_16f": _case(SD, 64, 64, 16, 4, 2, 25, **video),
    }
    return [dict(name=k, **v) for k, v in cases.items()]


def _log_int(rng, lo, hi, multiple):
    """A multiple of `multiple` between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / multiple)) * multiple))


def draw(rng):
    family = rng.choice(["sd", "sd", "sd", "sdxl", "video", "narrow", "narrow", "narrow_xl", "narrow_video", "tiny"])
    n = rng.randint(1, 4)
    more = dict(stride=rng.choice([1, 1, 1, 2, 3]), euler=rng.random() < 0.3, shift=rng.random() < 0.2,
                graphs=rng.random() < 0.7, edges=rng.random() < 0.6, ctx_len=rng.choice([77, 77, 77, 16, 120, 154]))
    if n >= 2 and rng.random() < 0.15:
        more.update(wrap=True, stride=1)
    elif rng.random() < 0.15:
        more.update(kind="components", drive=rng.randint(1, 4), stride=1, shift=False)
    steps = rng.randint(4, 30)
    warmup = rng.randint(1, 3)
    batch = rng.choice([1, 2, 2])
    if family == "sd":
        h, w = _log_int(rng, 32, 96, 8), _log_int(rng, 32, 96, 8)
        return _case(dict(SD, ctx_dim=rng.choice([768, 1024])), h, w, batch, n, warmup, steps, **more)
    if family == "sdxl":
        h, w = _log_int(rng, 48, 128, 4), _log_int(rng, 48, 128, 4)
        return _case(SDXL, h, w, batch, n, warmup, min(steps, 16), **more)
    if family == "video":
        frames = rng.randint(2, 16)
        h, w = _log_int(rng, 32, 64, 8), _log_int(rng, 32, 64, 8)
        return _case(SD, h, w, frames, n, warmup, min(steps, 12), frames=frames, heads_t=8, **more)
    if family == "narrow_video":
        frames = rng.randint(2, 16)
        return _case(SD_NARROW, _log_int(rng, 8, 32, 8), _log_int(rng, 8, 32, 8), frames, n, warmup, steps, frames=frames, heads_t=8, **more)
    more["dtype"] = rng.choice(["bf16", "bf16", "f32"])
    if family == "narrow":
        return _case(SD_NARROW, _log_int(rng, 16, 64, 8), _log_int(rng, 16, 64, 8), batch, n, warmup, steps, **more)
    if family == "narrow_xl":
        return _case(SDXL_NARROW, _log_int(rng, 16, 64, 4), _log_int(rng, 16, 64, 4), batch, n, warmup, steps, **more)
    more.update(dtype="f32", ctx_len=rng.choice([8, 16, 77]))
    return _case(TINY, _log_int(rng, 8, 32, 2), _log_int(rng, 8, 32, 2), batch, min(n, 3), warmup, steps, **more)


# ---- what a program keeps: loaded models and streams ------------------------------------------------------------------

def _config(case):
    ints = lambda s: [int(v) for v in s.split(",")]
    return dict(latent_channels=4, height=case["height"], width=case["width"], batch=case["batch"], channels=ints(case["channels"]),
                layers_per_block=case["layers"], transformer_depth=ints(case["depth"]), mid_depth=case["mid"], head_dim=case["head_dim"],
                gn_groups=case["groups"], ctx_len=case["ctx_len"], ctx_dim=case["ctx_dim"], pooled_dim=case["pooled"], frames=case["frames"],
                temporal_heads=case["heads_t"])


def _create(case):
    dtype = ad.AD_BF16 if case["dtype"] == "bf16" else ad.AD_F32
    warmup = max(case["warmup"], 1) if case["n"] > 1 else case["warmup"]
    return ad.AsyncDiff(_config(case), case["n"], warmup, case["stride"], dtype, wrap=case["wrap"])


_POOL = []                                    # N(0, 1) numbers the weights are cut from
_MODELS = collections.OrderedDict()           # model parameters -> loaded model; the last few
_STREAMS = []


def _pool():
    if not _POOL:
        g = torch.Generator(device=DEVICE)
        g.manual_seed(1000)
        _POOL.append(torch.randn(48 << 20, generator=g, device=DEVICE).cpu().numpy())
    return _POOL[0]


def _weights(manifest, std):
    """Weights and biases N(0, std); normalisation gains about 1, offsets about 0."""
    pool = _pool()
    scaled = pool * np.float32(std)
    out = {}
    for i, (name, shape) in enumerate(manifest):
        size = int(np.prod(shape))
        at = (i * 7919 * 64) % (pool.size - size)
        norm = len(shape) == 1 and name.rsplit(".", 2)[-2][:2] in ("gn", "ln")
        if norm:
            part = pool[at:at + size] * np.float32(0.1)
            out[name] = part + np.float32(1.0) if name.endswith(".g") else part
        else:
            out[name] = scaled[at:at + size].reshape(shape)
    return out


def _model(case):
    key = tuple((k, v) for k, v in sorted(case.items()) if k not in ("name", "kind", "drive", "steps", "euler", "shift", "graphs", "edges", "guidance"))
    if key in _MODELS:
        _MODELS.move_to_end(key)
        return _MODELS[key]
    while len(_MODELS) >= 12:
        torch.cuda.synchronize()
        _MODELS.popitem(last=False)[1].close()
    m = _create(case)
    m.allocate(DEVICE)
    # activations keep about unit size: 0.02 suits the 320-channel models
    m.load_weights(_weights(m.weight_manifest(), 0.02 * math.sqrt(320 / int(case["channels"].split(",")[0]))))
    _MODELS[key] = m
    return m


def _streams(count):
    while len(_STREAMS) < count:
        _STREAMS.append(torch.cuda.Stream(device=DEVICE))
    return _STREAMS[:count]


# ---- a pass -------------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    streams = _streams(6)
    m = _model(case)
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    frames = case["frames"]
    shape = (4, case["height"], case["width"])
    noise = torch.randn((frames,) + shape if frames else shape, generator=g, device=DEVICE)
    text = torch.randn(1 if frames else case["batch"], case["ctx_len"], case["ctx_dim"], generator=g, device=DEVICE)
    text = text.to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)
    pooled = torch.randn(case["batch"], case["pooled"], generator=g, device=DEVICE) if case["pooled"] else None
    state = dict(case=case, model=m, text=text, pooled=pooled, streams=streams[:case["n"] + case["stride"] - 1])
    sampler = ad.AD_EULER if case["euler"] else ad.AD_DDIM
    state["reset"] = lambda: m.reset(case["steps"], sampler=sampler, cfg_scale=case["guidance"], time_shift=case["shift"])
    m.reset(case["steps"], sampler=sampler)
    state["noise"] = noise * m.sampler_coeffs(0)[3]
    if case["kind"] == "components":
        store = {}
        parts = len(m.partition())
        for comp in range(1, parts + 1):
            for u in m.component_io(comp)[1]:
                b, h, w, c = m.tensor_shape(u)[0]
                last = comp == parts
                store[u] = torch.empty((b, c, h, w) if last else (b, h, w, c), device=DEVICE, dtype=torch.float32 if last else text.dtype)
        state["store"] = store
        state["io"] = [m.component_io(comp) for comp in range(1, parts + 1)]
    return state


def run(state):
    case, m, streams, text, pooled = (state[k] for k in ("case", "model", "streams", "text", "pooled"))
    here = torch.cuda.current_stream()
    streams[0].wait_stream(here)
    state["reset"]()
    if case["kind"] == "components":
        return _run_components(state, here)
    m.set_graph_mode(case["graphs"])
    m.set_edge_mode(case["edges"])
    with torch.cuda.stream(streams[0]):
        latent = state["noise"].clone()
    for s in streams[1:]:
        s.wait_stream(streams[0])
    while m.step(latent, text, streams, pooled=pooled) is not None:
        pass
    for s in streams:
        here.wait_stream(s)
        latent.record_stream(s)
    return latent


def _run_components(state, here):
    """The components one after the other, every step on fresh inputs."""
    case, m, text, pooled, store = (state[k] for k in ("case", "model", "text", "pooled", "store"))
    s = state["streams"][0]
    with torch.cuda.stream(s):
        latent = state["noise"].clone()
    m.precompute_text(text, s)
    last = len(m.units()) - 1
    for i in range(case["drive"]):
        scale = m.sampler_coeffs(i)[2]
        for comp, (ins, outs) in enumerate(state["io"], 1):
            m.component_forward(comp, [latent if u < 0 else store[u] for u in ins], i, text, [store[u] for u in outs], s, latent_scale=scale,
                                pooled=pooled)
        m.ddim_update(latent, store[last], i, case["guidance"], s)
    here.wait_stream(s)
    return [latent] + [store[u] for u in sorted(store)]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------

def work(case):
    """Multiply-adds of every component evaluation of the schedule, the text keys and values once.  Bytes: every evaluation reads
    its weights once (no cache holds them from one step to the next) and the stored tensors it takes, and writes those it
    gives; activations inside a component are not counted."""
    m = _create(case)
    m.reset(case["steps"])
    es = 2 if case["dtype"] == "bf16" else 4
    units, parts, rows = m.units(), m.partition(), m.schedule()
    if case["kind"] == "components":
        evals = [comp for _ in range(case["drive"]) for comp in range(1, len(parts) + 1)]
    else:
        evals = [r[1] for r in rows]
    text_rows = (1 if case["frames"] else case["batch"]) * case["ctx_len"]
    text_flops = lambda u: 4 * text_rows * u.c_in * case["ctx_dim"] * u.depth          # depth is 0 outside the transformers
    flops = [sum(u.flops - text_flops(u) for u in units[a:b + 1]) for a, b in parts]
    names = [u.name.decode() for u in units]
    where = {nm: k for k, (a, b) in enumerate(parts) for nm in names[a:b + 1]}
    size = [0] * len(parts)
    for name, shape in m.weight_manifest():
        n = int(np.prod(shape)) * es
        unit = next((nm for nm in names if name.startswith(nm + ".")), None)
        for k in range(len(parts)) if unit is None else [where[unit]]:       # the time embedding is part of every component
            size[k] += n
    for k in range(len(parts)):
        ins, outs = m.component_io(k + 1)
        size[k] += sum(m.tensor_shape(u)[1] for u in ins) + sum(m.tensor_shape(u)[1] for u in outs)
    m.close()
    return {"bytes": float(sum(size[c - 1] for c in evals)),
            "flops": float(sum(flops[c - 1] for c in evals) + sum(text_flops(u) for u in units))}


def tolerance(case):
    """Four times what the outputs move by when the same sums are taken in another order (other tiles, other splits of K): bf16
    2.6e-3 .. 6.6e-3 for a final latent, 1.6e-2 for the hidden states of the last component; fp32: 8e-7 against the same
    model in 64 bits at the listed sizes, more where the sums are longer."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 5e-5}
    return {"rel": 0.03, "max": 0.4} if case["kind"] == "components" else {"rel": 0.025, "max": 0.15}
