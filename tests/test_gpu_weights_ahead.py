"""A launch that asks for the weights of a later one computes what it computes without: which launches ask depends on where the model is cut."""
import numpy as np
import pytest
import torch

from paper_2406_06911_amd import binding as B

pytestmark = pytest.mark.gpu


def run(d, cuts, weights, noise, text, steps):
    n = len(cuts) + 1
    m = B.AsyncDiff(d, n, steps if n > 1 else 0, 1, B.AD_BF16, cuts=cuts or None)
    m.allocate("cuda:0")
    m.load_weights(weights(m.weight_manifest()))
    m.reset(steps)
    latent = noise.clone()
    streams = [torch.cuda.Stream(device="cuda:0")]
    torch.cuda.synchronize()
    while m.step(latent, text, streams) is not None:
        pass
    torch.cuda.synchronize()
    bytes_ = m.device_bytes()[0]
    m.close()
    return latent.cpu(), bytes_


# rows around the line of 512 (batch 1 and 2, ragged), K on both sides of 1280, temporal layers, a single workgroup row in the deepest level
@pytest.mark.parametrize("channels,depth,height,width,batch,frames", [([640, 1280], [1, 1], 46, 48, 1, 0), ([320, 1280], [2, 1], 46, 46, 2, 0), ([640, 1280], [1, 1], 26, 24, 3, 3)])
def test_results_do_not_depend_on_who_asks(channels, depth, height, width, batch, frames):
    d = dict(latent_channels=4, height=height, width=width, batch=batch, channels=channels, layers_per_block=1, transformer_depth=depth, mid_depth=1,
             head_dim=64, gn_groups=32, ctx_len=77, ctx_dim=256, pooled_dim=0, frames=frames, temporal_heads=8 if frames else 0)
    g = torch.Generator().manual_seed(5)
    pool = torch.randn(1 << 22, generator=g).numpy() * np.float32(0.02)

    def weights(manifest):
        out = {}
        for i, (name, shape) in enumerate(manifest):
            size = int(np.prod(shape))
            v = np.resize(pool[(i * 7919) % 100000:], size).reshape(shape)
            out[name] = v + np.float32(1) if len(shape) == 1 and name.endswith(".g") else v
        return out

    noise = torch.randn((frames, 4, height, width) if frames else (4, height, width), generator=g).to("cuda:0")
    text = torch.randn(1 if frames else batch, 77, 256, generator=g).to("cuda:0", torch.bfloat16)
    probe = B.AsyncDiff(d, 1, 0, 1, B.AD_BF16)
    units = len(probe.units())
    probe.close()
    whole, size = run(d, [], weights, noise, text, 2)
    assert size > 128 << 20                                  # a model whose launches ask
    assert torch.isfinite(whole).all()
    for cuts in (list(range(1, units)), [2, units // 2, units - 2]):       # a component a unit: nobody asks beyond it
        got, _ = run(d, cuts, weights, noise, text, 2)
        assert torch.equal(got, whole), cuts


def layers(units, manifest, batch):
    """The GEMMs of a range of units in order: weight, rows, columns, k of its taps (the text's keys and values come from the cache)."""
    shape, out = dict(manifest), []
    for u in units:
        name, rows, c = u.name.decode(), batch * u.h_out * u.w_out, u.c_out
        conv = lambda w: (w, rows, shape[w][0], shape[w][1] * shape[w][2] * shape[w][3])
        linear = lambda w, times=1: (w, rows, times * shape[w][0], shape[w][1])
        if ".res" in name:
            out += [conv(name + ".conv1.w"), conv(name + ".conv2.w")]
        elif ".tfm" in name:
            out.append(linear(name + ".proj_in.w"))
            for k in range(u.depth):
                s = "%s.%d." % (name, k)
                out += [linear(s + "attn1.q.w", 3)] + [linear(s + w) for w in ("attn1.o.w", "attn2.q.w", "attn2.o.w", "ff1.w", "ff2.w")]
            out.append(linear(name + ".proj_out.w"))
            if name + ".temp.q.w" in shape:
                out += [linear(name + ".temp.q.w", 3), linear(name + ".temp.o.w")]
        elif name == "conv_in":
            out.append((name + ".conv.w", rows, shape[name + ".conv.w"][0], 64))
        else:
            out.append(conv(name + ".conv.w"))
    return out


# both levels ask (2208 and 552 rows); the lower one has too few rows (432 and, of three frames, 312), so that nothing asks for its weights
@pytest.mark.parametrize("channels,depth,height,width,batch,frames,lower", [([640, 1280], [1, 1], 46, 48, 1, 0, True), ([640, 1280], [1, 2], 36, 48, 1, 0, False), ([640, 1280], [1, 1], 26, 24, 3, 3, False)])
def test_a_launch_asks_for_the_weights_of_the_one_behind_it(channels, depth, height, width, batch, frames, lower):
    """The last launch of a component asks for none: what follows runs on another stream."""
    d = dict(latent_channels=4, height=height, width=width, batch=batch, channels=channels, layers_per_block=1, transformer_depth=depth, mid_depth=1,
             head_dim=64, gn_groups=32, ctx_len=77, ctx_dim=256, pooled_dim=0, frames=frames, temporal_heads=8 if frames else 0)
    m = B.AsyncDiff(d, 4, 1, 1, B.AD_BF16, cuts=[2, 9, 16])
    m.allocate("cuda:0")
    manifest = m.weight_manifest()
    pool = torch.randn(1 << 20, generator=torch.Generator().manual_seed(5)).numpy() * np.float32(0.02)
    m.load_weights({n: np.resize(pool, int(np.prod(s))).reshape(s) for n, s in manifest})
    m.reset(4)
    text = torch.randn(1 if frames else batch, 77, 256, device="cuda:0").to(torch.bfloat16)
    stream = torch.cuda.current_stream()
    m.precompute_text(text, stream)
    asked = set()
    for comp, (first, last) in enumerate(m.partition(), 1):
        ins, outs = m.component_io(comp)
        new = lambda u, make: make(m.tensor_shape(u)[0], device="cuda:0", dtype=torch.float32 if u < 0 or u == len(m.units()) - 1 else torch.bfloat16)
        latent = torch.zeros((frames, 4, height, width) if frames else (4, height, width), device="cuda:0")
        m.profile(True)
        m.component_forward(comp, [latent if u < 0 else new(u, torch.ones) for u in ins], 0, text, [new(u, torch.empty) for u in outs], stream)
        torch.cuda.synchronize()
        records = m.profile_records(clear=False)
        at = [i for i, r in enumerate(records) if r[0].startswith("igemm")]
        got = [(records[i][0], records[i][4], B.lib.ad_profile_ahead(m._h, i)) for i in at]
        assert all(B.lib.ad_profile_ahead(m._h, i) == -1 for i in range(len(records)) if i not in at)
        m.profile_records()
        m.profile(False)
        want = layers(m.units()[first:last + 1], manifest, batch)
        assert len(got) == len(want), (got, want)
        for (kernel, (rows, n, k), ahead), this, behind in zip(got, want, want[1:] + [None]):
            assert (rows, n) == this[1:3] and k >= this[3], (kernel, rows, n, k, this)          # k includes a shortcut's
            wanted = -1
            if behind and any(kind in kernel for kind in ("_p3", "_d2", "_k2")) and not this[0].startswith("conv_in"):
                size = (behind[2] + 127) // 128 * 128 * behind[3] * 2
                if behind[1] >= 512 and behind[3] >= 1280 and size <= 16000000:
                    wanted = [w for w, _ in manifest].index(behind[0])
            assert ahead == wanted, (kernel, this, behind, ahead, wanted)
            if ahead >= 0:
                asked.add(manifest[ahead][0])
    m.close()
    assert any(w.endswith("conv2.w") for w in asked) and any(w.endswith("ff2.w") for w in asked)
    assert any(w.startswith("d1.0.tfm") for w in asked) == lower, asked
