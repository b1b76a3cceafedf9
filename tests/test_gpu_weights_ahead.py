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
