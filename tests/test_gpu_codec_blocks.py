"""The coder's kernels where their blocks of 32 symbols a lane end: containers against the oracle's word for word, and
decoded again. The deepest level codes all of an image, 3 * H * W latents over 16 lanes: below, at and above 32 and 64
symbols a lane, lanes of unequal length, and fewer latents than lanes. With heads the scales vary by latent."""
import numpy as np
import pytest

import paper_2206_08869_amd as iodf
from synth import make_blob, make_images
from synth.configs import PLAIN, FlowConfig
from util import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,levels,batch", [(2, 2, 1, 3), (10, 16, 1, 1), (12, 14, 1, 2), (2, 86, 1, 5), (2, 170, 1, 1),
                                              (2, 172, 1, 2), (24, 20, 2, 3), (32, 32, 3, 17)])
def test_containers_at_block_edges(H, W, levels, batch):
    import oracle
    import torch
    cfg = FlowConfig("blocks", H, W, batch, levels, 1, PLAIN, 32, 0, True, image_kind="uniform", seed_id=51)
    blob = make_blob(cfg)
    x = make_images(cfg, batch=batch)
    print("codec blocks", cfg, flush=True)
    w_ref, s_ref, _ = oracle.Model(blob).encode(x)
    flow = iodf.Flow(blob, max_batch=batch, device=0)
    words, sizes = flow.encode(to_gpu(x))
    torch.cuda.synchronize()
    assert np.array_equal(sizes.cpu().numpy().view(np.uint32), np.asarray(s_ref, np.uint32))
    assert np.array_equal(words.cpu().numpy().view(np.uint32), w_ref)
    x2 = flow.decode(words)
    torch.cuda.synchronize()
    assert np.array_equal(x2.cpu().numpy(), x) and flow.codec_errors() == (0, 0, 0)
    flow.close()
