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


# More images than two to a compute unit (256 of them): half a wave to a lane of at most 32 symbols, and containers packed by two
# workgroups or one (past 1024) instead of four. Else a whole wave and four, with the same results
@pytest.mark.parametrize("H,W,levels,batch,chunk,half", [
    (2, 84, 1, 512, True, False), (2, 84, 1, 513, False, True), (2, 86, 1, 513, True, False), (2, 2, 1, 513, False, True),   # 31.5, 32.25 symbols
    (2, 170, 1, 700, True, False), (16, 16, 2, 1025, False, True), (16, 20, 2, 600, False, True), (32, 16, 3, 520, True, True)])
def test_many_images_decode_as_few_do(H, W, levels, batch, chunk, half):
    import torch
    cfg = FlowConfig("many", H, W, batch, levels, 1, PLAIN, 32, 0, True, image_kind="uniform", seed_id=52)
    print("many images", cfg, flush=True)
    flow = iodf.Flow(make_blob(cfg), max_batch=batch, device=0)
    x = torch.randint(0, 256, (batch, 3, H, W), generator=torch.Generator().manual_seed(9), dtype=torch.uint8).cuda()
    words, sizes = flow.encode(x)
    few = [flow.encode(x[i:i + 256].contiguous()) for i in range(0, batch, 256)]
    assert torch.equal(words, torch.cat([w for w, _ in few])) and torch.equal(sizes, torch.cat([s for _, s in few]))
    flow.profile_begin(4096)
    assert torch.equal(flow.decode(words), x)
    ran = {k["name"] for k in flow.profile_end() if "decode" in k["name"]}
    assert ran == ({"k_rans_decode_chunk"} if chunk else set()) | ({"k_rans_decode_half"} if half else set())
    assert flow.codec_errors() == (0, 0, 0) and flow.range_errors() == 0
    # damaged containers: whatever comes out, it and the lanes counted as broken are the same
    slots = 16 * levels
    for what in range(5):
        bad = words.clone()
        if what == 0:
            bad[:, 1 + 3 * slots::3] ^= 0x5a5a5a           # payload
        elif what == 1:
            bad[::2, 2] += 5                               # a lane claims more words
        elif what == 2:
            bad[1::2, 0] = 1 << 30                         # absurd total
        elif what == 3:
            bad[:, 1 + slots:1 + 3 * slots] = -1           # states of all ones
        else:
            bad = bad[:, :1 + 3 * slots + 7].contiguous()  # cut short
        y = flow.decode(bad)
        counted = flow.codec_errors()[2]
        y_few, c_few = [], 0
        for i in range(0, batch, 256):
            y_few.append(flow.decode(bad[i:i + 256].contiguous()))
            c_few += flow.codec_errors()[2]
        assert torch.equal(y, torch.cat(y_few)) and counted == c_few, what
        assert counted > 0 or (H, W) == (2, 2)         # (too few latents for a word to be shed)
    flow.range_errors()
    assert torch.equal(flow.decode(words), x)
    flow.close()
