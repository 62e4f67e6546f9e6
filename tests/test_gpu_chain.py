"""Networks that run as one launch out of LDS, against the oracle, bit-exact: every kind of kernel (stream and
block-internal widths of one or two 64-channel planes, 1x1 and 3x3 second convolutions, no blocks at all) at the edges
of its pixel tiles, with groups of several images, and where the requantise has exact ties."""
import numpy as np
import pytest

import paper_2206_08869_amd as iodf
from synth import make_blob, make_images
from synth.configs import PLAIN, RESNET, FlowConfig
from util import to_gpu

pytestmark = pytest.mark.gpu


def _kernels(flow, x):
    """Names of the kernels one forward call runs, and its latents."""
    import torch
    flow.profile_begin(4096)
    z = flow.forward(x)[0]
    torch.cuda.synchronize()
    return {k["name"].split("<")[0] for k in flow.profile_end()}, z


def _check(cfg, batch, blob=None, kernel="k_chain", alone=True):
    """Forward and inverse against the oracle; `kernel` runs the networks (with `alone`: all of them)."""
    import oracle
    import torch
    blob = make_blob(cfg) if blob is None else blob
    x = make_images(cfg, batch=batch)
    print("chain", cfg, "batch", batch, flush=True)
    z_ref, c_ref = oracle.Model(blob).forward(x)
    flow = iodf.Flow(blob, max_batch=batch, device=0)
    for _rep in range(2):
        z, codes = flow.forward(to_gpu(x))
        torch.cuda.synchronize()
        assert np.array_equal(z.cpu().numpy(), z_ref)
        if cfg.heads:
            assert np.array_equal(codes.cpu().numpy(), c_ref)
        x2 = flow.inverse(z)
        torch.cuda.synchronize()
        assert np.array_equal(x2.cpu().numpy(), x)
    names, _ = _kernels(flow, to_gpu(x))
    ran = {n for n in names if n.startswith(("k_chain", "k_strip_block", "conv_igemm"))}
    assert kernel in ran and (not alone or ran == {kernel}), names
    flow.close()


# level-1 maps H/2 x W/2: 1, 2, 3..4 and 5..8 tiles of 32 pixels, full and ragged; images of more than 128 pixels run
# as one launch from an image for every fourth compute unit on (65), as strips below
@pytest.mark.parametrize("H,W,batch", [(8, 8, 1), (8, 16, 1), (12, 12, 2), (16, 16, 1), (16, 20, 3), (16, 32, 2),
                                       (2, 128, 2), (20, 26, 65), (24, 40, 67), (32, 32, 66)])
@pytest.mark.parametrize("width,keep,k2", [(128, 1.0, 3), (128, 0.4, 3), (128, 1.0, 1), (128, 0.4, 1), (64, 1.0, 3), (40, 0.8, 1)])
def test_tiles_and_widths(H, W, batch, width, keep, k2):
    _check(FlowConfig("chain", H, W, batch, 1, 1, RESNET, width, 2, False, keep=keep, seed_id=41, block_k2=k2), batch)


@pytest.mark.parametrize("width,unsigned", [(128, False), (128, True), (48, True)])
def test_plain_and_unsigned(width, unsigned):
    _check(FlowConfig("plain", 16, 16, 3, 2, 2, PLAIN, width, 0, True, seed_id=42, act_unsigned=unsigned), 3)
    _check(FlowConfig("plain", 32, 32, 34, 1, 2, PLAIN, width, 0, False, seed_id=42, act_unsigned=unsigned), 34)
    _check(FlowConfig("res_u", 16, 16, 3, 3, 1, RESNET, width, 1, True, seed_id=43, act_unsigned=unsigned, block_k2=3), 3)


# 4x4 and 2x2 maps: more images than compute units share workgroups, the last group is short
@pytest.mark.parametrize("batch", [257, 515])
def test_groups_of_images(batch):
    _check(FlowConfig("groups", 8, 8, batch, 2, 1, RESNET, 32, 1, True, seed_id=44), batch)


def test_ties_and_last_layers():
    """Multipliers that are powers of two reach exact halves (away from zero, not up); a 1x1 last layer; a last layer
    with a ReLU."""
    from synth.model import pack_blob, parse_blob
    cfg = FlowConfig("ties", 16, 16, 2, 2, 2, RESNET, 32, 2, True, seed_id=45)
    m = parse_blob(make_blob(cfg).copy())
    for n, net in enumerate(m["nets"]):
        for l, L in enumerate(net["layers"]):
            if n % 2 == 0:   # small weights and a coarse scale: many accumulators are odd multiples of half a code
                L["M"][:] = 1 << 30
                L["shift"][:] = 33
                L["W"] //= 32
                L["bias"] //= 256
            elif l + 1 == len(net["layers"]):   # ties in the last layer only: the hidden ones keep the short form
                L["M"][:] = 1 << 30
                L["shift"][:] = 37
        if n % 3 == 1:
            net["layers"][-1]["W"] = np.ascontiguousarray(net["layers"][-1]["W"][:, :, 1:2, 1:2])
        if n % 3 == 2:
            net["layers"][-1]["flags"] |= 1
    _check(cfg, 2, pack_blob(m), alone=False)   # ties in a shortcut layer: layer by layer


# strips: 24x40, 16x16 and 32x32 maps at batches that give one row, a few rows and the most rows a strip XX that are no multiple of a tile
@pytest.mark.parametrize("H,W,batch", [(48, 80, 1), (32, 32, 1), (32, 32, 13), (32, 32, 64), (64, 64, 3), (64, 64, 17), (64, 64, 66),
                                       (10, 52, 2), (34, 70, 9)])
@pytest.mark.parametrize("width,keep,k2,unsigned", [(128, 1.0, 3, False), (128, 0.4, 1, True), (64, 1.0, 3, True),
                                                    (128, 0.4, 3, False), (128, 1.0, 1, False), (48, 1.0, 1, True)])
def test_strips(H, W, batch, width, keep, k2, unsigned):
    _check(FlowConfig("strips", H, W, batch, 1, 1, RESNET, width, 2, False, keep=keep, seed_id=46, block_k2=k2,
                      act_unsigned=unsigned), batch, kernel="k_strip_block")


def _issued_macs(batch, h, w, rows, nc_x, nc_t, k2, run=1):
    """Multiply-accumulates that the matrix cores run for a residual block of nc_x (outside) and nc_t (inside) 32-channel chunks
    in strips of `rows` rows: whole tiles of 32 pixels, as many as the smallest kernel that holds the strip takes. `run` strips to a
    workgroup, of which those behind the first take the second convolution's tiles for both."""
    one = min(h, rows + 2 if k2 == 3 else rows)
    t1, t2 = next(t for t in ((2, 1), (3, 1), (3, 2), (4, 2), (6, 4)) if one * w <= 32 * t[0] and rows * w <= 32 * t[1])

    def layer(n_blk, tiles, taps, nc):
        share = 4 // (n_blk // (2 if n_blk == 4 and tiles >= 4 else 1))   # waves beside each other over the pixels
        return 32 * -(-tiles // share) * share * 32 * n_blk * taps * 32 * nc
    strips = -(-h // rows)
    firsts, two = -(-strips // run), layer(nc_x, t2, k2 * k2, nc_t)
    return batch * (firsts * (layer(nc_t, t1, 9, nc_x) + two) + (strips - firsts) * (layer(nc_t, t2, 9, nc_x) + two))


def _check_rows(cfg, batch, rows, nc_x, nc_t):
    """The rows that a forward call's strips took (256 compute units), told from the matrix work of a block's launch; the same
    images give the same latents in a small batch, and come back."""
    import torch
    print("rows", cfg, "batch", batch, flush=True)
    flow = iodf.Flow(make_blob(cfg), max_batch=batch, device=0)
    x = torch.randint(0, 256, (batch, 3, cfg.H, cfg.W), generator=torch.Generator().manual_seed(8), dtype=torch.uint8).cuda()
    flow.profile_begin(4096)
    z = flow.forward(x)[0]
    torch.cuda.synchronize()
    blocks = {k["name"]: k for k in flow.profile_end()}["k_strip_block"]
    h, w = cfg.H // 2, cfg.W // 2
    assert blocks["issued_macs"] == blocks["launches"] * _issued_macs(batch, h, w, rows, nc_x, nc_t, cfg.block_k2)
    assert torch.equal(z[-3:], flow.forward(x[-3:].contiguous())[0])
    assert torch.equal(flow.inverse(z), x)
    flow.close()


# Batches at which the most rows that give a strip to every compute unit would put two on some: other rows are taken
@pytest.mark.parametrize("H,batch,rows", [(64, 9, 2), (64, 24, 4), (32, 50, 4), (48, 40, 5)])
@pytest.mark.parametrize("keep,k2", [(1.0, 3), (0.7, 3), (1.0, 1)])
def test_strip_rows(H, batch, rows, keep, k2):
    cfg = FlowConfig("rows", H, H, batch, 1, 1, RESNET, 128, 2, False, keep=keep, seed_id=50, block_k2=k2)
    _check(cfg, batch, kernel="k_strip_block")
    _check_rows(cfg, batch, rows, 4, 3 if keep < 1 else 4)


# Fewer rows, more strips: where they save enough (five strips to two of seven rows), and not where many strips to a unit, or a
# third of the rows, cost what the estimate leaves out
@pytest.mark.parametrize("H,W,batch,width,keep,k2,rows", [
    (40, 32, 200, 64, 1.0, 3, 4), (40, 32, 200, 128, 1.0, 3, 4), (40, 32, 2048, 128, 1.0, 1, 4),
    (52, 38, 2048, 64, 1.0, 1, 6), (64, 38, 384, 128, 0.4, 3, 6), (110, 24, 1024, 128, 1.0, 3, 10), (34, 32, 111, 64, 1.0, 3, 6),
    (64, 18, 256, 128, 0.4, 1, 11)])
def test_strip_rows_where_more_strips_pay(H, W, batch, width, keep, k2, rows):
    _check_rows(FlowConfig("more_strips", H, W, batch, 1, 1, RESNET, width, 2, False, keep=keep, seed_id=50, block_k2=k2),
                batch, rows, width // 32, 2 if keep < 1 or width == 64 else 4)


# Strips that a workgroup takes one below the other (256 compute units; full rounds of two workgroups to each): 2, 4 and all 8
# strips of an image; just nine tenths of a round and just less; rounds that are not quite full or too empty; strips of eight and of
# three rows, 19 of them as ten and nine; strips of two rows, where the rows that are kept lie right behind those they replace (64 wide
# only: 128 wide, two rows of the 33 to 40 columns that take this kernel do not pay, and two of 48 are more than a workgroup moves
# between two strips, 768 pieces of 16 bytes). The run is told from the matrix work of a block's launch; the same images give the same
# latents in batches that take a strip to a workgroup (16 images of 24x48 maps a launch per layer).
RUNS = [(64, 64, 115, 4, 1), (64, 64, 116, 4, 2), (64, 64, 128, 4, 2), (64, 64, 256, 4, 4), (64, 64, 512, 4, 8), (64, 64, 237, 4, 4),
        (64, 64, 201, 4, 1), (80, 64, 102, 4, 2), (128, 32, 128, 8, 2), (114, 72, 256, 3, 10)]
KINDS = [(128, 1.0, False, 4, 4), (128, 0.7, True, 4, 3), (128, 0.4, False, 4, 2), (64, 1.0, True, 2, 2)]


@pytest.mark.parametrize("H,W,batch,rows,run,width,keep,unsigned,nc_x,nc_t", [r + k for r in RUNS for k in KINDS] + [
    (48, 80, 128, 2, 3, 64, 1.0, True, 2, 2), (48, 96, 128, 2, 1, 128, 0.4, False, 4, 2)])
def test_runs_of_strips(H, W, batch, rows, run, width, keep, unsigned, nc_x, nc_t):
    import torch
    cfg = FlowConfig("runs", H, W, batch, 1, 1, RESNET, width, 2, False, keep=keep, seed_id=54, block_k2=3, act_unsigned=unsigned)
    print("runs of strips", cfg, flush=True)
    flow = iodf.Flow(make_blob(cfg), max_batch=batch, device=0)
    x = torch.randint(0, 256, (batch, 3, H, W), generator=torch.Generator().manual_seed(9), dtype=torch.uint8).cuda()

    def blocks(part):
        flow.profile_begin(64)
        z = flow.forward(part)[0]
        torch.cuda.synchronize()
        return z, {k["name"]: k for k in flow.profile_end()}.get("k_strip_block")
    z, many = blocks(x)
    assert many["issued_macs"] == many["launches"] * _issued_macs(batch, H // 2, W // 2, rows, nc_x, nc_t, 3, run), (rows, run)
    _, few = blocks(x[:16])
    assert (W == 96) == (few is None)
    if few:
        per = few["issued_macs"] // few["launches"]
        assert any(per == _issued_macs(16, H // 2, W // 2, r, nc_x, nc_t, 3) for r in range(1, rows + 1))
    for i in range(0, batch, 16):
        assert torch.equal(z[i:i + 16], flow.forward(x[i:i + 16].contiguous())[0])
    assert torch.equal(flow.inverse(z), x)
    flow.close()


# 65 to 96 of 128 channels kept inside: blocks of 48 filters to a wave over four tiles and more, three waves of 32 below
# (64, 80 and 128 pixel maps, 130 to 256 as one launch; strips at every tile count); 97 take the kernels of 128
@pytest.mark.parametrize("H,W,batch,kernel", [(16, 16, 1, "k_chain"), (16, 20, 3, "k_chain"), (16, 32, 2, "k_chain"), (20, 26, 65, "k_chain"),
                                              (24, 40, 67, "k_chain"), (32, 32, 66, "k_chain"), (48, 80, 1, "k_strip_block"),
                                              (32, 32, 1, "k_strip_block"), (32, 32, 13, "k_strip_block"), (32, 32, 64, "k_strip_block"),
                                              (64, 64, 3, "k_strip_block"), (64, 64, 17, "k_strip_block"), (64, 64, 66, "k_strip_block"),
                                              (10, 52, 2, "k_strip_block"), (34, 70, 9, "k_strip_block")])
@pytest.mark.parametrize("keep,unsigned", [(0.75, False), (0.625, True), (65 / 128, False), (97 / 128, False)])
def test_three_quarters_kept(H, W, batch, kernel, keep, unsigned):
    _check(FlowConfig("kept", H, W, batch, 1, 1, RESNET, 128, 2, False, keep=keep, seed_id=49, block_k2=3, act_unsigned=unsigned),
           batch, kernel=kernel)


# Maps whose rows fill the largest strip kernel badly go layer by layer once more strips wait than run at once, or at
# once where a single row already takes that kernel; the same images give the same latents either way.
@pytest.mark.parametrize("H,batch,width,keep,k2,strips", [
    (64, 64, 128, 1.0, 3, True), (80, 24, 128, 1.0, 3, True), (80, 96, 128, 1.0, 3, False), (96, 96, 128, 1.0, 3, False),
    (128, 1, 128, 1.0, 3, False), (128, 48, 128, 1.0, 3, False), (128, 4, 128, 0.4, 3, True), (88, 6, 128, 0.4, 3, False),
    (104, 48, 128, 0.4, 3, False),
    (88, 128, 128, 1.0, 1, False), (96, 48, 128, 1.0, 1, True), (104, 96, 64, 1.0, 3, False), (128, 48, 64, 1.0, 3, True),
    (128, 48, 128, 0.4, 1, True)])
def test_strips_only_where_they_win(H, batch, width, keep, k2, strips):
    import torch
    cfg = FlowConfig("wide_maps", H, H, batch, 1, 1, RESNET, width, 2, False, keep=keep, seed_id=47, block_k2=k2)
    print("strips or layers", cfg, flush=True)
    flow = iodf.Flow(make_blob(cfg), max_batch=batch, device=0)
    x = torch.randint(0, 256, (batch, 3, H, H), generator=torch.Generator().manual_seed(5), dtype=torch.uint8).cuda()
    names, z = _kernels(flow, x)
    assert ("k_strip_block" in names) == strips and ("conv_igemm" in " ".join(names)) != strips, names
    few = min(batch, 3)
    _, z_few = _kernels(flow, x[-few:].contiguous())
    assert torch.equal(z[-few:], z_few)
    assert torch.equal(flow.inverse(z), x)
    flow.close()


# More images than a launch of strips of the cheapest rows could count (8 x 65535 of them): rows are taken with which it can
@pytest.mark.parametrize("H,W,batch,width,keep,k2", [(110, 38, 27756, 128, 1.0, 3), (18, 96, 61008, 128, 0.4, 1), (14, 86, 82850, 64, 1.0, 1)])
def test_strips_of_as_many_images_as_a_launch_counts(H, W, batch, width, keep, k2):
    import torch
    cfg = FlowConfig("many", H, W, batch, 1, 1, RESNET, width, 1, False, keep=keep, seed_id=53, block_k2=k2)
    print("many strips", cfg, flush=True)
    flow = iodf.Flow(make_blob(cfg), max_batch=batch, device=0)
    x = torch.randint(0, 256, (batch, 3, H, W), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda", dtype=torch.uint8)
    names, z = _kernels(flow, x)
    assert "k_strip_block" in names, names
    for part in (slice(0, 3), slice(batch - 3, batch)):
        assert torch.equal(z[part], _kernels(flow, x[part].contiguous())[1])
    assert torch.equal(flow.inverse(z), x)
    flow.close()


# Whole networks as one launch, but where kernels of whole tiles do too much padding for many images, and where two
# plain layers over a few large maps keep more compute units busy.
@pytest.mark.parametrize("H,W,batch,family,width,keep,k2,chain", [
    (10, 26, 256, RESNET, 128, 1.0, 3, True), (10, 26, 900, RESNET, 128, 1.0, 3, False), (16, 16, 900, RESNET, 128, 1.0, 3, True),
    (16, 20, 2560, RESNET, 128, 1.0, 3, False), (8, 8, 2560, RESNET, 128, 1.0, 3, False), (8, 8, 2048, RESNET, 128, 1.0, 3, True),
    (20, 26, 900, RESNET, 128, 1.0, 3, False), (20, 26, 900, RESNET, 128, 0.4, 3, True), (10, 26, 2560, RESNET, 128, 0.4, 3, False),
    (10, 26, 2560, RESNET, 128, 1.0, 1, False), (10, 26, 2560, RESNET, 128, 0.4, 1, True), (10, 26, 2560, RESNET, 64, 1.0, 3, True),
    (32, 32, 1, PLAIN, 128, 1.0, 1, False), (32, 32, 64, PLAIN, 128, 1.0, 1, True), (10, 26, 2560, PLAIN, 128, 1.0, 1, False)])
def test_one_launch_only_where_it_wins(H, W, batch, family, width, keep, k2, chain):
    import torch
    cfg = FlowConfig("ragged_maps", H, W, batch, 1, 1, family, width, 0 if family == PLAIN else 1, False, keep=keep, seed_id=48, block_k2=k2)
    print("one launch or layers", cfg, flush=True)
    flow = iodf.Flow(make_blob(cfg), max_batch=batch, device=0)
    x = torch.randint(0, 256, (batch, 3, H, W), generator=torch.Generator().manual_seed(6), dtype=torch.uint8).cuda()
    names, z = _kernels(flow, x)
    assert ("k_chain" in names) == chain and ("conv_igemm" in " ".join(names)) != chain, names
    few = min(batch, 70)
    _, z_few = _kernels(flow, x[-few:].contiguous())
    assert torch.equal(z[-few:], z_few)
    assert torch.equal(flow.inverse(z), x)
    flow.close()


@pytest.mark.parametrize("name,batch", [("cfg2", 64), ("cfg2", 3), ("paper_res32", 2), ("mini_dense", 5), ("deep6", 2), ("wide_resnet", 2)])
def test_convolution_launches_of_a_call(name, batch):
    """IODF_Q_CONV_LAUNCHES tells the launches that a call of max_batch images makes, whatever route its networks take."""
    import torch
    from util import gpu_flow, images
    flow = gpu_flow(name, batch)
    flow.profile_begin(4096)
    flow.forward(to_gpu(images(name, batch)))
    torch.cuda.synchronize()
    ran = sum(k["launches"] for k in flow.profile_end() if k["name"].startswith(("conv_igemm", "k_chain", "k_strip")))
    assert flow.query(iodf.IODF_Q_CONV_LAUNCHES) == ran
    flow.close()


def test_profile_of_strips_and_whole_networks():
    """Their launches report the matrix work that ran (no less than what the layers need, padding included), and blocks
    of two wide layers are in the wide-layer view."""
    import torch
    from util import gpu_flow, images
    flow = gpu_flow("cfg2", 4)   # level 1: strips of 16x16 maps, level 2: 8x8 maps as one launch
    flow.profile_begin(4096)
    flow.forward(to_gpu(images("cfg2", 4)))
    torch.cuda.synchronize()
    stats = {k["name"]: k for k in flow.profile_end()}
    for name in ("k_strip_in", "k_strip_block", "k_strip_last", "k_chain"):
        assert stats[name]["issued_macs"] >= stats[name]["macs"] > 0, stats[name]
    blocks = stats["k_strip_block"]
    for view in ("view: wide conv layers", "view: wide conv layers, levels 1-2"):
        assert (stats[view]["launches"], stats[view]["macs"]) == (blocks["launches"], blocks["macs"])
    # a workgroup takes one 8x8 map, two tiles of 32 pixels; its last layer, 12 filters of 32, runs over four
    per_image = 64 * 128 * (9 * 32 + 2 * (9 + 1) * 128) + 128 * 32 * 9 * 128
    assert stats["k_chain"]["issued_macs"] == 4 * stats["k_chain"]["launches"] * per_image
    flow.close()


# Calls of up to 32 kernels are launched directly, longer ones replayed: whole networks as one launch each, strips (ten launches a
# network), a launch per layer with the taps of the last one summed (four a network), and with the last one split along its 32
# k-tiles and finished by a kernel of its own (four a network too). Two more kernels take the pixels in and the latents out.
@pytest.mark.parametrize("family,width,depth,side,couplings,kernels,split", [
    (PLAIN, 32, 0, 8, 30, 32, False), (PLAIN, 32, 0, 8, 31, 33, False), (RESNET, 128, 8, 32, 3, 32, False), (RESNET, 128, 8, 32, 4, 42, False),
    (PLAIN, 256, 0, 8, 7, 30, False), (PLAIN, 256, 0, 8, 8, 34, False), (PLAIN, 2048, 0, 8, 7, 30, True), (PLAIN, 2048, 0, 8, 8, 34, True)])
def test_short_calls_are_launched_directly(family, width, depth, side, couplings, kernels, split):
    import torch
    from synth.model import pack_blob, parse_blob
    cfg = FlowConfig("short", side, side, 1, 1, couplings, family, width, depth, False, seed_id=54)
    print("short calls", cfg, flush=True)
    blob = make_blob(cfg)
    if split:
        m = parse_blob(blob.copy())
        for net in m["nets"]:
            net["layers"][-1]["W"] = np.ascontiguousarray(net["layers"][-1]["W"][:, :, 1:2, 1:2])
        blob = pack_blob(m)
    flow = iodf.Flow(blob, max_batch=2, device=0)
    x = to_gpu(make_images(cfg, batch=2))
    flow.profile_begin(4096)
    z = flow.forward(x[:1])[0]
    torch.cuda.synchronize()
    bracketed = sum(k["launches"] for k in flow.profile_end() if not k["name"].startswith("view:"))
    assert bracketed == kernels - couplings * split   # (a split layer and what finishes it are bracketed together)
    assert flow.query(iodf.IODF_Q_GRAPHS) == 0
    long = int(kernels > 32)
    for rep in range(2):
        assert torch.equal(flow.forward(x[:1])[0], z) and flow.query(iodf.IODF_Q_GRAPHS) == long * (1 if rep == 0 else 2)
        assert torch.equal(flow.inverse(z), x[:1]) and flow.query(iodf.IODF_Q_GRAPHS) == long * 2
    assert torch.equal(flow.forward(x)[0][:1], z) and flow.query(iodf.IODF_Q_GRAPHS) == long * 3
    flow.close()
