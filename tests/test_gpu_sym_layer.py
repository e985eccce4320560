"""The MoE layer in the paper's own format (moe_sym_forward: Q4_SYM weights,
Q8_F32 activations and h) against the oracle's layer in that format (GPU):
the full layer shape at one token with top-8 and top-4 of 256 and with 128
routed experts, a few tokens without a shared expert and with skipped slots,
and an exact-integer layer that must match bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2606_24031_amd as w4
from paper_2606_24031_amd import synth
from tests import moe_check
from tests.exact_layers import ExactLayer

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def pairs_workspace(T, H, I, k):
    """Bytes of the documented regions and y: what running pair by pair needs."""
    up = lambda n: (n + 255) // 256 * 256
    P = T * (k + 1)
    return up(T * H // 32 * 36) + up(4 * P * I) + up(P * I // 32 * 36) + up(4 * P * H)


def run_sym(x, ids, wts, w, H, I, E, k, grouped=None):
    """The layer on a workspace filled with a pattern; grouped: whether it is to
    run on the grouped kernels (which write past the documented regions and
    y), None: either."""
    T = x.shape[0]
    ws = w4.moe_sym_workspace(T, H, I, E, k)
    ws.fill_(0xEE)
    sgu = None if w["ws_gu"] is None else dev(w["ws_gu"])
    sd = None if w["ws_d"] is None else dev(w["ws_d"])
    out = w4.moe_sym_forward(dev(x), dev(ids), dev(wts), dev(w["w_gu"]), dev(w["w_d"]), sgu, sd,
                             H, I, E, k, ws)
    torch.cuda.synchronize()
    lay = w4.moe_sym_workspace_layout(T, H, I, E, k)
    P = T * k + T
    wsn = ws.cpu().numpy()
    if grouped is not None:
        assert bool((wsn[pairs_workspace(T, H, I, k):] != 0xEE).any()) == grouped, "path taken"
    h = wsn[lay["h"]:lay["h"] + P * I * 4].view(np.float32).reshape(P, I)
    hq = wsn[lay["hq"]:lay["hq"] + P * (I // 32) * 36].reshape(P, -1)
    xq = wsn[lay["xq"]:lay["xq"] + T * (H // 32) * 36].reshape(T, -1)
    assert np.array_equal(xq, oracle.q8_f32_quantize(x)), "Q8_F32(x)"
    return out.cpu().numpy(), h, hq


@pytest.fixture(scope="module")
def full_layer():
    H, I, E = 2048, 512, 256
    g = synth.rng(61)
    return dict(w_gu=synth.q4_sym_random_blocks(g, E * 2 * I, H),
                w_d=synth.q4_sym_random_blocks(g, E * H, I),
                ws_gu=synth.q4_sym_random_blocks(g, 2 * I, H),
                ws_d=synth.q4_sym_random_blocks(g, H, I))


@pytest.mark.parametrize("E,k", [(256, 8), (256, 4), (128, 8)])
def test_sym_layer_full_shape_one_token(full_layer, E, k):
    H, I = 2048, 512
    w = dict(full_layer)
    if E < 256:
        w["w_gu"] = w["w_gu"].reshape(256, -1)[:E].reshape(-1)
        w["w_d"] = w["w_d"].reshape(256, -1)[:E].reshape(-1)
    g = synth.rng(62 + E + k)
    x = synth.normal_f32(g, (1, H))
    ids, wts = synth.routing(g, 1, E, k)
    out, h, hq = run_sym(x, ids, wts, w, H, I, E, k)
    st = moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], w["ws_gu"],
                                   w["ws_d"], H, I, E, k)
    assert st["pairs"] == k + 1


def test_sym_layer_tokens_no_shared_skipped_slots():
    """Five tokens, no shared expert, a skipped slot and a repeated expert;
    I = 768 (three groups of eight blocks in the down rows)."""
    H, I, E, k, T = 1024, 768, 12, 4, 5
    g = synth.rng(63)
    w = dict(w_gu=synth.q4_sym_random_blocks(g, E * 2 * I, H),
             w_d=synth.q4_sym_random_blocks(g, E * H, I), ws_gu=None, ws_d=None)
    x = synth.normal_f32(g, (T, H))
    ids, wts = synth.routing(g, T, E, k)
    ids[1, 2] = -1
    ids[3, 1] = ids[3, 0]
    out, h, hq = run_sym(x, ids, wts, w, H, I, E, k)
    moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], None, None,
                              H, I, E, k)


@pytest.mark.parametrize("T,I,k,shared", [(2, 256, 1, False), (3, 512, 1, False), (2, 512, 1, True),
                                          (2, 1024, 1, False), (2, 512, 4, False),
                                          (2, 512, 4, True), (1, 256, 64, True)])
def test_sym_layer_slot_counts(T, I, k, shared):
    """Down and combine from one slot (no shared expert) to 65: a token's h
    blocks of less than one, of one and two whole rounds of single loads per
    thread, and of more; a repeated expert where k allows."""
    H, E = 768, 9
    g = synth.rng(68 + I + k)
    w = dict(w_gu=synth.q4_sym_random_blocks(g, E * 2 * I, H),
             w_d=synth.q4_sym_random_blocks(g, E * H, I),
             ws_gu=synth.q4_sym_random_blocks(g, 2 * I, H) if shared else None,
             ws_d=synth.q4_sym_random_blocks(g, H, I) if shared else None)
    x = synth.normal_f32(g, (T, H))
    ids = g.integers(-1, E, size=(T, k)).astype(np.int32)
    wts = np.abs(synth.normal_f32(g, (T, k)))
    out, h, hq = run_sym(x, ids, wts, w, H, I, E, k)
    moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], w["ws_gu"], w["ws_d"],
                              H, I, E, k)


def test_sym_layer_exact_integer_layer():
    """Every scale 1.0, integer activations and h with block maxima 127: the
    GPU's h, Q8_F32(h) and output equal the oracle's bit for bit (a block dot
    off by one anywhere changes them)."""
    H, I, E, k = 2048, 512, 8, 4
    check_exact(ExactLayer(64, H, I, E, k, [(3, [1, 5, -1, 7])], shared=True, lo=1), H, I, False)


def check_exact(L, H, I, grouped):
    w_gu, w_d, ws_gu, ws_d = L.sym()
    w = dict(w_gu=w_gu, w_d=w_d, ws_gu=ws_gu, ws_d=ws_d)
    out, h, hq = run_sym(L.x, L.ids, L.wts, w, H, I, L.E, L.k, grouped=grouped)
    r = oracle.moe_sym(L.x, L.ids, L.wts, w_gu, w_d, ws_gu, ws_d, H, I, L.E, L.k)
    pairs = moe_check.valid_pairs(L.ids, L.E, ws_gu is not None)
    assert np.array_equal(h[pairs].view(np.uint32), r.h[pairs].view(np.uint32)), "h"
    assert np.array_equal(hq[pairs], r.hq[pairs]), "Q8_F32(h)"
    assert np.array_equal(out.astype(np.float64), r.out), "layer output"


@pytest.mark.parametrize("E,k,clusters,shared", [
    # VALU chunks: three clusters of one chunk; chunks of 8, 8 and 4 rows
    (24, 8, [(8, range(0, 8)), (8, range(8, 16)), (8, range(16, 24))], False),
    (8, 8, [(20, range(8))], True),
    # tiles, cut at 64 rows: groups of 40, 70 (a full tile and one of 6 rows), 5,
    # 16 and 17; cut at 32 rows: 150 rows and the shared group
    (128, 8, [(40, range(0, 8)), (70, range(8, 16)), (5, range(16, 24)), (16, range(24, 32)),
              (17, range(32, 40))], False),
    (8, 8, [(150, range(8))], True)])
def test_sym_layer_exact_integer_layer_grouped(E, k, clusters, shared):
    H, I = 2048, 512
    L = ExactLayer(69 + E, H, I, E, k, [(n, list(e)) for n, e in clusters], shared=shared, lo=1)
    check_exact(L, H, I, True)


# The grouped kernels of this format: VALU chunks of up to 8 rows (13, 44 and
# 128 tokens), the matrix-core tiles above (129: one slice of the route ranked
# and finished in one launch; 160 and 400: with groups of a few rows and of
# more than 64, the routing being skewed), a skipped slot and a repeated
# expert; I = 256 (two stages of the tiles) to 768; H = 2304, past the VALU
# kernels' rows, on the tiles at 20 tokens; 40 slots per token; the largest expert
# count.
@pytest.mark.parametrize("T,H,I,E,k,shared", [(13, 2048, 512, 12, 8, True),
                                              (44, 1024, 512, 12, 4, True),
                                              (128, 1024, 512, 5, 2, False),
                                              (129, 768, 256, 9, 3, True),
                                              (160, 512, 768, 17, 4, True),
                                              (400, 256, 256, 40, 3, False),
                                              (20, 2304, 512, 6, 3, True),
                                              (12, 512, 512, 48, 40, True),
                                              (450, 256, 256, 1024, 2, True)])
def test_sym_layer_grouped(T, H, I, E, k, shared):
    print(f"sym grouped T={T} H={H} I={I} E={E} k={k}", flush=True)
    g = synth.rng(T + H + I + E)
    w = dict(w_gu=synth.q4_sym_random_blocks(g, E * 2 * I, H),
             w_d=synth.q4_sym_random_blocks(g, E * H, I),
             ws_gu=synth.q4_sym_random_blocks(g, 2 * I, H) if shared else None,
             ws_d=synth.q4_sym_random_blocks(g, H, I) if shared else None)
    x = synth.normal_f32(g, (T, H))
    x[1, :32] = 0.0                                     # a zero block
    ids, wts = synth.routing(g, T, E, k, bias_std=1.0)
    ids[2, 1] = -1
    ids[3, 1] = ids[3, 0]
    gpu_ids = ids.copy()
    gpu_ids[4, 0] = E                                   # out of range: skipped too
    ids[4, 0] = -1
    out, h, hq = run_sym(x, gpu_ids, wts, w, H, I, E, k, grouped=True)
    moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], w["ws_gu"], w["ws_d"],
                              H, I, E, k)


# Either side of the dispatch: the VALU chunks by the work of the pairs there
# are (200 of 512 x 1024, with and without a shared expert), the tiles (H past
# the chunks' rows, or more than 128 tokens) by how often tokens share an expert.
@pytest.mark.parametrize("T,H,I,E,k,shared,grouped", [(39, 1024, 512, 12, 4, True, False),
                                                      (40, 1024, 512, 12, 4, True, True),
                                                      (49, 1024, 512, 12, 4, False, False),
                                                      (50, 1024, 512, 12, 4, False, True),
                                                      (6, 2304, 768, 64, 8, True, False),
                                                      (12, 2304, 768, 64, 8, True, True),
                                                      (130, 1024, 768, 128, 1, False, False),
                                                      (200, 1024, 768, 128, 1, False, True)])
def test_sym_layer_dispatch(T, H, I, E, k, shared, grouped):
    print(f"sym dispatch T={T} H={H} I={I} E={E} k={k}", flush=True)
    g = synth.rng(T + H + I + E + 1)
    w = dict(w_gu=synth.q4_sym_random_blocks(g, E * 2 * I, H),
             w_d=synth.q4_sym_random_blocks(g, E * H, I),
             ws_gu=synth.q4_sym_random_blocks(g, 2 * I, H) if shared else None,
             ws_d=synth.q4_sym_random_blocks(g, H, I) if shared else None)
    x = synth.normal_f32(g, (T, H))
    ids, wts = synth.routing(g, T, E, k)
    out, h, hq = run_sym(x, ids, wts, w, H, I, E, k, grouped=grouped)
    moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], w["ws_gu"], w["ws_d"],
                              H, I, E, k)


def test_sym_layer_grouped_one_expert_in_every_slot():
    """A group of T * k = 480 rows at 60 tokens, on the VALU chunks."""
    T, H, I, E, k = 60, 512, 512, 3, 8
    g = synth.rng(66)
    w = dict(w_gu=synth.q4_sym_random_blocks(g, E * 2 * I, H),
             w_d=synth.q4_sym_random_blocks(g, E * H, I),
             ws_gu=synth.q4_sym_random_blocks(g, 2 * I, H),
             ws_d=synth.q4_sym_random_blocks(g, H, I))
    x = synth.normal_f32(g, (T, H))
    _, wts = synth.routing(g, T, 8, k)
    ids = np.full((T, k), 1, np.int32)
    out, h, hq = run_sym(x, ids, wts, w, H, I, E, k, grouped=True)
    moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], w["ws_gu"], w["ws_d"],
                              H, I, E, k)


@pytest.mark.parametrize("T", [2, 40, 136])
def test_sym_layer_scales_near_the_ends_of_fp32(T):
    """Activations near 6e36 (block scales near 1.4e35) against gate/up scales
    near 2e-38: the product of the two scales is ordinary, a block dot times the
    activation scale alone is beyond fp32.  Pair by pair, VALU chunks, tiles."""
    H, I, E, k = 512, 512, 12, 8
    g = synth.rng(67 + T)
    w_gu = synth.q4_sym_random_blocks(g, E * 2 * I, H).reshape(-1, 20).copy()
    w_gu[:, :4] = (w_gu[:, :4].copy().view(np.float32) * np.float32(3e-36)).view(np.uint8)
    w = dict(w_gu=w_gu.reshape(E * 2 * I, -1), w_d=synth.q4_sym_random_blocks(g, E * H, I),
             ws_gu=None, ws_d=None)
    x = synth.normal_f32(g, (T, H)) * np.float32(6e36)
    ids, wts = synth.routing(g, T, E, k)
    out, h, hq = run_sym(x, ids, wts, w, H, I, E, k, grouped=T > 2)
    assert np.isfinite(out).all()
    moe_check.check_sym_layer(out, h, hq, x, ids, wts, w["w_gu"], w["w_d"], None, None, H, I, E, k)


def test_sym_layer_grouped_workspace_and_in_place():
    """The documented regions and y alone (what a call of few tokens needs, per
    token) stay enough for any T: the layer then runs pair by pair, to the
    same result within the format's tolerance; out may be hidden itself."""
    T, H, I, E, k = 110, 1024, 512, 8, 2
    g = synth.rng(65)
    w_gu, w_d = (dev(synth.q4_sym_random_blocks(g, E * 2 * I, H)),
                 dev(synth.q4_sym_random_blocks(g, E * H, I)))
    x = synth.normal_f32(g, (T, H))
    ids, wts = synth.routing(g, T, E, k)
    small = pairs_workspace(T, H, I, k)
    full = w4.moe_sym_workspace(T, H, I, E, k)
    assert full.numel() > small
    outs = []
    for ws in (full, full[:small].clone()):
        y = dev(x)
        w4.moe_sym_forward(y, dev(ids), dev(wts), w_gu, w_d, None, None, H, I, E, k, ws, out=y)
        outs.append(y.cpu().numpy())
    # the two sum in another order: a few codes of h may flip by one step
    assert np.abs(outs[0] - outs[1]).max() <= 1e-2 * np.abs(outs[0]).max()
    with pytest.raises(w4.W4A8Error):
        w4.moe_sym_forward(dev(x), dev(ids), dev(wts), w_gu, w_d, None, None, H, I, E, k,
                           full[:small - 1].clone())
