"""The gated-delta-net recurrence (gdn_chunked_scan) against the oracle's
token-by-token recurrence in fp64 (GPU).

Tolerance: output element c of token t may differ by 2e-6 * |q_t| * smax_c
and the final state by 2e-6 * smax_c, smax_c the largest 2-norm over time of
column c of the head's state in the oracle: about 30 fp32 roundings (2^-24
each) of quantities of that size per chunk step, and the delta-rule update
is a contraction for beta in [0, 1] and unit keys, so errors do not grow
along the sequence (measured: below 4e-9 relative at 947 tokens).  A key-value memory
case (decay 1, step 1, orthonormal keys) is exact in fp32 and must match bit
for bit."""
import numpy as np
import pytest

import paper_2606_24031_amd as w4
from oracle.gdn import gdn_recurrent
from paper_2606_24031_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

REL = []     # (case, max error over the bound)


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def check(q, k, v, g, beta, s0, o, s, case):
    o_ref, s_ref, smax = gdn_recurrent(q, k, v, g, beta, s0)
    qn = np.sqrt((q.astype(np.float64) ** 2).sum(axis=2))            # [T, NH]
    bound_o = 2e-6 * qn[:, :, None] * smax[None, :, :] + 1e-30
    bound_s = 2e-6 * smax[:, None, :] + 1e-30
    eo = np.abs(o.astype(np.float64) - o_ref) / bound_o
    es = np.abs(s.astype(np.float64) - s_ref) / bound_s
    REL.append((case, float(eo.max()), float(es.max())))
    print(f"gdn {case}: max err/bound output {eo.max():.3g}, state {es.max():.3g}", flush=True)
    assert eo.max() <= 1.0, f"output error {eo.max():.3g} of the bound"
    assert es.max() <= 1.0, f"state error {es.max():.3g} of the bound"


# T: one token and up to 8 (the step kernel), 9 (the smallest chunked case, a
# ragged chunk), exactly one chunk, one past it, several chunks, the paper's
# 947-token prompt at its head shape (32 heads, 128 x 128)
@pytest.mark.parametrize("T,NH,DK,DV,state", [
    (1, 1, 128, 128, True), (5, 3, 128, 32, False), (8, 2, 128, 64, True),
    (9, 2, 64, 32, True), (32, 2, 128, 128, True),
    (33, 2, 64, 48, True), (100, 4, 128, 128, True), (947, 32, 128, 128, True)])
def test_gdn_matches_oracle(T, NH, DK, DV, state):
    g_ = synth.rng(1000 + T + NH)
    q, k, v, gate, beta, s0 = synth.gdn_inputs(g_, T, NH, DK, DV, with_state=state)
    o, s = w4.gdn_scan(dev(q), dev(k), dev(v), dev(gate), dev(beta), dev(s0))
    check(q, k, v, gate, beta, s0, o.cpu().numpy(), s.cpu().numpy(), f"T={T} NH={NH} DK={DK} DV={DV}")


# Two to four chunks (both register sets of the scan's loop, its exits), whole
# and ragged, and value columns that end inside a 16-column workgroup: 8 alone,
# 24 and 40 past one and two; 1 head and 8 (the per-XCD order)
@pytest.mark.parametrize("T", [10, 64, 65, 97])
@pytest.mark.parametrize("NH,DK,DV", [(1, 128, 8), (8, 64, 24), (3, 128, 40)])
def test_gdn_scan_edges(T, NH, DK, DV):
    g_ = synth.rng(2000 + T + NH + DV)
    q, k, v, gate, beta, s0 = synth.gdn_inputs(g_, T, NH, DK, DV, with_state=True)
    o, s = w4.gdn_scan(dev(q), dev(k), dev(v), dev(gate), dev(beta), dev(s0))
    check(q, k, v, gate, beta, s0, o.cpu().numpy(), s.cpu().numpy(), f"T={T} NH={NH} DK={DK} DV={DV}")


def test_gdn_state_handover_and_in_place_state():
    """Two calls (40, then 30 tokens) with the first call's final state as the
    second's initial state, written in place, against one 70-token run."""
    T, NH, DK, DV = 70, 2, 128, 64
    g_ = synth.rng(1100)
    q, k, v, gate, beta, s0 = synth.gdn_inputs(g_, T, NH, DK, DV)
    st = dev(s0)
    o1, _ = w4.gdn_scan(dev(q[:40]), dev(k[:40]), dev(v[:40]), dev(gate[:40]), dev(beta[:40]),
                        st, s_out=st)
    o2, _ = w4.gdn_scan(dev(q[40:]), dev(k[40:]), dev(v[40:]), dev(gate[40:]), dev(beta[40:]),
                        st, s_out=st)
    o = np.concatenate([o1.cpu().numpy(), o2.cpu().numpy()])
    check(q, k, v, gate, beta, s0, o, st.cpu().numpy(), "handover 40+30")


def test_gdn_memory_case_is_exact():
    """Decay 1, step 1, keys and queries orthonormal basis vectors (a key
    repeated later), integer values: every intermediate of the chunk form is
    a small integer combination of stored values, exact in fp32, so the
    outputs are the written values bit for bit."""
    DK, DV, NH = 128, 32, 2
    keys = [3, 17, 3, 100, 17, 0, 127, 3] * 5
    T = len(keys)
    g_ = synth.rng(1200)
    v = g_.integers(-64, 65, size=(T, NH, DV)).astype(np.float32)
    k = np.zeros((T, NH, DK), np.float32)
    for t, key in enumerate(keys):
        k[t, :, key] = 1.0
    gate = np.zeros((T, NH), np.float32)
    beta = np.ones((T, NH), np.float32)
    o, s = w4.gdn_scan(dev(k), dev(k), dev(v), dev(gate), dev(beta))
    assert np.array_equal(o.cpu().numpy(), v)
