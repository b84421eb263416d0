"""The one-wave-per-query-block forward (bf16, D = 128, 2,048 rows and up, heads
with even lists) against the two-wave kernel, which the parity tests hold to
the oracle: the same heads computed together (one-wave) and in two halves of
fewer than 2,048 rows (two-wave).  Each is within the parity bar (2e-2 + 2^-8
|ref|, each rounds P and O to bf16) of the exact result, so they differ by at
most twice that."""
import numpy as np
import pytest
import torch

import paper_2609_32882_amd as vsa2
from parity import MAX_ABS, REL_L2, ULP_REL, value_errors
from workload import Problem, Selection, Workload, make_inputs

pytestmark = pytest.mark.gpu

B2 = dict(dtype=1)
CASES = {
    # 33 cubes (rows not a multiple of anything), list lengths 16 (the shortest taken) and 33 (every block)
    "short": (Problem(1, 64, 64, 128, 12, 44, 4, **B2), Selection(0, 16), False),
    "all-blocks": (Problem(1, 64, 64, 128, 12, 44, 4, **B2), Selection(0, 33), False),
    # every axis cut: half-tiles without a real key, padding queries; grouped heads
    "padded-gqa": (Problem(1, 64, 16, 128, 7, 13, 22, **B2), Selection(0, 17), False),
    # lists longer than the 64 entries a wave holds at a time
    "long-lists": (Problem(1, 24, 24, 128, 16, 24, 16, **B2), Selection(0, 90), False),
    # ragged text tail; the text rows are longer than the paced ones
    "text": (Problem(1, 64, 64, 128, 12, 44, 4, text_len=70, **B2), Selection(0, 24), False),
    # large-magnitude blocks: two-term P in the training forward
    "skewed": (Problem(1, 64, 64, 128, 12, 44, 4, **B2), Selection(0, 20), True),
    # uneven lists: these heads stay with the two-wave kernel inside the same call
    "mass": (Problem(1, 64, 64, 128, 12, 44, 4, **B2), Selection(1, 0, 0.9, 30), True),
}


def assert_close(got, ref):
    _, beyond, rel = value_errors(got, ref, 2 * ULP_REL["bf16"])
    assert beyond <= 2 * MAX_ABS and rel <= REL_L2, (beyond, rel)


def slice_lists(r, rows, h0, h1):
    """CSR of the heads [h0, h1) (rows per head given)."""
    rp = r["row_ptr"][h0 * rows:h1 * rows + 1]
    return (rp - rp[0]).contiguous(), r["col_idx"][int(rp[0]):int(rp[-1])].contiguous()


@pytest.mark.parametrize("training", [False, True])
@pytest.mark.parametrize("name", CASES)
def test_one_wave_forward_matches_two_wave(name, training):
    p, sel, skewed = CASES[name]
    assert p.heads_q * p.N_joint >= 2048 and p.heads_q // 2 * p.N_joint < 2048
    x = make_inputs(Workload(name, p, sel, 77, skewed=skewed), with_grad=False)
    q, k, v = (torch.from_numpy(x[n]).bfloat16().cuda() for n in "qkv")
    R = (p.Rt, p.Rh, p.Rw)
    r = vsa2.route(p, sel, vsa2.pool(p, q, R), vsa2.pool(p, k, R))
    if p.text_len:
        r = vsa2.joint_lists(p, r)

    def run(p, q, k, v, rp, ci):
        out = vsa2.attn_fwd(p, q, k, v, rp, ci, training=training)
        o = out[0].float()
        return (o + out[2].float() if training else o).cpu().numpy(), out[1].cpu().numpy()

    o, lse = run(p, q, k, v, r["row_ptr"], r["col_idx"])
    again = run(p, q, k, v, r["row_ptr"], r["col_idx"])
    assert np.array_equal(o, again[0]) and np.array_equal(lse, again[1])
    half, hkv = p.heads_q // 2, p.heads_kv // 2
    for i in range(2):
        ph = p.replace(heads_q=half, heads_kv=hkv)
        rp, ci = slice_lists(r, p.N_joint, i * half, (i + 1) * half)
        oh, lh = run(ph, *(t[:, i * s:(i + 1) * s].contiguous() for t, s in ((q, half), (k, hkv), (v, hkv))), rp, ci)
        assert_close(o[:, i * half:(i + 1) * half], oh)
        got = lse[:, i * half:(i + 1) * half]
        assert np.array_equal(np.isinf(got), np.isinf(lh))
        fin = np.isfinite(lh)
        # sums of the same fp32 exponentials in another order
        assert np.abs(got[fin] - lh[fin]).max() <= 2e-5 * max(1.0, np.abs(lh[fin]).max())


def test_entries_outside_the_range_are_skipped():
    """-1 entries (as joint_lists emits for malformed ones) carry no weight."""
    p, sel, _ = CASES["short"]
    x = make_inputs(Workload("neg", p, sel, 78), with_grad=False)
    q, k, v = (torch.from_numpy(x[n]).bfloat16().cuda() for n in "qkv")
    rows, kk = p.heads_q * p.N, 18
    ci = torch.stack([torch.randperm(p.N)[:kk].sort()[0] for _ in range(rows)]).to(torch.int32)
    holes = ci.clone()
    holes[:, 0] = -1                      # first, middle and last entries
    holes[:, 7] = -1
    holes[::2, kk - 1] = p.N + 5
    rp = (torch.arange(rows + 1) * kk).to(torch.int32).cuda()
    o, lse = vsa2.attn_fwd(p, q, k, v, rp, holes.reshape(-1).contiguous().cuda())
    keep = (holes >= 0) & (holes < p.N)
    rp2 = torch.cat([torch.zeros(1, dtype=torch.int64), keep.sum(1).cumsum(0)]).to(torch.int32).cuda()
    o2, lse2 = vsa2.attn_fwd(p, q, k, v, rp2, holes[keep].contiguous().cuda())
    assert_close(o.float().cpu().numpy(), o2.float().cpu().numpy())
    assert float((lse - lse2).abs().max()) <= 2e-5 * max(1.0, float(lse2.abs().max()))
