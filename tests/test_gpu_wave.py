"""The one-wave-per-query-block forward (bf16, D = 128, from 2,048 rows of 320
blocks a head, heads with even lists) against the two-wave kernel, which the
parity tests hold to the oracle: the same heads computed together (one-wave) and
in two halves of fewer than 2,048 rows (two-wave); which kernel took which head
is read from the call's workspace.  Each is within the parity bar (2e-2 + 2^-8
|ref|, each rounds P and O to bf16) of the exact result, so they differ by at
most twice that."""
import numpy as np
import pytest
import torch

import paper_2609_32882_amd as vsa2
from parity import MAX_ABS, REL_L2, ULP_REL, value_errors
from workload import Problem, Selection, Workload, make_inputs

pytestmark = pytest.mark.gpu

PACE_BYTES = 8192      # pacing words, between the work order and the heads' averages

B2 = dict(dtype=1)
CASES = {
    # 330 cubes (rows not a multiple of anything), list lengths 24 (the shortest taken) and 330 (every block)
    "short": (Problem(1, 8, 8, 128, 12, 44, 40, **B2), Selection(0, 24), False),
    "all-blocks": (Problem(1, 8, 8, 128, 12, 44, 40, **B2), Selection(0, 330), False),
    # every axis cut: half-tiles without a real key, padding queries; grouped heads
    "padded-gqa": (Problem(1, 8, 2, 128, 15, 42, 30, **B2), Selection(0, 25), False),
    # lists longer than the 64 entries a wave holds at a time
    "long-lists": (Problem(1, 8, 8, 128, 12, 44, 40, **B2), Selection(0, 90), False),
    # ragged text tail; the text rows are longer than the paced ones
    "text": (Problem(1, 8, 8, 128, 12, 44, 40, text_len=70, **B2), Selection(0, 30), False),
    # large-magnitude blocks: in the training forward most rows take two-term P, and their heads the two-wave kernel
    "skewed": (Problem(1, 8, 8, 128, 12, 44, 40, **B2), Selection(0, 30), True),
    # uneven lists: these heads stay with the two-wave kernel inside the same call
    "mass": (Problem(1, 8, 8, 128, 12, 44, 40, **B2), Selection(1, 0, 0.9, 60), True),
}


def assert_close(got, ref):
    _, beyond, rel = value_errors(got, ref, 2 * ULP_REL["bf16"])
    assert beyond <= 2 * MAX_ABS and rel <= REL_L2, (beyond, rel)


def slice_lists(r, rows, h0, h1):
    """CSR of the heads [h0, h1) (rows per head given)."""
    rp = r["row_ptr"][h0 * rows:h1 * rows + 1]
    return (rp - rp[0]).contiguous(), r["col_idx"][int(rp[0]):int(rp[-1])].contiguous()


def one_wave_heads(p, row_ptr, qkv=None):
    """Per query head, the average list length where the rule gives the head to
    the one-wave kernel, else 0, computed on the host: at least 24 entries on
    average (below 8,192 rows), 7 of 8 rows within 1/16 of the average and, in
    training (qkv given), at most half of the query blocks flagged (a magnitude
    above 7, or NaN) and at most 0.7 flagged key blocks in an average list."""
    n = p.N_joint
    assert p.batch * p.heads_q * n < 8192
    lens = np.diff(row_ptr.cpu().numpy().astype(np.int64)).reshape(-1, n)
    avg = (lens.sum(1).astype(np.float32) / np.float32(n)).astype(np.float32)
    near = (np.abs(lens.astype(np.float32) - avg[:, None]) <= avg[:, None] * np.float32(1 / 16)).sum(1)
    take = (avg >= 24) & (near >= n - n // 8)
    if qkv is not None:
        fq, fk, fv = (~(t.float().abs() <= 7).reshape(-1, n, 64 * p.head_dim).all(-1).cpu().numpy() for t in qkv)
        take &= 2 * fq.sum(1) <= n
        take &= np.repeat((fk | fv).sum(1), p.heads_q // p.heads_kv) * avg <= 0.7 * n
    return np.where(take, avg, np.float32(0))


def _align256(n):
    return (n + 255) // 256 * 256


def forward(p, q, k, v, rp, ci, training):
    """O (with its remainder when training), LSE as numpy, and the per-head
    average list lengths that the library's rule stored (0: two-wave), or None
    below 2,048 rows.  Outputs are prefilled, so a row that no kernel writes shows."""
    P = vsa2.problem_from(p)
    st, wsb = vsa2.vsa2_attn_workspace(P, 0)
    assert st == 0
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    fill = 1.25e30
    o, o_lo = torch.full_like(q, fill), torch.full_like(q, fill)
    lse = torch.full((p.batch, p.heads_q, p.L_joint), fill, device="cuda")
    st = vsa2.vsa2_attn_fwd(P, q.data_ptr(), k.data_ptr(), v.data_ptr(), rp.data_ptr(), ci.data_ptr(), ci.numel(),
                            o.data_ptr(), lse.data_ptr(), o_lo.data_ptr() if training else None, ws.data_ptr(), wsb,
                            torch.cuda.current_stream().cuda_stream)
    assert st == 0, vsa2.STATUS_NAMES[st]
    rows, even = p.batch * p.heads_q * p.N_joint, None
    if rows >= 2048:
        assert p.N_joint >= 320          # else the workspace holds no averages
        at = _align256(4 * rows) + PACE_BYTES
        even = ws[at:at + 4 * p.batch * p.heads_q].view(torch.float32).cpu().numpy()
    out = o.float() + o_lo.float() if training else o.float()
    assert not (o.float() == torch.tensor(fill).bfloat16().float().item()).any() and not (lse == fill).any()
    return out.cpu().numpy(), lse.cpu().numpy(), even


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

    o, lse, even = forward(p, q, k, v, r["row_ptr"], r["col_idx"], training)
    want = one_wave_heads(p, r["row_ptr"], (q, k, v) if training else None)
    assert np.array_equal(even > 0, want > 0) and np.allclose(even, want, rtol=1e-6)
    assert (even == 0).all() if name == "mass" or (name == "skewed" and training) else (even > 0).all()
    again = forward(p, q, k, v, r["row_ptr"], r["col_idx"], training)
    assert np.array_equal(o, again[0]) and np.array_equal(lse, again[1])
    half, hkv = p.heads_q // 2, p.heads_kv // 2
    for i in range(2):
        ph = p.replace(heads_q=half, heads_kv=hkv)
        rp, ci = slice_lists(r, p.N_joint, i * half, (i + 1) * half)
        oh, lh, _ = forward(ph, *(t[:, i * s:(i + 1) * s].contiguous() for t, s in ((q, half), (k, hkv), (v, hkv))), rp, ci,
                            training)
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
    rows, kk = p.heads_q * p.N, 27
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
