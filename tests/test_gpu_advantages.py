"""Parity of the HIP espo_advantages with the CPU oracle, through the C ABI (needs an MI355X)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2605_29860_amd as espo  # noqa: E402
from paper_2605_29860_amd import workloads as W  # noqa: E402
import harness as H  # noqa: E402


def _say(msg):
    print(msg, flush=True)


def _batch(B, T, seed, lengths=None, stop_p=0.4, poison=True):
    g = torch.Generator().manual_seed(seed)
    rewards = torch.randn(B, T, generator=g)
    values = torch.rand(B, T, generator=g) * 2 - 1
    L = torch.randint(0, T + 1, (B,), generator=g) if lengths is None else torch.as_tensor(lengths)
    stopped = (torch.rand(B, generator=g) < stop_p).to(torch.uint8)
    if poison:
        pad = torch.arange(T)[None, :] >= L.clamp(0, T)[:, None]
        rewards[pad] = float("nan")
        values[pad] = float("nan")
    return rewards.cuda(), values.cuda(), L.to(torch.int32).cuda(), stopped.cuda()


@pytest.mark.parametrize("T", [1, 3, 4, 7, 8, 9, 64, 511, 512, 2047, 2048, 2049, 4100, 6151])
def test_shapes_and_ragged_lengths(T):
    _say(f"[case] advantages T={T}")
    B = 9
    L = [0, T, 1, max(T - 1, 0), T // 2, min(T, 2048), min(T, 2049), min(T, 513), T]
    for gamma, lam in ((1.0, 0.95), (0.99, 0.9), (1.0, 1.0), (0.9, 0.0)):
        r, v, Lt, s = _batch(B, T, seed=T, lengths=L)
        H.check_advantages(r, v, Lt, s, -1.0, gamma, lam)


def test_out_of_range_lengths_and_empty():
    _say("[case] advantages clamping / empty")
    B, T = 4, 100
    r, v, _, s = _batch(B, T, seed=1, lengths=[T, T, T, T], poison=False)
    L = torch.tensor([-3, T + 50, 0, 17], dtype=torch.int32).cuda()
    H.check_advantages(r, v, L, s, -1.0, 1.0, 0.95)
    e = torch.zeros(0, 5, device="cuda")
    espo.espo_advantages(e, e, torch.zeros(0, dtype=torch.int32, device="cuda"),
                         torch.zeros(0, dtype=torch.uint8, device="cuda"), -1.0, 1.0, 0.95, e.clone(), e.clone())
    with pytest.raises(espo.EspoError):
        espo.espo_advantages(r, v, L, s, -1.0, float("nan"), 0.95, torch.empty_like(r), torch.empty_like(r))


def test_closed_forms_on_device():
    _say("[case] advantages closed forms")
    # zero values, stopped: A_t = r_fail c^(L-1-t); gamma = lambda = 1: A_t = return-to-go - V_t
    B, T = 3, 5000
    z = torch.zeros(B, T, device="cuda")
    L = torch.tensor([5000, 3000, 1], dtype=torch.int32, device="cuda")
    st = torch.ones(B, dtype=torch.uint8, device="cuda")
    td, adv = torch.empty_like(z), torch.empty_like(z)
    espo.espo_advantages(z, z, L, st, -1.0, 1.0, 0.95, td, adv)
    a = adv.cpu().numpy().astype(np.float64)
    c = float(np.float32(0.95))
    for b, n in enumerate([5000, 3000, 1]):
        ref = -1.0 * c ** (n - 1 - np.arange(n))
        np.testing.assert_allclose(a[b, :n], ref, rtol=2e-5, atol=1e-30)
        assert (a[b, n:] == 0).all()
    r, v, Lr, s = _batch(6, 3000, seed=5)
    H.check_advantages(r, v, Lr, s, -2.0, 1.0, 1.0)


def test_config5_full_size():
    _say("[case] config 5 (B=1024, T=16384)")
    r, v, L, s = W.advantage_batch(device="cuda", poison=True, seed=5)
    assert r.shape == (1024, 16384)
    worst = H.check_advantages(r, v, L, s, -1.0, 1.0, 0.95)
    frac = float(s.float().mean())
    _say(f"  config 5: valid tokens {int(L.sum())}, stopped fraction {frac:.2f}, worst scaled error {worst:.2e}")
    assert 0.2 < frac < 0.4
    # a second call on the same inputs gives the same bits
    td1, adv1 = torch.empty_like(r), torch.empty_like(r)
    td2, adv2 = torch.empty_like(r), torch.empty_like(r)
    espo.espo_advantages(r, v, L, s, -1.0, 1.0, 0.95, td1, adv1)
    espo.espo_advantages(r, v, L, s, -1.0, 1.0, 0.95, td2, adv2)
    torch.cuda.synchronize()
    assert torch.equal(td1, td2) and torch.equal(adv1, adv2)


def test_ablation_variant_without_the_failure_penalty():
    _say("[case] advantages, variant C (no terminal penalty)")
    # Section 6, variant C: trajectories are truncated by the stop rule but get no failure reward.  That is this
    # call with every `stopped` flag zero: the truncated row keeps its stored last reward (0 in Algorithm 1).
    # Checked against the oracle, and against the full method on the same rows: only the rows that the rule had
    # stopped change, by r_fail (gamma lambda)^(L-1-t).
    r, v, L, s = W.advantage_batch(B=64, T=3000, len_lo=1, seed=31, device="cuda", poison=True)
    none = torch.zeros_like(s)
    H.check_advantages(r, v, L, none, -1.0, 1.0, 0.95)
    td_c, adv_c = torch.empty_like(r), torch.empty_like(r)
    td_a, adv_a = torch.empty_like(r), torch.empty_like(r)
    espo.espo_advantages(r, v, L, none, -1.0, 1.0, 0.95, td_c, adv_c)
    espo.espo_advantages(r, v, L, s, -1.0, 1.0, 0.95, td_a, adv_a)
    torch.cuda.synchronize()
    diff = (adv_a - adv_c).cpu().numpy().astype(np.float64)
    L_h, s_h = L.cpu().numpy(), s.cpu().numpy()
    assert s_h.any() and not s_h.all()
    c = float(np.float32(0.95))
    for b in range(64):
        n = int(L_h[b])
        want = -1.0 * c ** (n - 1 - np.arange(n)) if s_h[b] else np.zeros(n)   # the stored last reward of a stopped row is 0
        np.testing.assert_allclose(diff[b, :n], want, rtol=0, atol=1e-4)    # two fp32 scans of sums of size ~30
        assert (diff[b, n:] == 0).all()


@pytest.mark.parametrize("B", [513, 1025, 2500, 4096, 4097])
def test_many_rows(B):
    _say(f"[case] advantages B={B}")
    # More rows than workgroups fit on the chip at once: every row must still be processed
    # exactly once (outputs are pre-filled with a sentinel by the check), also with many equal
    # lengths, empty rows and lengths out of range.
    T = 260
    g = torch.Generator().manual_seed(B)
    L = torch.randint(0, T + 1, (B,), generator=g)
    L[::7] = T
    L[3::11] = 0
    L[5::13] = 17
    r, v, Lt, s = _batch(B, T, seed=B, lengths=L.tolist())
    H.check_advantages(r, v, Lt, s, -1.0, 1.0, 0.95)
    Lt[1] = -4
    Lt[2] = T + 100
    r = torch.nan_to_num(r, nan=0.0)
    v = torch.nan_to_num(v, nan=0.0)
    H.check_advantages(r, v, Lt, s, -0.5, 0.97, 0.9)
    # all rows of one length: the scans after the first 512 look their rows up by class of length and,
    # inside a class, by index; here that is one class, over several chunks of 1024 rows for the larger B
    r, v, Lt, s = _batch(B, T, seed=B + 1, lengths=[T - 1] * B)
    H.check_advantages(r, v, Lt, s, -1.0, 1.0, 0.95)


# --------------------------------------------------------------------------- terminal-reward form
def _terminal_batch(B, T, seed, lengths=None, stop_p=0.4):
    g = torch.Generator().manual_seed(seed)
    values = torch.rand(B, T, generator=g) * 2 - 1
    L = torch.randint(0, T + 1, (B,), generator=g) if lengths is None else torch.as_tensor(lengths)
    stopped = (torch.rand(B, generator=g) < stop_p).to(torch.uint8)
    term = torch.randint(0, 2, (B,), generator=g).float() + 0.25 * torch.randn(B, generator=g)
    values[torch.arange(T)[None, :] >= L.clamp(0, T)[:, None]] = float("nan")   # never to be read
    return values.cuda(), L.to(torch.int32).cuda(), stopped.cuda(), term.cuda()


@pytest.mark.parametrize("T", [1, 3, 4, 7, 8, 9, 64, 511, 512, 2047, 2048, 2049, 4100, 6151, 8192, 9000])
def test_terminal_form_shapes_and_options(T):
    _say(f"[case] advantages, terminal form T={T}")
    L = [0, T, 1, max(T - 1, 0), T // 2, min(T, 2048), min(T, 2049), min(T, 513), T, min(T, 4096), min(T, 4097)]
    v, Lt, s, term = _terminal_batch(len(L), T, seed=T, lengths=L)
    for gamma, lam in ((1.0, 0.95), (0.99, 0.9), (1.0, 1.0), (0.9, 0.0)):
        H.check_advantages_terminal(v, Lt, s, term, -1.0, gamma, lam, zero_padding=True, want_returns=True)
    H.check_advantages_terminal(v, Lt, s, term, -1.0, 1.0, 0.95, zero_padding=False, want_returns=True)
    H.check_advantages_terminal(v, Lt, s, term, -0.5, 1.0, 0.95, zero_padding=False, want_returns=False)
    H.check_advantages_terminal(v, Lt, s, term, -0.5, 1.0, 0.95, zero_padding=True, want_returns=False)


def test_terminal_form_equals_dense_form_bit_for_bit():
    _say("[case] advantages, terminal form vs dense form")
    B, T = 64, 9001
    v, L, s, term = _terminal_batch(B, T, seed=77)
    dense = torch.zeros(B, T, device="cuda")
    rows = torch.nonzero(L > 0).flatten()
    dense[rows, (L[rows] - 1).long()] = term[rows]
    td_d, adv_d = torch.empty_like(dense), torch.empty_like(dense)
    td_t, adv_t, ret = torch.empty_like(dense), torch.empty_like(dense), torch.empty_like(dense)
    espo.espo_advantages(dense, v, L, s, -1.0, 0.99, 0.95, td_d, adv_d)
    espo.espo_advantages_terminal(v, L, s, term, -1.0, 0.99, 0.95, td_t, adv_t, returns=ret)
    torch.cuda.synchronize()
    assert torch.equal(td_d, td_t) and torch.equal(adv_d, adv_t)
    valid = torch.arange(T, device="cuda")[None, :] < L[:, None]
    assert torch.equal(ret[valid], (adv_t + torch.nan_to_num(v))[valid]) and (ret[~valid] == 0).all()
    # lambda = 1: the value target is the discounted terminal reward, whatever the critic says
    espo.espo_advantages_terminal(v, L, s, term, -1.0, 0.999, 1.0, td_t, adv_t, returns=ret)
    torch.cuda.synchronize()
    r_end = torch.where(s > 0, torch.full_like(term, -1.0), term).double()
    dist = (L[:, None] - 1 - torch.arange(T, device="cuda")[None, :]).clamp(min=0).double()
    want = r_end[:, None] * float(np.float32(0.999)) ** dist
    err = (ret.double() - want).abs()[valid]
    assert float(err.max()) < 2e-4, float(err.max())     # ~9000 fp32 steps through values of size 1


def test_terminal_form_config5_full_size():
    _say("[case] config 5 in the terminal form (B=1024, T=16384)")
    r, v, L, s = W.advantage_batch(device="cuda", poison=True, seed=5)
    rows = torch.arange(r.shape[0], device="cuda")
    term = torch.nan_to_num(r[rows, (L - 1).clamp(min=0).long()])    # the survivors' terminal reward in {0, 1}
    worst = H.check_advantages_terminal(v, L, s, term, -1.0, 1.0, 0.95, zero_padding=False, want_returns=True)
    _say(f"  worst scaled error {worst:.2e}")
    worst = H.check_advantages_terminal(v, L, s, term, -1.0, 1.0, 0.95, zero_padding=True, want_returns=False)
    _say(f"  worst scaled error {worst:.2e}")


@pytest.mark.parametrize("part", range(5))
def test_seeded_sweep_of_both_forms(part):
    _say(f"[case] advantages, seeded sweep, part {part} (140 cases, both reward forms each)")
    rng = np.random.default_rng(4242 + part)
    worst = 0.0
    for case in range(part * 140, part * 140 + 140):
        T = int(rng.choice([rng.integers(1, 64), rng.integers(64, 5000), rng.integers(5000, 20000)]))
        B = int(rng.integers(1, 12))
        g = torch.Generator().manual_seed(7000 + case)
        v = (torch.rand(B, T, generator=g) * 2 - 1) * float(rng.choice([1.0, 30.0]))
        r = torch.randn(B, T, generator=g)
        L = torch.randint(0, T + 1, (B,), generator=g)
        pad = torch.arange(T)[None, :] >= L[:, None]
        v[pad] = float("nan")
        r[pad] = float("nan")
        s = (torch.rand(B, generator=g) < 0.4).to(torch.uint8)
        term = torch.randn(B, generator=g)
        gamma, lam = float(rng.choice([1.0, 0.99, 0.9])), float(rng.choice([0.95, 1.0, 0.0, 0.5]))
        r_fail = float(rng.choice([-1.0, -0.25, 0.0]))
        args = (v.cuda(), L.to(torch.int32).cuda(), s.cuda())
        try:
            worst = max(worst, H.check_advantages(r.cuda(), *args, r_fail, gamma, lam))
            worst = max(worst, H.check_advantages_terminal(*args, term.cuda(), r_fail, gamma, lam,
                                                           zero_padding=bool(rng.random() < 0.5),
                                                           want_returns=bool(rng.random() < 0.5)))
        except AssertionError as err:
            raise AssertionError(f"case {case}: T={T} B={B} gamma={gamma} lambda={lam} r_fail={r_fail}: {err}")
    _say(f"  worst scaled error {worst:.2e}")


@pytest.mark.parametrize("B,T", [(5, 1021), (5, 2045), (5, 2046), (5, 2048), (5, 2049), (5, 4099), (2, 8195), (513, 2047), (513, 2049), (513, 4093),
                                 (513, 4094), (513, 4096), (513, 4099), (514, 8193), (520, 9001), (1537, 8196)])
def test_rows_of_any_length_start_anywhere(B, T):
    # Rows whose length is no multiple of four start between 16-byte boundaries; short rows have workgroups of four
    # waves, several tiles long at most; from 513 long rows on the later ones are looked up by length.  Lengths sit at
    # the ends of tiles of 1024 and 4096 positions as counted from the boundary before a row.
    _say(f"[case] advantages B={B} T={T}")
    edges = [0, 1, 2, 3, 4, 5, 1021, 1022, 1023, 1024, 1025, 2048, 4093, 4094, 4095, 4096, 4097, T - 3, T - 1, T, T]
    lengths = [min(max(edges[b % len(edges)], 0), T) for b in range(B)]
    r, v, L, s = _batch(B, T, seed=T, lengths=lengths)
    H.check_advantages(r, v, L, s, -1.0, 1.0, 0.95)
    v, L, s, term = _terminal_batch(B, T, seed=T + 1, lengths=lengths)
    H.check_advantages_terminal(v, L, s, term, -1.0, 0.99, 0.97, zero_padding=True, want_returns=True)
    H.check_advantages_terminal(v, L, s, term, -1.0, 0.99, 0.97, zero_padding=False, want_returns=True)


# ------------------------------------------------------------------ trajectories stored back to back

def _packed(lens, seed, gaps=None, scale=1.0, stop_p=0.4):
    """Values, rewards, extents for the given lengths; `gaps[b]` unowned tokens (NaN) before trajectory b."""
    g = torch.Generator().manual_seed(seed)
    B = len(lens)
    gaps = [0] * B if gaps is None else gaps
    starts, pos = [], 0
    for b in range(B):
        pos += gaps[b]
        starts.append(pos)
        pos += lens[b]
    N = pos
    values = (torch.rand(N, generator=g) * 2 - 1) * scale
    rewards = torch.randn(N, generator=g)
    owned = torch.zeros(N, dtype=torch.bool)
    for b in range(B):
        owned[starts[b]:starts[b] + lens[b]] = True
    values[~owned] = float("nan")
    rewards[~owned] = float("nan")
    stopped = (torch.rand(B, generator=g) < stop_p).to(torch.uint8)
    term = torch.randn(B, generator=g)
    return values.cuda(), rewards.cuda(), starts, stopped.cuda(), term.cuda()


def _check_packed_both_forms(lens, seed, gaps=None, gamma=1.0, lam=0.95, r_fail=-1.0, scale=1.0):
    """With gaps the extents are not one running sum, so gapped layouts go one call per extent pair:
    cu = [start_b, end_b] is a valid one-trajectory call into the same arrays."""
    v, r, starts, s, term = _packed(lens, seed, gaps, scale)
    worst = 0.0
    if gaps is None:
        cu = torch.tensor(starts + [starts[-1] + lens[-1]] if lens else [0], dtype=torch.int64).cuda()
        worst = max(worst, H.check_advantages_packed(v, cu, s, r_fail, gamma, lam, rewards=r, want_returns=False))
        worst = max(worst, H.check_advantages_packed(v, cu, s, r_fail, gamma, lam, term=term, want_returns=True))
    else:
        for b in range(len(lens)):
            cu = torch.tensor([starts[b], starts[b] + lens[b]], dtype=torch.int64).cuda()
            worst = max(worst, H.check_advantages_packed(v, cu, s[b:b + 1], r_fail, gamma, lam, rewards=r, want_returns=True))
            worst = max(worst, H.check_advantages_packed(v, cu, s[b:b + 1], r_fail, gamma, lam, term=term[b:b + 1], want_returns=False))
    return worst


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 7, 8, 63, 64, 257, 4093, 4096, 4097, 8191, 8200, 12289])
def test_packed_every_alignment_of_start_and_end(L):
    _say(f"[case] packed advantages, L={L}")
    # neighbours of 1..3 tokens shift the start through all four alignments; each one is a trajectory itself
    lens = [L, 1, L, 2, L, 3, L, 0, L, 5, 0, 0, L]
    for gamma, lam in ((1.0, 0.95), (0.99, 0.9), (1.0, 1.0), (0.9, 0.0)):
        _check_packed_both_forms(lens, seed=L, gamma=gamma, lam=lam)


@pytest.mark.parametrize("B,mean", [(3, 1023), (3, 1025), (513, 500), (600, 2047), (600, 2049), (600, 4200)])
def test_packed_batches_of_short_and_long_trajectories(B, mean):
    # the number of waves and the order follow from the mean length; a few trajectories are many times as long
    _say(f"[case] packed advantages, B={B} mean length {mean}")
    g = torch.Generator().manual_seed(B + mean)
    lens = torch.randint(0, mean, (B,), generator=g).tolist()
    lens[0], lens[-1], lens[B // 2] = 0, 5 * mean + 3, 9 * mean + 1
    lens[1] = max(0, mean * B - (sum(lens) - lens[1]))
    _check_packed_both_forms(lens, seed=B)


@pytest.mark.parametrize("gamma,lam", [(1.0, 0.95), (0.999, 0.9995)])
def test_packed_long_trajectories_among_many_short_ones(gamma, lam):
    _say(f"[case] packed advantages, long trajectories in workgroups of four waves, gamma {gamma} lambda {lam}")
    # The waves follow from the mean length.  Of a long trajectory the tiles of 1024 tokens between the first and the last are
    # walked in pairs: none to eight of them here, both ends on and beside the edges, starts at all four alignments.
    lens = []
    for n in (2046, 2048, 2049, 2052, 3071, 3072, 3073, 3076, 4096, 4097, 5119, 5121, 6144, 6147, 7170, 8193, 9217, 10243, 30001):
        lens += [n] + [1, 2, 3, 7, 50][:1 + len(lens) % 4] * 8
    lens += [300] * 200
    assert 2 * (sum(lens) // len(lens)) <= 2048
    _check_packed_both_forms(lens, seed=11, gamma=gamma, lam=lam)


def test_packed_gaps_are_neither_read_nor_written():
    _say("[case] packed advantages, unowned gaps")
    lens = [5, 4096, 1, 300, 4099, 2, 8193]
    gaps = [3, 1, 2, 5, 0, 7, 1]
    _check_packed_both_forms(lens, seed=11, gaps=gaps)


def test_packed_extents_are_clipped_and_empty_batches():
    _say("[case] packed advantages, clipping / empty")
    v, r, starts, s, term = _packed([100, 50], seed=12)
    N = v.numel()
    td, adv = torch.full((N,), 7.0, device="cuda"), torch.full((N,), 7.0, device="cuda")
    ref_td, ref_adv = torch.full((N,), 7.0, device="cuda"), torch.full((N,), 7.0, device="cuda")
    espo.espo_advantages_packed(v, torch.tensor([0, 100, 150]).cuda(), s, -1.0, 1.0, 0.95, ref_td, ref_adv, terminal_reward=term)
    espo.espo_advantages_packed(v, torch.tensor([-9, 100, 10**12]).cuda(), s, -1.0, 1.0, 0.95, td, adv, terminal_reward=term)
    torch.cuda.synchronize()
    assert torch.equal(td, ref_td) and torch.equal(adv, ref_adv)
    td.fill_(7.0)
    espo.espo_advantages_packed(v, torch.tensor([120, 30, 10]).cuda(), s, -1.0, 1.0, 0.95, td, adv, terminal_reward=term)
    torch.cuda.synchronize()
    assert (td == 7.0).all()                                  # reversed extents hold no token
    H.check_advantages_packed(v, torch.tensor([-9, 100, 10**12]).cuda(), s, -1.0, 1.0, 0.95, rewards=r)
    e = torch.zeros(0, device="cuda")
    espo.espo_advantages_packed(e, torch.zeros(1, dtype=torch.int64, device="cuda"), torch.zeros(0, dtype=torch.uint8, device="cuda"),
                                -1.0, 1.0, 0.95, e.clone(), e.clone(), terminal_reward=e.clone())
    with pytest.raises(espo.EspoError):                       # both reward forms at once
        espo.espo_advantages_packed(v, torch.tensor([0, 100, 150]).cuda(), s, -1.0, 1.0, 0.95, td, adv, rewards=r, terminal_reward=term)
    with pytest.raises(espo.EspoError):                       # a view that starts 4 bytes into an allocation
        espo.espo_advantages_packed(v[1:], torch.tensor([0, 100, 149]).cuda(), s, -1.0, 1.0, 0.95, td[1:], adv[1:], terminal_reward=term)


def test_packed_config5_full_size():
    _say("[case] config 5 stored back to back (B=1024, lengths as in the padded workload)")
    r, v, L, s = W.advantage_batch(device="cuda", poison=False, seed=5)
    B, T = v.shape
    valid = torch.arange(T, device="cuda")[None, :] < L[:, None]
    cu = torch.zeros(B + 1, dtype=torch.int64, device="cuda")
    cu[1:] = torch.cumsum(L.long(), 0)
    vp, rp = v[valid].contiguous(), r[valid].contiguous()
    rows = torch.arange(B, device="cuda")
    term = r[rows, (L - 1).clamp(min=0).long()].contiguous()
    _say(f"  N = {vp.numel()} of {B * T}")
    worst = H.check_advantages_packed(vp, cu, s, -1.0, 1.0, 0.95, rewards=rp, want_returns=False)
    _say(f"  dense form: worst scaled error {worst:.2e}")
    worst = H.check_advantages_packed(vp, cu, s, -1.0, 1.0, 0.95, term=term, want_returns=True)
    _say(f"  terminal form: worst scaled error {worst:.2e}")


# From 257 rows on a workgroup of 8 waves walks a row, two spans of 256 tokens of a tile of 4096 to a wave: both sides of that line, with
# and without targets, lengths at the edges of spans, of a wave's first and second one, and of tiles.
@pytest.mark.parametrize("B,T", [(256, 8192), (257, 8192), (257, 8195), (513, 4612), (257, 4097), (257, 13824), (257, 13828)])
@pytest.mark.parametrize("gamma,lam", [(1.0, 0.95), (0.999, 0.9995)])
def test_rows_walked_by_two_spans_a_wave(B, T, gamma, lam):
    _say(f"[case] two spans a wave B={B} T={T} gamma={gamma} lambda={lam}")
    edges = [0, 1, 255, 256, 257, 2047, 2048, 2049, 2305, 4095, 4096, 4097, 6143, 6145, 8191, 8192, 8193, T - 1, T]
    L = [min(edges[b % len(edges)], T) for b in range(B)]
    r, v, Lt, s = _batch(B, T, seed=T + B, lengths=L)
    H.check_advantages(r, v, Lt, s, -1.0, gamma, lam)
    term = torch.randn(B, generator=torch.Generator().manual_seed(B)).cuda()
    for fill, returns in ((True, True), (False, True), (False, False)):
        H.check_advantages_terminal(v, Lt, s, term, -1.0, gamma, lam, zero_padding=fill, want_returns=returns)
    _check_packed_both_forms([max(n - b % 3, 0) for b, n in enumerate(L)], seed=T, gamma=gamma, lam=lam)


# Back to back with rewards and targets, 16 waves walk a row again beyond a mean length of 6912: both sides of that line.
@pytest.mark.parametrize("mean", [6912, 6913])
def test_packed_rewards_and_targets_of_long_trajectories(mean):
    _say(f"[case] packed advantages with rewards and targets, mean length {mean}")
    lens = [mean + (-1) ** b * (b // 2 * 47) for b in range(256)] + [mean]
    assert sum(lens) // len(lens) == mean
    v, r, starts, s, term = _packed(lens, seed=mean)
    cu = torch.tensor(starts + [starts[-1] + lens[-1]], dtype=torch.int64).cuda()
    H.check_advantages_packed(v, cu, s, -1.0, 1.0, 0.95, rewards=r, want_returns=True)


@pytest.mark.parametrize("part", range(4))
def test_packed_seeded_sweep(part):
    _say(f"[case] packed advantages, seeded sweep, part {part} (100 cases, both reward forms each)")
    rng = np.random.default_rng(5151 + part)
    worst = 0.0
    for case in range(part * 100, part * 100 + 100):
        B = int(rng.integers(1, 24))
        top = int(rng.choice([8, 200, 5000, 14000]))
        lens = [int(x) for x in rng.integers(0, top + 1, B)]
        for b in range(B):
            if rng.random() < 0.15:
                lens[b] = 0
        gamma, lam = float(rng.choice([1.0, 0.99, 0.9])), float(rng.choice([0.95, 1.0, 0.0, 0.5]))
        r_fail = float(rng.choice([-1.0, -0.25, 0.0]))
        try:
            worst = max(worst, _check_packed_both_forms(lens, 9000 + case, gamma=gamma, lam=lam, r_fail=r_fail,
                                                        scale=float(rng.choice([1.0, 30.0]))))
        except AssertionError as err:
            raise AssertionError(f"case {case}: lens={lens[:8]}... gamma={gamma} lambda={lam} r_fail={r_fail}: {err}")
    _say(f"  worst scaled error {worst:.2e}")
