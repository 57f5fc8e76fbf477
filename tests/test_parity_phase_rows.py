"""Rows that do not start on a 16-byte boundary or are not a whole number of 16-byte chunks long: the
kernels take each row as its whole aligned chunks and single entries at its ends (short bf16 rows
as the chunks that cover them) and write only the row's own entries. Every case compares lp,
loss_tok, flags and dlogits with the oracle, and checks that every byte of the buffers outside the
rows is left as it was (the entries between rows, before the first row and after the last)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_12070_amd as P

from helpers import compare_loss, oracle_anchor, oracle_params, run_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SENTINEL = 7.0                      # exactly representable in bf16


def _say(*a):
    print("[case]", *a, flush=True)


def _inputs(T, V, ld, off, seed):
    """Logits rows of length V at element offset `off` of a buffer, row stride ld; ids with
    the first and last entries of rows, a bad id, masked rows."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n = off + T * ld + 16
    buf = (torch.randn(n, generator=g, device=DEV) * 3).to(torch.bfloat16)
    z = buf[off:off + T * ld].view(T, ld)[:, :V]
    ids = torch.randint(0, V, (T,), generator=g, device=DEV)
    ids[0] = V - 1
    ids[1] = 0
    if T > 5:
        ids[5] = V + 3                   # bad id on a valid row
    mask = torch.ones(T, dtype=torch.uint8, device=DEV)
    mask[3::7] = 0
    anchor = oracle_anchor(z, ids.clamp(0, V - 1)).to(DEV)
    lp_ref = (anchor + 0.2 * torch.randn(T, generator=g, device=DEV, dtype=torch.float64)).float()
    lp_mu = (lp_ref.double() + 0.1 * torch.randn(T, generator=g, device=DEV,
                                                 dtype=torch.float64)).float()
    adv = torch.randn(T, generator=g, device=DEV)
    return buf, z, ids, mask, lp_mu, lp_ref, adv


def _outside(buf, off, T, ld, V):
    """Boolean mask of the buffer entries that belong to no row."""
    m = torch.ones(buf.numel(), dtype=torch.bool, device=buf.device)
    rows = off + torch.arange(T, device=buf.device)[:, None] * ld + torch.arange(V, device=buf.device)[None, :]
    m[rows.reshape(-1)] = False
    return m


CASES = [  # T, V, extra columns per row, element offset of row 0
    (40, 1, 0, 3), (40, 9, 0, 1), (300, 1003, 0, 0), (300, 1003, 5, 7), (200, 5003, 3, 1),
    (600, 8192, 1, 0), (120, 32001, 0, 5), (64, 50257, 0, 0), (64, 50257, 47, 2),
    (24, 151665, 271, 0), (24, 151937, 0, 6), (12, 155641, 0, 7),
]


@pytest.mark.parametrize("T,V,extra,off", CASES, ids=[f"T{c[0]}_V{c[1]}_x{c[2]}_o{c[3]}" for c in CASES])
def test_phase_rows_loss_and_untouched_neighbours(T, V, extra, off):
    ld = V + extra
    _say("phase rows", T, V, ld, off)
    buf, z, ids, mask, lp_mu, lp_ref, adv = _inputs(T, V, ld, off, seed=V + off)
    name = P.row_kernel_name(torch.bfloat16, V, ld)
    if (ld % 8 == 0) and (V % 8 == 0):
        assert "phase" not in name
    else:
        assert "phase" in name or "prefix" in name, name
    # dlogits into a second buffer with the same layout, filled with a sentinel
    dbuf = torch.full_like(buf, SENTINEL)
    d = dbuf[off:off + T * ld].view(T, ld)[:, :V]
    params = oracle_params((0.5, 2.0), (0.2, 0.2), "mask_weight", "const", 1.0)
    res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d,
                                       scale_mode="const")
    torch.cuda.synchronize()
    ref = run_oracle(z, ids, lp_mu, lp_ref, adv, mask, None, params)
    compare_loss(res, ref, params, torch.bfloat16)
    out = _outside(dbuf, off, T, ld, V)
    assert torch.all(dbuf[out] == SENTINEL), "entries outside the rows were written"
    # in place: the gradient overwrites the rows, and only the rows
    zin = buf.clone()
    zz = zin[off:off + T * ld].view(T, ld)[:, :V]
    res2 = P.decoupled_ppo_loss_fwd_bwd(zz, ids, lp_mu, lp_ref, adv, mask, dlogits=zz,
                                        scale_mode="const")
    torch.cuda.synchronize()
    assert torch.equal(zz.view(torch.int16), d.view(torch.int16)), "in place differs"
    assert torch.equal(zin[out].view(torch.int16), buf[out].view(torch.int16))
    assert torch.equal(res2.logp.view(torch.int32), res.logp.view(torch.int32))


@pytest.mark.parametrize("T,V,extra,off", CASES[:8], ids=[f"T{c[0]}_V{c[1]}_x{c[2]}_o{c[3]}" for c in CASES[:8]])
def test_phase_rows_forward_only(T, V, extra, off):
    ld = V + extra
    _say("phase rows forward", T, V, ld, off)
    buf, z, ids, mask, lp_mu, lp_ref, adv = _inputs(T, V, ld, off, seed=3 * V + off)
    lp = P.logprob_fwd(z, ids.clamp(0, V - 1))
    params = oracle_params((0.5, 2.0), (0.2, 0.2), "mask_weight", "const", 1.0)
    res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, want_dlogits=False,
                                       scale_mode="const")
    torch.cuda.synchronize()
    ref_lp, _ = oracle.logprob_fwd(oracle.bf16_bits_to_f64(
        z.cpu().view(torch.int16).numpy().view(np.uint16)), ids.clamp(0, V - 1).cpu().numpy())
    got = lp.cpu().double().numpy()
    assert np.all(np.abs(got - ref_lp) <= 2e-5 * np.maximum(np.abs(ref_lp), 1.0))
    ref = run_oracle(z, ids, lp_mu, lp_ref, adv, mask, None, params, want_dlogits=False)
    compare_loss(res, ref, params, torch.bfloat16, check_dlogits=False)


F32_CASES = [(300, 1003, 1), (200, 5003, 1), (120, 32001, 3), (40, 77821, 3)]


@pytest.mark.parametrize("T,V,extra", F32_CASES, ids=[f"T{c[0]}_V{c[1]}_x{c[2]}" for c in F32_CASES])
def test_fp32_ragged_rows_on_an_aligned_stride(T, V, extra):
    """fp32 rows whose length is not a multiple of 4 on a 16-byte stride: the resident kernel
    with its last entries loaded and stored one by one; the stride's padding is left alone."""
    ld = V + extra
    assert ld % 4 == 0
    _say("fp32 ragged rows", T, V, ld)
    assert P.row_kernel_name(torch.float32, V, ld).startswith("dppo::rows_f32_resident")
    g = torch.Generator(device=DEV).manual_seed(V)
    buf = torch.randn(T * ld, generator=g, device=DEV) * 3
    z = buf.view(T, ld)[:, :V]
    ids = torch.randint(0, V, (T,), generator=g, device=DEV)
    ids[0] = V - 1
    ids[2] = V - 2
    ids[5] = -1
    mask = torch.ones(T, dtype=torch.uint8, device=DEV)
    mask[3::7] = 0
    anchor = oracle_anchor(z, ids.clamp(0, V - 1)).to(DEV)
    lp_ref = (anchor + 0.2 * torch.randn(T, generator=g, device=DEV, dtype=torch.float64)).float()
    lp_mu = (lp_ref.double() + 0.1 * torch.randn(T, generator=g, device=DEV,
                                                 dtype=torch.float64)).float()
    adv = torch.randn(T, generator=g, device=DEV)
    dbuf = torch.full_like(buf, SENTINEL)
    d = dbuf.view(T, ld)[:, :V]
    params = oracle_params((0.5, 2.0), (0.2, 0.2), "mask_weight", "const", 1.0)
    res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d,
                                       scale_mode="const")
    lp = P.logprob_fwd(z, ids.clamp(0, V - 1))
    torch.cuda.synchronize()
    ref = run_oracle(z, ids, lp_mu, lp_ref, adv, mask, None, params)
    compare_loss(res, ref, params, torch.float32)
    assert torch.all(dbuf.view(T, ld)[:, V:] == SENTINEL)
    ref_lp, _ = oracle.logprob_fwd(z.cpu().double().numpy(), ids.clamp(0, V - 1).cpu().numpy())
    assert np.all(np.abs(lp.cpu().double().numpy() - ref_lp) <= 1e-5 * np.maximum(np.abs(ref_lp), 1.0))
    # in place
    zz = buf.clone().view(T, ld)
    P.decoupled_ppo_loss_fwd_bwd(zz[:, :V], ids, lp_mu, lp_ref, adv, mask, dlogits=zz[:, :V],
                                 scale_mode="const")
    torch.cuda.synchronize()
    assert torch.equal(zz[:, :V], d) and torch.equal(zz[:, V:], buf.view(T, ld)[:, V:])


def test_phase_rows_with_a_mismatched_gradient_layout_take_the_streaming_path():
    """dlogits at another offset within 16 bytes than the logits: the phase kernels cannot
    serve it, the streaming kernel does, with the same results."""
    T, V, ld, off = 50, 1003, 1003, 1
    buf, z, ids, mask, lp_mu, lp_ref, adv = _inputs(T, V, ld, off, seed=99)
    dbuf = torch.full((off + 1 + T * ld + 16,), SENTINEL, dtype=torch.bfloat16, device=DEV)
    d = dbuf[off + 1:off + 1 + T * ld].view(T, ld)[:, :V]
    params = oracle_params((0.5, 2.0), (0.2, 0.2), "mask_weight", "const", 1.0)
    res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d,
                                       scale_mode="const")
    torch.cuda.synchronize()
    ref = run_oracle(z, ids, lp_mu, lp_ref, adv, mask, None, params)
    compare_loss(res, ref, params, torch.bfloat16)
    out = _outside(dbuf, off + 1, T, ld, V)
    assert torch.all(dbuf[out] == SENTINEL)


def _random_cases(n=36, seed=2605):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        dtype = "bf16" if rng.random() < 0.7 else "f32"
        V = int(rng.choice([int(rng.integers(1, 64)), int(rng.integers(64, 4096)),
                            int(rng.integers(4096, 40000)), int(rng.integers(40000, 160000))]))
        extra = int(rng.choice([0, 0, int(rng.integers(1, 9)), 8 - V % 8]))
        off = int(rng.choice([0, 0, int(rng.integers(1, 8))]))
        T = int(max(2, min(400, 3_000_000 // max(V, 1))))
        out.append((i, dtype, T, V, extra, off, bool(rng.random() < 0.3), bool(rng.random() < 0.25)))
    return out


@pytest.mark.parametrize("i,dtype,T,V,extra,off,in_place,fwd_only", _random_cases(),
                         ids=[f"{c[0]}_{c[1]}_T{c[2]}_V{c[3]}_x{c[4]}_o{c[5]}" for c in _random_cases()])
def test_random_layouts_against_the_oracle(i, dtype, T, V, extra, off, in_place, fwd_only):
    """Seeded random layouts (dtype, V, stride, offset of the first row, T), with masked rows,
    bad ids, in place or into a second buffer, with or without dlogits: every output against
    the oracle, and no entry outside the rows written."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ld = V + extra
    _say("random layout", i, dtype, T, V, ld, off, in_place, fwd_only)
    g = torch.Generator(device=DEV).manual_seed(1000 + i)
    n = off + T * ld + 16
    buf = (torch.randn(n, generator=g, device=DEV) * 3).to(tdt)
    ref_buf = buf.clone()
    z = buf[off:off + T * ld].view(T, ld)[:, :V]
    ids = torch.randint(0, V, (T,), generator=g, device=DEV)
    ids[torch.rand(T, generator=g, device=DEV) < 0.05] = V
    mask = (torch.rand(T, generator=g, device=DEV) >= 0.15).to(torch.uint8)
    anchor = oracle_anchor(z, ids.clamp(0, V - 1)).to(DEV)
    lp_ref = (anchor + 0.2 * torch.randn(T, generator=g, device=DEV, dtype=torch.float64)).float()
    lp_mu = (lp_ref.double() + 0.1 * torch.randn(T, generator=g, device=DEV,
                                                 dtype=torch.float64)).float()
    adv = torch.randn(T, generator=g, device=DEV)
    params = oracle_params((0.5, 2.0), (0.2, 0.2), "mask_weight", "const", 1.0)
    ref = run_oracle(z, ids, lp_mu, lp_ref, adv, mask, None, params, want_dlogits=not fwd_only)
    out = _outside(buf, off, T, ld, V)
    if fwd_only:
        res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, want_dlogits=False,
                                           scale_mode="const")
        torch.cuda.synchronize()
        compare_loss(res, ref, params, tdt, check_dlogits=False)
        assert torch.equal(buf.view(torch.int16) if dtype == "bf16" else buf, ref_buf.view(torch.int16) if dtype == "bf16" else ref_buf)
        return
    if in_place:
        res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=z,
                                           scale_mode="const")
        torch.cuda.synchronize()
        compare_loss(res, ref, params, tdt)
        a, b = buf[out], ref_buf[out]
    else:
        dbuf = torch.full_like(buf, SENTINEL)
        d = dbuf[off:off + T * ld].view(T, ld)[:, :V]
        res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d,
                                           scale_mode="const")
        torch.cuda.synchronize()
        compare_loss(res, ref, params, tdt)
        a, b = dbuf[out], torch.full_like(dbuf[out], SENTINEL)
    if dtype == "bf16":
        a, b = a.view(torch.int16), b.view(torch.int16)
    assert torch.equal(a, b), "entries outside the rows were written"


ANY_CASES = [  # dtype, T, V, extra columns per row, element offset of row 0
    ("f32", 40, 1, 0, 1), ("f32", 40, 2, 0, 3), ("f32", 40, 3, 3, 2), ("f32", 60, 7, 0, 0),
    ("f32", 300, 1003, 0, 0), ("f32", 300, 1003, 2, 1), ("f32", 1200, 4101, 1, 3),
    ("f32", 64, 50257, 0, 0), ("f32", 24, 77818, 0, 2), ("f32", 12, 77823, 0, 1),
    ("f32", 600, 77829, 0, 1), ("f32", 20, 151937, 0, 3),
    ("bf16", 12, 155653, 0, 1), ("bf16", 520, 155661, 0, 0), ("bf16", 12, 262143, 4, 3),
]


@pytest.mark.parametrize("dtype,T,V,extra,off", ANY_CASES,
                         ids=[f"{c[0]}_T{c[1]}_V{c[2]}_x{c[3]}_o{c[4]}" for c in ANY_CASES])
def test_rows_that_start_anywhere(dtype, T, V, extra, off):
    """fp32 rows at any offset (shorter than a chunk, the resident shapes' limits, the prefix
    kernel's and the gap between them, which streams) and bf16 rows longer than the resident
    kernels: sampled ids at the first and last entries, in the whole chunks and in the entries
    before and after them, masked rows, a bad id, -inf at the row ends, a NaN row; the loss
    with dlogits (entries outside the rows untouched), in place, without dlogits, and the
    log-prob call: the same log-probs bit for bit where one kernel family serves them all (rows
    that the resident kernels hold)."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    E = 4 if dtype == "f32" else 8
    ld = V + extra
    _say("rows anywhere", dtype, T, V, ld, off)
    g = torch.Generator(device=DEV).manual_seed(V + off)
    n = off + T * ld + 16
    buf = (torch.randn(n, generator=g, device=DEV) * 3).to(dt)
    z = buf[off:off + T * ld].view(T, ld)[:, :V]
    if V > 3 * E:
        z[8, 0] = -float("inf")
        z[8, V - 1] = -float("inf")
    ids = torch.randint(0, V, (T,), generator=g, device=DEV)
    ids[0], ids[1], ids[5] = V - 1, 0, V + 3
    for i in range(min(12, V)):
        ids[10 + 2 * i % (T - 10)] = i               # every entry of the first chunks
        ids[11 + 2 * i % (T - 11)] = V - 1 - i
    mask = torch.ones(T, dtype=torch.uint8, device=DEV)
    mask[3::7] = 0
    anchor = oracle_anchor(z, ids.clamp(0, V - 1)).to(DEV)
    lp_ref = (anchor + 0.2 * torch.randn(T, generator=g, device=DEV, dtype=torch.float64)).float()
    lp_ref = lp_ref.nan_to_num(-7.0, neginf=-7.0)
    lp_mu = (lp_ref.double() + 0.1 * torch.randn(T, generator=g, device=DEV, dtype=torch.float64)).float()
    adv = torch.randn(T, generator=g, device=DEV)
    dbuf = torch.full_like(buf, SENTINEL)
    d = dbuf[off:off + T * ld].view(T, ld)[:, :V]
    params = oracle_params((0.5, 2.0), (0.2, 0.2), "mask_weight", "const", 1.0)
    kw = dict(scale_mode="const")
    res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d, **kw)
    fwd = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, want_dlogits=False, **kw)
    lp = P.logprob_fwd(z, ids.clamp(0, V - 1))
    torch.cuda.synchronize()
    ref = run_oracle(z, ids, lp_mu, lp_ref, adv, mask, None, params)
    compare_loss(res, ref, params, dt)
    compare_loss(fwd, ref, params, dt, check_dlogits=False)
    good = ((mask != 0) & (ids < V) & torch.isfinite(res.logp)).cpu().numpy()
    got, want = lp.cpu().double().numpy()[good], ref["lp"][good]
    assert np.all(np.abs(got - want) <= 2e-5 * np.maximum(np.abs(want), 1.0))
    aligned = off % E == 0 and ld % E == 0
    if (V if aligned else V + E - 1) <= 1024 * 19 * E:   # by the chunks a row may touch
        rows = (mask != 0) & (ids < V)
        for other in (fwd.logp, lp):
            assert torch.equal(res.logp[rows].view(torch.int32), other[rows].view(torch.int32))
    out = _outside(dbuf, off, T, ld, V)
    assert torch.all(dbuf[out] == SENTINEL), "entries outside the rows were written"
    zin = buf.clone()
    zz = zin[off:off + T * ld].view(T, ld)[:, :V]
    P.decoupled_ppo_loss_fwd_bwd(zz, ids, lp_mu, lp_ref, adv, mask, dlogits=zz, **kw)
    torch.cuda.synchronize()
    it = torch.int32 if dt == torch.float32 else torch.int16
    assert torch.equal(zz.contiguous().view(it), d.contiguous().view(it)), "in place differs"
    assert torch.equal(zin[out].view(it), buf[out].view(it))
    # dlogits at another offset within 16 bytes: the streaming kernel, one entry at a time
    if off == 0 and V < 60000:
        dbuf = torch.full_like(buf, SENTINEL)
        d2 = dbuf[1:1 + T * ld].view(T, ld)[:, :V]
        res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d2, **kw)
        torch.cuda.synchronize()
        compare_loss(res, ref, params, dt)
        assert torch.all(dbuf[_outside(dbuf, 1, T, ld, V)] == SENTINEL)
    # a NaN in an entry at an end reaches the whole row
    z[9] = float("nan") if V == 1 else z[9]
    z[9, V - 1] = float("nan")
    ids[9], mask[9] = 0, 1
    res = P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, dlogits=d, **kw)
    torch.cuda.synchronize()
    assert torch.isnan(res.logp[9]) and torch.isnan(d[9]).all()


SHORT_CASES = [  # dtype, T, V, extra columns per row, element offset of row 0
    ("bf16", 41, 2, 0, 5), ("bf16", 42, 8, 0, 0), ("bf16", 43, 511, 0, 1), ("bf16", 41, 512, 8, 0),
    ("bf16", 90, 513, 1, 7), ("bf16", 37, 2041, 0, 7), ("bf16", 64, 2048, 0, 0), ("bf16", 33, 2049, 0, 0),
    ("bf16", 30, 4089, 7, 7), ("bf16", 31, 4096, 0, 0), ("bf16", 30, 4097, 0, 3), ("bf16", 29, 8185, 0, 7),
    ("bf16", 30, 8193, 0, 0), ("bf16", 29, 12281, 0, 7), ("bf16", 30, 12288, 0, 0),
    ("bf16", 5000, 600, 0, 3),
    ("f32", 43, 255, 0, 1), ("f32", 41, 256, 0, 0), ("f32", 42, 1021, 0, 3), ("f32", 41, 1024, 4, 0),
    ("f32", 33, 1025, 0, 0), ("f32", 30, 2045, 0, 3), ("f32", 31, 2048, 0, 0), ("f32", 29, 4093, 0, 3),
    ("f32", 30, 4096, 0, 0), ("f32", 29, 6141, 0, 3), ("f32", 30, 6144, 0, 0), ("f32", 5000, 300, 0, 1),
]


@pytest.mark.parametrize("dtype,T,V,extra,off", SHORT_CASES,
                         ids=[f"{c[0]}_T{c[1]}_V{c[2]}_x{c[3]}_o{c[4]}" for c in SHORT_CASES])
def test_short_rows_one_wave_each(dtype, T, V, extra, off):
    """Rows that one wave works on: the ends of each capacity, of a wave's 64 chunks, and
    batches that leave waves of the last workgroup without a row."""
    name = P.row_kernel_name(torch.float32 if dtype == "f32" else torch.bfloat16, V, V + extra)
    assert "<256, " in name, name
    test_rows_that_start_anywhere(dtype, T, V, extra, off)


@pytest.mark.parametrize("dtype,T,V,grads", [("bf16", 1027, 700, True), ("bf16", 1027, 9001, False),
                                             ("bf16", 515, 160001, True), ("f32", 1027, 700, True),
                                             ("f32", 515, 30001, True), ("f32", 515, 90001, False),
                                             # batches long enough that the counters come from
                                             # atomics: past 65536 tokens, forward past 16384
                                             ("bf16", 65601, 12296, True), ("bf16", 65601, 12297, True),
                                             ("f32", 65601, 6150, True), ("bf16", 16384, 12296, False),
                                             ("bf16", 16385, 12296, False)])
def test_counters_from_flags_and_from_atomics(dtype, T, V, grads):
    """The counters and the loss are the same whether loss_sum derives them from the flags or the
    kernels add them (no flags written, or the atomics policy)."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(V)
    z = (torch.randn(T, V, generator=g, device=DEV) * 3).to(dt)
    ids = torch.randint(0, V, (T,), generator=g, device=DEV)
    ids[7] = -1
    mask = (torch.rand(T, generator=g, device=DEV) > 0.3).to(torch.uint8)
    mask[7] = 1
    lp = P.logprob_fwd(z, ids.clamp(0, V - 1))
    lp_ref = lp + 0.3 * torch.randn(T, generator=g, device=DEV)
    lp_mu = lp_ref + 0.6 * torch.randn(T, generator=g, device=DEV)
    adv = torch.randn(T, generator=g, device=DEV)
    for rd_mode in ("mask_weight", "weight"):
        def call(**kw):
            return P.decoupled_ppo_loss_fwd_bwd(z, ids, lp_mu, lp_ref, adv, mask, rd_mode=rd_mode,
                                                want_dlogits=grads, **kw)
        a, b = call(), call(want_flags=False)
        P.set_path_policy("auto+atomics")
        try:
            c = call()
        finally:
            P.set_path_policy("auto")
        torch.cuda.synchronize()
        f = a.flags.to(torch.int32)
        band, ppo = (f & P.FLAG_BAND) != 0, (f & P.FLAG_PPO) != 0
        act = ppo & band if rd_mode == "mask_weight" else ppo
        want = [int(mask.sum()), int(band.sum()), int(ppo.sum()), int(act.sum()), 1]
        for r in (a, b, c):
            assert r.stats.tolist() == want
            assert torch.equal(r.loss.view(torch.int32), a.loss.view(torch.int32))


@pytest.mark.parametrize("V,off", [(155661, 0), (155663, 5), (196625, 3), (262143, 1)])
def test_long_unaligned_rows_keep_small_probabilities(V, off):
    """bf16 rows that start anywhere and are longer than the resident kernels hold: their gradient
    is formed in fp32 from the logits, so an entry far below its neighbours keeps its value and
    every entry is rounded once, to bf16 (2^-8). Beside it the fp32 log-sum-exp and exponents of up
    to 80 (2e-5). Each length has entries in the resident part and, past it, in the tail."""
    T = 3
    assert "rows_bf16_prefix_phase" in P.row_kernel_name(torch.bfloat16, V, V)
    _say("long rows, small probabilities", V, off)
    g = torch.Generator(device=DEV).manual_seed(V)
    buf = torch.zeros(off + T * V + 16, dtype=torch.bfloat16, device=DEV)
    z = buf[off:off + T * V].view(T, V)
    z.copy_(torch.randn(T, V, generator=g, device=DEV) - 30)
    z[:, 3::13] += 40
    ids = torch.tensor([3, 16, V - 1], device=DEV)
    p = torch.softmax(z.double(), dim=1)
    lp = p.gather(1, ids[:, None])[:, 0].log().float()
    adv = torch.ones(T, device=DEV)
    d = torch.empty_like(buf)[off:off + T * V].view(T, V)
    P.decoupled_ppo_loss_fwd_bwd(z, ids, lp, lp, adv, dlogits=d, scale_mode="const")
    torch.cuda.synchronize()
    rel = ((d.double() - p) / p).scatter(1, ids[:, None], 0.0).abs().max()
    assert rel <= 2.0 ** -8 + 2e-5, float(rel)
