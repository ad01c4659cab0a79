"""GPU parity: specee_verify (arg-max of the full head + membership) against the oracle."""
import numpy as np
import pytest
import torch

from paper_2504_08850_amd import synth

from parity import close, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    from paper_2504_08850_amd import specee
    specee.lib()
    return specee


def run_verify(sp, h, g, W_d, ids, gate=None):
    out = sp.verify(dev(h), dev(g), W_d, dev(ids), gate=None if gate is None else dev(gate))
    torch.cuda.synchronize()
    return {k: host(v) for k, v in out.items()}


def check_verify(got, full, ids, what):
    """full: oracle logits [N][V].  The arg-max is unique only if the runner-up is not within tolerance."""
    N = full.shape[0]
    top = np.argsort(-full, axis=1)[:, :2]
    for n in range(N):
        best, second = full[n, top[n, 0]], full[n, top[n, 1]] if full.shape[1] > 1 else -np.inf
        close([got["max_logit"][n]], [best], 1.0, what + " max logit")
        if best - second > 4e-3 * max(1.0, abs(best)):
            assert got["token"][n] == top[n, 0], f"{what}: token of state {n}"
            assert got["hit"][n] == int(top[n, 0] in ids[n]), f"{what}: hit of state {n}"
        else:
            assert got["token"][n] in top[n], what
        assert got["hit"][n] == int(got["token"][n] in ids[n])


@pytest.mark.parametrize("d,V,N,K", [(64, 37, 1, 3), (1032, 1001, 2, 4), (4096, 515, 5, 4), (520, 4100, 64, 8),
                                     (2048, 300, 70, 2), (8, 1, 1, 1), (16384, 100, 2, 4)])
def test_verify_small(sp, oracle, d, V, N, K):
    rng = np.random.default_rng(d + V + N)
    h = rng.standard_normal((N, d)).astype(np.float16)
    g = (1 + 0.05 * rng.standard_normal(d)).astype(np.float16)
    W = (0.05 * rng.standard_normal((V, d))).astype(np.float16)
    full = oracle.lm_head_gemv(h, g, W)
    ids = rng.integers(0, V, size=(N, K)).astype(np.int32)
    ids[::2, 0] = full.argmax(axis=1)[::2]          # half of the states hit
    got = run_verify(sp, h, g, dev(W), ids)
    check_verify(got, full, ids, f"verify d={d} V={V} N={N}")
    ref = oracle.verify(h, g, W, ids)
    assert got["hit"].sum() > 0 or N == 1
    assert np.array_equal(ref["token"], full.argmax(axis=1))


def test_verify_tie_goes_to_lowest_id(sp):
    rng = np.random.default_rng(5)
    for N in (1, 4):
        h = rng.standard_normal((N, 256)).astype(np.float16)
        g = np.ones(256, np.float16)
        W = (0.01 * rng.standard_normal((700, 256))).astype(np.float16)
        boost = (0.5 * np.sign(h[0].astype(np.float32))).astype(np.float16)
        W[611] = boost
        W[87] = boost                                # identical rows: identical logits for state 0
        ids = np.tile(np.array([[611, 3]], np.int32), (N, 1))
        got = run_verify(sp, h, g, dev(W), ids)
        assert got["token"][0] == 87 and got["hit"][0] == 0


def test_verify_llama7b_and_agreement_with_lm_head(sp, oracle):
    c = synth.CONFIGS["C1"]
    lm_h = synth.lm_head(c.V, c.d, synth.lm_seed(c))
    lm_d = dev(lm_h)
    t = synth.make("C1", seed=2, lm=lm_h)
    oracle.set_threads(8)
    full = oracle.lm_head_gemv(t["hidden"], t["gamma"], lm_h)
    oracle.set_threads(1)
    ids = t["ids"].copy()
    got = run_verify(sp, t["hidden"], t["gamma"], lm_d, ids)
    check_verify(got, full, ids, "verify 32000x4096 miss")
    ids[0, 3] = full.argmax()
    got = run_verify(sp, t["hidden"], t["gamma"], lm_d, ids)
    check_verify(got, full, ids, "verify 32000x4096 hit")
    assert got["hit"][0] == 1
    # 16 states through the matrix-core path agree with the stored-logits path
    hid = synth.hidden(16, c.d, 77)
    gpu_full = host(sp.lm_head_gemv(dev(hid), dev(t["gamma"]), lm_d))
    ids16 = np.tile(ids, (16, 1))
    got = run_verify(sp, hid, t["gamma"], lm_d, ids16)
    assert np.array_equal(got["token"], gpu_full.argmax(axis=1))
    np.testing.assert_array_equal(got["max_logit"], gpu_full.max(axis=1))


@pytest.mark.parametrize("d,V,N,K,pattern", [(256, 700, 1, 4, "none"), (256, 700, 1, 4, "all"),
                                             (1032, 1001, 2, 4, "alternate"), (520, 4100, 5, 4, "alternate"),
                                             (520, 4100, 70, 8, "blocks"), (520, 4100, 70, 8, "none"),
                                             (520, 4100, 40, 2, "random")])
def test_verify_gated(sp, oracle, d, V, N, K, pattern):
    """Verification follows a positive prediction only (Sec. 4.3.3): states whose gate is 0 are skipped on
    the device and report token -1, max_logit 0, hit 0; the others match the ungated result."""
    rng = np.random.default_rng(d + V + N + len(pattern))
    h = rng.standard_normal((N, d)).astype(np.float16)
    g = (1 + 0.05 * rng.standard_normal(d)).astype(np.float16)
    W = (0.05 * rng.standard_normal((V, d))).astype(np.float16)
    full = oracle.lm_head_gemv(h, g, W)
    ids = rng.integers(0, V, size=(N, K)).astype(np.int32)
    ids[:, 0] = full.argmax(axis=1)
    gate = {"none": np.zeros(N, np.int32), "all": np.ones(N, np.int32),
            "alternate": (np.arange(N) % 2).astype(np.int32),
            "blocks": ((np.arange(N) // 16) % 2 * 7).astype(np.int32),     # whole 16-state blocks off, any non-zero = on
            "random": rng.integers(0, 2, N).astype(np.int32)}[pattern]
    W_d = dev(W)
    # poison the outputs first so that skipped states are seen to be written
    out = {"token": torch.full((N,), 123, dtype=torch.int32, device="cuda"),
           "max_logit": torch.full((N,), 9.0, dtype=torch.float32, device="cuda"),
           "hit": torch.full((N,), 5, dtype=torch.int32, device="cuda")}
    sp.verify(dev(h), dev(g), W_d, dev(ids), gate=dev(gate), out=out)
    torch.cuda.synchronize()
    got = {k: host(v) for k, v in out.items()}
    on = gate != 0
    assert np.all(got["token"][~on] == -1) and np.all(got["hit"][~on] == 0) and np.all(got["max_logit"][~on] == 0)
    if on.any():
        sub = {k: v[on] for k, v in got.items()}
        check_verify(sub, full[on], ids[on], f"gated verify {pattern} N={N}")
        ungated = run_verify(sp, h, g, W_d, ids)
        for k in got:
            assert np.array_equal(got[k][on], ungated[k][on]), k


def test_predict_then_gated_verify(sp, oracle):
    """The predictor's exit flags feed the verification without leaving the device."""
    c = synth.CONFIGS["T1"]
    t = synth.make("T1", seed=11, bias=True)
    lm_h = t["lm_head"]
    for threshold in (0.3, 0.5, 0.7):      # different mixes of exits
        ref = oracle.predict(t["hidden"], t["gamma"], lm_h, t["ids"], t["prev_probs"], t["W1"], t["w2"], t["b1"],
                             t["b2"], eps=c.eps, threshold=threshold)
        lm_d, hid_d, g_d, ids_d = dev(lm_h), dev(t["hidden"]), dev(t["gamma"]), dev(t["ids"])
        res = sp.predict(hid_d, g_d, lm_d, ids_d, dev(t["prev_probs"]), dev(t["W1"]), dev(t["w2"]), dev(t["b1"]),
                         dev(t["b2"]), eps=c.eps, threshold=threshold)
        out = sp.verify(hid_d, g_d, lm_d, ids_d, gate=res["exit"], eps=c.eps)
        torch.cuda.synchronize()
        flags = host(res["exit"])
        sure = np.abs(ref["scores"] - threshold) > 1e-4
        assert np.array_equal(flags[sure], ref["exit"][sure])
        vref = oracle.verify(t["hidden"], t["gamma"], lm_h, t["ids"], eps=c.eps)
        full = oracle.lm_head_gemv(t["hidden"], t["gamma"], lm_h, eps=c.eps)
        tok, hit = host(out["token"]), host(out["hit"])
        for n in range(c.B):
            if flags[n]:
                assert hit[n] == int(tok[n] in t["ids"][n])
                if tok[n] != vref["token"][n]:      # only a near-tie may differ
                    assert abs(full[n, tok[n]] - full[n].max()) <= 4e-3 * max(1.0, abs(full[n].max()))
            else:
                assert tok[n] == -1 and hit[n] == 0


@pytest.mark.parametrize("N", [3, 15, 16, 17, 31, 32, 33])
def test_multi_state_head_and_verify_by_tiles_of_states(sp, oracle, N):
    """One, two and four tiles of 16 states per workgroup, each with its last state and one more.  The bound is that of
    fp32 sums of exact products (x = hi + lo in halves): a term passes at most 32 additions of a matrix instruction, two
    accumulations per 32 columns and a few combining steps, each off by 2^-24 of what it has summed, and a lo below the
    normal halves is off by 2^-25.  Without the lo halves every N exceeds it four times over."""
    rng = np.random.default_rng(N)
    d, V, K = 1032, 261, 4
    h = rng.standard_normal((N, d)).astype(np.float16)
    g = (1 + 0.05 * rng.standard_normal(d)).astype(np.float16)
    w = (0.05 * rng.standard_normal((V, d))).astype(np.float16)
    ref = oracle.lm_head_gemv(h, g, w)
    got = sp.lm_head_gemv(dev(h), dev(g), dev(w)).cpu().numpy()
    x, w64 = np.abs(h.astype(np.float64) * g.astype(np.float64)), np.abs(w.astype(np.float64))
    r = 1.0 / np.sqrt((h.astype(np.float64) ** 2).mean(axis=1, keepdims=True) + 1e-5)
    bound = r * ((32 + 2 * ((d + 31) // 32) + 16) * 2.0 ** -24 * (x @ w64.T) + 2.0 ** -25 * w64.sum(axis=1))
    assert np.all(np.abs(got - ref) <= bound)
    ids = np.stack([rng.choice(V, K, replace=False) for _ in range(N)]).astype(np.int32)
    out = sp.verify(dev(h), dev(g), dev(w), dev(ids))
    torch.cuda.synchronize()
    # the same sums decide: the arg-max of the logits this library returns, bit for bit
    tok = out["token"].cpu().numpy()
    assert np.array_equal(tok, got.argmax(axis=1))
    assert np.array_equal(out["max_logit"].cpu().numpy(), got[np.arange(N), tok])


def head_rows(rng, V, d, group):
    """A head: what the library takes, and the same in float64 as weights and as bounds of what is summed for one."""
    if not group:
        w = (0.05 * rng.standard_normal((V, d))).astype(np.float16)
        return (dev(w),), w.astype(np.float64), np.abs(w.astype(np.float64))
    codes = rng.integers(0, 16, (V, d), dtype=np.uint32)
    q = (codes.reshape(V, d // 8, 8) << (4 * np.arange(8, dtype=np.uint32))).sum(axis=2, dtype=np.uint32)
    s = rng.uniform(0.004, 0.02, (V, d // group)).astype(np.float16)
    z = rng.uniform(5, 10, (V, d // group)).astype(np.float16)
    s64, z64 = (np.repeat(a.astype(np.float64), group, axis=1) for a in (s, z))
    return (dev(q.view(np.int32)), dev(s), dev(z), group), s64 * (codes - z64), s64 * (codes + z64)


@pytest.mark.parametrize("d,V,N,group,hscale", [
    (8, 1, 3, 0, 1.0), (72, 17, 16, 0, 1.0), (512, 16, 15, 0, 1.0), (520, 33, 17, 0, 1.0),  # rows end in a wavefront
    (576, 33, 17, 0, 1.0), (4608, 515, 16, 0, 1.0),                                         # the same, rows of whole lines
    (1032, 6007, 2, 0, 1.0), (2048, 4099, 64, 0, 1.0), (4096, 4111, 16, 0, 1.0),            # several tiles, passes of states
    (4104, 47, 15, 0, 1.0), (8192, 515, 16, 0, 1.0), (16384, 40, 3, 0, 1.0),                # two, two and four passes over rows
    (1024, 129, 8, 0, 2.0 ** -13), (1024, 129, 8, 0, 16000.0),
    (64, 2003, 15, 64, 1.0), (192, 1700, 16, 64, 1.0), (128, 8003, 2, 128, 1.0),
    (2048, 1603, 15, 64, 1.0), (3072, 1009, 16, 128, 1.0), (4096, 1103, 17, 128, 1.0),
    (4224, 1003, 16, 128, 1.0), (4608, 1601, 16, 64, 1.0), (5120, 1001, 16, 128, 1.0),
    (8192, 1503, 16, 64, 1.0), (16384, 1001, 16, 128, 1.0),
    (2048, 1603, 16, 128, 2.0 ** -13), (4608, 1603, 16, 64, 16000.0),
])
def test_head_of_several_states_by_shares_of_the_row(sp, d, V, N, group, hscale):
    """fp32 sums of exact products: a term passes at most 512 additions in a wavefront's share of the row (32 per matrix
    instruction, 16 of them), 16 shares, four passes and a handful of folds and factors, each off by 2^-24 of what it has
    summed.  x is scaled by its share's largest element to between 2^14 and 2^15 before it is cut into two halves, so that
    what lies below the normal halves is off by 2^-25 of that, at most 2^-39 of the largest."""
    rng = np.random.default_rng(d + V + N)
    h = (rng.standard_normal((N, d)).clip(-4, 4) * hscale).astype(np.float16)
    g = (1 + 0.05 * rng.standard_normal(d)).astype(np.float16)
    head, w, absw = head_rows(rng, V, d, group)
    logits, verify = (sp.lm_head_gemv_q4, sp.verify_q4) if group else (sp.lm_head_gemv, sp.verify)
    h64, g64 = h.astype(np.float64), g.astype(np.float64)
    r = 1.0 / np.sqrt((h64 ** 2).mean(axis=1, keepdims=True) + 1e-5)
    ref = r * ((h64 * g64) @ w.T)
    x = np.abs(h64 * g64)
    bound = r * ((512 + 16 + 4 + 16) * 2.0 ** -24 * (x @ absw.T) + 2.0 ** -39 * x.max(axis=1, keepdims=True) * absw.sum(axis=1))
    got = host(logits(dev(h), dev(g), *head, out=torch.full((N, V), float("nan"), device="cuda")))
    assert np.all(np.abs(got - ref) <= bound)
    ids = np.stack([rng.choice(V, min(V, 3), replace=False) for _ in range(N)]).astype(np.int32)
    v = {k: host(a) for k, a in verify(dev(h), dev(g), *head, dev(ids)).items()}
    # the same sums decide, and the lowest of equal rows wins
    assert np.array_equal(v["token"], got.argmax(axis=1)) and np.array_equal(v["max_logit"], got.max(axis=1))
    bad = h.copy()
    bad[0, d - 1], bad[N // 2, 0] = np.inf, np.nan
    b = host(logits(dev(bad), dev(g), *head))
    rest = np.setdiff1d(np.arange(N), [0, N // 2])
    assert np.isnan(b[[0, N // 2]]).all() and np.array_equal(b[rest], got[rest])


@pytest.mark.parametrize("d,V,N,group", [(72, 4000, 5, 0), (1024, 4001, 8, 0), (4096, 4111, 16, 0), (4104, 2003, 16, 0),
                                         (192, 4001, 16, 64), (2048, 1603, 16, 128), (3072, 1009, 16, 128),
                                         (4096, 1103, 16, 64), (4608, 1601, 16, 64), (8192, 1503, 16, 128)])
@pytest.mark.parametrize("large,gamma", [(30000.0, 2.0 ** -20), (1500.0, 2.0 ** -14), (30000.0, 0.0), (30000.0, 8.0),
                                         (2.0 ** -18, 1.0)])
def test_head_keeps_the_small_elements_beside_a_large_one(sp, d, V, N, group, large, gamma):
    """Hidden elements of very different size, the large ones where the RMSNorm weight is near zero: the small ones make the
    logits and must keep their 22 bits.  Also products that no half holds, and hidden states of subnormal halves.  548 additions, each off by at most 2^-24 of what it has
    summed and independent of the others, are off by sqrt(548 / 3) * 2^-24 = 8.1e-7 together; on codes scale * (sum of
    codes - zero * sum), whose parts have 2.5 times the root mean square of the difference."""
    rng = np.random.default_rng(d + V + N)
    h = rng.standard_normal((N, d)) * min(0.1, large)
    g = 1 + 0.05 * rng.standard_normal(d)
    if large > 1:
        h[:, [d // 7, d // 3]], g[[d // 7, d // 3]] = large, gamma
    h, g = h.astype(np.float16), g.astype(np.float16)
    head, w, _ = head_rows(rng, V, d, group)
    got = host((sp.lm_head_gemv_q4 if group else sp.lm_head_gemv)(dev(h), dev(g), *head, eps=0.0))
    h64 = h.astype(np.float64)
    ref = ((h64 * g.astype(np.float64)) @ w.T) / np.sqrt((h64 ** 2).mean(axis=1, keepdims=True))
    assert np.linalg.norm(got - ref) <= 8.1e-7 * (2.5 if group else 1.0) * np.linalg.norm(ref)


@pytest.mark.parametrize("d,V,N,group", [(4096, 6007, 16, 0), (1024, 300, 3, 0), (512, 20011, 5, 0), (4096, 8003, 16, 128),
                                         (512, 5003, 7, 64)])
def test_verify_of_several_states_on_as_many_workgroups_as_the_workspace_has_room_for(sp, d, V, N, group):
    """The queried workspace holds an arg-max candidate per tile of 16 rows or per CU, whichever is less (the kernels for
    other shapes leave one per 32 or 128 rows); what they leave is enough too, with the same outputs."""
    rng = np.random.default_rng(V)
    head, _, _ = head_rows(rng, V, d, group)
    verify, op = (sp.verify_q4, sp.OP_VERIFY_Q4) if group else (sp.verify, sp.OP_VERIFY)
    room = sp.workspace_bytes(op, sp.Dims(d, V, 2, 1, 1e-5, 0.5), N)
    assert room >= 2 * N * 4 * min(256, -(-V // 16))
    h, g = dev(rng.standard_normal((N, d)).astype(np.float16)), dev(np.ones(d, np.float16))
    ids = dev(rng.integers(0, V, (N, 2)).astype(np.int32))
    least = 2 * 256 * -(-N * 4 * -(-V // (32 if group else 128)) // 256)
    a, b = (verify(h, g, *head, ids, workspace=torch.full((n // 4,), 1e30, device="cuda")) for n in (room, least))
    assert all(torch.equal(a[k], b[k]) for k in ("token", "max_logit", "hit"))
    full = (sp.lm_head_gemv_q4 if group else sp.lm_head_gemv)(h, g, *head)
    assert torch.equal(a["token"].long(), full.argmax(dim=1)) and torch.equal(a["max_logit"], full.max(dim=1).values)


@pytest.mark.parametrize("d,large", [(2048, 0), (3072, 0), (4096, 0), (4608, 0), (5120, 0), (4096, 1500.0), (5120, 900.0)])
def test_fp16_head_of_several_states_sums_as_exactly_as_of_one(sp, d, large):
    """Both sum in 32 bits.  Of one state a lane adds d / 64 products in a row; of several, a chain of four matrix
    instructions makes 16 such additions at most, then four chains and the shares meet.  Errors against float64 as norms
    over 32000 logits each, a random quantity: a fifth more is allowed."""
    rng = np.random.default_rng(d)
    h, g = 0.3 * rng.standard_normal((4, d)) if large else rng.standard_normal((4, d)), 1 + 0.05 * rng.standard_normal(d)
    if large:
        h[:, [d // 7, d // 3]], g[[d // 7, d // 3]] = large, 0.02
    h, g = h.astype(np.float16), g.astype(np.float16)
    (w_d,), w, _ = head_rows(rng, 8000, d, 0)
    h64 = h.astype(np.float64)
    ref = ((h64 * g.astype(np.float64)) @ w.T) / np.sqrt((h64 ** 2).mean(axis=1, keepdims=True) + 1e-5)
    one = np.concatenate([host(sp.lm_head_gemv(dev(s[None]), dev(g), w_d)) for s in h])
    four = host(sp.lm_head_gemv(dev(h), dev(g), w_d))
    assert np.linalg.norm(four - ref) <= 1.2 * np.linalg.norm(one - ref)


def test_fp16_head_of_several_states_keeps_infinite_logits(sp):
    """A row with an infinite weight has an infinite logit, as in the sums for one state; both signs in it: NaN."""
    rng = np.random.default_rng(5)
    d, V = 1032, 300
    h = (1 + rng.random((4, d))).astype(np.float16)   # (x > 0 everywhere: the weight's sign is the logit's)
    w = (0.05 * rng.standard_normal((V, d))).astype(np.float16)
    w[17, 3], w[40, 1031], w[41, 600], w[41, 8] = np.inf, -np.inf, np.inf, -np.inf
    g = np.ones(d, np.float16)
    one = np.concatenate([host(sp.lm_head_gemv(dev(s[None]), dev(g), dev(w))) for s in h])
    four = host(sp.lm_head_gemv(dev(h), dev(g), dev(w)))
    for y in (one, four):
        assert (y[:, 17] == np.inf).all() and (y[:, 40] == -np.inf).all() and np.isnan(y[:, 41]).all()
        assert np.isfinite(np.delete(y, [17, 40, 41], axis=1)).all()
    assert (host(sp.verify(dev(h), dev(g), dev(w), dev(np.zeros((4, 1), np.int32)))["token"]) == 17).all()


def test_head_of_several_states_more_tiles_than_sums_wait_in_lds(sp):
    """Two passes over the rows and 33 tiles for the first workgroups: the sums of a row do not depend on the split."""
    d, V, N = 4104, 131100, 3
    gen = torch.Generator(device="cuda").manual_seed(1)
    h, g = torch.randn(N, d, generator=gen, device="cuda").half(), torch.ones(d, device="cuda").half()
    w = torch.randn(V, d, generator=gen, device="cuda", dtype=torch.float16)
    got = sp.lm_head_gemv(h, g, w)
    assert torch.equal(got[:, :1500], sp.lm_head_gemv(h, g, w[:1500].contiguous()))
    assert torch.equal(got[:, V - 1500:], sp.lm_head_gemv(h, g, w[V - 1500:].contiguous()))
    out = sp.verify(h, g, w, torch.zeros(N, 1, dtype=torch.int32, device="cuda"))
    assert torch.equal(out["token"].long(), got.argmax(dim=1)) and torch.equal(out["max_logit"], got.max(dim=1).values)


@pytest.mark.parametrize("d,V,N", [(8192, 12293, 17), (1024, 131200, 33), (16384, 6209, 64)])
def test_head_of_many_states_by_whole_lines(sp, d, V, N):
    """Rows of whole lines on heads above 192 MB, with 128 and 256 rows per workgroup and a last one that is not full.
    Sampled rows against float64: 2 * d additions (of hi and of lo), each off by at most 2^-24 of what it has summed and
    independent of the others, are off by sqrt(2 * d / 3) * 2^-24 together."""
    gen = torch.Generator(device="cuda").manual_seed(d)
    h, w = (torch.randn(n, d, generator=gen, device="cuda").half() for n in (N, V))
    g = (1 + 0.05 * torch.randn(d, generator=gen, device="cuda")).half()   # (x needs both halves)
    assert V * d * 2 > 192 << 20
    got = sp.lm_head_gemv(h, g, w)
    r = torch.rsqrt(h.double().pow(2).mean(1, keepdim=True) + 1e-5)
    for a, b in ((0, 300), (V // 2, V // 2 + 300), (V - 300, V)):
        ref = r * ((h.double() * g.double()) @ w[a:b].double().t().contiguous())
        assert (got[:, a:b] - ref).norm() <= (2 * d / 3) ** 0.5 * 2.0 ** -24 * ref.norm()
    v = sp.verify(h, g, w, torch.zeros(N, 1, dtype=torch.int32, device="cuda"))
    assert torch.equal(v["token"].long(), got.argmax(dim=1)) and torch.equal(v["max_logit"], got.max(dim=1).values)


@pytest.mark.parametrize("d,group", [(4096, 128), (4224, 128), (4608, 128), (4096, 64), (4160, 64), (4608, 64)])
def test_q4_head_of_several_states_with_and_without_the_hint(sp, d, group):
    """Codes above 72 MB are read with the non-temporal hint, the first and last rows of the same head without it."""
    V, n = 2 ** 28 // d + 33, 12001
    gen = torch.Generator(device="cuda").manual_seed(d)
    q = torch.randint(-2 ** 31, 2 ** 31 - 1, (V, d // 8), generator=gen, device="cuda", dtype=torch.int32)
    s, z = (torch.rand(V, d // group, generator=gen, device="cuda").half() for _ in range(2))
    h, g = torch.randn(2, d, generator=gen, device="cuda").half(), torch.ones(d, device="cuda").half()
    assert V * d // 2 > 72 << 20 > n * d // 2
    got = sp.lm_head_gemv_q4(h, g, q, s, 15 * z, group)
    for a, b in ((0, n), (V - n, V)):
        part = sp.lm_head_gemv_q4(h, g, q[a:b].contiguous(), s[a:b].contiguous(), 15 * z[a:b].contiguous(), group)
        assert torch.equal(got[:, a:b], part)
    v = sp.verify_q4(h, g, q, s, 15 * z, group, torch.zeros(2, 1, dtype=torch.int32, device="cuda"))
    assert torch.equal(v["token"].long(), got.argmax(dim=1)) and torch.equal(v["max_logit"], got.max(dim=1).values)
