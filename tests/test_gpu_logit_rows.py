"""Logits-given rows around the sizes where the serving kernel changes: a wave, 256, 512 or 1024
threads per row (80 logits per thread), beyond that pieces of a row or the long-row kernel; against the oracle, and against the
streaming kernel where rows hold masked or non-finite logits."""
import numpy as np
import pytest
import torch

from oracle import adwin_oracle as O
from paper_2605_28396_amd import synth
from tests import helpers as Hp
from tests.test_gpu_parity import B  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

DIAG = ("t_logp", "t_entropy", "t_rank")
BASE = ("kl", "c", "dz", "loss_prefix", "batch", "n_out", "n_adm_out", "status_dev")
SIZES = [8, 520, 5120, 5128, 20480, 20488, 40960, 40968, 81920, 81928]
LONG = [81928, 153600, 153608]


def _host(out):
    torch.cuda.synchronize()
    return {k: v.float().cpu().numpy() if v.dtype.is_floating_point else v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("V", SIZES)
def test_row_kernels_match_oracle(B, V):  # noqa: F811
    w = synth.Workload(f"rows_{V}", V, 0, 0, synth._offsets([3, 0, 1, 4]), np.array([2, 4, 1, 9], np.int32))
    p = synth.logits_problem(w)
    f = Hp.oracle_inputs(p)
    d = {k: v.cuda() for k, v in p.items()}
    rows = O.plan(w.offsets, w.window)["rows"]
    for est in (O.EST_EXPECTED, O.EST_SAMPLED):
        ref = O.supervise_from_logits(f["z_s"], f["z_t"], f["ids"], w.offsets, w.window, reduction=O.RED_SUM,
                                      grad_scale=-2.0, estimator=est)
        for want in (BASE, BASE + DIAG):
            got = _host(B.adwin_opd_from_logits(d["z_s"], d["z_t"], d["ids"], w.offsets, w.window,
                                                reduction=O.RED_SUM, grad_scale=-2.0, estimator=est, want=want))
            assert int(got["status_dev"][0]) == 0 and int(got["n_adm_out"][0]) == ref["n_adm"]
            Hp.assert_kl(got["kl"], ref["kl"])
            Hp.assert_cost(got["c"], ref["c"])
            Hp.assert_grad(got["dz"], ref["dz"], "dz", Hp.BF16_ULP, abs_cap=False)
            Hp.assert_close_rel(got["loss_prefix"], ref["loss_prefix"], Hp.LOSS_REL, "loss_prefix")
            if "t_rank" in got:
                for t in rows:
                    z, y = f["z_t"][t], int(f["ids"][t])
                    assert got["t_rank"][t] == O.teacher_rank(z, y)
                    assert abs(got["t_entropy"][t] - O.teacher_entropy(z)) <= 1e-4
                other = np.setdiff1d(np.arange(w.T), rows)
                assert not any(got[k][other].any() for k in DIAG)


@pytest.mark.parametrize("V", [8, 520, 5128, 20488, 81920])
def test_masked_and_nonfinite_rows_match_streaming(B, V):  # noqa: F811
    g = torch.Generator().manual_seed(V)
    T = 8
    z = [torch.randn((T, V), generator=g).to(torch.bfloat16) for _ in range(2)]
    lowest = torch.finfo(torch.bfloat16).min
    z[0][0, 1::2] = lowest                       # the type's lowest value as a mask, in both
    z[1][0, 1::2] = lowest
    z[1][1, ::3] = -float("inf")
    z[0][2, V // 2] = float("nan")
    z[1][3, V - 1] = float("inf")
    z[0][4] = -float("inf")
    z[0][5, 0] = 300.0                           # one entry holds the row
    ids = torch.tensor([0, 1, 0, 1, 0, 0, -1, V], dtype=torch.int32)     # two ids out of range
    d = [x.cuda() for x in (*z, ids)]
    off, win = np.array([0, T]), np.array([T], np.int32)
    outs = [_host(B.adwin_opd_from_logits(*d, off, win, want=BASE + DIAG, scheme=s, reduction=B.ADWIN_RED_SUM))
            for s in (B.ADWIN_LOGITS_AUTO, B.ADWIN_LOGITS_STREAMING)]
    a, b = outs
    for k in ("status_dev", "t_rank", "n_out"):
        assert np.array_equal(a[k], b[k]), k
    for k in ("kl", "c", "t_logp", "t_entropy"):     # fp32 sums in two orders
        assert np.allclose(a[k], b[k], rtol=1e-5, atol=1e-5 * max(1.0, np.abs(b[k]).max())), k
    # each side is a bf16 rounding of fp32 values within 1e-5 of each other: at most one ulp apart
    assert np.all(np.abs(a["dz"] - b["dz"]) <= 2 * Hp.BF16_ULP * np.abs(b["dz"]) + 1e-6 * np.abs(b["dz"]).max())


@pytest.mark.parametrize("V", LONG)
def test_long_rows_with_diagnostics_match_oracle(B, V):  # noqa: F811
    """The long-row kernel itself (the scheme that never cuts rows), up to and beyond its capacity."""
    w = synth.Workload(f"long_{V}", V, 0, 0, synth._offsets([2, 3]), np.array([1, 9], np.int32))
    p = synth.logits_problem(w)
    f = Hp.oracle_inputs(p)
    d = {k: v.cuda() for k, v in p.items()}
    ref = O.supervise_from_logits(f["z_s"], f["z_t"], f["ids"], w.offsets, w.window, reduction=O.RED_SUM)
    got = _host(B.adwin_opd_from_logits(d["z_s"], d["z_t"], d["ids"], w.offsets, w.window, reduction=O.RED_SUM,
                                        scheme=B.ADWIN_LOGITS_RESIDENT, want=BASE + DIAG))
    Hp.assert_kl(got["kl"], ref["kl"])
    Hp.assert_cost(got["c"], ref["c"])
    Hp.assert_grad(got["dz"], ref["dz"], "dz", Hp.BF16_ULP)
    for t in O.plan(w.offsets, w.window)["rows"]:
        z, y = f["z_t"][t], int(f["ids"][t])
        assert got["t_rank"][t] == O.teacher_rank(z, y)
        assert abs(got["t_entropy"][t] - O.teacher_entropy(z)) <= 1e-4
        assert abs(got["t_logp"][t] - O.teacher_logp(z, y)) <= 1e-4 * max(1.0, abs(O.teacher_logp(z, y)))
    assert got["t_rank"][1] == 0 and not got["t_entropy"][1]


@pytest.mark.parametrize("V,n_adm", [(81928, 1), (81928, 15), (102408, 156), (122880, 156), (81928, 157), (163848, 31), (81928, 257)])
def test_split_rows_match_whole_rows(B, V, n_adm):  # noqa: F811
    """Few long rows are cut into pieces (up to 140 or 156 rows, and where a second round of the compute
    units would be nearly empty); the same rows served whole differ by the order of fp32 sums."""
    g = torch.Generator().manual_seed(n_adm)
    off = np.array([0, 2, 2, 2 + n_adm, 5 + n_adm], np.int64)
    win = np.array([0, 7, n_adm, 0], np.int32)           # rows outside the windows on both sides
    T = int(off[-1])
    z = [(2 * torch.randn((T, V), generator=g)).to(torch.bfloat16) for _ in range(2)]
    z[1][2, 5] = float("nan")
    ids = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
    if n_adm > 2:
        ids[3], ids[4] = -1, V - 1
    d = [x.cuda() for x in (*z, ids)]
    for est in (O.EST_EXPECTED, O.EST_SAMPLED):
        for want in (BASE, BASE + DIAG):
            kw = dict(want=want, estimator=est, reduction=B.ADWIN_RED_SUM, grad_scale=-2.0)
            a = _host(B.adwin_opd_from_logits(*d, off, win, scheme=B.ADWIN_LOGITS_AUTO, **kw))
            b = _host(B.adwin_opd_from_logits(*d, off, win, scheme=B.ADWIN_LOGITS_STREAMING, **kw))
            for k in a:
                if a[k].dtype.kind == "i" or k == "t_rank":
                    assert np.array_equal(a[k], b[k]), k
                elif k == "dz":
                    assert np.all(np.abs(a[k] - b[k]) <= 2 * Hp.BF16_ULP * np.abs(b[k]) + 1e-6 * np.abs(b[k]).max())
                else:
                    assert np.allclose(a[k], b[k], rtol=2e-5, atol=1e-5 * max(1.0, np.abs(b[k]).max())), k


@pytest.mark.parametrize("V,rows", [(3256, 400), (8832, 400), (20480, 300), (81920, 200), (90000, 400), (151936, 500)])
def test_diagnostics_are_as_accurate_as_the_streaming_kernel(B, V, rows):  # noqa: F811
    """The sums over a row are fp32: however many logits one thread adds up, KL_t and the teacher
    entropy are as close to 64 bits as the streaming kernel's, whose 512 threads share a row (2-norm over
    the rows; 10 % for the scatter of the roundings over a few hundred rows)."""
    g = torch.Generator("cuda").manual_seed(V)
    z = [torch.randn((rows, V), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    ids = torch.randint(0, V, (rows,), generator=g, device="cuda", dtype=torch.int32)
    ref = {"kl": [], "t_entropy": []}
    for r in range(0, rows, 50):
        ls, lt = (torch.log_softmax(x[r:r + 50].double(), 1) for x in z)
        ref["kl"].append((ls.exp() * (ls - lt)).sum(1))
        ref["t_entropy"].append(-(lt.exp() * lt).sum(1))
    off, win = np.array([0, rows]), np.array([rows], np.int32)

    def errors(scheme):
        out = B.adwin_opd_from_logits(*z, ids, off, win, scheme=scheme, want=("kl",) + DIAG)
        return {k: float((out[k].double() - torch.cat(v)).norm()) for k, v in ref.items()}

    base = errors(B.ADWIN_LOGITS_STREAMING)
    for scheme in (B.ADWIN_LOGITS_AUTO, B.ADWIN_LOGITS_RESIDENT):
        got = errors(scheme)
        for k in ref:
            assert got[k] <= 1.1 * base[k], (scheme, k, got[k], base[k])


@pytest.mark.parametrize("V,n_adm,scheme", [
    (5120, 20, "AUTO"), (20480, 20, "AUTO"), (81920, 5, "AUTO"),      # a row's logits in registers
    (81928, 15, "AUTO"), (151936, 29, "AUTO"), (122880, 156, "AUTO"),  # rows cut into pieces
    (151936, 9, "RESIDENT"), (163848, 9, "RESIDENT"), (81928, 9, "STREAMING"),
])
def test_gradient_in_place(B, V, n_adm, scheme):  # noqa: F811
    """dz may be the storage of z_s or of z_t: the same bits as in an array of its own.  The sampled
    token's logits, which every workgroup of a row wants, lie anywhere in the row."""
    g = torch.Generator("cuda").manual_seed(V + n_adm)
    T = n_adm + 3
    off, win = np.array([0, 2, T]), np.array([0, n_adm], np.int32)     # rows outside the windows on both sides
    z = [torch.randn((T, V), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    ids = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    ids[2], ids[3] = 0, V - 1
    for est in (B.ADWIN_EST_EXPECTED, B.ADWIN_EST_SAMPLED):
        # with the sampled estimator the whole-row kernels of long rows read z_s[y] after dz is stored
        whole = V > 153600 or scheme != "AUTO"
        for which in ((0, 1) if est == B.ADWIN_EST_EXPECTED or not whole else (1,)):
            outs = []
            for in_place in (False, True):
                x = [q.clone() for q in z]
                call = B.LogitsCall(*x, ids, off, win, estimator=est, scheme=getattr(B, "ADWIN_LOGITS_" + scheme),
                                    reduction=B.ADWIN_RED_SUM, want=BASE + DIAG)
                if in_place:
                    call.out["dz"] = x[which]
                    call.p.dz = x[which].data_ptr()
                assert call.run() == B.ADWIN_OK
                outs.append({k: v.clone() for k, v in call.out.items()})
            for k in outs[0]:
                assert torch.equal(outs[0][k].view(torch.uint8), outs[1][k].view(torch.uint8)), (k, est, which)


def _long_rows(V, n, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    z = [torch.randn((n, V), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    return z, torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)


def test_resident_scheme_holds_for_any_number_of_rows(B):  # noqa: F811
    """An explicit scheme is the caller's choice: the long-row kernel's bits for 400 rows with
    diagnostics are those of the same rows in a call of 500, and AUTO, which takes the faster kernel for
    either, stays with the streaming kernel for the 400."""
    z, ids = _long_rows(151936, 500, 7)

    def run(n, scheme):
        out = B.adwin_opd_from_logits(z[0][:n], z[1][:n], ids[:n], np.array([0, n]), np.array([n], np.int32),
                                      reduction=O.RED_SUM, scheme=scheme, want=BASE + DIAG)
        return {k: out[k][:400] for k in ("kl", "c", "dz") + DIAG}

    few, many = run(400, B.ADWIN_LOGITS_RESIDENT), run(500, B.ADWIN_LOGITS_RESIDENT)
    auto, streaming = run(400, B.ADWIN_LOGITS_AUTO), run(400, B.ADWIN_LOGITS_STREAMING)
    for k in few:
        assert torch.equal(few[k].view(torch.uint8), many[k].view(torch.uint8)), k
        assert torch.equal(auto[k].view(torch.uint8), streaming[k].view(torch.uint8)), k


@pytest.mark.parametrize("V,n", [
    (40968, 256), (40968, 257), (51200, 300), (51208, 300), (69632, 257), (69640, 257), (69632, 903), (69632, 904),
    (69640, 512), (81920, 513), (81920, 561),
    (81928, 140), (81928, 141), (86016, 256), (86024, 216), (86024, 217), (86024, 257), (86024, 780), (86024, 781),
    (144000, 352), (144008, 352), (144008, 353), (151936, 156), (151936, 157), (180224, 256), (180232, 256),
    (131072, 513), (131072, 561),
])
def test_automatic_route_with_diagnostics(B, V, n):  # noqa: F811
    """On both sides of each line of the rule, AUTO gives the row outputs of the streaming kernel."""
    z, ids = _long_rows(V, n, V + n)
    off, win = np.array([0, n]), np.array([n], np.int32)
    auto, ref = (B.adwin_opd_from_logits(*z, ids, off, win, reduction=O.RED_SUM, scheme=s, want=BASE + DIAG)
                 for s in (B.ADWIN_LOGITS_AUTO, B.ADWIN_LOGITS_STREAMING))
    assert torch.equal(auto["t_rank"], ref["t_rank"])
    # fp32 sums in another order: KL and entropy of unit-variance logits lie near 1 and ln V
    for k in ("kl", "c", "t_entropy", "t_logp"):
        assert torch.allclose(auto[k], ref[k], rtol=2e-6, atol=1e-5), k
    assert torch.allclose(auto["dz"].float(), ref["dz"].float(), rtol=2 * Hp.BF16_ULP, atol=1e-6 * float(ref["dz"].float().abs().max()))


@pytest.mark.parametrize("want", [BASE, BASE + DIAG, BASE + DIAG + ("t_first_reject", "t_logp_mean")])
@pytest.mark.parametrize("V", [8, 5128, 20488, 40968, 81928, 400008])
def test_launches_of_a_call_share_its_work(B, V, want):  # noqa: F811
    """A plan that fits the launch of the rows is set up by it, and the tail of split rows (16 pieces at most,
    and more) runs in the launch of their gradient; status bits are then reported by another launch than the one
    that finds them.  The same call with rollouts of no rows behind it, whose plan does not fit, has the same
    rows bit for bit, and a rollout's loss is the fp32 of the mean of its rows' KL in 64 bits."""
    offsets, window = synth._offsets([6, 0, 20, 1]), np.array([4, 3, 17, 1], np.int32)
    g = torch.Generator().manual_seed(V)
    z = [torch.randn((27, V), generator=g).to(torch.bfloat16) for _ in range(2)]
    base_ids = torch.randint(0, V, (27,), generator=g, dtype=torch.int32)
    base_ids[[4, 24]] = -1                       # outside the windows: not reported
    z[1][5, 0] = float("nan")
    kw = dict(reduction=O.RED_SUM, want=want, topk=3 if "t_first_reject" in want else 0)
    for bad_id, excluded in ((False, False), (True, False), (False, True), (True, True)):
        zs, ids = z[0].clone(), base_ids.clone()
        ids[9] = V if bad_id else ids[9]
        zs[8, V - 1] = float("inf") if excluded else zs[8, V - 1]
        runs = []
        for extra in (0, 120):
            off = np.concatenate([offsets, np.full(extra, offsets[-1])])
            win = np.concatenate([window, np.zeros(extra, np.int32)]).astype(np.int32)
            runs.append(_host(B.adwin_opd_from_logits(zs.cuda(), z[1].cuda(), ids.cuda(), off, win, **kw)))
        a, b = runs
        status = (B.ADWIN_DEV_BAD_ID if bad_id else 0) | (B.ADWIN_DEV_NONFINITE if excluded else 0)
        assert int(a["status_dev"][0]) == int(b["status_dev"][0]) == status
        for k in a:
            x, y = a[k], b[k]
            if k == "t_logp_mean":               # its last row is the batch's
                x, y = np.concatenate([x[:-1], x[-1:]]), np.concatenate([y[:4], y[-1:]])
            elif k in ("loss_prefix", "n_out", "t_first_reject"):
                y = y[:4]
            assert np.array_equal(x, y), k
        for i in range(4):
            kl = a["kl"][offsets[i]:offsets[i] + min(window[i], offsets[i + 1] - offsets[i])].astype(np.float64)
            mean = kl.mean() if kl.size else 0.0
            assert abs(a["loss_prefix"][i] - mean) <= 2.0 ** -23 * abs(mean)
        assert excluded == (a["kl"][8] == 0.0) and bad_id == (a["c"][9] == 0.0)


@pytest.mark.parametrize("V,n_adm", [(81928, 210), (81928, 211), (81928, 400), (136008, 185), (136008, 186), (172008, 210),
                                     (190008, 256), (190008, 400), (190008, 401)])
def test_lines_of_split_rows(B, V, n_adm):  # noqa: F811
    """Both sides of the lines between rows in pieces and whole ones, as in test_split_rows_match_whole_rows."""
    z, ids = _long_rows(V, n_adm, V + n_adm)
    off, win = np.array([0, n_adm]), np.array([n_adm], np.int32)
    for want in (BASE, BASE + DIAG):
        a, b = (_host(B.adwin_opd_from_logits(*z, ids, off, win, reduction=O.RED_SUM, scheme=s, want=want))
                for s in (B.ADWIN_LOGITS_AUTO, B.ADWIN_LOGITS_STREAMING))
        for k in a:
            if a[k].dtype.kind == "i":
                assert np.array_equal(a[k], b[k]), k
            elif k == "dz":
                assert np.all(np.abs(a[k] - b[k]) <= 2 * Hp.BF16_ULP * np.abs(b[k]) + 1e-6 * np.abs(b[k]).max())
            else:
                assert np.allclose(a[k], b[k], rtol=2e-5, atol=1e-5 * max(1.0, np.abs(b[k]).max())), k


@pytest.mark.parametrize("V,n", [(82048, 2050), (151936, 1110), (163840, 1030)])
def test_long_rows_past_the_caches(B, V, n):  # noqa: F811
    """Logits of more than 320 MiB, in long rows of whole lines, go past the caches: the bits of the same kernel on the same
    rows in two calls, which keep them; rows outside the windows, too.  (V = 163,840: more logits than stay on chip.)"""
    assert 2 * n * V > 320 << 20 > n // 2 * 2 * V and V % 64 == 0
    z, ids = _long_rows(V, n, V)
    adm = np.zeros(n, bool)
    adm[:5] = adm[7:n - 13] = True
    kw = dict(reduction=O.RED_SUM, scheme=B.ADWIN_LOGITS_RESIDENT)

    def run(lo, hi, off, win, **more):
        return B.adwin_opd_from_logits(z[0][lo:hi], z[1][lo:hi], ids[lo:hi], np.array(off), np.array(win, np.int32), **{**kw, **more})

    for est in (O.EST_EXPECTED, O.EST_SAMPLED):
        for want in (BASE, BASE + DIAG):
            a = run(0, n, [0, 7, n], [5, n - 20], want=want, estimator=est)
            m = n // 2
            parts = [run(0, m, [0, 7, m], [5, m], want=want, estimator=est),
                     run(m, n, [0, n - m], [n - 13 - m], want=want, estimator=est)]
            for k in ("kl", "c", "dz") + (DIAG if "t_rank" in want else ()):
                b = torch.cat([x[k] for x in parts])
                assert torch.equal(a[k].view(torch.uint8), b.view(torch.uint8)), (k, est)
                assert not a[k][torch.from_numpy(~adm)].any()
            assert float(a["kl"].abs().max()) > 0
            auto = run(0, n, [0, 7, n], [5, n - 20], want=want, estimator=est, scheme=B.ADWIN_LOGITS_AUTO)
            assert torch.equal(a["dz"].view(torch.uint8), auto["dz"].view(torch.uint8))      # it serves them all


@pytest.mark.parametrize("V,n", [(82048, 2050), (86016, 1960), (151936, 1110), (180288, 940), (196608, 860)])
def test_results_do_not_depend_on_the_address(B, V, n):  # noqa: F811
    """Long rows of more than 320 MiB, at the lines of the rule that chooses between the streaming and the long-row kernel
    with diagnostics: the same bits from logits that begin a line and from logits that begin 16 bytes into one."""
    z, ids = _long_rows(V, n, V)
    shifted = []
    for x in z:
        shifted.append(torch.empty(x.numel() + 8, dtype=torch.bfloat16, device="cuda")[8:].view(x.shape))
        shifted[-1].copy_(x)
        assert x.data_ptr() % 128 == 0 and shifted[-1].data_ptr() % 128 == 16
    off, win = np.array([0, 7, n]), np.array([5, n - 20], np.int32)
    for want in (BASE, BASE + DIAG):
        a, b = (B.adwin_opd_from_logits(*x, ids, off, win, reduction=O.RED_SUM, want=want) for x in (z, shifted))
        for k in a:
            assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k
