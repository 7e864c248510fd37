"""GPU parity of the adaptive summary layer (Section 4.2, the summary-token equation)
against the fp64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import skipffn_oracle as O
from paper_2503_21817_amd import binding as B
from paper_2503_21817_amd import workloads as W
from helpers import REL_L2_TOL, bits_of, f64_of, rel_l2, to_dev_bf16

pytestmark = pytest.mark.gpu


def run_gpu(hid, tok, seg, wb, gout=None, gh0=None, flags=0, dw_init=None, saved=True):
    T, C = hid.shape
    S = len(seg) - 1
    d_h = to_dev_bf16(hid)
    d_tok = torch.from_numpy(np.ascontiguousarray(tok, dtype=np.int32)).cuda()
    d_seg = torch.from_numpy(np.ascontiguousarray(seg, dtype=np.int32)).cuda()
    d_w = to_dev_bf16(wb)
    out = torch.full((max(S, 1), C), float("nan"), dtype=torch.bfloat16, device="cuda")[:S]
    sv = torch.empty(B.skipffn_summary_saved_bytes(len(tok), S, C), dtype=torch.uint8, device="cuda") if saved else None
    ws = torch.empty(B.skipffn_summary_workspace_bytes(len(tok), S, C), dtype=torch.uint8, device="cuda")
    B.skipffn_summary_forward(d_h, d_tok, d_seg, d_w, out, saved=sv, workspace=ws)
    torch.cuda.synchronize()
    res = {"out": out, "saved": sv}
    if gout is not None:
        d_g = to_dev_bf16(gout)
        d_gh = to_dev_bf16(gh0)
        dw = torch.full((C,), float("nan"), dtype=torch.float32, device="cuda") if dw_init is None else dw_init
        B.skipffn_summary_backward(d_h, d_tok, d_seg, d_w, sv, d_g, d_gh, dw, workspace=ws, flags=flags)
        torch.cuda.synchronize()
        res["gh"] = d_gh
        res["dw"] = dw
    return res


def random_case(T, C, seg_lens, seed, scale=0.3):
    rng = np.random.default_rng(seed)
    hid = O.f64_to_bf16_bits(rng.standard_normal((T, C)))
    wb = O.f64_to_bf16_bits(rng.standard_normal(C) * scale / np.sqrt(C) * 4)
    n = int(sum(seg_lens))
    tok = rng.permutation(T)[:n].astype(np.int32)              # disjoint sets, any order
    seg = np.concatenate([[0], np.cumsum(seg_lens)]).astype(np.int32)
    gout = O.f64_to_bf16_bits(rng.standard_normal((len(seg_lens), C)))
    gh0 = O.f64_to_bf16_bits(rng.standard_normal((T, C)))
    return hid, tok, seg, wb, gout, gh0


CASES = [
    # T, C, set sizes
    (300, 256, (1, 16, 17, 33, 100)),         # one token, exactly one chunk, one over, several chunks
    (900, 1024, (576, 0, 200)),               # an empty set between two sets
    (64, 4096, (40,)),                        # backbone width
    (500, 264, (15, 31, 250)),                # C not a multiple of the thread count
    (200, 9000 // 8 * 8, (120,)),             # wide rows
    # one and two sets (bounds by scalar loads; an empty one first, last and alone), three (by the lanes of a wavefront)
    (20, 256, (16,)), (20, 256, (0,)), (40, 256, (17, 16)), (40, 256, (0, 33)), (40, 256, (33, 0)), (40, 256, (0, 33, 1)),
    # chunks + sets = 32 and 33: the two forms of the sum over chunks
    (600, 264, (472, 8)), (600, 264, (488, 8)),
]


@pytest.mark.parametrize("T,C,lens", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_summary_forward_backward_against_oracle(T, C, lens):
    hid, tok, seg, wb, gout, gh0 = random_case(T, C, lens, seed=7 + T)
    fo = O.summary_forward(hid, tok, seg, wb)
    bo = O.summary_backward(hid, tok, seg, wb, gout, gh0)
    r = run_gpu(hid, tok, seg, wb, gout, gh0)
    S = len(lens)
    got = f64_of(r["out"])
    nz = [i for i in range(S) if lens[i] > 0]
    assert rel_l2(got[nz], O.bf16_bits_to_f64(fo["out_bits"][nz])) < REL_L2_TOL
    for i in range(S):
        if lens[i] == 0:
            assert np.all(got[i] == 0)                      # empty set: zero row
    # fp32 intermediates kept for the backward: scores, log-sum-exp, x^s
    sv = r["saved"]
    n = len(tok)
    scores = sv[:n * 4].view(torch.float32).double().cpu().numpy()
    assert np.allclose(scores, fo["scores"], rtol=1e-4, atol=1e-4)
    off = (n * 4 + 255) // 256 * 256
    lse = sv[off:off + S * 4].view(torch.float32).double().cpu().numpy()
    assert np.allclose(lse[nz], fo["lse"][nz], rtol=1e-4, atol=1e-4)
    off += (S * 4 + 255) // 256 * 256
    xs = sv[off:off + S * C * 4].view(torch.float32).double().cpu().numpy().reshape(S, C)
    assert rel_l2(xs[nz], fo["xs"][nz]) < 1e-4
    # backward: listed rows within tolerance, the others untouched bit for bit
    gb = bits_of(r["gh"])
    listed = np.zeros(T, bool); listed[tok] = True
    assert np.array_equal(gb[~listed], gh0[~listed])
    assert rel_l2(O.bf16_bits_to_f64(gb[listed]), O.bf16_bits_to_f64(bo["gh_bits"][listed])) < REL_L2_TOL
    # the update itself (gradient minus what was there), which the bf16 sum above could hide
    upd_gpu = O.bf16_bits_to_f64(gb[listed]) - O.bf16_bits_to_f64(gh0[listed])
    upd_ref = O.bf16_bits_to_f64(bo["gh_bits"][listed]) - O.bf16_bits_to_f64(gh0[listed])
    big = np.abs(upd_ref) > 0.05                           # above the bf16 rounding of an O(1) sum
    if big.any():
        assert rel_l2(upd_gpu[big], upd_ref[big]) < 0.1
    assert rel_l2(r["dw"].double().cpu().numpy(), bo["dw"]) < REL_L2_TOL


def test_summary_on_the_paper_shaped_token_sets():
    """Configuration-2 token mix: per sequence the retained and the skipped visual tokens."""
    w = W.config(2)
    hid = W.make_hidden(w)
    tok, seg = W.make_summary_sets(w)
    wb = W.make_summary_weight(w)
    assert len(seg) == 2 * len(w.visual) + 1 and len(tok) == sum(w.visual)
    rng = np.random.default_rng(3)
    gout = O.f64_to_bf16_bits(rng.standard_normal((len(seg) - 1, w.C)))
    gh0 = W.make_grad(w)
    fo = O.summary_forward(hid, tok, seg, wb)
    bo = O.summary_backward(hid, tok, seg, wb, gout, gh0)
    r = run_gpu(hid, tok, seg, wb, gout, gh0)
    assert rel_l2(f64_of(r["out"]), O.bf16_bits_to_f64(fo["out_bits"])) < REL_L2_TOL
    gb = bits_of(r["gh"])
    listed = np.zeros(w.T, bool); listed[tok] = True
    assert np.array_equal(gb[~listed], gh0[~listed])
    assert rel_l2(O.bf16_bits_to_f64(gb[listed]), O.bf16_bits_to_f64(bo["gh_bits"][listed])) < REL_L2_TOL
    assert rel_l2(r["dw"].double().cpu().numpy(), bo["dw"]) < REL_L2_TOL


def test_out_of_range_tokens_and_bad_segments_are_ignored():
    hid, tok, seg, wb, gout, gh0 = random_case(120, 256, (30, 20), seed=5)
    bad = tok.copy()
    bad[3] = -1; bad[35] = 120; bad[36] = 2_000_000_000
    keep = np.ones(len(tok), bool); keep[[3, 35, 36]] = False
    tok_ok = tok[keep]
    seg_ok = np.array([0, 29, 47], dtype=np.int32)
    fo = O.summary_forward(hid, tok_ok, seg_ok, wb)
    bo = O.summary_backward(hid, tok_ok, seg_ok, wb, gout, gh0)
    r = run_gpu(hid, bad, seg, wb, gout, gh0)
    assert rel_l2(f64_of(r["out"]), O.bf16_bits_to_f64(fo["out_bits"])) < REL_L2_TOL
    gb = bits_of(r["gh"])
    listed = np.zeros(120, bool); listed[tok_ok] = True
    assert np.array_equal(gb[~listed], gh0[~listed])
    assert rel_l2(r["dw"].double().cpu().numpy(), bo["dw"]) < REL_L2_TOL
    # a segment table that runs past the token list is clamped to it
    seg_long = np.array([0, 30, 5000], dtype=np.int32)
    r2 = run_gpu(hid, tok, seg_long, wb)
    f2 = O.summary_forward(hid, tok, seg, wb)
    assert rel_l2(f64_of(r2["out"]), O.bf16_bits_to_f64(f2["out_bits"])) < REL_L2_TOL


def test_inference_without_saved_and_dw_accumulate_and_determinism():
    hid, tok, seg, wb, gout, gh0 = random_case(400, 512, (100, 150, 60), seed=9)
    a = run_gpu(hid, tok, seg, wb, saved=False)
    b = run_gpu(hid, tok, seg, wb, gout, gh0)
    assert torch.equal(a["out"].view(torch.int16), b["out"].view(torch.int16))
    c = run_gpu(hid, tok, seg, wb, gout, gh0)
    assert torch.equal(b["dw"], c["dw"]) and torch.equal(b["gh"].view(torch.int16), c["gh"].view(torch.int16))
    acc = torch.ones(512, dtype=torch.float32, device="cuda")
    d = run_gpu(hid, tok, seg, wb, gout, gh0, flags=B.FLAG_DW_ACCUMULATE, dw_init=acc)
    assert torch.allclose(d["dw"] - 1.0, b["dw"], rtol=1e-5, atol=1e-5)


def test_no_sets_is_a_no_op_and_zeroes_dw():
    C = 256
    d_h = torch.zeros((10, C), dtype=torch.bfloat16, device="cuda")
    tok = torch.zeros(0, dtype=torch.int32, device="cuda")
    seg = torch.zeros(1, dtype=torch.int32, device="cuda")
    w = torch.zeros(C, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros((0, C), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.skipffn_summary_workspace_bytes(0, 0, C), dtype=torch.uint8, device="cuda")
    B.skipffn_summary_forward(d_h, tok, seg, w, out, workspace=ws)
    dw = torch.full((C,), 5.0, dtype=torch.float32, device="cuda")
    sv = torch.empty(B.skipffn_summary_saved_bytes(0, 0, C), dtype=torch.uint8, device="cuda")
    B.skipffn_summary_backward(d_h, tok, seg, w, sv, out, d_h.clone(), dw, workspace=ws)
    torch.cuda.synchronize()
    assert torch.count_nonzero(dw).item() == 0


@pytest.mark.parametrize("C", [8, 1024, 1032, 2048, 2056, 4088, 4104])
def test_rows_held_in_registers(C):
    """Widths at the ends of the forms that hold the rows of a chunk in registers, and past the last; a chunk of one token, a full
    one, and sets of several."""
    test_summary_forward_backward_against_oracle(300, C, (1, 16, 17, 130))


@pytest.mark.parametrize("lens", [(1, 17, 130), (19,)], ids=str)      # sets found by the lanes of a wavefront; by scalar loads
@pytest.mark.parametrize("C", [1024, 2048, 4096, 4104])
def test_a_non_finite_row_outside_the_sets_changes_no_bit(C, lens):
    """Row 0 is in no set: sets that do not fill their last chunk, and a token index out of range, must not read its values in."""
    hid, tok, seg, wb, gout, gh0 = random_case(300, C, lens, seed=41 + C)
    tok = np.where(tok == 0, 299 if 299 not in tok else -1, tok).astype(np.int32)
    tok[-1] = 300
    clean = run_gpu(hid, tok, seg, wb, gout, gh0)
    for bits in (0x7F80, 0xFF80, 0x7FC0):                              # inf, -inf, NaN
        dirty = hid.copy()
        dirty[0] = bits
        r = run_gpu(dirty, tok, seg, wb, gout, gh0)
        for key in ("out", "gh"):
            assert np.array_equal(bits_of(r[key]), bits_of(clean[key])), key
        assert torch.equal(r["dw"], clean["dw"])
        assert np.all(np.isfinite(f64_of(r["out"])))


@pytest.mark.parametrize("lens", [(208, 240, 257), (4200, 3)], ids=str)
def test_many_chunks_a_set(lens):
    """13, 15 and 17 chunks (a batch of chunks that the merge of a set holds at once, less, more), and more than the 256 whose scales it
    stages at a time."""
    test_summary_forward_backward_against_oracle(sum(lens) + 10, 520, lens)
