"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on
the same seeded inputs.  Integer / byte results are compared bit for bit;
floating-point results by relative L2 error over retained rows, bound 1e-2
(bf16 inputs, fp32 accumulation, bf16 intermediates)."""
import numpy as np
import pytest
import torch

from oracle import skipffn_oracle as O
from paper_2503_21817_amd import binding as B
from paper_2503_21817_amd import workloads as W
from helpers import REL_L2_TOL, TWO_PART_GATE_UP, Problem, bits_of, f64_of, rel_l2, to_dev_bf16

pytestmark = pytest.mark.gpu


def run_compact(mask_np, want_pos=True):
    T = mask_np.shape[0]
    d_mask = torch.from_numpy(mask_np).cuda() if T else torch.empty(0, dtype=torch.uint8, device="cuda")
    idx = torch.full((max(T, 1),), -7, dtype=torch.int32, device="cuda")
    nr = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    pos = torch.full((max(T, 1),), -7, dtype=torch.int32, device="cuda") if want_pos else None
    ws = torch.empty(max(B.skipffn_compact_workspace_bytes(T), 16), dtype=torch.uint8, device="cuda")
    B.skipffn_compact(d_mask, idx, nr, pos, ws)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), int(nr.item()), None if pos is None else pos.cpu().numpy()


@pytest.mark.parametrize("T", [0, 1, 3, 64, 255, 256, 257, 1000, 4097, 16384, 29411, 262144,
                               262145, 300001, (1 << 20) + 37])
@pytest.mark.parametrize("kind", ["rand", "all0", "all1", "alt", "ends", "bytes"])
def test_compact_bit_exact(T, kind):
    rng = np.random.default_rng(T + len(kind))
    if kind == "rand":
        m = (rng.random(T) < 0.7).astype(np.uint8)
    elif kind == "all0":
        m = np.zeros(T, np.uint8)
    elif kind == "all1":
        m = np.ones(T, np.uint8)
    elif kind == "alt":
        m = (np.arange(T) % 2).astype(np.uint8)
    elif kind == "ends":
        m = np.ones(T, np.uint8); m[:1] = 0; m[-1:] = 0
    else:
        m = (rng.integers(0, 256, T) * (rng.random(T) < 0.5)).astype(np.uint8)
    print(f"compact T={T} kind={kind}", flush=True)
    idx, R, pos = run_compact(m)
    oidx, oR, opos = O.compact(m)
    assert R == oR
    assert np.array_equal(idx[:R], oidx)
    if T:
        assert np.all(idx[R:T] == -7)          # entries beyond R untouched
        assert np.array_equal(pos[:T], opos)


@pytest.mark.parametrize("cfg", [2, 3, 4])
def test_compact_on_workload_masks(cfg):
    w = W.config(cfg)
    m = W.make_mask(w)
    idx, R, pos = run_compact(m, want_pos=False)
    oidx, oR, _ = O.compact(m)
    assert R == oR == w.R and np.array_equal(idx[:R], oidx)


def gpu_forward(p, R_host=True, inplace=False, saved=True, flags=0):
    w = p.w
    bufs = B.SkipFFNBuffers(w.T, w.T if not R_host else w.R, w.C, w.I, training=saved)
    B.skipffn_compact(p.d_mask, bufs.idx, bufs.num_retained, None, bufs.compact_ws)
    hidden = p.d_hidden.clone()
    out = hidden if inplace else torch.full_like(hidden, float("nan"))
    B.skipffn_forward(hidden, out, bufs.idx, w.R if R_host else None, p.d_wg, p.d_wu, p.d_wd,
                      eps=w.eps, rms_gain=p.d_gain, num_retained=bufs.num_retained,
                      saved=bufs.saved, workspace=bufs.fwd_ws, flags=flags)
    torch.cuda.synchronize()
    return out, bufs


def gpu_backward(p, bufs, R_host=True, inplace=False, flags=0, dw=None, dgain=None):
    w = p.w
    grad = p.d_grad.clone()
    gh = grad if inplace else torch.full_like(grad, float("nan"))
    dt = torch.float32 if flags & B.FLAG_DW_FP32 else torch.bfloat16
    if dw is None:
        dw = [torch.full((w.I, w.C), float("nan"), dtype=dt, device="cuda"),
              torch.full((w.I, w.C), float("nan"), dtype=dt, device="cuda"),
              torch.full((w.C, w.I), float("nan"), dtype=dt, device="cuda")]
    B.skipffn_backward(grad, gh, bufs.idx, w.R if R_host else None, p.d_wg, p.d_wu, p.d_wd,
                       bufs.saved, dw[0], dw[1], dw[2], eps=w.eps, rms_gain=p.d_gain,
                       num_retained=bufs.num_retained, workspace=bufs.bwd_ws, flags=flags,
                       d_rms_gain=dgain)
    torch.cuda.synchronize()
    return gh, dw


SMALL = [
    W.config(1),
    W.small(C=512, I=1368, visual=(300, 411), text=(20, 35), keep=(130, 212), seed=11, name="ragged-2tiles"),
    W.small(C=264, I=520, visual=(700,), text=(9,), keep=(600,), seed=12, name="odd-dims-3tiles"),
    W.small(C=1024, I=2048, visual=(64,), text=(1,), keep=(0,), seed=13, name="one-row"),
]


@pytest.mark.parametrize("w", SMALL, ids=lambda w: w.name)
@pytest.mark.parametrize("gain", [False, True])
def test_forward_stage_by_stage(w, gain):
    print(f"forward stages {w.name} T={w.T} R={w.R} C={w.C} I={w.I} gain={gain}", flush=True)
    p = Problem(w, unit_gain=not gain, with_gain_tensor=gain)
    ref = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    out, bufs = gpu_forward(p)
    R = w.R
    idx = bufs.idx[:R].cpu().numpy()
    assert np.array_equal(idx, ref["idx"])
    sv = bufs.saved_views(R)
    # gathered input rows are bit copies
    assert np.array_equal(bits_of(sv["xrows"]), p.hidden[idx])
    assert rel_l2(f64_of(sv["rstd"]), ref["rstd"]) < 1e-6
    assert rel_l2(f64_of(sv["xn"]), ref["xn"]) < 3e-3          # one bf16 rounding: 2^-9 rms
    for k in ("G", "U", "H"):
        assert rel_l2(f64_of(sv[k]), ref[k]) < REL_L2_TOL, k
    # the transposed copy of the normalised rows is exact, its padding columns are zero
    xnT = bits_of(sv["xnT"])
    assert np.array_equal(xnT[:, :R], bits_of(sv["xn"]).T)
    assert not xnT[:, R:].any()
    # so is the transposed copy of silu(gate) * up that the gate/up epilogue (or, with few rows, a copy kernel) leaves
    HT = bits_of(sv["HT"])
    assert np.array_equal(HT[:, :R], bits_of(sv["H"]).T)
    assert not HT[:, R:].any()
    got = bits_of(out)
    skipped = p.mask != 0
    assert np.array_equal(got[skipped], p.hidden[skipped])      # bitwise passthrough
    e = rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(ref["out_bits"][idx]))
    assert e < REL_L2_TOL, e
    # the FFN update on its own (the residual can hide it when |y| << |x|)
    y_out, _ = gpu_forward(p, flags=B.FLAG_NO_RESIDUAL)
    yb = bits_of(y_out)
    assert np.array_equal(yb[skipped], p.hidden[skipped])
    ey = rel_l2(O.bf16_bits_to_f64(yb[idx]), ref["Y"])
    assert ey < REL_L2_TOL, ey


@pytest.mark.parametrize("w", SMALL, ids=lambda w: w.name)
@pytest.mark.parametrize("gain", [False, True])
def test_backward_against_oracle(w, gain):
    print(f"backward {w.name} T={w.T} R={w.R} C={w.C} I={w.I} gain={gain}", flush=True)
    p = Problem(w, unit_gain=not gain, with_gain_tensor=gain)
    ref = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    _, bufs = gpu_forward(p)
    gh, dw = gpu_backward(p, bufs)
    idx = ref["idx"]
    got = bits_of(gh)
    skipped = p.mask != 0
    assert np.array_equal(got[skipped], p.grad[skipped])
    e = rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(ref["dx_bits"][idx]))
    assert e < REL_L2_TOL, ("dx", e)
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        e = rel_l2(f64_of(t), ref[k])
        assert e < REL_L2_TOL, (k, e)
    # fp32 weight gradients, then accumulation on top of them: 2x
    gh32, dw32 = gpu_backward(p, bufs, flags=B.FLAG_DW_FP32)
    assert np.array_equal(bits_of(gh32), got)
    for t, k in zip(dw32, ("dw_gate", "dw_up", "dw_down")):
        assert rel_l2(f64_of(t), ref[k]) < REL_L2_TOL, k
    first = [t.clone() for t in dw32]
    gpu_backward(p, bufs, flags=B.FLAG_DW_FP32 | B.FLAG_DW_ACCUMULATE, dw=dw32)
    for t, f in zip(dw32, first):
        assert torch.equal(t, 2 * f)
    # bf16 accumulate onto zeros equals overwrite
    z = [torch.zeros_like(t) for t in dw]
    gpu_backward(p, bufs, flags=B.FLAG_DW_ACCUMULATE, dw=z)
    for t, f in zip(z, dw):
        assert torch.equal(t, f)


def test_invariants_on_gpu():
    w = W.small(C=512, I=1024, visual=(300,), text=(30,), keep=(77,), seed=21)
    p = Problem(w)
    out1, bufs = gpu_forward(p)
    # run twice: bitwise equal (deterministic reduction order)
    out2, _ = gpu_forward(p)
    assert torch.equal(out1.view(torch.int16), out2.view(torch.int16))
    # in place == out of place
    out3, _ = gpu_forward(p, inplace=True)
    assert torch.equal(out1.view(torch.int16), out3.view(torch.int16))
    # device-side R == host R
    out4, bufs4 = gpu_forward(p, R_host=False)
    assert torch.equal(out1.view(torch.int16), out4.view(torch.int16))
    gh1, dw1 = gpu_backward(p, bufs)
    gh2, dw2 = gpu_backward(p, bufs, inplace=True)
    gh4, dw4 = gpu_backward(p, bufs4, R_host=False)
    assert torch.equal(gh1.view(torch.int16), gh2.view(torch.int16))
    assert torch.equal(gh1.view(torch.int16), gh4.view(torch.int16))
    for a, b, c in zip(dw1, dw2, dw4):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        assert torch.equal(a.view(torch.int16), c.view(torch.int16))


def test_retain_all_and_retain_none():
    base = W.small(C=256, I=512, visual=(150,), text=(10,), keep=(150,), seed=31)
    p = Problem(base)
    assert not p.mask.any()
    out, bufs = gpu_forward(p)
    wide = [O.bf16_bits_to_f64(a) for a in (p.hidden, p.wg, p.wu, p.wd)]
    dense = O.dense_swiglu_layer(wide[0], wide[1], wide[2], wide[3], None, base.eps)
    assert rel_l2(f64_of(out), dense) < REL_L2_TOL
    none = W.small(C=256, I=512, visual=(150,), text=(0,), keep=(0,), seed=32)
    q = Problem(none)
    q.hidden[3, :4] = [0x7FC1, 0xFF80, 0x8000, 0x0001]
    q.d_hidden = to_dev_bf16(q.hidden)
    assert q.mask.all()
    out, bufs = gpu_forward(q)
    assert np.array_equal(bits_of(out), q.hidden)
    assert int(bufs.num_retained.item()) == 0
    gh, dw = gpu_backward(q, bufs)
    assert np.array_equal(bits_of(gh), q.grad)
    for t in dw:
        assert not t.view(torch.int16).any()
    # accumulate with R == 0 leaves dW alone
    keep = [torch.ones_like(t) for t in dw]
    gpu_backward(q, bufs, flags=B.FLAG_DW_ACCUMULATE, dw=keep)
    for t in keep:
        assert torch.equal(t, torch.ones_like(t))


def test_inference_forward_without_saved_buffer():
    w = W.small(C=512, I=1024, visual=(300,), text=(30,), keep=(77,), seed=21)
    p = Problem(w)
    a, _ = gpu_forward(p, saved=True)
    b, _ = gpu_forward(p, saved=False)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_skip_kv_cache_row_gather():
    rng = np.random.default_rng(5)
    T, D = 777, 1024
    cache = rng.integers(0, 65536, (T, D)).astype(np.uint16)
    m = (rng.random(T) < 0.75).astype(np.uint8)
    idx, R, _ = O.compact(m)
    src = to_dev_bf16(cache)
    dst = torch.zeros((R, D), dtype=torch.bfloat16, device="cuda")
    B.skipffn_gather_rows(src, dst, torch.from_numpy(idx).cuda(), R)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(dst), O.kv_skip_cache(cache, m))


@pytest.mark.parametrize("seed", range(6))
def test_random_shapes_forward_backward(seed):
    """Seeded random shapes: odd multiples of 8 for C and I, ragged R, one to three
    sequences; both R given by the host and R read on the device."""
    rng = np.random.default_rng(1000 + seed)
    C = 8 * int(rng.integers(8, 90))
    I = 8 * int(rng.integers(8, 200))
    nseq = int(rng.integers(1, 4))
    vis = [int(rng.integers(1, 400)) for _ in range(nseq)]
    txt = [int(rng.integers(0, 30)) for _ in range(nseq)]
    keep = [int(rng.integers(0, v + 1)) for v in vis]
    w = W.small(C=C, I=I, visual=vis, text=txt, keep=keep, seed=50 + seed, name=f"rand{seed}")
    print(f"random shape {seed}: T={w.T} R={w.R} C={C} I={I}", flush=True)
    if w.R == 0:
        pytest.skip("empty retained set is covered elsewhere")
    p = Problem(w, unit_gain=False, with_gain_tensor=bool(seed & 1))
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    idx = fo["idx"]
    sk = p.mask != 0
    for r_host in (True, False):
        out, bufs = gpu_forward(p, R_host=r_host, inplace=bool(seed & 2))
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
        gh, dw = gpu_backward(p, bufs, R_host=r_host, inplace=bool(seed & 2))
        gb = bits_of(gh)
        assert np.array_equal(gb[sk], p.grad[sk])
        assert rel_l2(O.bf16_bits_to_f64(gb[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
        for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
            assert rel_l2(f64_of(t), bo[k]) < REL_L2_TOL, (k, r_host)


@pytest.mark.parametrize("C,I", [(264, 200), (1096, 456), (456, 1096), (2056, 136), (192, 2056), (264, 8264)],
                         ids=lambda v: str(v))
@pytest.mark.parametrize("flags", [0, B.FLAG_BALANCED_SPLIT], ids=["", "core"])
def test_k_ranges_that_end_inside_a_slab(C, I, flags):
    """256-row tiles (R > 256) with contraction lengths that are no multiple of the 64-deep K slab, from
    3 to 130 slabs.  The forward of these narrow layers runs on tiles of all rows; the balanced split (a flag) and the
    widest I take it to the general core, where the backward always runs: its main loop runs its steady state (unmasked loads, offsets stepped per slab) up to
    the slabs at the end of the K range - and, in the dXn GEMM, of each of its two operand pairs - which
    take the guarded, masked path.  R = 300 is no multiple of 64 either (the weight-gradient GEMMs
    contract over it)."""
    w = W.small(C=C, I=I, visual=(330,), text=(12,), keep=(288,), seed=70 + C % 7, name=f"ktail-{C}-{I}")
    assert w.R == 300
    p = Problem(w, unit_gain=False, with_gain_tensor=True)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    idx, sk = fo["idx"], p.mask != 0
    for r_host in (True, False):
        out, bufs = gpu_forward(p, R_host=r_host, flags=flags)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
        sv = bufs.saved_views(w.R)
        for k in ("G", "U", "H"):
            assert rel_l2(f64_of(sv[k]), fo[k]) < REL_L2_TOL, k
        gh, dw = gpu_backward(p, bufs, R_host=r_host, flags=flags)
        gb = bits_of(gh)
        assert np.array_equal(gb[sk], p.grad[sk])
        assert rel_l2(O.bf16_bits_to_f64(gb[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
        for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
            assert rel_l2(f64_of(t), bo[k]) < REL_L2_TOL, (k, r_host)


BALANCED = [
    # (workload, what it exercises)
    W.small(C=512, I=1368, visual=(300, 411), text=(20, 35), keep=(130, 212), seed=21,
            name="bal-2groups-2tiles"),           # 2 m-tiles, K tail, aligned chunks + remainder pieces
    W.small(C=264, I=520, visual=(700,), text=(9,), keep=(600,), seed=22,
            name="bal-3tiles-short-k"),           # ragged C, few K slabs: q from the slab budget
    W.small(C=1024, I=2048, visual=(64,), text=(1,), keep=(0,), seed=23, name="bal-one-row"),
    W.small(C=256, I=9000, visual=(900, 600), text=(30, 12), keep=(450, 333), seed=24,
            name="bal-long-k-4tiles"),            # long K, remainder pieces spanning tiles
    W.small(C=4096, I=320, visual=(4400,), text=(30,), keep=(4100,), seed=25,
            name="bal-17-mtiles-16-workgroups"),  # more m-tiles than workgroups per group: a whole
                                                  # tile per workgroup first, the 17th split 5 ways
]


@pytest.mark.parametrize("w", BALANCED, ids=lambda w: w.name)
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_balanced_split_forward_backward(w, r_host):
    """The balanced K split of the down and dXn GEMMs (forced by flag: the cost model would
    not pick it at these sizes) against the oracle, with R known on the host and R read on
    the device (the plan is then recomputed in the kernels from the device-side count)."""
    p = Problem(w, unit_gain=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    idx = fo["idx"]
    sk = p.mask != 0
    out, bufs = gpu_forward(p, R_host=r_host, flags=B.FLAG_BALANCED_SPLIT)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
    gh, dw = gpu_backward(p, bufs, R_host=r_host, flags=B.FLAG_BALANCED_SPLIT)
    gb = bits_of(gh)
    assert np.array_equal(gb[sk], p.grad[sk])
    assert rel_l2(O.bf16_bits_to_f64(gb[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    # the split only changes the order of fp32 additions: results agree with the default path
    out2, bufs2 = gpu_forward(p, R_host=r_host)
    gh2, _ = gpu_backward(p, bufs2, R_host=r_host)
    a, b = f64_of(out)[idx], f64_of(out2)[idx]
    assert rel_l2(a, b) < 1e-2
    assert rel_l2(f64_of(gh)[idx], f64_of(gh2)[idx]) < 1e-2


KV_CASES = [
    # (leading dims, T, D, keep probability, destination capacity: "packed" or "prefill")
    ((3, 2, 4), 777, 128, 0.25, "packed"),      # layers x key/value x heads, LLaMA head size
    ((2, 2, 8), 616, 128, 0.30, "prefill"),     # compacted cache keeps the prefill capacity
    ((5,), 1000, 8, 0.5, "packed"),             # 16-byte rows
    ((70000,), 6, 8, 0.5, "packed"),            # more slabs than one grid dimension holds
    ((1, 1), 300, 1024, 1.0, "packed"),         # nothing skipped
]


@pytest.mark.parametrize("lead,T,D,keep,cap", KV_CASES, ids=lambda v: str(v).replace(" ", ""))
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_skip_kv_cache_whole_cache(lead, T, D, keep, cap, r_host):
    """Section 4.3 on a whole cache in one launch, bit for bit against the oracle."""
    rng = np.random.default_rng(31 + T)
    cache = rng.integers(0, 65536, lead + (T, D)).astype(np.uint16)
    m = (rng.random(T) >= keep).astype(np.uint8)
    want = O.kv_skip_cache_all(cache, m)
    R = want.shape[-2]
    mask = torch.from_numpy(m).cuda()
    idx = torch.empty(T, dtype=torch.int32, device="cuda")
    nret = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(B.skipffn_compact_workspace_bytes(T), 16), dtype=torch.uint8, device="cuda")
    B.skipffn_compact(mask, idx, nret, None, ws)
    src = to_dev_bf16(cache)
    rcap = T if (cap == "prefill" or not r_host) else R
    dst = torch.full(lead + (rcap, D), -1.0, dtype=torch.bfloat16, device="cuda")
    B.skipffn_kv_compact(src, dst, idx, R if r_host else None, num_retained=nret)
    torch.cuda.synchronize()
    got = bits_of(dst)
    assert np.array_equal(got[..., :R, :], want)
    # rows past R are left as they were
    assert np.all(got[..., R:, :] == bits_of(torch.full((1,), -1.0, dtype=torch.bfloat16))[0])


GAIN_CASES = [
    W.small(C=512, I=1368, visual=(300, 411), text=(20, 35), keep=(130, 212), seed=41, name="gain-2tiles"),
    W.small(C=264, I=520, visual=(700,), text=(9,), keep=(600,), seed=42, name="gain-odd-dims"),
    W.small(C=1024, I=256, visual=(64,), text=(1,), keep=(0,), seed=43, name="gain-one-row"),
    W.small(C=4104, I=128, visual=(40,), text=(3,), keep=(19,), seed=44, name="gain-wide-row"),   # C > 4096: streaming path
    W.small(C=264, I=128, visual=(300,), text=(6,), keep=(122,), seed=46, name="gain-32-strips"),  # the last in the small column sum
    W.small(C=264, I=128, visual=(300,), text=(7,), keep=(122,), seed=47, name="gain-33-strips"),
]


@pytest.mark.parametrize("w", GAIN_CASES, ids=lambda w: w.name)
@pytest.mark.parametrize("with_gain", [True, False], ids=["gain", "unit-gain"])
def test_rmsnorm_gain_gradient(w, with_gain):
    """d_rms_gain against the oracle (the gradient at g = 1 when no gain tensor is given);
    asking for it must not change dX; accumulate adds to what is there; R on the device."""
    p = Problem(w, unit_gain=not with_gain, with_gain_tensor=with_gain)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    idx = bo["idx"]
    _, bufs = gpu_forward(p)
    gh0, _ = gpu_backward(p, bufs)
    dgain = torch.full((w.C,), float("nan"), dtype=torch.float32, device="cuda")
    gh1, _ = gpu_backward(p, bufs, dgain=dgain)
    got = dgain.double().cpu().numpy()
    assert rel_l2(got, bo["dgain"]) < REL_L2_TOL
    assert rel_l2(f64_of(gh1)[idx], f64_of(gh0)[idx]) < 1e-6      # same sums, same order
    # deterministic: a second run gives the same bits
    dgain2 = torch.zeros_like(dgain)
    gpu_backward(p, bufs, dgain=dgain2)
    assert torch.equal(dgain, dgain2)
    # accumulate
    acc = torch.ones_like(dgain)
    dwa = [torch.zeros((w.I, w.C), dtype=torch.bfloat16, device="cuda"),
           torch.zeros((w.I, w.C), dtype=torch.bfloat16, device="cuda"),
           torch.zeros((w.C, w.I), dtype=torch.bfloat16, device="cuda")]
    gpu_backward(p, bufs, flags=B.FLAG_DW_ACCUMULATE, dw=dwa, dgain=acc)
    assert rel_l2(acc.double().cpu().numpy() - 1.0, bo["dgain"]) < REL_L2_TOL
    # R read on the device
    _, bufs_d = gpu_forward(p, R_host=False)
    dgain_d = torch.full((w.C,), float("nan"), dtype=torch.float32, device="cuda")
    gpu_backward(p, bufs_d, R_host=False, dgain=dgain_d)
    assert rel_l2(dgain_d.double().cpu().numpy(), bo["dgain"]) < REL_L2_TOL


def test_gain_gradient_with_nothing_retained_is_zero():
    w = W.small(C=256, I=512, visual=(50,), text=(0,), keep=(0,), seed=45, name="gain-empty")
    p = Problem(w)
    _, bufs = gpu_forward(p)
    dgain = torch.full((w.C,), 7.0, dtype=torch.float32, device="cuda")
    gpu_backward(p, bufs, dgain=dgain)
    assert torch.count_nonzero(dgain).item() == 0


TINY = [
    W.small(C=8, I=8, visual=(2,), text=(1,), keep=(0,), seed=71, name="tiny-8-8-one-row"),
    W.small(C=8, I=16, visual=(5,), text=(0,), keep=(5,), seed=72, name="tiny-8-16-all-kept"),
    W.small(C=24, I=8, visual=(70,), text=(3,), keep=(33,), seed=73, name="tiny-24-8"),
    W.small(C=8200, I=16, visual=(9,), text=(0,), keep=(4,), seed=74, name="wide-8200-16"),   # C beyond the register-resident row paths
]


@pytest.mark.parametrize("w", TINY, ids=lambda w: w.name)
def test_smallest_and_widest_shapes(w):
    """The minimum widths the interface allows (8), a single retained row, and a hidden size
    beyond the register-resident row kernels (streaming paths of RMSNorm forward/backward)."""
    p = Problem(w, unit_gain=False, with_gain_tensor=True)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    idx = fo["idx"]
    sk = p.mask != 0
    out, bufs = gpu_forward(p, flags=B.FLAG_NO_RESIDUAL)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    fo_nr = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps, no_residual=True)
    assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo_nr["out_bits"][idx])) < REL_L2_TOL
    out, bufs = gpu_forward(p)
    assert rel_l2(O.bf16_bits_to_f64(bits_of(out)[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
    dgain = torch.zeros(w.C, dtype=torch.float32, device="cuda")
    gh, dw = gpu_backward(p, bufs, flags=B.FLAG_DW_FP32, dgain=dgain)
    gb = bits_of(gh)
    assert np.array_equal(gb[sk], p.grad[sk])
    assert rel_l2(O.bf16_bits_to_f64(gb[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        assert rel_l2(t.double().cpu().numpy(), bo[k]) < REL_L2_TOL, k
    assert rel_l2(dgain.double().cpu().numpy(), bo["dgain"]) < REL_L2_TOL



@pytest.mark.parametrize("R", [1, 63, 64, 65, 127, 128, 129, 191, 255, 256, 257])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
@pytest.mark.parametrize("C,I", [(520, 1368), (1024, 1368), (2048, 2816)],
                         ids=["C520", "C1024", "C2048"])
def test_row_counts_around_the_tile_heights(R, r_host, C, I):
    """Row counts around 64, 128, 192 and 256, the heights of the tiles of all rows (257 is the first count on two of
    them), with split-K partial sums for the down projection and, from 65 to 256 rows at C = 2048, for gate/up; 1 to 64 rows
    run on the register path.  With the count on the device the row bound is T, which selects the
    variant."""
    visual = R - 7 if R > 7 else R
    text = R - visual
    T_pad = 40 if r_host else 0          # R-device: keep T (the bound) within the same variant
    w = W.small(C=C, I=I, visual=(visual + T_pad,), text=(text,), keep=(visual,), seed=300 + R,
                name=f"rows-{R}")
    assert w.R == R
    print(f"tile heights R={R} T={w.T} r_host={r_host}", flush=True)
    p = Problem(w, unit_gain=False, with_gain_tensor=True)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    fo_nr = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    for saved in (False, True):
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved, flags=B.FLAG_NO_RESIDUAL)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo_nr["out_bits"][idx])) < REL_L2_TOL
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved, inplace=True)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert rel_l2(f64_of(sv[k]), fo[k]) < REL_L2_TOL, k
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain, w.eps)
    gh, dw = gpu_backward(p, bufs, R_host=r_host)
    assert rel_l2(O.bf16_bits_to_f64(bits_of(gh)[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        assert rel_l2(f64_of(t), bo[k]) < REL_L2_TOL, k


@pytest.mark.parametrize("R_max", [300, 2000])
def test_buffers_sized_for_a_larger_row_bound(R_max):
    """Buffers sized once for R_max rows serve a call with fewer rows (here a count that takes one tile of all
    rows and more K splits than the bound's own configuration would)."""
    w = W.small(C=520, I=1368, visual=(200,), text=(13,), keep=(87,), seed=55, name="bound")
    p = Problem(w)
    bufs = B.SkipFFNBuffers(w.T, R_max, w.C, w.I, training=True)
    B.skipffn_compact(p.d_mask, bufs.idx, bufs.num_retained, None, bufs.compact_ws)
    out = p.d_hidden.clone()
    B.skipffn_forward(out, out, bufs.idx, w.R, p.d_wg, p.d_wu, p.d_wd, eps=w.eps, saved=bufs.saved,
                      workspace=bufs.fwd_ws)
    gh = p.d_grad.clone()
    dw = [torch.empty((w.I, w.C), dtype=torch.bfloat16, device="cuda"),
          torch.empty((w.I, w.C), dtype=torch.bfloat16, device="cuda"),
          torch.empty((w.C, w.I), dtype=torch.bfloat16, device="cuda")]
    B.skipffn_backward(gh, gh, bufs.idx, w.R, p.d_wg, p.d_wu, p.d_wd, bufs.saved, *dw, eps=w.eps,
                       workspace=bufs.bwd_ws)
    torch.cuda.synchronize()
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, None, w.eps)
    idx = fo["idx"]
    assert rel_l2(O.bf16_bits_to_f64(bits_of(out)[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
    assert rel_l2(O.bf16_bits_to_f64(bits_of(gh)[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        assert rel_l2(f64_of(t), bo[k]) < REL_L2_TOL, k


@pytest.mark.parametrize("R", [257, 300, 384, 385, 512 + 1, 512 + 128, 768 + 100])
@pytest.mark.parametrize("I", [1368, 8264], ids=["tiles-of-all-rows", "core"])
def test_last_tile_row_of_at_most_128_rows(R, I):
    """Row counts that leave 1 to 129 rows past a multiple of 256.  The wide layer (more gate/up tiles than CUs) runs its
    gate/up GEMM on tiles of 128 rows (257, 300, 384, 868), 192 (385, 513) or 256 (640), the last row of them cut off or
    whole.  The narrower layer runs on several tiles of all rows, the last one cut off.  Every row is checked on its
    own, forward and backward.  The intermediate width leaves a ragged column tile too."""
    from helpers import max_slice_rel_l2
    w = W.small(C=520, I=I, visual=(R + 30,), text=(9,), keep=(R - 9,), seed=900 + R, name=f"tail-{R}")
    assert w.R == R
    print(f"tail row R={R} T={w.T}", flush=True)
    p = Problem(w)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, None, w.eps)
    idx, sk = fo["idx"], p.mask != 0
    out, bufs = gpu_forward(p, saved=True, inplace=True)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k
    gh, dw = gpu_backward(p, bufs)
    gb = bits_of(gh)
    assert np.array_equal(gb[sk], p.grad[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(gb[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx]), axis=1) < REL_L2_TOL
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        assert rel_l2(f64_of(t), bo[k]) < REL_L2_TOL, k


@pytest.mark.parametrize("R,T", [(1, 2400), (100, 2400), (256, 2400), (257, 2400), (640, 2944), (700, 4400)])
def test_device_row_count_far_below_the_bound(R, T):
    """The tile map is laid over the effective rows: the bound has 10 to 18 tile rows (two or three panels),
    of which one to three are live - with a last row of at most 128 rows, a full one, or one in between.  The layer is
    wide enough for the 256-row tiles of the general core at this bound.  Every row is checked on its own."""
    from helpers import max_slice_rel_l2
    w = W.small(C=520, I=2056, visual=(T - 1,), text=(1,), keep=(R - 1,), seed=4000 + R)
    print(f"device count R={R} bound T={T}", flush=True)
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    out, bufs = gpu_forward(p, R_host=False)
    gx, dw = gpu_backward(p, bufs, R_host=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, None, w.eps)
    idx = fo["idx"]
    assert rel_l2(f64_of(out)[idx], O.bf16_bits_to_f64(fo["out_bits"][idx])) < REL_L2_TOL
    assert rel_l2(f64_of(gx)[idx], O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    assert max_slice_rel_l2(f64_of(out)[idx], O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL
    assert max_slice_rel_l2(f64_of(gx)[idx], O.bf16_bits_to_f64(bo["dx_bits"][idx]), axis=1) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k
    for a, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        assert rel_l2(f64_of(a), bo[k]) < REL_L2_TOL, k
    sk = p.mask != 0
    assert np.array_equal(bits_of(out)[sk], p.hidden[sk])


@pytest.mark.parametrize("R,T,C,I", [(0, 300, 520, 8200), (1, 300, 520, 8200), (64, 400, 520, 8200), (65, 700, 520, 8200),
                                     (129, 700, 1032, 2056), (193, 3000, 1032, 2056), (256, 3000, 520, 8200), (257, 3000, 520, 8200),
                                     (700, 3000, 1032, 2056), (5500, 6000, 520, 8200), (400, 4000, 2056, 1032),
                                     (600, 4000, 2056, 1032), (16450, 16700, 264, 520),
                                     (128, 500, 264, 16520), (129, 500, 264, 16520), (256, 500, 264, 16520)])
def test_every_path_of_a_device_row_count(R, T, C, I):
    """Inference with the count on the device and a bound for which the core runs: tiles of all rows of each height (the smallest
    and largest count of some, no row at all), K cut evenly, balanced (5500 rows) and whole, row counts past the list of
    plans.  Every row is checked on its own: xn, H and out are rounded to bf16, 2^-9 rms each."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(T - 1,), text=(1,), keep=(max(R - 1, 0),), seed=9000 + R)
    print(f"device count R={R} bound T={T} C={C} I={I}", flush=True)
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    if R == 0:
        p.mask[:] = 1
        p.d_mask.fill_(1)
    got = bits_of(gpu_forward(p, R_host=False, saved=False, flags=B.FLAG_NO_RESIDUAL)[0])
    sk = p.mask != 0
    assert np.array_equal(got[sk], p.hidden[sk])
    if R > 0:
        fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps, no_residual=True)
        idx = fo["idx"]
        assert len(idx) == R
        assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL


@pytest.mark.parametrize("R", [1, 15, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("C,I", [(136, 344), (512, 1368), (1032, 2056)], ids=["ragged-k", "whole-k", "batches-and-rest"])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_weights_streamed_to_registers(R, C, I, r_host):
    """A handful of rows: 1, 2 or 4 fragments of 16 rows, K ranges of a wavefront that are empty, shorter than a batch
    of loads, or end inside a k-step, column counts that are no multiple of 16; activations chunk-major (no
    saved buffer) and row-major.  Rows and columns are checked one by one."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + (0 if r_host is False else 23),), text=(1,), keep=(R - 1,), seed=5000 + R,
                name=f"few-{R}")
    assert w.R == R
    print(f"few rows R={R} T={w.T} C={C} I={I} r_host={r_host}", flush=True)
    p = Problem(w, unit_gain=False, with_gain_tensor=True)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    want = O.bf16_bits_to_f64(fo["out_bits"][idx])
    for saved in (False, True):
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved, flags=B.FLAG_NO_RESIDUAL)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        # bf16 rounding of xn, H and out (2^-9 rms each) on one row or one column of few elements
        assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), want, axis=1) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k
    full = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps)
    out, _ = gpu_forward(p, R_host=r_host, saved=False, inplace=True)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(full["out_bits"][idx]), axis=1) < REL_L2_TOL


@pytest.mark.parametrize("R,C,I", [(41, 2056, 7176), (64, 2048, 7168), (65, 264, 328), (128, 640, 1664), (129, 640, 1664),
                                   (192, 264, 328), (193, 136, 2056), (256, 640, 1664), (257, 264, 328), (385, 640, 1664),
                                   (640, 264, 1000),
                                   (300, 4096, 328), (65, 136, 4096), (200, 264, 8192), (256, 136, 12288), (300, 264, 4096)])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_tiles_of_all_rows(R, C, I, r_host):
    """Up to 256 rows in one tile of 64, 128, 192 or 256, more in several (the last one cut off): K ranges of a few slabs (fewer than the ring holds), ragged ones,
    whole ones, one split and several, column tiles that are cut off.  Where K is a multiple of 4096 workgroups start at
    different slabs of their range and wrap around: the whole range of gate/up (C = 4096), ranges of the split down GEMM
    shorter than the ring (I = 4096 at 65 rows), a little longer (8192, 12288) and in two row tiles."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + (0 if r_host is False else 23),), text=(1,), keep=(R - 1,), seed=6000 + R,
                name=f"all-rows-{R}")
    assert w.R == R
    print(f"tiles of all rows R={R} T={w.T} C={C} I={I} r_host={r_host}", flush=True)
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    out, bufs = gpu_forward(p, R_host=r_host, saved=True, flags=B.FLAG_NO_RESIDUAL)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    want = O.bf16_bits_to_f64(fo["out_bits"][idx])
    for axis in (0, 1):                  # every column and every row on its own
        assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), want, axis=axis) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k


@pytest.mark.parametrize("R,C,I", [(70, 136, 24), (66, 264, 3592), (130, 264, 5000), (200, 264, 9000), (256, 136, 14000), (48, 4104, 14344),
                                   (65, 136, 16392), (65, 136, 28680), (300, 136, 3592), (520, 136, 2184)])
@pytest.mark.parametrize("saved", [False, True], ids=["inference", "training"])
def test_gate_up_tile_columns(R, C, I, saved):
    """On 256 compute units: tiles of 16, 24, 40, 56 and 64 columns that one round of them holds, of 40 and 56 in two, of
    32 and 32 in two and three row tiles; the last tile of every row is cut off.  Every column of H is checked on its own."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + 23,), text=(1,), keep=(R - 1,), seed=6400 + R, name=f"columns-{I}")
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    out, bufs = gpu_forward(p, saved=saved, flags=B.FLAG_NO_RESIDUAL)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL
    if saved:
        sv = bufs.saved_views(R)
        for k in ("G", "U", "H"):
            assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=0) < REL_L2_TOL, k


@pytest.mark.parametrize("R", [1, 9, 16, 17])
@pytest.mark.parametrize("C,I", [(2056, 12296), (4104, 8200)], ids=["tiles", "registers-for-down"])
def test_decode_of_a_wide_layer(R, C, I):
    """A layer too wide for the register path of the gate/up GEMM.  Where the down GEMM has a column block for every CU, up to
    16 rows take that path, on the chunk-major result of the tiles; from 17 rows (and with a saved buffer) both run
    on tiles, as both do where the down GEMM is narrow and its K range long."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R,), text=(1,), keep=(R - 1,), seed=7000 + R, name=f"wide-{R}")
    assert w.R == R
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    idx, sk = fo["idx"], p.mask != 0
    want = O.bf16_bits_to_f64(fo["out_bits"][idx])
    for saved in (False, True):
        for r_host in (True, False):
            print(f"wide layer R={R} saved={saved} r_host={r_host}", flush=True)
            got = bits_of(gpu_forward(p, R_host=r_host, saved=saved)[0])
            assert np.array_equal(got[sk], p.hidden[sk])
            assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), want, axis=1) < REL_L2_TOL


@pytest.mark.parametrize("R,C,I,gain", [(1, 136, 344, True), (16, 2056, 520, True), (17, 1024, 1032, True), (64, 520, 344, False),
                                        (33, 2056, 7176, False), (64, 4096, 6600, False), (1, 2064, 12296, False)])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_norm_inside_the_gate_up_gemm(R, C, I, gain, r_host, inplace=False):
    """Without a saved buffer few rows are normalised by the gate/up GEMM, on registers (one, two and four row fragments, K
    ranges that end inside a step) and on 64-row tiles (one row, all of them, ragged K, workgroups that start at different
    slabs): rows 2^-12 to 2^12 times as large as others, one of zeros.  Rows are checked one by one: xn, H and out are
    rounded to bf16, 2^-9 rms each."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + (0 if r_host else min(23, 64 - R)),), text=(1,), keep=(R - 1,), seed=8500 + R, name=f"norm-{R}")
    assert w.R == R and w.T <= 66
    p = Problem(w, unit_gain=not gain, with_gain_tensor=gain)
    scale = 2.0 ** (torch.arange(w.T, device="cuda") * 5 % 25 - 12).float()
    if R > 8:
        scale[int(np.flatnonzero(p.mask == 0)[3])] = 0.0
    p.d_hidden = (p.d_hidden.float() * scale[:, None]).bfloat16()
    p.hidden = bits_of(p.d_hidden)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain if gain else None, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    got = bits_of(gpu_forward(p, R_host=r_host, saved=False, inplace=inplace, flags=B.FLAG_NO_RESIDUAL)[0])
    assert np.array_equal(got[sk], p.hidden[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL


@pytest.mark.parametrize("R,C,I", [(33, 2056, 7176), (64, 4096, 6600), (1, 2064, 12296)])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_norm_inside_the_gate_up_gemm_in_place(R, C, I, r_host):
    """The tiles do it where no skipped rows are copied; out of place (above) these sizes are normalised beside the copies."""
    test_norm_inside_the_gate_up_gemm(R, C, I, False, r_host, inplace=True)


@pytest.mark.parametrize("R,C,I", [(1, 2064, 12296), (64, 4096, 6600), (33, 2056, 7176), (20, 3072, 3072), (48, 1032, 7176), (64, 2048, 2056)])
def test_few_rows_are_not_rounded_after_their_norm(R, C, I):
    """1 / rms is applied to the sums of gate/up, whichever launch forms it: of what is rounded to bf16, up to 1.65e-3 rms of
    its size each (2^-8 / 2 over sqrt(3), by where in a binade it lies up to 1.46 times), H and the output remain: 2.3e-3.  Rounded rows
    add themselves twice, to gate and to up: 3.3e-3 and more."""
    w = W.small(C=C, I=I, visual=(R + 5,), text=(1,), keep=(R - 1,), seed=9200 + R + C, name=f"unrounded-{R}-{C}")
    assert w.R == R
    p = Problem(w)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps, no_residual=True)
    got = bits_of(gpu_forward(p, saved=False, flags=B.FLAG_NO_RESIDUAL)[0])
    assert rel_l2(O.bf16_bits_to_f64(got[fo["idx"]]), O.bf16_bits_to_f64(fo["out_bits"][fo["idx"]])) < 2.8e-3


@pytest.mark.parametrize("R,C,I", [(65, 4096, 8), (100, 4104, 72), (129, 2056, 264), (200, 4096, 520), (256, 3080, 1032),
                                   (9, 12296, 2056)],
                         ids=["one-column-tile", "ragged-k", "cut-off-tiles", "rotated-starts", "256-rows", "chunk-major-h"])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_gate_up_split_along_k(R, C, I, r_host):
    """Layers whose gate/up GEMM has few column tiles and a long K range: K is cut, the sums of gate and up meet in the
    reducing kernel.  One tile cut off at 8 columns, a K range that ends inside a slab, workgroups that start at different
    slabs of their range (C a multiple of 4096), H chunk-major for the register path of the down GEMM (9 rows of a
    layer above its weight limit, without a saved buffer).  Rows are checked one by one, and columns where they have 65
    entries or more: error and value of an entry are independent, so the largest of N relative errors of columns of n
    entries is the whole tensor's (4e-3) times about the root of the 1 - 1/N quantile of F(n, n) - 1.6 at n = 65 and
    N = 4104, but 4 at n = 9 and N = 12296."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + (0 if r_host is False else 23),), text=(1,), keep=(R - 1,), seed=8000 + R,
                name=f"split-gate-up-{R}")
    assert w.R == R
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    want = O.bf16_bits_to_f64(fo["out_bits"][idx])
    for saved in (False, True):
        print(f"split gate/up R={R} T={w.T} C={C} I={I} r_host={r_host} saved={saved}", flush=True)
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved, flags=B.FLAG_NO_RESIDUAL)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        for axis in (0, 1) if R >= 65 else (1,):
            assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), want, axis=axis) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k


@pytest.mark.parametrize("R,C,I", [(300, 16520, 72), (700, 12296, 136), (2305, 4104, 264)],
                         ids=["two-row-tiles", "three-row-tiles", "ten-row-tiles"])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_narrow_intermediate_width_with_many_rows(R, C, I, r_host):
    """More than 256 rows with I far below C: gate/up on several tiles of 256 rows, the down GEMM - more column tiles than
    CUs, a K range of two to five slabs - on the general core with its fused epilogue.  With the count on the device
    the last row tile of the bound is empty or cut off.  Every row is checked on its own."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + (300 if r_host is False else 23),), text=(1,), keep=(R - 1,), seed=9000 + R,
                name=f"short-k-{R}")
    assert w.R == R
    p = Problem(w, unit_gain=True, with_gain_tensor=False)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    want = O.bf16_bits_to_f64(fo["out_bits"][idx])
    for saved in (False, True):
        print(f"narrow I R={R} T={w.T} C={C} I={I} r_host={r_host} saved={saved}", flush=True)
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved, flags=B.FLAG_NO_RESIDUAL)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), want, axis=1) < REL_L2_TOL
    sv = bufs.saved_views(R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k


@pytest.mark.parametrize("R,C,I", [(9, 264, 8200), (17, 264, 8200), (64, 520, 8200), (40, 2056, 1032), (64, 4104, 520)],
                         ids=["9-long-k", "17-long-k", "64-long-k", "40-wide", "64-wide"])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_one_gemm_on_the_register_path(R, C, I, r_host):
    """Each GEMM of the forward pass chooses its path: gate/up on registers and, for a long K range, down on tiles (H
    row-major, normalised rows chunk-major without a saved buffer); or gate/up on tiles and down on registers (H
    chunk-major without a saved buffer).  Rows are checked one by one."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + (0 if r_host is False else 23),), text=(1,), keep=(R - 2 if r_host is False else R - 1,),
                seed=9500 + R, name=f"one-side-{R}")
    p = Problem(w, unit_gain=False, with_gain_tensor=True)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.gain, w.eps, no_residual=True)
    idx, sk = fo["idx"], p.mask != 0
    want = O.bf16_bits_to_f64(fo["out_bits"][idx])
    for saved in (False, True):
        print(f"one register GEMM R={w.R} T={w.T} C={C} I={I} r_host={r_host} saved={saved}", flush=True)
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved, flags=B.FLAG_NO_RESIDUAL)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), want, axis=1) < REL_L2_TOL
    sv = bufs.saved_views(w.R)
    for k in ("G", "U", "H"):
        assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k


@pytest.mark.parametrize("R", [0, 1, 64, 65, 130, 257])
@pytest.mark.parametrize("flags", [0, B.FLAG_DW_FP32, B.FLAG_DW_ACCUMULATE, B.FLAG_DW_FP32 | B.FLAG_DW_ACCUMULATE],
                         ids=["bf16", "fp32", "bf16-add", "fp32-add"])
def test_weight_gradients_of_more_tiles_than_compute_units(R, flags):
    """Every workgroup runs several tiles of dW as one stream of K slabs: 1 slab a tile (the loads run two tiles ahead) to 5,
    cut-off tiles at the right and lower edge, both data types, overwritten and added to; the row count on the device, 0
    included (zeros, or nothing added).  Bound: REL_L2_TOL; where a bf16 gradient is added to, the rounding of the sum with an
    old value of like size (2^-9 of it) is far inside it."""
    C, I = 2056, 8712                                    # 9 x 35 tiles of 256 x 256 for each matrix
    w = W.small(C=C, I=I, visual=(300,), text=(1 if R else 0,), keep=(max(R - 1, 0),), seed=610 + R, name=f"dw-stream-{R}")
    assert w.R == R
    p = Problem(w)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, None, w.eps)
    assert fo["R"] == R
    _, bufs = gpu_forward(p, R_host=False)
    dt = torch.float32 if flags & B.FLAG_DW_FP32 else torch.bfloat16
    rng = np.random.default_rng(R)
    add = bool(flags & B.FLAG_DW_ACCUMULATE)
    old = {}
    for k in ("dw_gate", "dw_up", "dw_down"):
        scale = max(float(np.sqrt(np.mean(bo[k] ** 2))), 1e-3)
        old[k] = torch.from_numpy((rng.standard_normal(bo[k].shape) * scale).astype(np.float32)).to(dt)
    _, dw = gpu_backward(p, bufs, R_host=False, flags=flags, dw=[old[k].cuda() for k in ("dw_gate", "dw_up", "dw_down")])
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        want = bo[k] + (old[k].to(torch.float64).numpy() if add else 0.0)
        got = t.to(torch.float64).cpu().numpy()
        if R == 0:
            assert np.array_equal(got, want), k
            continue
        assert rel_l2(got, want) < REL_L2_TOL, k
        # every row and column: REL_L2_TOL of its own size, plus, with one retained row, where a row of dW_gate is dG_i * xn and
        # a dG_i that cancels to nearly nothing keeps the rounding of its terms, REL_L2_TOL of a typical row times 4 (the
        # factors are normal, of at most 4 standard deviations over these counts).  A wrong tile edge would be off by 1
        for axis in (0, 1):
            err, size = np.linalg.norm(got - want, axis=axis), np.linalg.norm(want, axis=axis)
            assert np.all(err < REL_L2_TOL * (size + 4 * np.sqrt(np.mean(size ** 2)))), (k, axis)


@pytest.mark.parametrize("R,C,I", [(1, 136, 24), (33, 264, 688), (65, 1032, 3592), (300, 1032, 2056), (200, 2056, 5128), (600, 2056, 3080)],
                         ids=["one-tile", "parts-of-a-few-slabs", "8-parts", "two-tile-rows", "two-tiles-of-dw-each", "three-tile-rows"])
@pytest.mark.parametrize("flags", [0, B.FLAG_DW_FP32 | B.FLAG_DW_ACCUMULATE], ids=["bf16", "fp32-add"])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_input_gradient_beside_the_weight_gradients(R, C, I, flags, r_host):
    """dXn and dW_gate, dW_up in one launch: a workgroup for each tile of dW, lists of several (R on the host), K of dXn whole and in
    up to 8 parts, cut-off tiles at every edge, with rows that are skipped; dH in parts where C = 1032 and 2056.  Against the
    oracle, as the launches of their own that the balanced split takes; dW_down, which neither touches, bit for bit."""
    print(f"dxn beside dw R={R} C={C} I={I} flags={flags} r_host={r_host}", flush=True)
    w = W.small(C=C, I=I, visual=(R + 23,), text=(1,), keep=(R - 1,), seed=7700 + R, name=f"dxn-dw-{R}")
    assert w.R == R
    p = Problem(w)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, None, w.eps)
    _, bufs = gpu_forward(p, R_host=r_host)
    dt = torch.float32 if flags & B.FLAG_DW_FP32 else torch.bfloat16
    old = [torch.full(s, 0.5 if flags else float("nan"), dtype=dt, device="cuda") for s in ((I, C), (I, C), (C, I))]
    gh, dw = gpu_backward(p, bufs, R_host=r_host, flags=flags, dw=[t.clone() for t in old])
    gh2, dw2 = gpu_backward(p, bufs, R_host=r_host, flags=flags | B.FLAG_BALANCED_SPLIT, dw=[t.clone() for t in old])
    assert torch.equal(dw[2], dw2[2])
    idx, sk = bo["idx"], p.mask != 0
    for g in (gh, gh2):
        got = bits_of(g)
        assert np.array_equal(got[sk], p.grad[sk])
        assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    for t, k in [*zip(dw, ("dw_gate", "dw_up", "dw_down")), *zip(dw2, ("dw_gate", "dw_up", "dw_down"))]:
        # what was added to, 0.5, leaves a gradient's own digits: fp32 keeps them to 2^-24
        assert rel_l2(f64_of(t) - (0.5 if flags else 0.0), bo[k]) < REL_L2_TOL, k


@pytest.mark.parametrize("R,C,I,gain", [(1, 520, 8, False), (64, 520, 72, True), (65, 776, 264, False), (200, 1032, 3592, True), (300, 1544, 520, False),
                                        (600, 2056, 520, True), (250, 1544, 4000, False)],
                         ids=["one-chunk", "a-whole-tile", "ragged-parts", "two-parts", "two-tile-rows", "beyond-512-rows", "three-parts"])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_dh_in_parts_of_k(R, C, I, gain, r_host):
    """dH as fp32 slabs, the SwiGLU backward and the transposed copies from their sums: tiles of 64 x 64 cut off at every edge, parts of K
    that end inside a slab.  Every row of dX and every column and row of the weight gradients are as the oracle's: dG and dU
    are rounded to bf16, 2^-9 rms each; with one retained row a dG that cancels keeps the rounding of its terms, hence the typical
    size beside its own."""
    print(f"dh in parts R={R} C={C} I={I} gain={gain} r_host={r_host}", flush=True)
    w = W.small(C=C, I=I, visual=(R + 23,), text=(1,), keep=(R - 1,), seed=7900 + R, name=f"dh-parts-{R}")
    assert w.R == R
    p = Problem(w, unit_gain=not gain, with_gain_tensor=gain)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, p.gain if gain else None, w.eps)
    _, bufs = gpu_forward(p, R_host=r_host)
    gh, dw = gpu_backward(p, bufs, R_host=r_host)
    idx, sk = bo["idx"], p.mask != 0
    got = bits_of(gh)
    assert np.array_equal(got[sk], p.grad[sk])
    assert rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(bo["dx_bits"][idx])) < REL_L2_TOL
    for t, k in zip(dw, ("dw_gate", "dw_up", "dw_down")):
        g = f64_of(t)
        assert rel_l2(g, bo[k]) < REL_L2_TOL, k
        for axis in (0, 1):
            err, size = np.linalg.norm(g - bo[k], axis=axis), np.linalg.norm(bo[k], axis=axis)
            assert np.all(err < REL_L2_TOL * (size + 4 * np.sqrt(np.mean(size ** 2)))), (k, axis)


@pytest.mark.parametrize("R,I", [(257, 8264), (385, 8264), (481, 8264), (577, 8264), (673, 8264), (769, 8264), (1400, 12808)])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
@pytest.mark.parametrize("saved", [False, True], ids=["inference", "training"])
def test_gate_up_tile_heights(R, I, r_host, saved):
    """65 tile columns: without a saved buffer tiles of 128, 160, 192, 224, 256 and 128 rows, with one (heights of 64 rows
    only) of 128, 192, 192, 256, 256 and 128; row counts one past a tile's height, where the last is nearly empty.  101
    tile columns and 1400 rows: seven rows of 224-row tiles, or six of 256.
    Every row is checked on its own, the transposed copy bit for bit, zeros up to the next multiple of 64 rows included."""
    from helpers import max_slice_rel_l2
    w = W.small(C=264, I=I, visual=(R + 30,), text=(9,), keep=(R - 9,), seed=3300 + R, name=f"heights-{R}")
    assert w.R == R
    p = Problem(w)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    idx, sk = fo["idx"], p.mask != 0
    out, bufs = gpu_forward(p, R_host=r_host, saved=saved)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL
    if saved:
        sv = bufs.saved_views(R)
        for k in ("G", "U", "H"):
            assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k
        h, ht = bits_of(sv["H"]), bits_of(sv["HT"])
        assert np.array_equal(ht[:, :R], h.T)
        assert not ht[:, R:(R + 63) // 64 * 64].any()


@pytest.mark.parametrize("R,C,I,saved", TWO_PART_GATE_UP, ids=lambda v: str(v))
def test_gate_up_in_two_parts(R, C, I, saved):
    """Rows of 256-row tiles, then one row of 128 to 224 rows in the same launch, one row past the last height, K and the last
    tile column cut off; the row count on the host and on the device.  Every row is checked on its own, the transposed copy
    bit for bit."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + 30,), text=(9,), keep=(R - 9,), seed=3500 + R, name=f"two-parts-{R}")
    assert w.R == R
    p = Problem(w)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    idx, sk = fo["idx"], p.mask != 0
    for r_host in (True, False):
        print(f"two parts R={R} C={C} I={I} saved={saved} R_host={r_host}", flush=True)
        out, bufs = gpu_forward(p, R_host=r_host, saved=saved)
        got = bits_of(out)
        assert np.array_equal(got[sk], p.hidden[sk])
        assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL
        if saved:
            sv = bufs.saved_views(R)
            for k in ("G", "U", "H"):
                assert max_slice_rel_l2(f64_of(sv[k]), fo[k], axis=1) < REL_L2_TOL, k
            h, ht = bits_of(sv["H"]), bits_of(sv["HT"])
            assert np.array_equal(ht[:, :R], h.T)
            assert not ht[:, R:(R + 63) // 64 * 64].any()


@pytest.mark.parametrize("R,C,I", [(257, 1032, 8264), (769, 1032, 8264), (961, 1032, 8264), (1153, 1032, 8264),
                                   (1793, 4104, 72), (1921, 4104, 72), (2401, 4104, 72), (2881, 4104, 72)])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_down_tile_heights(R, C, I, r_host):
    """The down GEMM on 256 compute units: eight K ranges into fp32 slabs, then (I = 72) one with the residual in its epilogue,
    each on tiles of 128, 160, 192 and 224 rows; row counts one past a tile's height, where the last is nearly empty.
    Every row is checked on its own."""
    from helpers import max_slice_rel_l2
    w = W.small(C=C, I=I, visual=(R + 30,), text=(9,), keep=(R - 9,), seed=3400 + R, name=f"down-heights-{R}")
    assert w.R == R
    p = Problem(w)
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    idx, sk = fo["idx"], p.mask != 0
    out, _ = gpu_forward(p, R_host=r_host)
    got = bits_of(out)
    assert np.array_equal(got[sk], p.hidden[sk])
    assert max_slice_rel_l2(O.bf16_bits_to_f64(got[idx]), O.bf16_bits_to_f64(fo["out_bits"][idx]), axis=1) < REL_L2_TOL


@pytest.mark.parametrize("R", [1, 64, 65, 200, 300, 773, 1400])
@pytest.mark.parametrize("r_host", [True, False], ids=["R-host", "R-device"])
def test_weights_that_are_not_finite_stay_in_their_columns(R, r_host):
    """An infinite weight makes a column of H infinite (here in every row: its gate and the weighted activation are positive),
    a NaN makes one NaN.  Past the row count the transposed copy is zero all the same, so the gradient of an infinite column
    is infinite where it has one sign in every row, and the other columns are as ever."""
    C, I, c_in, i_inf, i_nan = 264, 8264, 17, 4101, 133
    w = W.small(C=C, I=I, visual=(R + 30,), text=(1,), keep=(R - 1,), seed=3600 + R, name=f"non-finite-{R}")
    assert w.R == R
    p = Problem(w)
    p.hidden[:, c_in] &= 0x7FFF                          # positive activations in column c_in, gradients in column 0
    p.grad[:, 0] &= 0x7FFF
    p.wg[i_inf, :] = 0
    p.wg[i_inf, c_in] = 0x3F80                           # gate = that activation
    fo = O.skipffn_forward(p.hidden, p.mask, p.wg, p.wu, p.wd, None, w.eps)
    bo = O.skipffn_backward(p.hidden, p.mask, p.wg, p.wu, p.wd, p.grad, None, w.eps)
    p.wu[i_inf, c_in] = 0x7F80                           # infinity
    p.wg[i_nan, c_in] = 0x7FC0                           # NaN
    p.d_hidden, p.d_grad, p.d_wg, p.d_wu = (to_dev_bf16(x) for x in (p.hidden, p.grad, p.wg, p.wu))
    assert np.all(p.hidden[fo["idx"], c_in] != 0) and np.all(p.grad[fo["idx"], 0] != 0)
    _, bufs = gpu_forward(p, R_host=r_host)
    _, dw = gpu_backward(p, bufs, R_host=r_host)
    ht = bits_of(bufs.saved_views(R)["HT"])
    assert not ht[:, R:(R + 63) // 64 * 64].any()
    assert np.all(ht[i_inf, :R] == 0x7F80)
    got = f64_of(dw[2])
    assert got[0, i_inf] == np.inf
    assert np.isnan(got[:, i_nan]).all()
    finite = np.delete(np.arange(I), [i_inf, i_nan])
    assert rel_l2(got[:, finite], bo["dw_down"][:, finite]) < REL_L2_TOL
