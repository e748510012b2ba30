"""Work splits of few-row plans that leave part of the GPU idle: shorter
context and decode chunks, against the oracle; and which problems the
allocation-free entry point takes: those whose partials fit its scratch."""
import ctypes
import random

import pytest

import oracle
import paper_2403_08845_amd as bif
import workloads

from .parity import assert_parity


def _ceil(a, b):
    return -(-a // b)


def _coarse_bytes(b, h, g, d, m_c, m_d):
    """Workspace of the longest few-row chunks (context 1024..2048 keys, a
    quarter of the context; decode chunks halved down to 128 keys)."""
    p, M, units = h // g, b * (h // g), b * g
    assert M <= 64
    ctx = min(2048, max(1024, 128 * _ceil(_ceil(m_c, 4), 128)))
    dec = min(1024, max(128, 128 * _ceil(m_d, 128)))
    while dec > 128 and units * _ceil(m_d, dec) < 128:
        dec //= 2
    rows = (g * _ceil(m_c, ctx) * M, units * _ceil(m_d, 32 * _ceil(dec, 32)) * 4 * p)
    off = 0
    for r in rows:
        for size in (r * d * 4, r * 8):
            off = 256 * _ceil(off + size, 256)
    return 256 * _ceil(off + 4, 256)


def _noalloc_status(b, h, g, d, m_c, m_d, n=1, kv="bf16"):
    """Status of an allocation-free call with an unaligned pointer: ESCRATCH, or
    for a problem that fits whatever the later argument checks say."""
    fake = ctypes.c_void_p(256)
    dims = bif.noalloc_dims(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated")
    return bif.lib().bifattn_decode_noalloc(ctypes.byref(dims), ctypes.c_void_p(8), fake, fake,
                                            fake, fake, fake, None, None, fake, None)


def test_noalloc_takes_the_problems_whose_longest_chunks_fit():
    """What fits with the longest chunks is taken whatever the plan's own; of
    few-row plans, whose own chunks are no longer, nothing else is."""
    rng = random.Random(4)
    seen = {True: 0, False: 0}
    for _ in range(4000):
        p = rng.choice((1, 2, 4, 8))
        b = rng.randint(1, 64 // p)
        g = rng.randint(1, 1200)
        d = rng.choice((64, 128))
        m_c = rng.choice((rng.randint(1, 300), rng.randint(300, 9000)))
        m_d = rng.randint(1, 1100)
        if m_c + m_d > 60000:
            continue
        need = _coarse_bytes(b, g * p, g, d, m_c, m_d)
        if not (40 << 20) < need < (90 << 20):
            continue
        st = _noalloc_status(b, g * p, g, d, m_c, m_d)
        fits = need <= bif.NOALLOC_SCRATCH_BYTES
        if fits or b * p <= 32:
            assert (st == bif.ESCRATCH) == (not fits), (b, g, p, d, m_c, m_d, need, st)
        seen[fits] += 1
    assert min(seen.values()) > 20, seen


@pytest.mark.parametrize("case", [
    # b, h, g, d, m_c, m_d, n, kv: two thirds of the scratch or less with the
    # plan's own chunks, more than all of it with others that nothing would run
    (64, 169, 169, 128, 37728, 112, 1, "int4"),
    (187, 61, 61, 128, 1382, 14, 2, "int8"),
    (1491, 6, 3, 128, 856, 30, 2, "bf16"),
    (60, 720, 180, 64, 816, 116, 1, "bf16"),
    (37, 400, 400, 64, 42654, 0, 1, "fp8_e4m3"),
], ids=lambda c: "b%d_h%d_g%d_d%d_mc%d_md%d_n%d_%s" % c)
def test_noalloc_takes_a_problem_that_fits(case):
    assert _noalloc_status(*case) != bif.ESCRATCH


@pytest.mark.parametrize("g", [1, 2, 85, 128, 255, 256, 257, 270, 298, 299, 600])
@pytest.mark.parametrize("p", [1, 8, 33])
def test_splits_of_any_number_of_groups(g, p):
    """Groups around the number of CUs, context lengths around the chunk bounds."""
    for m_c in (1, 200, 256, 257, 300, 511, 513, 1000, 2049, 9000):
        for b in (1, 3, 40):
            assert _noalloc_status(b, g * p, g, 128, m_c, 16) != bif.OK  # no crash: EALIGN, EHIP ...


def test_noalloc_refuses_what_cannot_fit():
    # the outputs' own partials: 64 rows of 4000 groups, one split, four decode waves
    assert _noalloc_status(64, 4000, 4000, 128, 100, 100) == bif.ESCRATCH


@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # b, h, g, d, m_c, m_d, n, kv
    (2, 32, 8, 128, 3001, 200, 1, "bf16"),   # 256-key chunks, the last one short
    (3, 16, 4, 64, 257, 40, 2, "bf16"),      # one key in the second chunk
    (1, 4, 1, 128, 1, 1, 1, "bf16"),         # the smallest
    (16, 8, 4, 128, 5000, 300, 1, "int8"),   # 256-key chunks, one decode chunk of 384
    (8, 32, 8, 128, 6000, 1000, 1, "bf16"),  # 32 rows per group, two decode chunks
    (1, 64, 1, 128, 3000, 100, 1, "bf16"),   # 64 rows of one unit
    (4, 40, 40, 128, 1300, 600, 1, "int4"),
    (9, 32, 32, 64, 2100, 30, 1, "fp8_e4m3"),
], ids=lambda c: "b%d_h%d_g%d_d%d_mc%d_md%d_n%d_%s" % c)
def test_short_chunks_match_the_oracle(case):
    import torch
    from .gpu_util import to_device
    b, h, g, d, m_c, m_d, n, kv = case
    x = workloads.make_inputs(b, h, g, d, m_c, m_d, seed=1900 + m_c, ragged=True, n=n, kv=kv,
                              poison_tail=True)
    dev = to_device(x)
    outs = []
    with bif.Plan(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated") as plan:
        info = plan.info()
        print(f"[case] {case} {info}", flush=True)
        assert info["ctx_kernel"] == 0 and info["ctx_keys_per_block"] <= 1024
        for call in (lambda *a: bif.bifattn_decode_scaled(plan, *a),
                     lambda *a: bif.bifattn_decode_noalloc(
                         bif.noalloc_dims(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated"), *a)):
            out = torch.full(tuple(x["q"].shape), float("nan"), dtype=torch.float32, device="cuda")
            call(dev["q"], dev["Kc"], dev["Vc"], dev["Kd"], dev["Vd"], dev["lens"],
                 dev["k_scale"], dev["v_scale"], out)
            torch.cuda.synchronize()
            outs.append(out)
    assert torch.equal(*outs)
    assert_parity(outs[0].cpu().double().numpy(), oracle.attention(**x), str(case), x=x)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # b, h, g, d, m_c, m_d, n, kv
    (33, 32, 1, 128, 2000, 64, 1, "bf16"),     # two query tiles per unit, an odd work-group count
    (17, 48, 3, 128, 777, 300, 1, "bf16"),     # 272 rows per group, one idle row block wave
    (19, 32, 8, 128, 1500, 90, 1, "bf16"),     # 76 rows per group: four-wave work-groups
    (33, 16, 1, 128, 900, 1100, 1, "fp8_e4m3"),  # two decode chunks
    (13, 20, 4, 128, 640, 70, 4, "int8"),      # tokens
    (65, 8, 8, 128, 3000, 5, 1, "int4"),       # one decode tile
    (70, 4, 1, 128, 130, 1, 1, "bf16"),        # a second key chunk of two keys
    (33, 4, 4, 128, 500, 60, 1, "bf16"),       # 33 rows per group: one row in the second wave
    (16, 4, 1, 128, 64, 40, 1, "int8"),        # 64 rows, one stage
    (33, 2, 2, 64, 700, 33, 1, "bf16"),        # d = 64: four waves,
    (50, 24, 2, 64, 1111, 130, 1, "bf16"),     # three row blocks or more, an idle wave
    (128, 32, 1, 64, 9000, 64, 1, "bf16"),     # eight waves, two query tiles per unit
    (64, 32, 2, 64, 9001, 40, 1, "fp8_e4m3"),
    (64, 32, 2, 64, 9001, 40, 1, "int8"),
    (64, 32, 2, 64, 9001, 40, 2, "int4"),
    (20, 8, 4, 64, 1, 3, 1, "int4"),           # one context key
], ids=lambda c: "b%d_h%d_g%d_d%d_mc%d_md%d_n%d_%s" % c)
def test_many_rows_in_one_launch_equal_two(case, monkeypatch):
    """The decode work-groups in the 32x32 context kernel's launch: the same
    bits as in a launch of their own, the same as without a plan, and the
    oracle's result."""
    import torch
    from .gpu_util import to_device
    b, h, g, d, m_c, m_d, n, kv = case
    x = workloads.make_inputs(b, h, g, d, m_c, m_d, seed=2000 + m_c, ragged=True, n=n, kv=kv,
                              poison_tail=True)
    dev = to_device(x)
    args = [dev[k] for k in ("q", "Kc", "Vc", "Kd", "Vd", "lens", "k_scale", "v_scale")]
    outs = []

    def run(call):
        outs.append(torch.full(tuple(x["q"].shape), float("nan"), dtype=torch.float32, device="cuda"))
        call(*args, outs[-1])
        torch.cuda.synchronize()

    dims = bif.noalloc_dims(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated")
    for fork in ("1", "0"):
        monkeypatch.setenv("BIFATTN_FORK", fork)
        with bif.Plan(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated") as plan:
            info = plan.info()
            print(f"[case] {case} {info}", flush=True)
            assert info["ctx_kernel"] == 2 and info["side_stream"] == 0 and info["fused"] == int(fork)
            run(lambda *a: bif.bifattn_decode_scaled(plan, *a))
    monkeypatch.delenv("BIFATTN_FORK")
    run(lambda *a: bif.bifattn_decode_noalloc(dims, *a))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert_parity(outs[0].cpu().double().numpy(), oracle.attention(**x), str(case), x=x)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # b, h, g, d, m_c, n, kv: rows that fill the combine's work-groups or not,
    # the smallest, the few-row and the many-row kernels
    (1, 1, 1, 128, 1, 1, "bf16"),
    (3, 5, 5, 64, 40, 1, "bf16"),
    (7, 6, 2, 128, 50, 1, "int8"),
    (9, 33, 1, 128, 64, 1, "bf16"),
    (43, 24, 2, 64, 128, 2, "bf16"),
    (77, 40, 1, 64, 100, 1, "int4"),
    (1100, 33, 1, 64, 64, 1, "bf16"),    # many rows, of units past 32
], ids=lambda c: "b%d_h%d_g%d_d%d_mc%d_n%d_%s" % c)
def test_one_partial_per_row(case):
    """A context's one split without decode rows, whose combine has a kernel of
    its own; a scale that is not positive is flagged there too."""
    import torch
    from .gpu_util import to_device
    b, h, g, d, m_c, n, kv = case
    x = workloads.make_inputs(b, h, g, d, m_c, 0, seed=2500 + m_c, n=n, kv=kv)
    dev = to_device(x)
    with bif.Plan(b, h, g, d, m_c, 0, n=n, kv=kv, path="bifurcated") as plan:
        info = plan.info()
        print(f"[case] {case} {info}", flush=True)
        assert info["ctx_splits"] == 1 and info["dec_splits"] == 0
        out = torch.full(tuple(x["q"].shape), float("nan"), dtype=torch.float32, device="cuda")
        args = [dev[k] for k in ("q", "Kc", "Vc", "Kd", "Vd", "lens", "k_scale", "v_scale")]
        bif.bifattn_decode_scaled(plan, *args, out)
        assert bif.bifattn_plan_status(plan) == bif.OK
        assert_parity(out.cpu().double().numpy(), oracle.attention(**x), str(case), x=x)
        if kv != "bf16":
            args[7] = args[7].clone()
            args[7][-1] = 0.0
            bif.bifattn_decode_scaled(plan, *args, out)
            assert bif.bifattn_plan_status(plan) == bif.ESCALE


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 1536, 32, 128, 3079, 1024), (1, 512, 8, 128, 30000, 64),
                                   (1, 2560, 64, 64, 1833, 512)])
def test_four_query_tiles_leave_work_groups_for_the_decode_part(shape):
    """With 33 to 64 query rows in one unit a work-group fills a CU: the chunks of
    a step that fits the GPU leave an eighth of the CUs to the decode part."""
    with bif.Plan(*shape) as plan:
        info = plan.info()
        assert info["ctx_kernel"] == 0 and info["ctx_blocks"] <= 224


@pytest.mark.gpu
def test_many_row_splits_use_the_slots_there_are():
    """Three four-wave work-groups of d = 64 fit a CU, two of d = 128; a last round
    of few work-groups, or CUs of which some hold two and most one, are avoided."""
    def blocks(*shape, **kw):
        with bif.Plan(*shape, **kw) as plan:
            info = plan.info()
            print(f"[case] {shape} {info}", flush=True)
            assert info["ctx_kernel"] == 2
            return info["ctx_blocks"]
    assert 384 < blocks(40, 40, 40, 64, 12000, 100) <= 768       # one row block: 320 -> 480 or so
    assert blocks(27, 16, 8, 128, 35226, 0, n=2) <= 256           # was 296: 44.0 us, now 36.2
    assert 512 < blocks(43, 2048, 32, 64, 919, 0, kv="int4") <= 768  # was two rounds of eight waves


@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # b, h, g, d, m_c, m_d, n, kv: 65 to 80 MiB of partials with the plan's own
    # splits, 43 to 55 with longer chunks
    (130, 256, 8, 64, 9303, 32, 1, "int4"),
    (30, 536, 67, 64, 8851, 5, 2, "int8"),
    (52, 300, 60, 128, 14829, 11, 1, "int8"),
], ids=lambda c: "b%d_h%d_g%d_d%d_mc%d_md%d_n%d_%s" % c)
def test_noalloc_with_longer_chunks(case):
    """A problem whose partials pass the scratch with its plan's splits and fit it
    with longer chunks: sampled rows against the oracle, every row against the
    plan's result (the two round their weights apart: 2^-9 / sqrt(3) each)."""
    import numpy as np
    import torch
    from .gpu_util import sample_rows, to_device
    b, h, g, d, m_c, m_d, n, kv = case
    rng = np.random.default_rng(2600 + m_c)
    cols, std = (d // 2, 21.25 ** 0.5) if kv == "int4" else (d, 73.9)  # of uniform codes
    codes = lambda *s: rng.integers(0, 256, (*s, cols), dtype=np.uint8)
    q = rng.standard_normal((b, h, d) if n == 1 else (b, h, n, d), dtype=np.float32)
    x = dict(q=workloads.f32_to_bf16_bits(q), Kc=codes(g, m_c), Vc=codes(g, m_c),
             Kd=codes(b, g, m_d), Vd=codes(b, g, m_d),
             lens=rng.integers(n, m_d + 1, b).astype(np.int32), kv=kv,
             k_scale=np.full(g, 1 / std, np.float32), v_scale=np.full(g, 1 / std, np.float32))
    dev = to_device(x)
    args = [dev[k] for k in ("q", "Kc", "Vc", "Kd", "Vd", "lens", "k_scale", "v_scale")]
    outs = [torch.full(tuple(x["q"].shape), float("nan"), device="cuda") for _ in range(2)]
    with bif.Plan(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated") as plan:
        info = plan.info()
        print(f"[case] {case} {info}", flush=True)
        rows = b * (h // g) * n * g
        parts = info["ctx_splits"] + info["dec_splits"]
        assert rows * parts * (d + 2) * 4 > bif.NOALLOC_SCRATCH_BYTES
        bif.bifattn_decode_scaled(plan, *args, outs[0])
        torch.cuda.synchronize()
    dims = bif.noalloc_dims(b, h, g, d, m_c, m_d, n=n, kv=kv, path="bifurcated")
    bif.bifattn_decode_noalloc(dims, *args, outs[1])
    torch.cuda.synchronize()
    assert bool(torch.isfinite(outs[1]).all())
    rel = float((outs[0] - outs[1]).norm() / outs[0].norm())
    assert 0 < rel < 4e-3, rel
    ri, rj = sample_rows(b, h, x["lens"], 24, seed=7)
    rt = np.arange(ri.size, dtype=np.int32) % n
    out = outs[1].cpu().double().numpy().reshape(b, h, n, d)[ri, rj, rt]
    assert_parity(out, oracle.attention_rows(**x, rows_i=ri, rows_j=rj, rows_t=rt), str(case), x=x)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,n", [((2, 80, 40, 128, 10456, 116), 4), ((3, 40, 40, 128, 8792, 14), 1),
                                     ((4, 32, 32, 128, 3174, 683), 1), ((2, 96, 24, 64, 16186, 486), 2)])
def test_few_row_context_work_groups_fill_whole_cus(shape, n):
    """Not a few more context work-groups than CUs (160 to 280 of them with the
    even share alone)."""
    with bif.Plan(*shape, n=n) as plan:
        info = plan.info()
        assert info["ctx_kernel"] == 0
        assert info["ctx_blocks"] <= 256 or info["ctx_blocks"] > 298, info
