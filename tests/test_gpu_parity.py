"""GPU parity: every stage of the HIP path, called through the C ABI, against the fp64
oracle on the same seeded inputs.

Bars: index maps bit-exact (similarities within 1e-6 of the threshold are counted and
excused); attention mass within 2e-3 elementwise; merged K/V within 2e-3 plus the unit
roundoff of the cache dtype they are stored in (row-normalised), and within one storage ulp
of the exact value up to 2e-5 of the row maximum; singleton sets bit-identical.  Each stage is fed oracle-made
inputs (mass rounded to fp32, index maps), never outputs of the HIP path.
"""
import math
import os
import sys

import numpy as np
import pytest
import torch

from oracle import ref
from paper_2407_08454_amd import binding as kb
from paper_2407_08454_amd import synth

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, file=sys.stderr, flush=True)


def _rand(shape, dtype, seed):
    return synth.to_storage(np.random.default_rng(seed).standard_normal(shape, dtype=np.float32), dtype)


def _slices(seed, B, H, n_list, N, d, G, dtype, rho=None):
    """(B, H) independent slices from the workload generator, right-padded to N."""
    Q = np.empty((B, H * G, N, d), synth.storage_numpy_dtype(dtype))
    K = np.empty((B, H, N, d), Q.dtype)
    V = np.empty_like(K)
    for b in range(B):
        for h in range(H):
            q, k, v, _ = synth.gen_slice(seed, b * H + h, n_list[b], d, G, rho, dtype, N)
            Q[b, h * G:(h + 1) * G], K[b, h], V[b, h] = q, k, v
    return Q, K, V


# ---------------------------------------------------------------------------------------------
# similarities out of the score pass (kvm_attn_mass_sim)
# ---------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype,N,lens,G", [("f16", 700, [700, 333, 0], 2), ("bf16", 700, [641, 700, 1], 1),
                                            ("f32", 300, [300, 77, 0], 2), ("f16", 8200, [8200, 5000, 513], 1),
                                            ("bf16", 8704, [8704, 8193, 64], 2)])
def test_attn_mass_sim_gives_the_scan_s_similarities(dtype, N, lens, G):
    """The column-sum kernels also write the adjacent-key cosines (the split kernel in small launches, in full ones the
    two-block kernel below 8192 tokens and the four-block kernel from there on; the streaming scan for fp32): against
    the oracle's similarities to the bar of the scan, zero at token 0, on padding and around a zero-norm key; the scores
    bit for bit those of kvm_attn_mass; and the sets identified from these similarities are the oracle's.  The rows
    alone, and repeated until the launch is full."""
    B, H = len(lens), 2
    Q, K, V = _slices(51, B, H, lens, N, 128, G, dtype)
    K[0, 1, 40] = 0                                          # a zero-norm key: similarity 0 to both neighbours
    K[0, 0, 31:34] = K[0, 0, 31]                             # identical keys across a 32-row block edge: similarity 1
    full = "attn_colsum_pipe_kernel" if N >= 8192 else "attn_colsum_kernel"
    for copies, kernel in ((1, "attn_colsum_split_kernel"), ({300: 8, 700: 22}.get(N, 3), full)):
        _say(f"mass + similarities in one pass: {dtype} N={N} lens={lens} G={G}, {copies} copies ({kernel})")
        _check_attn_mass_sim(Q, K, dtype, G, lens, copies, kernel)


def _check_attn_mass_sim(Q, K, dtype, G, lens, copies, kernel):
    rows, H, N, _ = K.shape
    Qd, Kd = gu.to_dev(Q, dtype).repeat(copies, 1, 1, 1), gu.to_dev(K, dtype).repeat(copies, 1, 1, 1)
    lens, K, B = lens * copies, np.tile(K, (copies, 1, 1, 1)), rows * copies
    sh = kb.make_shape(Kd, G, gu.lens_dev(lens))
    params = kb.kvm_params_for_budget(0.5)
    ws = torch.empty(max(kb.kvm_workspace_bytes(sh, params), 256), dtype=torch.uint8, device="cuda")
    mass = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    mass2 = torch.full_like(mass, float("nan"))
    sim = torch.full_like(mass, float("nan"))
    kb.kvm_attn_mass(sh, Qd, Kd, mass, ws)
    assert kernel in gu.kernels_of(lambda: kb.kvm_attn_mass_sim(sh, Qd, Kd, mass2, sim, ws))
    assert torch.equal(mass.view(torch.int32), mass2.view(torch.int32))
    m32 = mass.cpu().numpy()
    o = ref.identify_sets(K, m32.astype(np.float64), dtype, params.budget, params.recent_ratio, params.heavy_ratio,
                          params.threshold, True, kb.kvm_out_capacity(sh, params), lens)
    o["cap_rows"] = kb.kvm_out_capacity(sh, params)
    g_sim = sim.cpu().numpy()
    np.testing.assert_allclose(g_sim, o["sim"], atol=2e-6)
    for b, n in enumerate(lens):
        assert (g_sim[b, :, n:] == 0).all() and (n == 0 or (g_sim[b, :, 0] == 0).all())
    assert (g_sim[::rows, 1, 40:42] == 0).all() and (np.abs(g_sim[::rows, 0, 32:34] - 1) <= 2e-6).all()
    # sets from these similarities
    given = kb.KvmParams.from_buffer_copy(params)
    given.sim_given = 1
    cap = kb.kvm_out_capacity(sh, params)
    i32 = dict(dtype=torch.int32, device="cuda")
    out = dict(set_id=torch.full((B, H, N), -7, **i32), set_start=torch.full((B, H, cap + 1), -7, **i32),
               pivot=torch.full((B, H, cap), -7, **i32), n_sets=torch.full((B, H), -7, **i32), status=torch.full((B, H), -7, **i32))
    kb.kvm_identify_sets(sh, given, Kd, mass, out["set_id"], out["set_start"], out["pivot"], out["n_sets"], sim, out["status"], ws)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in out.items()}
    excused, near = gu.compare_maps(g, o, lens, N, params.threshold, "sets from the score pass's similarities")
    _say(f"  slices excused by a similarity at the threshold: {excused} (near-threshold similarities: {near})")


# ---------------------------------------------------------------------------------------------
# (a) aggregated attention mass
# ---------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 31, 63, 64, 65, 257, 600])
def test_mass_small_sizes(dtype, n):
    _say(f"mass dtype={dtype} n={n}")
    Q, K, _ = _slices(11, 1, 3, [n], n, 128, 1, dtype)
    want = ref.attn_mass(Q, K, dtype)
    got = gu.gpu_mass(Q, K, dtype)
    gu.assert_mass_close(got, want, None, n, f"{dtype} n={n}")
    assert got.sum() == pytest.approx(3 * n, rel=1e-4)


@pytest.mark.parametrize("dtype,G", [("bf16", 4), ("f16", 2), ("f32", 4)])
def test_mass_grouped_queries_and_ragged(dtype, G):
    lens = [300, 129, 0, 1, 256]
    N = 320
    _say(f"mass ragged dtype={dtype} G={G} lens={lens} N={N}")
    Q, K, _ = _slices(12, len(lens), 2, lens, N, 128, G, dtype)
    want = ref.attn_mass(Q, K, dtype, G=G, seq_lens=lens)
    got = gu.gpu_mass(Q, K, dtype, G=G, seq_lens=lens)
    gu.assert_mass_close(got, want, lens, N, f"{dtype} G={G} ragged")


def test_mass_config1_and_determinism():
    cfg = synth.CONFIGS[1]
    _say("mass config 1 (N=512 fp32), two runs")
    Q, K, V, _ = synth.gen_config(cfg)
    want = ref.attn_mass(Q, K, "f32")
    got = gu.gpu_mass(Q, K, "f32")
    err = gu.assert_mass_close(got, want, None, 512, "config 1")
    _say(f"  worst relative error {err:.2e}")
    assert np.array_equal(got, gu.gpu_mass(Q, K, "f32"))          # no atomics: bitwise repeatable


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_mass_scores_rising_far_above_the_first_keys(dtype):
    """Scores that grow by hundreds along the sequence: a softmax reference taken from the first
    keys cannot be held (the exponentials overflow), so in a full launch the row statistics have to
    come out of the repeat that updates the maximum at every block.  A small launch does that anyway
    (and adds up the parts of several waves)."""
    n = 700
    _say(f"mass: rising scores, {dtype}")
    rng = np.random.default_rng(12)
    q = rng.standard_normal((1, 3, n, 128)).astype(np.float32)
    k = rng.standard_normal((1, 3, n, 128)).astype(np.float32)
    # head 0: every query and key shares a component that grows with the position
    ramp = np.linspace(0.0, 60.0, n, dtype=np.float32)
    q[0, 0, :, 0] = 40.0
    k[0, 0, :, 0] = ramp
    # head 1: a single late key far above everything before it
    q[0, 1, :, 1] = 30.0
    k[0, 1, 400, 1] = 90.0
    # head 2: all scores zero except two late keys, 127.2 to 127.6 binary orders above the rest and held
    # by different halves of a wave: each half's sum of exponentials is finite, their sum is not
    q[0, 2], k[0, 2] = 0.0, 0.0
    q[0, 2, :, 2] = 30.0
    k[0, 2, 400, 2] = k[0, 2, 404, 2] = 33.355
    Q, K = synth.to_storage(q, dtype), synth.to_storage(k, dtype)
    want = ref.attn_mass(Q, K, dtype)
    for copies, kernels in ((1, ["attn_lse_split_kernel"]), (45, ["attn_lse_kernel", "attn_lse_redo_kernel"])):
        got = gu.gpu_mass(Q, K, dtype, copies=copies, kernels=kernels)
        assert np.isfinite(got).all()
        # the mass sits on few keys here; compare where the oracle's mass is not negligible and
        # require the rest to be small
        big = want > 1e-6
        assert (np.abs(got[big] - want[big]) / want[big]).max() <= gu.TOL
        assert np.abs(got[~big]).max() <= 2e-6 and got.sum() == pytest.approx(3 * n, rel=1e-4)


def test_mass_large_scores_do_not_overflow():
    # keys and queries scaled so that raw scores reach the hundreds: the row maximum must be used
    n = 200
    Q, K, _ = _slices(13, 1, 2, [n], n, 128, 1, "f16")
    Q = (Q.astype(np.float32) * 6).astype(np.float16)
    K = (K.astype(np.float32) * 6).astype(np.float16)
    want = ref.attn_mass(Q, K, "f16")
    for copies, kernels in ((1, ["attn_lse_split_kernel"]), (100, ["attn_lse_kernel"])):
        got = gu.gpu_mass(Q, K, "f16", copies=copies, kernels=kernels)
        # columns that receive next to nothing are compared absolutely
        assert np.isfinite(got).all() and got.sum() == pytest.approx(2 * n, rel=1e-4)
        big = want > 1e-6
        assert (np.abs(got - want)[big] / want[big]).max() <= gu.TOL


def _held_reference_case(dtype, orders, n):
    """Equal queries and, among zero keys, a few whose scores lie `orders` binary orders above theirs (rounded to the type)."""
    q, k = np.zeros((1, 6, n, 128), np.float32), np.zeros((1, 6, n, 128), np.float32)
    q[:, :, :, 2] = 30.0
    top = orders * math.sqrt(128.0) / (30.0 * math.log2(math.e))
    k[0, 0, 300, 2] = top                                     # one wave sees it
    k[0, 1, [200, 300], 2] = top                              # two waves, the others stay with zeros
    k[0, 2, [255, 575], 2] = top, 2 * top                     # again and higher, late
    # one wave sees both, the second on the diagonal of 64 rows that all see it: what was held before is scaled down there
    k[0, 3, [200, 320], 2] = top                              # (blocks 6 and 10 of 32 keys: the same wave of four; the same half of its lanes)
    k[0, 4, [328, 576], 2] = top                              # (blocks 10 and 18: of eight as well)
    k[0, 5, [204, 320], 2] = top                              # (in the two halves of the lanes)
    Q, K = synth.to_storage(q, dtype), synth.to_storage(k, dtype)
    return Q, K, ref.attn_mass(Q, K, dtype)


def _check_held_reference(got, want):
    big = want > 1e-6
    assert np.isfinite(got).all() and (np.abs(got[big] - want[big]) / want[big]).max() <= gu.TOL
    assert np.abs(got[~big]).max(initial=0.0) <= 2e-6


HELD_ORDERS = [40.0, 63.5, 64.5, 95.0, 97.0, 100.0, 126.3, 126.9, 128.5, 300.0]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("orders", HELD_ORDERS)
@pytest.mark.parametrize("n", [600, 2100])                    # four waves a workgroup, eight
def test_mass_split_held_reference(dtype, orders, n):
    """The split row statistics hold a wave's reference from its first block on: late keys around and beyond the 2^96 at
    which a workgroup starts again with the maximum updated, in one wave or in two, after it or on its last block."""
    _say(f"mass, held reference: {dtype} {orders} binary orders, n={n}")
    Q, K, want = _held_reference_case(dtype, orders, n)
    _check_held_reference(gu.gpu_mass(Q, K, dtype, kernels=["attn_lse_split_kernel"]), want)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("orders", HELD_ORDERS)
@pytest.mark.parametrize("n,copies", [(600, 26), (2100, 11)])
def test_mass_full_held_reference(dtype, orders, n, copies):
    """The full row statistics hold the reference of the first 64 keys to the diagonal, and leave a tile whose held sums
    passed 2^96 to the repeat launch."""
    _say(f"mass, held reference in full launches: {dtype} {orders} binary orders, n={n}")
    Q, K, want = _held_reference_case(dtype, orders, n)
    _check_held_reference(gu.gpu_mass(Q, K, dtype, copies=copies, kernels=["attn_lse_kernel", "attn_lse_redo_kernel"]), want)


@pytest.mark.parametrize("G,lens,N,copies", [
    (1, [1], 1, 1), (1, [15], 16, 1), (2, [17, 16, 0], 17, 1), (1, [40, 33, 31], 48, 2), (4, [49, 130], 130, 1), (3, [350, 1, 0, 256], 350, 1),
    (1, [700, 513], 770, 3), (4, [600], 600, 4), (2, [500, 250, 37], 500, 4), (2, [500, 250, 37], 500, 5)])
def test_mass_fp32_smallest_launches(G, lens, N, copies):
    """The fp32 kernels of 16 rows, four and eight waves, alone and with the other pass in the kernels of 32 rows (G > 1 and many
    copies: the row statistics have G times the slices): edges of a 16-row block, padding, heads, against the oracle
    (fp32 sums of N terms: 8 * 2^-24 sqrt(N) of a column's sum, and the exponent's own 1e-5)."""
    _say(f"mass, smallest fp32 launches: G={G} lens={lens} N={N} x{copies}")
    Q, K, _ = _slices(31, len(lens), 1, lens, N, 128, G, "f32")
    got = gu.gpu_mass(Q, K, "f32", G=G, seq_lens=lens, copies=copies, kernels=["attn_lse_split_kernel", "attn_colsum_split_kernel"])
    want = ref.attn_mass(Q, K, "f32", G=G, seq_lens=lens)
    for b, n in enumerate(lens):
        assert (got[b, :, n:] == 0).all()
        assert (np.abs(got[b, :, :n] - want[b, :, :n]) <= (1e-5 + 8 * 2.0 ** -24 * math.sqrt(N)) * want[b, :, :n]).all()


def test_mass_fp32_split_rule():
    """Where the fp32 split launches change kernels: up to 256 blocks of 32 rows 16 rows and eight waves a workgroup, up to 384 blocks
    16 rows and four waves, beyond 32 rows.  One slice repeated: the same bits within a range, other orders of the fp32 sums and
    so other bits on its other side (all three add up the same 1000 terms: 8 * 2^-24 sqrt(N) of a sum, and the exponent's 1e-5)."""
    N = 1000                                                  # 32 blocks a slice
    _say("mass, fp32 split rule")
    Q, K, _ = _slices(37, 1, 1, [N], N, 128, 1, "f32")
    bits = {c: gu.gpu_mass(Q, K, "f32", copies=c, kernels=["attn_lse_split_kernel", "attn_colsum_split_kernel"]) for c in (1, 8, 9, 12, 13, 16)}
    for a, b in ((1, 8), (9, 12), (13, 16)):
        assert np.array_equal(bits[a], bits[b]), (a, b)
    for a, b in ((8, 9), (12, 13), (8, 13)):
        assert not np.array_equal(bits[a], bits[b]), (a, b)
    want = ref.attn_mass(Q, K, "f32")
    for c in bits:
        assert (np.abs(bits[c] - want) <= (1e-5 + 8 * 2.0 ** -24 * math.sqrt(N)) * want).all(), c


@pytest.mark.parametrize("dtype,G,lens,N,copies,kernels", [
    ("f16", 1, [2304, 0, 2048, 1, 1793, 1025, 257, 512], 2304, 7, ["attn_lse_kernel", "attn_colsum_kernel"]),
    ("bf16", 2, [2100, 1800, 1, 0, 700, 2304], 2304, 9, ["attn_lse_kernel", "attn_colsum_kernel"]),
    ("f32", 1, [1200, 0, 1, 1024, 897, 129], 1200, 5, ["attn_lse_kernel", "attn_colsum_kernel"]),
    ("f16", 1, [8704, 0, 4097, 1, 513, 7000], 8704, 3, ["attn_lse_kernel", "attn_colsum_pipe_kernel"])])
def test_mass_tiles_paired_within_a_slice(dtype, G, lens, N, copies, kernels):
    """Full launches pair the long and the short tiles of every slice by its own length: even and odd numbers of tiles, one,
    none.  Against the split kernels, which pair nothing (other order of N fp32 additions: 8 * 2^-24 sqrt(N) of a sum);
    every padded token is a zero."""
    _say(f"mass, paired tiles: {dtype} G={G} lens={lens} N={N} x{copies}")
    Q, K, _ = _slices(29, len(lens), 1, lens, N, 128, G, dtype)
    small = gu.gpu_mass(Q, K, dtype, G=G, seq_lens=lens)
    full = gu.gpu_mass(Q, K, dtype, G=G, seq_lens=lens, copies=copies, kernels=kernels)
    for b, n in enumerate(lens):
        assert (full[b, :, n:] == 0).all() and (full[b, :, :n] > 0).all()
        assert (np.abs(full[b, :, :n] - small[b, :, :n]) <= 8 * 2.0 ** -24 * math.sqrt(N) * small[b, :, :n]).all()


@pytest.mark.parametrize("dtype,G,lens,N,copies", [
    ("f16", 1, [1], 1, 400), ("bf16", 1, [33, 31], 33, 240), ("f32", 1, [65, 32], 65, 80),   # edges of a 32-row block
    ("f16", 2, [97, 64, 0], 97, 140), ("bf16", 4, [300, 129, 0, 1, 256], 320, 50), ("f32", 4, [300, 129, 0, 1, 256], 320, 20),
    ("f16", 1, [2100, 1500, 2049], 2100, 35), ("bf16", 4, [600, 257], 600, 70), ("f32", 2, [257, 600], 600, 20),
    ("f16", 1, [8200, 5000, 513], 8200, 8), ("bf16", 2, [8704, 8193], 8704, 10)])
def test_mass_small_and_full_launches(dtype, G, lens, N, copies):
    """A launch that cannot fill the chip goes to the split kernels (four or eight waves share a row tile), a full one
    to the kernels that stream a tile for 256 rows (512 from 8192 tokens on): the same slices alone and repeated until
    the launch is full, both against the oracle (up to 2200 tokens) and against each other, with the similarities and
    from the caller's row statistics too, on rising scores in one slice.  Between the two only the order of the fp32
    additions differs: N terms, none above the sum, 2^-24 sqrt(N) < 6e-6 of it and 8 times that as the bar."""
    _say(f"mass, small and full launch: {dtype} G={G} lens={lens} N={N} x{copies}")
    B = len(lens)
    Q, K, _ = _slices(23, B, 1, lens, N, 128, G, dtype)
    q0, k0 = synth.to_f64(Q[:1], dtype).astype(np.float32), synth.to_f64(K[:1], dtype).astype(np.float32)
    q0[..., 0], k0[..., 0] = 40.0, np.linspace(0.0, 60.0, N, dtype=np.float32)   # no held maximum fits these
    Q[:1], K[:1] = synth.to_storage(q0, dtype), synth.to_storage(k0, dtype)
    Qd, Kd = gu.to_dev(Q, dtype), gu.to_dev(K, dtype)

    def run(rep):
        q, k = Qd.repeat(rep, 1, 1, 1), Kd.repeat(rep, 1, 1, 1)
        sh = kb.make_shape(k, G, gu.lens_dev(lens * rep))
        ws = torch.empty(max(kb.kvm_workspace_bytes(sh), 256), dtype=torch.uint8, device="cuda")
        out = [torch.full((B * rep, 1, N), float("nan"), dtype=torch.float32, device="cuda") for _ in range(3)]
        kb.kvm_attn_mass_sim(sh, q, k, out[0], out[1], ws)
        if N <= 2200:
            kb.kvm_attn_mass_from_lse(sh, q, k, torch.from_numpy(lse).cuda().repeat(rep, 1, 1), out[2], ws)
        torch.cuda.synchronize()
        for t in out:                                        # every copy the same bits
            assert torch.equal(t.view(torch.int32).view(rep, -1), t.view(torch.int32)[:B].view(1, -1).expand(rep, -1))
        return [t[:B].cpu().numpy() for t in out]

    def close(got, want, tol):
        big = want > 1e-6                                     # (columns of the rising slice that receive next to nothing)
        assert np.isfinite(got).all() and (np.abs(got - want)[big] / want[big]).max() <= tol
        assert not (~big).any() or np.abs(got[~big]).max() <= 2e-6

    if N <= 2200:
        lse = ref.row_lse(Q, K, dtype, G=G, seq_lens=lens).astype(np.float32)
        want = ref.attn_mass(Q, K, dtype, G=G, seq_lens=lens)
    few, full = run(1), run(copies)
    if N <= 2200:
        for got in (few[0], full[0], few[2], full[2]):
            close(got, want, gu.TOL)
    for b, n in enumerate(lens):
        assert (few[0][b, :, n:] == 0).all() and (full[0][b, :, n:] == 0).all()
    # the rising slice's scores reach 200 in units of the exponent: an fp32 rounding of the score is 2^-16 of a term
    if B > 1:
        close(full[0][1:], few[0][1:].astype(np.float64), 5e-5)
    close(full[0], few[0].astype(np.float64), 2e-3)
    np.testing.assert_allclose(full[1], few[1], atol=2e-6)


# slices of a launch -> does the split kernel take the row statistics, the column sums (else the full kernels do)
@pytest.mark.parametrize("dtype,N,G,expect", [
    ("f16", 96, 1, {256: (1, 1), 257: (0, 0)}), ("bf16", 97, 1, {128: (1, 1), 129: (1, 0), 256: (1, 0), 257: (0, 0)}),
    ("f16", 256, 1, {128: (1, 1), 192: (1, 0), 193: (0, 0)}), ("f16", 448, 1, {192: (1, 1), 193: (0, 0)}),
    ("bf16", 512, 1, {160: (1, 1), 161: (0, 0)}), ("f16", 1000, 1, {96: (1, 1), 97: (0, 0)}),
    ("f16", 192, 2, {384: (0, 1), 385: (0, 0)}), ("bf16", 256, 2, {96: (1, 1), 97: (0, 1), 256: (0, 1), 257: (0, 0)}),
    ("f16", 224, 4, {384: (0, 1), 385: (0, 0)}), ("bf16", 256, 4, {320: (0, 1), 321: (0, 0)}),
    ("f16", 1800, 1, {64: (1, 1), 65: (0, 0)}), ("f32", 128, 1, {128: (1, 1), 129: (0, 0)})])
def test_mass_on_both_sides_of_the_split_rule(dtype, N, G, expect):
    """One slice repeated to the numbers of slices where the choice between split and full kernels turns: which kernels
    ran, every copy the same bits, and the oracle's scores."""
    _say(f"mass around the split rule: {dtype} N={N} G={G} {expect}")
    Q, K, _ = _slices(31, 1, 1, [N], N, 128, G, dtype)
    want = ref.attn_mass(Q, K, dtype, G=G)
    for count, (lse, colsum) in expect.items():
        q, k = gu.to_dev(Q, dtype).repeat(count, 1, 1, 1), gu.to_dev(K, dtype).repeat(count, 1, 1, 1)
        sh = kb.make_shape(k, G)
        ws = torch.empty(max(kb.kvm_workspace_bytes(sh), 256), dtype=torch.uint8, device="cuda")
        mass = torch.full((count, 1, N), float("nan"), dtype=torch.float32, device="cuda")
        names = gu.kernels_of(lambda: kb.kvm_attn_mass(sh, q, k, mass, ws))
        assert ("attn_lse_split_kernel" in names, "attn_colsum_split_kernel" in names) == (lse, colsum), (count, names)
        assert torch.equal(mass.view(torch.int32), mass[:1].view(torch.int32).expand(count, 1, N))
        gu.assert_mass_close(mass[:1].cpu().numpy(), want, None, N, f"{count} slices")


def test_maps_of_a_slice_alone_and_in_a_full_launch():
    """Small and full launches add a slice's scores up in different orders, so the last bits of the scores depend on how
    many slices a call covers, and with them a top-k or a pivot where two scores nearly tie.  Nothing else may: both
    launches' maps are what the oracle's rule gives on the scores of that launch, and those agree to their rounding."""
    N, rows, copies = 1000, 4, 25
    _say("maps of a slice alone and in a full launch")
    Q, K, _ = _slices(37, rows, 1, [N] * rows, N, 128, 1, "f16")
    params = kb.kvm_params_for_budget(0.5)
    few = gu.gpu_mass(Q, K, "f16", kernels=["attn_colsum_split_kernel"])
    full = gu.gpu_mass(Q, K, "f16", copies=copies, kernels=["attn_colsum_kernel"])
    assert (np.abs(full - few) / few).max() <= 5e-5          # N terms: see test_mass_small_and_full_launches
    for mass in (few, full):
        g, o = _identify_both(K, mass.astype(np.float64), "f16", params)
        gu.compare_maps(g, o, None, N, params.threshold, "maps on this launch's scores")


@pytest.mark.parametrize("dtype,N,G", [("f16", 97, 2), ("bf16", 200, 1), ("f32", 70, 2), ("bf16", 2016, 1)])
@pytest.mark.parametrize("lengths", ["none", "equal", "different"])
def test_mass_split_launch_of_every_slice_count(dtype, N, G, lengths):
    """The split kernels deal the slices out in turn, or (16-bit types, equal lengths) as one, two, four and whole groups
    of eight (fewer than eight slices from 32 tiles on): every number of slices up to 17 has to give every slice the bits
    it gets alone (no slice left out or taken twice: the outputs start as NaN)."""
    _say(f"mass, 1 to 17 slices: {dtype} N={N} G={G} lengths: {lengths}")
    lens = [N - (3 * (b % 5) if lengths == "different" else 0) for b in range(17)]
    Q, K, _ = _slices(29, 17, 1, lens, N, 128, G, dtype)
    Qd, Kd = gu.to_dev(Q, dtype), gu.to_dev(K, dtype)

    def run(rows):
        q, k = Qd[rows].contiguous(), Kd[rows].contiguous()
        sh = kb.make_shape(k, G, None if lengths == "none" else gu.lens_dev(lens[rows]))
        ws = torch.full((max(kb.kvm_workspace_bytes(sh), 256),), 255, dtype=torch.uint8, device="cuda")
        out = torch.full((2, len(lens[rows]), N), float("nan"), dtype=torch.float32, device="cuda")
        names = gu.kernels_of(lambda: kb.kvm_attn_mass_sim(sh, q, k, out[0].view(-1, 1, N), out[1].view(-1, 1, N), ws))
        assert {"attn_lse_split_kernel", "attn_colsum_split_kernel"} <= names
        return out.view(torch.int32)

    alone = torch.cat([run(slice(b, b + 1)) for b in range(17)], dim=1)
    for count in range(2, 18):
        assert torch.equal(run(slice(0, count)), alone[:, :count]), f"{count} slices"
    gu.assert_mass_close(alone[0].view(torch.float32).cpu().numpy()[:, None], ref.attn_mass(Q, K, dtype, G=G, seq_lens=lens), lens, N)


def _single_pass(Q, K, dtype, G=1, copies=1, sim=False):
    """Scores of `copies` copies of the slices with the workspace of a program that runs the whole pass (all of the same
    length: short sequences then take the single score pass), which come out with the same bits; the kernels' names."""
    Qd, Kd = gu.to_dev(Q, dtype).repeat(copies, 1, 1, 1), gu.to_dev(K, dtype).repeat(copies, 1, 1, 1)
    sh = kb.make_shape(Kd, G)
    ws = torch.full((kb.kvm_workspace_bytes(sh, kb.kvm_params_for_budget(0.5)),), 255, dtype=torch.uint8, device="cuda")
    mass = torch.full((2,) + Kd.shape[:3], float("nan"), dtype=torch.float32, device="cuda")
    if sim:
        names = gu.kernels_of(lambda: kb.kvm_attn_mass_sim(sh, Qd, Kd, mass[0], mass[1], ws))
    else:
        names = gu.kernels_of(lambda: kb.kvm_attn_mass(sh, Qd, Kd, mass[0], ws))
    torch.cuda.synchronize()
    bits = mass[0].view(torch.int32).view(copies, -1)
    assert torch.equal(bits, bits[:1].expand_as(bits))
    return mass[:, :Q.shape[0]].cpu().numpy(), names


# the tiles of 16 and 32 rows and keys, the numbers of waves and of tiles a wave (128, 256, 512, 1024 tokens), the longest rows
@pytest.mark.parametrize("dtype,N,G,copies", [
    ("f16", 1, 1, 1), ("bf16", 31, 3, 1), ("f16", 32, 1, 70), ("f32", 15, 2, 1), ("f32", 17, 1, 66), ("f16", 33, 4, 3), ("bf16", 128, 1, 9),
    ("f16", 129, 2, 1), ("f32", 256, 1, 65), ("f32", 257, 3, 1), ("f16", 256, 1, 64), ("bf16", 257, 1, 2), ("f16", 511, 8, 1), ("f16", 513, 1, 33),
    ("f32", 513, 1, 2), ("bf16", 1000, 4, 1), ("f16", 1024, 1, 65), ("f32", 1025, 1, 2), ("bf16", 1025, 1, 1), ("f16", 2048, 2, 1),
    ("f32", 2049, 1, 1), ("f32", 4096, 1, 1)])
def test_mass_single_pass(dtype, N, G, copies):
    """The scores of short sequences from one score pass, against the oracle (fp32 sums of N terms: 8 * 2^-24 sqrt(N) of a column's
    sum, and the exponent's own 1e-5), against the two passes that the smallest workspace leaves, and the same bits with
    the similarities asked for."""
    _say(f"mass, single pass: {dtype} N={N} G={G} x{copies}")
    Q, K, _ = _slices(41, 2, 1, [N, N], N, 128, G, dtype)
    want = ref.attn_mass(Q, K, dtype, G=G)
    (got, _), names = _single_pass(Q, K, dtype, G, copies)
    assert names == {"attn_single_kernel", "attn_single_sum_kernel"}
    tol = 1e-5 + 8 * 2.0 ** -24 * math.sqrt(N)
    assert (np.abs(got - want) <= tol * want).all()
    two = gu.gpu_mass(Q, K, dtype, G=G, copies=copies)        # (a workspace without the room)
    assert (np.abs(got - two) <= tol * want).all()
    (again, sim), names = _single_pass(Q, K, dtype, G, copies, sim=True)
    assert "attn_single_kernel" in names and "cosine_scan_kernel" in names
    assert np.array_equal(again.view(np.int32), got.view(np.int32))
    cap = kb.kvm_out_capacity(kb.make_shape(gu.to_dev(K, dtype), G), kb.kvm_params_for_budget(0.5))
    np.testing.assert_allclose(sim, ref.identify_sets(K, want, dtype, 0.5, 0.17, 0.12, 0.75, True, cap)["sim"], atol=2e-6)


@pytest.mark.parametrize("dtype,N,G", [("f16", 300, 1), ("bf16", 70, 3), ("f32", 100, 2)])
@pytest.mark.parametrize("slices", [1, 2, 5, 7, 8, 9, 15, 33, 57, 63, 65, 68, 71, 103])
def test_mass_single_pass_of_every_slice_count(dtype, N, G, slices):
    """Whole eights of slices take turns and what is left over goes out before them in fours, twos and ones: every slice gets all of its
    workgroups, with the same bits, and the oracle's scores."""
    _say(f"mass, single pass, {slices} slices: {dtype} N={N} G={G}")
    Q, K, _ = _slices(50, 1, 1, [N], N, 128, G, dtype)
    want = ref.attn_mass(Q, K, dtype, G=G)
    (got, _), names = _single_pass(Q, K, dtype, G, slices)
    assert "attn_single_kernel" in names
    assert (np.abs(got - want) <= (1e-5 + 8 * 2.0 ** -24 * math.sqrt(N)) * want).all()


@pytest.mark.parametrize("dtype,N,G", [("f16", 64, 1), ("bf16", 257, 3), ("f32", 300, 2)])
def test_mass_sim_single_pass_takes_two_launches(dtype, N, G):
    """The similarities come from the launch that adds the column sums up: a scan of its own would cost short sequences more than
    the second score pass that it replaces.  (Results: test_mass_single_pass.)"""
    _say(f"mass and similarities, launches: {dtype} N={N} G={G}")
    Q, K, _ = _slices(42, 1, 2, [N], N, 128, G, dtype)
    _, names = _single_pass(Q, K, dtype, G, sim=True)
    assert names == {"attn_single_kernel", "cosine_scan_kernel"}


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("orders", HELD_ORDERS + [-40.0, -300.0, 1000.0])
def test_mass_single_pass_reference(dtype, orders):
    """Rows whose scores lie far from the reference that the rows before left: the sums that leave 2^-32 .. 2^96 are worked
    out again with a maximum of their own (one slice, one unit of rows a workgroup, and 45, several).  An fp32 rounding
    of a score of `orders` binary orders is 2^-24 of it: the rows' statistics and terms within 4 of those."""
    _say(f"mass, single pass, scores {orders} binary orders off, {dtype}")
    Q, K, want = _held_reference_case(dtype, orders, 600)
    tol = 1e-5 + 4 * abs(orders) * 2.0 ** -24 * math.log(2.0)
    for copies in (1, 45):
        (got, _), names = _single_pass(Q, K, dtype, copies=copies)
        assert "attn_single_kernel" in names and np.isfinite(got).all()
        big = want > 1e-6
        assert (np.abs(got[big] - want[big]) / want[big]).max() <= tol
        assert np.abs(got[~big]).max(initial=0.0) <= 2e-6


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("offset", [-3000.0, -60.0, 60.0, 3000.0])
def test_mass_single_pass_common_offset(dtype, offset):
    """All scores of a row moved by the same amount, and rising scores: the reference moves along.  (Tolerance: the scores'
    own rounding, a few 2^-24 of their size each, sums of 128 products in fp32.)"""
    n = 700
    _say(f"mass, single pass, common offset {offset}, {dtype}")
    rng = np.random.default_rng(3)
    q, k = (rng.standard_normal((1, 2, n, 128)).astype(np.float32) for _ in range(2))
    q[..., 0] = 20.0
    k[:, 0, :, 0] = offset * math.sqrt(128.0) / 20.0
    k[:, 1, :, 0] = np.linspace(0.0, 60.0, n, dtype=np.float32)
    Q, K = synth.to_storage(q, dtype), synth.to_storage(k, dtype)
    want = ref.attn_mass(Q, K, dtype)
    (got, _), names = _single_pass(Q, K, dtype)
    assert "attn_single_kernel" in names and np.isfinite(got).all()
    big = want > 1e-6
    assert (np.abs(got[big] - want[big]) / want[big]).max() <= 1e-5 + 16 * max(abs(offset), 110.0) * 2.0 ** -24
    assert np.abs(got[~big]).max(initial=0.0) <= 2e-6


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("scales", [(1.0, 8.0, 40.0, 0.1), (40.0, 40.0, 40.0, 40.0), (100.0, 1.0, 1.0, 100.0)])
def test_mass_single_pass_heads_of_different_scale(dtype, scales):
    """Query heads whose log-sum-exps lie far apart, and rows of one head that do (scores that spread like N(0, 40^2)), in launches of
    one unit of rows a workgroup and of several.  (Tolerance as for a common offset; scores go up to five times the scale.)"""
    _say(f"mass, single pass, heads scaled by {scales}, {dtype}")
    n, G = 1000, len(scales)
    Q, K, _ = _slices(46, 1, 1, [n], n, 128, G, "f32")
    Q, K = synth.to_storage(Q * np.asarray(scales, np.float32).reshape(1, G, 1, 1), dtype), synth.to_storage(K, dtype)
    want = ref.attn_mass(Q, K, dtype, G=G)
    tol = 1e-5 + 16 * 5 * max(scales) / math.log(2.0) * 2.0 ** -24
    for copies in (1, 9, 300):
        (got, _), names = _single_pass(Q, K, dtype, G, copies=copies)
        assert "attn_single_kernel" in names and np.isfinite(got).all()
        big = want > 1e-6
        assert (np.abs(got[big] - want[big]) / want[big]).max() <= tol
        assert np.abs(got[~big]).max(initial=0.0) <= 2e-6


@pytest.mark.parametrize("dtype,size", [("f16", 6e4), ("f16", 1e4), ("bf16", 1e9), ("f32", 6e4), ("f32", 1e9)])
def test_mass_single_pass_of_very_large_scores(dtype, size):
    """One key and one query so large that every score with them is finite but decides its row alone: weights of one and zero, which
    no rounding of a row's log-sum-exp (2^11 and more at these sizes) may turn into others."""
    _say(f"mass, single pass, a row of {size}, {dtype}")
    n = 300
    rng = np.random.default_rng(51)
    q, k = (rng.standard_normal((1, 2, n, 128)).astype(np.float32) for _ in range(2))
    k[0, 0, n // 4], q[0, 0, n // 2] = size, size
    Q, K = synth.to_storage(q, dtype), synth.to_storage(k, dtype)
    want = ref.attn_mass(Q, K, dtype)
    for copies in (1, 150):
        (got, _), names = _single_pass(Q, K, dtype, copies=copies)
        assert "attn_single_kernel" in names and np.isfinite(got).all()
        big = want > 1e-6
        assert (np.abs(got[big] - want[big]) / want[big]).max() <= 2e-5
        assert np.abs(got[~big]).max(initial=0.0) <= 2e-6


@pytest.mark.parametrize("slices,N,scale", [(2, 1000, 8.0), (1, 500, 4.0), (1, 3000, 4.0)])
def test_mass_single_pass_fp32_is_as_exact_as_the_two_passes(slices, N, scale):
    """Scores of some size, where the rounding of their sums of products shows: the error against the oracle, 2-norm, of the single
    pass and of the two passes that the smallest workspace leaves.  (No larger; a tenth for the luck of one input.)"""
    _say(f"mass, single pass, exactness in fp32, {slices} x {N}, scale {scale}")
    Q, K, _ = _slices(47, 1, slices, [N], N, 128, 1, "f32")
    Q = (Q * np.float32(scale)).astype(np.float32)
    want = ref.attn_mass(Q, K, "f32")
    (one, _), names = _single_pass(Q, K, "f32")
    assert "attn_single_kernel" in names
    two = gu.gpu_mass(Q, K, "f32")
    assert np.linalg.norm(one - want) <= 1.1 * np.linalg.norm(two - want)


def test_mass_single_pass_rule():
    """Which calls take the single pass: enough workspace, no lengths, short rows; 16-bit rows beyond 1024 tokens up to 2^18
    query rows.  (Sizes and names only: the launches of the rule's far sides are small.)"""
    _say("mass, single pass rule")
    params = kb.kvm_params_for_budget(0.5)

    def takes(dtype, N, copies=1, G=1, lens=None, room=True):
        K = torch.zeros((copies, 1, N, 128), dtype=gu.TORCH_DT[dtype], device="cuda")
        Q = torch.zeros((copies, G, N, 128), dtype=gu.TORCH_DT[dtype], device="cuda")
        sh = kb.make_shape(K, G, gu.lens_dev(lens))
        least, most = kb.kvm_workspace_bytes(sh), kb.kvm_workspace_bytes(sh, params)
        ws = torch.empty(most if room else most - 1, dtype=torch.uint8, device="cuda")
        mass = torch.empty((copies, 1, N), dtype=torch.float32, device="cuda")
        names = gu.kernels_of(lambda: kb.kvm_attn_mass(sh, Q, K, mass, ws))
        single = "attn_single_kernel" in names
        assert not single or most > least
        n = N if lens is None else lens[0]
        harmonic = G * np.cumsum((1.0 / np.arange(1, n + 1))[::-1])[::-1]
        np.testing.assert_allclose(mass[0, 0, :n].cpu().numpy(), harmonic, rtol=1e-5)   # zero scores: sums of 1 / t
        return single

    assert takes("f16", 1024, 300) and takes("bf16", 2048) and takes("f32", 4096) and takes("f16", 40, G=1024)
    assert not takes("f16", 2049) and not takes("f32", 4097) and not takes("f16", 8, G=1025)
    assert not takes("f16", 700, lens=[700]) and not takes("f16", 700, room=False)
    assert takes("f16", 1025, 255) and not takes("f16", 1025, 256) and not takes("bf16", 2048, 33, G=4)


@pytest.mark.parametrize("dtype,n", [("f16", 100000), ("bf16", 70001), ("f32", 20000), ("f16", 131071), ("f16", 2 ** 22)])
def test_mass_long_sequence_against_a_closed_form(dtype, n):
    """Too long for the oracle's n^2 loop, so the scores are given a shape whose column sums have
    a closed form at any length: every query is beta e_1, hence row t is a softmax of the same
    numbers c alpha_j (alpha_j = first component of key j) cut off at j <= t, and
    mass_j = exp(c alpha_j) * sum over t >= j of 1 / (sum over i <= t of exp(c alpha_i)).
    Head 1 has zero queries: harmonic numbers.  The other components of the keys are noise."""
    _say(f"mass: closed form at n={n}, {dtype}")
    rng = np.random.default_rng(19)
    beta = 8.0
    # the longest cases: one head, no decode step (time); 131071 is about the longest that the split kernels take
    heads = 1 if n > 10 ** 5 else 2
    k = rng.standard_normal((1, heads, n, 128), dtype=np.float32)
    q = np.zeros((1, heads, n, 128), np.float32)
    q[0, 0, :, 0] = beta
    K, Q = synth.to_storage(k, dtype), synth.to_storage(q, dtype)
    del k, q
    alpha = synth.to_f64(np.ascontiguousarray(K[0, 0, :, 0]), dtype)   # as stored
    e = np.exp(beta / math.sqrt(128.0) * alpha)
    tail = np.cumsum((1.0 / np.cumsum(e))[::-1])[::-1]        # sum over t >= j of 1 / Z_t
    Hn = np.concatenate([[0.0], np.cumsum(1.0 / np.arange(1, n + 1))])
    want = np.stack([e * tail, Hn[n] - Hn[:n]][:heads])[None]
    got = gu.gpu_mass(Q, K, dtype)
    err = gu.assert_mass_close(got, want, None, n, f"closed form n={n}")
    _say(f"  worst relative error {err:.2e}")
    # one decode step on top: the same closed form one token further, from the library's own scores
    if heads == 2:
        short = gu.gpu_mass(Q, K, dtype, seq_lens=[n - 1])
        again = gu.gpu_mass_append(np.ascontiguousarray(Q[:, :, n - 1]), K, short, dtype, seq_lens=[n])
        gu.assert_mass_close(again, want, None, n, f"closed form n={n}, last row appended")


@pytest.mark.parametrize("dtype,G,lens,N", [("f16", 1, [600], 600), ("bf16", 4, [300, 129, 0, 1, 256], 320),
                                            ("f32", 2, [257, 64], 257), ("f16", 1, [2100, 1500], 2100)])
def test_mass_from_row_statistics_of_the_caller(dtype, G, lens, N):
    """The row statistics come from the oracle (rounded to fp32, as a prefill kernel would hand
    them over); entries past a slice's length are poisoned to show that they are not read."""
    _say(f"mass from row statistics dtype={dtype} G={G} lens={lens} N={N}")
    Q, K, _ = _slices(14, len(lens), 2, lens, N, 128, G, dtype)
    lse = ref.row_lse(Q, K, dtype, G=G, seq_lens=lens).astype(np.float32)
    for b, n in enumerate(lens):
        lse[b, :, n:] = np.nan
    want = ref.attn_mass(Q, K, dtype, G=G, seq_lens=lens)
    got = gu.gpu_mass_from_lse(Q, K, lse, dtype, G=G, seq_lens=lens)
    gu.assert_mass_close(got, want, lens, N, f"{dtype} G={G} from row statistics")
    # and it is the map that the two-pass entry point computes
    two_pass = gu.gpu_mass(Q, K, dtype, G=G, seq_lens=lens)
    assert np.abs(got - two_pass).max() <= 1e-4 * max(1.0, np.abs(two_pass).max())


@pytest.mark.parametrize("dtype,G,lens,N", [("f16", 1, [600], 600), ("bf16", 4, [300, 129, 0, 1, 256, 257], 320),
                                            ("f32", 2, [255, 64], 257), ("f16", 1, [5000, 4097], 5000)])
def test_mass_append_one_query_row(dtype, G, lens, N):
    """Decode-time update: the same fp32 scores before the call on both sides (random, with a
    marker past each row's length that must survive), the newest token's query from the generator."""
    _say(f"mass append dtype={dtype} G={G} lens={lens} N={N}")
    Q, K, _ = _slices(15, len(lens), 2, lens, N, 128, G, dtype)
    q_new = np.ascontiguousarray(np.stack([Q[b, :, max(n - 1, 0)] for b, n in enumerate(lens)]))
    before = (np.random.default_rng(16).random((len(lens), 2, N)) * 3 + 0.01).astype(np.float32)
    for b, n in enumerate(lens):
        before[b, :, n:] = -5.0
    want = ref.attn_mass_append(q_new, K, before.astype(np.float64), dtype, G=G, seq_lens=lens)
    got = gu.gpu_mass_append(q_new, K, before, dtype, G=G, seq_lens=lens)
    for b, n in enumerate(lens):
        assert np.all(got[b, :, n:] == -5.0), "entries past the length were touched"
        if n:
            rel = np.abs(got[b, :, :n] - want[b, :, :n]) / want[b, :, :n]
            assert rel.max() <= gu.TOL, f"row {b}: relative error {rel.max():.3e}"
            # the row that was added sums to G
            added = got[b, :, :n].astype(np.float64).sum(axis=1) - before[b, :, :n - 1].astype(np.float64).sum(axis=1)
            assert added == pytest.approx(G, rel=1e-3)


@pytest.mark.parametrize("dtype,G,lens,N", [
    ("f16", 8, [300, 0, 65], 300), ("bf16", 17, [129, 1, 1100], 1100), ("f16", 33, [200], 256),   # more heads than waves, than ACC_HEADS
    ("f16", 1, [32768, 32769], 32832), ("bf16", 3, [32769, 700, 40001], 40001), ("f32", 4, [33000], 33000), ("f16", 17, [33000], 33000),
    ("f16", 1, [262144, 262145], 270000), ("bf16", 2, [527000], 527000), ("f16", 17, [263000], 263000)])
def test_mass_append_many_heads_and_long_rows(dtype, G, lens, N):
    """Decode-time update where the waves of a workgroup take several heads, in several turns, where they share the statistics
    of a row (beyond 512 * 64 keys) and where a workgroup takes several chunks of keys (beyond 256 * 1024)."""
    _say(f"mass append, heads and lengths: {dtype} G={G} lens={lens} N={N}")
    rng = np.random.default_rng(N + G)
    B = len(lens)
    K = synth.to_storage(rng.standard_normal((B, 1, N, 128), dtype=np.float32), dtype)
    q_new = synth.to_storage(rng.standard_normal((B, G, 128), dtype=np.float32), dtype)
    before = (rng.random((B, 1, N)) * 1e-3).astype(np.float32)
    for b, n in enumerate(lens):
        before[b, :, n:] = -5.0
    got = gu.gpu_mass_append(q_new, K, before, dtype, G=G, seq_lens=lens)
    want = ref.attn_mass_append(q_new, K, before.astype(np.float64), dtype, G=G, seq_lens=lens)
    for b, n in enumerate(lens):
        assert np.all(got[b, :, n:] == -5.0), "entries past the length were touched"
        if n:
            # what was added, to the rounding of the sum with what was there (2^-24 of 1e-3, far below an average entry of G / n)
            add, want_add = (x[b, 0, :n].astype(np.float64) for x in (got, want))
            add[:n - 1] -= before[b, 0, :n - 1]
            want_add[:n - 1] -= before[b, 0, :n - 1]
            assert (np.abs(add - want_add) <= 1e-4 * want_add + 2.0 ** -23 * want[b, 0, :n]).all()
            assert add.sum() == pytest.approx(G, rel=1e-5)


def test_mass_append_continues_the_prefill_pass():
    """Prefill scores of the first n0 tokens, then appends token by token: the result has to be
    the prefill scores of all n1 tokens (both from the library; the oracle checks the end state)."""
    n0, n1, dtype = 300, 316, "f16"
    _say(f"mass: prefill of {n0} tokens + {n1 - n0} appends against a prefill of {n1}")
    Q, K, _ = _slices(17, 1, 3, [n1], n1, 128, 1, dtype)
    mass = gu.gpu_mass(Q, K, dtype, seq_lens=[n0])
    assert np.all(mass[:, :, n0:] == 0)
    for n in range(n0 + 1, n1 + 1):
        mass = gu.gpu_mass_append(np.ascontiguousarray(Q[:, :, n - 1]), K, mass, dtype, seq_lens=[n])
    want = ref.attn_mass(Q, K, dtype)
    gu.assert_mass_close(mass, want, None, n1, "prefill + appends")
    direct = gu.gpu_mass(Q, K, dtype)
    assert np.abs(mass - direct).max() <= 1e-4 * np.abs(direct).max()


@pytest.mark.parametrize("cut", [77, 6000, 9000, 16000])
@pytest.mark.parametrize("dtype,H", [("f16", 64), ("bf16", 32), ("f32", 16)])
def test_streamed_launches_give_the_bits_of_small_ones(dtype, H, cut):
    """From 128 MiB of keys (decode-time scores) and 256 MiB (scan) on, rows are read with the non-temporal hint, each slice
    by its own length: with its second row shorter by `cut` a batch streams in both kernels, in one, in none of that row; the
    merge writes with the hint where its rows and the caches come to 256 MiB.  Nothing else differs, so every slice has the bits it gets in a call of its own, ragged last tiles included."""
    B, N = 2, 16381 if dtype == "f32" else 16384
    esz = 4 if dtype == "f32" else 2
    _say(f"streamed launches: {dtype}, {B * H} slices of {N} ({B * H * N * 128 * esz >> 20} MiB of keys)")
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    K = gu.randn_gpu((B, H, N, 128), dt, 41)
    q = gu.randn_gpu((B, H, 128), dt, 42)
    params = kb.kvm_params_for_budget(0.35)
    results = []
    for K_part, q_part in ((K, q), (K[1:, H - 1:].contiguous(), q[1:, H - 1:].contiguous())):
        lens = torch.tensor([N, N - cut][-K_part.shape[0]:], dtype=torch.int32, device="cuda")
        shape = kb.make_shape(K_part, 1, lens)
        buf = kb.Buffers(shape, params, "cuda", dt, with_sim=True)
        buf.mass.fill_(0.25)
        kb.kvm_attn_mass_append(shape, q_part, K_part, buf.mass, buf.ws)
        kb.kvm_identify_sets(shape, params, K_part, buf.mass, buf.set_id, buf.set_start, buf.pivot, buf.n_sets, buf.sim,
                             buf.status, buf.ws)
        kb.kvm_merge(shape, params, K_part, K_part, buf.set_start, buf.pivot, buf.n_sets, buf.K_out, buf.V_out, None, buf.ws)
        rows = int(buf.n_sets[-1, -1])
        results.append([t[-1, -1].cpu() for t in (buf.mass, buf.sim, buf.set_id, buf.set_start, buf.pivot)] +
                       [t[-1, -1, :rows].cpu() for t in (buf.K_out, buf.V_out)])
    for name, a, b in zip(("mass", "sim", "set_id", "set_start", "pivot", "K_out", "V_out"), *results):
        assert torch.equal(a, b), name


def test_mass_append_large_scores():
    n, dtype = 700, "bf16"
    _say("mass append: scores in the hundreds")
    rng = np.random.default_rng(18)
    k = rng.standard_normal((1, 2, n, 128)).astype(np.float32) * 5
    q = k[:, :, 123] * 4                                      # the query picks out key 123 with a score near 5000
    K, q_new = synth.to_storage(k, dtype), synth.to_storage(np.ascontiguousarray(q), dtype)
    before = np.ones((1, 2, n), np.float32)
    want = ref.attn_mass_append(q_new, K, before.astype(np.float64), dtype)
    got = gu.gpu_mass_append(q_new, K, before, dtype)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= gu.TOL * np.abs(want).max() and got[0, 0, 123] == pytest.approx(2.0, rel=1e-3)


# ---------------------------------------------------------------------------------------------
# (b) merging sets
# ---------------------------------------------------------------------------------------------

def _identify_both(K, mass64, dtype, params, lens=None):
    mass32 = mass64.astype(np.float32)
    B, H, N, _ = K.shape
    g = gu.gpu_identify(K, mass32, dtype, params, lens)
    o = ref.identify_sets(K, mass32.astype(np.float64), dtype, params.budget, params.recent_ratio,
                          params.heavy_ratio, params.threshold, bool(params.enforce_budget), g["cap_rows"], lens,
                          pivot_rule=params.pivot_rule, pivot_seed=params.pivot_seed, set_rule=params.set_rule)
    return g, o


def _compare_anchor_maps(g, o, what):
    """Anchor rule: one flipped comparison moves every set below it, so a slice is either
    bit-identical or, when the oracle saw a similarity within NEAR of the threshold, excused."""
    B, H = o["n_sets"].shape
    excused = 0
    for b in range(B):
        for h in range(H):
            same = all(np.array_equal(g[k][b, h], o[k][b, h]) for k in ("set_id", "set_start", "pivot")) and \
                g["n_sets"][b, h] == o["n_sets"][b, h] and g["status"][b, h] == o["status"][b, h]
            if not same:
                assert o["anchor_margin"][b, h] <= gu.NEAR, \
                    f"{what} slice ({b},{h}): maps differ although no comparison came closer than " \
                    f"{o['anchor_margin'][b, h]:.2e} to the threshold"
                excused += 1
    return excused


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_identify_anchor_rule(dtype):
    n = 1500
    lens = [n, 1037, 0, 1]
    _say(f"identify: anchor rule, {dtype}, lens {lens}")
    Q, K, V = _slices(24, 4, 3, lens, n, 128, 1, dtype)
    mass = np.random.default_rng(8).random((4, 3, n)) + 0.01
    total_excused = 0
    for budget, thr, enforce in ((0.5, 0.75, True), (0.5, 0.5, False), (0.15, 0.9, True), (1.0, -2.0, False)):
        params = kb.make_params(budget, 0.3 * budget, 0.2 * budget, threshold=thr, enforce_budget=enforce,
                                set_rule=kb.KVM_SETS_ANCHOR)
        g, o = _identify_both(K, mass, dtype, params, lens)
        total_excused += _compare_anchor_maps(g, o, f"anchor {dtype} thr {thr}")
        gu.check_partition(g, lens, n, g["cap_rows"])
        np.testing.assert_allclose(g["sim"], o["sim"], atol=2e-6)        # still the adjacent similarities
        if budget == 0.15:
            assert (o["status"][0] & kb.KVM_SLICE_INFEASIBLE).all()       # this rule has no fallback
    _say(f"  excused slices: {total_excused}")
    assert total_excused <= 4


def test_identify_anchor_rule_special_keys():
    n = 400
    _say("identify: anchor rule on a turning key, identical keys, zero rows")
    K = np.zeros((1, 3, n, 128), np.float32)
    t = np.arange(n)
    K[0, 0, :, 0], K[0, 0, :, 1] = np.cos(0.1 * t), np.sin(0.1 * t)       # sets of 8 against the anchor
    K[0, 1] = np.arange(1, 129)                                           # identical keys
    K[0, 2] = np.random.default_rng(0).standard_normal((n, 128))
    K[0, 2, 50:60] = 0                                                    # zero-norm keys: similarity 0
    mass = np.linspace(2, 1, n)[None, None].repeat(3, 1)
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False, set_rule=kb.KVM_SETS_ANCHOR)
    g, o = _identify_both(K, mass, "f32", params)
    assert _compare_anchor_maps(g, o, "anchor special") == 0
    assert g["n_sets"][0, 0] == 50 and g["n_sets"][0, 1] == 1


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 255, 256, 257, 1000, 4096, 5000])
def test_identify_sizes(dtype, n):
    _say(f"identify dtype={dtype} n={n}")
    Q, K, V = _slices(21, 2, 2, [n, n], n, 128, 1, dtype)
    rng = np.random.default_rng(n)
    mass = rng.random((2, 2, n)) ** 3 + 1e-3
    params = kb.kvm_params_for_budget(0.5)
    g, o = _identify_both(K, mass, dtype, params)
    np.testing.assert_allclose(g["sim"], o["sim"], atol=2e-6)
    exc, near = gu.compare_maps(g, o, None, n, params.threshold, f"{dtype} n={n}")
    _say(f"  excused slices {exc}, near-threshold similarities {near}")
    gu.check_partition(g, None, n, g["cap_rows"])


@pytest.mark.parametrize("budget", [0.5, 0.35])
def test_identify_with_oracle_mass_on_workload_slices(budget):
    n = 1024
    _say(f"identify on oracle mass, budget={budget}")
    Q, K, V = _slices(22, 1, 6, [n], n, 128, 1, "f16")
    mass = ref.attn_mass(Q, K, "f16")
    params = kb.kvm_params_for_budget(budget)
    g, o = _identify_both(K, mass, "f16", params)
    exc, near = gu.compare_maps(g, o, None, n, params.threshold, f"budget {budget}")
    assert (o["n_sets"] <= math.floor(budget * n)).all() and (g["status"] == 0).all()
    _say(f"  sets per slice {g['n_sets'].ravel().tolist()}, excused {exc}, near {near}")


def test_identify_ragged_and_padding_garbage():
    lens = [700, 64, 0, 1, 333, 1023]
    N = 1024
    _say(f"identify ragged lens={lens}")
    Q, K, V = _slices(23, len(lens), 2, lens, N, 128, 1, "bf16")
    mass = np.random.default_rng(5).random((len(lens), 2, N)) + 0.01
    params = kb.kvm_params_for_budget(0.35)
    g, o = _identify_both(K, mass, "bf16", params, lens)
    gu.compare_maps(g, o, lens, N, params.threshold, "ragged")
    gu.check_partition(g, lens, N, g["cap_rows"])
    for b, n in enumerate(lens):
        assert (g["sim"][b, :, n:] == 0).all()


def test_identify_special_keys():
    n, d = 300, 128
    _say("identify: identical keys, orthogonal keys, zero row")
    params = kb.make_params(1.0, 0.1, 0.05, enforce_budget=False)
    mass = np.linspace(2, 1, n)[None, None].repeat(3, 1)
    K = np.zeros((1, 3, n, d), np.float32)
    K[0, 0] = np.arange(1, d + 1)                      # identical keys
    K[0, 1, np.arange(n), np.arange(n) % d] = 1.0      # neighbours orthogonal
    K[0, 2] = np.random.default_rng(0).standard_normal((n, d))
    K[0, 2, 100:110] = K[0, 2, 100]                    # a run of equal keys ...
    K[0, 2, 105] = 0                                   # ... split by a zero-norm key
    g, o = _identify_both(K, mass, "f32", params)
    gu.compare_maps(g, o, None, n, params.threshold, "special keys")
    assert g["n_sets"][0, 0] == 30 + 15 + 1 and g["n_sets"][0, 1] == n
    assert g["sim"][0, 2, 105] == 0 and g["sim"][0, 2, 106] == 0


@pytest.mark.parametrize("dtype,scale", [("f16", 2.0 ** -20), ("f16", 200.0), ("bf16", 1e-15), ("bf16", 1e15), ("f32", 1e-15)])
def test_identify_key_magnitudes(dtype, scale):
    """Keys in the subnormal range of the storage type, and very small and very large keys: the
    similarity does not depend on the scale of the keys."""
    n = 500
    _say(f"identify: keys scaled by {scale} ({dtype})")
    rng = np.random.default_rng(5)
    x = np.zeros((1, 2, n, 128), np.float32)
    x[0, :, 0] = rng.standard_normal((2, 128))
    for t in range(1, n):                                    # AR(1) keys, similarity around the threshold
        x[0, :, t] = 0.75 * x[0, :, t - 1] + np.sqrt(1 - 0.75 ** 2) * rng.standard_normal((2, 128))
    K = synth.to_storage((x * scale).astype(np.float32), dtype)
    mass = rng.uniform(1, 2, (1, 2, n))
    params = kb.kvm_params_for_budget(0.5)
    g, o = _identify_both(K, mass, dtype, params)
    np.testing.assert_allclose(g["sim"], o["sim"], atol=2e-6)
    gu.compare_maps(g, o, None, n, params.threshold, f"{dtype} scale {scale}")


def test_identify_ties_in_mass():
    n = 2000
    _say("identify: heavy ties in the scores (top-k and pivot tie-breaks)")
    Q, K, V = _slices(24, 1, 4, [n], n, 128, 1, "f16", rho=0.97)
    rng = np.random.default_rng(3)
    mass = rng.integers(1, 6, size=(1, 4, n)).astype(np.float64)      # five distinct values only
    mass[0, 3] = 1.0                                                    # all equal
    for budget in (0.5, 0.35):
        params = kb.kvm_params_for_budget(budget)
        g, o = _identify_both(K, mass, "f16", params)
        gu.compare_maps(g, o, None, n, params.threshold, f"ties budget {budget}")


@pytest.mark.parametrize("n", [1535, 1536, 4096, 4097])
def test_identify_select_on_both_sides_of_the_histogram_copies(n):
    """The radix select counts its first digit in eight copies from 1536 tokens on: scores that agree in no, one, two,
    three or all four bytes of their order-preserving key (the top-k threshold then falls in each digit in turn), and
    random keys, whose fallback selects among similarities of both signs."""
    _say(f"identify: digits of the select, n={n}")
    rng = np.random.default_rng(n)
    K = synth.to_storage(rng.standard_normal((1, 5, n, 128)).astype(np.float32), "f16")
    mass = np.empty((1, 5, n), np.float32)
    mass[0, 0] = np.exp2(rng.uniform(-60, 60, n))
    for h, low_bits in enumerate((24, 16, 8, 0), 1):
        mass[0, h] = (0x3f000000 + rng.integers(0, 1 << low_bits, n)).astype(np.uint32).view(np.float32)
    params = kb.kvm_params_for_budget(0.35)
    g, o = _identify_both(K, mass.astype(np.float64), "f16", params)
    gu.compare_maps(g, o, None, n, params.threshold, f"n={n}")


@pytest.mark.parametrize("n", [255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384])
def test_identify_on_both_sides_of_the_workgroup_sizes(n):
    """A slice gets as many threads as it needs, of 4, 8 or 16 tokens: sets, sets' ends and pivots that cross a thread's, a
    wave's and the last thread's edge, thresholds that a digit of the select settles early and ties that none does, with
    and without the budget rule, in rows as long as the stride and one shorter."""
    _say(f"identify: workgroup sizes, n={n}")
    rng = np.random.default_rng(n)
    base = rng.standard_normal((3, 128)).astype(np.float32)
    K = rng.standard_normal((2, 3, n, 128)).astype(np.float32)
    K[:, 1] = base[np.arange(n) % 3]                          # adjacent similarities of three values: ties in the budget rule
    K[:, 2] = base[np.arange(n) // 97 % 3] * rng.uniform(0.5, 2, (n, 1))   # runs of 97 keys of one direction
    K = synth.to_storage(K, "f16")
    mass = np.exp(rng.standard_normal((2, 3, n))).astype(np.float32)
    mass[:, 1] = rng.integers(1, 4, n)                        # ties in the top-k and the pivots
    for budget in (0.5, 0.35):
        params = kb.kvm_params_for_budget(budget)
        lens = [n, n - 1]
        g, o = _identify_both(K, mass.astype(np.float64), "f16", params, lens)
        gu.compare_maps(g, o, lens, n, params.threshold, f"n={n} budget {budget}")


@pytest.mark.parametrize("case", ["fallback", "fallback_ties", "no_enforce"])
def test_identify_budget_rule(case):
    n = 1500
    _say(f"identify budget rule: {case}")
    rng = np.random.default_rng(7)
    if case == "fallback_ties":
        # keys cycle through three directions: every boundary similarity takes one of three values
        base = rng.standard_normal((3, 128)).astype(np.float32)
        K = base[np.arange(n) % 3][None, None].copy()
    else:
        K = rng.standard_normal((1, 1, n, 128)).astype(np.float32)     # neighbours nearly orthogonal
    K = np.concatenate([K, _slices(25, 1, 1, [n], n, 128, 1, "f32", rho=0.8)[1]], axis=1)
    mass = rng.random((1, 2, n)) + 0.1
    params = kb.make_params(0.4, 0.1, 0.1, threshold=0.75, enforce_budget=(case != "no_enforce"))
    g, o = _identify_both(K, mass, "f32", params)
    exc, near = gu.compare_maps(g, o, None, n, params.threshold, case)
    _say(f"  status {g['status'].ravel().tolist()} n_sets {g['n_sets'].ravel().tolist()} excused {exc}")
    if case == "no_enforce":
        assert g["status"][0, 0] == 0 and g["n_sets"][0, 0] == n and g["cap_rows"] == n
    else:
        assert g["status"][0, 0] == kb.KVM_SLICE_FALLBACK and g["n_sets"][0, 0] == math.floor(0.4 * n)


def test_identify_infeasible_budget_is_reported():
    n = 400
    _say("identify: conserved tokens alone exceed the budget")
    K = np.random.default_rng(1).standard_normal((1, 1, n, 128)).astype(np.float32)
    mass = np.random.default_rng(2).random((1, 1, n)) + 0.1
    params = kb.make_params(0.3, 0.15, 0.15, threshold=2.0)             # nothing can merge at threshold 2
    g, o = _identify_both(K, mass, "f32", params)
    gu.compare_maps(g, o, None, n, params.threshold, "infeasible")
    want = kb.KVM_SLICE_FALLBACK | kb.KVM_SLICE_INFEASIBLE | kb.KVM_SLICE_TRUNCATED
    assert g["status"][0, 0] == want and g["n_sets"][0, 0] > g["cap_rows"]


def test_identify_and_merge_at_the_maximum_length():
    """One slice of 2^22 tokens, the longest sequence the library accepts (one more is refused)."""
    n, dtype = 2 ** 22, "f16"
    _say(f"identify + merge at N={n}")
    rng = np.random.default_rng(29)
    # keys that share a direction for a stretch and then jump (mean stretch 32 tokens): within a
    # stretch adjacent keys have cosine similarity near 0.9, across a jump near 0
    noise = rng.standard_normal((n, 128), dtype=np.float32)
    stretch = np.cumsum(rng.random(n) < 1 / 32)
    direction = rng.standard_normal((int(stretch[-1]) + 1, 128), dtype=np.float32)
    k = np.float32(math.sqrt(0.9)) * direction[stretch] + np.float32(math.sqrt(0.1)) * noise
    del noise, direction
    K = synth.to_storage(k[None, None], dtype)
    V = synth.to_storage(rng.standard_normal((1, 1, n, 128), dtype=np.float32), dtype)
    del k
    mass = rng.random((1, 1, n)) ** 3 + 1e-3
    params = kb.kvm_params_for_budget(0.5)
    g, o = _identify_both(K, mass, dtype, params)
    np.testing.assert_allclose(g["sim"], o["sim"], atol=2e-6)
    exc, near = gu.compare_maps(g, o, None, n, params.threshold, "maximum length")
    _say(f"  sets {int(o['n_sets'][0, 0])}, excused slices {exc}, near-threshold similarities {near}")
    gu.check_partition(g, None, n, g["cap_rows"])
    res = _merge_both(K, V, dtype, params, o)
    _check_merge(K, V, dtype, o, *res, "maximum length")
    sh = kb.KvmShape(1, 1, 1, n + 1, 128, kb.KVM_F16, None)
    assert kb.kvm_workspace_bytes(sh, params) == 0 and b"too large" in kb.load_library().kvm_last_error()


@pytest.mark.parametrize("rule", ["adjacent", "anchor"])
def test_identify_and_merge_beyond_the_short_sequence_paths(rule):
    """40000 tokens: longer than any staging buffer sized for the usual prompts (the anchor walk
    reads its inputs from global memory from 16385 tokens on), with a ragged second row."""
    n = 40000
    lens = [n, 33333]
    _say(f"identify + merge, {rule} sets, N={n}, lens {lens}")
    Q, K, V = _slices(27, 2, 2, lens, n, 128, 1, "f16")
    del Q
    mass = np.random.default_rng(10).random((2, 2, n)) ** 3 + 1e-3
    params = kb.kvm_params_for_budget(0.5)
    if rule == "anchor":
        params.set_rule = kb.KVM_SETS_ANCHOR
    g, o = _identify_both(K, mass, "f16", params, lens)
    np.testing.assert_allclose(g["sim"], o["sim"], atol=2e-6)
    if rule == "anchor":
        exc = _compare_anchor_maps(g, o, "long anchor")
    else:
        exc, _ = gu.compare_maps(g, o, lens, n, params.threshold, "long adjacent")
    _say(f"  excused slices {exc}; sets {o['n_sets'].tolist()}")
    assert exc <= 1
    gu.check_partition(g, lens, n, g["cap_rows"])
    o["cap_rows"] = g["cap_rows"]
    res = _merge_both(K, V, "f16", params, o, lens)
    _check_merge(K, V, "f16", o, *res, f"long {rule}")


def test_identify_with_similarities_carried_over_the_decode_steps():
    """Sets for a growing sequence with the similarities kept from call to call: a full call at
    n0 tokens, then per new token one new similarity (kvm_sim_append) and a call that trusts the
    buffer.  Every step must give the maps of a call that scans K itself, and the last one the
    oracle's (same fp32 scores on both sides)."""
    n0, n1, N, dtype = 700, 716, 720, "bf16"
    lens1 = [n1, n1 - 300]
    _say(f"identify over decode steps {n0}..{n1} with carried similarities (second row 300 shorter)")
    Q, K, V = _slices(28, 2, 2, lens1, N, 128, 1, dtype)
    del Q, V
    mass = (np.random.default_rng(11).random((2, 2, N)) ** 3 + 1e-3).astype(np.float32)
    Kd, md = gu.to_dev(K, dtype), torch.from_numpy(mass).cuda()
    full = kb.kvm_params_for_budget(0.5)
    carried = kb.kvm_params_for_budget(0.5)
    carried.sim_given = 1
    sim = torch.full((2, 2, N), float("nan"), dtype=torch.float32, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")

    def run(params, lens, sim_buf):
        sl = gu.lens_dev(lens)
        sh = kb.make_shape(Kd, 1, sl)
        cap = kb.kvm_out_capacity(sh, params)
        o = dict(set_id=torch.full((2, 2, N), -7, **i32), set_start=torch.full((2, 2, cap + 1), -7, **i32),
                 pivot=torch.full((2, 2, cap), -7, **i32), n_sets=torch.full((2, 2), -7, **i32),
                 status=torch.full((2, 2), -7, **i32))
        ws = torch.empty(max(kb.kvm_workspace_bytes(sh, params), 256), dtype=torch.uint8, device="cuda")
        if params.sim_given:
            kb.kvm_sim_append(sh, Kd, sim_buf)
        kb.kvm_identify_sets(sh, params, Kd, md, o["set_id"], o["set_start"], o["pivot"], o["n_sets"], sim_buf,
                             o["status"], ws)
        torch.cuda.synchronize()
        return o

    run(full, [n0, n0 - 300], sim)
    for n in range(n0 + 1, n1 + 1):
        lens = [n, n - 300]
        got = run(carried, lens, sim)
        fresh_sim = torch.empty_like(sim)
        want = run(full, lens, fresh_sim)
        for k in want:
            assert torch.equal(got[k], want[k]), f"n={n}: {k} differs from the call that scans K"
        for b, nb in enumerate(lens):
            assert torch.equal(sim[b, :, :nb], fresh_sim[b, :, :nb]), f"n={n}: carried similarities differ"
    o = ref.identify_sets(K, mass.astype(np.float64), dtype, full.budget, full.recent_ratio, full.heavy_ratio,
                          full.threshold, True, got["set_start"].shape[2] - 1, lens1)
    g = {k: v.cpu().numpy() for k, v in got.items()}
    g["sim"] = sim.cpu().numpy()
    exc, _ = gu.compare_maps(g, o, lens1, N, full.threshold, "carried similarities")
    assert exc == 0


# ---------------------------------------------------------------------------------------------
# (c) Gaussian-kernel merge
# ---------------------------------------------------------------------------------------------

def _merge_both(K, V, dtype, params, o, lens=None):
    ko, vo, w, Kt, Vt = gu.gpu_merge(K, V, dtype, params, o["set_start"], o["pivot"], o["n_sets"], lens)
    rk, rv, rw = ref.merge(K, V, dtype, o["set_start"], o["pivot"], o["n_sets"], params.sigma_mode, params.sigma,
                           bool(params.value_scale_by_set_size), lens, weights=params.weights)
    return ko, vo, w, rk, rv, rw, Kt, Vt


def _check_merge(K, V, dtype, o, ko, vo, w, rk, rv, rw, Kt, Vt, what):
    B, H, N, d = K.shape
    worst_k = worst_v = worst_w = 0.0
    for b in range(B):
        for h in range(H):
            M = min(int(o["n_sets"][b, h]), o["cap_rows"])
            if M == 0:
                continue
            ek = gu.row_rel_err(ko[b, h, :M], rk[b, h, :M])
            ev = gu.row_rel_err(vo[b, h, :M], rv[b, h, :M])
            worst_k, worst_v = max(worst_k, ek.max()), max(worst_v, ev.max())
            # beyond the one rounding to the cache dtype only fp32 accumulation error remains
            xk = gu.ulp_excess(ko[b, h, :M], rk[b, h, :M], dtype).max()
            xv = gu.ulp_excess(vo[b, h, :M], rv[b, h, :M], dtype).max()
            assert xk <= 2e-5 and xv <= 2e-5, f"{what}: error beyond one storage ulp {xk:.2e}/{xv:.2e}"
            st = o["set_start"][b, h]
            single = np.flatnonzero(np.diff(st[:M + 1]) == 1)
            src = st[single]
            k64, v64 = synth.to_f64(K[b, h], dtype), synth.to_f64(V[b, h], dtype)
            assert np.array_equal(ko[b, h, single], k64[src]), f"{what}: singleton key rows are not bit-identical"
            assert np.array_equal(vo[b, h, single], v64[src]), f"{what}: singleton value rows are not bit-identical"
            if w is not None:
                n_cov = st[M]
                worst_w = max(worst_w, np.abs(w[b, h, :n_cov] - rw[b, h, :n_cov]).max())
    tol = gu.kv_tol(dtype)
    assert worst_k <= tol and worst_v <= tol, f"{what}: merged K/V error {worst_k:.3e}/{worst_v:.3e} > {tol:.3e}"
    assert worst_w <= 1e-5, f"{what}: weight error {worst_w:.3e}"
    return worst_k, worst_v, worst_w


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("budget", [0.5, 0.35])
def test_merge_on_workload_slices(dtype, budget):
    n = 1536
    _say(f"merge dtype={dtype} budget={budget}")
    Q, K, V = _slices(31, 2, 3, [n, n], n, 128, 1, dtype)
    mass = np.random.default_rng(9).random((2, 3, n)) ** 3 + 1e-3
    params = kb.kvm_params_for_budget(budget)
    cap = math.floor(budget * n)
    o = ref.identify_sets(K, mass, dtype, params.budget, params.recent_ratio, params.heavy_ratio, params.threshold,
                          True, cap)
    res = _merge_both(K, V, dtype, params, o)
    errs = _check_merge(K, V, dtype, o, *res, f"{dtype} budget {budget}")
    _say(f"  worst K/V/w errors {errs[0]:.2e} {errs[1]:.2e} {errs[2]:.2e}; "
         f"largest set {int(np.diff(o['set_start'][0, 0, :o['n_sets'][0, 0] + 1]).max())}")


@pytest.mark.parametrize("rule,seed", [(kb.KVM_PIVOT_LAST, 0), (kb.KVM_PIVOT_RANDOM, 0), (kb.KVM_PIVOT_RANDOM, 2 ** 63 + 12345)])
@pytest.mark.parametrize("dtype,n", [("f16", 4096), ("bf16", 777)])
def test_identify_pivot_rules(rule, seed, dtype, n):
    _say(f"identify: pivot rule {rule}, seed {seed}, {dtype} n={n}")
    Q, K, V = _slices(23, 2, 3, [n, n - 5], n, 128, 1, dtype)
    mass = np.random.default_rng(n).random((2, 3, n)) + 0.01
    for budget, thr, enforce in ((0.5, 0.75, True), (0.2, 0.95, True), (1.0, 0.6, False)):   # plain, fallback + truncation, free
        params = kb.make_params(budget, 0.3 * budget, 0.2 * budget, threshold=thr, enforce_budget=enforce,
                                pivot_rule=rule, pivot_seed=seed)
        g, o = _identify_both(K, mass, dtype, params, [n, n - 5])
        gu.compare_maps(g, o, [n, n - 5], n, params.threshold, f"pivot rule {rule} budget {budget}")
        gu.check_partition(g, [n, n - 5], n, g["cap_rows"])


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("scale", [True, False])
def test_merge_average_weights(dtype, scale):
    n = 1500
    _say(f"merge: average weights, {dtype}, value scale {scale}")
    Q, K, V = _slices(34, 1, 3, [n], n, 128, 1, dtype)
    mass = np.random.default_rng(7).random((1, 3, n)) + 0.01
    params = kb.make_params(0.5, 0.17, 0.12, weights=kb.KVM_WEIGHTS_AVERAGE, pivot_rule=kb.KVM_PIVOT_LAST,
                            value_scale_by_set_size=scale)
    o = ref.identify_sets(K, mass, dtype, 0.5, 0.17, 0.12, 0.75, True, n // 2, pivot_rule=ref.PIVOT_LAST)
    res = _merge_both(K, V, dtype, params, o)
    _check_merge(K, V, dtype, o, *res, f"average {dtype}")
    # one long set (two sweeps in the kernel) and the fixed-sigma field set at the same time: ignored
    params = kb.make_params(1.0, 0.0, 0.0, threshold=-2.0, enforce_budget=False, weights=kb.KVM_WEIGHTS_AVERAGE,
                            sigma_mode=kb.KVM_SIGMA_FIXED, sigma=0.01, value_scale_by_set_size=scale)
    o = ref.identify_sets(K, mass, dtype, 1.0, 0.0, 0.0, -2.0, False, n)
    res = _merge_both(K, V, dtype, params, o)
    _check_merge(K, V, dtype, o, *res, f"average, one set, {dtype}")


@pytest.mark.parametrize("mode", ["fixed_sigma", "no_value_scale", "fixed_sigma_small"])
def test_merge_variants(mode):
    n = 800
    _say(f"merge variant {mode}")
    Q, K, V = _slices(32, 1, 4, [n], n, 128, 1, "f16")
    mass = np.random.default_rng(4).random((1, 4, n)) + 0.01
    kw = dict(fixed_sigma=dict(sigma_mode=kb.KVM_SIGMA_FIXED, sigma=5.0),
              fixed_sigma_small=dict(sigma_mode=kb.KVM_SIGMA_FIXED, sigma=0.5),
              no_value_scale=dict(value_scale_by_set_size=False))[mode]
    params = kb.make_params(0.5, 0.17, 0.12, **kw)
    o = ref.identify_sets(K, mass, "f16", 0.5, 0.17, 0.12, 0.75, True, n // 2)
    res = _merge_both(K, V, "f16", params, o)
    _check_merge(K, V, "f16", o, *res, mode)


def test_merge_degenerate_sets():
    n, d = 3000, 128
    _say("merge: one set spanning the whole slice; identical keys; ragged; truncated capacity")
    rng = np.random.default_rng(6)
    lens = [n, 37, 0]
    K = rng.standard_normal((3, 2, n, d)).astype(np.float32)
    V = rng.standard_normal((3, 2, n, d)).astype(np.float32)
    K[0, 1] = K[0, 1, 0]                                  # identical keys: uniform weights
    mass = rng.random((3, 2, n)) + 0.1
    params = kb.make_params(1.0, 0.0, 0.0, threshold=-2.0, enforce_budget=False)   # everything merges
    o = ref.identify_sets(K, mass, "f32", 1.0, 0.0, 0.0, -2.0, False, n, lens)
    assert o["n_sets"].ravel().tolist() == [1, 1, 1, 1, 0, 0]
    res = _merge_both(K, V, "f32", params, o, lens)
    _check_merge(K, V, "f32", o, *res, "degenerate")
    # truncated: more sets than rows of capacity -> only the stored sets are merged
    params = kb.make_params(0.3, 0.15, 0.15, threshold=2.0)
    o = ref.identify_sets(K, mass, "f32", 0.3, 0.15, 0.15, 2.0, True, math.floor(0.3 * n), lens)
    assert (o["status"][0] & kb.KVM_SLICE_TRUNCATED).all()
    res = _merge_both(K, V, "f32", params, o, lens)
    _check_merge(K, V, "f32", o, *res, "truncated")


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("mode", ["gaussian", "fixed_sigma", "average", "no_value_scale"])
def test_merge_sets_around_the_length_a_workgroup_takes_over(dtype, mode):
    """Hand-made partitions with sets of 512 tokens (still one wave's), 513 and 2000 tokens (merged by a
    whole workgroup), short sets and singletons between them, ragged lengths; every weighting."""
    n = 3600
    _say(f"merge: long sets, {dtype}, {mode}")
    rng = np.random.default_rng(77)
    lens = [n, 1500, 513]
    Q, K, V = _slices(34, 3, 2, lens, n, 128, 1, dtype, rho=0.97)
    sizes = [[512, 513, 5, 1, 2000, 17, 1, 1, 64, 486], [700, 1, 1, 513, 285], [513]]
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    if mode == "fixed_sigma":
        params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 4.0
    elif mode == "average":
        params.weights = kb.KVM_WEIGHTS_AVERAGE
    elif mode == "no_value_scale":
        params.value_scale_by_set_size = 0
    cap = n
    st = np.zeros((3, 2, cap + 1), np.int32)
    pv = np.full((3, 2, cap), -1, np.int32)
    ns = np.zeros((3, 2), np.int32)
    for b in range(3):
        assert sum(sizes[b]) == lens[b]
        for h in range(2):
            starts = np.concatenate([[0], np.cumsum(sizes[b])])
            M = len(sizes[b])
            st[b, h, :M + 1] = starts
            st[b, h, M + 1:] = lens[b]
            pv[b, h, :M] = starts[:-1] + rng.integers(0, sizes[b])
            ns[b, h] = M
    o = dict(set_start=st, pivot=pv, n_sets=ns, cap_rows=cap)
    res = _merge_both(K, V, dtype, params, o, lens)
    _check_merge(K, V, dtype, o, *res, f"long sets {dtype} {mode}")


@pytest.mark.parametrize("sets", [1, 64, 65, 4096, 4097, 4160, 4161, 8000, 8193])
def test_merge_finds_the_sets_of_a_tile(sets):
    """A wave looks for the first set of its tile with 64 probes a round: set counts at the edges of one (64),
    two (4160) and three rounds, set sizes of 1 and 2 with a long set first and one last (the long sets are
    looked up 4096 at a time, so from 4097 sets on the last one is found in a later turn), a ragged second row."""
    rng = np.random.default_rng(sets)
    sizes = [rng.integers(1, 3, sets), rng.integers(1, 2, sets)]
    for s in sizes:
        s[0] += 520
        s[-1] += 700
    lens = [int(s.sum()) for s in sizes]
    n = max(lens)
    _say(f"merge: {sets} sets over {lens} tokens")
    Q, K, V = _slices(35, 2, 1, lens, n, 128, 1, "f16", rho=0.97)
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    st = np.zeros((2, 1, n + 1), np.int32)
    pv = np.full((2, 1, n), -1, np.int32)
    for b in range(2):
        starts = np.concatenate([[0], np.cumsum(sizes[b])])
        st[b, 0, :sets + 1], st[b, 0, sets + 1:] = starts, lens[b]
        pv[b, 0, :sets] = starts[:-1] + rng.integers(0, sizes[b])
    o = dict(set_start=st, pivot=pv, n_sets=np.full((2, 1), sets, np.int32), cap_rows=n)
    res = _merge_both(K, V, "f16", params, o, lens)
    _check_merge(K, V, "f16", o, *res, f"{sets} sets")


@pytest.mark.parametrize("slices", [64, 65])
def test_merge_gives_the_same_bits_for_every_tile_size(slices):
    """Tiles of 16 tokens up to 2^18 tokens, of 32 beyond: slices of a launch on either side of the line have to
    give the bits of the same slice merged alone (16-token tiles)."""
    n = 4096
    _say(f"merge: {slices} slices of {n} tokens")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(slices)
    K = torch.randn((1, slices, n, 128), generator=gen, device="cuda").to(torch.float16)
    K[:, :, 1::3] = K[:, :, 0::3][:, :, :K[:, :, 1::3].shape[2]]
    K[:, :, 1000:1700] = K[:, :, 1000:1001]                 # one long set
    V = torch.randn((1, slices, n, 128), generator=gen, device="cuda").to(torch.float16)
    params = kb.make_params(1.0, 0.1, 0.1, enforce_budget=False)
    sh = kb.make_shape(K, 1, None)
    buf = kb.Buffers(sh, params, "cuda", torch.float16)
    buf.mass.copy_(torch.rand((1, slices, n), generator=gen, device="cuda"))
    kb.kvm_identify_sets(sh, params, K, buf.mass, buf.set_id, buf.set_start, buf.pivot, buf.n_sets, None, buf.status, buf.ws)
    buf.K_out.fill_(7.0)
    buf.V_out.fill_(7.0)
    kb.kvm_merge(sh, params, K, V, buf.set_start, buf.pivot, buf.n_sets, buf.K_out, buf.V_out, None, buf.ws)
    for h in (0, slices // 2, slices - 1):
        one = slice(h, h + 1)
        Ki, Vi = K[:, one].contiguous(), V[:, one].contiguous()
        Ko, Vo = torch.full_like(buf.K_out[:, one], 7.0), torch.full_like(buf.V_out[:, one], 7.0)
        maps = [t[:, one].contiguous() for t in (buf.set_start, buf.pivot, buf.n_sets)]
        kb.kvm_merge(kb.make_shape(Ki, 1, None), params, Ki, Vi, *maps, Ko, Vo, None, buf.ws)
        assert torch.equal(Ko.view(torch.int16), buf.K_out[:, one].contiguous().view(torch.int16))
        assert torch.equal(Vo.view(torch.int16), buf.V_out[:, one].contiguous().view(torch.int16))


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("mode", ["adaptive", "fixed", "average"])
def test_merge_gives_the_same_bits_by_one_wave_four_or_the_refresh(dtype, mode):
    """Sets of more than 128 tokens are summed in four parts: by four waves in launches of up to 96 K tokens and in the
    refresh, one after the other by one wave beyond.  Sizes at the edges of a batch, of the split and of its parts (the last
    ones of which are empty for 129 to 144 tokens), rows and weights bit for bit the same, and the oracle's."""
    _say(f"merge: the same bits by one wave, four and the refresh, {dtype} {mode}")
    sizes = np.array([1, 16, 17, 2, 64, 65, 127, 128, 129, 144, 145, 1, 1, 160, 176, 177, 192, 193, 255, 256, 257, 31, 400, 497, 511, 512, 3])
    n, M = int(sizes.sum()), len(sizes)
    copies = 3 * 2 ** 15 // n + 1
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    rng = np.random.default_rng(5)
    Q, K, V = _slices(36, 1, 1, [n], n, 128, 1, dtype, rho=0.9)
    starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    piv = (starts[:-1] + rng.integers(0, sizes)).astype(np.int32)
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    if mode == "fixed":
        params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 9.0
    if mode == "average":
        params.weights = kb.KVM_WEIGHTS_AVERAGE
    results = []
    for S in (1, copies):
        Kd, Vd = (gu.to_dev(x, dtype).expand(1, S, n, 128).contiguous() for x in (K, V))
        sh = kb.make_shape(Kd, 1, None)
        b = kb.Buffers(sh, params, "cuda", dt, with_debug=True)
        for t, v, fill in ((b.set_start, starts, n), (b.pivot, piv, -1)):
            t.fill_(fill)
            t[0, :, :len(v)] = torch.from_numpy(v).cuda()
        b.n_sets.fill_(M)
        kb.kvm_merge(sh, params, Kd, Vd, b.set_start, b.pivot, b.n_sets, b.K_out, b.V_out, b.w, b.ws)
        results.append([t[0, -1].clone() for t in (b.K_out[:, :, :M], b.V_out[:, :, :M], b.w)])
        b.K_out.zero_()
        b.V_out.zero_()
        none = [torch.full_like(t, -1) for t in (b.set_id, b.set_start, b.pivot)] + [torch.zeros_like(b.n_sets)]
        kb.kvm_merge_refresh(sh, params, Kd, Vd, *none, b.set_start, b.pivot, b.n_sets, b.K_out, b.V_out, None, b.ws)
        results.append([t[0, -1].clone() for t in (b.K_out[:, :, :M], b.V_out[:, :, :M])])
    for other in results[1:]:
        for name, x, y in zip("KVw", results[0], other):
            assert torch.equal(x, y), name
    rk, rv, _ = ref.merge(K, V, dtype, starts[None, None], piv[None, None], np.full((1, 1), M, np.int32), sigma_mode=params.sigma_mode,
                          sigma=params.sigma, weights=params.weights)
    for got, want in zip(results[0], (rk, rv)):
        err = np.abs(got.double().cpu().numpy() - want[0, 0, :M]).max(axis=-1) / np.abs(want[0, 0, :M]).max(axis=-1)
        assert err.max() <= gu.TOL + 2.0 ** (-8 if dtype == "bf16" else -11)      # fp32 arithmetic, one rounding to the cache type


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_merge_sets_of_two_batches(dtype):
    """Sets of 17 to 32 tokens keep their second batch in registers: all sizes around them, the pivot in either batch, rows
    the same with and without the weights written, by the refresh, and the oracle's (fp32 sums, one rounding to the type)."""
    _say(f"merge: sets of two batches, {dtype}")
    rng = np.random.default_rng(8)
    sizes = np.concatenate([np.arange(14, 36), [1, 1, 1], np.arange(35, 13, -1), [48, 49]])
    n, M = int(sizes.sum()), len(sizes)
    Q, K, V = _slices(41, 1, 1, [n], n, 128, 1, dtype, rho=0.9)
    starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    piv = (starts[:-1] + rng.integers(0, sizes)).astype(np.int32)
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    Kd, Vd = gu.to_dev(K, dtype), gu.to_dev(V, dtype)
    sh = kb.make_shape(Kd, 1, None)
    b = kb.Buffers(sh, params, "cuda", Kd.dtype, with_debug=True)
    for t, v, fill in ((b.set_start, starts, n), (b.pivot, piv, -1)):
        t.fill_(fill)
        t[0, 0, :len(v)] = torch.from_numpy(v).cuda()
    b.n_sets.fill_(M)
    results = []
    for w in (b.w, None):
        kb.kvm_merge(sh, params, Kd, Vd, b.set_start, b.pivot, b.n_sets, b.K_out, b.V_out, w, b.ws)
        results.append([t[0, 0, :M].clone() for t in (b.K_out, b.V_out)])
    none = [torch.full_like(t, -1) for t in (b.set_id, b.set_start, b.pivot)] + [torch.zeros_like(b.n_sets)]
    kb.kvm_merge_refresh(sh, params, Kd, Vd, *none, b.set_start, b.pivot, b.n_sets, b.K_out, b.V_out, None, b.ws)
    results.append([t[0, 0, :M].clone() for t in (b.K_out, b.V_out)])
    for other in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(results[0], other))
    rk, rv, rw = ref.merge(K, V, dtype, starts[None, None], piv[None, None], np.full((1, 1), M, np.int32))
    for got, want in zip(results[0], (rk, rv)):
        err = np.abs(got.double().cpu().numpy() - want[0, 0, :M]).max(axis=-1) / np.abs(want[0, 0, :M]).max(axis=-1)
        assert err.max() <= gu.TOL + 2.0 ** (-8 if dtype == "bf16" else -11)
    assert np.abs(b.w.cpu().numpy() - rw).max() <= gu.TOL


def test_merge_rounds_bf16_rows_like_the_storage_type():
    """The merged rows' rounding to bf16, on means that are exact in fp32: of two equal rows the row itself for every finite pattern whose
    sum does not overflow, subnormals among them; of two neighbours, half way between them, the even one; NaN stays NaN."""
    _say("merge: rounding of bf16 rows")
    x = np.arange(65536, dtype=np.uint16).reshape(512, 128)
    up = np.minimum(x.astype(np.uint32) + 1, 65535).astype(np.uint16)
    params = kb.make_params(1.0, 0.0, 0.0, value_scale_by_set_size=False, enforce_budget=False, weights=kb.KVM_WEIGHTS_AVERAGE)
    n, M = 1024, 512
    starts = np.full((1, 1, n + 1), n, np.int32)
    starts[..., :M] = 2 * np.arange(M)
    pivot = np.full((1, 1, n), -1, np.int32)
    pivot[..., :M] = starts[..., :M]
    for other in (x, up):
        rows = np.stack([x, other], 1).reshape(1, 1, n, 128)
        Ko, Vo, _, _, _ = gu.gpu_merge(rows, rows, "bf16", params, starts, pivot, np.full((1, 1), M, np.int32))
        f = (rows.astype(np.uint32) << 16).view(np.float32).reshape(M, 2, 128)
        with np.errstate(all="ignore"):
            mean = (f[:, 0] + f[:, 1]) * np.float32(0.5)
            exact = (f[:, 0].astype(np.float64) + f[:, 1]) * 0.5
        u = mean.view(np.uint32)
        want = ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)
        sure, nan = np.isfinite(f).all(axis=1) & (mean == exact), np.isnan(f).any(axis=1)
        assert sure.mean() > 0.98
        for got in (Ko[0, 0, :M], Vo[0, 0, :M]):
            assert np.array_equal(got[sure].astype(np.float32), want[sure])
            assert np.isnan(got[nan]).all()


@pytest.mark.parametrize("N,copies,rows", [(1, 20200, 13), (40, 600, 13), (100, 210, 13), (256, 80, 13), (700, 29, 13), (4096, 22, 3), (4097, 22, 3)])
def test_merge_of_large_launches_of_short_slices(N, copies, rows):
    """Launches of more than 2^18 tokens deal out slices of up to 128 tiles in groups of eight, each group starting at
    another tile: one to 129 tiles a slice, slice counts that leave a rest, ragged lengths.  Every copy of a slice has to
    give the bits of that slice in a small launch, and nothing beyond its rows is written."""
    lens = [N - (N * b) // (2 * rows) for b in range(rows)]
    _say(f"merge: {copies} copies of {rows} slices of {lens[-1]}..{N} tokens")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    K = torch.randn((rows, 1, N, 128), generator=gen, device="cuda").to(torch.float16)
    if N > 40:
        K[:, :, 10:35] = K[:, :, 10:11]                       # a set across the edge of a tile
    V = torch.randn((rows, 1, N, 128), generator=gen, device="cuda").to(torch.float16)
    mass = torch.rand((rows, 1, N), generator=gen, device="cuda")
    params = kb.make_params(1.0, 0.1, 0.1, threshold=0.02, enforce_budget=False)

    def run(rep):
        k, v = K.repeat(rep, 1, 1, 1), V.repeat(rep, 1, 1, 1)
        sh = kb.make_shape(k, 1, gu.lens_dev(lens * rep))
        buf = kb.Buffers(sh, params, "cuda", torch.float16)
        buf.mass.copy_(mass.repeat(rep, 1, 1))
        kb.kvm_identify_sets(sh, params, k, buf.mass, buf.set_id, buf.set_start, buf.pivot, buf.n_sets, None, buf.status, buf.ws)
        w = torch.full((rows * rep, 1, N), 7.0, dtype=torch.float32, device="cuda")
        buf.K_out.fill_(7.0)
        buf.V_out.fill_(7.0)
        kb.kvm_merge(sh, params, k, v, buf.set_start, buf.pivot, buf.n_sets, buf.K_out, buf.V_out, w, buf.ws)
        return [t.view(rep, rows, -1) for t in (buf.K_out.view(torch.int16), buf.V_out.view(torch.int16), w.view(torch.int32))]

    assert rows * N <= 1 << 18 < rows * N * copies
    for few, many in zip(run(1), run(copies)):
        assert torch.equal(many, few.expand_as(many))


@pytest.mark.parametrize("slices", [2, 33])
def test_merge_with_empty_sets_between(slices):
    """Maps that a caller made itself may hold sets without tokens: up to 64 sets may start in a tile of tokens, whatever
    its size (16 tokens in a small launch, 32 in a large one), and the sets with tokens have to come out as from the same
    maps without the empty ones."""
    n, empty = 8192, 20
    _say(f"merge: {empty} empty sets at three places, {slices} slices")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(slices)
    K, V = (torch.randn((1, slices, n, 128), generator=gen, device="cuda").to(torch.float16) for _ in range(2))
    starts = np.arange(0, n, 3)
    at = [0, 1001, len(starts) - 1]                          # empty sets in front of these sets
    keep = np.arange(len(starts)) + empty * np.searchsorted(at, np.arange(len(starts)), side="right")
    padded = np.insert(starts, np.repeat(at, empty), np.repeat(starts[at], empty))
    assert np.array_equal(padded[keep], starts)
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    sh = kb.make_shape(K, 1)
    out = []
    for st in (starts, padded):
        set_start = torch.full((1, slices, n + 1), n, dtype=torch.int32, device="cuda")
        pivot = torch.full((1, slices, n), -1, dtype=torch.int32, device="cuda")
        set_start[:, :, :len(st)] = pivot[:, :, :len(st)] = torch.from_numpy(st.astype(np.int32)).cuda()
        n_sets = torch.full((1, slices), len(st), dtype=torch.int32, device="cuda")
        o = [torch.full((1, slices, n, 128), 7.0, dtype=torch.float16, device="cuda") for _ in range(2)]
        ws = torch.empty(kb.kvm_workspace_bytes(sh, params), dtype=torch.uint8, device="cuda")
        kb.kvm_merge(sh, params, K, V, set_start, pivot, n_sets, *o, None, ws)
        out.append(o)
    for want, got in zip(*out):
        assert torch.equal(got[:, :, torch.from_numpy(keep).cuda()].view(torch.int16), want[:, :, :len(starts)].view(torch.int16))


def test_merge_tolerates_inconsistent_maps():
    n = 256
    _say("merge: out-of-range map entries are clamped, nothing faults")
    Q, K, V = _slices(33, 1, 1, [n], n, 128, 1, "f16")
    params = kb.make_params(0.5, 0.1, 0.1)
    cap = n // 2
    st = np.full((1, 1, cap + 1), 10 ** 9, np.int32)
    st[0, 0, :4] = [-5, 3, 2, 100000]
    pv = np.full((1, 1, cap), -(10 ** 9), np.int32)
    ko, vo, w, Kt, Vt = gu.gpu_merge(K, V, "f16", params, st, pv, np.array([[10 ** 6]], np.int32), want_w=False)
    assert np.isfinite(ko).all() and np.isfinite(vo).all()


@pytest.mark.parametrize("dtype,mode", [("f16", "gaussian"), ("bf16", "fixed_sigma"), ("f32", "average")])
def test_merge_refresh_over_decode_steps(dtype, mode):
    """Decode-time loop on a growing sequence: scores updated by one query row, one new similarity,
    sets identified again, and the compacted cache brought up to date by kvm_merge_refresh (rows of
    unchanged sets moved, the others merged again).  After every one of 20 steps the cache must be,
    bit for bit, what kvm_merge gives on the new maps; the last one is also held against the oracle.
    The second batch row is 300 tokens shorter and one slice has a run of identical keys, i.e. a set
    long enough for the workgroup-per-set kernel that keeps growing."""
    n0, steps, N = 1500, 20, 1536
    n1 = n0 + steps
    lens1 = [n1, n1 - 300]
    _say(f"merge refresh over decode steps {n0}..{n1}, {dtype}, {mode}")
    Q, K, V = _slices(41, 2, 2, lens1, N, 128, 1, dtype)
    K[0, 1, 200:n1] = K[0, 1, 200]                         # one long run of identical keys, up to the newest token
    params = kb.kvm_params_for_budget(0.5)
    if mode == "fixed_sigma":
        params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 4.0
    elif mode == "average":
        params.weights = kb.KVM_WEIGHTS_AVERAGE
    Qd, Kd, Vd = gu.to_dev(Q, dtype), gu.to_dev(K, dtype), gu.to_dev(V, dtype)
    tdt = gu.TORCH_DT[dtype]
    i32 = dict(dtype=torch.int32, device="cuda")

    def shape_at(lens):
        sl = gu.lens_dev(lens)
        return kb.make_shape(Kd, 1, sl)

    sh = shape_at([n0, n0 - 300])
    cap = kb.kvm_out_capacity(sh, params)
    ws = torch.empty(max(kb.kvm_workspace_bytes(sh, params), 256), dtype=torch.uint8, device="cuda")
    mass = torch.empty((2, 2, N), dtype=torch.float32, device="cuda")
    sim = torch.empty((2, 2, N), dtype=torch.float32, device="cuda")
    maps = [dict(set_id=torch.full((2, 2, N), -7, **i32), set_start=torch.full((2, 2, cap + 1), -7, **i32),
                 pivot=torch.full((2, 2, cap), -7, **i32), n_sets=torch.full((2, 2), -7, **i32),
                 status=torch.full((2, 2), -7, **i32)) for _ in range(2)]
    Ko = torch.zeros((2, 2, cap, 128), dtype=tdt, device="cuda")
    Vo = torch.zeros_like(Ko)
    n_changed = torch.full((2, 2), -1, **i32)

    def identify(sh, m, given):
        params.sim_given = 1 if given else 0
        kb.kvm_identify_sets(sh, params, Kd, mass, m["set_id"], m["set_start"], m["pivot"], m["n_sets"], sim, m["status"], ws)

    # prefill: the whole pass once
    kb.kvm_attn_mass(sh, Qd, Kd, mass, ws)
    identify(sh, maps[0], False)
    kb.kvm_merge(sh, params, Kd, Vd, maps[0]["set_start"], maps[0]["pivot"], maps[0]["n_sets"], Ko, Vo, None, ws)
    cur = 0
    total_changed = 0
    bits = torch.int32 if dtype == "f32" else torch.int16
    for step in range(1, steps + 1):
        lens = [n0 + step, n0 + step - 300]
        sh = shape_at(lens)
        q_new = torch.stack([Qd[b, :, n - 1] for b, n in enumerate(lens)]).contiguous()
        kb.kvm_attn_mass_append(sh, q_new, Kd, mass, ws)
        kb.kvm_sim_append(sh, Kd, sim)
        new = 1 - cur
        identify(sh, maps[new], True)
        kb.kvm_merge_refresh(sh, params, Kd, Vd, maps[cur]["set_id"], maps[cur]["set_start"], maps[cur]["pivot"],
                             maps[cur]["n_sets"], maps[new]["set_start"], maps[new]["pivot"], maps[new]["n_sets"], Ko, Vo,
                             n_changed, ws)
        Kf = torch.zeros_like(Ko)
        Vf = torch.zeros_like(Vo)
        kb.kvm_merge(sh, params, Kd, Vd, maps[new]["set_start"], maps[new]["pivot"], maps[new]["n_sets"], Kf, Vf, None, ws)
        torch.cuda.synchronize()
        ns = maps[new]["n_sets"].cpu().numpy()
        for b in range(2):
            for h in range(2):
                M = min(int(ns[b, h]), cap)
                assert torch.equal(Ko[b, h, :M].view(bits), Kf[b, h, :M].view(bits)), f"step {step} slice ({b},{h}): K rows differ"
                assert torch.equal(Vo[b, h, :M].view(bits), Vf[b, h, :M].view(bits)), f"step {step} slice ({b},{h}): V rows differ"
        ch = n_changed.cpu().numpy()
        assert (ch >= 1).all() and (ch <= ns).all()          # the set that holds the newest token is always new
        total_changed += int(ch.sum())
        cur = new
    _say(f"  sets merged again per step and slice: {total_changed / (steps * 4):.1f} of about {int(ns.mean())}")
    assert total_changed < 0.2 * steps * ns.sum()            # the point of the call: most rows are kept
    # the final state against the oracle: maps from the library's own scores, merged rows to the merge bar
    params.sim_given = 0
    m_g = mass.cpu().numpy()
    o = ref.identify_sets(K, m_g.astype(np.float64), dtype, params.budget, params.recent_ratio, params.heavy_ratio,
                          params.threshold, True, cap, lens1)
    g = {k: v.cpu().numpy() for k, v in maps[cur].items()}
    g["cap_rows"] = cap
    exc, _ = gu.compare_maps(g, o, lens1, N, params.threshold, "refresh, final maps")
    assert exc == 0
    rk, rv, _ = ref.merge(K, V, dtype, o["set_start"], o["pivot"], o["n_sets"], params.sigma_mode, params.sigma,
                          bool(params.value_scale_by_set_size), lens1, weights=params.weights)
    for b in range(2):
        for h in range(2):
            M = min(int(o["n_sets"][b, h]), cap)
            assert gu.row_rel_err(gu.to_host_f64(Ko[b, h, :M]), rk[b, h, :M]).max() <= gu.kv_tol(dtype)
            assert gu.row_rel_err(gu.to_host_f64(Vo[b, h, :M]), rv[b, h, :M]).max() <= gu.kv_tol(dtype)
            assert gu.ulp_excess(gu.to_host_f64(Ko[b, h, :M]), rk[b, h, :M], dtype).max() <= 2e-5
            assert gu.ulp_excess(gu.to_host_f64(Vo[b, h, :M]), rv[b, h, :M], dtype).max() <= 2e-5


# ---------------------------------------------------------------------------------------------
# whole pass
# ---------------------------------------------------------------------------------------------

def _explained_by_near_ties_in_mass(m_o, oi, og, ge, n, what):
    """The library's maps (equal to the oracle's rule on the library's own scores, checked before)
    differ from the oracle's maps on the oracle's scores: the first decision that went the other
    way has to be one between scores that the two sides agree on to within the tolerance of the
    scores themselves.  Conserved sets first (the exact top-k); if they agree the sets agree and
    only pivots can differ."""
    m = m_o[0, 0, :n]
    P_o, P_g = oi["protected"][0, 0, :n].astype(bool), og["protected"][0, 0, :n].astype(bool)
    if not np.array_equal(P_o, P_g):
        n_rec = int(P_o[::-1].argmin()) if not P_o.all() else n       # length of the trailing conserved window
        heavy = np.flatnonzero(P_o[:n - n_rec])
        assert len(heavy), f"{what}: conserved tokens differ without a top-k selection"
        T = m[heavy].min()                                            # the smallest selected score
        odd = np.flatnonzero(P_o != P_g)
        worst = np.abs(m[odd] / T - 1).max()
        assert worst <= 2.5 * gu.TOL, f"{what}: conserved tokens differ at scores {worst:.2e} away from the k-th largest"
        return "top-k near-tie"
    assert np.array_equal(ge["set_id"][0, 0, :n], oi["set_id"][0, 0, :n]), f"{what}: same conserved tokens, different sets"
    M = min(int(oi["n_sets"][0, 0]), oi["cap_rows"])
    pg, po = ge["pivot"][0, 0, :M], oi["pivot"][0, 0, :M]
    odd = np.flatnonzero(pg != po)
    assert len(odd), f"{what}: maps differ but neither conserved tokens, sets nor pivots do"
    worst = np.abs(m[pg[odd]] / m[po[odd]] - 1).max()
    assert worst <= 2.5 * gu.TOL, f"{what}: pivots differ between scores {worst:.2e} apart"
    return "pivot near-tie"


def _whole_pass(Q, K, V, dtype, G, params, lens, sample, what, device_tensors=None, slice_of=None,
                sim_from_score_pass=False):
    """GPU: the three calls back to back on all slices.  Oracle: the same on sampled slices.
    Stage by stage the oracle's inputs are its own.  End to end the library's maps must be exactly
    what the oracle's rule gives on the library's own fp32 scores (themselves checked against the
    oracle's scores first), the only excuse being a similarity within 1e-6 of the threshold; where
    they differ from the oracle's maps on the oracle's scores the deciding scores must be a near-tie.
    With device_tensors = (Qd, Kd, Vd) the inputs are already on the GPU and slice_of(b, h) returns
    the host copy (Q (G, N, d), K (N, d), V (N, d)) of a sampled slice.  sim_from_score_pass: the
    similarities come from kvm_attn_mass_sim instead of the sets' own scan of K."""
    if device_tensors is None:
        Qd, Kd, Vd = gu.to_dev(Q, dtype), gu.to_dev(K, dtype), gu.to_dev(V, dtype)
        slice_of = lambda b, h: (Q[b, h * G:(h + 1) * G], K[b, h], V[b, h])
    else:
        Qd, Kd, Vd = device_tensors
    sl = gu.lens_dev(lens)
    sh = kb.make_shape(Kd, G, sl)
    buf = kb.Buffers(sh, params, "cuda", gu.TORCH_DT[dtype], with_debug=True)
    kb.compress(sh, params, Qd, Kd, Vd, buf, sim_from_score_pass=sim_from_score_pass)
    torch.cuda.synchronize()
    B, H, N, d = Kd.shape
    g = dict(set_id=buf.set_id.cpu().numpy(), set_start=buf.set_start.cpu().numpy(), pivot=buf.pivot.cpu().numpy(),
             n_sets=buf.n_sets.cpu().numpy(), status=buf.status.cpu().numpy(), sim=buf.sim.cpu().numpy())
    gu.check_partition(g, lens, N, buf.cap, what)
    mass_g = buf.mass.cpu().numpy()
    differing = excused = 0
    for (b, h) in sample:
        n = N if lens is None else int(lens[b])
        _say(f"  {what}: oracle on slice ({b},{h}) n={n}")
        q_s, k_s, v_s = slice_of(b, h)
        Qs = np.ascontiguousarray(q_s)[None]
        Ks, Vs = np.ascontiguousarray(k_s)[None, None], np.ascontiguousarray(v_s)[None, None]
        ls = None if lens is None else [n]
        if G > 1:      # the query heads in parallel: the grouped score is the sum of the heads' scores
            m_o = ref.attn_mass(Qs.transpose(1, 0, 2, 3).copy(), np.repeat(Ks, G, 0), dtype,
                                seq_lens=None if ls is None else ls * G).sum(0, keepdims=True)
        else:
            m_o = ref.attn_mass(Qs, Ks, dtype, seq_lens=ls)
        gu.assert_mass_close(mass_g[b:b + 1, h:h + 1], m_o, ls, N, f"{what} ({b},{h})")
        # stage (b) and (c) on the oracle's own fp32-rounded mass
        m32 = m_o.astype(np.float32)
        gi = gu.gpu_identify(Ks, m32, dtype, params, ls)
        ident = lambda mass64, seed: ref.identify_sets(
            Ks, mass64, dtype, params.budget, params.recent_ratio, params.heavy_ratio, params.threshold,
            bool(params.enforce_budget), gi["cap_rows"], ls, pivot_rule=params.pivot_rule, pivot_seed=seed,
            set_rule=params.set_rule)
        oi = ident(m32.astype(np.float64), params.pivot_seed)
        anchor = params.set_rule == kb.KVM_SETS_ANCHOR
        if anchor:
            _compare_anchor_maps(gi, oi, f"{what} ({b},{h})")
        else:
            gu.compare_maps(gi, oi, ls, N, params.threshold, f"{what} ({b},{h})")
        res = _merge_both(Ks, Vs, dtype, params, oi, ls)
        _check_merge(Ks, Vs, dtype, oi, *res, f"{what} ({b},{h})")
        # end to end.  The draws of the random pivot depend on the slice's index in the call.
        seed_here = (params.pivot_seed + ((b * H + h) << 32)) % (1 << 64)
        ge = {k: g[k][b:b + 1, h:h + 1] for k in ("set_id", "set_start", "pivot", "n_sets", "status")}
        ge["cap_rows"] = buf.cap
        # (i) the oracle's rule on the library's own scores: bit-exact, similarities at the threshold excused
        og = ident(mass_g[b:b + 1, h:h + 1].astype(np.float64), seed_here)
        if anchor:
            excused += _compare_anchor_maps(ge, og, f"{what} ({b},{h}) on the library's scores")
        else:
            excused += gu.compare_maps(ge, og, ls, N, params.threshold, f"{what} ({b},{h}) on the library's scores")[0]
        # (ii) against the oracle's maps on the oracle's scores
        oe = oi if params.pivot_rule != kb.KVM_PIVOT_RANDOM else ident(m32.astype(np.float64), seed_here)
        same = all(np.array_equal(ge[k][0, 0], oe[k][0, 0]) for k in ("set_id", "set_start", "pivot"))
        if same:
            M = min(int(oe["n_sets"][0, 0]), buf.cap)
            rk, rv = res[3], res[4]
            if oe is not oi:
                rk, rv, _ = ref.merge(Ks, Vs, dtype, oe["set_start"], oe["pivot"], oe["n_sets"], params.sigma_mode,
                                      params.sigma, bool(params.value_scale_by_set_size), ls, weights=params.weights)
            ek = gu.row_rel_err(gu.to_host_f64(buf.K_out[b, h, :M]), rk[0, 0, :M]).max() if M else 0.0
            ev = gu.row_rel_err(gu.to_host_f64(buf.V_out[b, h, :M]), rv[0, 0, :M]).max() if M else 0.0
            assert ek <= gu.kv_tol(dtype) and ev <= gu.kv_tol(dtype), \
                f"{what} ({b},{h}): end-to-end K/V error {ek:.2e}/{ev:.2e}"
        else:
            differing += 1
            near_sim = np.abs(oe["sim"][0, 0, 1:n] - params.threshold).min() <= gu.NEAR if n > 1 else False
            if anchor:
                near_sim = oe["anchor_margin"][0, 0] <= gu.NEAR
            why = "similarity at the threshold" if near_sim else \
                _explained_by_near_ties_in_mass(m_o, oe, og, ge, n, f"{what} ({b},{h})")
            _say(f"  {what} ({b},{h}): end-to-end maps differ from the oracle's on its own scores: {why}")
    _say(f"  {what}: {differing} of {len(sample)} sampled slices have end-to-end maps that differ "
         f"(each explained by a near-tie); {excused} excused by a similarity at the threshold")
    return g


def test_whole_pass_config1():
    cfg = synth.CONFIGS[1]
    _say("whole pass: config 1")
    Q, K, V, _ = synth.gen_config(cfg)
    g = _whole_pass(Q, K, V, "f32", 1, kb.kvm_params_for_budget(0.5), None, [(0, 0)], "config 1")
    assert g["n_sets"][0, 0] <= 256 and g["status"][0, 0] == 0


@pytest.mark.parametrize("cfg_id,layers,budget", [(2, 2, 0.5), (2, 1, 0.35), (3, 1, 0.35)])
def test_whole_pass_reduced_layers(cfg_id, layers, budget):
    cfg = synth.CONFIGS[cfg_id]
    _say(f"whole pass: config {cfg_id}, {layers} layer(s), budget {budget}")
    Q, K, V, lens = synth.gen_config(cfg, layers=layers)
    H = cfg["H_kv"]
    sample = [(0, 0), (layers - 1, H - 1), (0, H // 2)]
    g = _whole_pass(Q, K, V, cfg["dtype"], cfg["G"], kb.kvm_params_for_budget(budget), lens, sample,
                    f"config {cfg_id}")
    assert (g["n_sets"] <= math.floor(budget * cfg["N"])).all()
    _say(f"  mean M/n = {g['n_sets'].mean() / cfg['N']:.3f}, fallback slices {(g['status'] != 0).sum()}")


def test_whole_pass_config4_grouped_queries_long():
    cfg = synth.CONFIGS[4]
    _say("whole pass: config 4 shape (G=4, N=16384), one layer")
    Q, K, V, lens = synth.gen_config(cfg, layers=1)
    g = _whole_pass(Q, K, V, "bf16", 4, kb.kvm_params_for_budget(0.5), None, [(0, 3)], "config 4")
    # the same pass with the similarities written by the column-sum kernels (one layer: the split kernel, two: the
    # four-block kernel): the same maps, unless a similarity sits within the two paths' rounding of the threshold
    params = kb.kvm_params_for_budget(0.5)
    for layers, kernel in ((1, "attn_colsum_split_kernel"), (2, "attn_colsum_pipe_kernel")):
        Qd, Kd, Vd = (gu.to_dev(x, "bf16").repeat(layers, 1, 1, 1) for x in (Q, K, V))
        sh = kb.make_shape(Kd, 4, None)
        bufs = [kb.Buffers(sh, params, "cuda", torch.bfloat16, with_sim=True) for _ in range(2)]
        kb.compress(sh, params, Qd, Kd, Vd, bufs[0])
        assert kernel in gu.kernels_of(lambda: kb.compress(sh, params, Qd, Kd, Vd, bufs[1], sim_from_score_pass=True))
        assert torch.equal(bufs[0].mass, bufs[1].mass)
        np.testing.assert_allclose(bufs[1].sim.cpu().numpy(), bufs[0].sim.cpu().numpy(), atol=2e-6)
        for h in range(8):
            same = all(torch.equal(getattr(bufs[0], k)[:, h], getattr(bufs[1], k)[:, h]) for k in ("set_id", "set_start", "pivot", "n_sets"))
            near = (bufs[0].sim[:, h, 1:] - params.threshold).abs().min().item() <= 2e-6
            assert same or near, f"head {h}: maps differ between the two ways to get the similarities"
    assert (g["n_sets"] <= 8192).all()


def test_whole_pass_config5_ragged_batch():
    cfg = dict(synth.CONFIGS[5], H_kv=4)         # four of the 32 heads of one layer, all four lengths
    _say("whole pass: config 5 shape (B=4 ragged, N=16384 padded), one layer, 4 heads")
    Q, K, V, lens = synth.gen_config(cfg, layers=1)
    g = _whole_pass(Q, K, V, "f16", 1, kb.kvm_params_for_budget(0.35), lens, [(0, 0), (1, 1), (2, 2), (3, 3)],
                    "config 5")
    for b, n in enumerate(lens):
        assert (g["n_sets"][b] <= math.floor(0.35 * n)).all()


def test_whole_pass_config2_full_size_sampled():
    """The headline workload whole (1024 slices in one launch of every kernel, as the benchmark
    times it): the oracle on a spread sample of slices, size-independent properties on all."""
    cfg = synth.CONFIGS[2]
    L, H, N = cfg["layers"], cfg["H_kv"], cfg["N"]
    _say(f"whole pass: config 2 at full size ({L} layers x {H} heads)")
    Q, K, V, lens = synth.gen_config(cfg)
    sample = [(0, 0), (L - 1, H - 1), (7, 13), (16, 5), (21, 30), (30, 1)]
    params = kb.kvm_params_for_budget(0.5)
    g = _whole_pass(Q, K, V, "f16", 1, params, lens, sample, "config 2 full")
    assert g["n_sets"].shape == (L, H) and (g["n_sets"] <= N // 2).all() and (g["n_sets"] > 0).all()
    assert (g["status"] == 0).all()
    # every attention row sums to one, so a slice's scores sum to its length
    Kd = gu.to_dev(K, "f16")
    sh = kb.make_shape(Kd, 1, None)
    mass = torch.empty((L, H, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(kb.kvm_workspace_bytes(sh, params), dtype=torch.uint8, device="cuda")
    kb.kvm_attn_mass(sh, gu.to_dev(Q, "f16"), Kd, mass, ws)
    tot = mass.double().sum(-1).cpu().numpy()
    assert np.abs(tot / N - 1).max() <= 1e-5, f"scores of a slice do not sum to n: {np.abs(tot / N - 1).max():.2e}"
    assert (mass[:, :, 0] >= 1).all() and (mass[:, :, N - 1] <= 1).all() and (mass > 0).all()


@pytest.mark.parametrize("cfg_id,budget", [(3, 0.35), (4, 0.5)])
def test_whole_pass_large_configs_full_size_sampled(cfg_id, budget):
    """Workloads 3 and 4 whole, as the benchmark launches them; the oracle on one slice of every
    length from the last layer (the highest addresses), partition properties on all slices."""
    cfg = synth.CONFIGS[cfg_id]
    _say(f"whole pass: config {cfg_id} at full size")
    Q, K, V, lens = synth.gen_config(cfg)
    B, H = K.shape[0], cfg["H_kv"]
    per = cfg["batch"]
    sample = [(B - per + i, (7 * i + 3) % H) for i in range(per)] + [(0, 0)]
    g = _whole_pass(Q, K, V, cfg["dtype"], cfg["G"], kb.kvm_params_for_budget(budget), lens, sample,
                    f"config {cfg_id} full")
    n_b = np.full(B, cfg["N"]) if lens is None else np.asarray(lens)
    assert (g["n_sets"] <= np.floor(budget * n_b)[:, None]).all() and (g["n_sets"] > 0).all()


def test_whole_pass_config5_full_size_sampled():
    """Workload 5 whole (4 x 32 x 32 slices padded to 16384 tokens, 16 GiB per tensor, offsets
    beyond 2^32 together with per-sequence lengths), in the launch the benchmark times.  The
    inputs are generated and copied to the GPU one layer at a time, so the host never holds more
    than one layer; the host copies of the sampled slices (one of every length from the last layer,
    one from the first) are kept for the oracle."""
    cfg = synth.CONFIGS[5]
    budget = 0.35
    L, per, H, G, N, d, dtype = cfg["layers"], cfg["batch"], cfg["H_kv"], cfg["G"], cfg["N"], cfg["d"], cfg["dtype"]
    B = L * per
    _say("whole pass: config 5 at full size, filled layer by layer")
    tdt = gu.TORCH_DT[dtype]
    Qd = torch.empty((B, H * G, N, d), dtype=tdt, device="cuda")
    Kd = torch.empty((B, H, N, d), dtype=tdt, device="cuda")
    Vd = torch.empty((B, H, N, d), dtype=tdt, device="cuda")
    sample = [(B - per + i, (7 * i + 3) % H) for i in range(per)] + [(0, 0)]
    kept = {}
    lens = None
    for layer, (Q, K, V, sl) in enumerate(synth.gen_config_layers(cfg)):
        b0 = layer * per
        Qd[b0:b0 + per].copy_(gu.to_dev(Q, dtype))
        Kd[b0:b0 + per].copy_(gu.to_dev(K, dtype))
        Vd[b0:b0 + per].copy_(gu.to_dev(V, dtype))
        for (b, h) in sample:
            if b0 <= b < b0 + per:
                kept[(b, h)] = (Q[b - b0, h * G:(h + 1) * G].copy(), K[b - b0, h].copy(), V[b - b0, h].copy())
        lens = sl if lens is None else np.concatenate([lens, sl])
        if layer % 8 == 7:
            _say(f"  {layer + 1} of {L} layers on the GPU")
    g = _whole_pass(None, None, None, dtype, G, kb.kvm_params_for_budget(budget), lens, sample, "config 5 full",
                    device_tensors=(Qd, Kd, Vd), slice_of=lambda b, h: kept[(b, h)])
    assert (g["n_sets"] <= np.floor(budget * np.asarray(lens))[:, None]).all() and (g["n_sets"] > 0).all()


@pytest.mark.parametrize("variant", ["average_last", "gaussian_random", "fixed_sigma", "anchor_sets"])
def test_whole_pass_variants(variant):
    """The configurations the paper compares its method with (Section 4.2 first experiment,
    Section 5.4), end to end on two layers of the headline shape."""
    cfg = synth.CONFIGS[2]
    _say(f"whole pass: variant {variant}")
    Q, K, V, lens = synth.gen_config(cfg, layers=2)
    params = kb.kvm_params_for_budget(0.5)
    if variant == "average_last":
        params.weights, params.pivot_rule = kb.KVM_WEIGHTS_AVERAGE, kb.KVM_PIVOT_LAST
    elif variant == "gaussian_random":
        params.pivot_rule, params.pivot_seed = kb.KVM_PIVOT_RANDOM, 2024
    elif variant == "anchor_sets":
        params.set_rule, params.enforce_budget = kb.KVM_SETS_ANCHOR, 0
    else:
        params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 5.0
    g = _whole_pass(Q, K, V, "f16", 1, params, lens, [(0, 0), (1, 31)], variant)
    if variant != "anchor_sets":
        assert (g["n_sets"] <= cfg["N"] // 2).all()
    else:
        _say(f"  anchor rule: mean M/n = {g['n_sets'].mean() / cfg['N']:.3f}")


@pytest.mark.parametrize("case", range(12))
def test_whole_pass_random_shapes(case):
    """Seeded random shapes, lengths, group sizes, types, budgets and variants: every slice of a
    small batch goes through the oracle."""
    rng = np.random.default_rng(1000 + case)
    dtype = ["f16", "bf16", "f32"][case % 3]
    B, H, G = int(rng.integers(1, 4)), int(rng.integers(1, 4)), int(rng.choice([1, 2, 4]))
    N = int(rng.choice([1, 63, 64, 65, 255, 256, 257, 511, 513, 700, 1025, 1300]))
    lens = [int(x) for x in rng.integers(0, N + 1, B)]
    lens[int(rng.integers(0, B))] = N                        # one sequence at full length
    budget = float(rng.choice([0.35, 0.5, 0.8]))
    params = kb.kvm_params_for_budget(budget)
    params.weights = int(rng.choice([kb.KVM_WEIGHTS_GAUSSIAN, kb.KVM_WEIGHTS_AVERAGE]))
    params.pivot_rule = int(rng.choice([kb.KVM_PIVOT_MAX_SCORE, kb.KVM_PIVOT_LAST, kb.KVM_PIVOT_RANDOM]))
    params.pivot_seed = int(rng.integers(0, 1 << 40))
    params.set_rule = int(rng.choice([kb.KVM_SETS_ADJACENT, kb.KVM_SETS_ANCHOR]))
    params.threshold = float(rng.choice([0.6, 0.75, 0.9]))
    _say(f"random shapes {case}: {dtype} B={B} H={H} G={G} N={N} lens={lens} budget={budget} "
         f"weights={params.weights} pivot={params.pivot_rule} sets={params.set_rule} eps={params.threshold}")
    Q, K, V = _slices(2000 + case, B, H, lens, N, 128, G, dtype)
    sample = [(b, h) for b in range(B) for h in range(H)]
    _whole_pass(Q, K, V, dtype, G, params, lens, sample, f"random shapes {case}", sim_from_score_pass=case % 2 == 1)


# ---------------------------------------------------------------------------------------------
# comparison workload: eviction by score
# ---------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_evict_matches_the_oracle(dtype):
    n = 2100
    lens = [n, 1000, 0, 1, 77]
    _say(f"evict: {dtype}, lens {lens}")
    Q, K, V = _slices(35, 5, 2, lens, n, 128, 1, dtype)
    rng = np.random.default_rng(9)
    mass = (rng.random((5, 2, n)) + 0.01).astype(np.float32)
    mass[0, 0, 300:700] = mass[0, 0, 300]                    # ties: the lower index is kept first
    for budget, recent in ((0.5, 0.17), (0.35, 0.08), (0.3, 0.3), (1.0, 0.0)):   # plain, plain, window only, keep all
        params = kb.make_params(budget, recent, 0.0)
        Kd, Vd = gu.to_dev(K, dtype), gu.to_dev(V, dtype)
        sh = kb.make_shape(Kd, 1, gu.lens_dev(lens))
        cap = kb.kvm_out_capacity(sh, params)
        kept = torch.full((5, 2, cap), -7, dtype=torch.int32, device="cuda")
        n_kept = torch.full((5, 2), -7, dtype=torch.int32, device="cuda")
        Ko = torch.zeros((5, 2, cap, 128), dtype=gu.TORCH_DT[dtype], device="cuda")
        Vo = torch.zeros_like(Ko)
        ws = torch.empty(kb.kvm_workspace_bytes(sh, params), dtype=torch.uint8, device="cuda")
        kb.kvm_evict(sh, params, Kd, Vd, torch.from_numpy(mass).cuda(), kept, n_kept, Ko, Vo, ws)
        torch.cuda.synchronize()
        ok, on, oko, ovo = ref.evict(K, V, mass.astype(np.float64), dtype, budget, recent, cap, lens)
        assert np.array_equal(n_kept.cpu().numpy(), on) and np.array_equal(kept.cpu().numpy(), ok)
        gk, gv = gu.to_host_f64(Ko), gu.to_host_f64(Vo)
        for b in range(5):
            for h in range(2):
                m = int(on[b, h])
                assert np.array_equal(gk[b, h, :m], oko[b, h, :m]) and np.array_equal(gv[b, h, :m], ovo[b, h, :m])
                assert (gk[b, h, m:] == 0).all()              # rows beyond the kept ones are not written


def _random_partition(rng, n, p_boundary, long_run=None):
    """Set starts and pivots of a random contiguous partition of n tokens."""
    if n == 0:
        return np.zeros(0, np.int64), np.zeros(0, np.int64)
    is_start = rng.random(n) < p_boundary
    is_start[0] = True
    if long_run is not None:
        is_start[long_run[0] + 1:long_run[1]] = False
    starts = np.flatnonzero(is_start)
    ends = np.append(starts[1:], n)
    return starts, starts + (rng.random(len(starts)) * (ends - starts)).astype(np.int64)


def _maps_of(starts_list, pivots_list, lens, N, cap):
    S = len(starts_list)
    sid = np.full((S, N), -1, np.int32)
    sst = np.zeros((S, cap + 1), np.int32)
    pv = np.full((S, cap), -1, np.int32)
    ns = np.zeros(S, np.int32)
    for i, (starts, piv) in enumerate(zip(starts_list, pivots_list)):
        M = len(starts)
        ns[i] = M
        sst[i, :M], sst[i, M:], pv[i, :M] = starts, lens[i], piv
        for s, (a, b) in enumerate(zip(starts, list(starts[1:]) + [lens[i]])):
            sid[i, a:b] = s
    return sid, sst, pv, ns


def test_merge_refresh_random_map_changes():
    """Hand-made pairs of valid maps (not from kvm_identify_sets): random partitions, then boundaries toggled
    anywhere, pivots changed, a few tokens appended, sets of more than 512 tokens among them, so that rows move
    up and down in one call and the set count changes by more than one.  kvm_merge_refresh on the cache of the
    old maps must give the bits of kvm_merge on the new maps.  (A longer run of this generator, 15000 cases,
    was clean.)"""
    rng = np.random.default_rng(77)
    for case in range(120):
        dtype = ["f16", "bf16", "f32"][case % 3]
        N = int(rng.choice([3, 64, 300, 1000, 1537, 3000]))
        B, H = int(rng.integers(1, 3)), int(rng.integers(1, 3))
        S = B * H
        grow = int(rng.integers(0, 3))
        new_b = [int(rng.integers(max(1, N // 2), N + 1)) for _ in range(B)]
        old_b = [max(0, n - grow) for n in new_b]
        lens_new, lens_old = [new_b[i // H] for i in range(S)], [old_b[i // H] for i in range(S)]
        params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
        if case % 4 == 1:
            params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 3.0
        if case % 4 == 2:
            params.weights = kb.KVM_WEIGHTS_AVERAGE
        if case % 20 == 0:
            _say(f"merge refresh on random map changes: case {case}, {dtype}, N={N}, {S} slices")
        K = synth.to_storage(rng.standard_normal((B, H, N, 128), dtype=np.float32), dtype)
        V = synth.to_storage(rng.standard_normal((B, H, N, 128), dtype=np.float32), dtype)
        Kd, Vd = gu.to_dev(K, dtype), gu.to_dev(V, dtype)
        cap, p_boundary = N, float(rng.choice([0.02, 0.2, 0.6]))
        o_st, o_pv, n_st, n_pv = [], [], [], []
        for i in range(S):
            n0, n1 = lens_old[i], lens_new[i]
            long_run = None
            if n0 > 700 and rng.random() < 0.4:
                a = int(rng.integers(0, n0 - 600))
                long_run = (a, a + int(rng.integers(520, 600)))
            st, pv = _random_partition(rng, n0, p_boundary, long_run)
            o_st.append(st), o_pv.append(pv)
            is_start = np.zeros(n1, bool)
            is_start[st] = True
            for _ in range(int(rng.integers(0, 6))):
                j = int(rng.integers(1, max(2, n1)))
                if j < n1:
                    is_start[j] = ~is_start[j]
            if n1 > n0:
                is_start[n0:n1] = rng.random(n1 - n0) < 0.7
            is_start[0] = True
            st2 = np.flatnonzero(is_start)
            en2 = np.append(st2[1:], n1)
            old_piv = {int(a): int(q) for a, q in zip(st, pv)}
            old_end = {int(a): int(b) for a, b in zip(st, np.append(st[1:], n0))}
            pv2 = np.empty(len(st2), np.int64)
            for s_, (a, b) in enumerate(zip(st2, en2)):
                keep = int(a) in old_piv and old_end[int(a)] == int(b) and rng.random() < 0.95
                pv2[s_] = old_piv[int(a)] if keep else a + int(rng.random() * (b - a))
            n_st.append(st2), n_pv.append(pv2)
        old = _maps_of(o_st, o_pv, lens_old, N, cap)
        new = _maps_of(n_st, n_pv, lens_new, N, cap)
        shapes = ((B, H, N), (B, H, cap + 1), (B, H, cap), (B, H))
        d_old = [torch.from_numpy(a.reshape(shp)).cuda() for a, shp in zip(old, shapes)]
        d_new = [torch.from_numpy(a.reshape(shp)).cuda() for a, shp in zip(new, shapes)]
        sh_old, sh_new = kb.make_shape(Kd, 1, gu.lens_dev(old_b)), kb.make_shape(Kd, 1, gu.lens_dev(new_b))
        ws = torch.empty(max(kb.kvm_workspace_bytes(sh_new, params), 256), dtype=torch.uint8, device="cuda")
        Ko = torch.zeros((B, H, cap, 128), dtype=gu.TORCH_DT[dtype], device="cuda")
        Vo, Kf, Vf = torch.zeros_like(Ko), torch.zeros_like(Ko), torch.zeros_like(Ko)
        kb.kvm_merge(sh_old, params, Kd, Vd, d_old[1], d_old[2], d_old[3], Ko, Vo, None, ws)
        kb.kvm_merge_refresh(sh_new, params, Kd, Vd, *d_old, d_new[1], d_new[2], d_new[3], Ko, Vo, None, ws)
        kb.kvm_merge(sh_new, params, Kd, Vd, d_new[1], d_new[2], d_new[3], Kf, Vf, None, ws)
        torch.cuda.synchronize()
        bits = torch.int32 if dtype == "f32" else torch.int16
        for i in range(S):
            b, h = divmod(i, H)
            M = int(new[3][i])
            assert torch.equal(Ko[b, h, :M].view(bits), Kf[b, h, :M].view(bits)) and \
                torch.equal(Vo[b, h, :M].view(bits), Vf[b, h, :M].view(bits)), \
                f"case {case} ({dtype}, N={N}) slice {i}: refreshed rows differ from a full merge (M {int(old[3][i])} -> {M})"


@pytest.mark.parametrize("dtype,mode", [("f16", "adaptive"), ("bf16", "fixed"), ("f32", "adaptive"), ("f32", "average")])
@pytest.mark.parametrize("slices", [1, 256, 257])
def test_merge_refresh_with_one_workgroup_size_or_the_other(dtype, mode, slices):
    """Up to 256 slices a workgroup of 1024 threads refreshes a slice, its sets of more than 512 tokens too; beyond, one of 512
    threads, and the long sets follow in a launch of their own.  Rows that move up and down over several batches, changed sets
    of one, four and sixteen waves: the bits of a full merge of the new maps."""
    _say(f"merge refresh, {slices} slices: {dtype} {mode}")
    rng = np.random.default_rng(9)
    old = [1] * 300 + [600, 513, 200, 129, 17, 5] + [1] * 200 + [40, 3] + [1] * 100
    new = [1] * 290 + [4, 6] + [600, 514, 199, 129, 17, 5] + [1] * 200 + [20, 20, 3] + [1] * 100   # (same tokens, other sets)
    n = sum(old)
    assert sum(new) == n
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    if mode == "fixed":
        params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 9.0
    if mode == "average":
        params.weights = kb.KVM_WEIGHTS_AVERAGE
    _, K, V = _slices(44, 1, 1, [n], n, 128, 1, dtype, rho=0.9)
    Kd, Vd = (gu.to_dev(x, dtype).expand(1, slices, n, 128).contiguous() for x in (K, V))
    sh = kb.make_shape(Kd, 1, None)
    b = kb.Buffers(sh, params, "cuda", gu.TORCH_DT[dtype])

    def maps(sizes, shift):
        starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        piv = (starts[:-1] + np.minimum(np.asarray(sizes) - 1, np.where(np.asarray(sizes) > 500, shift, 0))).astype(np.int32)
        out = [torch.full_like(t, f) for t, f in ((b.set_id, -1), (b.set_start, n), (b.pivot, -1), (b.n_sets, len(sizes)))]
        for t, v in zip(out, (np.repeat(np.arange(len(sizes), dtype=np.int32), sizes), starts, piv)):
            t[0, :, :len(v)] = torch.from_numpy(v).cuda()
        return out

    before, after = maps(old, 7), maps(new, 9)               # (the set of 600 tokens keeps its extent and changes its pivot)
    kb.kvm_merge(sh, params, Kd, Vd, *before[1:], b.K_out, b.V_out, None, b.ws)
    names = gu.kernels_of(lambda: kb.kvm_merge_refresh(sh, params, Kd, Vd, *before, *after[1:], b.K_out, b.V_out, None, b.ws))
    assert ("merge_long_kernel" in names) == (slices > 256)
    Kf, Vf = torch.zeros_like(b.K_out), torch.zeros_like(b.V_out)
    kb.kvm_merge(sh, params, Kd, Vd, *after[1:], Kf, Vf, None, b.ws)
    torch.cuda.synchronize()
    M, bits = len(new), torch.int32 if dtype == "f32" else torch.int16
    for got, want in ((b.K_out, Kf), (b.V_out, Vf)):
        assert torch.equal(got[:, :, :M].view(bits), want[:, :, :M].view(bits))


@pytest.mark.parametrize("slices,N,kernel", [(1, 512, "refresh_kernel"), (1, 513, "refresh_kernel_few"), (256, 300, "refresh_kernel"),
                                             (256, 513, "refresh_kernel_few"), (257, 513, "refresh_kernel")])
def test_merge_refresh_workgroup_size(slices, N, kernel):
    """1024 threads a slice up to 256 slices, where a set can be longer than 512 tokens; 512 otherwise.  Unchanged maps: the rows
    stay as they are."""
    _say(f"merge refresh, {slices} slices of {N}: {kernel}")
    K = gu.randn_gpu((1, slices, N, 128), torch.float16, 48)
    sh, params = kb.make_shape(K, 1, None), kb.kvm_params_for_budget(0.5)
    b = kb.Buffers(sh, params, "cuda", torch.float16)
    b.mass.copy_(torch.rand_like(b.mass))
    kb.kvm_identify_sets(sh, params, K, b.mass, b.set_id, b.set_start, b.pivot, b.n_sets, None, b.status, b.ws)
    kb.kvm_merge(sh, params, K, K, b.set_start, b.pivot, b.n_sets, b.K_out, b.V_out, None, b.ws)
    Ks, maps = b.K_out.clone(), [t.clone() for t in (b.set_id, b.set_start, b.pivot, b.n_sets)]
    names = gu.kernels_of(lambda: kb.kvm_merge_refresh(sh, params, K, K, *maps, b.set_start, b.pivot, b.n_sets, b.K_out, b.V_out, None, b.ws))
    assert kernel in names
    assert torch.equal(b.K_out.view(torch.int16), Ks.view(torch.int16))


@pytest.mark.parametrize("dtype,slices,sets", [("f16", 1, 1), ("f32", 1, 4096), ("f16", 1, 4097), ("bf16", 3, 9000), ("bf16", 64, 1030),
                                               ("f32", 100, 1025), ("f16", 128, 1040), ("f32", 129, 1025), ("f16", 257, 2048), ("bf16", 257, 2049), ("f32", 257, 4500)])
def test_merge_refresh_of_many_sets(dtype, slices, sets):
    """Every thread of a refresh compares four sets at a time, 4096 or 2048 a workgroup: numbers of sets at the edges of such a turn
    and beyond it, mostly single tokens whose rows move by one, in both directions, past sets that were split and joined.  With the
    whole workspace, where few slices of this many rows find room for two workgroups each, and with the smallest, one each
    (test_merge_refresh_shared_slices asks for every number).  The bits of a full merge of the new maps."""
    _say(f"merge refresh of {sets} sets, {slices} slices: {dtype}")
    rng = np.random.default_rng(sets)
    new = np.ones(sets, np.int64)
    new[rng.choice(sets, min(sets, 40), replace=False)] = rng.integers(2, 40, min(sets, 40))
    old, i = [], 0
    while i < sets:                                          # (one set in sixty was two, one pair in sixty was one set)
        what = rng.integers(0, 60)
        if what == 0 and new[i] > 1:
            old += [1, int(new[i]) - 1]
        elif what == 1 and i + 1 < sets:
            old.append(int(new[i] + new[i + 1]))
            i += 1
        else:
            old.append(int(new[i]))
        i += 1
    n = int(new.sum())
    assert sum(old) == n
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    _, K, V = _slices(45, 1, 1, [n], n, 128, 1, dtype, rho=0.9)
    Kd, Vd = (gu.to_dev(x, dtype).expand(1, slices, n, 128).contiguous() for x in (K, V))
    sh = kb.make_shape(Kd, 1, None)
    b = kb.Buffers(sh, params, "cuda", gu.TORCH_DT[dtype])

    def maps(sizes):
        starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        out = [torch.full_like(t, f) for t, f in ((b.set_id, -1), (b.set_start, n), (b.pivot, -1), (b.n_sets, len(sizes)))]
        for t, v in zip(out, (np.repeat(np.arange(len(sizes), dtype=np.int32), sizes), starts, starts[:-1])):
            t[0, :, :len(v)] = torch.from_numpy(v).cuda()
        return out

    before, after = maps(old), maps(new)
    kb.kvm_merge(sh, params, Kd, Vd, *before[1:], b.K_out, b.V_out, None, b.ws)
    Ks, Vs = b.K_out.clone(), b.V_out.clone()
    changed = torch.full((2, 1, slices), -1, dtype=torch.int32, device="cuda")
    kb.kvm_merge_refresh(sh, params, Kd, Vd, *before, *after[1:], b.K_out, b.V_out, changed[0], b.ws)
    least = slices * ((n + 63) // 64 + n // 513 + 3 + 2 * n + 1) * 4
    kb.kvm_merge_refresh(sh, params, Kd, Vd, *before, *after[1:], Ks, Vs, changed[1], torch.empty(least, dtype=torch.uint8, device="cuda"))
    Kf, Vf = torch.zeros_like(b.K_out), torch.zeros_like(b.V_out)
    kb.kvm_merge(sh, params, Kd, Vd, *after[1:], Kf, Vf, None, b.ws)
    torch.cuda.synchronize()
    bits = torch.int32 if dtype == "f32" else torch.int16
    for got, want in ((b.K_out, Kf), (b.V_out, Vf), (Ks, Kf), (Vs, Vf)):
        assert torch.equal(got[:, :, :sets].view(bits), want[:, :, :sets].view(bits))
    kept = len(set(zip(before[1][0, 0].tolist(), before[1][0, 0, 1:len(old) + 1].tolist())) &
               set(zip(after[1][0, 0].tolist(), after[1][0, 0, 1:sets + 1].tolist())))
    assert bool((changed == sets - kept).all())


@pytest.mark.parametrize("dtype,mode", [("f16", "adaptive"), ("bf16", "fixed"), ("f32", "adaptive"), ("f16", "average"), ("f32", "fixed")])
@pytest.mark.parametrize("parts,slices", [(1, 3), (2, 3), (4, 3), (2, 65), (2, 128), (4, 64), (1, 129)])
def test_merge_refresh_shared_slices(dtype, mode, parts, slices):
    """One, two or four workgroups a slice, by the lists that the workspace has room for: rows that move over three or more batches in both
    directions, changed sets of a wave, of four waves and of the whole workgroup.  The bits of a full merge of the new maps, and the
    number of changed sets from one of the workgroups."""
    sets = 3300 if slices <= 3 else 2100
    _say(f"merge refresh, {slices} slices by {parts} workgroups each: {dtype} {mode}")
    few, many = sets // 3, sets - sets // 3
    old = [1] * few + [3, 40] + [1] * few + [600, 200, 513, 20] + [1] * many
    new = [1] * few + [20, 20, 3] + [1] * (few - 6) + [4, 2] + [601, 199, 130, 383, 20] + [1] * (many - 9) + [5, 4]
    # (from old to new the rows of the middle move down by two and those of the end up by one)
    n = sum(old)
    assert n == sum(new) and len(new) > 2 * 1024
    params = kb.make_params(1.0, 0.0, 0.0, enforce_budget=False)
    if mode == "fixed":
        params.sigma_mode, params.sigma = kb.KVM_SIGMA_FIXED, 9.0
    if mode == "average":
        params.weights = kb.KVM_WEIGHTS_AVERAGE
    _, K, V = _slices(49, 1, 1, [n], n, 128, 1, dtype, rho=0.9)
    Kd, Vd = (gu.to_dev(x, dtype).expand(1, slices, n, 128).contiguous() for x in (K, V))
    sh = kb.make_shape(Kd, 1, None)
    b = kb.Buffers(sh, params, "cuda", gu.TORCH_DT[dtype])

    def maps(sizes):
        starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        out = [torch.full_like(t, f) for t, f in ((b.set_id, -1), (b.set_start, n), (b.pivot, -1), (b.n_sets, len(sizes)))]
        for t, v in zip(out, (np.repeat(np.arange(len(sizes), dtype=np.int32), sizes), starts, starts[:-1])):
            t[0, :, :len(v)] = torch.from_numpy(v).cuda()
        return out

    # the lists of one workgroup a slice, and behind them those of every further one
    lists = slices * ((n + 63) // 64 + n // 513 + 3 + 2 * n + 1) + (parts - 1) * slices * (n + 2 + n // 513 + 1)
    bits = torch.int32 if dtype == "f32" else torch.int16
    ends = set(zip(np.cumsum([0] + old).tolist(), np.cumsum(old).tolist()))
    for here, there in ((old, new), (new, old)):
        before, after = maps(here), maps(there)
        kb.kvm_merge(sh, params, Kd, Vd, *before[1:], b.K_out, b.V_out, None, b.ws)
        changed = torch.full((1, slices), -1, dtype=torch.int32, device="cuda")
        ws = torch.empty(4 * lists, dtype=torch.uint8, device="cuda")
        names = gu.kernels_of(lambda: kb.kvm_merge_refresh(sh, params, Kd, Vd, *before, *after[1:], b.K_out, b.V_out, changed, ws))
        assert names == {"refresh_kernel_few" if parts == 1 else f"refresh_kernel_{parts}"}
        Kf, Vf = torch.zeros_like(b.K_out), torch.zeros_like(b.V_out)
        kb.kvm_merge(sh, params, Kd, Vd, *after[1:], Kf, Vf, None, b.ws)
        torch.cuda.synchronize()
        for got, want in ((b.K_out, Kf), (b.V_out, Vf)):
            assert torch.equal(got[:, :, :len(there)].view(bits), want[:, :, :len(there)].view(bits))
        kept = len(ends & set(zip(np.cumsum([0] + new).tolist(), np.cumsum(new).tolist())))
        assert bool((changed == len(there) - kept).all())


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_evict_merge_values_matches_the_oracle(dtype):
    """Value-only merging (comparison workload): kept positions and keys bit-exact, the averaged values
    to the bar of the merged rows.  Scores fall with the position in slice (0, 1), so the kept tokens
    crowd at both ends and one of them averages hundreds of values (the part a whole wave sums)."""
    n = 2100
    lens = [n, 1000, 0, 1, 77]
    _say(f"evict + value merge: {dtype}, lens {lens}")
    Q, K, V = _slices(36, 5, 2, lens, n, 128, 1, dtype)
    rng = np.random.default_rng(10)
    mass = (rng.random((5, 2, n)) + 0.01).astype(np.float32)
    mass[0, 1] = (3.0 - np.arange(n) / n + 0.001 * rng.random(n)).astype(np.float32)
    mass[0, 0, 300:700] = mass[0, 0, 300]
    for budget, recent in ((0.5, 0.17), (0.35, 0.08), (0.05, 0.01), (0.3, 0.3), (1.0, 0.0)):
        params = kb.make_params(budget, recent, 0.0)
        Kd, Vd = gu.to_dev(K, dtype), gu.to_dev(V, dtype)
        sh = kb.make_shape(Kd, 1, gu.lens_dev(lens))
        cap = kb.kvm_out_capacity(sh, params)
        kept = torch.full((5, 2, cap), -7, dtype=torch.int32, device="cuda")
        n_kept = torch.full((5, 2), -7, dtype=torch.int32, device="cuda")
        Ko = torch.zeros((5, 2, cap, 128), dtype=gu.TORCH_DT[dtype], device="cuda")
        Vo = torch.zeros_like(Ko)
        ws = torch.empty(kb.kvm_workspace_bytes(sh, params), dtype=torch.uint8, device="cuda")
        kb.kvm_evict_merge_values(sh, params, Kd, Vd, torch.from_numpy(mass).cuda(), kept, n_kept, Ko, Vo, ws)
        torch.cuda.synchronize()
        ok, on, oko, ovo, cnt = ref.evict_merge_values(K, V, mass.astype(np.float64), dtype, budget, recent, cap, lens)
        assert np.array_equal(n_kept.cpu().numpy(), on) and np.array_equal(kept.cpu().numpy(), ok)
        gk, gv = gu.to_host_f64(Ko), gu.to_host_f64(Vo)
        worst, longest = 0.0, 0
        for b in range(5):
            for h in range(2):
                m = int(on[b, h])
                assert np.array_equal(gk[b, h, :m], oko[b, h, :m])
                assert (gk[b, h, m:] == 0).all() and (gv[b, h, m:] == 0).all()    # rows beyond the kept ones are not written
                if m == 0:
                    continue
                lone = cnt[b, h, :m] == 1
                assert np.array_equal(gv[b, h, :m][lone], ovo[b, h, :m][lone])    # nothing received: the same bits
                err = gu.row_rel_err(gv[b, h, :m], ovo[b, h, :m]).max()
                assert err <= gu.kv_tol(dtype), f"slice ({b},{h}) budget {budget}: value error {err:.3e}"
                assert gu.ulp_excess(gv[b, h, :m], ovo[b, h, :m], dtype).max() <= 2e-5
                worst, longest = max(worst, float(err)), max(longest, int(cnt[b, h, :m].max()))
        _say(f"  budget {budget}: worst value error {worst:.2e}, longest mean over {longest} values")
        if budget == 0.05:
            assert longest > 64                               # the cooperative part ran


# ---------------------------------------------------------------------------------------------
# streams and graphs: the calls only enqueue work on the caller's stream
# ---------------------------------------------------------------------------------------------

def _outputs(buf):
    names = ("mass", "set_id", "set_start", "pivot", "n_sets", "status", "K_out", "V_out")
    return {k: getattr(buf, k).clone() for k in names}


def _same_outputs(a, b, what):
    M = a["n_sets"].clamp(max=a["K_out"].shape[2])
    for k in ("mass", "set_id", "set_start", "pivot", "n_sets", "status"):
        assert torch.equal(a[k], b[k]), f"{what}: {k} differs"
    for k in ("K_out", "V_out"):                      # rows past the set count are not written
        for bb in range(M.shape[0]):
            for h in range(M.shape[1]):
                m = int(M[bb, h])
                assert torch.equal(a[k][bb, h, :m], b[k][bb, h, :m]), f"{what}: {k} differs in slice ({bb},{h})"


def test_stream_handle_with_and_without_torchs_raw_call(monkeypatch):
    """The binding asks torch for the current stream's handle alone where it can; the public way has to give the same one."""
    _say("binding: the current stream's handle")
    side = torch.cuda.Stream()
    for stream in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(stream):
            assert kb._stream() == stream.cuda_stream
            with monkeypatch.context() as m:
                m.setattr(kb, "_current_raw_stream", None)
                assert kb._stream() == stream.cuda_stream


@pytest.mark.parametrize("rule", ["adjacent", "anchor"])
def test_whole_pass_on_a_side_stream_and_replayed_from_a_graph(rule):
    """Nothing in the three calls allocates, synchronises or leaves the caller's stream: the pass
    can be enqueued on a side stream and captured into a graph.  Every replay (with other work
    and synchronisations in between, and with new inputs in the same buffers) has to give the
    bits of the plain run on the same inputs; the kernels use no atomics."""
    _say(f"whole pass, {rule} sets: side stream, then graph capture and three replays")
    n, dtype = 1300, "f16"
    inputs = [_slices(seed, 1, 4, [n], n, 128, 1, dtype) for seed in (41, 42)]
    dev = [[gu.to_dev(x, dtype) for x in trio] for trio in inputs]
    params = kb.kvm_params_for_budget(0.5)
    if rule == "anchor":
        params.set_rule = kb.KVM_SETS_ANCHOR
        params.enforce_budget = 0
    Qs, Ks, Vs = (torch.empty_like(t) for t in dev[0])      # the buffers the graph reads
    shape = kb.make_shape(Ks, 1, None)
    buf = kb.Buffers(shape, params, "cuda", torch.float16)
    plain = []
    for Qd, Kd, Vd in dev:                                  # default stream, no graph
        Qs.copy_(Qd), Ks.copy_(Kd), Vs.copy_(Vd)
        kb.compress(shape, params, Qs, Ks, Vs, buf)
        torch.cuda.synchronize()
        plain.append(_outputs(buf))
    assert not torch.equal(plain[0]["set_id"], plain[1]["set_id"])

    side = torch.cuda.Stream()
    Qs.copy_(dev[0][0]), Ks.copy_(dev[0][1]), Vs.copy_(dev[0][2])
    buf.mass.fill_(-1.0)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        kb.compress(shape, params, Qs, Ks, Vs, buf)
    side.synchronize()
    _same_outputs(_outputs(buf), plain[0], "side stream")

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kb.compress(shape, params, Qs, Ks, Vs, buf)
    for which in (1, 0, 1):
        Qs.copy_(dev[which][0]), Ks.copy_(dev[which][1]), Vs.copy_(dev[which][2])
        buf.mass.fill_(-1.0)
        buf.set_id.fill_(-9)
        graph.replay()
        torch.cuda.synchronize()
        _same_outputs(_outputs(buf), plain[which], f"graph replay with input {which}")
        # unrelated work of the program between the replays
        other = gu.gpu_mass(inputs[which][0], inputs[which][1], dtype)
        assert np.isfinite(other).all()


# ---------------------------------------------------------------------------------------------
# addressing: tensors of more than 2^32 elements
# ---------------------------------------------------------------------------------------------

def test_every_stage_on_tensors_of_more_than_2_pow_32_elements():
    """260 x 32 slices of 4096 tokens: Q, K and V hold 4.36e9 elements each, slice (256, 0)
    starts at element 2^32 exactly.  The bulk is a small generated block repeated on the
    device; five slices around that boundary and at both ends carry data of their own and
    are compared with the oracle, each stage fed the same inputs on both sides."""
    N, d, H, B, dtype = 4096, 128, 32, 260, "f16"
    free, _ = torch.cuda.mem_get_info()
    if free < 60 * 2 ** 30:
        pytest.skip("needs 60 GiB of free device memory")
    _say("stages on 260 x 32 x 4096 x 128 tensors (offsets past 2^32 elements)")
    base = _slices(51, 2, H, [N, N], N, d, 1, dtype)
    Qd, Kd, Vd = (gu.to_dev(x, dtype).repeat(B // 2, 1, 1, 1) for x in base)
    assert Kd.numel() > 2 ** 32 and Kd.is_contiguous()
    sample = [(0, 0), (255, H - 1), (256, 0), (256, 1), (B - 1, H - 1)]
    S = len(sample)
    Qu, Ku, Vu = _slices(52, S, 1, [N] * S, N, d, 1, dtype)                 # (S, 1, N, d) each
    rng = np.random.default_rng(53)
    mass_base = (rng.random((2, H, N)) ** 3 + 1e-3).astype(np.float32)
    mass_u = (rng.random((S, 1, N)) ** 3 + 1e-3).astype(np.float32)
    mass_in = torch.from_numpy(mass_base).cuda().repeat(B // 2, 1, 1)
    for i, (b, h) in enumerate(sample):
        Qd[b, h], Kd[b, h], Vd[b, h] = (gu.to_dev(x[i, 0], dtype) for x in (Qu, Ku, Vu))
        mass_in[b, h] = torch.from_numpy(mass_u[i, 0]).cuda()
    params = kb.kvm_params_for_budget(0.5)
    shape = kb.make_shape(Kd, 1, None)
    buf = kb.Buffers(shape, params, "cuda", torch.float16, with_debug=True)

    # (a) aggregated scores
    kb.kvm_attn_mass(shape, Qd, Kd, buf.mass, buf.ws)
    torch.cuda.synchronize()
    want = ref.attn_mass(Qu, Ku, dtype)
    got = np.stack([buf.mass[b, h].cpu().numpy() for b, h in sample])[:, None]
    err = gu.assert_mass_close(got, want, None, N, "large tensors")
    _say(f"  mass: worst relative error {err:.2e}")
    # (b), (c) on scores given to both sides
    kb.kvm_identify_sets(shape, params, Kd, mass_in, buf.set_id, buf.set_start, buf.pivot, buf.n_sets, buf.sim,
                         buf.status, buf.ws)
    kb.kvm_merge(shape, params, Kd, Vd, buf.set_start, buf.pivot, buf.n_sets, buf.K_out, buf.V_out, buf.w, buf.ws)
    torch.cuda.synchronize()
    o = ref.identify_sets(Ku, mass_u.astype(np.float64), dtype, params.budget, params.recent_ratio, params.heavy_ratio,
                          params.threshold, True, buf.cap)
    rk, rv, rw = ref.merge(Ku, Vu, dtype, o["set_start"], o["pivot"], o["n_sets"], params.sigma_mode, params.sigma,
                           bool(params.value_scale_by_set_size), None, weights=params.weights)
    pick = lambda t: np.stack([t[b, h].cpu().numpy() for b, h in sample])[:, None]
    g = dict(set_id=pick(buf.set_id), set_start=pick(buf.set_start), pivot=pick(buf.pivot),
             n_sets=np.array([[int(buf.n_sets[b, h])] for b, h in sample]),
             status=np.array([[int(buf.status[b, h])] for b, h in sample]), sim=pick(buf.sim), cap_rows=buf.cap)
    np.testing.assert_allclose(g["sim"], o["sim"], atol=2e-6)
    exc, near = gu.compare_maps(g, o, None, N, params.threshold, "large tensors")
    _say(f"  maps: {exc} excused slices, {near} near-threshold similarities")
    assert exc == 0
    ko = np.stack([gu.to_host_f64(buf.K_out[b, h]) for b, h in sample])[:, None]
    vo = np.stack([gu.to_host_f64(buf.V_out[b, h]) for b, h in sample])[:, None]
    _check_merge(Ku, Vu, dtype, o, ko, vo, pick(buf.w), rk, rv, rw, None, None, "large tensors")
    # eviction by score: kept positions and rows, bit for bit (reuses the merge's output buffers)
    buf.K_out.zero_(), buf.V_out.zero_()
    kb.kvm_evict(shape, params, Kd, Vd, mass_in, buf.pivot, buf.n_sets, buf.K_out, buf.V_out, buf.ws)
    torch.cuda.synchronize()
    ek, en, eko, evo = ref.evict(Ku, Vu, mass_u.astype(np.float64), dtype, params.budget, params.recent_ratio, buf.cap, None)
    for i, (b, h) in enumerate(sample):
        m = int(en[i, 0])
        assert int(buf.n_sets[b, h]) == m and np.array_equal(buf.pivot[b, h].cpu().numpy(), ek[i, 0])
        assert np.array_equal(gu.to_host_f64(buf.K_out[b, h, :m]), eko[i, 0, :m])
        assert np.array_equal(gu.to_host_f64(buf.V_out[b, h, :m]), evo[i, 0, :m])
    # decode-time calls: one more query row on the given scores, one similarity
    q_new = Qd[:, :, N - 1].contiguous()
    kept_before = buf.mass.clone()                                           # the scores of stage (a)
    work = mass_in.clone()
    kb.kvm_attn_mass_append(shape, q_new, Kd, work, buf.ws)
    sim2 = torch.full_like(buf.sim, float("nan"))
    kb.kvm_sim_append(shape, Kd, sim2)
    torch.cuda.synchronize()
    want = ref.attn_mass_append(np.ascontiguousarray(Qu[:, :, N - 1]), Ku, mass_u.astype(np.float64), dtype)
    for i, (b, h) in enumerate(sample):
        rel = np.abs(work[b, h].cpu().numpy() - want[i, 0]) / want[i, 0]
        assert rel.max() <= gu.TOL, f"append on slice ({b},{h}): {rel.max():.2e}"
        assert float(sim2[b, h, N - 1]) == float(buf.sim[b, h, N - 1]) and bool(torch.isnan(sim2[b, h, :N - 1]).all())
    # the column pass alone, on row statistics from the oracle
    lse = torch.zeros((B, H, N), dtype=torch.float32, device="cuda")
    lse_u = ref.row_lse(Qu, Ku, dtype).astype(np.float32)
    for i, (b, h) in enumerate(sample):
        lse[b, h] = torch.from_numpy(lse_u[i, 0]).cuda()
    kb.kvm_attn_mass_from_lse(shape, Qd, Kd, lse, buf.mass, buf.ws)
    torch.cuda.synchronize()
    for i, (b, h) in enumerate(sample):
        assert torch.allclose(buf.mass[b, h], kept_before[b, h], rtol=1e-4, atol=0), f"from row statistics, slice ({b},{h})"
    buf.mass.copy_(kept_before)
    # the repeated bulk: every copy of a block slice must give the bits of the first copy
    for b, h in ((2, 5), (258, 5), (257, H - 1)):
        b0 = b % 2
        if (b, h) in sample or (b0, h) in sample:
            continue
        assert torch.equal(buf.mass[b, h], buf.mass[b0, h]) and torch.equal(buf.set_id[b, h], buf.set_id[b0, h])
        m = int(buf.n_sets[b0, h])                                           # by now the kept rows of the eviction
        assert int(buf.n_sets[b, h]) == m
        assert torch.equal(buf.K_out[b, h, :m], buf.K_out[b0, h, :m]) and torch.equal(buf.V_out[b, h, :m], buf.V_out[b0, h, :m])
