"""GPU parity of the correlator (afc_correlate) against the CPU oracle.

Inputs are seeded channelised samples drawn directly in the block layout
(workloads.make_channelised); the oracle receives the same values in its
natural [S][N] layout.  int8: bit-exact against exact integer sums.  fp16 and
fp32: float32 accumulation of exactly representable products, compared per
baseline with the error normalised by sqrt(V_ii V_jj).
"""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import gather_rows, log, normalised_error, vis_to_complex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def afc():
    import paper_1609_04205_amd as afc
    return afc


def _oracle_channel(zn, dtype, flags=None):
    if dtype == "i8":
        V, W_ = oracle.xcorr_int(zn, flags)
        return V, W_
    V, W_ = oracle.xcorr(zn.astype(np.float64), flags)
    return V, W_


CASES = [
    # (dtype, B, Na, S, per-subband S or None, flagged antennas or None, channels to check)
    ("i8", 2, 48, 1024, None, None, range(64)),
    ("f16", 2, 48, 1024, None, None, range(0, 64, 7)),
    ("f32", 2, 48, 1024, None, None, range(0, 64, 7)),
    ("i8", 1, 70, 37, None, [3, 69], range(0, 64, 9)),        # N = 140: ragged against 128 and 64 tiles
    ("f16", 1, 70, 37, None, [0], range(0, 64, 9)),
    ("f32", 1, 70, 37, None, [1], range(0, 64, 9)),
    ("i8", 2, 33, 100, [100, 61], [5], range(0, 64, 13)),     # spectra >= S_b ignored although nonzero
    ("f32", 2, 33, 100, [3, 100], None, range(0, 64, 13)),
    ("i8", 1, 1, 5, None, None, range(64)),                   # one antenna
    ("f16", 1, 64, 16, None, None, range(0, 64, 21)),         # exactly one 128 tile
    # three 128-row tiles (off-diagonal tiles load their column operands
    # directly) with stage counts that are not a multiple of the register ring
    ("i8", 2, 150, 300, [300, 171], [7], range(0, 64, 13)),
    ("f16", 1, 150, 77, None, None, range(0, 64, 13)),
    # one spectrum block (one real stage, the rest of the register ring padding)
    ("i8", 2, 100, 8, [8, 1], [99], range(0, 64, 17)),
    ("f16", 1, 100, 3, None, None, range(0, 64, 17)),
]


@pytest.mark.parametrize("dtype,B,Na,S,S_sb,flagged,chans", CASES)
def test_correlate_matches_oracle(afc, dev, dtype, B, Na, S, S_sb, flagged, chans):
    log(f"xengine {dtype} B={B} Na={Na} S={S} S_sb={S_sb} flagged={flagged}")
    z = W.make_channelised(B, 64, S, 2 * Na, dtype, seed=Na * 7 + S, device=dev)
    if S_sb is not None:
        # fill the slots beyond each subband's S_b with nonzero values: they must be ignored
        zf = W.make_channelised(B, 64, S, 2 * Na, dtype, seed=99, device=dev)
        z = torch.where(z == 0, zf, z)
    fl = None
    if flagged is not None:
        fl_np = np.zeros((B, Na), np.uint8)
        fl_np[:, flagged] = 1
        fl = torch.from_numpy(fl_np).to(dev)
    vis, w = afc.correlate(z, n_spectra=S, n_spectra_per_sb=S_sb, flags=fl)
    torch.cuda.synchronize()
    vis_np = vis.cpu().numpy()
    w_np = w.cpu().numpy()
    zn_all = W.blocked_to_natural(z.cpu(), z.shape[2] * 8).numpy()
    for b in range(B):
        Sb_ = S if S_sb is None else S_sb[b]
        fb = None if fl is None else fl_np[b]
        for ch in chans:
            zn = zn_all[b, ch, :Sb_]
            Vref, Wref = _oracle_channel(zn, dtype, fb)
            if dtype == "i8":
                np.testing.assert_array_equal(vis_np[b, ch].astype(np.int64), Vref)
            else:
                got = vis_to_complex(vis_np[b, ch])
                ref = Vref
                err = normalised_error(got, ref, Na)
                if fb is not None:
                    a_, b_ = np.tril_indices(Na)
                    hit = (fb[a_] == 1) | (fb[b_] == 1)
                    assert np.all(got[hit] == 0)
                    err = err[~hit]
                assert err.max() <= 1e-5, (b, ch, err.max())
            np.testing.assert_array_equal(w_np[b], Wref)


def test_autocorrelations_exactly_real(afc, dev):
    z = W.make_channelised(1, 64, 200, 96, "f32", seed=3, device=dev)
    vis, _ = afc.correlate(z, n_spectra=200)
    v = vis.cpu().numpy()
    d = np.array([a * (a + 1) // 2 + a for a in range(48)])
    assert np.all(v[:, :, d, 0, 0, 1] == 0) and np.all(v[:, :, d, 1, 1, 1] == 0)
    assert np.all(v[:, :, d, 0, 0, 0] >= 0) and np.all(v[:, :, d, 1, 1, 0] >= 0)


def test_int8_extreme_values_exact(afc, dev):
    """All samples at +-127 (the largest products) stay exact; -128 is never produced."""
    g = torch.Generator(device=dev)
    g.manual_seed(11)
    S = 3051
    bits = torch.randint(0, 2, (1, 64, (S + 7) // 8, 96, 8, 2), generator=g, device=dev)
    z = (bits * 254 - 127).to(torch.int8)
    z[:, :, -1, :, S % 8:, :] = 0
    vis, _ = afc.correlate(z, n_spectra=S)
    v = vis.cpu().numpy()
    zn = W.blocked_to_natural(z.cpu(), z.shape[2] * 8).numpy()
    for ch in (0, 33):
        Vref, _ = oracle.xcorr_int(zn[0, ch, :S])
        np.testing.assert_array_equal(v[0, ch].astype(np.int64), Vref)


@pytest.mark.parametrize("dtype,B,Na,S", [("i8", 2, 576, 3051), ("f16", 1, 576, 763), ("i8", 2, 150, 300),
                                          ("f16", 1, 150, 77), ("i8", 1, 70, 37)])
def test_repeated_launches_bit_identical(afc, dev, dtype, B, Na, S):
    """The DMA ring's stage barrier orders the refill of a stage buffer after
    every wave's reads of it; a missing wait would show as launches that
    differ.  Every repeat (with other work queued in between) must equal the
    first bit for bit, on 128-wide diagonal and off-diagonal tiles and
    ragged tails."""
    log(f"xengine repeats {dtype} B={B} Na={Na} S={S}")
    z = W.make_channelised(B, 64, S, 2 * Na, dtype, seed=12, device=dev)
    fl = torch.zeros((B, Na), dtype=torch.uint8, device=dev)
    fl[:, Na // 3] = 1
    vis = torch.empty(afc.visibility_shape(B, Na), dtype=torch.int32 if dtype == "i8" else torch.float32,
                      device=dev)
    afc.correlate(z, n_spectra=S, out=vis, flags=fl, want_weights=False)
    torch.cuda.synchronize()
    first = vis.view(torch.int32).clone()
    for _ in range(6):
        vis.fill_(-1)
        _ = torch.randn(4096, device=dev).sum()
        afc.correlate(z, n_spectra=S, out=vis, flags=fl, want_weights=False)
        torch.cuda.synchronize()
        assert torch.equal(vis.view(torch.int32), first)
    del z, vis, first
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", ["i8", "f16"])
def test_checked_and_check_free_stores_agree(afc, dev, dtype):
    """Channel 0's tiles store through the checked path when weights are
    asked for and through the check-free one otherwise (interior
    off-diagonal 128-wide tiles): the visibilities are the same bit for bit,
    with and without flagged antennas."""
    Na, S = 576, 300
    z = W.make_channelised(2, 64, S, 2 * Na, dtype, seed=21, device=dev)
    for flagged in ([], [0, 200, 575]):
        fl = torch.zeros((2, Na), dtype=torch.uint8, device=dev)
        if flagged:
            fl[:, flagged] = 1
        v_w, _ = afc.correlate(z, n_spectra=S, flags=fl)
        v_n, _ = afc.correlate(z, n_spectra=S, flags=fl, want_weights=False)
        torch.cuda.synchronize()
        assert torch.equal(v_w.view(torch.int32), v_n.view(torch.int32)), flagged
    del z, v_w, v_n
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", ["i8", "f16", "f32"])
def test_full_size_sampled(afc, dev, dtype):
    """AARTFAAC-12 shape: 1152 receivers, 16 subbands, 3051 spectra, sampled baselines."""
    Na, B, S = 576, 16, 3051
    log(f"xengine full size {dtype}")
    z = W.make_channelised(B, 64, S, 2 * Na, dtype, seed=5, device=dev)
    vis, w = afc.correlate(z, n_spectra=S)
    torch.cuda.synchronize()
    rng = np.random.default_rng(1)
    for _ in range(6):
        sb = int(rng.integers(B))
        ch = int(rng.integers(64))
        ants = sorted(set(rng.choice(Na, size=5, replace=False).tolist() + [Na - 1, 0]))
        inputs = [2 * a + p for a in ants for p in range(2)]
        rows = gather_rows(z, sb, ch, inputs, S)
        pos = {i: k for k, i in enumerate(inputs)}
        pairs, where = [], []
        for ia, a in enumerate(ants):
            for b in ants[: ia + 1]:
                for p in range(2):
                    for q in range(2):
                        pairs.append((pos[2 * a + p], pos[2 * b + q]))
                        where.append((a * (a + 1) // 2 + b, p, q))
        pairs = np.array(pairs)
        blv = np.array([x[0] for x in where])
        got = vis[sb, ch, torch.as_tensor(blv, device=dev)].cpu().numpy()     # [n][2][2][2]
        gp = np.array([got[k, where[k][1], where[k][2]] for k in range(len(where))])
        if dtype == "i8":
            ref = oracle.xcorr_pairs_int(rows, pairs)
            np.testing.assert_array_equal(gp.astype(np.int64), ref)
        else:
            ref = oracle.xcorr_pairs(rows.astype(np.float64), pairs)
            autos = {pos[i]: oracle.xcorr_pairs(rows.astype(np.float64), np.array([[pos[i], pos[i]]]))[0].real
                     for i in inputs}
            den = np.sqrt([autos[i] * autos[j] for i, j in pairs])
            err = np.abs((gp[:, 0] + 1j * gp[:, 1]) - ref) / den
            assert err.max() <= 1e-5
    assert int(w.min()) == S and int(w.max()) == S
    del z, vis
    torch.cuda.empty_cache()


def _natural_f32(z, S):
    zn = W.blocked_to_natural(z.cpu(), S).numpy().astype(np.float64)
    return zn[..., 0] + 1j * zn[..., 1]                     # [B][64][S][N]


# tile widths of fp32 launches: 75 antennas x 1 subband 64, 48 x 4 128 (from the
# launch size); 100 x 1 128 with an interior off-diagonal tile
@pytest.mark.parametrize("B,Na,S", [(1, 75, 97), (4, 48, 40), (1, 100, 200), (1, 150, 65), (2, 32, 17)])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -56, 2.0 ** 50])
def test_f32_split_and_its_range(afc, dev, B, Na, S, scale):
    """fp32 samples are split into bf16 parts where every nonzero one lies in
    [2^-50, 2^50), and multiplied on the fp32 matrix cores otherwise (scaled
    cases): both within the fp32 bound, normalised by sqrt(V_ii V_jj)."""
    log(f"xengine f32 split B={B} Na={Na} S={S} scale={scale}")
    z = W.make_channelised(B, 64, S, 2 * Na, "f32", seed=Na + S, device=dev) * scale
    z[:, :, :, 3] = 0.0                                     # a dead receiver is in range
    v, _ = afc.correlate(z, n_spectra=S)
    a, c = np.tril_indices(Na)
    got = v.cpu().numpy().astype(np.float64)
    zn = _natural_f32(z, S)
    for b in range(B):
        for ch in (0, 41):
            x = zn[b, ch].T
            V = x @ x.conj().T
            d = np.sqrt(np.maximum(V.diagonal().real, 1e-300))
            for p in range(2):
                for q in range(2):
                    g = got[b, ch, :, p, q, 0] + 1j * got[b, ch, :, p, q, 1]
                    err = np.abs(g - V[2 * a + p, 2 * c + q]) / (d[2 * a + p] * d[2 * c + q])
                    err[(2 * a + p == 3) | (2 * c + q == 3)] = 0.0
                    assert err.max() <= 1e-5, (b, ch, p, q, err.max())
            dead = got[b, ch][(a == 1)][:, 1]
            assert np.all(dead == 0)


@pytest.mark.parametrize("B,Na", [(1, 75), (1, 100), (1, 150)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38, 2.0 ** -140])
def test_f32_values_out_of_the_split_range(afc, dev, B, Na, bad):
    """One sample that the split cannot hold leaves the visibilities of the
    other receivers as they were (to the fp32 bound) and gives its own the
    value of the fp32 products: with a real part of +-Inf against finite
    samples of nonzero parts, infinities and no NaN."""
    log(f"xengine f32 out of range Na={Na} value={bad}")
    S, rcv = 70, 2 * Na - 3
    z = W.make_channelised(B, 64, S, 2 * Na, "f32", seed=5, device=dev)
    ref, _ = afc.correlate(z, n_spectra=S)
    y = z.clone()
    y[0, 7, 5, rcv, 2, 0] = float(bad)
    got, _ = afc.correlate(y, n_spectra=S)
    a, c = np.tril_indices(Na)
    r, g = ref.cpu().numpy(), got.cpu().numpy()
    same = np.ones(64, bool)
    same[7] = False
    np.testing.assert_array_equal(r[0, same], g[0, same])
    auto = np.sqrt(np.abs(r[0, 7][a == c][:, [0, 1], [0, 1], 0]).astype(np.float64)).reshape(-1)    # [N]
    for p in range(2):
        for q in range(2):
            hit = (2 * a + p == rcv) | (2 * c + q == rcv)
            d = np.abs(g[0, 7, ~hit, p, q].astype(np.float64) - r[0, 7, ~hit, p, q]).max(-1)
            assert (d / (auto[2 * a + p] * auto[2 * c + q])[~hit]).max() <= 2e-5
            v = g[0, 7, hit & (a != c), p, q]
            if v.size == 0:
                continue
            if np.isnan(bad):
                assert np.isnan(v).all()
            elif np.isinf(bad):
                assert np.isinf(v).all()
            else:
                x = W.blocked_to_natural(y.cpu(), S).numpy().astype(np.float64)[0, 7]
                x = x[..., 0] + 1j * x[..., 1]
                k = np.flatnonzero(hit & (a != c))
                e = (x[:, 2 * a[k] + p] * x[:, 2 * c[k] + q].conj()).sum(0)
                fin = np.abs(e) < 1e38                      # (above: float32 overflows in either form)
                m = np.abs(x).max(0)
                err = np.abs((v[fin, 0] + 1j * v[fin, 1]) - e[fin])
                assert np.all(err <= 1e-5 * S * (m[2 * a[k] + p] * m[2 * c[k] + q])[fin])


@pytest.mark.parametrize("dtype", ["i8", "f16", "f32"])
@pytest.mark.parametrize("Na,S,B", [(100, 1000, 12), (128, 700, 10), (48, 1500, 8), (33, 1200, 24)])
def test_tile_width_does_not_change_results(afc, dev, dtype, Na, S, B):
    """The tile width follows the launch's size: one of these subbands alone
    takes 64-wide tiles (fp32 at 100 and 128 antennas 128-wide), all of them
    together 128-wide ones (at 66 receivers 64-wide).  The sums run over the
    spectra in the same order either way: identical bit for bit, flags,
    weights and ragged lengths among them."""
    log(f"xengine tile widths {dtype} Na={Na} S={S} B={B}")
    z = W.make_channelised(B, 64, S, 2 * Na, dtype, seed=Na, device=dev)
    fl = torch.zeros((B, Na), dtype=torch.uint8, device=dev)
    fl[:, 5] = 1
    S_sb = [S - 13 * b for b in range(B)]
    v, w = afc.correlate(z, n_spectra=S, n_spectra_per_sb=S_sb, flags=fl)
    for b in (0, B - 1):
        v1, w1 = afc.correlate(z[b:b + 1].contiguous(), n_spectra=S, n_spectra_per_sb=S_sb[b:b + 1], flags=fl[b:b + 1])
        assert torch.equal(v1[0].view(torch.int32), v[b].view(torch.int32)), b
        assert torch.equal(w1[0], w[b])
    del z, v
    torch.cuda.empty_cache()


@pytest.mark.parametrize("Na,B", [(33, 1), (8, 4), (48, 1), (48, 2), (75, 1), (8, 8)])
@pytest.mark.parametrize("S", [1, 31, 32, 33, 128, 129, 401])
def test_int8_groups_of_a_small_launch(afc, dev, Na, B, S):
    """A launch that leaves the CUs mostly empty gives each int8 tile four or
    two groups of waves, which share its stages of 32 spectra: fewer stages
    than groups, one each, remainders, ragged lengths, flags and weights, up to
    the workgroup counts where the groups change (256 and 512)."""
    log(f"xengine int8 groups Na={Na} B={B} S={S}")
    z = W.make_channelised(B, 64, S, 2 * Na, "i8", seed=Na + S, device=dev)
    S_sb = [max(1, S - 5 * b) for b in range(B)]
    fl_np = np.zeros((B, Na), np.uint8)
    fl_np[:, 3] = 1
    vis, w = afc.correlate(z, n_spectra=S, n_spectra_per_sb=S_sb, flags=torch.from_numpy(fl_np).to(dev))
    vis_np, w_np = vis.cpu().numpy(), w.cpu().numpy()
    zn = W.blocked_to_natural(z.cpu(), z.shape[2] * 8).numpy()
    for b in {0, B - 1}:
        for ch in (0, 41, 63):
            V, W_ = oracle.xcorr_int(zn[b, ch, :S_sb[b]], fl_np[b])
            np.testing.assert_array_equal(vis_np[b, ch].astype(np.int64), V)
            np.testing.assert_array_equal(w_np[b], W_)


@pytest.mark.parametrize("B,Na,S", [(1, 75, 97), (4, 48, 40), (1, 100, 200), (1, 150, 65), (4, 100, 200)])
@pytest.mark.parametrize("power", [-20, -30])
def test_f32_split_goes_by_the_receivers_scale(afc, dev, B, Na, S, power):
    """A sample far below its receiver's others does not take a tile off the
    bf16 split (among samples of 1e-9, some lie below any bound on a single
    one): the split's products scale exactly, so samples times 2^power give
    the visibilities times 2^(2 power) bit for bit."""
    log(f"xengine f32 scale B={B} Na={Na} S={S} power={power}")
    z = W.make_channelised(B, 64, S, 2 * Na, "f32", seed=Na + S, device=dev)
    z[:, :, 0, ::2, 1, 0] = 2.0 ** -33                      # scaled: 2^-53, 2^-63
    ref, _ = afc.correlate(z, n_spectra=S)
    got, _ = afc.correlate(z * 2.0 ** power, n_spectra=S)
    assert torch.equal(got, ref * 2.0 ** (2 * power))


# fp32 tiles of one subband alone and of all together: 64 and 128 wide at 48
# antennas and at 100 x 4 (with a tile off the diagonal), 128 and 64 at 100 x 2
@pytest.mark.parametrize("B,Na,S", [(4, 48, 300), (4, 100, 200), (2, 100, 33)])
@pytest.mark.parametrize("case", ["inf", "large", "late", "small", "all"])
def test_f32_out_of_range_antennas_leave_the_others_alone(afc, dev, B, Na, S, case):
    """A baseline's bits depend on the samples of its own two antennas: one that
    the bf16 split cannot hold changes no bit of the others' visibilities, and
    its own are the same in tiles of either width, weights and flags too."""
    log(f"xengine f32 out-of-range antennas B={B} Na={Na} S={S} {case}")
    z = W.make_channelised(B, 64, S, 2 * Na, "f32", seed=Na, device=dev)
    fl = torch.zeros((B, Na), dtype=torch.uint8, device=dev)
    fl[:, 5] = 1
    ref, wref = afc.correlate(z, n_spectra=S, flags=fl)
    y, ants = z.clone(), [3, Na - 2]
    for a in ants if case != "all" else range(Na):
        if case == "inf":
            y[:, :, 0, 2 * a + 1, 2, 1] = np.inf
        elif case == "large":
            y[:, :, :, 2 * a] *= 2.0 ** 55
        elif case == "late":
            y[:, :, (S - 1) // 8, 2 * a, (S - 1) % 8, 0] = 2.0 ** 51
        else:
            y[:, :, :, 2 * a:2 * a + 2] *= 2.0 ** -56
    got, w = afc.correlate(y, n_spectra=S, flags=fl)
    assert torch.equal(w, wref)
    if case != "all":
        a, c = np.tril_indices(Na)
        rest = torch.from_numpy(~(np.isin(a, ants) | np.isin(c, ants))).to(dev)
        assert torch.equal(got[:, :, rest], ref[:, :, rest])
    for b in range(B):
        v1, w1 = afc.correlate(y[b:b + 1].contiguous(), n_spectra=S, flags=fl[b:b + 1])
        assert torch.equal(v1[0].view(torch.int32), got[b].view(torch.int32)), b
        assert torch.equal(w1[0], w[b])


@pytest.mark.parametrize("dtype,Na,B,S,tile", [("i8", 40, 8, 1000, 128), ("i8", 128, 3, 64, 64), ("i8", 1500, 1, 16, 128),
                                               ("f16", 33, 8, 200, 128), ("f16", 100, 3, 300, 64),
                                               ("f32", 48, 4, 100, 128), ("f32", 288, 1, 2, 64), ("f32", 75, 3, 1, 64)])
def test_tile_width_by_the_lengths(afc, dev, dtype, Na, B, S, tile):
    """Launches whose faster tile width the sizes without the integration
    lengths, or without the stores, do not tell: the plan takes the rule's."""
    log(f"tile width {dtype} Na={Na} B={B} S={S}")
    plan = afc.Plan(Na, [S] * B, [dtype] * B)
    assert plan.info().tile == tile
    plan.close()
