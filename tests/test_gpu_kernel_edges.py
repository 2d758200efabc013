"""GPU parity at the sizes where a kernel or a branch of a launch can go wrong:
tile edges, remainders, the smallest and largest of a range, both sides of a
rule on sizes.  Integer results and fixed-order fp32 results are compared with
the CPU oracle bit for bit; other bounds are derived where they are used."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_17652_amd as F

pytestmark = pytest.mark.gpu

DEV = "cuda"
D = 128


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F.lib()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def status(st):
    torch.cuda.synchronize()
    return int(st.item()) & 0xFFFFFFFF


def threshold_keys(rng, n, kdt):
    """Keys on and one unit in the last place beside the cell boundaries T * s of
    their block, signed zeros, and magnitudes far below a cell."""
    K = (rng.standard_normal((n, D)) * np.exp(rng.standard_normal(D))).astype(kdt)
    for c in range(0, D, 3):
        a = np.float16(np.exp(rng.uniform(-6, 6)))
        s = np.float32(a) / np.float32(8)
        k = (rng.integers(-8, 9, n) * s).astype(kdt)
        side = rng.integers(-1, 2, n)
        k = np.where(side == 0, k, np.nextafter(k, np.where(side > 0, np.inf, -np.inf).astype(kdt), dtype=kdt))
        tiny = rng.random(n) < 0.2
        k[tiny] = (rng.choice([-1.0, 1.0, -0.0, 0.0], tiny.sum()) * s * 2.0 ** rng.integers(-30, -10, tiny.sum())).astype(kdt)
        k[::64] = np.float32(a)  # the block maximum
        K[:, c] = np.clip(k, -np.float32(a), np.float32(a)).astype(kdt)
    return K


@pytest.mark.parametrize("kdt", [np.float32, np.float16])
@pytest.mark.parametrize("U,nb_cap,ld", [(52, 67, 128), (3, 67, 160), (17, 256, 128)])
def test_pack_tiles(kdt, U, nb_cap, ld):
    """Workgroups of 16 blocks (the first and the last shape) and one wave per
    item (the second) at odd block strides: ragged ends inside a tile, empty
    units, padded rows, keys at the cell boundaries, NaN and infinite keys."""
    rng = np.random.default_rng(7 * U + nb_cap)
    cap = nb_cap * 64
    ns = [int(x) for x in rng.integers(0, cap + 1, U)]
    ns[:3] = [cap, cap - 1, 1023]
    if U > 6:
        ns[3:7] = [0, 1, 1024, 1025]
    K = torch.full((U, cap, ld), float("nan"), dtype=torch.float32 if kdt == np.float32 else torch.float16, device=DEV)
    host = {}
    for u in range(min(U, 7)):
        k = threshold_keys(rng, ns[u], kdt)
        if u == 2:
            k[70, 5], k[71, 6], k[200, 5], k[1000, 9] = np.nan, np.inf, -np.inf, np.nan
        host[u] = k
        K[u, :ns[u], :D] = dev(k)
    for u in range(7, U):
        K[u, :ns[u], :D] = torch.randn((ns[u], D), device=DEV).to(K.dtype)
    st = F.new_status()
    planes, scales = F.fathom_pack(K[:, :, :D], dev(np.array(ns, np.int64)), nb_cap=nb_cap, dev_status=st)
    assert status(st) == (F.FATHOM_DEV_NONFINITE | F.FATHOM_DEV_SCALE_OVERFLOW)
    for u, k in host.items():
        op, os_, _ = oracle.pack(k.astype(np.float32), nb_cap=nb_cap)
        assert np.array_equal(scales[u].cpu().numpy().view(np.uint16), os_), f"scales unit {u} n={ns[u]}"
        assert np.array_equal(planes[u].cpu().numpy().view(np.uint64), op), f"planes unit {u} n={ns[u]}"


@pytest.mark.parametrize("kdt", [np.float32, np.float16])
@pytest.mark.parametrize("U,cap,pad", [(3, 1, 0), (1, 8195, 0), (2, 4099, 3), (600, 17, 8), (1, 262200, 0)])
def test_rotate_keys_runs(kdt, U, cap, pad):
    """Runs of 16 to 512 tokens per workgroup with ragged last groups of four,
    empty and one-token units, and rows whose stride rules out 16-byte loads
    (pad 3); bit-exact to the oracle on sampled rows of every unit checked."""
    rng = np.random.default_rng(U + cap)
    ld = D + pad
    tdt = torch.float32 if kdt == np.float32 else torch.float16
    K = torch.randn((U, cap, ld), device=DEV).to(tdt)
    ns = rng.integers(0, cap + 1, U)
    ns[0] = cap
    mu = rng.standard_normal((U, D)).astype(np.float32)
    V = rng.standard_normal((U, D, D)).astype(np.float32)
    st = F.new_status()
    out = torch.full((U, cap, D), 7.0, device=DEV)
    F.fathom_klt_rotate_keys(K[:, :, :D], dev(ns.astype(np.int64)), dev(mu), dev(V), out=out, dev_status=st)
    assert status(st) == 0
    for u in sorted({0, U // 2, U - 1}):
        n = int(ns[u])
        rows = np.unique(np.concatenate([np.arange(min(n, 600)), np.arange(max(0, n - 600), n)])).astype(np.int64)
        got = out[u, dev(rows)].cpu().numpy()
        ref = oracle.klt_rotate_keys(K[u, dev(rows), :D].cpu().numpy(), mu[u], V[u])
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (u, n)
        assert bool((out[u, n:] == 7.0).all())  # rows past n are left as they were


@pytest.mark.parametrize("kdt", [np.float32, np.float16])
@pytest.mark.parametrize("U,cap,pad,offset", [(1, 1, 0, 0.0), (3, 259, 3, 1.0), (9, 1030, 0, 300.0), (1, 20011, 8, 1.0)])
def test_calibrate_chunks(kdt, U, cap, pad, offset):
    """Calibration over 1 to 54 chunks per unit with ragged last steps of four
    tokens, empty, one-key and rank-deficient units, a mean far from zero, and
    strides that rule out 16-byte loads.  Bounds, with L the largest eigenvalue:
    fp32 mean; |eigenvalue error|, |C v - lambda v| and |V^T V - I| of an fp32
    Jacobi (128 x 128, backward error a few hundred units in the last place):
    2e-5 L, 1e-4 L, 1e-5."""
    rng = np.random.default_rng(U * 1000 + cap)
    A = rng.standard_normal((D, D)) * np.geomspace(3.0, 0.05, D)
    ns = rng.integers(0, cap + 1, U)
    ns[0] = cap
    if U > 2:
        ns[1:3] = [0, 2]
    K = rng.standard_normal((U, cap, D + pad))
    K[:, :, :D] = K[:, :, :D] @ A.T + offset * rng.standard_normal(D)
    K = K.astype(kdt)
    st = F.new_status()
    mu, V, lam = (t.cpu().numpy().astype(np.float64) for t in
                  F.fathom_klt_calibrate(dev(K)[:, :, :D], dev(ns.astype(np.int64)), dev_status=st))
    assert status(st) == 0
    for u in range(U):
        k = K[u, :ns[u], :D].astype(np.float64)
        m = k.mean(0) if len(k) else np.zeros(D)
        C = (k - m).T @ (k - m) / max(len(k), 1)
        w = np.linalg.eigvalsh(C)[::-1]
        L = max(w[0], 1e-300)
        assert np.abs(mu[u] - m).max() <= 1.2e-7 * np.abs(m).max() + 1e-30
        assert np.abs(lam[u] - w).max() <= 2e-5 * L and (np.diff(lam[u]) <= 0).all()
        assert np.abs(C @ V[u] - V[u] * lam[u]).max() <= 1e-4 * L
        assert np.abs(V[u].T @ V[u] - np.eye(D)).max() <= 1e-5
        if ns[u] <= 1:
            assert (V[u] == np.eye(D)).all() and (lam[u] == 0).all()
        else:
            assert (V[u][np.abs(V[u]).argmax(0), np.arange(D)] > 0).all()


def topk_rows(rng, kind, n):
    if kind == "narrow":  # one binade: every digit has to be refined
        return (1000.0 + rng.standard_normal(n) * 0.01).astype(np.float32)
    if kind == "equal":  # more equal scores than a list holds, few above them
        s = np.full(n, 2.5, np.float32)
        s[rng.integers(0, max(n, 1), 40 if n else 0)] = 3.0
        return s
    if kind == "late":  # the equal scores at the threshold only in the last third
        s = -np.abs(rng.standard_normal(n)).astype(np.float32)
        s[2 * n // 3:] = 0.0
        s[n // 2:n // 2 + 9] = -0.0
        return s
    if kind == "cluster":  # equal scores inside the list: the row is sorted
        return np.where(rng.random(n) < 0.01, np.float32(4.0), rng.standard_normal(n)).astype(np.float32)
    s = rng.standard_normal(n).astype(np.float32)
    s[rng.random(n) < 0.01] = np.nan
    s[rng.random(n) < 0.01] = np.inf
    return s


@pytest.mark.parametrize("kind", ["narrow", "equal", "late", "cluster", "special"])
@pytest.mark.parametrize("k,lo,tail", [(1, 0, 0), (500, 4, 32), (2048, 0, 0), (8192, 3, 1)])
def test_topk_refinement(kind, k, lo, tail):
    """fathom_topk where rows take one, two or three digits, where the equal
    scores at the threshold do not fit the list (index order decides), where a
    list holds many equal scores, and at the ends of chunks of 4096: indices and
    values equal to the oracle's."""
    rng = np.random.default_rng(k)
    ns = [40961, 20000, 4096, lo + tail + 1, 8193]
    ld = 40970
    s = np.zeros((len(ns), 2, ld), np.float32)
    for u, n in enumerate(ns):
        for h in range(2):
            s[u, h, :n] = topk_rows(rng, kind, n)
    st = F.new_status()
    idx, val = F.fathom_topk(dev(s), dev(np.array(ns, np.int64)), k, lo, tail, dev_status=st)
    flags, want = status(st), 0
    idx, val = idx.cpu().numpy(), val.cpu().numpy()
    for u, n in enumerate(ns):
        for h in range(2):
            oi, ov, ost = oracle.topk(s[u, h, :n], k, lo, tail)
            want |= ost
            assert np.array_equal(idx[u, h], oi), (u, h)
            assert np.array_equal(val[u, h], ov, equal_nan=True), (u, h)
    assert flags == want


@pytest.mark.parametrize("G,qdt", [(1, np.float32), (3, np.float16), (4, np.float16), (8, np.float32)])
@pytest.mark.parametrize("U,nb_cap", [(43, 90), (2, 19), (80, 90)])
def test_scan_stages(G, qdt, U, nb_cap):
    """fathom_scan with four blocks and one block a wave, 0 to 128 active channels
    (none to four stages), every depth, ragged ends and a score row shorter than
    the keys; bit-exact to the oracle's fp32 order."""
    rng = np.random.default_rng(G * 100 + U)
    cap = nb_cap * 64
    ns = rng.integers(1, cap + 1, U)
    ns[0], ns[1] = cap, 1025
    K = torch.randn((U, cap, D), device=DEV)
    planes, scales = F.fathom_pack(K, dev(ns.astype(np.int64)), nb_cap=nb_cap)
    q = rng.standard_normal((U, G, D)).astype(qdt)
    depths = rng.integers(0, 5, (U, D)).astype(np.uint8)
    depths[rng.random((U, D)) < 0.4] = 0
    depths[0], depths[1] = 0, 0
    depths[0, [0, 63, 64, 127]] = [1, 2, 3, 4]
    if U > 2:
        depths[2], depths[3, :], depths[4, :65] = 4, 0, 1
    ld = cap - 70
    st = F.new_status()
    s = F.fathom_scan(planes, scales, dev(ns.astype(np.int64)), dev(q), dev(depths), ld_s=ld, dev_status=st)
    assert status(st) == 0
    for u in range(min(U, 8)):
        n = int(ns[u])
        ref = oracle.scores_f32(planes[u].cpu().numpy().view(np.uint64), scales[u].cpu().numpy().view(np.uint16), n,
                                q[u].astype(np.float32), depths[u])
        m = min(n, ld)
        assert np.array_equal(s[u, :, :m].cpu().numpy().view(np.uint32), ref[:, :m].view(np.uint32)), u


@pytest.mark.parametrize("G", [1, 4, 8])
def test_alloc_depths_extremes(G):
    """Importances from subnormal to 1e38, equal and zero ones, and every budget's
    ends: the 32-bit candidate keys and the early end of the search against the
    oracle's exact candidates; top-r ranks with equal weights."""
    rng = np.random.default_rng(G)
    U = 9
    q = rng.standard_normal((U, G, D)).astype(np.float32)
    var = np.exp(rng.standard_normal((U, D))).astype(np.float32)
    var[1] = np.exp(rng.uniform(-103, 80, D)).astype(np.float32)      # subnormal to huge
    q[2], var[2] = 1.0, 1.0                                            # all equal
    q[3] = np.round(q[3])                                              # many equal, many zero
    var[3] = 4.0 ** rng.integers(-3, 4, D)
    var[4] = 0.0
    var[5, 1:] = 0.0
    var[6, ::2] = 0.0
    q[7] *= np.float32(1e-22)                                          # squares in the subnormals
    q[8] *= np.float32(1e18)
    for B in (0, 1, 2, 47, 128, 500, 511, 512):
        st = F.new_status()
        d, th = F.fathom_alloc_depths(dev(q), dev(var), F.FATHOM_WATERFILL, B, dev_status=st)
        d, th, flags = d.cpu().numpy(), th.cpu().numpy(), status(st)
        want = 0
        for u in range(U):
            od, oth, ost = oracle.alloc_waterfill(q[u], var[u], B)
            want |= ost
            assert np.array_equal(d[u], od), (B, u)
            assert th[u] == np.float32(oth), (B, u)
        assert flags == want
    for r in (0, 1, 63, 127, 128):
        d, th = F.fathom_alloc_depths(dev(q), None, F.FATHOM_UNIFORM_TOPR, r)
        for u in range(U):
            od = oracle.alloc_topr(q[u], r)[0]
            assert np.array_equal(d[u].cpu().numpy(), od), (r, u)


def depth_row(rng, spec):
    """Depths with spec = {depth: channel count} on channels drawn at random."""
    d = np.zeros(D, np.uint8)
    ch = rng.permutation(D)
    at = 0
    for t, c in spec.items():
        d[ch[at:at + c]] = t
        at += c
    return d


@pytest.mark.parametrize("G,qdt", [(4, np.float16), (3, np.float32), (1, np.float32)])
def test_scan_topk_81_to_128_cells(G, qdt):
    """Units of 81 to 128 depth bits in the cell filter at eight slices (the
    caller bounds the bits by 128): 32 channels at 4 planes, 128 one-plane
    channels (every channel of the unit), 81 cells (a ragged last row group), 100
    channels of mixed depth, water-filling at 96 bits, and units of few cells
    beside them; odd block strides, a window with lo and tail, k = 1 and 300.  The
    filter serves them (no fallback flag at k = 300); without a bound the same
    units take the wide pass.  Both bit-exact to the oracle."""
    ns = [70000, 23456, 40001, 30000, 50000, 64, 20000, 30001]
    rng = np.random.default_rng(300 + G)
    U, cap = len(ns), max(ns)
    K = torch.randn((U, cap, D), device=DEV) * torch.exp(torch.randn((U, 1, D), device=DEV))
    n = dev(np.array(ns, np.int64))
    q = rng.standard_normal((U, G, D)).astype(qdt)
    var = np.exp(2 * rng.standard_normal((U, D))).astype(np.float32)
    dn = F.fathom_alloc_depths(dev(q), dev(var), F.FATHOM_WATERFILL, 96)[0].cpu().numpy()
    specs = {0: {4: 32}, 1: {1: 128}, 2: {4: 17, 1: 13}, 3: {1: 72, 2: 28}, 4: {4: 31, 3: 1, 1: 1}, 5: {4: 32},
             7: {2: 3}}
    for u, spec in specs.items():
        dn[u] = depth_row(rng, spec)
    assert [int(dn[u].sum()) for u in specs] == [128, 128, 81, 128, 128, 128, 6]
    assert dn[6].sum() <= 96
    for nb_cap in (1094, 1101):
        planes, scales = F.fathom_pack(K, n, nb_cap=nb_cap)
        P, S = planes.cpu().numpy().view(np.uint64), scales.cpu().numpy().view(np.uint16)
        ref = [oracle.scores_f32(P[u], S[u], ns[u], q[u].astype(np.float32), dn[u]) for u in range(U)]
        for k, lo, tail in [(300, 0, 0), (300, 4, 32), (1, 0, 0)]:
            want = [[oracle.topk(ref[u][h], k, lo, tail) for h in range(G)] for u in range(U)]
            for bound in (128, 0):
                st = F.new_status()
                idx, val = F.fathom_scan_topk(planes, scales, n, dev(q), dev(dn), k, lo, tail, dev_status=st,
                                              max_unit_bits=bound)
                s = status(st)
                assert s & ~(F.FATHOM_DEV_TOPK_SHORT | F.FATHOM_DEV_TOPK_FALLBACK) == 0, (bound, hex(s))
                assert k == 1 or not s & F.FATHOM_DEV_TOPK_FALLBACK, (bound, lo)
                for u in range(U):
                    for h in range(G):
                        oi, ov, _ = want[u][h]
                        assert np.array_equal(idx[u, h].cpu().numpy(), oi), (bound, k, u, h)
                        assert np.array_equal(val[u, h].cpu().numpy(), ov, equal_nan=True), (bound, k, u, h)


@pytest.mark.parametrize("k", [0, 1, 92, 128, 220, 257, 476, 512, 513])
@pytest.mark.parametrize("U", [3, 45, 70])
def test_sparse_attn_row_lists(k, U):
    """Row lists of 1 to 17 chunks on both sides of the one-workgroup rule (at most
    8 chunks, 9 with 12 rows, 16 with 180, 8 with more than 256), with sink and local rows, skipped
    entries, a short unit, an empty unit and empty chunks.  Bound: the oracle's,
    1e-5 of the softmax-weighted mean of |V|, at most 1e-5 max |V|."""
    rng = np.random.default_rng(k + U)
    G, cap = 4, 700
    ns = rng.integers(1, cap + 1, U)
    ns[:3] = [cap, 40, 0]
    K = rng.standard_normal((U, cap, D)).astype(np.float16)
    V = rng.standard_normal((U, cap, D)).astype(np.float16)
    q = rng.standard_normal((U, G, D)).astype(np.float32)
    for sink, local in [(0, 0), (4, 32)]:
        idx = np.full((U, G, k), -1, np.int32)
        for u in range(U):
            for h in range(G):
                m = min(k, int(ns[u]))
                idx[u, h, rng.permutation(k)[:m]] = rng.permutation(int(ns[u]))[:m]
        idx[0, 0, : min(k, 64)] = -1  # a head whose first chunks are empty
        out = F.fathom_sparse_attn(dev(q), dev(K), dev(V), dev(ns.astype(np.int64)), dev(idx), sink, local).cpu().numpy()
        for u in [0, 1, 2, U - 1]:
            ref = oracle.sparse_attn(q[u], K[u, :ns[u]], V[u, :ns[u]], idx[u], sink, local, 1 / np.sqrt(D))
            assert np.abs(out[u] - ref).max() <= 1e-5 * np.abs(V[u].astype(np.float32)).max(), (u, sink)


def filtered_rows(ws, U, G, k):
    """Rows [U][G] that the filter served, from the workspace of a call: a threshold
    and a survivor list that holds the top k.  Layout: a threshold a row, then a
    256-byte line a row whose first word counts the survivors; the list's capacity
    is twice min(2k + 2048, 16384)."""
    R = U * G
    tau = ws[: 4 * R].view(torch.float32).cpu().numpy()
    at = (4 * R + 255) // 256 * 256
    cnt = ws[at: at + 256 * R].view(torch.int32).view(R, 64)[:, 0].cpu().numpy()
    return (np.isfinite(tau) & (cnt >= k) & (cnt <= 2 * min(2 * k + 2048, 16384))).reshape(U, G)


@pytest.mark.parametrize("k", [1, 1000, 1024, 1025, 2048, 2049])
@pytest.mark.parametrize("U", [28, 36])
def test_scan_topk_many_rows(U, k):
    """112 and 144 rows: more than one round of the chip at 8 rank parts a row, so 1,
    2 or 8 parts by rows and k; a unit with many equal scores (keys drawn from four
    blocks), one whose ends are inside a sampled quad (odd stride), and windows.
    Bit-exact to the oracle; the filter serves all but a few rows of the other units
    from k = 1000 (the rank pass is reached, not only the exact rows; a threshold
    misses by chance in one row of some thousands)."""
    rng = np.random.default_rng(k)
    G, cap = 4, 24003
    ns = rng.integers(16000, cap + 1, U)
    ns[0] = cap
    torch.manual_seed(1000 * U + k)
    K = torch.randn((U, cap, D), device=DEV) * torch.exp(torch.randn((U, 1, D), device=DEV))
    K[1] = K[1, :256].repeat(94, 1)[:cap]
    n = dev(ns.astype(np.int64))
    planes, scales = F.fathom_pack(K, n)
    q = rng.standard_normal((U, G, D)).astype(np.float16)
    var = np.exp(2 * rng.standard_normal((U, D))).astype(np.float32)
    d, _ = F.fathom_alloc_depths(dev(q), dev(var), F.FATHOM_WATERFILL, 48)
    ws = torch.empty((F.fathom_scan_topk_workspace_size(U, G, 64 * planes.shape[-1], k),), dtype=torch.uint8, device=DEV)
    for lo, tail in [(0, 0), (4, 32)]:
        st = F.new_status()
        idx, val = F.fathom_scan_topk(planes, scales, n, dev(q), d, k, lo, tail, ws=ws, dev_status=st, max_unit_bits=48)
        assert status(st) & ~F.FATHOM_DEV_TOPK_FALLBACK == 0
        served = filtered_rows(ws, U, G, k)
        served[1] = True
        assert k == 1 or (~served).sum() <= 2
        for u in [0, 1, 2, 13, U - 1]:
            ref = oracle.scores_f32(planes[u].cpu().numpy().view(np.uint64), scales[u].cpu().numpy().view(np.uint16),
                                    int(ns[u]), q[u].astype(np.float32), d[u].cpu().numpy())
            for h in range(G):
                oi, ov, _ = oracle.topk(ref[h], k, lo, tail)
                assert np.array_equal(idx[u, h].cpu().numpy(), oi), (u, h, lo)
                assert np.array_equal(val[u, h].cpu().numpy(), ov, equal_nan=True), (u, h, lo)


@pytest.mark.parametrize("G,qdt", [(5, np.float32), (6, np.float16), (8, np.float16)])
@pytest.mark.parametrize("B", [48, 64, 80, 96, 200])
def test_scan_topk_more_than_4_heads(G, qdt, B):
    """5 to 8 query heads: the cell filter 4 heads at a time for every slice count
    (and units above the bound, which are computed exactly), beside a unit that is
    computed directly and an empty one; with and without a bound, which takes the
    exact path.  Bit-exact to the oracle, and the fallback flag as documented; the
    flag is raised for more than 4 heads either way, so that the filter served the
    long units' rows, both fours of them, is read from the workspace."""
    rng = np.random.default_rng(G * B)
    ns = [40000, 23457, 2000, 0, 33000]
    U, cap, k = len(ns), 40000, 300
    torch.manual_seed(G * B)
    K = torch.randn((U, cap, D), device=DEV) * torch.exp(torch.randn((U, 1, D), device=DEV))
    n = dev(np.array(ns, np.int64))
    planes, scales = F.fathom_pack(K, n)
    q = rng.standard_normal((U, G, D)).astype(qdt)
    var = np.exp(2 * rng.standard_normal((U, D))).astype(np.float32)
    d, _ = F.fathom_alloc_depths(dev(q), dev(var), F.FATHOM_WATERFILL, B)
    P, S, dn = planes.cpu().numpy().view(np.uint64), scales.cpu().numpy().view(np.uint16), d.cpu().numpy()
    ref = [oracle.scores_f32(P[u], S[u], ns[u], q[u].astype(np.float32), dn[u]) for u in range(U)]
    ws = torch.empty((F.fathom_scan_topk_workspace_size(U, G, 64 * planes.shape[-1], k),), dtype=torch.uint8, device=DEV)
    for lo, tail in [(0, 0), (4, 32)]:
        for bound in (min(B, 96), 0):
            st = F.new_status()
            idx, val = F.fathom_scan_topk(planes, scales, n, dev(q), d, k, lo, tail, ws=ws, dev_status=st, max_unit_bits=bound)
            assert status(st) == (F.FATHOM_DEV_TOPK_FALLBACK | F.FATHOM_DEV_TOPK_SHORT)
            assert (filtered_rows(ws, U, G, k)[[0, 1, 4]] == (B <= bound)).all(), (lo, bound)
            for u in range(U):
                for h in range(G):
                    oi, ov, _ = oracle.topk(ref[u][h], k, lo, tail)
                    assert np.array_equal(idx[u, h].cpu().numpy(), oi), (u, h, lo, bound)
                    assert np.array_equal(val[u, h].cpu().numpy(), ov, equal_nan=True), (u, h, lo, bound)


@pytest.mark.parametrize("k,bound", [(300, 48), (560, 48), (620, 48), (2048, 48), (4096, 48), (2048, 0), (4096, 128)])
@pytest.mark.parametrize("clumped", [False, True])
def test_scan_topk_large_k(k, bound, clumped):
    """k from 1/110 to 1/8 of the keys: the samples of tau are a block's two largest
    scores or its r-th largest (k above about 1/53), in the cell filter and the
    wide pass.  With independent keys the filter serves every row (no fallback
    flag); with the large scores in a few blocks it may not, and the result is the
    same.  Bit-exact to the oracle."""
    rng = np.random.default_rng(k)
    U, G = 5, 4
    ns = [32768, 32701, 40000, 36007, 33333]
    cap = max(ns)
    K = torch.randn((U, cap, D), device=DEV) * torch.exp(torch.randn((U, 1, D), device=DEV))
    if clumped:
        K[:, :1000] *= 6.0
    n = dev(np.array(ns, np.int64))
    planes, scales = F.fathom_pack(K, n)
    q = rng.standard_normal((U, G, D)).astype(np.float16)
    var = np.exp(2 * rng.standard_normal((U, D))).astype(np.float32)
    d, _ = F.fathom_alloc_depths(dev(q), dev(var), F.FATHOM_WATERFILL, 48 if bound == 48 else 100)
    P, S, dn = planes.cpu().numpy().view(np.uint64), scales.cpu().numpy().view(np.uint16), d.cpu().numpy()
    st = F.new_status()
    idx, val = F.fathom_scan_topk(planes, scales, n, dev(q), d, k, 4, 32, dev_status=st, max_unit_bits=bound)
    assert status(st) & ~F.FATHOM_DEV_TOPK_FALLBACK == 0
    assert clumped or status(st) == 0
    for u in range(U):
        ref = oracle.scores_f32(P[u], S[u], ns[u], q[u].astype(np.float32), dn[u])
        for h in range(G):
            oi, ov, _ = oracle.topk(ref[h], k, 4, 32)
            assert np.array_equal(idx[u, h].cpu().numpy(), oi), (u, h)
            assert np.array_equal(val[u, h].cpu().numpy(), ov, equal_nan=True), (u, h)


@pytest.mark.parametrize("G", [4, 6])
def test_scan_topk_sample_steps(G):
    """Sample steps of 1 to 4 planes on both sides of the 64th active channel and
    with 1 to 4 channels in the last step; windows whose lo and n leave most
    sampled quads without a key, units below lo.  k is small beside the windows,
    so the filter serves every row of at most 4 heads (no fallback flag: a sample
    above its key's score would leave fewer than k survivors).  Bit-exact to the
    oracle."""
    rng = np.random.default_rng(40 + G)
    ns = [60000, 27000, 60000, 20011, 33, 52345, 60000]
    U, cap, k = len(ns), max(ns), 30
    tail_of = [[1, 2, 1, 3], [4], [2, 2, 4, 1, 1, 1, 1, 3, 3], [1, 1, 4, 4, 1], [3, 1, 1], [2], [4, 3]]
    dn = np.zeros((U, D), np.uint8)
    for u, tl in enumerate(tail_of):
        seq = [1] * (66 if u % 2 == 0 else 3) + tl
        dn[u, np.sort(rng.permutation(D)[:len(seq)])] = seq
    K = torch.randn((U, cap, D), device=DEV) * torch.exp(torch.randn((U, 1, D), device=DEV))
    n = dev(np.array(ns, np.int64))
    q = rng.standard_normal((U, G, D)).astype(np.float16)
    planes, scales = F.fathom_pack(K, n)
    P, S = planes.cpu().numpy().view(np.uint64), scales.cpu().numpy().view(np.uint16)
    ref = [oracle.scores_f32(P[u], S[u], ns[u], q[u].astype(np.float32), dn[u]) for u in range(U)]
    for lo, tail in [(0, 0), (20000, 100), (24575, 1)]:
        for bound in (128, 0):
            st = F.new_status()
            idx, val = F.fathom_scan_topk(planes, scales, n, dev(q), dev(dn), k, lo, tail, dev_status=st,
                                          max_unit_bits=bound)
            s = status(st)
            assert s & ~(F.FATHOM_DEV_TOPK_SHORT | F.FATHOM_DEV_TOPK_FALLBACK) == 0, hex(s)
            assert G > 4 or not s & F.FATHOM_DEV_TOPK_FALLBACK, (lo, bound)
            for u in range(U):
                for h in range(G):
                    oi, ov, _ = oracle.topk(ref[u][h], k, lo, tail)
                    assert np.array_equal(idx[u, h].cpu().numpy(), oi), (u, h, lo, bound)
                    assert np.array_equal(val[u, h].cpu().numpy(), ov, equal_nan=True), (u, h, lo, bound)


def spectrum_keys(rng, kind, n):
    """Keys [n][128] of a covariance with the named spectrum in a random basis."""
    Q = np.linalg.qr(rng.standard_normal((D, D)))[0]
    s = {"decaying": np.geomspace(3.0, 0.05, D), "isotropic": np.ones(D), "steep": np.geomspace(30.0, 1e-3, D),
         "outlier": np.where(np.arange(D) < 4, 40.0, np.exp(0.5 * rng.standard_normal(D)))}[kind]
    return (rng.standard_normal((n, D)) * s) @ Q.T


@pytest.mark.parametrize("kind", ["decaying", "isotropic", "steep", "outlier"])
def test_calibrate_orthonormal(kind):
    """The basis is orthonormal to the rounding of its entries, so that (qV).(kV)
    is q.k, and decorrelates the keys to it.  Bounds: entries rounded to fp32 (2^-24
    relative) move the dot product of two unit columns by at most 2^-23, so
    |V^T V - I|_F <= 128 * 2^-23, and V by at most 2^-24 sqrt(128) in the 2-norm of its
    entries, so the off-diagonal of V^T C V by twice that share of |C|_F (twice more
    where close eigenvalues leave rotations out: the isotropic covariances)."""
    rng = np.random.default_rng(len(kind))
    ns = [6000, 3001, 129, 40, 2]
    K = np.zeros((len(ns), max(ns), D), np.float32)
    for u, n in enumerate(ns):
        K[u, :n] = spectrum_keys(rng, kind, n)
    _, V, _ = F.fathom_klt_calibrate(dev(K), dev(np.array(ns, np.int64)))
    V = V.cpu().numpy().astype(np.float64)
    for u, n in enumerate(ns):
        assert np.linalg.norm(V[u].T @ V[u] - np.eye(D)) <= D * 2.0 ** -23, (u, n)
        x = K[u, :n].astype(np.float64) - K[u, :n].astype(np.float64).mean(0)
        C = x.T @ x / n
        W = V[u].T @ C @ V[u]
        off = np.linalg.norm(W - np.diag(np.diag(W))) / np.linalg.norm(C)
        assert off <= (4 if kind == "isotropic" else 2) * 2.0 ** -24 * np.sqrt(D), (u, n, off)


def test_calibrate_few_keys():
    """Units of 2 to 7 keys: the covariance has at most 6 directions, and the other
    eigenvalues are rounding error of either sign.  None is negative, and the depth
    allocation takes them as variances: no status bit, no plane for a channel whose
    variance is zero while others are not."""
    rng = np.random.default_rng(11)
    U = 48
    ns = 2 + np.arange(U) % 6
    K = (rng.standard_normal((U, 7, D)) * np.exp(rng.standard_normal(D)) + 3.0).astype(np.float32)
    n = dev(ns.astype(np.int64))
    _, V, lam = F.fathom_klt_calibrate(dev(K), n)
    assert bool((lam >= 0).all())
    q = F.fathom_klt_rotate_q(dev(rng.standard_normal((U, 4, D)).astype(np.float32)), V)
    st = F.new_status()
    d, _ = F.fathom_alloc_depths(q, lam, F.FATHOM_WATERFILL, 4, dev_status=st)
    assert status(st) == 0
    assert bool(((d > 0) <= (lam > 0)).all())


@pytest.mark.parametrize("U,cap", [(1, 1), (3, 18), (2, 1027), (5, 4099), (1, 70001)])
def test_rotate_keys_in_place(U, cap):
    """fp32 keys rotated into their own rows, with ragged ends of groups and runs,
    an empty unit, and U = 1 with any unit stride: the bits of a call with an
    output of its own, and rows past n left as they were."""
    rng = np.random.default_rng(cap)
    ns = rng.integers(0, cap + 1, U)
    ns[0] = cap
    if U > 2:
        ns[1] = 0
    n = dev(ns.astype(np.int64))
    K = torch.randn((U, cap, D), device=DEV)
    mu = dev(rng.standard_normal((U, D)).astype(np.float32))
    V = dev(rng.standard_normal((U, D, D)).astype(np.float32))
    ref = K.clone()
    F.fathom_klt_rotate_keys(K, n, mu, V, out=ref)
    F.fathom_klt_rotate_keys(K, n, mu, V, out=K)
    assert torch.equal(K.view(torch.int32), ref.view(torch.int32))


@pytest.mark.parametrize("share", [1.0, 0.8, 0.5, 0.1])
def test_topk_shared_bins(share):
    """A share of a row's scores in one bin of every digit (one value), the rest
    spread: the first pass adds up a wave's lanes of one bin, or not, by chunk;
    odd ends of chunks and rows of one score.  Indices and values equal to the
    oracle's."""
    rng = np.random.default_rng(int(10 * share))
    ns = [12289, 4096, 65, 1, 8191]
    s = rng.standard_normal((len(ns), 3, max(ns))).astype(np.float32)
    s = np.where(rng.random(s.shape) < share, np.float32(0.75), s)
    for k in (1, 70, 2500):
        idx, val = F.fathom_topk(dev(s), dev(np.array(ns, np.int64)), k)
        idx, val = idx.cpu().numpy(), val.cpu().numpy()
        for u, n in enumerate(ns):
            for h in range(3):
                oi, ov, _ = oracle.topk(s[u, h, :n], k, 0, 0)
                assert np.array_equal(idx[u, h], oi) and np.array_equal(val[u, h], ov, equal_nan=True), (k, u, h)


@pytest.mark.parametrize("n,k,lo", [(131072, 1, 0), (131071, 1024, 5), (262144, 8192, 0), (1 << 20, 300, 4),
                                    (4096 * 4096 + 70001, 2000, 3)])
def test_topk_ties_by_chunk(n, k, lo):
    """More equal scores at the threshold than a list holds, standing late, spread
    thin, in every second chunk, and from the window's start on, with few and with
    k - 1 scores above them; the last shape counts two chunks together.  The first
    equal ones in index order: indices and values equal to the oracle's."""
    rng = np.random.default_rng(k)
    s = -1.0 - rng.random((4, n)).astype(np.float32)
    ties = max(4 * k + 4096, n // 8)
    s[0, n - ties:] = 0.0
    s[1, rng.permutation(n)[:ties]] = 0.0
    s[2, (np.arange(n) - lo) // 4096 % 2 == 1] = 0.0
    s[3] = 0.0
    s[0, rng.integers(lo, n, min(k, 50) - 1)] = 2.0
    s[1, lo + rng.permutation(n - lo)[: k - 1]] = rng.integers(1, 9, k - 1)
    s[3, ::3] = -0.0
    idx, val = F.fathom_topk(dev(s[:, None]), dev(np.full(4, n, np.int64)), k, lo, 0)
    idx, val = idx.cpu().numpy(), val.cpu().numpy()
    for u in range(4):
        oi, ov, _ = oracle.topk(s[u], k, lo, 0)
        assert np.array_equal(idx[u, 0], oi), u
        assert np.array_equal(val[u, 0], ov), u


@pytest.mark.parametrize("kind", ["round", "outlier", "narrow", "pair", "normal", "same"])
@pytest.mark.parametrize("R,n,k", [(10, 1000, 40), (10, 30000, 8192), (100, 9001, 2048), (104, 9001, 5000), (200, 7000, 700),
                                   (400, 3000, 30), (400, 9001, 2048)])
def test_topk_uneven_lists(kind, R, n, k):
    """Lists whose interpolated sub-buckets are uneven (scores rounded to quarters,
    an outlier above or below the rest, one binade, two values, one value), short
    ones and long ones, beside even ones: 8, 4, 2 and 1 workgroups a row.  Indices
    and values equal to the oracle's."""
    rng = np.random.default_rng(R + k)
    s = rng.standard_normal((R, 1, n)).astype(np.float32)
    if kind == "round":
        s = np.round(4 * s) / 4
    elif kind == "outlier":
        s[:, 0, 7] = 1e30
        s[::2, 0, n - 1] = np.inf
    elif kind == "narrow":
        s = (1000 + 1e-3 * s).astype(np.float32)
    elif kind == "pair":
        s = np.where(s > 2.5, np.float32(2), np.float32(1))
    elif kind == "same":
        s[:] = -3.0
    idx, val = F.fathom_topk(dev(s), dev(np.full(R, n, np.int64)), k)
    idx, val = idx.cpu().numpy(), val.cpu().numpy()
    for u in sorted({0, 1, 7, 8, R // 2, R - 1}):
        oi, ov, _ = oracle.topk(s[u, 0], k, 0, 0)
        assert np.array_equal(idx[u, 0], oi), u
        assert np.array_equal(val[u, 0], ov), u


@pytest.mark.parametrize("k", [1000, 2000])
def test_scan_topk_rank_equal_scores(k):
    """136 rows, one and two rank parts a row, with units whose best keys are 62 or
    70 equal blocks: 3968 equal scores are ranked, 4480 are more than a sub-bucket
    may hold (4096), so the rows are computed exactly, as the flag says.  Bit-exact
    to the oracle."""
    rng = np.random.default_rng(k)
    U, G, nb = 34, 4, 375
    n = dev(np.full(U, 64 * nb, np.int64))
    q = rng.standard_normal((U, G, D)).astype(np.float32)
    torch.manual_seed(k)
    K = torch.randn((U, 64 * nb, D), device=DEV) * torch.exp(torch.randn((U, 1, D), device=DEV))
    d, _ = F.fathom_alloc_depths(dev(q), dev(np.ones((U, D), np.float32)), F.FATHOM_WATERFILL, 48)
    for m in (62, 70):
        Km = K.clone()
        Km.view(U, nb, 64, D)[:2, dev(rng.permutation(nb)[:m])] = dev(16 * q[:2].sum(1)).view(2, 1, 1, D)
        planes, scales = F.fathom_pack(Km, n)
        st = F.new_status()
        idx, val = F.fathom_scan_topk(planes, scales, n, dev(q), d, k, dev_status=st, max_unit_bits=48)
        assert status(st) == (F.FATHOM_DEV_TOPK_FALLBACK if 64 * m > 4096 else 0), m
        for u in (0, 1, 2, U - 1):
            ref = oracle.scores_f32(planes[u].cpu().numpy().view(np.uint64), scales[u].cpu().numpy().view(np.uint16),
                                    64 * nb, q[u], d[u].cpu().numpy())
            for h in range(G):
                oi, ov, _ = oracle.topk(ref[h], k, 0, 0)
                assert u > 1 or ov[0] == ov[-1]  # the equal ones fill the top k
                assert np.array_equal(idx[u, h].cpu().numpy(), oi) and np.array_equal(val[u, h].cpu().numpy(), ov), (m, u, h)


@pytest.mark.parametrize("kdt", [np.float32, np.float16])
@pytest.mark.parametrize("U,max_new", [(5, 1), (5, 300), (7, 4000), (90, 1), (20, 300)])
def test_pack_append_blocks(kdt, U, max_new):
    """Appends on both sides of the rule of 96 blocks (a token a lane, or 16): blocks
    of 1, 63 and 64 tokens, keys at the cell boundaries, signed zeros, NaN, infinite
    and tiny keys, padded rows, a unit that does not grow and one whose lengths are
    refused.  Bit-exact to the oracle's pack of the longer prefix; blocks past the
    end and the refused unit stay as they were."""
    rng = np.random.default_rng(U + max_new)
    nb_cap, ld = 70, 136
    n_old = rng.integers(0, 64 * nb_cap - max_new, U)
    n_old[:4] = [128, 191, 127, 40]
    n = n_old + rng.integers(1, max_new + 1, U)
    n[3], n_old[4], n[4] = n_old[3], 100, 99  # no growth; refused
    K = torch.full((U, 64 * nb_cap, ld), float("nan"), dtype=torch.float32 if kdt == np.float32 else torch.float16, device=DEV)
    host = {}
    for u in range(U):
        m = int(max(n[u], n_old[u]))
        if u < 7:
            k = threshold_keys(rng, m, kdt)
            if u < 2:
                k[m - 1, 3], k[m - 2, 4], k[m - 1, 5], k[m - 1, 6] = np.nan, np.inf, -np.inf, -0.0
                k[(m - 1) // 64 * 64:, 7] = 1e-8
            host[u] = k
            K[u, :m, :D] = dev(k)
        else:
            K[u, :m, :D] = torch.randn((m, D), device=DEV).to(K.dtype)
    planes = torch.full((U, D, 4, nb_cap), 0x5A5A5A5A, dtype=torch.int64, device=DEV)
    scales = torch.full((U, D, nb_cap), 0x1234, dtype=torch.int16, device=DEV)
    for u in range(U):  # the store before: packed up to n_old, not zeroed past it
        p, s = F.fathom_pack(K[u:u + 1, :, :D], dev(n_old[u:u + 1].astype(np.int64)), nb_cap=nb_cap)
        b = (int(n_old[u]) + 63) // 64
        planes[u, :, :, :b], scales[u, :, :b] = p[0, :, :, :b], s[0, :, :b]
    before = planes.clone(), scales.clone()
    st = F.new_status()
    F.fathom_pack_append(K[:, :, :D], dev(n_old.astype(np.int64)), dev(n.astype(np.int64)), max_new, planes, scales, dev_status=st)
    assert status(st) == (F.FATHOM_DEV_NONFINITE | F.FATHOM_DEV_SCALE_OVERFLOW | F.FATHOM_DEV_BAD_N)
    assert torch.equal(planes[4], before[0][4]) and torch.equal(scales[4], before[1][4])
    for u in (0, 1, 2, 3) + ((5, 6) if U > 6 else ()):
        b = (int(n[u]) + 63) // 64
        op, os_, _ = oracle.pack(host[u][:n[u]].astype(np.float32), nb_cap=nb_cap)
        assert np.array_equal(planes[u, :, :, :b].cpu().numpy().view(np.uint64), op[:, :, :b]), u
        assert np.array_equal(scales[u, :, :b].cpu().numpy().view(np.uint16), os_[:, :b]), u
        assert torch.equal(planes[u, :, :, b:], before[0][u, :, :, b:]) and torch.equal(scales[u, :, b:], before[1][u, :, b:])


@pytest.mark.parametrize("G", [1, 5])
def test_alloc_depths_nonfinite(G):
    """Importances outside the defined inputs stand above every candidate, infinite
    ones below NaN and those below negative ones (as their bit patterns do): the
    channels above the water line keep 4 planes, and a water line among them is
    infinite or NaN.  Three such channels of each kind, budgets that put the line
    into every group; NONFINITE is raised."""
    rng = np.random.default_rng(G)
    q = rng.standard_normal((1, G, D)).astype(np.float32)
    var = np.exp(rng.standard_normal((1, D))).astype(np.float32)
    neg, nan, inf = [3, 64, 127], [0, 65, 70], [5, 63, 126]
    var[0, neg], var[0, nan], var[0, inf] = -1.0, np.nan, np.inf
    rest = var.copy()
    rest[0, neg + nan + inf] = 0.0
    for B in (0, 11, 12, 23, 24, 35, 36, 60, 511):
        st = F.new_status()
        d, th = F.fathom_alloc_depths(dev(q), dev(var), F.FATHOM_WATERFILL, B, dev_status=st)
        d, th = d.cpu().numpy()[0], float(th.item())
        assert status(st) == F.FATHOM_DEV_NONFINITE
        want = np.zeros(D, np.uint8)
        want[neg] = 4
        if B < 24:
            assert np.isnan(th), B
        elif B < 36:
            want[nan] = 4
            assert th == np.inf, B
        else:
            od, oth, _ = oracle.alloc_waterfill(q[0], rest[0], B - 36)
            want = od.copy()
            want[neg + nan + inf] = 4
            assert th == np.float32(oth), B
        assert np.array_equal(d, want), B
