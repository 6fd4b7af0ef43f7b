"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.

Bars: bit-exact for momentum (float32, stated rounding order), sign packing,
vote, counts and the fused update; PolarNS within 2e-2 relative Frobenius error
of the float32 oracle with >= 99.9 % sign agreement on entries with
|x| > 1e-3 * max|x|.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import signmuon_oracle as O

pytestmark = pytest.mark.gpu

NS_REL_TOL = 2e-2
SIGN_AGREE = 0.999


@pytest.fixture(scope="module")
def P():
    import paper_2605_16311_amd as pkg
    return pkg


@pytest.fixture(scope="module")
def ctx(P):
    c = P.Context()
    yield c
    torch.cuda.synchronize()
    c.close()


# Settings of the context's tuning switches (GEMM tile, grouping of the K steps, storage of the s x s
# matrices) under which the Newton-Schulz and whole-step cases are repeated; "auto" is what a caller gets.
VARIANTS = {
    "auto": dict(),
    "t128-pairs-upper": dict(gemm_tile=128),
    "t256-pairs-upper": dict(gemm_tile=256),
    "t128-pairs-full": dict(gemm_tile=128, ns_store="full"),
    "t256-pairs-full": dict(gemm_tile=256, ns_store="full"),
    "t128-single-upper": dict(gemm_tile=128, ns_path="single"),
    "t256-single-upper": dict(gemm_tile=256, ns_path="single"),
    "t256-single-full": dict(gemm_tile=256, ns_path="single", ns_store="full"),
    "t128-stepwise": dict(gemm_tile=128, ns_path="stepwise"),
    "t256-stepwise": dict(gemm_tile=256, ns_path="stepwise"),
}


@pytest.fixture(scope="module", params=list(VARIANTS))
def vctx(P, request):
    c = P.Context(**VARIANTS[request.param])
    yield c
    torch.cuda.synchronize()
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bf16_dev(a_f32):
    return dev(np.asarray(a_f32, np.float32)).bfloat16()


def bf16_host(t):
    return t.float().cpu().numpy()


def ns_check(got, ref, what=""):
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    rel = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30)
    big = np.abs(ref) > 1e-3 * np.max(np.abs(ref))
    agree = np.mean((got[big] >= 0) == (ref[big] >= 0)) if big.any() else 1.0
    assert rel <= NS_REL_TOL, f"{what}: rel Frobenius {rel:.3e}"
    assert agree >= SIGN_AGREE, f"{what}: sign agreement {agree:.5f}"
    return rel, agree


# ------------------------------------------------------------------ a1
@pytest.mark.parametrize("M,r,c,wd", [(4, 256, 256, 0.0), (3, 37, 53, 0.0), (2, 64, 576, 0.1),
                                      (5, 129, 100, 0.05), (1, 1, 1, 0.0), (2, 1000, 2048, 0.0)])
def test_momentum_bit_exact(P, ctx, M, r, c, wd):
    g = wl.worker_grads("single256", 0, r, c, M=M)
    m0 = wl.normal((M, r, c), stream=21)
    w = wl.weights(r, c)
    ref = O.momentum_update(m0, g, w, 0.9, wd, dtype=np.float32)
    mom, x = dev(m0), torch.empty((M, r, c), dtype=torch.bfloat16, device="cuda")
    ss = torch.empty(M, dtype=torch.float32, device="cuda")
    P.signmuon_momentum(ctx, mom, dev(g), dev(w) if wd else None, 0.9, wd, x_bf16=x, sumsq=ss)
    got = mom.cpu().numpy()
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
    assert np.array_equal(bf16_host(x), wl.from_bf16_bits(wl.to_bf16_bits(ref)))
    ss_ref = np.sum(ref.astype(np.float64) ** 2, axis=(1, 2))
    assert np.allclose(ss.cpu().numpy(), ss_ref, rtol=1e-5)
    # second step from the new state, no side outputs
    ref2 = O.momentum_update(ref, g, w, 0.9, wd, dtype=np.float32)
    P.signmuon_momentum(ctx, mom, dev(g), dev(w) if wd else None, 0.9, wd)
    assert np.array_equal(mom.cpu().numpy().view(np.uint32), ref2.view(np.uint32))


@pytest.mark.parametrize("chunks", [1, 1023, 1024, 1025, 8191, 8192, 8193])
def test_momentum_sums_of_squares(P, ctx, chunks):
    """Edges of the sum over a worker's partial sums (of 1024 entries): 1024 threads, eight loads each at a time."""
    M, n = 2, 1024 * chunks - 3
    mom = torch.randn((M, 1, n), generator=torch.Generator("cuda").manual_seed(chunks), device="cuda")
    ss = torch.empty(M, dtype=torch.float32, device="cuda")
    P.signmuon_momentum(ctx, mom, torch.zeros_like(mom), None, 0.9, 0.0, sumsq=ss)
    ref = mom.cpu().numpy().astype(np.float64) ** 2
    # positive terms: at most 37 roundings of 2^-24 lie between an entry and the sum (partial 11, thread 16, trees 10)
    assert np.allclose(ss.cpu().numpy(), ref.sum(axis=(1, 2)), rtol=37 * 2.0 ** -24, atol=0)


# ------------------------------------------------------------------ a5
@pytest.mark.parametrize("n", [1, 7, 8, 63, 64, 65, 1000, 4096, 65536 + 13, 300001])
@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_sign_pack_bit_exact(P, ctx, n, dt):
    batch = 3
    x = wl.normal((batch, n), stream=22, block=n)
    sv = wl.special_values_f32()
    x[0, : min(n, sv.size)] = sv[: min(n, sv.size)]
    x[1, ::3] = 0.0
    x[2, 1::5] = -0.0
    if dt == "bf16":
        xb = wl.from_bf16_bits(wl.to_bf16_bits(x))
        u = dev(wl.to_bf16_bits(x).view(np.int16)).view(torch.bfloat16)
    else:
        xb, u = x, dev(x)
    stride = O.packed_stride_bytes(n)
    out = torch.full((batch, stride + 8), 0xAA, dtype=torch.uint8, device="cuda")
    P.signmuon_sign_pack(ctx, u, "1bit", out)
    got = out.cpu().numpy()
    for b in range(batch):
        assert np.array_equal(got[b, :stride], O.pack_bits(O.sign_entries(xb[b]))), (n, dt, b)
        assert np.all(got[b, stride:] == 0xAA)          # nothing written past the row
    o8 = torch.full((batch, n + 5), 7, dtype=torch.int8, device="cuda")
    P.signmuon_sign_pack(ctx, u, "int8", o8)
    g8 = o8.cpu().numpy()
    for b in range(batch):
        assert np.array_equal(g8[b, :n], O.signs_pm1(xb[b]))
        assert np.all(g8[b, n:] == 7)


def test_sign_pack_empty_and_errors(P, ctx):
    u = torch.empty((2, 0), dtype=torch.float32, device="cuda")
    out = torch.zeros((2, 8), dtype=torch.uint8, device="cuda")
    P.signmuon_sign_pack(ctx, u, "1bit", out)
    u = torch.zeros((1, 100), dtype=torch.float32, device="cuda")
    with pytest.raises(P.SignMuonError):
        P.signmuon_sign_pack(ctx, u, "1bit", torch.zeros((1, 8), dtype=torch.uint8, device="cuda"))
    with pytest.raises(P.SignMuonError):
        P.signmuon_sign_pack(ctx, u, "int8", torch.zeros((1, 50), dtype=torch.int8, device="cuda"))


# ------------------------------------------------------------------ a6 (+ a8)
@pytest.mark.parametrize("M", [1, 2, 3, 4, 8, 16, 33, 300])
@pytest.mark.parametrize("n", [1, 5, 64, 100, 4099, 70001])
def test_vote_bit_exact(P, ctx, M, n):
    rng = wl.rng_for(23, block=M, worker=n)
    S = rng.choice(np.array([-1, 1], np.int8), size=(M, n), p=[0.45, 0.55])
    S[:, : min(n, 4)] = 1
    if M % 2 == 0 and n > 8:
        S[: M // 2, 5] = 1
        S[M // 2:, 5] = -1                                    # a forced tie
    packed = np.stack([O.pack_bits((S[p] > 0).astype(np.uint8)) for p in range(M)])
    stride = packed.shape[1]
    vote_ref, tot_ref = O.majority_vote_int8(S)
    vote1_ref, c_ref = O.majority_vote_bits(packed, M, n)
    assert np.array_equal(vote_ref, vote1_ref)
    w0 = wl.normal((n,), stream=24, block=n)
    lr = 0.01
    w_ref = O.apply_update(w0.reshape(1, n), vote_ref.reshape(1, n), lr, dtype=np.float32).reshape(n)
    for fmt, signs, counts_ref, sb in (("1bit", packed, c_ref, stride), ("int8", S, tot_ref, n)):
        d_signs = dev(signs)
        # voted bits
        vb = torch.full((stride + 8,), 0x55, dtype=torch.uint8, device="cuda")
        P.signmuon_majority_vote(ctx, d_signs, fmt, M, n, sb, voted=vb, vfmt="bits")
        g = vb.cpu().numpy()
        assert np.array_equal(g[:stride], O.pack_bits((vote_ref > 0).astype(np.uint8))), (fmt, M, n)
        assert np.all(g[stride:] == 0x55)
        # expanded formats + counts + fused update, one call each
        cnt = torch.full((n + 4,), -7, dtype=torch.int32, device="cuda")
        w = dev(np.concatenate([w0, np.full(4, 3.0, np.float32)]))
        v8 = torch.full((n + 4,), 9, dtype=torch.int8, device="cuda")
        P.signmuon_majority_vote(ctx, d_signs, fmt, M, n, sb, voted=v8, vfmt="int8", counts=cnt, w=w, lr_scaled=lr)
        assert np.array_equal(v8.cpu().numpy()[:n], vote_ref) and np.all(v8.cpu().numpy()[n:] == 9)
        assert np.array_equal(cnt.cpu().numpy()[:n], counts_ref) and np.all(cnt.cpu().numpy()[n:] == -7)
        gw = w.cpu().numpy()
        assert np.array_equal(gw[:n].view(np.uint32), w_ref.view(np.uint32)) and np.all(gw[n:] == 3.0)
        vb16 = torch.zeros((n + 4,), dtype=torch.bfloat16, device="cuda")
        P.signmuon_majority_vote(ctx, d_signs, fmt, M, n, sb, voted=vb16, vfmt="bf16")
        assert np.array_equal(bf16_host(vb16)[:n], vote_ref.astype(np.float32)) and np.all(bf16_host(vb16)[n:] == 0)
        vf = torch.zeros((n + 4,), dtype=torch.float32, device="cuda")
        P.signmuon_majority_vote(ctx, d_signs, fmt, M, n, sb, voted=vf, vfmt="f32")
        assert np.array_equal(vf.cpu().numpy()[:n], vote_ref.astype(np.float32)) and np.all(vf.cpu().numpy()[n:] == 0)


@pytest.mark.parametrize("M", [1, 2, 3, 7, 8, 31, 32, 100, 255, 256])
@pytest.mark.parametrize("n", [32, 64 * 37, 32 * 2049, 256 * 300 + 32])
def test_vote_word_aligned_without_counts(P, ctx, M, n):
    """n % 32 == 0, no counts: the form the step uses (bit-sliced counting, one thread per 32-bit word);
    voted bf16 and the fused update in one call, against the scalar definition (eq. mv_def)."""
    rng = wl.rng_for(27, block=M, worker=n)
    S = rng.choice(np.array([-1, 1], np.int8), size=(M, n), p=[0.5, 0.5])
    if M % 2 == 0:
        S[: M // 2, 3::17] = 1
        S[M // 2:, 3::17] = -1                                # forced ties -> +1
    packed = np.stack([O.pack_bits((S[p] > 0).astype(np.uint8)) for p in range(M)])
    stride = packed.shape[1]
    vote_ref, _ = O.majority_vote_int8(S)
    w0 = wl.normal((n,), stream=28, block=n)
    lr = 0.0625
    w_ref = O.apply_update(w0.reshape(1, n), vote_ref.reshape(1, n), lr, dtype=np.float32).reshape(n)
    w = dev(np.concatenate([w0, np.full(8, 3.0, np.float32)]))
    vb16 = torch.full((n + 8,), 5.0, dtype=torch.bfloat16, device="cuda")
    P.signmuon_majority_vote(ctx, dev(packed), "1bit", M, n, stride, voted=vb16, vfmt="bf16", w=w, lr_scaled=lr)
    gv = bf16_host(vb16)
    assert np.array_equal(gv[:n], vote_ref.astype(np.float32)) and np.all(gv[n:] == 5.0), (M, n)
    gw = w.cpu().numpy()
    assert np.array_equal(gw[:n].view(np.uint32), w_ref.view(np.uint32)) and np.all(gw[n:] == 3.0), (M, n)


@pytest.mark.parametrize("M", [1, 2, 16, 127, 300])
@pytest.mark.parametrize("n", [16, 4096, 65536 + 16])
def test_vote_int8_sixteen_entry_groups(P, ctx, M, n):
    """int8 signs with n % 16 == 0 and aligned rows (one thread per 16 entries): int32 sums, voted int8 and
    bf16, fused update, against the scalar definition; sums beyond the int8 range at M = 300."""
    rng = wl.rng_for(30, block=M, worker=n)
    S = rng.choice(np.array([-1, 1], np.int8), size=(M, n), p=[0.5, 0.5])
    if M % 2 == 0:
        S[: M // 2, 1::13] = 1
        S[M // 2:, 1::13] = -1                                # forced ties -> +1
    S[:, 0] = 1                                               # sum = M (overflows int8 at M = 300)
    vote_ref, tot_ref = O.majority_vote_int8(S)
    w0 = wl.normal((n,), stream=31, block=n)
    lr = 0.03125
    w_ref = O.apply_update(w0.reshape(1, n), vote_ref.reshape(1, n), lr, dtype=np.float32).reshape(n)
    d_signs = dev(S)
    cnt = torch.full((n + 16,), -7, dtype=torch.int32, device="cuda")
    w = dev(np.concatenate([w0, np.full(16, 3.0, np.float32)]))
    v8 = torch.full((n + 16,), 9, dtype=torch.int8, device="cuda")
    P.signmuon_majority_vote(ctx, d_signs, "int8", M, n, n, voted=v8, vfmt="int8", counts=cnt, w=w, lr_scaled=lr)
    assert np.array_equal(v8.cpu().numpy()[:n], vote_ref) and np.all(v8.cpu().numpy()[n:] == 9)
    assert np.array_equal(cnt.cpu().numpy()[:n], tot_ref) and np.all(cnt.cpu().numpy()[n:] == -7)
    gw = w.cpu().numpy()
    assert np.array_equal(gw[:n].view(np.uint32), w_ref.view(np.uint32)) and np.all(gw[n:] == 3.0)
    vb16 = torch.full((n + 16,), 5.0, dtype=torch.bfloat16, device="cuda")
    P.signmuon_majority_vote(ctx, d_signs, "int8", M, n, n, voted=vb16, vfmt="bf16")
    gv = bf16_host(vb16)
    assert np.array_equal(gv[:n], vote_ref.astype(np.float32)) and np.all(gv[n:] == 5.0)


@pytest.mark.parametrize("M", [1, 7, 8, 9, 20])
@pytest.mark.parametrize("n", [15, 17, 1023, 1024, 1041, 4095, 4097, 8200])
def test_vote_int8_runs_of_a_wave(P, ctx, M, n):
    """int8 values of the whole range in rows that start anywhere, around the 16 entries of a lane, the 1024 of a wave
    and the 4096 of a workgroup, and around groups of eight workers: sums, votes and update in one call and alone."""
    rng = wl.rng_for(65, block=M, worker=n)
    S = rng.integers(-128, 128, size=(M, n + 3), dtype=np.int8)
    tot = S[:, :n].astype(np.int32).sum(axis=0)
    vote = np.where(tot >= 0, 1, -1)
    w0, lr = wl.normal((n,), stream=66, block=n), 0.03125
    w_ref = O.apply_update(w0.reshape(1, n), vote.reshape(1, n), lr, dtype=np.float32).reshape(n)
    base = dev(np.concatenate([np.zeros(1, np.int8), S.reshape(-1)]))
    signs = base[1:]                                          # one byte past an aligned address
    for voted in (None, "int8", "bf16", "f32"):
        cnt = torch.full((n + 4,), -7, dtype=torch.int32, device="cuda")
        w = dev(np.concatenate([w0, np.full(4, 3.0, np.float32)]))
        v = None if voted is None else torch.full((n + 4,), 9, device="cuda", dtype=dict(
            int8=torch.int8, bf16=torch.bfloat16, f32=torch.float32)[voted])
        P.signmuon_majority_vote(ctx, signs, "int8", M, n, n + 3, voted=v, vfmt=voted or "bits", counts=cnt, w=w, lr_scaled=lr)
        assert np.array_equal(cnt.cpu().numpy()[:n], tot) and np.all(cnt.cpu().numpy()[n:] == -7)
        gw = w.cpu().numpy()
        assert np.array_equal(gw[:n].view(np.uint32), w_ref.view(np.uint32)) and np.all(gw[n:] == 3.0)
        if v is not None:
            gv = v.float().cpu().numpy()
            assert np.array_equal(gv[:n], vote.astype(np.float32)) and np.all(gv[n:] == 9.0)


ONE_ROUND = 1 << 21    # entries: the line between the vote kernels on a card of 256 compute units


@pytest.mark.parametrize("fmt", ["1bit", "int8"])
@pytest.mark.parametrize("M,n", [(1, ONE_ROUND), (1, ONE_ROUND + 1), (4, ONE_ROUND + 1039), (7, ONE_ROUND + 4094), (8, ONE_ROUND + 33), (9, ONE_ROUND), (9, ONE_ROUND + 1),
                                 (12, ONE_ROUND + 1039), (9, 2 * ONE_ROUND + 8), (16, 2 * ONE_ROUND - 16), (16, 2 * ONE_ROUND), (17, 2 * ONE_ROUND + 8), (31, ONE_ROUND + 15), (32, ONE_ROUND + 17),
                                 (248, 70), (249, 3), (500, 1)])
def test_vote_on_both_sides_of_the_lines_between_its_kernels(P, ctx, fmt, M, n):
    """Launches of up to one round of waves and beyond, with and without counts, up to 7 workers, 8 int8 and 31 1-bit ones
    and more, ends of the buffer at any place in a lane's entries: every format of the votes, sums and update."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * 31 + n)
    S = torch.randint(0, 2, (M, n), generator=gen, device="cuda", dtype=torch.int8)
    w0 = torch.randn((n,), generator=gen, device="cuda")
    sums = S.sum(0, dtype=torch.int32)
    vote = torch.where(2 * sums >= M, 1.0, -1.0)
    if fmt == "1bit":
        stride = O.packed_stride_bytes(n)
        bits = torch.zeros((M, 8 * stride), dtype=torch.uint8, device="cuda")
        bits[:, :n] = S.view(torch.uint8)
        place = (2 ** torch.arange(8, device="cuda")).to(torch.uint8)
        signs = (bits.view(M, stride, 8) * place).sum(-1, dtype=torch.uint8).contiguous()
    else:
        stride, signs, sums = n, 2 * S - 1, 2 * sums - M
    lr = 2.0 ** -6
    w_ref = w0 - lr * vote                                    # lr * vote is exact: one rounding, as in the kernels
    for counts, update in ((False, False), (True, False), (False, True), (True, True)):
        for vfmt, dt in ((None, None), ("int8", torch.int8), ("bf16", torch.bfloat16), ("f32", torch.float32)):
            if not (counts or update or vfmt):
                continue
            cnt = torch.full((n + 4,), -7, dtype=torch.int32, device="cuda") if counts else None
            w = torch.cat([w0, torch.full((4,), 3.0, device="cuda")]) if update else None
            v = torch.full((n + 4,), 9, dtype=dt, device="cuda") if vfmt else None
            P.signmuon_majority_vote(ctx, signs, fmt, M, n, stride, voted=v, vfmt=vfmt or "bits", counts=cnt, w=w, lr_scaled=lr)
            what = (fmt, M, n, counts, update, vfmt)
            if counts:
                assert torch.equal(cnt[:n], sums) and bool((cnt[n:] == -7).all()), what
            if update:
                assert torch.equal(w[:n], w_ref) and bool((w[n:] == 3.0).all()), what
            if vfmt:
                assert torch.equal(v[:n].float(), vote) and bool((v[n:] == 9).all()), what


@pytest.mark.parametrize("M", [255, 256, 257, 263, 264, 511, 513, 1031])
@pytest.mark.parametrize("n", [1, 129, 64 * 37])
def test_vote_bits_of_many_workers(P, ctx, M, n):
    """Voted bits by carry-save addition of eight words (256 workers and more), every remainder of eight, counts around the
    threshold and around powers of two."""
    rng = wl.rng_for(71, block=M, worker=n)
    S = rng.integers(0, 2, size=(M, n), dtype=np.uint8)
    half = (M + 1) // 2
    for i, k in enumerate([half, half - 1, 0, M, 128, 255, 256 if M > 255 else 254]):
        if i < n:                                             # exactly k of M set in entry i
            S[:, i] = 0
            S[rng.permutation(M)[:min(k, M)], i] = 1
    packed = np.stack([O.pack_bits(S[p]) for p in range(M)])
    ref = O.pack_bits((2 * S.astype(np.int64).sum(axis=0) >= M).astype(np.uint8))
    vb = torch.full((packed.shape[1] + 8,), 0x55, dtype=torch.uint8, device="cuda")
    P.signmuon_majority_vote(ctx, dev(packed), "1bit", M, n, packed.shape[1], voted=vb, vfmt="bits")
    got = vb.cpu().numpy()
    assert np.array_equal(got[:-8], ref) and np.all(got[-8:] == 0x55)


@pytest.mark.parametrize("sign_fmt", ["1bit", "int8"])
@pytest.mark.parametrize("M,Kp", [(9, 0), (3, 0), (9, 1)])
def test_step_votes_beyond_one_round_over_padded_rows(P, ctx, sign_fmt, M, Kp):
    """More entries in a step's vote than one round of the kernel of four entries per lane: rows of odd length, a whole
    row's matrix and a tiny one in the launch, votes into padded rows (Kp) and flat ones."""
    run_step_case(P, ctx, [(1100, 1999), (64, 128), (5, 1)], M, sign_fmt=sign_fmt, Kp=Kp, K=0, check_ns_blocks=())


@pytest.mark.parametrize("snr", [0.25, 1.0])
def test_majority_vote_sign_error_falls_like_inverse_sqrt_m(P, ctx, snr):
    """Lemma "Majority vote improves sign reliability": with M independent workers whose gradient entries are
    g + sigma z (symmetric unimodal noise), the vote's sign-error rate is at most sigma / (sqrt(M) |g|).  The
    library's pack + vote on synthetic entries: the measured rate matches the exact binomial value (ties -> +1),
    obeys the bound and falls with M."""
    from scipy import stats
    n = 1 << 20
    g = np.where(np.arange(n) % 2 == 0, snr, -snr).astype(np.float32)      # sigma = 1
    prev = 1.0
    p1 = float(stats.norm.cdf(-snr))                                       # one worker's failure probability
    for M in (1, 4, 16, 64):
        z = wl.normal((M, n), stream=32, block=M, worker=int(snr * 100))
        u = dev((g[None, :] + z).astype(np.float32))
        stride = O.packed_stride_bytes(n)
        bits = torch.zeros((M, stride), dtype=torch.uint8, device="cuda")
        P.signmuon_sign_pack(ctx, u, "1bit", bits)
        v8 = torch.zeros((n,), dtype=torch.int8, device="cuda")
        P.signmuon_majority_vote(ctx, bits, "1bit", M, n, stride, voted=v8, vfmt="int8")
        vote = v8.cpu().numpy()
        fail = float(np.mean(vote != np.sign(g)))
        # exact: entries with g > 0 fail iff fewer than M/2 workers are right; with g < 0 a tie also fails
        k = np.arange(M + 1)
        pmf = stats.binom.pmf(k, M, 1.0 - p1)                              # number of correct workers
        q_pos = pmf[2 * k < M].sum()
        q_neg = pmf[2 * k <= M].sum()
        q = 0.5 * (q_pos + q_neg)
        assert abs(fail - q) <= 5.0 * np.sqrt(q * (1 - q) / n) + 1e-6, (M, fail, q)
        assert fail <= 1.0 / (np.sqrt(M) * snr) + 1e-3, (M, fail)
        assert fail < prev or M == 1
        prev = fail


def test_vote_ignores_garbage_tail_bits_and_dropped_worker(P, ctx):
    M, n = 5, 70
    rng = wl.rng_for(25)
    S = rng.choice(np.array([-1, 1], np.int8), size=(M, n))
    packed = np.stack([O.pack_bits((S[p] > 0).astype(np.uint8)) for p in range(M)])
    ref, _ = O.majority_vote_int8(S)
    dirty = packed.copy()
    dirty[:, n // 8] |= np.uint8(0xFF << (n % 8) & 0xFF)      # set padding bits in every worker
    dirty[:, n // 8 + 1:] = 0xFF
    vb = torch.zeros((16,), dtype=torch.uint8, device="cuda")
    P.signmuon_majority_vote(ctx, dev(dirty), "1bit", M, n, 16, voted=vb, vfmt="bits")
    assert np.array_equal(vb.cpu().numpy(), O.pack_bits((ref > 0).astype(np.uint8)))
    # a dropped worker: vote over the first M-1 rows only
    ref4, _ = O.majority_vote_int8(S[:4])
    P.signmuon_majority_vote(ctx, dev(packed), "1bit", 4, n, 16, voted=vb, vfmt="bits")
    assert np.array_equal(vb.cpu().numpy(), O.pack_bits((ref4 > 0).astype(np.uint8)))


# ------------------------------------------------------------------ a2-a4
NS_CASES = [
    # (batch, rows, cols, steps, scale, coeffs)
    (4, 256, 256, 5, "fro", O.PAPER_COEFFS),
    (2, 64, 576, 5, "fro", O.PAPER_COEFFS),
    (2, 576, 64, 5, "fro", O.PAPER_COEFFS),
    (3, 128, 320, 3, "fro", O.PAPER_COEFFS),
    (2, 200, 136, 5, "fro", O.PAPER_COEFFS),        # padding in both dimensions, tall
    (2, 100, 333, 4, "fro", O.PAPER_COEFFS),        # padding, wide, odd sizes
    (1, 512, 1152, 5, "fro", O.PAPER_COEFFS),
    (2, 256, 256, 1, "fro", O.PAPER_COEFFS),
    (2, 192, 448, 0, "fro", O.PAPER_COEFFS),        # K = 0: only the scaling
    (2, 256, 384, 5, "spectral", O.PAPER_COEFFS),
    (2, 384, 256, 5, "spectral", O.PAPER_COEFFS),
    (2, 128, 128, 4, "none", O.PAPER_COEFFS),
    (2, 192, 320, 3, "fro", (2.0, -1.5, 0.5)),      # quintic polynomial (step-by-step form)
    (2, 192, 320, 4, "fro", (1.6, -0.6, 0.0)),      # cubic with a > 3/2 (step-by-step form)
    (2, 256, 640, 2, "fro", O.PAPER_COEFFS),        # shortest short-side recurrence
    (2, 320, 192, 7, "fro", O.PAPER_COEFFS),        # two segments (5 + 2), tall
    (2, 256, 640, 10, "fro", O.PAPER_COEFFS),       # two full segments, wide
    (1, 512, 512, 10, "spectral", O.PAPER_COEFFS),  # square, near convergence
    (2, 136, 200, 6, "fro", O.PAPER_COEFFS),        # padding + two segments (5 + 1)
    (2, 192, 448, 8, "fro", O.PAPER_COEFFS),        # segments 5 + 3: two steps at a time, then one
    (2, 448, 192, 9, "fro", O.PAPER_COEFFS),        # segments 5 + 4: two pairs, tall
    (2, 256, 384, 5, "fro", (1.25, -0.4, 0.0)),     # another cubic on the short-side recurrence
    (2, 256, 384, 4, "none", (1.4, -0.45, 0.0)),
    (2, 320, 512, 5, "fro", O.PAPER_COEFFS),        # short side 320: a whole and a partial 256-block
    (1, 640, 576, 5, "fro", O.PAPER_COEFFS),        # short side 576 (tall): three blocks, the last partial
    (1, 640, 640, 4, "fro", O.PAPER_COEFFS),        # square, 2.5 blocks
]


@pytest.mark.parametrize("batch,r,c,steps,scale,coeffs", NS_CASES)
@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_polar_ns_against_fp32_oracle(P, vctx, batch, r, c, steps, scale, coeffs, dt):
    ctx = vctx
    x = wl.normal((batch, r, c), stream=26, block=r, worker=c)
    if scale == "none":
        x = x / (1.05 * np.linalg.norm(x, ord=2, axis=(1, 2), keepdims=True)).astype(np.float32)
    v0 = wl.start_vectors(batch, c, block=r)
    if dt == "bf16":
        xin = wl.from_bf16_bits(wl.to_bf16_bits(x))
        xd = dev(wl.to_bf16_bits(x).view(np.int16)).view(torch.bfloat16)
    else:
        xin, xd = x, dev(x)
    P.signmuon_polar_ns(ctx, xd, steps, coeffs=coeffs, scale=scale, power_iters=2, eps=1e-12,
                        v0=dev(v0) if scale == "spectral" else None)
    got = xd.float().cpu().numpy()
    for b in range(batch):
        ref = O.polar_ns(xin[b], steps, coeffs, scale, 2, 1e-12, v0[b], dtype=np.float32)
        ns_check(got[b], ref, f"{(batch, r, c, steps, scale, dt)} item {b}")


@pytest.mark.parametrize("batch,r,c", [(1, 1, 1), (3, 60, 70), (2, 200, 65), (2, 128, 300), (40, 129, 150), (41, 256, 192),
                                       (40, 250, 256)])
@pytest.mark.parametrize("steps", [2, 3, 4, 5, 7])
def test_polar_ns_one_workgroup_per_matrix(P, ctx, batch, r, c, steps):
    """Small matrices, whose products of a segment run in one launch: every length of a segment, short sides at and
    around the sizes of its two kernels (128, 256) and of its 32-blocks."""
    x = wl.normal((batch, r, c), stream=61, block=r, worker=steps)
    xd = dev(x)
    P.signmuon_polar_ns(ctx, xd, steps)
    got = xd.cpu().numpy()
    for b in (0, batch - 1):
        ref = O.polar_ns(x[b], steps, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32)
        ns_check(got[b], ref, f"{(batch, r, c, steps)} item {b}")


@pytest.mark.parametrize("batch,r,c,s,l", [(3, 100, 150, 128, 192), (41, 250, 200, 256, 256)])
@pytest.mark.parametrize("steps,products", [(2, 2), (3, 5), (4, 7), (5, 10), (8, 15)])
def test_work_booked_for_products_in_one_launch(P, batch, r, c, s, l, steps, products):
    """signmuon_profile_work beside the times of a set that runs on chip (s, l: the padded sides): per product the
    32 x 32 blocks on and above the diagonal, clipped to the matrix; per segment A_0 read and P written once; a Gram
    launch writes A_0 as packed blocks."""
    from paper_2605_16311_amd import binding as B
    segments, su = (steps + 4) // 5, min(r, c)
    ctx = P.Context()
    x = dev(wl.normal((batch, r, c), stream=64, block=r, worker=c))
    P.signmuon_polar_ns(ctx, x, steps)
    ctx.profile_enable(1 << B.SM_K_NS_SMALL | 1 << B.SM_K_NS_GRAM)
    ctx.profile_reset()
    P.signmuon_polar_ns(ctx, x, steps)
    (small_n, small_ms), (gram_n, _) = ctx.profile_read(B.SM_K_NS_SMALL), ctx.profile_read(B.SM_K_NS_GRAM)
    small, gram = ctx.profile_work(B.SM_K_NS_SMALL), ctx.profile_work(B.SM_K_NS_GRAM)
    ctx.close()
    side = [min(32, su - b) for b in range(0, su, 32)]
    area = sum(side[i] * side[j] for j in range(len(side)) for i in range(j + 1))
    packed = s * (s + 32) // 2
    assert small_n == gram_n == segments and small_ms > 0
    assert small == (batch * products * 2.0 * area * su, batch * products * 2.0 * s ** 3,
                     batch * segments * 2.0 * (packed + s * s))
    assert gram[2] == batch * segments * 2.0 * (s * l + packed)


@pytest.mark.parametrize("ns_path", ["pairs", "stepwise"])
@pytest.mark.parametrize("r,c", [(64, 64), (100, 333), (333, 100), (448, 192), (192, 448)])
def test_polar_ns_with_tiles_of_64(P, ns_path, r, c):
    x = wl.normal((2, r, c), stream=62, block=r, worker=c)
    xd = dev(x)
    cc = P.Context(gemm_tile=64, ns_path=ns_path)
    P.signmuon_polar_ns(cc, xd, 5)
    got = xd.cpu().numpy()
    cc.close()
    for b in range(2):
        ref = O.polar_ns(x[b], 5, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32)
        ns_check(got[b], ref, f"{(r, c, ns_path)} item {b}")


@pytest.mark.parametrize("opts", [dict(ns_store="full"), dict(ns_path="single", ns_store="full"), dict(gemm_tile=64, ns_path="single")])
@pytest.mark.parametrize("steps", [2, 3, 5])
@pytest.mark.parametrize("batch,s", [(1, 64), (2, 128), (1, 180), (1, 256), (3, 320), (40, 330), (1, 576)])
def test_polar_ns_products_of_few_tiles(P, opts, steps, batch, s):
    """Products in a ring of LDS stages, one to nine slices of K (fewer than there are stages, and every remainder by three
    and four), with every kind of added term; 40 of 330: the three-stage ring.  Both sides of the matrix."""
    for r, c in ((s, s + 70), (s + 70, s)):
        x = wl.normal((batch, r, c), stream=64, block=r, worker=c)
        xd = dev(x)
        ctx = P.Context(**opts)
        P.signmuon_polar_ns(ctx, xd, steps)
        ctx.close()
        got = xd.cpu().numpy()
        for b in {0, batch - 1}:
            ns_check(got[b], O.polar_ns(x[b], steps, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32),
                     f"{(batch, r, c, steps, opts)} item {b}")


@pytest.mark.parametrize("steps", [1, 4, 5])
@pytest.mark.parametrize("batch,s,l", [(36, 384, 384), (37, 384, 384), (13, 640, 640), (14, 640, 640), (12, 641, 641), (24, 300, 650)])
def test_polar_ns_around_one_round_of_short_tiles(P, ctx, batch, s, l, steps):
    """Both sides of the lines between tiles of 64 and 128: all tiles of 64 in one round, ten slices of K and eleven."""
    x = wl.normal((batch, s, l), stream=67, block=s, worker=l)
    xd = dev(x)
    P.signmuon_polar_ns(ctx, xd, steps)
    got = xd.cpu().numpy()
    for b in (0, batch - 1):
        ns_check(got[b], O.polar_ns(x[b], steps, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32), f"{(batch, s, l)} item {b}")


@pytest.mark.parametrize("opts", [dict(gemm_tile=128), dict(gemm_tile=256), dict(gemm_tile=256, ns_store="full"),
                                  dict(gemm_tile=128, ns_path="stepwise")])
@pytest.mark.parametrize("r,c", [(1152, 1408), (1408, 1152)])
@pytest.mark.parametrize("batch", [2, 6])
def test_polar_ns_on_grids_of_several_tile_bands(P, opts, r, c, batch):
    """The GEMM kernels list a matrix's tiles in bands of 4 (256-wide tiles) or 8 (128-wide) tile rows.  A short
    side of 1152 is 4.5 and 9 tiles: the symmetric products and the apply run over a full band and a ragged
    one, in both operand orientations.  The symmetric launches of two matrices have 90 tiles of 128, one round of a
    card of 256 compute units: three LDS stages, whole s x s matrices; those of six have 270: two stages, of the s x s
    matrices the blocks on and above the diagonal.  256-wide tiles have two stages either way."""
    ctx = P.Context(**opts)
    x = wl.normal((batch, r, c), stream=27, block=r, worker=c)
    xd = dev(wl.to_bf16_bits(x).view(np.int16)).view(torch.bfloat16)
    xin = wl.from_bf16_bits(wl.to_bf16_bits(x))
    P.signmuon_polar_ns(ctx, xd, 5, scale="fro")
    got = xd.float().cpu().numpy()
    for b in (0, batch - 1):
        ns_check(got[b], O.polar_ns(xin[b], 5, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32),
                 f"{(batch, r, c, opts)} item {b}")
    torch.cuda.synchronize()
    ctx.close()


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("steps", [1, 5, 6])
@pytest.mark.parametrize("batch,r,c,off", [(2, 100, 72, 0), (1, 72, 100, 0), (3, 130, 136, 0), (3, 130, 136, 2), (2, 1, 8, 0), (9, 700, 648, 0)])
def test_polar_ns_writes_the_callers_matrix_alone(P, ctx, batch, r, c, off, steps, dt):
    """Rows of whole 16-byte pieces, which the last apply writes itself (one to three tiles of either size), and rows or
    starts that are not: the same result, and nothing before or behind the matrices."""
    n = batch * r * c
    x = dev(wl.normal((batch, r, c), stream=65, block=r, worker=c))
    buf = torch.full((n + 96,), 7.0, device="cuda", dtype=dt)
    buf[32 + off:32 + off + n] = x.flatten().to(dt)
    xin = buf[32 + off:32 + off + n].clone()
    P.signmuon_polar_ns(ctx, buf[32 + off:32 + off + n].view(batch, r, c), steps)
    assert bool((buf[:32 + off] == 7).all()) and bool((buf[32 + off + n:] == 7).all())
    got = buf[32 + off:32 + off + n].float().cpu().numpy().reshape(batch, r, c)
    xin = xin.float().cpu().numpy().reshape(batch, r, c)
    for b in {0, batch - 1}:
        ns_check(got[b], O.polar_ns(xin[b], steps, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32), f"item {b}")


def test_polar_ns_zero_matrix_and_errors(P, ctx):
    x = torch.zeros((2, 64, 128), dtype=torch.float32, device="cuda")
    P.signmuon_polar_ns(ctx, x, 5)
    assert torch.all(x == 0) and not torch.isnan(x).any()
    with pytest.raises(P.SignMuonError):
        P.signmuon_polar_ns(ctx, x, 5, scale="spectral")          # no v0
    with pytest.raises(P.SignMuonError):
        P.signmuon_polar_ns(ctx, x, -1)


# ------------------------------------------------------------------ whole step
def run_step_case(P, ctx, shapes, M, *, sign_fmt, Kp, K=5, scale="fro", wd=0.0, rsqrt=False, stream=31,
                  grads=None, check_ns_blocks=None):
    n = len(shapes)
    lr, beta = 1e-3, 0.9
    W0 = [wl.weights(r, c, block=i, stream=stream) for i, (r, c) in enumerate(shapes)]
    G = grads or [wl.normal((M, r, c), stream=stream, block=i, worker=7) for i, (r, c) in enumerate(shapes)]
    M0 = [0.1 * wl.normal((M, r, c), stream=stream, block=i, worker=8) for i, (r, c) in enumerate(shapes)]
    V0 = [wl.start_vectors(M, c, block=i, stream=stream) for i, (r, c) in enumerate(shapes)]
    w = [dev(a) for a in W0]
    mom = [dev(a) for a in M0]
    grad = [dev(a) for a in G]
    v0 = [dev(a) for a in V0] if scale == "spectral" else None
    d = [r * c for r, c in shapes]
    sstride = [O.packed_stride_bytes(x) if sign_fmt == "1bit" else x for x in d]
    signs = [torch.zeros((M, s), dtype=torch.uint8, device="cuda") for s in sstride]
    counts = [torch.zeros((x,), dtype=torch.int32, device="cuda") for x in d]
    u_out = [torch.zeros((M, r, c), dtype=torch.bfloat16, device="cuda") for r, c in shapes]
    d_out = [torch.zeros((r, c), dtype=torch.bfloat16, device="cuda") for r, c in shapes]
    plan = P.StepPlan(w, mom, grad, beta=beta, lr=lr, ns_steps=K, weight_decay=wd, scale=scale, v0=v0,
                      sign_fmt=sign_fmt, local_polar_steps=Kp, update_rsqrt_mn=rsqrt,
                      signs_out=signs, counts_out=counts, u_out=u_out, d_out=d_out)
    P.signmuon_step(ctx, plan)
    torch.cuda.synchronize()
    for i, (r, c) in enumerate(shapes):
        # a1: momentum bit-exact
        m_ref = O.momentum_update(M0[i], G[i], W0[i], beta, wd, dtype=np.float32)
        assert np.array_equal(mom[i].cpu().numpy().view(np.uint32), m_ref.view(np.uint32)), f"momentum block {i}"
        U = bf16_host(u_out[i])
        # a2-a4: U against the float32 oracle (on selected blocks: it is the slow part)
        if check_ns_blocks is None or i in check_ns_blocks:
            for p in range(M):
                ref = O.polar_ns(m_ref[p], K, O.PAPER_COEFFS, scale, 2, 1e-12, V0[i][p], dtype=np.float32)
                ns_check(U[p], ref, f"U block {i} worker {p}")
        # a5: the oracle's packing of the GPU's own U, bit-exact
        if sign_fmt == "1bit":
            s_ref = np.stack([O.pack_bits(O.sign_entries(U[p])) for p in range(M)])
            vote_ref, c_ref = O.majority_vote_bits(s_ref, M, d[i])
        else:
            s_ref = np.stack([O.signs_pm1(U[p]).reshape(-1) for p in range(M)]).view(np.uint8)
            vote_ref, c_ref = O.majority_vote_int8(s_ref.view(np.int8))
        assert np.array_equal(signs[i].cpu().numpy(), s_ref), f"signs block {i}"
        # a6: vote / counts of those signs, bit-exact
        assert np.array_equal(counts[i].cpu().numpy(), c_ref), f"counts block {i}"
        S_bar = vote_ref.reshape(r, c)
        D = bf16_host(d_out[i])
        if Kp == 0:
            assert np.array_equal(D, S_bar.astype(np.float32)), f"vote block {i}"
        elif check_ns_blocks is None or i in check_ns_blocks:
            # a7: local polar of the voted matrix against the float32 oracle
            ref = O.local_polar(S_bar, Kp, O.PAPER_COEFFS, scale, 2, 1e-12, V0[i][0], dtype=np.float32)
            ns_check(D, ref, f"D block {i}")
        # a8: W - step * D with the GPU's own D, bit-exact
        w_ref = O.apply_update(W0[i], D, lr, rsqrt, dtype=np.float32)
        assert np.array_equal(w[i].cpu().numpy().view(np.uint32), w_ref.view(np.uint32)), f"W block {i}"
    return plan


def test_step_single256(P, vctx):
    """256x256, M=4, N(0,1) gradients from zero momentum, 5 NS steps, 1-bit, no local polar."""
    ctx = vctx
    cfg = wl.WORKLOADS["single256"]
    shapes, M = cfg["shapes"], cfg["M"]
    G = [wl.worker_grads("single256", 0, 256, 256)]
    run_step_case(P, ctx, shapes, M, sign_fmt="1bit", Kp=0, grads=G)


@pytest.mark.parametrize("sign_fmt", ["1bit", "int8"])
@pytest.mark.parametrize("Kp", [0, 3])
def test_step_mixed_set(P, vctx, sign_fmt, Kp):
    ctx = vctx
    # (200, 160) and (96, 224): signs packed by the apply GEMM with zero padding in both dimensions;
    # (100, 72): rows that do not pack into whole words (separate sign-pack launch)
    shapes = [(64, 192), (192, 64), (64, 192), (128, 128), (100, 72), (64, 192), (200, 160), (96, 224)]
    run_step_case(P, ctx, shapes, 3, sign_fmt=sign_fmt, Kp=Kp, wd=0.1, rsqrt=(Kp > 0))


@pytest.mark.parametrize("batch,r,c", [(8, 641, 700), (8, 764, 710), (7, 830, 770), (1, 1990, 2010), (5, 641, 700), (5, 700, 641),
                                       (5, 710, 764), (5, 764, 710), (5, 770, 830), (5, 830, 770)])
def test_polar_ns_in_one_round_of_tiles_of_128(P, ctx, batch, r, c):
    """Launches of 129 to 256 tiles of 128 with more than ten slices of K, which take three LDS stages on a card of 256
    compute units; last tiles are half empty.  Batches of 7 and 8: the symmetric products, 11, 12 and 13 slices (every
    remainder by three), while their applies have 288 tiles or more and keep two stages.  Batches of 5: the applies (180
    to 245 tiles), 11, 12 and 13 slices, wide and tall.  One matrix of 1990 x 2010: both, 32 slices."""
    x = wl.normal((batch, r, c), stream=63, block=r, worker=c)
    xd = dev(x)
    P.signmuon_polar_ns(ctx, xd, 5)
    again = dev(x)
    cc = P.Context(gemm_tile=256)   # two stages
    P.signmuon_polar_ns(cc, again, 5)
    cc.close()
    got, other = xd.cpu().numpy(), again.cpu().numpy()
    for b in (0, batch - 1):
        ref = O.polar_ns(x[b], 5, O.PAPER_COEFFS, "fro", 2, 1e-12, None, dtype=np.float32)
        ns_check(got[b], ref, f"{(batch, r, c)} item {b}")
        ns_check(other[b], ref, f"{(batch, r, c)} item {b}, two stages")


@pytest.mark.parametrize("sign_fmt", ["1bit", "int8"])
@pytest.mark.parametrize("Kp", [0, 3])
@pytest.mark.parametrize("K", [0, 5])
def test_step_with_rows_of_any_length(P, sign_fmt, Kp, K):
    """Signs in padded rows, votes, updates and copies of rows that are no multiple of anything, next to whole rows."""
    for opts in (dict(), dict(gemm_tile=64)):
        c = P.Context(**opts)
        run_step_case(P, c, [(129, 101), (64, 128), (67, 33), (1, 7), (5, 1)], 3, sign_fmt=sign_fmt, Kp=Kp, K=K, wd=0.1)
        c.close()


@pytest.mark.parametrize("sign_fmt", ["1bit", "int8"])
@pytest.mark.parametrize("K,Kp", [(0, 0), (5, 0), (2, 3)])
def test_step_results_do_not_depend_on_the_taps_of_signs(P, ctx, sign_fmt, K, Kp):
    """No tap, a tap of every block's signs (from which the vote then reads padded blocks), of the padded blocks alone and
    of some of them: the same momentum, weights and counts to the bit, and the same signs wherever they are tapped."""
    shapes, M = [(129, 101), (64, 128), (67, 33), (1, 7), (5, 1), (1100, 1999)], 9
    padded = {i for i, (r, c) in enumerate(shapes) if c % 64}
    first = None
    for tapped in (set(), set(range(6)), padded, {0, 1}, {5}):
        w = [dev(wl.weights(r, c, block=i, stream=70)) for i, (r, c) in enumerate(shapes)]
        grad = [dev(wl.normal((M, r, c), stream=70, block=i, worker=1)) for i, (r, c) in enumerate(shapes)]
        mom = [torch.zeros_like(g) for g in grad]
        size = [O.packed_stride_bytes(r * c) if sign_fmt == "1bit" else r * c for r, c in shapes]
        signs = [torch.zeros((M, n), dtype=torch.uint8, device="cuda") if i in tapped else None for i, n in enumerate(size)]
        counts = [torch.zeros((r * c,), dtype=torch.int32, device="cuda") for r, c in shapes]
        plan = P.StepPlan(w, mom, grad, beta=0.9, lr=1e-3, ns_steps=K, sign_fmt=sign_fmt, local_polar_steps=Kp,
                          signs_out=signs if tapped else None, counts_out=counts)
        P.signmuon_step(ctx, plan)
        got = [t.cpu() for t in w + mom + counts]
        seen = {i: signs[i].cpu() for i in tapped}
        if first is None:
            first, sign_ref = got, {}
        assert all(torch.equal(a, b) for a, b in zip(got, first)), tapped
        for i, t in seen.items():
            assert torch.equal(t, sign_ref.setdefault(i, t)), (tapped, i)


@pytest.mark.parametrize("special", [False, True])
def test_step_signs_written_by_the_apply_alone(P, vctx, special):
    """Without a u_out tap the last apply writes only the packed signs (U is never stored; the bits come
    straight from the accumulators).  The same step with all taps (checked against the oracle by the cases
    above; there the signs are taken from the stored bf16 U) must give the same signs, counts and W.
    special: a column of entries near the bottom of the fp32 range (its outputs fall among the
    denormals, negative ones included), a NaN (the whole matrix turns NaN: all signs -1) and a zero matrix."""
    # (64, 100) cannot be packed by the GEMM; (200, 160) is packed with padding in both dimensions;
    # (320, 576) and (576, 320) span two tiles of 256 each way with a ragged second tile
    ctx = vctx
    shapes, M = [(128, 256), (256, 128), (192, 192), (64, 100), (200, 160), (320, 576), (576, 320)], 3
    outs = []
    for tapped in (True, False):
        w = [dev(wl.weights(r, c, block=i)) for i, (r, c) in enumerate(shapes)]
        mom = [torch.zeros((M, r, c), device="cuda") for r, c in shapes]
        g_host = [wl.normal((M, r, c), stream=29, block=i) for i, (r, c) in enumerate(shapes)]
        if special:
            sgn = np.where(wl.normal((M, 128), stream=30) >= 0, 1.0, -1.0).astype(np.float32)
            g_host[0][:, :, 5] = sgn * np.float32(3e-37)
            g_host[1][0, 7, 9] = np.float32("nan")
            g_host[2][1] = 0.0
            sgn = np.where(wl.normal((M, 320), stream=35) >= 0, 1.0, -1.0).astype(np.float32)
            g_host[5][:, :, 300] = sgn * np.float32(3e-37)          # a column in the second 256-tile
            g_host[6][2, 400, 17] = np.float32("nan")
        grad = [dev(g) for g in g_host]
        d = [r * c for r, c in shapes]
        signs = [torch.zeros((M, O.packed_stride_bytes(x)), dtype=torch.uint8, device="cuda") for x in d]
        counts = [torch.zeros((x,), dtype=torch.int32, device="cuda") for x in d]
        u_out = [torch.zeros((M, r, c), dtype=torch.bfloat16, device="cuda") for r, c in shapes] if tapped else None
        plan = P.StepPlan(w, mom, grad, beta=0.9, lr=1e-2, ns_steps=5, sign_fmt="1bit", local_polar_steps=2,
                          signs_out=signs, counts_out=counts, u_out=u_out)
        P.signmuon_step(ctx, plan)
        torch.cuda.synchronize()
        outs.append(([t.cpu().numpy() for t in signs], [t.cpu().numpy() for t in counts], [t.cpu().numpy() for t in w]))
    for a, b in zip(outs[0], outs[1]):
        for x, y in zip(a, b):
            assert np.array_equal(x.view(np.uint8), y.view(np.uint8))


def test_step_replays_from_a_hip_graph(P):
    """After the first call (which plans and clears the workspace) a step only enqueues kernels on the
    context's stream, so it can be captured once and replayed.  Four replays, with eager work and
    synchronisations between them, must leave W and the momentum bit-identical to four eager steps."""
    shapes, M = [(128, 256), (256, 128), (192, 192), (64, 100)], 3

    def fresh():
        w = [dev(wl.weights(r, c, block=i, stream=33)) for i, (r, c) in enumerate(shapes)]
        mom = [torch.zeros((M, r, c), device="cuda") for r, c in shapes]
        grad = [dev(wl.normal((M, r, c), stream=33, block=i)) for i, (r, c) in enumerate(shapes)]
        return w, mom, grad

    results = []
    for use_graph in (False, True):
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            w, mom, grad = fresh()
            ctx = P.Context(stream=side)
            plan = P.StepPlan(w, mom, grad, beta=0.9, lr=1e-2, ns_steps=5, sign_fmt="1bit", local_polar_steps=3)
            P.signmuon_step(ctx, plan)                      # plans the workspace
            side.synchronize()
            snaps = []
            if use_graph:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=side):
                    P.signmuon_step(ctx, plan)
            for rep in range(4):
                if use_graph:
                    graph.replay()
                else:
                    P.signmuon_step(ctx, plan)
                torch.cuda.synchronize()
                scratch = torch.randn((1 << 16,), device="cuda").sum().item()      # unrelated eager work between replays
                assert np.isfinite(scratch)
                snaps.append(([t.cpu().numpy().copy() for t in w], [t.cpu().numpy().copy() for t in mom]))
            ctx.close()
        results.append(snaps)
    for rep in range(4):
        for a, b in zip(results[0][rep][0] + results[0][rep][1], results[1][rep][0] + results[1][rep][1]):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), f"replay {rep}"


def test_step_with_normalized_sign_update(P, ctx):
    """update scale mode 2: W <- W - lr S / max(PowerIter(S), eps) with S the voted sign (the appendix's
    "normalized sign").  The vote is checked bit-exactly from the GPU's own U; the step size, which every entry
    of a block shares, against the float32 oracle's PowerIter on the same S and start vector."""
    shapes, M, lr = [(128, 256), (200, 160), (64, 100), (256, 128)], 3, 0.05
    W0 = [wl.weights(r, c, block=i, stream=34) for i, (r, c) in enumerate(shapes)]
    G = [wl.normal((M, r, c), stream=34, block=i) for i, (r, c) in enumerate(shapes)]
    V0 = [wl.start_vectors(M, c, block=i, stream=34) for i, (r, c) in enumerate(shapes)]
    w = [dev(a) for a in W0]
    mom = [torch.zeros((M, r, c), device="cuda") for r, c in shapes]
    grad = [dev(a) for a in G]
    u_out = [torch.zeros((M, r, c), dtype=torch.bfloat16, device="cuda") for r, c in shapes]
    d_out = [torch.zeros((r, c), dtype=torch.bfloat16, device="cuda") for r, c in shapes]
    plan = P.StepPlan(w, mom, grad, beta=0.9, lr=lr, ns_steps=3, power_iters=2, v0=[dev(a) for a in V0],
                      update_rsqrt_mn="op_norm", u_out=u_out, d_out=d_out)
    P.signmuon_step(ctx, plan)
    torch.cuda.synchronize()
    for i, (r, c) in enumerate(shapes):
        U = u_out[i].float().cpu().numpy()
        signs = np.stack([O.pack_bits(O.sign_entries(U[p])) for p in range(M)])
        vote, _ = O.majority_vote_bits(signs, M, r * c)
        S = vote.reshape(r, c).astype(np.float32)
        assert np.array_equal(d_out[i].float().cpu().numpy(), S)
        moved = (W0[i].astype(np.float64) - w[i].cpu().numpy().astype(np.float64)) * S      # = step, entry by entry
        step_ref = lr / float(O.power_iter(S, 2, 1e-12, V0[i][0]))
        assert abs(moved.mean() - step_ref) <= 1e-3 * step_ref, (i, moved.mean(), step_ref)
        assert np.all(np.abs(moved - moved.mean()) <= 2e-3 * step_ref)                      # one step size per block
    with pytest.raises(P.SignMuonError):                                                    # not with a local polar step
        P.signmuon_step(ctx, P.StepPlan(w, mom, grad, beta=0.9, lr=lr, ns_steps=3, v0=[dev(a) for a in V0],
                                        update_rsqrt_mn="op_norm", local_polar_steps=2))


@pytest.mark.parametrize("mode", ["fused", "separate"])
@pytest.mark.parametrize("batch,r,c", [(2, 9, 16500), (3, 300, 70), (1, 2050, 64), (2, 130, 4100), (1, 1, 1)])
def test_polar_ns_spectral_scale_of_any_width(P, mode, batch, r, c):
    """Shares of the row chunks (narrow matrices), several quads per thread, more columns than the threads keep."""
    x = wl.normal((batch, r, c), stream=66, block=r, worker=c)
    v0 = wl.start_vectors(batch, c, block=r)
    ctx = P.Context(power_iter=mode)
    xd = dev(x)
    P.signmuon_polar_ns(ctx, xd, 1, scale="spectral", power_iters=2, eps=1e-12, v0=dev(v0))
    ctx.close()
    got = xd.cpu().numpy()
    for b in range(batch):
        ns_check(got[b], O.polar_ns(x[b], 1, O.PAPER_COEFFS, "spectral", 2, 1e-12, v0[b], dtype=np.float32), f"{(r, c)} item {b}")


def test_step_spectral(P, vctx):
    run_step_case(P, vctx, [(128, 256), (256, 128)], 2, sign_fmt="1bit", Kp=2, scale="spectral")


@pytest.mark.parametrize("mode", ["fused", "separate", "auto"])
def test_step_spectral_power_iteration_forms(P, mode):
    """Alg. PowerIter over a set that spans every form: matrices for each column-strip count of the fused pass
    (one read of X for X v and X^T u), one too wide for it (a pass per product), ragged row chunks and padding."""
    shapes = [(72, 4608), (200, 160), (96, 1800), (130, 2304), (64, 3000), (70, 4000), (300, 64)]
    ctx = P.Context(power_iter=mode)
    run_step_case(P, ctx, shapes, 2, sign_fmt="1bit", Kp=1, K=3, scale="spectral", stream=37)
    torch.cuda.synchronize()
    ctx.close()


def test_nan_worker_on_a_padded_shape_does_not_leak_into_other_blocks(P):
    """A NaN in one worker's gradient turns that worker's whole matrix NaN (every sign -1), zero padding of its
    slots in the working layout included.  After the vote those slots hold other blocks' voted matrices, so
    the padding is cleared again: the blocks without a NaN worker must come out exactly as in a run where
    the NaN is replaced by an ordinary number.  200 x 160 pads both dimensions; K = 7 makes both working
    buffers carry apply outputs; the local polar step reads the voted matrices with their padding."""
    shapes, M = [(200, 160)] * 3 + [(136, 200)] * 2, 3

    def run(ctx, poisoned):
        G = [wl.normal((M, r, c), stream=36, block=i) for i, (r, c) in enumerate(shapes)]
        if poisoned:
            G[0][1, 3, 4] = np.float32("nan")
            G[3][2, 100, 150] = np.float32("inf")
        w = [dev(wl.weights(r, c, block=i, stream=36)) for i, (r, c) in enumerate(shapes)]
        mom = [torch.zeros((M, r, c), device="cuda") for r, c in shapes]
        d_out = [torch.zeros((r, c), dtype=torch.bfloat16, device="cuda") for r, c in shapes]
        plan = P.StepPlan(w, mom, [dev(g) for g in G], beta=0.9, lr=1e-2, ns_steps=7, local_polar_steps=3, d_out=d_out)
        P.signmuon_step(ctx, plan)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in w], [bf16_host(t) for t in d_out]

    c0 = P.Context()
    w_ref, d_ref = run(c0, False)
    c0.close()
    c1 = P.Context()
    w_bad, d_bad = run(c1, True)
    w_after, d_after = run(c1, False)          # the same context, after it has seen the NaN
    c1.close()
    for i in range(len(shapes)):
        assert np.isfinite(w_ref[i]).all() and np.isfinite(d_ref[i]).all()
        assert np.array_equal(w_after[i], w_ref[i]) and np.array_equal(d_after[i], d_ref[i]), f"block {i} after the NaN"
    for i in (1, 2, 4):                        # blocks whose workers are all finite
        assert np.array_equal(w_bad[i], w_ref[i]) and np.array_equal(d_bad[i], d_ref[i]), f"block {i} beside the NaN"
    for i in (0, 3):                           # the vote tolerates the non-finite worker (its signs are all -1)
        assert np.isfinite(w_bad[i]).all() and np.isfinite(d_bad[i]).all()


def test_step_signsgd_limit_and_zero_gradients(P, ctx):
    # K = 0, beta = 0, M = 1: W - lr * sign(G)
    r, c = 48, 80
    G = wl.normal((1, r, c), stream=32)
    W0 = wl.weights(r, c, stream=32)
    w, mom, grad = [dev(W0)], [torch.zeros((1, r, c), device="cuda")], [dev(G)]
    plan = P.StepPlan(w, mom, grad, beta=0.0, lr=0.25, ns_steps=0)
    P.signmuon_step(ctx, plan)
    ref = O.signmuon_step(W0, np.zeros_like(G), G, beta=0.0, lr=0.25, ns_steps=0, dtype=np.float32)
    assert np.array_equal(w[0].cpu().numpy(), ref["W"])
    # all-zero gradients from zero state: every sign bit is 1, W decreases by lr
    w = [torch.ones((r, c), device="cuda")]
    z = [torch.zeros((3, r, c), device="cuda")]
    plan = P.StepPlan(w, [z[0].clone()], z, beta=0.9, lr=0.5, ns_steps=5)
    P.signmuon_step(ctx, plan)
    assert torch.all(w[0] == 0.5)


def test_step_is_deterministic_and_repeatable(P, ctx):
    shapes, M = [(128, 256), (256, 128)], 4
    outs = []
    for _ in range(2):
        W0 = [wl.weights(r, c, block=i, stream=33) for i, (r, c) in enumerate(shapes)]
        w = [dev(a) for a in W0]
        mom = [torch.zeros((M, r, c), device="cuda") for r, c in shapes]
        grad = [dev(wl.normal((M, r, c), stream=33, block=i)) for i, (r, c) in enumerate(shapes)]
        plan = P.StepPlan(w, mom, grad, beta=0.9, lr=1e-2, ns_steps=5, local_polar_steps=2)
        for _ in range(3):
            P.signmuon_step(ctx, plan)
        outs.append([t.cpu().numpy() for t in w + mom])
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
