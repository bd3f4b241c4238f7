"""Product sumchecks at the sizes where the round kernels change over, byte for byte against the oracle's C tier:
one block per evaluation in the last rounds (512, 256, 128, 64 and fewer pairs), few and many partial sums per round
(one, up to 64, more than 512)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[1, 0], ids=["helpers", "apart"])
def ctx(request, lib):
    """Every size both ways: the last rounds in one launch with helper blocks, and with launches of their own, which then run at
    sizes that they see in no other way."""
    c = lib.Context(0)
    c.set_round_helpers(request.param)
    yield c
    c.close()


@pytest.mark.parametrize("d", [1, 2, 3, 5, 8, 10, 11, 12, 13, 14, 17, 19, 20])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_product_rounds(lib, ctx, k, d):
    from oracle import c_oracle
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(100 * k + d)
    raws = [uniform_fr_limbs(rng, 1 << d).tobytes() for _ in range(k)]
    if d == 12:     # the largest element everywhere: sums of lazy values at the top of their range
        from oracle.field import R_MOD
        raws = [int(R_MOD - 1).to_bytes(32, "little") * (1 << d) for _ in range(k)]
    tabs = [lib.fr_tensor_upload(ctx, r, (1 << d,)) for r in raws]
    tr = lib.Transcript(7)
    got = lib.sumcheck_product(ctx, tabs, tr)
    proof, chal, digest = c_oracle.product_prove(raws, 7)
    assert got["proof"] == proof and got["points"] == chal and tr.digest() == digest


# The last rounds with helper blocks: fewer rounds than they take, 16, 32 and 64 helpers with the smallest and largest slices, after a
# round of its own and after passes of two rounds; and the block that closes the rounds alone, as when no helper reports
@pytest.mark.parametrize("d", [7, 8, 9, 12, 13, 14, 15, 16, 17, 18])
@pytest.mark.parametrize("k", [2, 3])
def test_product_rounds_with_helpers(lib, k, d):
    import paper_2307_16273_amd as zk
    from oracle import c_oracle
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(900 * k + d)
    raws = [uniform_fr_limbs(rng, 1 << d).tobytes() for _ in range(k)]
    if d == 14:     # the largest element everywhere: sums of lazy values at the top of their range
        from oracle.field import R_MOD
        raws = [int(R_MOD - 1).to_bytes(32, "little") * (1 << d) for _ in range(k)]
    proof, chal, digest = c_oracle.product_prove(raws, 3)
    own = zk.Context(0)
    tabs = [zk.fr_tensor_upload(own, r, (1 << d,)) for r in raws]
    # HELPERS_ON after HELPERS_ABSENT and the other way round: launches follow each other with either outcome
    for mode in (1, 2, 1, 1, 0, 2, 2, 1):
        own.set_round_helpers(mode)
        tr = zk.Transcript(3)
        got = zk.sumcheck_product(own, tabs, tr)
        assert got["proof"] == proof and got["points"] == chal and tr.digest() == digest, mode
    own.close()


# zkReLU's last i-rounds with helper blocks: three rounds and nine, behind rounds on the integers (d < 10) and behind the contraction; an odd number
# of columns (the last helper has one), one pair of them, 64 of two slices (all 64 helpers and 16 for the equations); and the leader alone
@pytest.mark.parametrize("d", [7, 8, 9, 10, 13, 15])
@pytest.mark.parametrize("q,r,ga", [(32, 16, True), (33, 31, True), (5, 2, False), (1, 1, True), (1, 1, False), (20, 13, True)])
def test_zkrelu_rounds_with_helpers(lib, d, q, r, ga):
    import torch
    import paper_2307_16273_amd as zk
    from oracle import c_oracle
    rng = np.random.default_rng(70 * d + q)
    b = 1 << (q + r - 1)
    z, g = (rng.integers(-b, b - 1, 1 << d, dtype=np.int64, endpoint=True) for _ in range(2))
    z[0], g[-1] = -b, b - 1
    ot = c_oracle.Transcript(4)
    want = c_oracle.zkrelu_prove(z, g if ga else None, q, r, ot)
    own = zk.Context(0)
    zd, gd = torch.from_numpy(z).cuda(), torch.from_numpy(g).cuda() if ga else None
    for mode in (1, 2, 1, 0, 2, 1):
        own.set_round_helpers(mode)
        tr = zk.Transcript(4)
        assert zk.zkrelu_prove(own, zd, gd, tr, q, r)["proof"] == want and tr.digest() == ot.digest(), mode
    own.close()


# A wait that is given up (at once here) fails the call and changes nothing of the caller's.  Words of its messages stay in the helpers' mail,
# valid ones in the places of the next call's: that one, on other inputs, gives its own proof.
@pytest.mark.parametrize("k,d", [(2, 9), (3, 12), (2, 14), (3, 15)])
def test_product_after_a_wait_that_was_given_up(lib, k, d):
    import paper_2307_16273_amd as zk
    from oracle import c_oracle
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(40 * k + d)
    own = zk.Context(0)
    raws = [[uniform_fr_limbs(rng, 1 << d).tobytes() for _ in range(k)] for _ in range(2)]
    tabs = [[zk.fr_tensor_upload(own, r, (1 << d,)) for r in side] for side in raws]
    want = [c_oracle.product_prove(side, 3) for side in raws]
    lib.sumcheck_product(own, tabs[0], lib.Transcript(3))       # the kernel's code is there: all helpers report in time from now on
    for turn in range(4):
        own.set_helper_wait(0)
        tr = zk.Transcript(3)
        before = tr.digest()
        with pytest.raises(zk.ZkdlError, match="ZKDL_EHIP"):
            zk.sumcheck_product(own, tabs[turn & 1], tr)
        assert tr.digest() == before
        own.set_helper_wait(4000000)
        for side in (1 - (turn & 1), turn & 1):
            tr = zk.Transcript(3)
            got = zk.sumcheck_product(own, tabs[side], tr)
            assert (got["proof"], got["points"], tr.digest()) == want[side], (turn, side)
    own.close()


@pytest.mark.parametrize("d,q,r,ga", [(9, 32, 16, True), (12, 5, 2, False), (15, 20, 13, True)])
def test_zkrelu_after_a_wait_that_was_given_up(lib, d, q, r, ga):
    import torch
    import paper_2307_16273_amd as zk
    from oracle import c_oracle
    rng = np.random.default_rng(d)
    b = 1 << (q + r - 1)
    own = zk.Context(0)
    ins, want = [], []
    for _ in range(2):
        z, g = (rng.integers(-b, b - 1, 1 << d, dtype=np.int64, endpoint=True) for _ in range(2))
        ot = c_oracle.Transcript(4)
        want.append((c_oracle.zkrelu_prove(z, g if ga else None, q, r, ot), ot.digest()))
        ins.append((torch.from_numpy(z).cuda(), torch.from_numpy(g).cuda() if ga else None))
    lib.zkrelu_prove(own, *ins[0], lib.Transcript(4), q, r)
    for turn in range(4):
        own.set_helper_wait(0)
        tr = zk.Transcript(4)
        before = tr.digest()
        with pytest.raises(zk.ZkdlError, match="ZKDL_EHIP"):
            zk.zkrelu_prove(own, *ins[turn & 1], tr, q, r)
        assert tr.digest() == before
        own.set_helper_wait(4000000)
        for side in (1 - (turn & 1), turn & 1):
            tr = zk.Transcript(4)
            got = zk.zkrelu_prove(own, *ins[side], tr, q, r)
            assert (got["proof"], tr.digest()) == want[side], (turn, side)
    own.close()


def test_rounds_beside_other_work(lib):
    """Additions over 1 GB on another stream hold the compute units that the helpers need: some launches find their helpers, some do not."""
    import paper_2307_16273_amd as zk
    import torch
    from oracle import c_oracle
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(77)
    own, side, x = zk.Context(0), torch.cuda.Stream(), torch.ones(1 << 28, device="cuda")
    cases = []
    for k, d in ((2, 9), (3, 12), (2, 15), (3, 15)):
        raws = [uniform_fr_limbs(rng, 1 << d).tobytes() for _ in range(k)]
        cases.append(([zk.fr_tensor_upload(own, r, (1 << d,)) for r in raws], c_oracle.product_prove(raws, 3)[::2]))
    z = rng.integers(-1 << 40, 1 << 40, 1 << 12, dtype=np.int64)
    ot = c_oracle.Transcript(3)
    cases.append((torch.from_numpy(z).cuda(), (c_oracle.zkrelu_prove(z, None, 32, 16, ot), ot.digest())))
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(60):
            x.add_(1.0)
    for turn in range(8):
        for given, want in cases:
            tr = zk.Transcript(3)
            got = zk.sumcheck_product(own, given, tr) if isinstance(given, list) else zk.zkrelu_prove(own, given, None, tr, 32, 16)
            assert (got["proof"], tr.digest()) == want, turn
    torch.cuda.synchronize()
    own.close()


@pytest.mark.parametrize("mode", [0, 2])
@pytest.mark.parametrize("shape", [(8, 16, 256, 8), (2, 4, 2048, 4), (1, 2, 1024, 2), (64, 2, 64, 2)])
def test_matmul_and_hadamard_without_helpers(lib, ctx, shape, mode):
    """The two forms of the matrix product and the Hadamard product (from 2^17 entries on: the equality factor built for the last launch)."""
    import paper_2307_16273_amd as zk
    import torch
    n, d1, d2, d3 = shape
    rng = np.random.default_rng(4)
    own = zk.Context(0)
    a, b = (torch.from_numpy(rng.integers(-9999, 9999, s, dtype=np.int32)).cuda() for s in ((n, d1, d2), (n, d2, d3)))
    x, y = (torch.from_numpy(rng.integers(-9999, 9999, (n * d2 * 256,), dtype=np.int32)).cuda() for _ in range(2))
    out = []
    for c, m in ((ctx, None), (own, mode)):
        if m is not None:
            c.set_round_helpers(m)
        ta, tb = zk.tensor_wrap_int(c, a, a.shape), zk.tensor_wrap_int(c, b, b.shape)
        tx, ty = zk.tensor_wrap_int(c, x), zk.tensor_wrap_int(c, y)
        tr = zk.Transcript(1)
        out.append([bytes(f(c, *t, tr)["proof"]) for f, t in ((zk.sumcheck_matmul, (ta, tb)), (zk.sumcheck_matmul_ft, (ta, tb)),
                                                              (zk.sumcheck_hadamard, (tx, ty)))] + [tr.digest()])
    own.close()
    assert out[0] == out[1]


@pytest.mark.parametrize("mode", [0, 2])
@pytest.mark.parametrize("form", ["plain", "linked", "ft", "update"])
def test_windows_without_helpers(lib, form, mode):
    """Whole windows and the update, as a partition with few compute units or a full device proves them."""
    import paper_2307_16273_amd as zk
    import torch
    from workloads import fcnn_window, CONFIG_SEED
    wit = {k: torch.from_numpy(np.ascontiguousarray(x)).cuda() if isinstance(x, np.ndarray) else x
           for k, x in fcnn_window(CONFIG_SEED + 5, n_layers=4, width=64, batch=16, steps=2).items()}
    own, out = zk.Context(0), []
    for m in (1, mode):
        own.set_round_helpers(m)
        tr = zk.Transcript(6)
        if form == "update":
            g = np.random.default_rng(5).integers(-1 << 40, 1 << 40, 1 << 12, dtype=np.int64)
            got = zk.update_prove(own, g, tr, 26, 30)
        else:
            got = zk.aggregate_prove(own, wit, tr, linked=form == "linked", ft=form == "ft")
        out.append((bytes(got["proof"]), got["points"], tr.digest()))
    own.close()
    assert out[0] == out[1]


# Every length of the stream's unfinished block in front of a sumcheck: the claim's and the first round's frames are taken
# together, and the draw behind them has one closing block or two.
@pytest.mark.parametrize("k", [1, 2, 3])
def test_first_round_behind_any_unfinished_block(lib, ctx, k):
    from oracle import protocols as P
    from oracle.field import fr_array_from_le
    from oracle.transcript import Transcript
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(50 + k)
    raws = [uniform_fr_limbs(rng, 4).tobytes() for _ in range(k)]
    tabs = [lib.fr_tensor_upload(ctx, r, (4,)) for r in raws]
    arrays = [fr_array_from_le(r, 4) for r in raws]
    for pad in range(64):
        tr, ot = lib.Transcript(pad), Transcript(pad)
        for t in (tr, ot):
            t.absorb(b"pad", bytes(range(pad)))
        for _ in range(2):       # the second one behind the finals of the first
            got = lib.sumcheck_product(ctx, tabs, tr)
            buf, _, vs = P.product_prove(arrays, ot)
            assert got["proof"] == buf and got["points"] == vs and tr.digest() == ot.digest(), pad


@pytest.mark.parametrize("shape", [(1, 2, 2, 1), (1, 1, 4, 2), (2, 2, 2, 2), (4, 1, 1, 1)])
def test_matmul_behind_any_unfinished_block(lib, ctx, shape):
    """The same for claims that are written but not absorbed, or copied (the two forms of the matrix product)."""
    import torch
    from oracle import protocols as P
    from oracle.field import fr_array
    from oracle.transcript import Transcript
    n, d1, d2, d3 = shape
    rng = np.random.default_rng(3)
    a, b = rng.integers(-99, 99, (n, d1, d2), dtype=np.int32), rng.integers(-99, 99, (n, d2, d3), dtype=np.int32)
    ta, tb = (lib.tensor_wrap_int(ctx, torch.from_numpy(x).cuda(), x.shape) for x in (a, b))
    for ours, theirs in ((lib.sumcheck_matmul, P.matmul_prove), (lib.sumcheck_matmul_ft, P.matmul_ft_prove)):
        for pad in range(0, 64, 3):
            tr, ot = lib.Transcript(pad), Transcript(pad)
            for t in (tr, ot):
                t.absorb(b"pad", bytes(range(pad)))
            got = ours(ctx, ta, tb, tr)
            buf = theirs(fr_array(a), list(a.shape), fr_array(b), list(b.shape), ot)[0]
            assert got["proof"] == buf and tr.digest() == ot.digest(), pad


# (log2 rows, Q, R, backward slice): below, at and above the size from which the first five rounds come from one
# contraction; one and two words of columns, columns that do not fill a group of 32, the widest recompositions
@pytest.mark.parametrize("d,q,r,ga", [(9, 32, 16, True), (10, 32, 16, True), (10, 32, 16, False), (10, 32, 32, True),
                                      (10, 1, 1, True), (11, 5, 2, True), (11, 33, 31, False), (12, 26, 30, False),
                                      (13, 16, 8, True), (14, 31, 28, True), (16, 32, 16, True), (17, 24, 13, False)])
def test_zkrelu_first_rounds(lib, ctx, d, q, r, ga):
    import torch
    from oracle import c_oracle
    rng = np.random.default_rng(1000 + d)
    b = 1 << (q + r - 1)
    vals = [rng.integers(-b, b - 1, 1 << d, dtype=np.int64, endpoint=True) for _ in range(2)]
    for x in vals:       # the ends of the range, where signed digits carry the furthest
        x[:6] = [b - 1, -b, 0, -1, b // 2, -(b // 2)]
        x[-2:] = [b - 1, -b]
    z, g = vals[0], vals[1] if ga else None
    tr = lib.Transcript(5)
    got = lib.zkrelu_prove(ctx, torch.from_numpy(z).cuda(), None if g is None else torch.from_numpy(g).cuda(), tr, q, r)
    ot = c_oracle.Transcript(5)
    assert got["proof"] == c_oracle.zkrelu_prove(z, g, q, r, ot)
    assert tr.digest() == ot.digest()


# the last i-rounds in one block (up to four of them, from eight pairs of rows on; one or two where the others have helper blocks): fewer
# rounds than that, none at all, and the rounds before them on the integers or on columns; one column to 64, tables of j from 2 entries to 64
@pytest.mark.parametrize("d", list(range(0, 11)))
@pytest.mark.parametrize("q,r,ga", [(1, 1, True), (2, 1, False), (33, 31, True), (20, 13, False)])
def test_zkrelu_short_rounds(lib, ctx, d, q, r, ga):
    import torch
    from oracle import c_oracle
    rng = np.random.default_rng(d + q)
    b = 1 << (q + r - 1)
    z, g = (rng.integers(-b, b - 1, 1 << d, dtype=np.int64, endpoint=True) for _ in range(2))
    z[0], g[-1] = -b, b - 1
    tr, ot = lib.Transcript(9), c_oracle.Transcript(9)
    got = lib.zkrelu_prove(ctx, torch.from_numpy(z).cuda(), torch.from_numpy(g).cuda() if ga else None, tr, q, r)
    assert got["proof"] == c_oracle.zkrelu_prove(z, g if ga else None, q, r, ot)
    assert tr.digest() == ot.digest()


# columns written by the round that sums them, which the default threshold does from 2^22 rows on (here from 64 `fill`): groups of
# 16 columns that are not full, all of them in a thread or one each; one block of threads that is not full, one that is, several
@pytest.mark.parametrize("fill,d,q,r,ga", [(f, *c) for f in (1, 16, 32) for c in
                                           ((10, 1, 1, True), (10, 9, 8, True), (11, 16, 16, False), (11, 33, 31, True), (12, 26, 30, False))
                                           if 64 * f <= 1 << c[0]] +
                         [(32, 11, 1, 1, True), (32, 11, 9, 8, True), (1, 14, 32, 16, True), (1, 15, 9, 8, True), (256, 15, 26, 30, False),
                          (1, 16, 32, 16, True), (1024, 16, 33, 31, True)])
@pytest.mark.parametrize("helpers", [1, 0])
def test_zkrelu_columns_in_one_pass(lib, fill, d, q, r, ga, helpers):
    import torch
    import paper_2307_16273_amd as zk
    from oracle import c_oracle
    rng = np.random.default_rng(d + q)
    b = 1 << (q + r - 1)
    z, g = (rng.integers(-b, b - 1, 1 << d, dtype=np.int64, endpoint=True) for _ in range(2))
    c2 = zk.Context(0)
    c2.set_fill_threads(fill)
    c2.set_round_helpers(helpers)
    got = lib.zkrelu_prove(c2, torch.from_numpy(z).cuda(), torch.from_numpy(g).cuda() if ga else None, lib.Transcript(9), q, r)
    assert got["proof"] == c_oracle.zkrelu_prove(z, g if ga else None, q, r, c_oracle.Transcript(9))
    c2.close()


def test_zkrelu_constant_rows(lib, ctx):
    """Every row the most negative value: the largest digit sums of one sign."""
    import torch
    from oracle import c_oracle
    for val in (-(1 << 47), (1 << 47) - 1, -1):
        z = np.full(1 << 12, val, dtype=np.int64)
        got = lib.zkrelu_prove(ctx, torch.from_numpy(z).cuda(), torch.from_numpy(z).cuda(), lib.Transcript(6), 32, 16)
        assert got["proof"] == c_oracle.zkrelu_prove(z, z, 32, 16, c_oracle.Transcript(6))


def test_zkrelu_range_error(lib, ctx):
    import torch
    z = np.zeros(1 << 11, dtype=np.int64)
    z[1500] = 1 << 47
    tr = lib.Transcript(8)
    before = tr.digest()
    with pytest.raises(lib.ZkdlError) as e:
        lib.zkrelu_prove(ctx, torch.from_numpy(z).cuda(), None, tr, 32, 16)
    assert e.value.code == -2 and tr.digest() == before


# from 2^16 entries on (the two sizes below: one launch, or a launch per round): two rounds per pass, one or two pairs of rounds left over for
# the last launch, one value of the batch or many per block; tables whose signed digits are all as large as they get
@pytest.mark.parametrize("k,d,fill", [(2, 14, "random"), (2, 15, "digits"), (2, 16, "random"), (2, 17, "digits"), (3, 16, "digits"),
                                      (3, 17, "top"), (2, 21, "random"), (3, 20, "digits"), (3, 20, "mixed"),
                                      (3, 21, "random"), (3, 22, "top")])
def test_product_pairs_of_rounds(lib, ctx, k, d, fill):
    from oracle import c_oracle
    from oracle.field import R_MOD
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(k * d)
    n = 1 << d
    consts = {"digits": [R_MOD - int("80" * 31, 16), R_MOD - 1 - int("80" * 31, 16), int("7f" * 31, 16)],
              "top": [R_MOD - 1, 0, 1], "mixed": [R_MOD - 1, 0, None], "random": [None] * 3}[fill]
    raws = [uniform_fr_limbs(rng, n).tobytes() if c is None else (c << 261) * pow(1 << 522, -1, R_MOD) % R_MOD for c in consts[:k]]
    raws = [r if isinstance(r, bytes) else int(r).to_bytes(32, "little") * n for r in raws]
    if fill == "mixed":      # two tables differ in one entry only
        raws[1] = raws[0][:32 * (n - 1)] + (5).to_bytes(32, "little")
    tabs = [lib.fr_tensor_upload(ctx, r, (n,)) for r in raws]
    for rep in range(2):     # the second one with the work memory as the first one left it
        tr = lib.Transcript(9)
        got = lib.sumcheck_product(ctx, tabs, tr)
        if rep == 0:
            proof, chal, digest = c_oracle.product_prove(raws, 9)
        assert got["proof"] == proof and got["points"] == chal and tr.digest() == digest
    assert tabs[0].download() == raws[0]


# Constants whose internal form (times 2^261, less r, in signed 8-bit digits) has a digit -128 on both sides: the digit
# sums are as large as the number of values per block lets them be.  2^27 entries are the first size at which a block
# per compute unit would take more than 2^16 values.
@pytest.mark.parametrize("factors", [(6, 6), (2, 3, 6)])
def test_product_of_constants_at_2p27(lib, ctx, factors):
    import torch
    from oracle import protocols as P
    from oracle.field import R_MOD
    from oracle.transcript import Transcript
    d = 27
    tabs = {}
    for f in set(factors):
        tabs[f] = lib.fr_tensor_upload(ctx, torch.full((1 << d,), f, dtype=torch.int32, device="cuda"), (1 << d,))
    tr, ot = lib.Transcript(31), Transcript(31)
    got = lib.sumcheck_product(ctx, [tabs[f] for f in factors], tr)
    for t in tabs.values():
        t.free()
    proof, vs = P.product_verify(got["proof"], len(factors), d, ot)
    assert got["points"] == vs and tr.digest() == ot.digest()
    assert got["claims"] == list(factors)
    # every table stays constant, so g_t is: the product times the 2^(d - t - 1) pairs
    product = int(np.prod(factors))
    assert proof.claim0 == (product << d) % R_MOD
    assert [list(g) for g in proof.rounds] == [[(product << (d - t - 1)) % R_MOD] * (len(factors) + 1) for t in range(d)]


def test_verifier_of_more_rounds_than_a_batch(lib):
    """The device verifier works 32 rounds of a sumcheck out together; 2^26 gradients make one of 33.  Against the host's, which goes
    round by round: the accepted proof, and one with an element of every round changed, the second batch's among them."""
    import torch
    from oracle.field import R_MOD
    c2 = lib.Context(0)
    g = torch.Generator(device="cuda").manual_seed(4)
    gw = torch.randint(-2 ** 40, 2 ** 40, (1 << 26,), generator=g, device="cuda", dtype=torch.int64)
    tr = lib.Transcript(5)
    proof = lib.update_prove(c2, gw, tr, 26, 30)["proof"]
    rounds = 27 + 6
    # the zkReLU sumcheck's rounds: four elements each, behind the claim that their first two add up to
    words = [int.from_bytes(proof[k:k + 32], "little") for k in range(0, len(proof) - 31, 4)]
    start = [4 * k for k in range(8, len(words) - 16) if (words[k] + words[k + 8]) % R_MOD == words[k - 8] and words[k - 8] > 1 << 200]
    start = [s for s in start if s + 128 * rounds <= len(proof)][0]

    def both(data):
        t1, t2 = lib.Transcript(5), lib.Transcript(5)
        a, b = lib.aggregate_verify(c2, data, t1), lib.aggregate_verify(None, data, t2)
        assert a["verdict"] == b["verdict"] and a["points"] == b["points"] and t1.digest() == t2.digest()
        return a["verdict"]

    assert both(proof) == 0
    for t in range(rounds):
        for k in (0, 3):
            bad = bytearray(proof)
            at = start + 128 * t + 32 * k
            x = (int.from_bytes(bad[at:at + 32], "little") + 1) % R_MOD
            bad[at:at + 32] = x.to_bytes(32, "little")
            assert both(bytes(bad)) != 0, (t, k)
            if k:
                bad[at:at + 32] = R_MOD.to_bytes(32, "little")       # not canonical
                assert both(bytes(bad)) != 0, (t, k)
    c2.close()
