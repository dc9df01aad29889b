"""Bit-exact parity where the library's arithmetic changes form: moduli on
either side of the floating-point range, of 2^60 and of every size in one
chain, digits of one to sixteen primes, and extreme residues, at rings whose
passes take each geometry and launches of each size class."""
import numpy as np
import pytest

import oracle as O
import paper_2603_22437_amd as H
import seeded_inputs as S

pytestmark = pytest.mark.gpu


def _primes(two_n, start, count, taken, step):
    """`count` primes = 1 mod 2N from `start` on, upwards (step 1) or down."""
    out, x = [], start // two_n * two_n + 1
    if step > 0 and x < start:
        x += two_n
    if step < 0 and x >= start:
        x -= two_n
    while len(out) < count:
        if S.is_prime(x) and x not in taken:
            out.append(x)
            taken.add(x)
        x += step * two_n
    return out


def _params(kind, log_n):
    two_n, taken = 2 << log_n, set()
    limit = (1 << 50) + (1 << 44)     # moduli from 2^26 to here run on doubles
    pick = lambda start, count, step: _primes(two_n, start, count, taken, step)
    if kind == "edges":     # both sides of every boundary, in one chain
        q = (pick(1 << 60, 1, -1) + pick(limit, 1, -1) + pick(limit, 1, 1) +
             pick(1 << 26, 1, 1) + pick(1 << 26, 1, -1) + pick(1 << 45, 1, 1) +
             pick(1 << 52, 1, 1))
        p, dnum = pick(1 << 50, 1, -1) + pick(1 << 60, 1, -1) + pick(1 << 58, 1, 1), 3
    elif kind == "wide":    # moduli up to 2^61 (whole-word conversions)
        q = pick(1 << 61, 1, -1) + pick(1 << 50, 2, -1) + pick(1 << 60, 1, 1) + pick(1 << 40, 1, 1)
        p, dnum = pick(1 << 61, 2, -1), 3
    elif kind == "long":    # one digit of sixteen primes, fifteen special primes
        q = pick(1 << 60, 1, -1) + pick(1 << 50, 15, -1)
        p, dnum = pick(1 << 60, 15, -1), 1
    else:                   # "many": one prime a digit
        q = pick(1 << 60, 1, -1) + pick(1 << 50, 11, 1)
        p, dnum = pick(1 << 60, 1, -1), 12
    return dict(name=f"{kind}/{log_n}", log_n=log_n, n=1 << log_n, q=q, p=p, dnum=dnum,
                scale=2.0 ** 40)


def _residues(mods, n, kind, seed):
    if kind == "uniform":
        return S.uniform_residues(mods, n, seed, 2)
    out = np.empty((2, len(mods), n), dtype=np.uint64)
    for i, q in enumerate(mods):
        out[:, i] = q - 1 if kind == "top" else np.where(np.arange(n) % 2, q // 2, q // 2 + 1)
    return out


@pytest.mark.parametrize("kind,log_n", [("edges", 11), ("edges", 14), ("edges", 15), ("edges", 16),
                                        ("edges", 17), ("wide", 12), ("wide", 15), ("long", 12),
                                        ("many", 13)])
def test_mixed_moduli_match_oracle(kind, log_n):
    prm = _params(kind, log_n)
    o, ctx = O.Oracle(prm), H.Context.from_params(prm)
    sk, s_o = ctx.keygen_secret(1), o.keygen_secret(1)
    step = 3
    g = o.galois_element(step)
    gks, gko = ctx.keygen_rotation(sk, [step], 5), {g: o.keygen_galois(s_o, g, 5)}
    rlk, rlk_o = ctx.keygen_relin(sk, 7), o.keygen_relin(s_o, 7)
    assert np.array_equal(ctx.switch_key_export(rlk), rlk_o)
    assert np.array_equal(ctx.switch_key_export(ctx.switch_key_import(rlk_o)), rlk_o)
    levels = sorted({0, 1, o.L // 2, o.L - 1}) if log_n < 15 else sorted({0, o.L - 1})
    for level in levels:
        for i, values in enumerate(("uniform", "top", "middle")):
            r = _residues(o.qmods(level), o.n, values, 60 + level)
            ct, ct_o = ctx.ciphertext_import(r, level, 2.0 ** 40), O.Ciphertext(r, level, 2.0 ** 40)
            same = lambda x, y, what: np.testing.assert_array_equal(
                ctx.ciphertext_export(x)[0], y.polys, f"{what}, level {level}, {values}")
            same(ct, ct_o, "import and export")
            same(ctx.rotate(ct, step, gks), o.rotate(ct_o, step, gko), "rotate")
            if i:
                continue
            many = ctx.rotate_many([ct] * 1 + [ctx.ciphertext_import(r, level, 2.0 ** 40)
                                               for _ in range(6)], step, gks)
            for y in many:
                same(y, o.rotate(ct_o, step, gko), "rotate_many")
            same(ctx.rotate_hoisted(ct, [step], gks)[0],
                 o.rotate_hoisted(ct_o, [step], gko)[0], "rotate_hoisted")
            t, t_o = ctx.mul(ct, ct), o.tensor(ct_o, ct_o)
            same(ctx.relinearize(t, rlk), o.relinearize(t_o, rlk_o), "relinearize")
            if level:
                same(ctx.rescale(ct), o.rescale(ct_o), "rescale")
                same(ctx.rescale(t), o.rescale(t_o), "rescale of three parts")


@pytest.mark.parametrize("name,level,count", [("tiny", 2, 1), ("mix15", 11, 3), ("mix15", 0, 2),
                                              ("vital", 23, 1), ("vital", 12, 9)])
def test_rotations_in_place_match_copies(name, level, count):
    """A rotation that writes its own input: the last launch reads both parts
    through the automorphism while other workgroups write them."""
    prm = S.params(name)
    ctx = H.Context.from_params(prm)
    sk = ctx.keygen_secret(1)
    steps = [1, 7, ctx.n_slots - 1]
    gks = ctx.keygen_rotation(sk, steps, 5)
    mods = prm["q"][: level + 1]
    for rep, step in enumerate(steps):
        rs = [S.uniform_residues(mods, ctx.n, 100 * rep + i, 2) for i in range(count)]
        cts = [ctx.ciphertext_import(r, level, prm["scale"]) for r in rs]
        want = [ctx.ciphertext_export(ctx.rotate(c, step, gks))[0] for c in cts]
        if count == 1:
            ctx.rotate(cts[0], step, gks, out=cts[0])
        else:
            ctx.rotate_many(cts, step, gks, outs=cts)
        for c, w in zip(cts, want):
            np.testing.assert_array_equal(ctx.ciphertext_export(c)[0], w)


@pytest.mark.parametrize("kind,level,count", [("specials", 10, 12), ("chain", 11, 16)])
def test_pairs_across_2_60_match_oracle(kind, level, count):
    """Launches large enough to convert two targets in a workgroup, where the
    integer moduli of a pair lie on either side of 2^60: the last q and the
    first special prime of the ModUp, and two of the q chain in the ModDown."""
    log_n, two_n, taken = 15, 2 << 15, set()
    low = _primes(two_n, 1 << 55, 12, taken, -1)
    high = _primes(two_n, 1 << 61, 4, taken, -1)
    if kind == "specials":   # digits 0 and 1 pair (q_10, p_0)
        q, p, dnum = low, high, 3
    else:                    # the ModUp's targets are special primes alone
        q = [low[0], high[0], low[1], high[1]] + low[2:10]
        p, dnum = _primes(two_n, 1 << 59, 4, taken, -1), 1
    prm = dict(name=f"pairs/{kind}", log_n=log_n, n=1 << log_n, q=q, p=p, dnum=dnum,
               scale=2.0 ** 40)
    o, ctx = O.Oracle(prm), H.Context.from_params(prm)
    sk, s_o = ctx.keygen_secret(1), o.keygen_secret(1)
    step = 3
    g = o.galois_element(step)
    gks, gko = ctx.keygen_rotation(sk, [step], 5), {g: o.keygen_galois(s_o, g, 5)}
    for values in ("uniform", "top"):
        r = _residues(o.qmods(level), o.n, values, 70 + level)
        want = o.rotate(O.Ciphertext(r, level, 2.0 ** 40), step, gko).polys
        cts = [ctx.ciphertext_import(r, level, 2.0 ** 40) for _ in range(count)]
        for y in ctx.rotate_many(cts, step, gks):
            np.testing.assert_array_equal(ctx.ciphertext_export(y)[0], want, f"{kind}, {values}")


@pytest.mark.parametrize("name,level,count,together",
                         [("edge11", 0, 1, True), ("edge11", 2, 7, True), ("gest12", 11, 1, True),
                          ("gest12", 11, 16, True), ("mid14", 7, 2, True), ("mid14", 7, 3, False),
                          ("mix15", 11, 1, True), ("mix15", 11, 2, False),
                          ("edge17", 0, 1, False)])
def test_small_switches_match_oracle(name, level, count, together):
    """Switches whose tiles all run at once take their key products in one
    launch and the tail by itself; on either side of that line rotations (into
    other ciphertexts and in place) and relinearizations are bit-exact."""
    if name == "mid14":
        taken = set()
        q = _primes(2 << 14, 1 << 60, 1, taken, -1) + _primes(2 << 14, 1 << 50, 7, taken, -1)
        prm = dict(name=name, log_n=14, n=1 << 14, q=q, dnum=3, scale=2.0 ** 40,
                   p=_primes(2 << 14, 1 << 60, 3, taken, -1))
    else:
        prm = S.params(name)
    o, ctx = O.Oracle(prm), H.Context.from_params(prm)
    sk, s_o = ctx.keygen_secret(1), o.keygen_secret(1)
    step = 5
    g = o.galois_element(step)
    gks, gko = ctx.keygen_rotation(sk, [step], 5), {g: o.keygen_galois(s_o, g, 5)}
    rlk, rlk_o = ctx.keygen_relin(sk, 7), o.keygen_relin(s_o, 7)
    rs = [S.uniform_residues(o.qmods(level), o.n, 90 + i, 2) for i in range(count)]
    cts = [ctx.ciphertext_import(r, level, 2.0 ** 40) for r in rs]
    cts_o = [O.Ciphertext(r, level, 2.0 ** 40) for r in rs]
    same = lambda got, want, what: [
        np.testing.assert_array_equal(ctx.ciphertext_export(x)[0], y.polys, what)
        for x, y in zip(got, want)]
    outs = [ctx.ciphertext() for _ in cts]
    ctx.trace(True)
    ctx.rotate_many(cts, step, gks, outs=outs)
    names = [r[0] for r in ctx.trace_read()]
    ctx.trace(False)
    last = "ks_moddown_tail" if together else "ks_inner_tail"
    assert names[-1] == last and names.count("ks_contig_inner") == 1, names
    want = [o.rotate(c, step, gko) for c in cts_o]
    same(outs, want, "rotate_many")
    prods = [ctx.mul(c, c) for c in cts]
    ctx.rotate_many(cts, step, gks, outs=cts)
    same(cts, want, "in place")
    ctx.relinearize_many(prods, rlk, outs=prods)
    same(prods, [o.relinearize(o.tensor(c, c), rlk_o) for c in cts_o], "relinearize in place")


def test_largest_ring_batches_match_oracle():
    """At N = 2^17 large launches too convert one target a workgroup (two take
    LDS that leaves a CU one small workgroup); a batch of rotations is
    bit-exact."""
    taken, two_n = set(), 2 << 17
    q = _primes(two_n, 1 << 60, 1, taken, -1) + _primes(two_n, 1 << 50, 5, taken, -1)
    prm = dict(name="batch17", log_n=17, n=1 << 17, q=q, p=_primes(two_n, 1 << 60, 2, taken, -1),
               dnum=3, scale=2.0 ** 40)
    o, ctx = O.Oracle(prm), H.Context.from_params(prm)
    sk, s_o = ctx.keygen_secret(1), o.keygen_secret(1)
    g = o.galois_element(3)
    gks, gko = ctx.keygen_rotation(sk, [3], 5), {g: o.keygen_galois(s_o, g, 5)}
    r = S.uniform_residues(o.qmods(5), o.n, 44, 2)
    cts = [ctx.ciphertext_import(r, 5, 2.0 ** 40) for _ in range(12)]
    outs = [ctx.ciphertext() for _ in cts]
    ctx.trace(True)
    ctx.rotate_many(cts, 3, gks, outs=outs)
    grids = {x[0]: x[1] for x in ctx.trace_read()}
    ctx.trace(False)
    # three digits of two limbs, each to the six other limbs
    assert grids["ks_modup_strided"][1:] == (18, 12), grids
    want = o.rotate(O.Ciphertext(r, 5, 2.0 ** 40), 3, gko).polys
    for y in outs:
        np.testing.assert_array_equal(ctx.ciphertext_export(y)[0], want)


@pytest.mark.parametrize("bits", [50, 57])
def test_largest_ring_splits_match_oracle(bits):
    """Every split of the full transforms at N = 2^17, the 1024-point pass
    among them, on doubles and on integers: imports, products and exports."""
    taken, two_n = set(), 2 << 17
    q = _primes(two_n, 1 << 60, 1, taken, -1) + _primes(two_n, 1 << bits, 2, taken, -1)
    prm = dict(name=f"splits17/{bits}", log_n=17, n=1 << 17, q=q, dnum=3, scale=2.0 ** 40,
               p=_primes(two_n, 1 << 60, 1, taken, -1))
    o, ctx = O.Oracle(prm), H.Context.from_params(prm)
    tried = []
    for i, split in enumerate((9, 8, 10)):
        ctx.set_ntt_split(split)
        tried.append(ctx.ntt_split())
        for values in ("uniform", "top"):
            r = _residues(o.qmods(2), o.n, values, 81 + i)
            ct, ct_o = ctx.ciphertext_import(r, 2, 2.0 ** 40), O.Ciphertext(r, 2, 2.0 ** 40)
            np.testing.assert_array_equal(ctx.ciphertext_export(ct)[0], r)
            np.testing.assert_array_equal(ctx.ciphertext_export(ctx.mul(ct, ct))[0],
                                          o.tensor(ct_o, ct_o).polys, f"{split}, {values}")
    assert tried == [9, 8, 10]
