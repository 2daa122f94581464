"""The calls that a program serving encrypted decode steps makes, as cases for timing and comparison.

Every case goes through the public binding (paper_2602_11470_amd.binding).  A program keeps for its lifetime: the
context of its ring, its rotation keys, the plans that hold the encoded weights, the rotary-embedding objects.  They
are made once per case here.  What changes from call to call -- the ciphertexts, and with them the encrypted cache --
is made from the seed.

Inputs: the limbs of a ciphertext are uniform residues under their moduli (that is what an encryption under this scheme
looks like without the secret key), so the input ciphertexts are drawn directly as such residues; weights are
N(0, 0.02^2) matrices, encoded by the library.  Client-side calls (encode, encrypt, decrypt, key generation) are
synchronous set-up on host buffers and no part of a served step; they are not timed here.

Every output is a ciphertext: whole 64-bit words, the same for every correct implementation of these calls, so the
tolerance is "exact" throughout, and there is no floating-point output whose distance from 64-bit arithmetic could be
taken.

Cases (op):
  product    x W for an encrypted row and a plaintext matrix (cm_vmm_pt, cm_vmm_pt_multi for several matrices of one
             input, token-batched plans in the prompt phase)
  ctproduct  one ciphertext-ciphertext multiplication: tensor product, relinearisation, rescale
  rotate     one rotation, or several hoisted rotations of one ciphertext
  rope       rotary embedding of one token's queries (tau >= 0) or of a token group (tau = -1)
  qk, sv     query times K cache, scores times V cache, decode phase or a query group of the prompt phase
  step       the attention of one decode step: append the token's key and value, query times K, scores times V
  gqa        grouped-query attention on a cache that stores every KV head once: query times K and scores times V
"""
import math

import torch

from paper_2602_11470_amd import binding as B
from paper_2602_11470_amd import inputs

# ring degree, ciphertext primes, special primes, primes per key-switch digit (benchmark configurations 1, 2-4 and 5)
RINGS = {"4096: 5+1": (4096, 5, 1, 1), "65536: 24+4": (65536, 24, 4, 4), "65536: 36+6": (65536, 36, 6, 6)}
BIG = "65536: 24+4"
FORMS = {"plain": {}, "raised": {"raised_sums": True}, "direct": {"direct_giants": True}, "unrolled": {"unrolled_ladders": True}}


def _product(name, ring, d_in, d_out, level, form, count=1, tokens=False):
    return dict(name=name, op="product", ring=ring, d_in=d_in, d_out=d_out, level=level, form=form, count=count, tokens=tokens)


def _attention(name, op, heads, dim, level, context, index, shared, group=False, unrolled=True):
    return dict(name=name, op=op, ring=BIG, heads=heads, dim=dim, level=level, context=context, index=index, shared=shared,
                group=group, unrolled=unrolled)


def listed():
    return [
        # the smallest call: a 64 x 64 product on the small ring, Algorithm 1 as printed (what smoke() runs)
        _product("product_64_small_ring", "4096: 5+1", 64, 64, 4, "plain"),
        # one 4096 x 4096 projection, input at the top level, whole product in the extended basis (bench.py's step)
        _product("product_4096_top", BIG, 4096, 4096, 23, "unrolled"),
        # the same projection at the level the paper runs it at
        _product("product_4096_low", BIG, 4096, 4096, 4, "unrolled"),
        # MLP down projection near the end of the modulus chain
        _product("product_mlp_down_low", BIG, 16384, 4096, 3, "unrolled"),
        # q / k / v projections of one token of a 2048-wide model, in the middle of the chain
        _product("product_qkv_2048_mid", BIG, 2048, 2048, 13, "unrolled", count=3),
        # prompt phase: a group of 32 tokens against a 1024-wide projection
        _product("product_tokens_1024", BIG, 1024, 1024, 9, "direct", tokens=True),
        # ciphertext-ciphertext multiplication at the paper's middle level
        dict(name="ctproduct_mid", op="ctproduct", ring=BIG, level=13),
        # rotary embedding of one token's queries (32 heads of 128 dims) at the paper's level
        dict(name="rope_low", op="rope", ring=BIG, heads=32, dim=128, level=3, tau=5),
        # attention of one decode step at the paper's level, 1000 cached tokens, cache with the key index
        _attention("step_low", "step", 32, 128, 3, 1000, True, 1),
        # query times K without the index: copy mask before the sum over the dims
        _attention("qk_mid", "qk", 32, 128, 12, 1000, False, 128),
        # scores times V with the cache at its highest level
        _attention("sv_top", "sv", 32, 128, 22, 1024, False, 1),
        # grouped-query attention: 8 KV heads, 4 query heads each, 2500 cached tokens, key index
        dict(name="gqa_mid", op="gqa", ring=BIG, heads=8, dim=128, group=4, level=9, context=2500, index=True),
    ]


def draw(rng):
    def logpick(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["small", "product", "product", "tokens", "ctproduct", "rotate", "rope", "qk", "sv", "step", "gqa"])
    if op == "small":
        d = 2 ** rng.randint(5, 9)
        a = rng.choice([1, 1, 2, 4])
        i, o = rng.choice([(d, d * a), (d * a, d)])
        return _unnamed(_product("", "4096: 5+1", i, o, rng.randint(2, 4), rng.choice(list(FORMS))))
    if op == "product":
        ring = rng.choice([BIG, BIG, BIG, "65536: 36+6"])
        d = 2 ** rng.randint(8, 12 if ring == BIG else 11)
        a = rng.choice([1, 1, 2, 4])
        i, o = rng.choice([(d, d * a), (d * a, d)])
        top = {8: 23, 9: 23, 10: 23, 11: 23, 12: 23, 13: 9, 14: 4}[int(math.log2(d * a))]
        level = min(top, logpick(1, 23)) if ring == BIG else logpick(4, 35)
        form = rng.choice(["unrolled", "unrolled", "unrolled", "direct", "raised", "plain"])
        count = rng.choice([1, 1, 2, 3]) if d * a <= 2048 and form != "plain" else 1
        return _unnamed(_product("", ring, i, o, level, form, count=count))
    if op == "tokens":
        d = 2 ** rng.randint(7, 10)
        return _unnamed(_product("", BIG, d, d, logpick(1, 9 if d == 1024 else 17), rng.choice(["direct", "raised"]), tokens=True))
    if op == "ctproduct":
        ring = rng.choice([BIG, BIG, "65536: 36+6"])
        return dict(op=op, ring=ring, level=rng.randint(1, 23 if ring == BIG else 35))
    if op == "rotate":
        return dict(op=op, ring=BIG, level=rng.randint(1, 23), steps=rng.choice([1, 1, 3, 7, 11]), first=rng.randint(1, 4000))
    if op == "rope":
        heads, dim = rng.choice([(32, 128), (32, 64), (12, 64), (8, 128)])
        return dict(op=op, ring=BIG, heads=heads, dim=dim, level=logpick(1, 23), tau=rng.choice([0, 5, 7, -1]))
    heads, dim = rng.choice([(32, 128), (32, 64), (12, 64)])
    room = 32768 // (1 << (heads - 1).bit_length())                     # tokens one cache holds
    context = min(room, logpick(16, 2048))
    if op == "gqa":
        return dict(op="gqa", ring=BIG, heads=8, dim=128, group=rng.choice([2, 4]), level=rng.randint(4, 9), context=logpick(64, 4000),
                    index=True)
    if op == "qk":
        index = rng.random() < 0.4
        shared = 1 if index else rng.choice([dim, dim, dim // 8])
        return _unnamed(_attention("", "qk", heads, dim, logpick(2, 12), min(context, 1024), index, shared, group=rng.random() < 0.3))
    if op == "sv":
        return _unnamed(_attention("", "sv", heads, dim, logpick(2, 22), context, False, 1, group=rng.random() < 0.3,
                                   unrolled=rng.random() < 0.8))
    return _unnamed(_attention("", "step", heads, dim, logpick(2, 12), context, True, 1))


def _unnamed(c):
    c.pop("name", None)
    return c


# ---- what a program keeps ----------------------------------------------------------------------------------
_contexts = {}
_kept = {}            # handles of the case in hand: one case at a time


def _context(ring):
    if ring not in _contexts:
        n, n_q, n_p, _ = RINGS[ring]
        _contexts[ring] = B.config1() if n == 4096 else B.llama_ring(n_q, n_p)
    return _contexts[ring]


def _keep(case, make):
    key = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if key not in _kept:
        _kept.clear()
        _kept[key] = make()
    return _kept[key]


def _keys(ctx, steps, relin):
    return ctx.keygen_rotations(ctx.keygen_secret(1), sorted(set(steps)), 2, with_relin=relin)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _ciphertext(ctx, level, gen, ct=None):
    ct = ct or B.Ct(ctx, level)
    limbs = ct.buf[: 2 * (level + 1) * ctx.n].view(2, level + 1, ctx.n)
    for i, q in enumerate(ctx.moduli()[: level + 1]):
        limbs[:, i].random_(0, int(q), generator=gen)
    ct.d = B.cm_ct(ct.buf.data_ptr(), level, 2, ctx.scale)
    return ct


def _words(ct):
    return ct.buf[: ct.ncomp * (ct.level + 1) * ct.ctx.n]


def _cache(case, ctx, gen, level):
    dim, index = case["dim"], case["index"]
    kv = ctx.kv_create(case["heads"], dim, level, r_i=max(1, dim // 8), unrolled_ladders=case.get("unrolled", True),
                       shared_dims=case.get("shared", 1), key_index=index)
    t = ctx.S // ((1 << (case["heads"] - 1).bit_length()) * dim)
    one = B.Ct(ctx, level)
    op = case["op"]
    for c in range(-(-case["context"] // t) if not index or op == "step" else 0):
        kv.load(B.CM_QK, c, _ciphertext(ctx, level, gen, one))
    for k in range(dim if op != "qk" else 0):
        kv.load(B.CM_SV, k, _ciphertext(ctx, level, gen, one))
    for k in range(dim if index else 0):
        kv.load(B.CM_KV_INDEX, k, _ciphertext(ctx, level, gen, one))
    kv.set_tokens(case["context"])
    return kv


def prepare(case, seed):
    ctx, op, gen, level = _context(case["ring"]), case["op"], _gen(seed), case.get("level")
    s = dict(case=case, ctx=ctx)
    if op == "product":
        def make():
            kw = dict(level=level, token_batch=case["tokens"], **FORMS[case["form"]])
            plans = [ctx.vmm_plan(case["d_in"], case["d_out"], W=inputs.vmm_inputs(7 + i, case["d_in"], case["d_out"])[1], **kw)
                     for i in range(case["count"])]
            return plans, _keys(ctx, plans[0].steps(), False)
        s["plans"], s["keys"] = _keep(case, make)
        s["x"] = _ciphertext(ctx, level, gen)
        s["y"] = [B.Ct(ctx, level - 1) for _ in s["plans"]]
    elif op == "ctproduct":
        s["keys"] = _keep(case, lambda: _keys(ctx, [], True))
        s["x"], s["y"] = _ciphertext(ctx, level, gen), _ciphertext(ctx, level, gen)
    elif op == "rotate":
        s["steps"] = [case["first"] + 17 * i for i in range(case["steps"])]
        s["keys"] = _keep(case, lambda: _keys(ctx, s["steps"], False))
        s["x"] = _ciphertext(ctx, level, gen)
    elif op == "rope":
        def make():
            rope = ctx.rope(case["heads"], case["dim"], level, 129, case["tau"])
            return rope, _keys(ctx, rope.steps(), False)
        s["rope"], s["keys"] = _keep(case, make)
        s["x"], s["y"] = _ciphertext(ctx, level, gen), B.Ct(ctx, level - 1)
    elif op == "gqa":
        s["kv"] = _cache(case, ctx, gen, level)
        s["gqa"] = ctx.gqa(s["kv"], case["group"])
        s["keys"] = _keep(case, lambda: _keys(ctx, s["kv"].steps() + s["gqa"].steps(), True))
        s["q"] = _ciphertext(ctx, level + 1, gen)
        s["scores"] = [_ciphertext(ctx, level, gen) for _ in range(case["group"])]
    else:
        s["kv"] = _cache(case, ctx, gen, level)
        s["keys"] = _keep(case, lambda: _keys(ctx, s["kv"].steps(), True))
        s["q"], s["scores"] = _ciphertext(ctx, level, gen), _ciphertext(ctx, level, gen)
        s["k_new"], s["v_new"] = (_ciphertext(ctx, level + 1, gen) for _ in range(2)) if op == "step" else (None, None)
    return s


def run(s):
    case, ctx, keys = s["case"], s["ctx"], s["keys"]
    op = case["op"]
    if op == "product":
        if case["count"] == 1:
            return [_words(ctx.vmm_pt(keys, s["plans"][0], s["x"], out=s["y"][0]))]
        return [_words(y) for y in ctx.vmm_pt_multi(keys, s["plans"], s["x"], outs=s["y"])]
    if op == "ctproduct":
        return _words(ctx.rescale(ctx.relinearize(keys, ctx.mul_ct(s["x"], s["y"]))))
    if op == "rotate":
        if len(s["steps"]) == 1:
            return _words(ctx.rotate(keys, s["x"], s["steps"][0]))
        return [_words(r) for r in ctx.rotate_hoisted(keys, s["x"], s["steps"])]
    if op == "rope":
        return _words(ctx.rope_apply(keys, s["rope"], s["x"], out=s["y"]))
    if op == "gqa":
        scores = ctx.gqa_qk(keys, s["gqa"], s["q"])
        return [_words(c) for c in scores] + [_words(ctx.gqa_sv(keys, s["gqa"], s["scores"]))]
    kv, group = s["kv"], case["group"]
    if op == "qk":
        return _words(ctx.vmm_kv(keys, kv, B.CM_QK_GROUP if group else B.CM_QK, s["q"]))
    if op == "sv":
        return _words(ctx.vmm_kv(keys, kv, B.CM_SV_GROUP if group else B.CM_SV, s["scores"]))
    # one decode step: the new token joins the cache, then the query and the scores meet it (the appended key and value
    # show in the two results).  A pass starts from the same token count, as the next layer's cache would.
    kv.set_tokens(case["context"] - 1)
    kv.append(keys, s["k_new"], s["v_new"])
    return [_words(ctx.vmm_kv(keys, kv, B.CM_QK, s["q"])), _words(ctx.vmm_kv(keys, kv, B.CM_SV, s["scores"]))]


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def _log2(x):
    return max(0, (int(x) - 1).bit_length())


def _runs(steps):
    """Rotations of a rotate-and-add ladder of that many steps, unrolled in runs of up to three."""
    runs = -(-steps // 3)
    return sum(2 ** (steps // runs + (1 if r < steps % runs else 0)) - 1 for r in range(runs))


def _rotations(case):
    """(rotation keys, plaintext products) of one product."""
    S = RINGS[case["ring"]][0] // 2
    d, big = sorted((case["d_in"], case["d_out"]))
    t, tp = S // d, S // big
    pre, red = (tp, t) if case["d_in"] > case["d_out"] else (t, tp)
    if case["tokens"]:
        tp = pre = red = 1
    m = d // tp
    cheap = case["tokens"] or case["form"] != "plain"
    ri = 1 << ((_log2(m) + 1) // 2)
    ri = 2 * ri if cheap and 2 * ri <= m else ri
    ro = m // ri
    count = _runs if case["form"] == "unrolled" else int
    giants = ro - 1 if case["form"] in ("direct", "unrolled") else min(1, ro - 1)
    return count(_log2(pre)) + ri - 1 + giants + count(_log2(red)), m


def work(case):
    n, _, n_p, alpha = RINGS[case["ring"]]
    level, op, w = case["level"], case["op"], 8
    poly = w * n * (level + 1)                                            # one polynomial at the input's level

    def key(lv):                                                          # the stored half of one key at level lv
        return -(-(lv + 1) // alpha) * (lv + 1 + n_p) * w * n

    def switch(lv):                                                       # multiply-adds of one key switch's inner product
        return 2 * 2 * -(-(lv + 1) // alpha) * (lv + 1 + n_p) * n
    if op == "product":
        rot, m = _rotations(case)
        return {"bytes": rot * key(level) + case["count"] * (m * poly + 2 * level * w * n) + 2 * poly,
                "flops": rot * switch(level) + case["count"] * m * 2 * 2 * (level + 1) * n}
    if op == "ctproduct":
        return {"bytes": key(level) + 4 * poly + 2 * level * w * n, "flops": switch(level) + 8 * (level + 1) * n}
    if op == "rotate":
        return {"bytes": case["steps"] * (key(level) + 2 * poly) + 2 * poly, "flops": case["steps"] * switch(level)}
    if op == "rope":
        return {"bytes": 2 * key(level) + 5 * poly + 2 * level * w * n, "flops": 2 * switch(level) + 12 * (level + 1) * n}
    hp, dim = 1 << _log2(case["heads"]), case["dim"]
    t = n // 2 // (hp * dim)
    ri, ro = max(1, dim // 8), dim // max(1, dim // 8)
    res = _runs(_log2(t))
    index, group = case["index"], case.get("group")
    per = 8 * (level + 1) * n                                             # multiply-adds of one tensor product
    sv = {"bytes": (ri - 1 + ro - 1 + 1 + (0 if group else res)) * key(level) + dim * 2 * poly + 4 * poly,
          "flops": (ri + ro + ro + (0 if group else res)) * switch(level) + dim * per}
    if op == "sv":
        return sv
    nk = -(-case["context"] // t)
    if index:
        qk = {"bytes": (ri - 1 + ro - 1 + 1 + (0 if group else _log2(t))) * key(level) + dim * 2 * poly + 4 * poly,
              "flops": (ri + ro + ro + (0 if group else _log2(t))) * switch(level) + dim * per}
    else:
        e2 = _runs(_log2(dim // case["shared"]))
        qk = {"bytes": (case["shared"] - 1 + e2 + 1 + (0 if group else _log2(t))) * key(level) + nk * 2 * poly + 4 * poly,
              "flops": (nk * (1 + e2) + case["shared"]) * switch(level) + nk * per + nk * 2 * 2 * level * n}
    if op == "qk":
        return qk
    if op == "step":
        up = 2 * poly // (level + 1) * (level + 2)
        app = {"bytes": (ri - 1 + ro - 1) * key(level + 1) + 2 * up + (2 * dim + 1) * 4 * poly,
               "flops": (ri + ro) * switch(level + 1) + (2 * dim + 1) * 4 * (level + 2) * n}
        return {k: qk[k] + sv[k] + app[k] for k in ("bytes", "flops")}
    g = case["group"]                                                     # gqa: the keys and the cache once, the products g times
    moves = {"bytes": 4 * (g - 1) * key(level + 1), "flops": 4 * (g - 1) * switch(level + 1)}
    return {"bytes": qk["bytes"] + sv["bytes"] + moves["bytes"] + 2 * g * 2 * poly,
            "flops": g * (qk["flops"] + sv["flops"]) + moves["flops"]}


def tolerance(case):
    return "exact"
