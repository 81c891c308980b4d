"""GPU: the branches of the launch rules, each at the sizes where it can go wrong, device against device or against
plain torch (the parity of the paths themselves with the oracle is test_gpu_parity.py)."""
import pytest
import torch

from paper_2404_15949_amd import corm
from tests import harness

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# kv dtype, G, Hkv, d, P, m, Tcap, position of the first key, thr_scale, holes
SEEDS = [
    ("bf16", 1, 2, 128, 700, 64, 704, 0, 1.0, False),      # one whole block of queries
    ("bf16", 1, 2, 128, 515, 97, 517, 0, 1.0, False),      # tail and rows of no whole piece
    ("bf16", 2, 1, 128, 640, 200, 672, 32, 1.0, False),    # positions shifted by a word; seven workgroups per key block
    ("bf16", 1, 128, 64, 700, 600, 704, 0, 1.0, False),    # one workgroup per key block over 38 tiles: more than the
                                                           # 32 that the boolean ring's histories hold
    ("bf16", 4, 2, 64, 600, 130, 640, 3, 1.0, False),      # positions shifted by no piece
    ("bf16", 8, 1, 64, 300, 48, 320, 0, 1.0, True),        # keys missing: general blocks next to fast ones
    ("f32", 1, 2, 64, 520, 80, 576, 0, 1.0, False),
    ("f32", 2, 2, 128, 333, 100, 352, 0, 1.0, True),       # 32 keys per wave
    ("f32", 8, 1, 128, 400, 33, 448, 32, 1.0, False),
    ("bf16", 2, 2, 128, 512, 64, 512, 0, 0.0, False),      # threshold 0: everything is important
    ("bf16", 2, 2, 128, 512, 64, 512, 0, 1e30, False),     # and one that nothing reaches
    ("bf16", 1, 40, 128, 300, 32, 320, 0, 2.5, False),     # many units with a block that is not whole
    ("bf16", 8, 24, 128, 500, 300, 512, 0, 1.0, False),    # a block is half of the heads of 16 queries; 152 tiles, and the
                                                           # ring's end inside a tile
    ("bf16", 4, 48, 128, 700, 421, 704, 0, 1.0, False),    # a block is all heads of 16 queries
    ("bf16", 2, 96, 64, 900, 770, 960, 0, 1.0, False),     # ... and of 32
    ("f32", 1, 128, 128, 700, 600, 704, 0, 1.0, False),    # blocks of two tiles, runs of 16 blocks
]


@pytest.mark.parametrize("case", range(len(SEEDS)))
def test_seed_decides_by_the_score_on_every_ring(case):
    """Every ring type starts from the same fp32 score of a (query, key) pair and decides by one comparison, so with the
    fp32 ring as the witness the others follow bit for bit: a bf16 ring holds its rounding to nearest even, the
    boolean ring is "score >= c/t", and last_hit is the latest step whose stored score reaches c/t -- whatever way
    (bands of raw logits, thresholds before rounding) the kernel takes to that decision."""
    dtype, G, Hkv, d, P, m, Tcap, first, c, holes = SEEDS[case]
    print("[case]", SEEDS[case], flush=True)
    B, Hq = 2, G * Hkv
    g = torch.Generator(device=DEV).manual_seed(case)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    K = torch.randn(B, Hkv, P, d, device=DEV, generator=g).to(tdt)
    q = torch.randn(B, Hq, m, d, device=DEV, generator=g).to(tdt)
    pos = torch.arange(P, device=DEV)
    if holes:   # drop every 7th key of the first half
        pos = pos[(pos >= P // 2) | (pos % 7 != 3)]
    n = len(pos)
    t_last = P + first
    got = {}
    for ring in ("f32", "bf16", "bit"):
        st = corm.LayerState(B, Hq, Hkv, d, P, Tcap + first, m + 1, 8, dtype, thr_scale=c, device=DEV, score_dtype=ring)
        st.K[:, :, :n] = K[:, :, pos]
        st.pos[:, :, :n] = (pos + first).int()
        st.lens.fill_(n)
        t = torch.full((B,), t_last, dtype=torch.int32, device=DEV)
        st.prefill_seed(q, t, torch.zeros_like(t))      # m < w: nothing is moved
        torch.cuda.synchronize()
        assert int(st.status.item()) == 0
        got[ring] = st
    steps = torch.arange(t_last - m + 1, t_last + 1, device=DEV)
    rows = (steps - 1) % (m + 1)
    seen = (pos + first).view(1, -1) < steps.view(-1, 1)                                   # [m, n]
    score = got["f32"].ring[:, :, rows][..., pos + first]                                  # [B, Hq, m, n]
    # rows are normalized: fp32 sums of at most 700 terms
    total = torch.where(seen, score, 0).double().sum(-1)
    assert (total - 1).abs().max() < 1e-5
    assert torch.equal(got["bf16"].ring[:, :, rows][..., pos + first][..., seen], score.bfloat16()[..., seen])
    thr = torch.tensor(c, dtype=torch.float32, device=DEV) / steps.float()
    for ring, stored in (("f32", score), ("bf16", score.bfloat16().float()), ("bit", score)):
        hit = (stored >= thr.view(-1, 1)) & seen
        want = torch.where(hit, steps.view(-1, 1).int(), 0).amax(2).view(B, Hkv, G, n).amax(2)
        assert torch.equal(got[ring].last_hit[:, :, :n], want), ring
    words = got["bit"].ring[:, :, rows].contiguous()
    bits = (words.unsqueeze(-1) >> torch.arange(32, device=DEV)) & 1
    bits = bits.flatten(-2)[..., pos + first].bool()
    assert torch.equal(bits & seen, (score >= thr.view(-1, 1)) & seen)
    if c == 0.0:
        assert bool((bits | ~seen).all())
    if c == 1.0:
        assert bool(hit.any()) and not bool(hit.all())


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 128)])
@pytest.mark.parametrize("Lcap", [1, 64, 513, 4097, 16384, 16385])
def test_compact_on_both_sides_of_the_slab_limit(dtype, d, Lcap):
    """A unit per kind of mask, at the edges of 64-slot words, of a batch of rows and of the longest unit that one launch could
    hold (by slabs up to 513 slots here, the longer ones by chunks; the rule's own limits and long slabs are the next test);
    the survivors, their metadata and kept_idx against an index operation of torch, exactly."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(Lcap)
    kinds = ["all", "first", "last", "none", "third", "half", "tail", "one"]
    U = len(kinds)
    st = corm.LayerState(1, U, U, d, Lcap, Lcap, 1, 1, dtype, device=DEV, want_masks=True, want_ring=False)
    st.K.copy_(torch.randn(1, U, Lcap, d, device=DEV, generator=g).to(tdt))
    st.V.copy_(torch.randn(1, U, Lcap, d, device=DEV, generator=g).to(tdt))
    st.pos.copy_(torch.arange(Lcap, device=DEV, dtype=torch.int32))
    st.last_hit.copy_(torch.randint(0, 99, (1, U, Lcap), device=DEV, generator=g, dtype=torch.int32))
    lens = [Lcap, Lcap, Lcap, Lcap, Lcap, max(Lcap - 5, 0), Lcap, Lcap // 2]
    st.lens.copy_(torch.tensor([lens], dtype=torch.int32))
    keep = torch.ones(U, Lcap, dtype=torch.bool, device=DEV)
    keep[1, 0] = False
    keep[2, -1] = False
    keep[3] = False
    keep[4] = torch.rand(Lcap, device=DEV, generator=g) < 0.33
    keep[5] = torch.rand(Lcap, device=DEV, generator=g) < 0.5
    keep[6, Lcap - Lcap // 3:] = False
    keep[7, Lcap // 4] = False
    st.keep.copy_(keep.unsqueeze(0))
    before = {k: getattr(st, k).clone() for k in ("K", "V", "pos", "last_hit")}
    print("[case]", dtype, d, Lcap, flush=True)
    corm.corm_compact(st.desc, st.K, st.V, st.pos, st.last_hit, st.lens, st.keep, st.kept_idx, st.workspace)
    torch.cuda.synchronize()
    for u, kind in enumerate(kinds):
        idx = torch.nonzero(keep[u, :lens[u]]).squeeze(1)
        n = len(idx)
        assert int(st.lens[0, u]) == n, kind
        assert torch.equal(st.kept_idx[0, u, :n].long(), idx), kind
        for name, old in before.items():
            assert torch.equal(getattr(st, name)[0, u, :n], old[0, u, idx]), (kind, name)


# kv dtype, d, units, Lcap: both sides of the limits between one launch of slabs and two of chunks (slots of a unit, by
# the walks of the launch; walks; workgroups of very many short units)
COMPACTS = [("bf16", 64, 5, 2816), ("bf16", 64, 5, 2817), ("bf16", 64, 70, 2304), ("bf16", 64, 70, 2305),
            ("bf16", 128, 5, 4352), ("bf16", 128, 5, 4353), ("f32", 64, 64, 3072), ("f32", 64, 64, 3073),
            ("f32", 128, 5, 4352), ("f32", 128, 5, 4353), ("bf16", 128, 383, 4360), ("bf16", 128, 384, 4360),
            ("bf16", 64, 768, 16384), ("bf16", 64, 8, 16384), ("f32", 128, 910, 512), ("f32", 128, 911, 512)]


@pytest.mark.parametrize("case", range(len(COMPACTS)))
def test_compact_on_both_sides_of_the_launch_rule(case):
    """Units of several kinds of mask and length against a stable sort of torch, exactly."""
    dtype, d, U, Lcap = COMPACTS[case]
    print("[case]", COMPACTS[case], flush=True)
    g = torch.Generator(device=DEV).manual_seed(case)
    st = corm.LayerState(1, U, U, d, Lcap, Lcap, 1, 1, dtype, device=DEV, want_masks=True, want_ring=False)
    st.K.copy_(torch.randn(1, U, 1, d, device=DEV, generator=g) + torch.arange(Lcap, device=DEV).view(1, 1, Lcap, 1))
    st.V.copy_(torch.randn(1, U, Lcap, 1, device=DEV, generator=g).expand(1, U, Lcap, d))
    st.pos.copy_(torch.arange(Lcap, device=DEV, dtype=torch.int32))
    st.last_hit.copy_(torch.randint(0, 99, (1, U, Lcap), device=DEV, generator=g, dtype=torch.int32))
    st.lens.copy_(torch.randint(0, Lcap + 1, (1, U), device=DEV, generator=g))
    st.lens[0, ::2] = Lcap
    share = torch.tensor([1.0, 0.5, 0.999, 0.0, 0.97], device=DEV)[torch.arange(U, device=DEV) % 5]
    keep = torch.rand(U, Lcap, device=DEV, generator=g) < share.view(U, 1)
    keep[::7, 0] = False
    st.keep.copy_(keep.unsqueeze(0))
    keep &= torch.arange(Lcap, device=DEV) < st.lens.view(U, 1)
    order = torch.argsort((~keep).to(torch.int8), dim=-1, stable=True)
    n = keep.sum(-1)
    before = {k: getattr(st, k).clone() for k in ("K", "V", "pos", "last_hit")}
    corm.corm_compact(st.desc, st.K, st.V, st.pos, st.last_hit, st.lens, st.keep, st.kept_idx, st.workspace)
    torch.cuda.synchronize()
    assert torch.equal(st.lens.view(U).long(), n)
    kept = torch.arange(Lcap, device=DEV) < n.view(U, 1)
    assert bool(((st.kept_idx[0] == order) | ~kept).all())
    for u in range(U):
        for name, old in before.items():
            assert torch.equal(getattr(st, name)[0, u, :n[u]], old[0, u, order[u, :n[u]]]), (name, u)


def _compaction_time(U, d, Lcap):
    """us per corm_compact that takes the first slot of every unit away."""
    st = corm.LayerState(1, U, U, d, Lcap, Lcap, 1, 1, "bf16", device=DEV, want_masks=True, want_ring=False)
    st.keep.fill_(1)
    st.keep[:, :, 0] = 0
    st.lens.fill_(Lcap)

    def step():
        corm.corm_compact(st.desc, st.K, st.V, st.pos, st.last_hit, st.lens, st.keep, None, st.workspace)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            step()
    best = float("inf")
    for _ in range(5):
        st.lens.fill_(Lcap)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 20)
    return best


@pytest.mark.parametrize("U,d", [(1, 128), (8, 64)])
def test_few_long_units_are_not_left_to_a_few_serial_walks(U, d):
    """The longest units that slabs could compact against units of one slot more, which they cannot: about the same work,
    so about the same time (measured 1.0; by slabs 3.7 and 2.9 times as long)."""
    at, beyond = _compaction_time(U, d, 16384), _compaction_time(U, d, 16385)
    print("[case]", U, d, round(at, 1), round(beyond, 1), flush=True)
    assert at < 1.8 * beyond


# kv dtype, G, Hkv, d, Lcap: few units whose heads are shared by workgroups (1, 2, 4, 8 of them), lengths on both sides
# of a part and of the number of parts one wave folds
ROUTES = [("bf16", 8, 1, 64, 1000), ("f32", 8, 2, 64, 520), ("f32", 4, 3, 128, 700), ("bf16", 4, 40, 64, 900),
          ("f32", 2, 30, 128, 515), ("bf16", 1, 4, 64, 1600), ("bf16", 1, 4, 64, 1601), ("f32", 2, 1, 64, 400),
          # both sides of the workgroups up to which the record launch has a thread per key: 512, with eight heads a unit 768
          ("f32", 1, 128, 64, 1600), ("f32", 1, 129, 64, 1600), ("bf16", 2, 128, 64, 1600), ("f32", 2, 129, 64, 1600),
          ("bf16", 4, 128, 128, 1600), ("bf16", 4, 129, 64, 1600), ("bf16", 8, 192, 64, 1600), ("bf16", 8, 193, 128, 1600)]


@pytest.mark.parametrize("ring", ["f32", "bit", None])
@pytest.mark.parametrize("case", range(len(ROUTES)))
def test_default_route_of_a_small_launch_equals_torch(case, ring):
    """One step by the route the rules choose against a softmax in float64 on the same stored bits: out, the recorded row and
    last_hit.  out: fp32 sums of at most 1600 terms and a 2^x of about 1 ulp: 1e-5 of the largest element.  A score
    within that of c/t may fall on either side."""
    dtype, G, Hkv, d, Lcap = ROUTES[case]
    print("[case]", ROUTES[case], ring, flush=True)
    B, Hq, tdt = 1, G * Hkv, torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(case)
    st = corm.LayerState(B, Hq, Hkv, d, Lcap, Lcap, 4, 4, dtype, device=DEV, want_ring=ring is not None, score_dtype=ring)
    lens = torch.randint(1, Lcap, (B, Hkv), device=DEV, generator=g, dtype=torch.int32)
    lens.view(-1)[0] = Lcap - 1
    st.K.copy_(torch.randn(B, Hkv, Lcap, d, device=DEV, generator=g).to(tdt))
    st.V.copy_(torch.randn(B, Hkv, Lcap, d, device=DEV, generator=g).to(tdt))
    st.pos.copy_(torch.arange(Lcap, device=DEV, dtype=torch.int32))
    st.lens.copy_(lens)
    q = torch.randn(B, Hq, d, device=DEV, generator=g).to(tdt)
    k, v = (torch.randn(B, Hkv, d, device=DEV, generator=g).to(tdt) for _ in range(2))
    t = torch.full((B,), Lcap, dtype=torch.int32, device=DEV)
    st.step_attend(q, k, v, t, t)                       # the window is not full: nothing goes
    torch.cuda.synchronize()
    assert int(st.status.item()) == 0
    for h in range(Hkv):
        n = int(lens[0, h])
        K = torch.cat([st.K[0, h, :n], k[0, h][None]]).double()
        V = torch.cat([st.V[0, h, :n], v[0, h][None]]).double()
        a = torch.softmax(q[0, h * G:(h + 1) * G].double() @ K.t().contiguous() / d ** 0.5, dim=-1)
        want = a @ V
        got = st.out[0, h * G:(h + 1) * G].double()
        assert ((got - want).abs().amax(1) <= 1e-5 * want.abs().amax(1)).all()
        assert torch.equal(st.K[0, h, n], k[0, h]) and torch.equal(st.V[0, h, n], v[0, h])
        # (without a ring on a bf16 cache the score is compared as a bf16 ring would hold it: half an ulp, 2^-8 at most)
        clear = (a * Lcap - 1).abs() > (2.0 ** -8 if ring is None and dtype == "bf16" else 0) + 1e-4
        hits = a * Lcap >= 1
        pos = torch.cat([torch.arange(n, device=DEV), torch.tensor([Lcap - 1], device=DEV)])
        assert torch.equal(st.pos[0, h, :n + 1].long(), pos)
        sure = clear.all(0)
        assert torch.equal((st.last_hit[0, h, :n + 1] == Lcap)[sure], hits.any(0)[sure])
        if ring == "f32":
            row = st.ring[0, h * G:(h + 1) * G, (Lcap - 1) % 4][:, pos].double()
            assert ((row - a).abs() <= 1e-5 * a + 1e-9).all()
        if ring == "bit":
            words = st.ring[0, h * G:(h + 1) * G, (Lcap - 1) % 4]
            bits = ((words[:, pos // 32] >> (pos % 32)) & 1).bool()
            assert torch.equal(bits[clear], hits[clear])


@pytest.mark.parametrize("Lcap", [600, 16500])
@pytest.mark.parametrize("poison", ["init", 0x7f, 0xff, "random"])
def test_evict_on_a_workspace_that_no_attend_filled(Lcap, poison):
    """corm_step_evict reads a unit's slots and survivors from the workspace.  After corm_workspace_init there are none;
    whatever else the workspace holds, only the call's own units are written (units in front of and behind them are
    the witnesses) and lens stays within its range."""
    print("[case]", Lcap, poison, flush=True)
    U, d = 3, 64
    st = corm.LayerState(1, U, U, d, Lcap, Lcap, 4, 4, "f32", device=DEV, want_ring=False)
    g = torch.Generator(device=DEV).manual_seed(1)
    K, V = (torch.randn(U + 2, Lcap, d, device=DEV, generator=g) for _ in range(2))
    pos, hit, idx = (torch.randint(0, 99, (U + 2, Lcap), device=DEV, generator=g, dtype=torch.int32) for _ in range(3))
    lens = torch.full((U + 2,), Lcap // 2, dtype=torch.int32, device=DEV)
    arrays = [K, V, pos, hit, lens, idx]
    before = [a.clone() for a in arrays]
    if poison == "init":
        st.workspace.fill_(0x7f)
        corm.corm_workspace_init(st.desc, st.workspace)
    elif poison == "random":
        st.workspace.copy_(torch.randint(0, 256, st.workspace.shape, device=DEV, generator=g, dtype=torch.uint8))
    else:
        st.workspace.fill_(poison)
    corm.corm_step_evict(st.desc, K[1:], V[1:], lens[1:], pos[1:], hit[1:], idx[1:], st.workspace)
    torch.cuda.synchronize()
    for a, b in zip(arrays, before):
        assert torch.equal(a[0], b[0]) and torch.equal(a[-1], b[-1])
    assert ((lens[1:-1] >= 0) & (lens[1:-1] <= Lcap)).all()
    if poison == "init":
        assert (lens[1:-1] == 0).all()
        assert torch.equal(K, before[0]) and torch.equal(V, before[1])


def _bit_hits(ring, rows, pos):
    """Recorded booleans [B, Hq, len(rows), len(pos)] of a boolean ring."""
    words = ring[:, :, rows].contiguous()
    bits = (words.unsqueeze(-1) >> torch.arange(32, device=DEV)) & 1
    return bits.flatten(-2)[..., pos].bool()


POISON = {"nan": (0x7fc0, 0x7fc00000), "-nan": (0xffc0, 0xffc00000), "inf": (0x7f80, 0x7f800000), "-inf": (0xff80, 0xff800000)}


@pytest.mark.parametrize("c", [0.0, 1.0])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
def test_seed_with_logits_that_are_not_finite(dtype, d, c):
    """A key with NaN of either sign, or an infinity of either sign, in one element: Def. 3.1 compares scores, so a score
    that is not a number is minor and one that is 0 reaches the threshold 0, on every ring type and whichever way the
    kernel decides.  The scores an fp32 ring holds are the witness; comparisons of them are exact.  Keys in front of the
    first tail query take the kernel's fast blocks (with a bf16 ring only those whose rows are finite), those among the tail its general
    ones: both get a poisoned key."""
    print("[case]", dtype, d, c, flush=True)
    P, m, Hkv = 600, 80, len(POISON)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d)
    K = torch.randn(1, Hkv, P, d, device=DEV, generator=g).to(tdt)
    q = torch.randn(1, Hkv, m, d, device=DEV, generator=g).to(tdt)
    for h, (bf16, f32) in enumerate(POISON.values()):
        raw = K.view(torch.int32 if dtype == "f32" else torch.int16)
        value = f32 if dtype == "f32" else bf16
        raw[0, h, 5, 0] = raw[0, h, P - 9, 0] = value - (1 << (32 if dtype == "f32" else 16)) if value >> (31 if dtype == "f32" else 15) else value
    steps = torch.arange(P - m + 1, P + 1, device=DEV)
    rows, pos = (steps - 1) % (m + 1), torch.arange(P, device=DEV)
    seen = pos.view(1, -1) < steps.view(-1, 1)
    got = {}
    for ring in ("f32", "bf16", "bit"):
        st = corm.LayerState(1, Hkv, Hkv, d, P, P, m + 1, 8, dtype, thr_scale=c, device=DEV, score_dtype=ring)
        st.preload(K, torch.zeros_like(K))
        t = torch.full((1,), P, dtype=torch.int32, device=DEV)
        st.prefill_seed(q, t, torch.zeros_like(t))
        torch.cuda.synchronize()
        got[ring] = st
    score = got["f32"].ring[:, :, rows][..., pos]
    thr = torch.tensor(c, dtype=torch.float32, device=DEV) / steps.float()
    wrong = []
    for ring, stored in (("f32", score), ("bf16", score.bfloat16().float()), ("bit", score)):
        hit = (stored >= thr.view(-1, 1)) & seen
        want = torch.where(hit, steps.view(-1, 1).int(), 0).amax(2)
        for h, kind in enumerate(POISON):
            if not torch.equal(got[ring].last_hit[:, h], want[:, h]):
                wrong.append((ring, kind, "last_hit"))
            if ring == "bit" and not torch.equal(_bit_hits(got[ring].ring, rows, pos)[:, h] & seen, hit[:, h]):
                wrong.append((ring, kind, "bits"))
    assert not wrong, wrong


# kv dtype, d, query heads per KV head, m: tails that end in a fast block of the kernel (64 queries; of fp32 rows of 512 bytes 32, over all heads)
LASTS = [("bf16", 128, 1, 64), ("bf16", 128, 1, 128), ("bf16", 64, 1, 64), ("f32", 64, 1, 64), ("f32", 128, 1, 32), ("f32", 128, 1, 64),
         ("bf16", 128, 2, 64), ("bf16", 64, 4, 16)]


@pytest.mark.parametrize("ring", ["f32", "bf16", "bit", None])
@pytest.mark.parametrize("case", range(len(LASTS)))
def test_seed_latest_hit_of_rows_that_are_not_finite(case, ring):
    """A key with +inf in one element makes the logit of a query +inf or -inf by that element's sign, and a row with +inf has no
    finite sum: its scores are 0, that of the key itself no number; the others are finite rows with a score of 0 for the key.  At
    threshold 0 every other key's latest hit is therefore the last step, whichever of the last 16 queries and those 16 before them have such a row;
    the key's own is the last step one of whose heads has a finite row."""
    dtype, d, G, m = LASTS[case]
    print("[case]", LASTS[case], ring, flush=True)
    P, Hkv = 600, 8
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(case)
    K = torch.randn(1, Hkv, P, d, device=DEV, generator=g).to(tdt)
    K[:, :, 5, 0] = float("inf")
    q = torch.randn(1, G * Hkv, m, d, device=DEV, generator=g).to(tdt)
    up = torch.rand(1, Hkv, G, m, device=DEV, generator=g) < 0.5
    up[:, ::2, :, -16:] = True            # the last 16 queries have such rows, those before them do not
    up[:, ::2, :, :-16] = False
    up[:, 1] = torch.arange(m, device=DEV) % 2 == 1
    q[..., 0] = torch.where(up.view(1, G * Hkv, m), 1.0, -1.0).to(tdt)
    st = corm.LayerState(1, G * Hkv, Hkv, d, P, 608, m + 1, 8, dtype, thr_scale=0.0, device=DEV, want_ring=ring is not None,
                         score_dtype=ring or "bf16")
    st.preload(K, torch.zeros_like(K))
    t = torch.full((1,), P, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    assert int(st.status.item()) == 0
    want = torch.full((1, Hkv, P), P, dtype=torch.int32, device=DEV)
    steps = torch.arange(P - m + 1, P + 1, device=DEV, dtype=torch.int32)
    want[:, :, 5] = torch.where(~up.all(2), steps, 0).amax(-1)
    assert torch.equal(st.last_hit, want)


@pytest.mark.parametrize("score", ["f32", "bf16", "bit"])
@pytest.mark.parametrize("dtype,d,G", [("bf16", 64, 1), ("f32", 128, 4)])
def test_seed_of_as_many_queries_as_a_call_takes(dtype, d, G, score):
    """65535 groups of 16 queries, each of which attends to one key (its logit is 79 or more above the others: a score of 1 against
    thresholds of 1/2 and up): the latest hits are in the last groups, whose numbers fill 16 bits, and with fp32 rows of four
    heads the queries reach beyond 2^31 bytes."""
    print("[case]", dtype, d, G, score, flush=True)
    m, P = 65535 * 16, 64
    t_last = m + P
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    st = corm.LayerState(1, G, 1, d, P, t_last, m + 1, 8, dtype, thr_scale=0.5 * t_last, device=DEV, want_ring=False, score_dtype=score)
    K = (30.0 * torch.eye(P, d, device=DEV)).to(tdt).view(1, 1, P, d)
    st.preload(K, torch.zeros_like(K))
    j = torch.arange(m, device=DEV)
    key = (7 * j.view(1, m) + 3 * torch.arange(G, device=DEV).view(G, 1)) % P
    q = torch.zeros(1, G, m, d, device=DEV, dtype=tdt).scatter_(3, key.view(1, G, m, 1), 30.0)
    t = torch.full((1,), t_last, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    assert int(st.status.item()) == 0
    want = torch.zeros(P, dtype=torch.int64, device=DEV)
    want.scatter_reduce_(0, key.flatten(), (P + 1 + j).expand(G, m).flatten(), "amax")
    assert bool((want > t_last - 64).all()) and torch.equal(st.last_hit[0, 0].long(), want)


@pytest.mark.parametrize("ring", ["f32", "bf16", "bit"])
def test_seed_with_a_threshold_of_minus_zero(ring):
    """thr_scale = -0.0 passes the descriptor's check (it is not below 0) and is the threshold 0: every key is important to
    every query that sees it."""
    P, m = 300, 32
    g = torch.Generator(device=DEV).manual_seed(3)
    K, q = (torch.randn(1, 2, n, 64, device=DEV, generator=g).bfloat16() for n in (P, m))
    st = corm.LayerState(1, 2, 2, 64, P, P, m + 1, 8, "bf16", thr_scale=-0.0, device=DEV, score_dtype=ring)
    st.preload(K, K)
    t = torch.full((1,), P, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    assert (st.last_hit == P).all()


@pytest.mark.parametrize("P", [256, 300])
def test_seed_bits_next_to_positions_without_a_column(P):
    """Keys at positions the ring has no column for are skipped and flagged; the words that hold the valid positions of the same
    64 slots are those of a ring that was clear before."""
    Tcap, m, d = 225, 16, 64
    g = torch.Generator(device=DEV).manual_seed(P)
    K, q = (torch.randn(1, 2, n, d, device=DEV, generator=g).bfloat16() for n in (P, m))
    got = []
    for before in (0, -1):
        st = corm.LayerState(1, 2, 2, d, P, Tcap, m + 1, 8, "bf16", device=DEV, score_dtype="bit")
        st.preload(K, K)
        st.ring.fill_(before)
        t = torch.full((1,), Tcap, dtype=torch.int32, device=DEV)
        st.prefill_seed(q, t, torch.zeros_like(t))
        torch.cuda.synchronize()
        assert int(st.status.item()) == corm.CORM_DEV_BAD_STEP
        got.append(st)
    steps = torch.arange(Tcap - m + 1, Tcap + 1, device=DEV)
    pos = torch.arange(Tcap, device=DEV)
    seen = pos.view(1, -1) < steps.view(-1, 1)
    a, b = (_bit_hits(st.ring, (steps - 1) % (m + 1), pos) & seen for st in got)
    assert bool(a.any()) and torch.equal(a, b)
    assert torch.equal(got[0].last_hit, got[1].last_hit)


@pytest.mark.parametrize("w,words", [(2044, 262657), (16383, 32770)])
def test_seed_bits_in_a_ring_of_two_gigabytes(w, words):
    """Stores that a lane has no part in go to an offset behind the head's ring, 0x7ffffff0 at most: a ring of just that
    many bytes, and one whose last words lie behind that offset.  Only the tail's rows may change."""
    P, m, t_last, d = 64, 64, 300, 64
    print("[case]", w, words, flush=True)
    g = torch.Generator(device=DEV).manual_seed(5)
    K, q = (torch.randn(1, 1, n, d, device=DEV, generator=g).bfloat16() for n in (P, m))
    st = corm.LayerState(1, 1, 1, d, P, words * 32, w, 8, "bf16", device=DEV, score_dtype="bit")
    st.preload(K, K)
    st.ring.fill_(-1)
    t = torch.full((1,), t_last, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    flat = st.ring.view(w, words)
    steps = torch.arange(t_last - m + 1, t_last + 1, device=DEV)
    rows = (steps - 1) % w
    hits = _bit_hits(st.ring, rows, torch.arange(P, device=DEV))[0, 0]
    assert bool(hits.any()) and not bool(hits.all())
    assert torch.equal(torch.where(hits, steps.view(-1, 1).int(), 0).amax(0), st.last_hit[0, 0])
    flat[rows] = -1
    assert bool((flat == -1).all())


@pytest.mark.parametrize("t_last", [300, 330])   # the ring wraps in the second and in the first block of queries
@pytest.mark.parametrize("ring,Tcap", [("bf16", 12000000), ("f32", 6000000), ("bit", 180000000)])
def test_seed_in_a_ring_beyond_32_bit_offsets(ring, Tcap, t_last):
    """A head's ring of more than 2 GiB, whose fast blocks address the rows of a tile: the same bits as in a short one."""
    P, m, w, d = 160, 90, 97, 128
    print("[case]", ring, t_last, flush=True)
    g = torch.Generator(device=DEV).manual_seed(7)
    K, q = (torch.randn(1, 1, n, d, device=DEV, generator=g).bfloat16() for n in (P, m))
    got = []
    for columns in (Tcap, 512):
        st = corm.LayerState(1, 1, 1, d, P, columns, w, 8, "bf16", device=DEV, score_dtype=ring)
        st.preload(K, K)
        t = torch.full((1,), t_last, dtype=torch.int32, device=DEV)
        st.prefill_seed(q, t, torch.zeros_like(t))
        torch.cuda.synchronize()
        n = P // 32 if ring == "bit" else P
        got.append((st.ring[..., :n].clone(), st.last_hit))
        assert not bool(st.ring[..., n:].any())
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert bool(got[0][1].any())


# kv dtype, G, Hkv, d, P, m, scaled logit of the keys (log2) in the first and in the second half of the prompt
SUM_RANGES = [
    ("bf16", 1, 2, 128, 700, 64, 0, 0),          # few units: a query tile per wave, the keys in segments
    ("bf16", 1, 2, 128, 700, 64, 150, 150),      # references far from 0,
    ("bf16", 1, 2, 64, 700, 64, -150, -150),
    ("bf16", 2, 2, 128, 1300, 40, -150, 150),    # different ones in different segments
    ("bf16", 4, 2, 64, 1300, 33, 150, 3),
    ("bf16", 1, 300, 128, 530, 130, -90, 0),     # more units: four query tiles per wave, two segments
    ("bf16", 1, 300, 64, 530, 70, 0, 0),
    ("f32", 2, 2, 64, 1300, 50, -150, 0),
    ("f32", 1, 2, 128, 700, 90, 150, 150),       # key blocks of 128
    ("f32", 1, 300, 128, 300, 70, 0, 120),
    ("bf16", 1, 600, 128, 530, 130, -150, 150),  # four query tiles per wave, one segment: the reference rises within it,
    ("bf16", 1, 600, 64, 530, 200, 150, -150),   # or stays while the terms vanish
]


@pytest.mark.parametrize("case", range(len(SUM_RANGES)))
def test_seed_sums_over_the_range_of_the_logits(case):
    """The sum of a row is taken against a reference that follows the logits (test_seed_sums_that_the_reference_cannot_follow has
    the rows where it cannot): scores against softmax in 64 bits.  Keys and queries are nearly constant vectors, so the d products of a logit x all have
    its sign: summed in fp32 in any order they carry at most d 2^-24 |x|, the few operations after them 8 2^-24 |x|, and a
    score is e to that."""
    dtype, G, Hkv, d, P, m, lo, hi = SUM_RANGES[case]
    print("[case]", SUM_RANGES[case], flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(case)
    unit = (d ** 0.5 / 1.4426950408889634) / d            # a key of this constant has a scaled logit of 1 with the query 1
    level = torch.where(torch.arange(P, device=DEV) < P // 2, lo, hi).view(1, 1, P, 1)
    K = ((level + torch.randn(1, Hkv, P, 1, device=DEV, generator=g)) * unit +
         0.05 * torch.randn(1, Hkv, P, d, device=DEV, generator=g)).to(tdt)
    q = (1 + 0.05 * torch.randn(1, Hkv * G, m, d, device=DEV, generator=g)).to(tdt)
    st = corm.LayerState(1, Hkv * G, Hkv, d, P, P, m + 1, 8, dtype, device=DEV, score_dtype="f32")
    st.preload(K, torch.zeros_like(K))
    t = torch.full((1,), P, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    steps = torch.arange(P - m + 1, P + 1, device=DEV)
    seen = torch.arange(P, device=DEV).view(1, -1) < steps.view(-1, 1)
    got = st.ring[0][:, (steps - 1) % (m + 1)][..., :P].double()
    for h in range(0, Hkv * G, 7 if Hkv > 8 else 1):
        s = (q[0, h].double() @ K[0, h // G].double().t().contiguous() / d ** 0.5).masked_fill(~seen, float("-inf"))
        want = torch.softmax(s, dim=-1)
        tol = 0.7 * (d + 8) * 2.0 ** -24 * (max(abs(lo), abs(hi)) + 16)   # (log2 units; 16: the spread within a level)
        assert ((got[h] - want).abs() <= tol * want + 1e-30)[seen].all(), h


# kv dtype, G, Hkv, d, P, m, (lane groups, in the first n keys) that differ, their scaled logit (log2), scaled logit of the others, the
# query that is 2^13 times the others, slots without a column.  Key i is lane group i % 16 // 4's.  Few units have one query
# tile per wave, which looks at 64 keys at a time, 600 of them with 9 or more tiles four, which look at 16.
INF = float("inf")
FAR_SUMS = [
    ("bf16", 1, 2, 128, 700, 64, ((0,), 64), -1.2e6, -300, None, 0),       # a lane group's first keys; the keys in segments
    ("bf16", 1, 2, 128, 700, 64, ((1,), 64), -INF, -300, None, 0),
    ("bf16", 2, 2, 64, 1300, 40, ((2, 3), 64), -1.2e6, -300, None, 0),
    ("bf16", 1, 600, 128, 530, 130, ((1,), 16), -1.2e6, -300, None, 0),    # one segment
    ("bf16", 1, 600, 64, 530, 130, ((3,), 16), -INF, -300, None, 0),
    ("bf16", 4, 150, 128, 300, 64, ((0, 2), 16), -INF, -300, None, 0),
    ("f32", 2, 2, 64, 1300, 50, ((0,), 64), -1.2e6, -300, None, 0),
    ("f32", 1, 2, 128, 700, 90, ((1, 2, 3), 64), -INF, -300, None, 0),
    ("bf16", 1, 600, 128, 530, 130, ((0,), 16), -1.2e6, -126, None, 0),    # the group's sum is positive, and not whole
    ("bf16", 1, 2, 128, 700, 64, ((0,), 64), 2e6, -300, None, 0),
    ("bf16", 4, 2, 64, 600, 33, ((0, 1, 2, 3), 64), -INF, 150, None, 0),   # all groups, and more than one block
    ("bf16", 1, 600, 128, 530, 130, ((0, 1, 2, 3), 96), -INF, -300, None, 0),
    ("bf16", 1, 2, 128, 700, 64, ((), 0), 0, 1.5e6, None, 0),              # every row beyond 10^6
    ("f32", 1, 2, 64, 700, 64, ((), 0), 0, -1.5e6, None, 0),
    ("bf16", 1, 600, 128, 530, 130, ((), 0), 0, 300, 21, 0),               # one query of the workgroup beyond it
    ("bf16", 1, 2, 128, 700, 64, ((), 0), 0, -300, 5, 0),
    ("bf16", 1, 2, 128, 700, 64, ((), 0), 0, -300, None, 4),               # the first block is seen in part, and one group
    ("bf16", 1, 600, 64, 530, 130, ((), 0), 0, -300, None, 52),            # sees none of it
    ("f32", 1, 2, 128, 700, 64, ((), 0), 0, -300, None, 61),
]


@pytest.mark.parametrize("ring", ["f32", "bf16", "bit"])
@pytest.mark.parametrize("case", range(len(FAR_SUMS)))
def test_seed_sums_that_the_reference_cannot_follow(case, ring):
    """Rows whose sum cannot be taken in the first walk over the keys, wholly or in one lane group, are walked again against their
    maximum: scores against softmax in 64 bits, rows that sum to 1.  A logit is the sum of two products, exact in fp32 in any
    order; scaling, the difference to the reference and exp2 round once each, at up to 32 + |log2 score| after the difference, and
    the sums of up to 1300 positive terms add less than 100 roundings: together (132 + |log2 score|) 2^-24, in exp2 times ln 2."""
    dtype, G, Hkv, d, P, m, (groups, n), special, others, big, gone = FAR_SUMS[case]
    print("[case]", FAR_SUMS[case], ring, flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(case)
    scale = float(1 / torch.tensor(float(d)).sqrt() * torch.tensor(1.4426950408889634))      # (in fp32, as the library does)
    K = torch.zeros(1, Hkv, P, d, device=DEV)
    K[..., 0] = others / scale
    step = 5 if abs(others) > 1e5 else 0.5
    K[..., 1] = torch.randint(-4, 5, (1, Hkv, P), device=DEV, generator=g) * step
    slots = [i for i in range(n) if i % 16 // 4 in groups]
    K[:, :, slots, 0] = special / scale
    K[:, :, slots, 1] = 0
    K = K.to(torch.bfloat16).to(tdt)                     # (both elements exact in bf16, their sum in fp32)
    q = torch.zeros(1, Hkv * G, m, d, device=DEV)
    q[..., :2] = 1
    if big is not None:
        q[:, :, big] *= 2 ** 13
    q = q.to(tdt)
    st = corm.LayerState(1, Hkv * G, Hkv, d, P, P, m + 1, 8, dtype, device=DEV, score_dtype=ring)
    st.preload(K, torch.zeros_like(K))
    pos = torch.arange(P, device=DEV) - gone             # the first `gone` lie in front of the ring's columns
    st.pos[:] = pos.int()
    t_last = P - gone
    t = torch.full((1,), t_last, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    assert int(st.status.item()) == (corm.CORM_DEV_BAD_STEP if gone else 0)
    steps = torch.arange(t_last - m + 1, t_last + 1, device=DEV)
    rows = (steps - 1) % (m + 1)
    seen = (pos.view(1, -1) < steps.view(-1, 1)) & (pos >= 0)
    for h in range(0, Hkv * G, 37 if Hkv > 8 else 1):
        raw = K[0, h // G, :, 0].double() + K[0, h // G, :, 1].double()
        x = (q[0, h, :, :1].double() * raw * scale).masked_fill(~seen, -INF)
        z = torch.exp2(x - x.amax(-1, keepdim=True))
        want = z / z.sum(-1, keepdim=True)
        tol = 0.7 * 2.0 ** -24 * (132 - torch.log2(want.clamp(min=1e-36))) * want
        thr = 1.0 / steps.double().view(-1, 1)
        if ring == "bit":
            hits = _bit_hits(st.ring, rows, pos.clamp(min=0))[0, h]
            sure = seen & ((want - thr).abs() > tol)
            assert torch.equal(hits[sure], (want >= thr)[sure]), h
            continue
        got = st.ring[0, h][rows][:, :P - gone].double()
        want, tol, seen_h = (a[:, gone:] for a in (want, tol, seen))
        if ring == "bf16":
            tol = tol * 1.01 + 2.0 ** -8 * want
        else:
            assert ((torch.where(seen_h, got, 0.0).sum(-1) - 1).abs() <= 200 * 2.0 ** -24).all(), h
        assert ((got - want).abs() <= tol + 2e-36)[seen_h].all(), h


# kv dtype, G, units, d, P, m: so many that the keys of a query block stay in one segment
LONG_SUMS = [("bf16", 4, 768, 64, 8192, 64), ("bf16", 4, 768, 64, 16300, 64), ("bf16", 4, 768, 128, 2048, 64), ("f32", 4, 224, 64, 32768, 64)]


@pytest.mark.parametrize("sink", [0, 24])
@pytest.mark.parametrize("case", range(len(LONG_SUMS)))
def test_seed_sums_of_long_rows(case, sink):
    """The sum of a long row behind a few keys that hold nearly all of it: every score is its term over that sum, so the row
    sums to 1 within the sum's roundings.  A lane adds up the tiles of 256 keys and then those sums, a chain of 16 + P / 256
    roundings at most; 20 more for terms, quotient and the four lane groups."""
    dtype, G, units, d, P, m = LONG_SUMS[case]
    print("[case]", LONG_SUMS[case], sink, flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(case)
    K = torch.randn(1, units, P, d, device=DEV, generator=g, dtype=tdt) * 0.9
    K[..., 0] = 0
    K[:, :, :16, 0] = sink / (1.4426950408889634 / d ** 0.5)
    q = torch.randn(1, units * G, m, d, device=DEV, generator=g).to(tdt)
    q[..., 0] = 1
    st = corm.LayerState(1, units * G, units, d, P, P, m + 1, 8, dtype, device=DEV, score_dtype="f32")
    st.preload(K, K)
    t = torch.full((1,), P, dtype=torch.int32, device=DEV)
    st.prefill_seed(q, t, torch.zeros_like(t))
    torch.cuda.synchronize()
    steps = torch.arange(P - m + 1, P + 1, device=DEV)
    seen = torch.arange(P, device=DEV).view(1, -1) < steps.view(-1, 1)
    worst = 0.0
    for h in range(0, units * G, 97):
        row = torch.where(seen, st.ring[0, h][(steps - 1) % (m + 1)], 0.0)
        worst = max(worst, float((row.double().sum(-1) - 1).abs().max()))
    print("[worst]", worst, flush=True)
    assert worst <= (36 + P / 256) * 2.0 ** -24


# kv dtype, G, Hkv, d, Lcap, ring, w (two sequences each): up to the limits of the one-launch step
SMALL = [
    ("f32", 1, 4, 64, 640, "f32", 8), ("f32", 1, 3, 64, 576, "bit", 8), ("f32", 2, 2, 128, 208, None, 4), ("f32", 4, 1, 128, 80, "bf16", 4),
    ("bf16", 1, 2, 128, 640, "bf16", 8), ("bf16", 1, 5, 64, 1024, "bit", 6), ("bf16", 2, 2, 64, 832, "bf16", 8), ("bf16", 4, 2, 64, 320, "f32", 5),
    ("bf16", 4, 3, 64, 300, "bit", 8), ("bf16", 1, 100, 128, 1024, None, 8), ("f32", 2, 1, 64, 65, "bf16", 3), ("bf16", 1, 1, 128, 1, "bit", 2),
    ("f32", 1, 2, 64, 64, "f32", 3), ("f32", 1, 2, 128, 320, "bit", 8), ("f32", 2, 3, 64, 416, "f32", 6), ("f32", 4, 2, 64, 160, "bf16", 6),
    ("f32", 1, 100, 64, 1024, "bf16", 8), ("bf16", 2, 100, 64, 1023, "bit", 8), ("bf16", 4, 100, 64, 1024, "f32", 5), ("f32", 1, 100, 128, 512, "bf16", 6),
    ("f32", 2, 100, 128, 408, "bit", 8), ("f32", 4, 100, 128, 256, "f32", 4),
]

# and beyond one of them
NOT_SMALL = [
    ("f32", 1, 4, 64, 641), ("f32", 2, 2, 128, 209), ("f32", 4, 1, 128, 81), ("bf16", 1, 2, 128, 641), ("bf16", 1, 5, 64, 1025),
    ("bf16", 2, 2, 64, 833), ("bf16", 4, 2, 64, 321), ("f32", 1, 100, 64, 1025), ("f32", 1, 100, 128, 513), ("f32", 2, 100, 128, 409),
    ("f32", 4, 100, 128, 257), ("f32", 8, 1, 64, 32), ("bf16", 8, 2, 64, 64), ("bf16", 2, 1, 128, 65), ("bf16", 4, 1, 128, 64),
    ("f32", 1, 128, 64, 64),
]


def _small_states(case, n):
    """n layers in the same state (units that are empty, full or hold an invalid length, a position without a column), and a
    generator of steps: (q, k, v, t, t_first), steps at which the window is full or not, one of them without a column."""
    dtype, G, Hkv, d, Lcap, ring, w = SMALL[case]
    print("[case]", SMALL[case], flush=True)
    B, Hq, Tcap = 2, G * Hkv, Lcap + 40
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(case)
    lens = torch.randint(0, Lcap + 1, (B, Hkv), device=DEV, generator=g, dtype=torch.int32)
    edge = [0, Lcap, max(Lcap - 1, 0), min(Lcap, 512), min(Lcap, 511), Lcap + 7, -3, min(Lcap, 128), min(Lcap, 127)]
    for i, e in enumerate(edge):
        if i < B * Hkv:
            lens.view(-1)[(i + case) % (B * Hkv)] = e
    rows = [torch.randn(B, Hkv, Lcap, d, device=DEV, generator=g).to(tdt) for _ in range(2)]
    pos = torch.arange(Lcap, device=DEV, dtype=torch.int32).expand(B, Hkv, Lcap).clone()
    pos[0, 0, Lcap // 2] = Tcap + 5
    hit = torch.randint(0, Lcap + 4, (B, Hkv, Lcap), device=DEV, generator=g, dtype=torch.int32)
    states = []
    for _ in range(n):
        st = corm.LayerState(B, Hq, Hkv, d, Lcap, Tcap, w, 3, dtype, device=DEV, want_ring=ring is not None, want_masks=True,
                             score_dtype=ring)
        st.K.copy_(rows[0]), st.V.copy_(rows[1]), st.pos.copy_(pos), st.last_hit.copy_(hit), st.lens.copy_(lens)
        states.append(st)

    def steps():
        t = torch.tensor([Lcap + 1, Lcap + 3], dtype=torch.int32, device=DEV)
        for step in range(10):
            q = torch.randn(B, Hq, d, device=DEV, generator=g).to(tdt)
            k, v = (torch.randn(B, Hkv, d, device=DEV, generator=g).to(tdt) for _ in range(2))
            ts = t + step
            if step == 7:
                ts[1] = Tcap + 1
            yield step, q, k, v, ts, ts - (0 if step % 4 == 3 else w)
    return states, steps()


def _same(a, b, step, names):
    for name in names:
        x, y = getattr(a, name), getattr(b, name)
        if x is None and y is None:
            continue
        if x.is_floating_point():        # (NaN in the same places)
            assert torch.equal(x.isnan(), y.isnan()), (name, step)
            x, y = x.nan_to_num(0, 1e38, -1e38), y.nan_to_num(0, 1e38, -1e38)
        assert torch.equal(x, y), (name, step)


@pytest.mark.parametrize("poison", [None, INF, -INF, float("nan")])
@pytest.mark.parametrize("case", range(len(SMALL)))
def test_small_units_in_one_launch_equal_the_split_launches(case, poison):
    """A step of small units in one launch against attend, record and compact: the same bits in the cache, the decisions, the
    survivors, out and the ring, with finite keys and with one that is not in every other unit."""
    (a, b), steps = _small_states(case, 2)
    assert harness.step_is_one_launch(a)
    if poison is not None:
        for st in (a, b):
            st.K[0, ::2, st.Lcap // 3, 5] = poison
    for step, q, k, v, t, t_first in steps:
        for st, path in ((a, 0), (b, 1)):
            st.keep.zero_(), st.kept_idx.zero_()
            st.step(q, k, v, t, t_first, opts=corm.corm_launch_opts(path, 0, None, None))
        torch.cuda.synchronize()
        _same(a, b, step, ("out", "ring", "lens", "pos", "last_hit", "K", "V", "keep", "kept_idx", "status"))


@pytest.mark.parametrize("case", range(len(SMALL)))
def test_small_units_step_like_the_calls_that_do_a_part_of_it(case):
    """What the header says of corm_decode_step, with default options: its bits are those of append, attend, mask and compact, and of
    the two phases; the deferred step with dead_num = 0 reproduces it slot for slot (its recent-r rule goes by position: units with
    room, and keys at the positions in front of the step's)."""
    (a, two, lazy, single), steps = _small_states(case, 4)
    room = max(a.Lcap - 8, 0)
    n = a.lens.clamp(0, room)
    before = torch.tensor([a.Lcap, a.Lcap + 2], device=DEV).view(2, 1, 1)
    for st in (a, two, lazy, single):
        st.lens.copy_(n)
        st.pos.copy_(before - n.unsqueeze(-1) + torch.arange(a.Lcap, device=DEV))
    for step, q, k, v, t, t_first in steps:
        if step > min(room, 6):
            break
        a.step(q, k, v, t, t_first)
        two.step_attend(q, k, v, t, t_first)
        two.step_evict()
        lazy.step_lazy(q, k, v, t, t_first, 0, 1)
        s = single
        corm.corm_append(s.desc, s.K, s.V, s.lens, s.pos, s.last_hit, k, v, t, s.status)
        corm.corm_decode_attend(s.desc, q, s.K, s.V, s.lens, s.pos, t, s.ring, s.last_hit, s.out, s.workspace, status=s.status)
        corm.corm_evict_mask_summary(s.desc, s.last_hit, s.lens, t, t_first, s.keep)
        corm.corm_compact(s.desc, s.K, s.V, s.pos, s.last_hit, s.lens, s.keep, s.kept_idx, s.workspace)
        torch.cuda.synchronize()
        live = torch.arange(a.Lcap, device=DEV) < a.lens.unsqueeze(-1)
        for other in (two, lazy, single):
            _same(a, other, step, ("out", "ring", "lens", "status"))
            for name in ("pos", "last_hit", "K", "V"):
                assert torch.equal(getattr(a, name)[live], getattr(other, name)[live]), (name, step)


@pytest.mark.parametrize("dtype,G,Hkv,d,Lcap", NOT_SMALL)
def test_what_is_not_small_takes_the_launches_of_its_path(dtype, G, Hkv, d, Lcap):
    assert not harness.step_is_one_launch(corm.LayerState(2, G * Hkv, Hkv, d, Lcap, Lcap + 8, 4, 3, dtype, device=DEV, want_ring=False))


@pytest.mark.parametrize("case", [0, 4, 6])
def test_a_step_of_small_units_with_events_brackets_the_launch_that_streams(case):
    """The events of corm_launch_opts lie around the launch that streams K and V alone: a step with events takes the split launches."""
    (a, b), steps = _small_states(case, 2)
    a.workspace.fill_(0x5a)
    for step, q, k, v, t, t_first in steps:
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record(), e1.record()      # (creates the handles)
        a.step(q, k, v, t, t_first, opts=corm.make_opts(0, (e0.cuda_event, e1.cuda_event)))
        b.step(q, k, v, t, t_first)
        torch.cuda.synchronize()
        assert e0.elapsed_time(e1) > 0
        _same(a, b, step, ("out", "ring", "lens", "keep"))
        if step == 0:
            assert not bool((a.workspace == 0x5a).all())
            break


# query heads per KV head, d, capacity: 15, 16 and 17 parts of a full unit (up to 16 a wave folds an item alone), 68 parts of 128
# keys and 70 of 512 (more than a wave holds one of per lane)
OUTS = [(1, 64, 1900), (8, 128, 2048), (2, 128, 2100), (4, 128, 8600), (1, 128, 35700)]


@pytest.mark.parametrize("case", range(len(OUTS)))
def test_out_of_a_split_unit_whatever_its_parts(case):
    """out of the split launches against softmax in 64 bits, for units of every number of parts, empty ones among them (out 0).
    A weight's logit is a sum of d products of at most 8 / d each in the log2 domain, rounded d times; with exp2, the factors
    between parts and the sums (over the parts of a key's lane, its wave and unit) less than 200 more roundings of terms that are
    all weights times |v|."""
    G, d, Lcap = OUTS[case]
    print("[case]", OUTS[case], flush=True)
    g = torch.Generator(device=DEV).manual_seed(case)
    full = [0, 1, 15, 63, 64, 511, 512, 513, 1500, 1920, 2047, Lcap // 2 + 1, Lcap - 1, Lcap]
    lens = [n for n in full if n <= Lcap]
    B = len(lens)
    st = corm.LayerState(B, G, 1, d, Lcap, Lcap, 16, 8, "f32", device=DEV, want_ring=False)
    scale = float(torch.tensor(float(d)).rsqrt() * 1.4426950408889634)
    q = torch.rand(B, G, d, device=DEV, generator=g) * 2 - 1
    st.K[:] = (torch.rand(B, 1, Lcap, d, device=DEV, generator=g) * 2 - 1) * (8 / d / scale)
    st.V[:] = torch.randn(B, 1, Lcap, d, device=DEV, generator=g)
    st.pos[:] = torch.arange(Lcap, device=DEV).int()
    st.lens[:] = torch.tensor(lens, device=DEV, dtype=torch.int32).view(B, 1)
    st.out.fill_(7.0)
    t = torch.full((B,), Lcap, dtype=torch.int32, device=DEV)
    assert corm.corm_selected_path(st.desc) == 1
    corm.corm_decode_attend(st.desc, q, st.K, st.V, st.lens, st.pos, t, st.ring, st.last_hit, st.out, st.workspace,
                            status=st.status)
    torch.cuda.synchronize()
    assert int(st.status.item()) == 0
    for b, n in enumerate(lens):
        if n == 0:
            assert not st.out[b].any()
            continue
        k, v = st.K[b, 0, :n].double(), st.V[b, 0, :n].double()
        a = torch.softmax(q[b].double() @ k.t().contiguous() / d ** 0.5, -1)
        tol = 2.0 ** -24 * (8 * d + 200) * (a @ v.abs())
        assert ((st.out[b].double() - a @ v).abs() <= tol).all(), n


# query heads per KV head, d, units, capacity: the record launch by its rules (workgroups of one, two and four chunks; a thread per key or
# two keys a thread; out by workgroups of its own, by waves or whole ones, or by those that record)
RECORDS = [(8, 64, 768, 512), (8, 64, 769, 512), (8, 128, 512, 256), (8, 128, 513, 256), (8, 64, 1024, 512), (8, 128, 600, 2048), (8, 64, 1030, 2100),
           (4, 128, 130, 9000), (1, 64, 1100, 300), (2, 64, 600, 600), (4, 64, 40, 4096), (1, 128, 3, 20000)]


@pytest.mark.parametrize("case", range(len(RECORDS)))
def test_record_launch_by_its_rules(case):
    """out and last_hit of one attend call over units of every fill, empty ones among them (out 0), against softmax in 64 bits.  Tolerance of out
    as in test_out_of_a_split_unit_whatever_its_parts; a score within 1e-4 of c/t may fall on either side."""
    G, d, U, Lcap = RECORDS[case]
    print("[case]", RECORDS[case], flush=True)
    g = torch.Generator(device=DEV).manual_seed(case)
    st = corm.LayerState(1, G * U, U, d, Lcap, Lcap, 16, 8, "f32", device=DEV, want_ring=False)
    lens = torch.randint(0, Lcap + 1, (U,), device=DEV, generator=g, dtype=torch.int32)
    edges = [n for n in (Lcap, 0, 1, 511, 512, 513, 2048, 4095, 7 * 512, 8192) if n <= Lcap][:U]
    lens[:len(edges)] = torch.tensor(edges, device=DEV, dtype=torch.int32)
    scale = float(torch.tensor(float(d)).rsqrt() * 1.4426950408889634)
    q = torch.rand(1, G * U, d, device=DEV, generator=g) * 2 - 1
    st.K[:] = (torch.rand(1, U, Lcap, d, device=DEV, generator=g) * 2 - 1) * (8 / d / scale)
    st.V[:] = torch.randn(1, U, Lcap, d, device=DEV, generator=g)
    st.pos[:] = torch.arange(Lcap, device=DEV).int()
    st.lens[0] = lens
    st.out.fill_(7.0)
    t = torch.full((1,), Lcap, dtype=torch.int32, device=DEV)
    opts = corm.make_opts(path=1)
    corm.corm_decode_attend(st.desc, q, st.K, st.V, st.lens, st.pos, t, st.ring, st.last_hit, st.out, st.workspace,
                            status=st.status, opts=opts)
    torch.cuda.synchronize()
    assert int(st.status.item()) == 0
    slot = torch.arange(Lcap, device=DEV)
    step = max(1, 2 ** 21 // Lcap)
    for u in range(0, U, step):
        n = lens[u:u + step].long().view(-1, 1, 1)
        held = slot.view(1, 1, -1) < n
        k, v = st.K[0, u:u + step].double(), st.V[0, u:u + step].double()
        qu = q.view(U, G, d)[u:u + step].double()
        s = torch.matmul(k, qu.transpose(1, 2).contiguous()).transpose(1, 2) / d ** 0.5
        a = torch.softmax(s.masked_fill(~held, float("-inf")), -1)
        a = torch.where(held, a, 0.0)
        tol = 2.0 ** -24 * (8 * d + 200) * torch.matmul(a, v.abs())
        out = st.out.view(U, G, d)[u:u + step].double()
        assert ((out - torch.matmul(a, v)).abs() <= tol).all(), u
        assert not out[(n == 0).view(-1)].any()
        sure = ((a * Lcap - 1).abs() > 1e-4).all(1)
        hit = (a * Lcap >= 1).any(1)
        assert torch.equal((st.last_hit[0, u:u + step] == Lcap)[sure], hit[sure]), u
