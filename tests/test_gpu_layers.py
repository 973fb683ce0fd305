"""keydiff_prefill_block_layers where the steps of its layers share launches, against keydiff_prefill_block layer by
layer (which the oracle checks elsewhere): positions, rows and scores bit for bit, outputs within the attention's bar
(the keys are cut into fewer ranges)."""
import numpy as np
import pytest

import paper_2504_15364_amd as kd
from helpers import ATTN_ATOL

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _blocks(heads, T, B, seed):
    hq, hkv, d = heads
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shift = torch.randn((1, hkv, 1, d), generator=gen, device="cuda")
    for t in range(0, T, B):
        n = min(B, T - t)
        q, k, v = (torch.randn((1, h, n, d), generator=gen, device="cuda") for h in (hq, hkv, hkv))
        yield t, q.bfloat16(), (k + shift).bfloat16(), v.bfloat16()


def _same_state(a, b, where):
    assert a.len == b.len, where
    n = a.len
    pa, pb = a.positions(), b.positions()
    assert torch.equal(pa, pb), f"positions differ {where}"
    for x, y in ((a.key_rows(), b.key_rows()), (a.value_rows(), b.value_rows())):
        assert torch.equal(x[:, :, :n].view(torch.int16), y[:, :, :n].view(torch.int16)), f"rows differ {where}"
    assert torch.equal(a.scores().view(torch.int32), b.scores().view(torch.int32)), f"key sums differ {where}"
    assert a.status() == 0 and b.status() == 0


@pytest.mark.parametrize("heads,N,B,T,layers,kw", [
    ((8, 2, 128), 512, 128, 1100, 2, {}),                                              # ragged last block
    ((8, 2, 128), 512, 128, 900, 17, {}),                                              # more layers than a launch takes
    ((6, 2, 128), 300, 48, 650, 5, {"anchor_mode": kd.ANCHOR_MEAN_UNIT_KEY}),           # waves without query rows
    ((4, 1, 64), 256, 32, 480, 16, {"layout": kd.LAYOUT_ORDERED}),                      # (shifted by the selection)
    ((8, 2, 64), 512, 64, 820, 2, {"layout": kd.LAYOUT_ORDERED}),                       # (likewise)
    ((4, 1, 128), 640, 160, 1480, 16, {"layout": kd.LAYOUT_ORDERED}),                   # the shifts of a full launch, two chunks to wait for
    ((8, 2, 128), 900, 128, 1600, 2, {"layout": kd.LAYOUT_ORDERED}),
    ((14, 2, 128), 384, 64, 640, 3, {"window_W": 64}),
    ((8, 2, 128), 300, 256, 1000, 1, {}),                                              # one layer: the step of prefill_block
], ids=["2", "17", "5-helper", "16-ordered-short", "2-ordered-short", "16-ordered", "2-ordered", "3-window", "1"])
def test_layers_in_one_launch(heads, N, B, T, layers, kw):
    kw = {"layout": kd.LAYOUT_FILL, **kw}
    a, b = ([kd.KeyDiffCache(kd.KeyDiffConfig(1, *heads, N, B, **kw)) for _ in range(layers)] for _ in range(2))
    for i, blks in enumerate(zip(*(_blocks(heads, T, B, 100 + l) for l in range(layers)))):
        t = blks[0][0]
        by_layer = i == 5 and kw["layout"] == kd.LAYOUT_FILL and not kw.get("window_W")
        if by_layer:
            # a block on which the layers run one by one and leave evictions pending
            outs = []
            for l, (_, q, k, v) in enumerate(blks):
                outs.append(a[l].prefill_block_deferred(q, k, v, t, carry=a[l - 1] if layers > 1 else None))
        else:
            outs = kd.prefill_block_layers(a, [x[1] for x in blks], [x[2] for x in blks], [x[3] for x in blks], t)
        for l, (_, q, k, v) in enumerate(blks):
            want = b[l].prefill_block(q, k, v, t)
            assert float((outs[l].float() - want.float()).abs().max()) <= ATTN_ATOL, (t, l)
        assert all(bool(c.plan()[3] & 4) == (layers > 1 and not by_layer) for c in a), (t, a[0].plan())   # launches were shared
        assert all(c.plan()[3] == 0 for c in b)
        assert layers < 16 or a[0].plan()[0] <= b[0].plan()[0]
    for l in range(layers):
        _same_state(a[l], b[l], f"layer {l}")
        a[l].close()
        b[l].close()


@pytest.mark.parametrize("kind", ["chain", "in-place", "common-inputs"])
def test_layers_that_touch_one_anothers_memory_keep_their_order(kind):
    heads, N, B, T, layers = (8, 2, 128), 64, 32, 160, 3
    a, b = ([kd.KeyDiffCache(kd.KeyDiffConfig(1, *heads, N, B, layout=kd.LAYOUT_FILL)) for _ in range(layers)] for _ in range(2))
    for blks in zip(*(_blocks(heads, T, B, 300 + l) for l in range(layers))):
        t = blks[0][0]
        got = []
        for caches in (a, b):
            qs, ks, vs = ([x[i].clone() for x in blks] for i in (1, 2, 3))
            if kind == "chain":          # a layer's output is the next layer's queries
                outs = [torch.zeros_like(q) for q in qs]
                qs = [qs[0]] + outs[:-1]
            elif kind == "in-place":
                outs = qs
            else:                        # inputs in common: nothing is written that another layer reads
                outs = [torch.zeros_like(q) for q in qs]
                ks[1] = vs[0]
            if caches is a:
                kd.prefill_block_layers(caches, qs, ks, vs, t, out=outs)
                assert all(bool(c.plan()[3] & 4) == (kind == "common-inputs") for c in a)
            else:
                for c, q, k, v, o in zip(caches, qs, ks, vs, outs):
                    c.prefill_block(q, k, v, t, out=o)
            got.append(outs)
        for x, y in zip(*got):
            assert float((x.float() - y.float()).abs().max()) <= ATTN_ATOL, t
    for l in range(layers):
        _same_state(a[l], b[l], f"layer {l}")
        a[l].close()
        b[l].close()


@pytest.mark.parametrize("heads,N,B,kw", [
    ((8, 2, 128), 12300, 128, {}),                                   # scores alone in the registers of the selection
    ((4, 1, 64), 12288 - 64, 64, {}),                                # the last length with positions there too
    ((4, 1, 64), 20500, 64, {}),                                     # read from memory in every pass
    ((4, 1, 64), 20480 - 64, 64, {"layout": kd.LAYOUT_ORDERED}),     # the last length in registers
    ((8, 2, 128), 20600, 128, {"layout": kd.LAYOUT_ORDERED}),
], ids=["12428", "12288", "20564", "20480-ordered", "20728-ordered"])
def test_layers_with_long_caches_in_one_launch(heads, N, B, kw):
    hq, hkv, d = heads
    kw = {"layout": kd.LAYOUT_FILL, **kw}
    a, b = ([kd.KeyDiffCache(kd.KeyDiffConfig(1, *heads, N, B, **kw)) for _ in range(2)] for _ in range(2))
    pos = torch.arange(N, dtype=torch.int32, device="cuda").expand(1, hkv, N).contiguous()
    for l, pair in enumerate(zip(a, b)):
        (_, _, k, v), = _blocks(heads, N, N, 700 + l)
        for c in pair:
            c.load(k, v, pos)
    for blks in zip(*(_blocks(heads, 3 * B, B, 800 + l) for l in range(2))):
        t = N + blks[0][0]
        outs = kd.prefill_block_layers(a, [x[1] for x in blks], [x[2] for x in blks], [x[3] for x in blks], t)
        assert all(c.plan()[3] & 4 for c in a), a[0].plan()
        for l, (_, q, k, v) in enumerate(blks):
            want = b[l].prefill_block(q, k, v, t)
            assert float((outs[l].float() - want.float()).abs().max()) <= ATTN_ATOL, (t, l)
    for l in range(2):
        _same_state(a[l], b[l], f"layer {l}")
        a[l].close()
        b[l].close()


@pytest.mark.parametrize("d,N,B", [(64, 736, 32), (64, 737, 32), (64, 500, 260), (128, 352, 32), (128, 353, 32), (128, 190, 190),
                                   (64, 40, 1), (128, 60, 7)])
@pytest.mark.parametrize("call", ["block", "layers", "deferred"])
def test_short_ordered_caches_are_shifted_by_the_selection(d, N, B, call):
    # up to 48 K elements of K a head (768 rows of 64, 384 of 128) the selection shifts the rows of an ORDERED cache, in
    # passes of 512 or 256; beyond, the workgroups around it do, or a launch of its own.  The retained rows are those of the FILL layout, in order.
    heads, layers = (8, 2, d), 2 if call == "layers" else 1
    a, b = ([kd.KeyDiffCache(kd.KeyDiffConfig(1, *heads, N, B, layout=lay)) for _ in range(layers)]
            for lay in (kd.LAYOUT_ORDERED, kd.LAYOUT_FILL))
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = [torch.randn((1, 2, N, d), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    pos = torch.arange(N, dtype=torch.int32, device="cuda").expand(1, 2, N).contiguous()
    for c in a + b:
        c.load(*x, pos)
    for blks in zip(*(_blocks(heads, 4 * B + B // 2, B, 500 + l) for l in range(layers))):
        t = N + blks[0][0]
        for caches in (a, b):
            if call == "layers":
                kd.prefill_block_layers(caches, [y[1] for y in blks], [y[2] for y in blks], [y[3] for y in blks], t)
            elif call == "deferred":
                caches[0].prefill_block_deferred(*blks[0][1:], t)
            else:
                caches[0].prefill_block(*blks[0][1:], t)
    for ca, cb in zip(a, b):
        pa, pb = ca.positions(), cb.positions().sort(-1)
        assert torch.equal(pa, pb.values)
        for ra, rb in ((ca.key_rows(), cb.key_rows()), (ca.value_rows(), cb.value_rows())):
            pick = pb.indices[..., None].expand(-1, -1, -1, d)
            assert torch.equal(ra[:, :, :N].view(torch.int16), rb[:, :, :N].gather(2, pick).view(torch.int16))
        assert torch.allclose(ca.scores(), cb.scores().gather(2, pb.indices), rtol=1e-6, atol=1e-7)
        assert ca.status() == 0 and cb.status() == 0
        ca.close()
        cb.close()


@pytest.mark.parametrize("anchor", [kd.ANCHOR_MEAN_KEY, kd.ANCHOR_MEAN_UNIT_KEY], ids=["mean", "unit"])
@pytest.mark.parametrize("d,N,E", [(128, 2900, 100), (128, 2816, 256), (128, 1500, 300), (64, 2900, 100), (64, 2560, 512), (64, 700, 520)])
def test_ordered_eviction_carried_leaves_what_one_inside_the_step_leaves(d, N, E, anchor):
    # The keys an ORDERED eviction takes out of the key sum are read by all waves of a passenger and by half of those of
    # step_post, in batches of 256 rows (or 128, 256 of 64): positions, rows and scores are the same bits either way.  The evicted keys
    # have exponents up to 40 apart, so that every score shows the order in which they were summed.
    hq, hkv, T = 8, 2, N + E
    rng = np.random.default_rng(N + E + d)
    keys = 1.0 + 0.3 * rng.standard_normal((1, hkv, T, d))
    far = np.stack([rng.permutation(T)[:E] for _ in range(hkv)])
    for h in range(hkv):
        keys[0, h, far[h]] = np.exp2(rng.integers(-20, 21, size=(E, 1))) * (1.0 + 0.05 * rng.standard_normal((E, d)))
    keys = torch.from_numpy(keys.astype(np.float32)).cuda().bfloat16()
    values = torch.randn(keys.shape, generator=torch.Generator(device="cuda").manual_seed(E), device="cuda").bfloat16()
    pos = torch.arange(N, dtype=torch.int32, device="cuda").expand(1, hkv, N).contiguous()
    q = torch.zeros((1, hq, E, d), dtype=torch.bfloat16, device="cuda")
    block = (q, keys[:, :, N:].contiguous(), values[:, :, N:].contiguous())
    a, b, other = (kd.KeyDiffCache(kd.KeyDiffConfig(1, hq, hkv, d, N, E, layout=kd.LAYOUT_ORDERED, anchor_mode=anchor)) for _ in range(3))
    for c in (a, b):
        c.load(keys[:, :, :N].contiguous(), values[:, :, :N].contiguous(), pos)
    a.prefill_block(*block, N)
    b.prefill_block_deferred(*block, N, carry=other)
    other.prefill_block_deferred(*block, 0, carry=b)
    assert other.plan()[3] & 1
    _same_state(a, b, "carried")
    assert torch.all(a.positions().diff(dim=-1) > 0)
    for c in (a, b, other):
        c.close()


@pytest.mark.parametrize("heads,batch,N,B,layers,lay,want", [
    # ORDERED, three layers or more: sharing puts the row shifts of all of them behind the attention
    ((32, 8, 128), 1, 4096, 128, 3, kd.LAYOUT_ORDERED, 4),
    ((32, 8, 128), 2, 4096, 128, 3, kd.LAYOUT_ORDERED, 2),     # twice the rows: 38.8 us a layer and block shared, 34.4 riding
    ((32, 8, 64), 4, 2048, 128, 3, kd.LAYOUT_ORDERED, 2),
    ((32, 8, 64), 4, 2048, 128, 4, kd.LAYOUT_ORDERED, 4),
    ((32, 8, 128), 2, 4096, 128, 8, kd.LAYOUT_ORDERED, 4),
    ((8, 2, 128), 1, 1024, 128, 4, kd.LAYOUT_ORDERED, 4),      # few row tiles: 6.3 us shared, 14.0 riding
    ((8, 2, 64), 1, 1100, 64, 3, kd.LAYOUT_ORDERED, 4),
    # FILL: 192 row tiles of each layer in 256 compute units, or 48 in ranges of 240 workgroups
    ((28, 4, 128), 8, 2048, 200, 2, kd.LAYOUT_FILL, 1),
    ((28, 4, 128), 2, 8192, 200, 2, kd.LAYOUT_FILL, 1),
    ((28, 4, 128), 2, 4096, 200, 2, kd.LAYOUT_FILL, 4),
    ((28, 4, 128), 4, 4096, 200, 3, kd.LAYOUT_ORDERED, 1),     # 288 row tiles of three layers: a second round for 32
    ((28, 4, 128), 1, 4096, 200, 3, kd.LAYOUT_ORDERED, 4),
    ((24, 8, 128), 8, 2048, 128, 2, kd.LAYOUT_FILL, 4),
    ((32, 8, 128), 1, 8192, 128, 4, kd.LAYOUT_FILL, 4),
    ((28, 4, 128), 1, 8192, 256, 2, kd.LAYOUT_FILL, 4),
], ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_layers_share_launches_where_that_is_faster(heads, batch, N, B, layers, lay, want):
    # which way calls of the measured shapes go (256 compute units): the bit of plan()[3] on every layer of the second evicting block
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the plans are for 256 compute units")
    hq, hkv, d = heads
    gen = torch.Generator(device="cuda").manual_seed(5)
    caches = [kd.KeyDiffCache(kd.KeyDiffConfig(batch, *heads, N, B, layout=lay)) for _ in range(layers)]
    pos = torch.arange(N, dtype=torch.int32, device="cuda").expand(batch, hkv, N).contiguous()
    rows = torch.randn((batch, hkv, N, d), generator=gen, device="cuda").bfloat16()
    for c in caches:
        c.load(rows, rows, pos)
    q = torch.randn((batch, hq, B, d), generator=gen, device="cuda").bfloat16()
    for i in range(2):
        k = torch.randn((batch, hkv, B, d), generator=gen, device="cuda").bfloat16()
        kd.prefill_block_layers(caches, [q] * layers, [k] * layers, [k] * layers, N + i * B)
    plans = [c.plan() for c in caches]
    assert all(pl[3] & want for pl in plans), plans
    for c in caches:
        c.finish()
        assert c.status() == 0
        c.close()


def _counters(cache):
    """The part of a cache's metadata that counts the workgroups of each head that have started in launches that shift rows: the last
    thing in it, 32 words apart."""
    heads = cache.cfg.batch * cache.cfg.n_kv_heads
    torch.cuda.synchronize()
    return cache._meta[-((heads * 128 + 255) // 256 * 256):].view(torch.int32)[:heads * 32:32]


def _started(cache):
    return _counters(cache).clone()


def _start_order(cache, by):
    """Adds `by` to what a cache says about how many workgroups have started."""
    _counters(cache).add_(by)
    torch.cuda.synchronize()


@pytest.mark.parametrize("heads,batch,N,B,layers,kw,units", [
    ((8, 2, 128), 1, 390, 32, 1, {}, 1),                                         # the fewest rows: beyond what the selection shifts itself
    ((8, 2, 128), 1, 900, 300, 1, {}, 1),                                         # rows that land ten chunks below
    ((4, 1, 64), 1, 1000, 7, 1, {"window_W": 90}, 1),
    ((4, 1, 64), 1, 12288 - 50, 50, 1, {"anchor_mode": kd.ANCHOR_MEAN_UNIT_KEY}, 1),  # the last length
    ((8, 8, 128), 4, 2000, 130, 1, {}, 10),                                          # ten units a thread, merged by few workgroups
    ((32, 8, 128), 1, 4097, 1, 1, {}, 5),                                           # one row, behind step_few and its merge
    ((24, 8, 128), 1, 4096, 128, 3, {}, 15),                                         # fifteen units, several layers
    ((8, 2, 64), 1, 2000, 100, 16, {}, 5),
    ((28, 4, 128), 4, 1024, 200, 1, {}, 3),                                          # few ranges and many rows to merge: four pieces a thread
    ((24, 8, 128), 2, 2048, 256, 2, {}, 11),                                         # likewise, one a thread
    ((16, 8, 128), 2, 8192, 64, 1, {}, 18),                                          # eighteen units
], ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else None)
def test_rows_shifted_around_the_selection(heads, batch, N, B, layers, kw, units):
    # ORDERED caches beyond what the selection shifts itself: the rows wait in the registers of the workgroups around it.  The rows retained are
    # those of the FILL layout, in order, over steps that follow one another and with a ragged one; a launch starts a selection and
    # a workgroup for every `units` times 4096 elements of K of every head.
    hq, hkv, d = heads
    a, b = ([kd.KeyDiffCache(kd.KeyDiffConfig(batch, *heads, N, B, layout=lay, **kw)) for _ in range(layers)]
            for lay in (kd.LAYOUT_ORDERED, kd.LAYOUT_FILL))
    gen = torch.Generator(device="cuda").manual_seed(N + B)

    def draw(h, n):
        return torch.randn((batch, h, n, d), generator=gen, device="cuda").bfloat16()

    t = N
    if kw.get("window_W"):   # (needs consecutive positions from an empty cache on)
        t = 0
    else:
        rows = draw(hkv, N), draw(hkv, N)
        pos = torch.arange(N, dtype=torch.int32, device="cuda").expand(batch, hkv, N).contiguous()
        for c in a + b:
            c.load(*rows, pos)
    for n in [B] * (N // B + 1 if t == 0 else 0) + [B, B, (B + 1) // 2, B]:
        blk = [[draw(h, n) for _ in range(layers)] for h in (hq, hkv, hkv)]
        outs, before = [], [_started(c) for c in a]
        for caches in (a, b):
            if layers > 1:
                outs.append(kd.prefill_block_layers(caches, *blk, t))
            else:
                outs.append([caches[0].prefill_block(*(x[0] for x in blk), t)])
        for x, y in zip(*outs):
            assert float((x.float() - y.float()).abs().max()) <= ATTN_ATOL, t
        if a[0].len == N and t >= N and torch.cuda.get_device_properties(0).multi_processor_count == 256:
            want = 1 + -(-(N + n) * d // (units * 4096))
            assert all(torch.equal(_started(c) - x, torch.full_like(x, want)) for c, x in zip(a, before)), (t, want)
        t += n
    for ca, cb in zip(a, b):
        pa, pb = ca.positions(), cb.positions().sort(-1)
        assert torch.equal(pa, pb.values)
        for ra, rb in ((ca.key_rows(), cb.key_rows()), (ca.value_rows(), cb.value_rows())):
            pick = pb.indices[..., None].expand(-1, -1, -1, d)
            assert torch.equal(ra[:, :, :N].view(torch.int16), rb[:, :, :N].gather(2, pick).view(torch.int16))
        assert ca.status() == 0 and cb.status() == 0
        ca.close()
        cb.close()


def _loaded(batch, heads, N, B, seed, layouts, **kw):
    """Caches of the given layouts, holding the same N rows each."""
    hq, hkv, d = heads
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rows = [torch.randn((batch, hkv, N, d), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    pos = torch.arange(N, dtype=torch.int32, device="cuda").expand(batch, hkv, N).contiguous()
    caches = [kd.KeyDiffCache(kd.KeyDiffConfig(batch, *heads, N, B, layout=lay, **kw)) for lay in layouts]
    for c in caches:
        c.load(*rows, pos)
    return caches


@pytest.mark.parametrize("heads,N,B,how", [((8, 2, 128), 2000, 100, "finish"), ((4, 1, 64), 3000, 33, "scores"), ((32, 8, 128), 4097, 1, "step")])
def test_pending_eviction_is_finished_around_its_selection(heads, N, B, how):
    # An eviction that found no launch to ride in, finished by a call on its own cache: with nothing to merge, the workgroups around the
    # selection only shift.  Positions and rows are those of the step that evicts by itself.
    a, b = _loaded(1, heads, N, B, 9, [kd.LAYOUT_ORDERED] * 2)
    gen = torch.Generator(device="cuda").manual_seed(10)
    hq, hkv, d = heads
    for i in range(3):
        q, k, v = (torch.randn((1, h, B, d), generator=gen, device="cuda").bfloat16() for h in (hq, hkv, hkv))
        t = N + i * B
        out, before = a.prefill_block_deferred(q, k, v, t), _started(a)
        if how == "finish":
            a.finish()
        elif how == "scores":
            a.scores()
        want = b.prefill_block(q, k, v, t)
        assert float((out.float() - want.float()).abs().max()) <= ATTN_ATOL, t
        if how != "step":   # (else the next step finishes it)
            shifted = _started(a) - before
            assert bool((shifted > 0).all()) and torch.equal(_started(a), _started(b))
            _same_state(a, b, f"after {t}")
    _same_state(a, b, "at the end")
    a.close()
    b.close()


@pytest.mark.parametrize("heads,N,B,layers", [
    ((6, 3, 128), 6000, 100, 1),      # three heads: a head's workgroups start on all XCDs, the chip holds neither both launches nor half of them
    ((8, 2, 128), 8192, 128, 1),
    ((24, 8, 128), 4096, 64, 3),
    ((4, 1, 64), 3000, 20, 5),
    ((6, 3, 128), 12400, 300, 1),     # too long for the launch of the selection: the shift is one of its own, three chunks to wait for
    ((12, 6, 64), 12400, 130, 3),
    ((32, 8, 128), 8192, 128, 3),     # ... or rides in the attention launch of another layer
], ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_ordered_caches_on_two_streams(heads, N, B, layers):
    # Row shifts of different caches overlap on the chip, each in a launch whose workgroups wait for one another.  Every
    # cache ends as it does where nothing else runs.
    steps, kinds = 12, [kd.LAYOUT_ORDERED] * 2 * layers
    groups = []
    for g in range(2):
        both = _loaded(1, heads, N, B, 40 + g, kinds)
        gen = torch.Generator(device="cuda").manual_seed(60 + g)
        blks = [[[torch.randn((1, h, B, heads[2]), generator=gen, device="cuda").bfloat16() for _ in range(layers)]
                 for h in (heads[0], heads[1], heads[1])] for _ in range(steps)]
        outs = [[[torch.empty_like(q) for q in blk[0]] for blk in blks] for _ in range(2)]
        groups.append((both[:layers], both[layers:], blks, outs))

    def step(caches, blk, out, t):
        if layers > 1:
            kd.prefill_block_layers(caches, *blk, t, out=out)
        else:
            caches[0].prefill_block(*(x[0] for x in blk), t, out=out[0])

    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for i in range(steps):
        for (a, _, blks, outs), s in zip(groups, streams):
            with torch.cuda.stream(s):
                step(a, blks[i], outs[0][i], N + i * B)
    for (a, *_), s in zip(groups, streams):
        for c in a:
            c.finish(s)
    torch.cuda.synchronize()
    for a, b, blks, outs in groups:
        for i in range(steps):
            step(b, blks[i], outs[1][i], N + i * B)
        torch.cuda.synchronize()
        for x, y in zip(*outs):
            assert all(torch.equal(p.view(torch.int16), q.view(torch.int16)) for p, q in zip(x, y))
        for l in range(layers):
            _same_state(a[l], b[l], f"layer {l}")
            a[l].close()
            b[l].close()


@pytest.mark.parametrize("heads,N,B", [((4, 1, 64), 1000, 40), ((8, 2, 128), 900, 100)])
def test_selection_by_a_workgroup_that_started_second(heads, N, B):
    # Whichever workgroup of a head starts first selects, the others take its rows from the lowest up: here the first to start is told that it
    # is none of them, so that the next one selects, whatever its number, and the topmost rows of a head are nobody's.
    hq, hkv, d = heads
    a, b = _loaded(1, heads, N, B, 7, (kd.LAYOUT_ORDERED, kd.LAYOUT_FILL))
    gen = torch.Generator(device="cuda").manual_seed(8)
    q, k, v = (torch.randn((1, h, B, d), generator=gen, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    _start_order(a, -1)
    out = a.prefill_block(q, k, v, N)
    want = b.prefill_block(q, k, v, N)
    assert float((out.float() - want.float()).abs().max()) <= ATTN_ATOL
    pa, pb = a.positions(), b.positions().sort(-1)
    assert torch.equal(pa, pb.values)
    assert a.status() != 0 and b.status() == 0
    unit = 4096 // d   # rows a chunk: one 16-byte unit a thread, half of 1024 threads for the keys
    chunks = -(-(N + B) // unit)
    here = pa < (chunks - 1) * unit           # rows of the chunks that had a workgroup (before it, position = row)
    assert bool(here.any())
    for ra, rb in ((a.key_rows(), b.key_rows()), (a.value_rows(), b.value_rows())):
        got, ref = ra[:, :, :N].view(torch.int16), rb[:, :, :N].gather(2, pb.indices[..., None].expand(-1, -1, -1, d)).view(torch.int16)
        assert torch.equal(got[here], ref[here])
    a.close()
    b.close()


def test_rows_stay_where_a_wait_expires():
    # No workgroup is told that it selects: the waits for the eviction bitmap, which are bounded, expire.  The status word says so and no row has moved.
    heads, N, B = (4, 1, 64), 1000, 40
    a, = _loaded(1, heads, N, B, 7, (kd.LAYOUT_ORDERED,))
    gen = torch.Generator(device="cuda").manual_seed(8)
    q, k, v = (torch.randn((1, h, B, 64), generator=gen, device="cuda").bfloat16() for h in (4, 1, 1))
    before = torch.cat([a.key_rows()[:, :, :N], k], 2), torch.cat([a.value_rows()[:, :, :N], v], 2)
    _start_order(a, 1)
    a.prefill_block(q, k, v, N)
    assert a.status() != 0
    for rows, want in zip((a.key_rows(), a.value_rows()), before):
        assert torch.equal(rows[:, :, :N + B].view(torch.int16), want.view(torch.int16))
    a.close()


@pytest.mark.parametrize("hq,hkv,d,Bt,anchor", [
    (7, 1, 128, 1, kd.ANCHOR_MEAN_KEY),        # seven workgroups for seven rows
    (28, 4, 128, 1, kd.ANCHOR_MEAN_KEY),
    (28, 4, 64, 2, kd.ANCHOR_MEAN_KEY),        # fourteen rows of a head
    (16, 1, 64, 1, kd.ANCHOR_MEAN_UNIT_KEY),   # the anchor by all waves together
    (1, 1, 128, 3, kd.ANCHOR_MEAN_KEY),
    (32, 1, 128, 1, kd.ANCHOR_MEAN_KEY),       # two workgroups share a key range
])
def test_generation_steps_against_plain_attention(hq, hkv, d, Bt, anchor):
    # steps of few query rows behind a long cache: every wave forms the anchor of a single token by itself, and the partials are merged by a
    # workgroup a row.  Outputs against float64; the rows that stay are those of the highest scores' complement, as keydiff_scores of the same rows has them.
    N, G = 4100, hq // hkv
    gen = torch.Generator(device="cuda").manual_seed(hq * 131 + d + Bt)

    def draw(h, n):
        return torch.randn((1, h, n, d), generator=gen, device="cuda").bfloat16()

    cache = kd.KeyDiffCache(kd.KeyDiffConfig(1, hq, hkv, d, N, Bt, layout=kd.LAYOUT_ORDERED, anchor_mode=anchor))
    K, V = draw(hkv, N), draw(hkv, N)
    cache.load(K, V, torch.arange(N, dtype=torch.int32, device="cuda").expand(1, hkv, N).contiguous())
    full = kd.KeyDiffCache(kd.KeyDiffConfig(1, hq, hkv, d, N + Bt, Bt, layout=kd.LAYOUT_ORDERED, anchor_mode=anchor))
    pos = torch.arange(N, device="cuda").expand(hkv, N)
    for i in range(3):
        q, k, v = draw(hq, Bt), draw(hkv, Bt), draw(hkv, Bt)
        t = N + i * Bt
        out = cache.prefill_block(q, k, v, t)
        K, V = torch.cat([K, k], 2), torch.cat([V, v], 2)
        pos = torch.cat([pos, torch.arange(t, t + Bt, device="cuda").expand(hkv, Bt)], 1)
        kk, vv = (x[0].double().repeat_interleave(G, 0) for x in (K, V))
        logits = (q[0].double()[:, :, None, :] * kk[:, None]).sum(-1) / d ** 0.5
        late = torch.arange(N + Bt, device="cuda")[None, :] > N + torch.arange(Bt, device="cuda")[:, None]
        w = logits.masked_fill(late, -torch.inf).softmax(-1)
        want = (w[..., None] * vv[:, None]).sum(2)
        assert float((out[0].double() - want).abs().max()) <= ATTN_ATOL, t
        full.load(K.contiguous(), V.contiguous(), pos[None].int().contiguous())
        scores = full.scores()[0].double()
        leave = torch.zeros_like(scores, dtype=torch.bool).scatter_(1, scores.topk(Bt, 1).indices, True)   # (no two scores are alike)
        keep = (~leave).nonzero()[:, 1].view(hkv, N)
        pos = pos.gather(1, keep)
        K, V = (x.gather(2, keep[None, :, :, None].expand(-1, -1, -1, d)) for x in (K, V))
        assert torch.equal(cache.positions()[0].long(), pos), t
    assert cache.status() == 0
    cache.close()
    full.close()
