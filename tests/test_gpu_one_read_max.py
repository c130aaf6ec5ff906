"""The form with one read of G for the largest magnitude of the whole vector: forced at small sizes by its testing hook, every
driver, one and several fills, blocks and groups that end inside the vector, every number of records around the halves of the
ring that they wait in and around the room for them, ties, values and weights that are not finite, and the decision that the
sample makes on the device.  Codes, scales and estimates equal the oracle's (or the two-read form's) bit for bit."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

from gpu_util import cyclic_csr, monotone_csr, random_csr, to_device

pytestmark = pytest.mark.gpu


def _code(rng, kind, n, k, width):
    return (cyclic_csr(rng, n, min(n, width)) if kind == "cyclic" else monotone_csr(rng, n, k, width) if kind == "interval"
            else random_csr(rng, n, k, width))


def _check(G_host, csr, k, bits, w, mask, unfused=False, graph=False, seed=77, step=9):
    """What agc_debug_sketch_last says of the last pass."""
    import torch
    n, d = len(bits), G_host.shape[1]
    ctx = api.Context(n, k, d, scale_mode=api.AGC_SCALE_MAXABS, unfused_step=unfused)
    ctx.agc_set_code(*csr)
    ctx.agc_debug_sketch_max(1)
    codes, scales, ghat = ctx.alloc_outputs(bits)
    for t in codes:
        t.fill_(0x5A)
    G = to_device(G_host)

    def run():
        ctx.agc_step(G, bits, w, mask, seed, step, codes, scales, ghat)
    run()
    if graph:
        torch.cuda.synchronize()
        side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            run()
    for _ in range(3 if graph else 1):   # the next pass finds what the last one left behind
        ghat.fill_(float("nan"))
        g.replay() if graph else run()
        torch.cuda.synchronize()
    o_streams, o_scales, o_ghat = O.step(G_host, O.Csr(*csr, k), bits, w, mask, seed, step, api.AGC_SCALE_MAXABS)
    assert np.array_equal(scales.cpu().numpy().view(np.uint32).ravel(), o_scales.view(np.uint32).ravel())
    for i in range(n):
        assert np.array_equal(codes[i].cpu().numpy(), o_streams[i]), i
    assert np.array_equal(ghat.cpu().numpy().view(np.uint32), o_ghat.view(np.uint32))
    last = ctx.agc_debug_sketch_last()
    ctx.close()
    assert last["one_read"] and last["groups"] == -(-d // 1024) and not last["bound_failed"]
    return last


def _draw(rng, n, most):
    return (rng.integers(2, most + 1, n).astype(np.uint8), rng.uniform(0.2, 3.0, n).astype(np.float32),
            (rng.random(n) < 0.7).astype(np.uint8))


@pytest.mark.parametrize("kind,width", [("cyclic", s) for s in range(1, 9)] + [("interval", w) for w in (2, 4, 8)] + [("general", 5)])
@pytest.mark.parametrize("d", [1, 255, 1024, 40000 + 77])
def test_every_driver(kind, width, d):
    """Few values that are not zero, so that the records fit whatever the sample saw: a block has 266 / width +- 16 / sqrt(width)
    (one standard deviation) of them, each coded by at most `width` workers, and room for 512 records."""
    rng = np.random.default_rng([d, width, len(kind)])
    n = k = 13
    bits, w, mask = _draw(rng, n, 9)
    G = rng.standard_normal((k, d)) * (rng.random((k, d)) < 0.08 / width)
    last = _check(G.astype(np.float32), _code(rng, kind, n, k, width), k, bits, w, mask, graph=width == 4)
    assert last["left"] == 0


@pytest.mark.parametrize("n,most", [(1, 16), (2, 3), (7, 16), (8, 4), (9, 2), (31, 16), (33, 16), (64, 5), (97, 3), (161, 2), (256, 6)])
@pytest.mark.parametrize("law", ["normal", "layered", "sparse"])
def test_workers_widths_and_fills(n, most, law):
    """Blocks that overflow, all of them or some, and blocks that do not, in one to several fills of the staging area."""
    rng = np.random.default_rng([n, most])
    k, d = n, 3 * 1024 * 12 + 300
    csr = _code(rng, "cyclic" if n % 2 else "interval", n, k, 4)
    bits, w, mask = _draw(rng, n, most)
    G = rng.standard_normal((k, d))
    if law == "layered":
        G = G * np.repeat(10.0 ** rng.uniform(-4, 1, 36 + 1), 1024)[:d]
    elif law == "sparse":
        G = G * (rng.random((k, d)) < 0.01)
    last = _check(G.astype(np.float32), csr, k, bits, w, mask, unfused=n % 3 == 0)
    if law == "sparse":
        assert last["left"] == 0


@pytest.mark.parametrize("kind,width,n", [("cyclic", s, 13) for s in range(1, 9)] + [("interval", w, 13) for w in (2, 4, 8)]
                         + [("general", 5, 13), ("cyclic", 4, 70), ("interval", 4, 97), ("general", 5, 70), ("cyclic", 2, 161)])
def test_scales_that_the_sample_has_not_seen(kind, width, n):
    """The largest value of every row lies in one block, which in one of three trials at least is not one of the two that are sampled:
    the scales can only come from the sketch itself, whose bounds lay far below them (every value that is not 0 a record) in the
    blocks that began before that one was done."""
    rng = np.random.default_rng([n, width, len(kind)])
    d, k = 64 * 256 + 77, n
    bits, w, mask = _draw(rng, n, 9)
    csr = _code(rng, kind, n, k, width)
    G = (1e-3 * rng.standard_normal((k, d))).astype(np.float32)
    left = []
    for block in (0, 31, 64):
        one = G.copy()
        one[:, 256 * block + 5] = rng.uniform(40.0, 50.0, k)
        left.append(_check(one, csr, k, bits, w, mask)["left"])
    assert max(left) > 0


@pytest.mark.parametrize("records", [0, 1, 2, 255, 256, 257, 511, 512, 513, 768])
def test_records_around_the_ring_and_the_room(records):
    """A known number of them in every block: values of the scale's size, which always leave level 0, spread over the workers or
    all of the last ones.  Sixteen workers have room for 512."""
    rng = np.random.default_rng(records)
    n, d = 16, 5 * 1024 + 512
    csr = (np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), np.ones(n, np.float32))
    bits, w, mask = _draw(rng, n, 8)
    for spread in (True, False):
        G = np.zeros((n, d // 256, 256), np.float32)
        for b in range(d // 256):
            at = rng.choice(n * 256, records, replace=False) if spread else np.arange(n * 256 - records, n * 256)
            G[at // 256, b, at % 256] = rng.choice([-1.0, 1.0], records)
        last = _check(G.reshape(n, d), csr, n, bits, w, mask)
        assert last["left"] == (0 if records <= 512 else 6)


def test_ties_take_the_secondary_draw():
    """Every coordinate of a worker but one the same: a draw ties with the low half of the one grid position once in 65536."""
    rng = np.random.default_rng(6)
    n, d = 4, 200 * 1024
    csr = cyclic_csr(rng, n, 1)
    G = np.full((n, d), 1e-3, np.float32) * np.float32(1 + 0.1 * rng.random((n, 1)))
    G[:, 500] = 0.03
    bits = np.array([2, 3, 4, 4], np.uint8)
    ties = 0
    for i in range(n):
        f = O.encode(G, O.Csr(*csr, n), i)
        low = int(O.grid_pos(f[0], O.inv16(np.float32(np.abs(f).max()), bits[i]), bits[i])) & 0xFFFF
        ties += sum(O.draw(77, 9, i, m)[0] == low for m in range(d))
    assert ties >= 4, ties
    _check(G, csr, n, bits, np.ones(n, np.float32), np.ones(n, np.uint8))


def _outputs(ctx, G, bits, w, mask):
    import torch
    codes, scales, ghat = ctx.alloc_outputs(bits)
    ctx.agc_step(G, bits, w, mask, 3, 4, codes, scales, ghat)
    torch.cuda.synchronize()
    return ([c.cpu().numpy() for c in codes] + [scales.cpu().numpy().view(np.uint32).ravel(), ghat.cpu().numpy()],
            ctx.agc_debug_sketch_last())


@pytest.mark.parametrize("value", [np.nan, np.inf, 3e38, 1e-42])
@pytest.mark.parametrize("as_weight", [False, True])
def test_extreme_values_give_what_two_reads_give(value, as_weight):
    rng = np.random.default_rng(9)
    n, d = 6, 70 * 1024 + 5
    bits, w, mask = _draw(rng, n, 4)
    mask[:] = 1
    G = (rng.standard_normal((n, d)) * (rng.random((n, d)) < 0.02)).astype(np.float32)
    if as_weight:
        w[1] = value
    else:
        G[2, 4321] = value
    csr, G = cyclic_csr(rng, n, 2), to_device(G)
    outs = []
    for mode in (1, 2):
        ctx = api.Context(n, n, d)
        ctx.agc_set_code(*csr)
        ctx.agc_debug_sketch_max(mode)
        out, last = _outputs(ctx, G, bits, w, mask)
        outs.append(out)
        assert last["one_read"] == (mode == 1)
        ctx.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b, equal_nan=a.dtype == np.float32)


@pytest.mark.parametrize("law", ["heavy", "alike"])
def test_the_sample_decides(law):
    """Sizes that the rule takes.  Heavy tails take one read; where values are alike everywhere the sample sees that the blocks
    would overflow and two reads are made; layers, and a return from them."""
    import torch
    rng = np.random.default_rng(10)
    n, d = 32, (1 << 25) + 333
    bits, w, mask = np.full(n, 3, np.uint8), np.ones(n, np.float32), (rng.random(n) < 0.7).astype(np.uint8)
    csr = cyclic_csr(rng, n, 3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    G = api.padded_rows(n, d)
    for j in range(n):
        G[j].normal_(generator=gen)
        if law == "heavy":
            G[j].pow_(7)
    outs = []
    for mode in (0, 2):
        ctx = api.Context(n, n, d)
        ctx.agc_set_code(*csr)
        ctx.agc_debug_sketch_max(mode)
        for layers in ([], [1 << 24, d], []):
            ctx.agc_set_layers(np.array(layers, np.int64))
            out, last = _outputs(ctx, G, bits, w, mask)
            assert last["one_read"] == (mode == 0 and not layers)
            if last["one_read"]:
                assert last["bound_failed"] == (law == "alike")
                assert last["left"] == last["groups"] if law == "alike" else last["left"] < last["groups"] // 10
            outs.append(out)
        ctx.close()
    for a, b in zip(outs[:3], outs[3:]):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
    assert all(np.array_equal(x, y) for x, y in zip(outs[0], outs[2]))


@pytest.mark.parametrize("rooms", [0.5, 0.9, 1.1])
def test_bounded_values_take_one_read_where_it_is_faster(rooms):
    """Values of which one in a hundred is the largest there is, so the sample's bounds do not rise, and as many records in a block
    as the stated part of its room: 32 workers with two bits have 8192 coded values and room for 1024.  Records of a block
    are within 1024 * rooms +- 31 (one standard deviation), the expectations of the sampled blocks within 1 % of each other, and what
    these cost, half the part that they fill or all, is to be at most 0.5 - 4 / 32."""
    import torch
    rng = np.random.default_rng(12)
    n, d = 32, (1 << 25) + 333
    bits, w, mask = np.full(n, 2, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    G = api.padded_rows(n, d)
    for j in range(n):
        G[j].normal_(generator=gen).mul_((rooms / 8 - 0.01) / 0.99 / (2 / np.pi) ** 0.5)
        largest = torch.rand(d, device="cuda", generator=gen) < 0.01
        G[j][largest] = torch.sign(G[j][largest])
    csr = cyclic_csr(rng, n, 1)
    outs = []
    for mode in (0, 2):
        ctx = api.Context(n, n, d)
        ctx.agc_set_code(*csr)
        ctx.agc_debug_sketch_max(mode)
        out, last = _outputs(ctx, G, bits, w, mask)
        ctx.close()
        assert last["one_read"] == (mode == 0)
        if mode == 0:
            assert last["bound_failed"] == (rooms > 0.75)
            assert last["left"] == (last["groups"] if rooms > 0.75 else 0)
        outs.append(out)
    assert all(np.array_equal(a, b) for a, b in zip(*outs))


def test_the_hook_keeps_its_mode():
    """Forced by the hook, the sample does not decide, also with the workspace that is taken again after layers; the hook of the other
    kind of scale changes nothing.  Back by the rule, a vector this short is read twice."""
    rng = np.random.default_rng(13)
    n, d = 16, 64 * 256
    bits, w, mask = np.full(n, 8, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    csr, G = cyclic_csr(rng, n, 2), to_device(rng.standard_normal((n, d)).astype(np.float32))   # alike: every block overflows
    ctx = api.Context(n, n, d)
    ctx.agc_set_code(*csr)
    ctx.agc_debug_sketch_max(1)
    outs = []
    for between in (lambda: None, lambda: (ctx.agc_set_layers(np.array([256, d], np.int64)), ctx.agc_set_layers(np.array([], np.int64))),
                    lambda: ctx.agc_debug_sketch(0), lambda: ctx.agc_debug_sketch(2), lambda: ctx.agc_set_code(*csr)):
        between()
        out, last = _outputs(ctx, G, bits, w, mask)
        assert last["one_read"] and not last["bound_failed"] and last["left"] > 0
        outs.append(out)
    ctx.agc_debug_sketch_max(0)
    out, last = _outputs(ctx, G, bits, w, mask)
    assert not last["one_read"]
    for other in outs:
        assert all(np.array_equal(a, b) for a, b in zip(out, other))
    ctx.close()


def test_the_hook_refuses_other_scales():
    for kw in (dict(scale_mode=api.AGC_SCALE_L2), dict(bucket=256)):
        ctx = api.Context(2, 2, 4096, **kw)
        with pytest.raises(api.AgcError):
            ctx.agc_debug_sketch_max(1)
        ctx.close()
    ctx = api.Context(2, 2, 4096)
    with pytest.raises(api.AgcError):
        ctx.agc_debug_sketch_max(3)
    ctx.close()
