"""The form with one read of G (Euclidean scale of the whole vector): forced at small sizes by its testing hook, every
driver, one and several fills of the staging area, blocks and groups that end inside the vector, blocks with more records
than there is room for, samples that mislead in either direction, values and weights that are not finite.  Codes, scales
and estimates equal the oracle's bit for bit, twice in a row and from a replayed graph.  A block with more records than there
is room for takes the kernel of the two-read form, so every test also asks which groups of blocks did."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

from gpu_util import cyclic_csr, monotone_csr, random_csr, to_device

pytestmark = pytest.mark.gpu


def _code(rng, kind, n, k, width):
    return (cyclic_csr(rng, n, min(n, width)) if kind == "cyclic" else monotone_csr(rng, n, k, width) if kind == "interval"
            else random_csr(rng, n, k, width))


M64 = 2 ** 64 - 1


def _mix(x):
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & M64
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & M64
    return x ^ (x >> 31)


def _sampled_blocks(d, seed, step):
    """The blocks that the bounds are estimated from (sample_block in csrc/agc_dispatch.h)."""
    nblocks = -(-d // 256)
    samples = min(max(nblocks // 32, 1), 512)
    length, longer = divmod(nblocks, samples)
    golden = 0x9E3779B97F4A7C15
    salt = _mix((seed + _mix((step + golden) & M64)) & M64)
    return [e * length + min(e, longer) + (((_mix((salt + golden * e) & M64) >> 32) * (length + (e < longer))) >> 32)
            for e in range(samples)]


def _check(G_host, csr, k, bits, w, mask, unfused=False, graph=False, seed=77, step=9, oracle=None):
    """What agc_debug_sketch_last says of the last pass."""
    import torch
    n, d = len(bits), G_host.shape[1]
    ctx = api.Context(n, k, d, scale_mode=api.AGC_SCALE_L2, unfused_step=unfused)
    ctx.agc_set_code(*csr)
    ctx.agc_debug_sketch(1)
    codes, scales, ghat = ctx.alloc_outputs(bits)
    for t in codes:
        t.fill_(0x5A)
    ghat.fill_(float("nan"))
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
        if graph:
            ghat.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
        else:
            run()
    torch.cuda.synchronize()
    o_streams, o_scales, o_ghat = oracle or O.step(G_host, O.Csr(*csr, k), bits, w, mask, seed, step, api.AGC_SCALE_L2)
    assert np.array_equal(scales.cpu().numpy().view(np.uint32).ravel(), o_scales.view(np.uint32).ravel())
    for i in range(n):
        assert np.array_equal(codes[i].cpu().numpy(), o_streams[i]), i
    got = ghat.cpu().numpy()
    nan = np.isnan(o_ghat)   # the payload of a NaN is nobody's contract
    assert np.array_equal(np.isnan(got), nan) and np.array_equal(got.view(np.uint32)[~nan], o_ghat.view(np.uint32)[~nan])
    last = ctx.agc_debug_sketch_last()
    ctx.close()
    assert last["one_read"] and last["groups"] == -(-d // 1024)
    return last


def _draw(rng, n, most):
    return (rng.integers(2, most + 1, n).astype(np.uint8), rng.uniform(0.2, 3.0, n).astype(np.float32),
            (rng.random(n) < 0.7).astype(np.uint8))


@pytest.mark.parametrize("kind,width", [("cyclic", s) for s in range(1, 9)] + [("interval", w) for w in (2, 4, 8)] + [("general", 5)])
@pytest.mark.parametrize("d", [1, 255, 1024, 40000 + 77])
def test_every_driver(kind, width, d):
    """Widths whose records fit at these lengths."""
    rng = np.random.default_rng([d, width, len(kind)])
    n = k = 13
    bits, w, mask = _draw(rng, n, {1: 6, 255: 2, 1024: 2}.get(d, 4))
    last = _check(rng.standard_normal((k, d)).astype(np.float32), _code(rng, kind, n, k, width), k, bits, w, mask)
    assert last["left"] == 0 and not last["bound_failed"]


@pytest.mark.parametrize("n,most", [(1, 16), (2, 3), (7, 16), (8, 4), (9, 2), (31, 16), (32, 9), (33, 16), (64, 5), (97, 3),
                                    (161, 2), (256, 2), (256, 6)])
@pytest.mark.parametrize("law", ["normal", "heavy", "layered", "sparse"])
def test_workers_widths_and_fills(n, most, law):
    """Wide codes overflow their blocks' room for records (all, or with layers of very different size some of them), the rest
    of the group's blocks and of the vector do not.  With few values that are not zero wide codes fit as well, in one to
    thirteen fills."""
    rng = np.random.default_rng([n, most])
    k, d = n, 3 * 1024 * 12 + 300 if n < 256 or law != "sparse" else 1024 * 300 + 300
    csr = _code(rng, "cyclic" if n % 2 else "interval", n, k, 4)
    bits, w, mask = _draw(rng, n, most)
    G = rng.standard_normal((k, d))
    if law == "heavy":
        G = G * np.exp(2.0 * rng.standard_normal((k, d)))
    elif law == "layered":
        G = G * np.repeat(10.0 ** rng.uniform(-4, 1, 36 + 1), 1024)[:d]
    elif law == "sparse":
        G = G * (rng.random((k, d)) < (0.01 if n <= 33 else 0.05 if n < 256 else 0.0015))
    last = _check(G.astype(np.float32), csr, k, bits, w, mask, unfused=n % 3 == 0, graph=n == 33)
    if law == "sparse":
        assert last["left"] <= last["groups"] // 4 and not last["bound_failed"]


@pytest.mark.parametrize("kind,n,k,width", [("general", 5, 1, 1), ("general", 5, 17, 17), ("general", 33, 127, 9), ("general", 3, 128, 128),
                                            ("general", 7, 129, 70), ("interval", 128, 128, 8), ("interval", 140, 150, 4)])
def test_rows_that_the_sample_holds_and_more(kind, n, k, width):
    """Up to 128 rows of a sampled block wait in LDS, more are gathered; rows of the code shorter and longer than a wave."""
    rng = np.random.default_rng([n, k])
    for d, most in ((500, 2), (64 * 256 + 77, 4)) if n < 100 else ((128 * 256 + 77, 2),):
        last = _check(rng.standard_normal((k, d)).astype(np.float32), _code(rng, kind, n, k, width), k, *_draw(rng, n, most))
        assert last["left"] <= (last["groups"] // 4 if d > 500 else 0) and not last["bound_failed"]


@pytest.mark.parametrize("where", ["one", "two", "three", "elsewhere", "nowhere", "sign", "large", "small"])
def test_samples_that_mislead(where):
    """Eight of 280 blocks are sampled and the two largest left out.  All of the vector's norm in one or two of them, or in none:
    there is no bound, and the blocks that hold it overflow.  In three: the bound lies above the scale and everything
    takes the second read."""
    rng = np.random.default_rng(5)
    n = k = 11
    d = 70 * 1024
    sampled = _sampled_blocks(d, 77, 9)
    assert len(sampled) == 8 and len(set(sampled)) == 8
    loud = {"one": sampled[2:3], "two": sampled[3:5], "three": sampled[1:8:3], "nowhere": [],
            "elsewhere": [b for b in range(20, 36) if b not in sampled]}.get(where, range(280))
    csr = cyclic_csr(rng, n, 3)
    bits, w, mask = _draw(rng, n, 3 if where == "large" else 8)
    G = np.zeros((k, 280, 256), np.float32)
    G[:, list(loud)] = rng.standard_normal((k, len(loud), 256))
    G = G.reshape(k, d)
    if where == "sign":
        G = np.copysign(np.float32(0), rng.standard_normal((k, d))).astype(np.float32)
        G[:, 3] = 1.0
    G *= np.float32({"large": 1e18, "small": 1e-42}.get(where, 1.0))
    last = _check(G, csr, k, bits, w, mask)
    assert last["bound_failed"] == (where == "three")
    assert where == "small" or last["left"] == {"three": 70, "nowhere": 0, "sign": 0, "large": 0}.get(where, len({b // 4 for b in loud}))


def test_ties_take_the_secondary_draw():
    """Every coordinate of a worker the same: a draw ties with the low half of the one grid position once in 65536."""
    rng = np.random.default_rng(6)
    n = k = 4
    d = 200 * 1024
    bits, w, mask = np.array([2, 3, 4, 4], np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    csr = cyclic_csr(rng, n, 1)
    G = np.full((k, d), 1e-3, np.float32) * np.float32(1 + 0.1 * rng.random((k, 1)))
    ties = 0
    for i in range(n):
        f = O.encode(G, O.Csr(*csr, k), i)
        low = int(O.grid_pos(f[0], O.inv16(O.scale_l2(f), bits[i]), bits[i])) & 0xFFFF
        ties += sum(O.draw(77, 9, i, m)[0] == low for m in range(d))
    assert ties >= 4, ties
    last = _check(G, csr, k, bits, w, mask)
    assert last["left"] == 0 and not last["bound_failed"]


@pytest.mark.parametrize("weight", [0.0, -0.0, -2.5, 1e-38, 3e38])
def test_weights(weight):
    rng = np.random.default_rng(8)
    n = k = 6
    bits, w, mask = _draw(rng, n, 4)
    w[:3] = weight
    mask[:] = 1
    last = _check(rng.standard_normal((k, 5000)).astype(np.float32), cyclic_csr(rng, n, 2), k, bits, w, mask)
    assert last["bound_failed"] == (weight == 3e38) and last["left"] == (5 if weight == 3e38 else 0)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("as_weight", [False, True])
def test_what_is_not_finite_gives_what_two_reads_give(value, as_weight):
    """Against the form with two reads, since the oracle defines nothing here: scales, codes and estimates."""
    import torch
    rng = np.random.default_rng(9)
    n, k, d = 6, 6, 70 * 1024 + 5
    csr = cyclic_csr(rng, n, 2)
    bits, w, mask = _draw(rng, n, 4)
    G = rng.standard_normal((k, d)).astype(np.float32)
    if as_weight:
        w[1] = value
        mask[1] = 1
    else:
        G[2, 4321] = value
    outs = []
    for mode in (1, 2):
        ctx = api.Context(n, k, d, scale_mode=api.AGC_SCALE_L2)
        ctx.agc_set_code(*csr)
        ctx.agc_debug_sketch(mode)
        codes, scales, ghat = ctx.alloc_outputs(bits)
        ctx.agc_step(to_device(G), bits, w, mask, 3, 4, codes, scales, ghat)
        torch.cuda.synchronize()
        outs.append([c.cpu().numpy() for c in codes] + [scales.cpu().numpy().view(np.uint32), ghat.cpu().numpy()])
        last = ctx.agc_debug_sketch_last()
        assert last["one_read"] == (mode == 1) and last["left"] == last["groups"] and last["bound_failed"] == (mode == 1)
        ctx.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b, equal_nan=a.dtype == np.float32)


def test_the_rule_takes_it_and_layers_do_not():
    """A vector long enough for the rule, ragged end, in a context whose layers are switched on and off; the last pass on a
    stream of its own."""
    import torch
    rng = np.random.default_rng(10)
    n, k, d = 32, 32, (1 << 20) + 333
    csr = cyclic_csr(rng, n, 3)
    bits, w, mask = _draw(rng, n, 4)
    G_host = rng.standard_normal((k, d)).astype(np.float32)
    G = to_device(G_host)
    outs = []
    side = torch.cuda.Stream()
    for mode in (0, 2):
        ctx = api.Context(n, k, d, scale_mode=api.AGC_SCALE_L2)
        ctx.agc_set_code(*csr)
        ctx.agc_debug_sketch(mode)
        for turn, layers in enumerate(([], [512 * 256, d], [], [])):
            if turn in (1, 2):
                ctx.agc_set_layers(np.array(layers, np.int64))
            codes, scales, ghat = ctx.alloc_outputs(bits)
            ghat.fill_(float("nan"))
            if turn == 3:
                side.wait_stream(torch.cuda.current_stream())
                with torch.cuda.stream(side):
                    ctx.agc_step(G, bits, w, mask, 3, 4, codes, scales, ghat)
            else:
                ctx.agc_step(G, bits, w, mask, 3, 4, codes, scales, ghat)
            torch.cuda.synchronize()
            last = ctx.agc_debug_sketch_last()
            assert last["one_read"] == (mode == 0 and not layers) and last["left"] == 0 and not last["bound_failed"]
            outs.append([c.cpu().numpy() for c in codes] + [scales.cpu().numpy().view(np.uint32).ravel(), ghat.cpu().numpy().view(np.uint32)])
        ctx.close()
    for a, b in zip(outs[:4], outs[4:]):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
    for again in outs[2:4]:
        assert all(np.array_equal(x, y) for x, y in zip(outs[0], again))
    o_streams, o_scales, o_ghat = O.step(G_host, O.Csr(*csr, k), bits, w, mask, 3, 4, api.AGC_SCALE_L2)
    assert all(np.array_equal(x, y) for x, y in zip(outs[0], [*o_streams, o_scales.view(np.uint32).ravel(), o_ghat.view(np.uint32)]))


@pytest.mark.parametrize("width", [4096, 16384])
@pytest.mark.parametrize("first,width_of_codes", [(20.0, 2), (0.05, 4)])
def test_gradients_made_of_matrices_do_not_mislead_the_sample(width, first, width_of_codes):
    """The first 256 columns of every row much larger or smaller than the others: neither fails the bounds nor puts them so low
    that blocks overflow."""
    rng = np.random.default_rng(12)
    n, d = 12, 1 << 20
    bits, w, mask = np.full(n, width_of_codes, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    G_host = rng.standard_normal((n, d), dtype=np.float32).reshape(n, -1, width)
    G_host[:, :, :256] *= np.float32(first)
    G = to_device(G_host.reshape(n, d))
    ctx = api.Context(n, n, d, scale_mode=api.AGC_SCALE_L2)
    ctx.agc_set_code(*cyclic_csr(rng, n, 2))
    ctx.agc_debug_sketch(1)
    codes, scales, ghat = ctx.alloc_outputs(bits)
    for step in range(6):
        ctx.agc_step(G, bits, w, mask, 2, step, codes, scales, ghat)
        assert ctx.agc_debug_sketch_last() == dict(one_read=True, groups=1024, left=0, bound_failed=False), step
    ctx.close()


def test_a_norm_in_one_part_of_the_vector_is_seen():
    """All but a millionth of it in a 32nd: two of the sampled blocks are left out of the bound, and it must not be two of two."""
    rng = np.random.default_rng(14)
    n, d = 12, 1 << 20
    bits, w, mask = np.full(n, 2, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    G = to_device(rng.standard_normal((n, d), dtype=np.float32))
    G[:, d // 3: d // 3 + d // 32] *= 200
    ctx = api.Context(n, n, d, scale_mode=api.AGC_SCALE_L2)
    ctx.agc_set_code(*cyclic_csr(rng, n, 2))
    ctx.agc_debug_sketch(1)
    codes, scales, ghat = ctx.alloc_outputs(bits)
    for step in range(6):
        ctx.agc_step(G, bits, w, mask, 2, step, codes, scales, ghat)
        assert ctx.agc_debug_sketch_last() == dict(one_read=True, groups=1024, left=0, bound_failed=False), step
    ctx.close()


def test_groups_left_over_are_spread_over_the_chip():
    """The same number of blocks with more records than there is room for, one in every 64 of the vector or one in every four
    of its first sixteenth: the kernels behind the scales take the same time (on one of the eight dies alone the former
    would take several times as long as on all)."""
    rng = np.random.default_rng(13)
    n, d = 32, 1 << 23
    bits, w, mask = np.full(n, 8, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    ctx = api.Context(n, n, d, scale_mode=api.AGC_SCALE_L2)
    ctx.agc_set_code(*cyclic_csr(rng, n, 2))
    ctx.agc_debug_sketch(1)
    codes, scales, ghat = ctx.alloc_outputs(bits)
    G = to_device(rng.standard_normal((n, d), dtype=np.float32))
    G.view(n, -1, 256)[:, ::64] *= 20
    took = []
    for _ in range(2):
        best = float("inf")
        for step in range(12):
            ctx.agc_profile_enable(step >= 2)
            ctx.agc_profile_read()
            ctx.agc_step(G, bits, w, mask, 2, step, codes, scales, ghat)
            last = ctx.agc_debug_sketch_last()
            assert last["left"] == 512 and not last["bound_failed"], last
            if step >= 2:
                best = min(best, ctx.agc_profile_read()["quantize"][0])
        took.append(best)
        blocks = G.view(n, -1, 256)
        blocks[:, ::64] /= 20
        blocks[:, :2048:4] *= 20
    ctx.close()
    assert took[0] < 1.35 * took[1], took


def test_memory_is_held_only_where_a_step_can_use_it():
    """Signs and records come with the code (a program that only decodes sets none), go with layers and come back without them."""
    import torch
    rng = np.random.default_rng(15)
    n, d = 64, 1 << 22
    need = (d // 256) * (2 * 1024 + 8 * 900)   # more than 900 records a block

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]
    before = free()
    ctx = api.Context(n, n, d, scale_mode=api.AGC_SCALE_L2)
    assert before - free() < need // 4
    ctx.agc_set_code(*cyclic_csr(rng, n, 4))
    with_code = free()
    assert before - with_code > need
    ctx.agc_set_layers(np.array([d // 2, d], np.int64))
    assert before - free() < need // 4
    ctx.agc_set_layers([])
    assert before - free() > need
    ctx.agc_debug_sketch(2)
    assert before - free() < need // 4
    ctx.agc_debug_sketch(0)
    assert before - free() > need
    ctx.close()
    assert before - free() < need // 4


def test_the_hook_tells_the_form():
    rng = np.random.default_rng(11)
    n, d = 5, 40 * 1024 + 9
    bits, w, mask = np.full(n, 2, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8)
    G = rng.standard_normal((n, d)).astype(np.float32)
    G[:, 7 * 1024: 8 * 1024] *= 1e4   # four of the 161 blocks hold the norm: more records than there is room for
    ctx = api.Context(n, n, d, scale_mode=api.AGC_SCALE_L2)
    ctx.agc_set_code(*cyclic_csr(rng, n, 2))
    codes, scales, ghat = ctx.alloc_outputs(bits)
    none = dict(one_read=False, groups=0, left=0, bound_failed=False)
    assert ctx.agc_debug_sketch_last() == none
    ctx.agc_debug_sketch(1)
    ctx.agc_step(to_device(G), bits, w, mask, 1, 2, codes, scales, ghat)
    last = ctx.agc_debug_sketch_last()
    assert last["one_read"] and last["groups"] == 41 and not last["bound_failed"] and last["left"] == 1
    ctx.agc_debug_sketch(2)
    ctx.agc_step(to_device(G), bits, w, mask, 1, 2, codes, scales, ghat)
    assert ctx.agc_debug_sketch_last() == none
    ctx.close()


def test_the_hook_refuses_other_scales():
    for kw in (dict(scale_mode=api.AGC_SCALE_MAXABS), dict(scale_mode=api.AGC_SCALE_L2, bucket=256)):
        ctx = api.Context(2, 2, 4096, **kw)
        with pytest.raises(api.AgcError):
            ctx.agc_debug_sketch(1)
        with pytest.raises(api.AgcError):
            ctx.agc_debug_sketch(3)
        ctx.close()


@pytest.mark.parametrize("groups", [1024, 1025, 1280, 1281])
@pytest.mark.parametrize("n,most", [(64, 5), (5, 16), (131, 4)])
@pytest.mark.parametrize("fused", [True, False])
def test_fills_by_the_length_of_the_vector(groups, n, most, fused):
    """Four, five and six workgroups of the code-making kernel on a compute unit have fills of their own: the lengths where their
    number changes, in one to many fills, against two reads."""
    import torch
    rng = np.random.default_rng([groups, n])
    d = groups * 1024 - 77
    csr = cyclic_csr(rng, n, 3)
    bits, w, mask = rng.integers(2, most + 1, n).astype(np.uint8), rng.uniform(0.2, 3.0, n).astype(np.float32), (rng.random(n) < 0.7).astype(np.uint8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    G = api.padded_rows(n, d)
    G.normal_(generator=gen)
    if most == 16:   # every value that is not 0 is a record: 77 +- 15 of them in a block (one standard deviation), room for 160
        G.mul_(torch.rand(G.shape, device="cuda", generator=gen) < 0.02)
    outs = []
    for mode in (1, 2):
        ctx = api.Context(n, n, d, scale_mode=api.AGC_SCALE_L2, unfused_step=not fused)
        ctx.agc_set_code(*csr)
        ctx.agc_debug_sketch(mode)
        codes, scales, ghat = ctx.alloc_outputs(bits)
        ctx.agc_step(G, bits, w, mask, 3, 4, codes, scales, ghat)
        torch.cuda.synchronize()
        last = ctx.agc_debug_sketch_last()
        ctx.close()
        assert last["one_read"] == (mode == 1)
        if mode == 1:
            assert last["groups"] == groups and not last["bound_failed"] and last["left"] < groups // 10
        outs.append([*codes, scales.view(torch.int32), ghat.view(torch.int32)])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
