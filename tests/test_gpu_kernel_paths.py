"""Small GPU tests of single kernel paths at the sizes and alignments where they can go wrong."""
import ctypes
import time

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import oracle
    import paper_2303_02868_amd as apm
    from gpu_helpers import DEV


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [1, 7, 9, 100, 511, 512, 1024, 1025, 2048, 2049, 4095, 4097, 3 * 4096 + 5])
def test_pack_and_unpack_at_every_address_are_bit_exact_and_write_nothing_else(dtype, n):
    """Any byte address on either side (vectors, head and tail of the copy kernel): pages and tensors
    hold the same bytes, and the bytes around an unpacked tensor keep their value."""
    E, eb = 4096, 2 if dtype == "bf16" else 4
    kind, st = (apm.APM_BF16, apm.APM_G16) if dtype == "bf16" else (apm.APM_F32, apm.APM_P32)
    raw = torch.randint(0, 256, (n * eb + 32,), dtype=torch.uint8, device=DEV,
                        generator=torch.Generator(device=DEV).manual_seed(n))
    for src_off in (0, 1, 2, 4, 6, 8, 13, 16):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, 5, state_mask=1 << st)
        apm.apm_pack_tensors(pool, st, apm.make_tensors([n], kind, [raw.data_ptr() + src_off]), 1)
        for dst_off in (0, 1, 2, 4, 6, 8, 13):
            out = torch.full((n * eb + 32,), 77, dtype=torch.uint8, device=DEV)
            apm.apm_unpack(pool, st, apm.make_tensors([n], kind, [out.data_ptr() + dst_off]), 1)
            torch.cuda.synchronize()
            assert torch.equal(out[dst_off:dst_off + n * eb], raw[src_off:src_off + n * eb]), (src_off, dst_off)
            assert (out[:dst_off] == 77).all() and (out[dst_off + n * eb:] == 77).all(), (src_off, dst_off)
        pool.destroy()


@pytest.mark.parametrize("n_t", [1, 439, 440, 441, 880, 881, 2500])
def test_pack_and_unpack_of_many_tensors_are_bit_exact(n_t):
    """Tensor counts around what one launch carries in its arguments and around the count from which
    the addresses are staged; empty tensors, tiny ones and ones of several pages, in mixed order."""
    E = 512
    numels = [(0, 3, E - 1, E, 2 * E + 5, 17)[(7 * k) % 6] for k in range(n_t)]
    numels[-1] = E + 9
    off = [sum(numels[:k]) for k in range(n_t)]
    src = torch.arange(sum(numels), device=DEV, dtype=torch.float32)
    dst = torch.full_like(src, -1.0)
    n_pages = sum(-(-n // E) for n in numels)
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n_pages, state_mask=1)
    lists = [apm.make_tensors(numels, apm.APM_F32, [t.data_ptr() + 4 * o for o in off]) for t in (src, dst)]
    apm.apm_pack_tensors(pool, apm.APM_P32, lists[0], n_t)
    apm.apm_unpack(pool, apm.APM_P32, lists[1], n_t)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)
    pool.destroy()


@pytest.mark.parametrize("numels,align", [([1000, 17, 70000, 300001, 9] * 3, 1), ([1000, 17, 70000, 300001, 9] * 3, 4), ([5] * 3 + [4099] * 5 + [1 << 21], 16),
                                          ([32 << 20, 12345, 7, (1 << 19) + 1, 300], 16), ([32 << 20, 12345, 7, (1 << 19) + 1, 300], 1),
                                          ([(66 << 20) + 5, 300, (1 << 19) + 1], 16)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pack_and_unpack_of_long_and_short_segments_are_bit_exact(dtype, numels, align):
    """Segments of all length classes in one grid; aligned lists below and above the size from which a
    workgroup is one wavefront, and views of one flat buffer at odd distances.  The pages hold what the oracle's plan
    says, and nothing else."""
    kind, st, dt = (apm.APM_BF16, apm.APM_G16, torch.int16) if dtype == "bf16" else (apm.APM_F32, apm.APM_P32, torch.int32)
    E, n_t, off, at = 65536, len(numels), [], 0
    for k, n in enumerate(numels):
        at += -at % align + (k % 5 if align == 1 else 0)
        off.append(at)
        at += n
    src = torch.randint(-30000, 30000, (at + 64,), device=DEV, dtype=dt, generator=torch.Generator(device=DEV).manual_seed(at))
    out = torch.full_like(src, -7)
    want = torch.full_like(src, -7)
    plan = oracle.plan_pack(numels, E)
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, sum(-(-n // E) for n in numels), state_mask=1 << st)
    lists = [apm.make_tensors(numels, kind, [t.data_ptr() + o * t.element_size() for o in off]) for t in (src, out)]
    apm.apm_pack_tensors(pool, st, lists[0], n_t)
    apm.apm_unpack(pool, st, lists[1], n_t)
    torch.cuda.synchronize()
    pages = torch.as_tensor(_Region(pool, st, plan.n_pages * E * src.element_size() // 2), device=DEV).view(dt).view(plan.n_pages, E)
    placed = torch.zeros_like(pages)
    for s in plan.segments:
        at = off[s.tensor] + s.tensor_off
        placed[s.page, s.page_off:s.page_off + s.n] = src[at:at + s.n]
    assert torch.equal(pages, placed)
    for o, n in zip(off, numels):
        want[o:o + n] = src[o:o + n]
    assert torch.equal(out, want)
    pool.destroy()


@pytest.mark.parametrize("clip", [0.0, 0.01])
@pytest.mark.parametrize("n_t,listed", [(1, "all"), (147, "odd"), (219, "all"), (221, "reversed"), (441, "all"), (450, "reversed"),
                                        (700, "odd"), (900, "all"), (1500, "reversed")])
def test_fused_step_equals_the_page_step_for_any_tensor_count_and_list(n_t, listed, clip):
    """Gradients read from / parameters written to tensors against the same gradients packed into
    pages: same kernels, so the same bits.  Counts around what one stage launch carries (440 words:
    a listed page, a gradient address, a parameter address each take one), several launches, the ring."""
    E = 512
    numels = [(3, E - 1, E, 2 * E + 5, 17)[(3 * k) % 5] for k in range(n_t)]
    off = [0]
    for n in numels:
        off.append(off[-1] + (n + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(n_t)
    g = (torch.randn(off[-1], device=DEV, generator=gen) * 1e-3).bfloat16()
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, apm.APM_SKIP_NONE)
    got = []
    for fused in (False, True):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, sum(-(-n // E) for n in numels) + 3)
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)
        n = apm.lib().apm_pool_pages_in_use(pool.handle)
        pages = {"all": None, "odd": list(range(1, n, 2)), "reversed": list(range(n))[::-1]}[listed]
        count = n if pages is None else len(pages)
        norm = torch.zeros(count, device=DEV) if count else torch.zeros(1, device=DEV)
        q = torch.zeros_like(g)
        if fused:
            apm.apm_page_adamw_step_fused(pool, pages, count, 3, hyper, lst(g), lst(q), n_t, norm, None)
        else:
            apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
            apm.apm_page_adamw_step(pool, pages, count, 3, hyper, norm, None)
            apm.apm_unpack(pool, apm.APM_P16, lst(q), n_t)
        out = [norm, q]
        for st in (apm.APM_P32, apm.APM_M32, apm.APM_V32):
            out.append(torch.zeros_like(p0))
            apm.apm_unpack(pool, st, lst(out[-1]), n_t)
        torch.cuda.synchronize()
        got.append(out)
        pool.destroy()
    assert got[0][2].ne(p0).any() or listed == "odd"
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("E,numels", [(8, [8, 3, 17]), (16384, [16384, 16383, 40000, 5]), (32776, [32776 * 3 + 257, 16385, 70001, 1]),
                                      (66 * 16384, [66 * 16384 + 12345, 64 * 16384 + 1, 66 * 16384 * 2, 300])])
@pytest.mark.parametrize("form", ["run", "reversed", "fused"])
def test_clipped_update_with_and_without_waiting(E, numels, form):
    """The clipped update hands sums and scales from wavefront to wavefront: the same bits when every
    wavefront computes them by itself; norms against 64 bits (an fp32 rounding of an fp64 sum)."""
    n_t, off = len(numels), [0]
    for n in numels:
        off.append(off[-1] + (n + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(E)
    g = (torch.randn(off[-1], device=DEV, generator=gen) * 1e-2).bfloat16()
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.05, apm.APM_SKIP_NONE)
    got = []
    for wait in (True, False):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, sum(-(-n // E) for n in numels) + 1)
        if not wait:   # wavefronts compute what they would wait for
            assert apm.lib().apm_test_set_wait_limit(ctypes.c_void_p(pool.handle), 0) == 0
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)
        apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        n = apm.lib().apm_pool_pages_in_use(pool.handle)
        norm, q = torch.full((n,), -1.0, device=DEV), torch.zeros_like(g)
        pages = list(range(n))[::-1] if form == "reversed" else None
        if form == "fused":
            apm.apm_page_adamw_step_fused(pool, pages, n, 3, hyper, lst(g), lst(q), n_t, norm, None)
        else:
            apm.apm_page_adamw_step(pool, pages, n, 3, hyper, norm, None)
            apm.apm_unpack(pool, apm.APM_P16, lst(q), n_t)
        out = [norm, q]
        for st in (apm.APM_P32, apm.APM_M32, apm.APM_V32):
            out.append(torch.zeros_like(p0))
            apm.apm_unpack(pool, st, lst(out[-1]), n_t)
        torch.cuda.synchronize()
        got.append(out)
        pool.destroy()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    plan = oracle.plan_pack(numels, E)
    sq = torch.zeros(n, dtype=torch.float64, device=DEV)
    for s in plan.segments:
        sq[s.page] += g[off[s.tensor] + s.tensor_off:off[s.tensor] + s.tensor_off + s.n].double().square().sum()
    want = sq.sqrt().flip(0) if form == "reversed" else sq.sqrt()
    assert torch.allclose(got[0][0].double(), want, rtol=2.0 ** -23, atol=0.0)


@pytest.mark.parametrize("clip,skip,norms", [(0.0, 0, False), (0.02, 0, True), (0.02, 1, True)])
@pytest.mark.parametrize("listed,micro,shift", [("all", 1, 0), ("all", 3, 0), ("reversed", 2, 0), ("odd", 2, 0), ("all", 2, 1), ("middle", 2, 0), ("more", 2, 0)])
@pytest.mark.parametrize("E,n_t", [(8, 3), (8, 5000), (2056, 1000), (4104, 1000), (49160, 9)])
def test_delayed_hand_over_equals_the_synchronous_step(E, n_t, listed, micro, shift, clip, skip, norms):
    """The hand-over copies used extents and leaves sums for the update; further micro-batches are added in
    bf16.  Same bits as a synchronous step on the summed gradient: extents around the copy's and the sums'
    items, more listed pages than one launch or four carry, consecutive pages and pages beyond the layout,
    a source that is not 16-byte aligned (shift)."""
    numels = [(E + 3, 3 * E, E // 2 + 1, 16385, 1)[k % 5] if E > 8 else 5 for k in range(n_t)]
    n = oracle.plan_pack(numels, E).n_pages
    gen = torch.Generator(device=DEV).manual_seed(n)
    flat = torch.randn(n * E, device=DEV, generator=gen) * 0.02
    pools = []
    for _ in range(2):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n + 2)
        off = [sum(numels[:k]) for k in range(n_t)]
        apm.apm_pack_tensors(pool, apm.APM_P32, apm.make_tensors(numels, apm.APM_F32, [flat.data_ptr() + 4 * o for o in off]), n_t)
        pools.append(pool)
    pages = {"all": None, "more": None, "odd": list(range(1, n, 2)), "reversed": list(range(n))[::-1], "middle": list(range(1, n - 1))}[listed]
    count = len(pages) if pages is not None else n + 2 if listed == "more" else n
    norm, mask = [torch.full((n + 2,), -1.0, device=DEV) for _ in range(2)], [torch.full((n + 2,), 9, device=DEV, dtype=torch.uint8) for _ in range(2)]
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, skip)
    if norms:
        apm.apm_delayed_set_outputs(pools[1], norm[1], mask[1])
    raw = [torch.zeros((n + 2) * E + 8, device=DEV, dtype=torch.bfloat16) for _ in range(micro)]
    for t in (1, 2, 3):
        gs = []
        for k in range(micro):
            raw[k] = torch.zeros((n + 2) * E + 8, device=DEV, dtype=torch.bfloat16)
            g = raw[k][shift if k == 0 else 0:][:(n + 2) * E]
            g.copy_((torch.randn((n + 2) * E, device=DEV, generator=gen) * 1e-2).bfloat16())
            if skip:
                g.view(n + 2, E)[::3] = 0
            gs.append(g)
        total = gs[0].clone()
        for g in gs[1:]:
            total = total + g
        view = torch.as_tensor(_Region(pools[0], apm.APM_G16, (n + 2) * E), device=DEV)
        view.copy_(total.view(torch.int16))
        apm.apm_page_adamw_step(pools[0], pages, count, t, hyper, norm[0] if norms else None, mask[0] if norms else None)
        apm.apm_step_delayed(pools[1], pages, count, gs[0].data_ptr(), hyper)
        for g in gs[1:]:
            apm.apm_delayed_accumulate(pools[1], pages, count, g.data_ptr())
        torch.cuda.synchronize()
    apm.apm_step_delayed(pools[1], pages, count, None, hyper)
    torch.cuda.synchronize()
    if norms:
        assert torch.equal(norm[0][:count], norm[1][:count]) and torch.equal(mask[0][:count], mask[1][:count])
    for st, kind in ((apm.APM_P32, apm.APM_F32), (apm.APM_M32, apm.APM_F32), (apm.APM_V32, apm.APM_F32), (apm.APM_P16, apm.APM_BF16)):
        out = [torch.zeros(sum(numels), device=DEV, dtype=torch.float32 if st < 3 else torch.bfloat16) for _ in range(2)]
        for pool, o in zip(pools, out):
            apm.apm_unpack(pool, st, apm.make_tensors(numels, kind, [o.data_ptr() + o.element_size() * x for x in off]), n_t)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]), st
    for pool in pools:
        pool.destroy()


@pytest.mark.parametrize("clip", [0.0, 0.02])
@pytest.mark.parametrize("numels", [[3 * 4096 + 5], [4096, 9, 9, 9]])
def test_a_hand_over_of_no_pages_is_accepted(numels, clip):
    """An iteration that touched no listed page: the gradient handed over before is applied, nothing is taken over and
    the next call applies nothing (layouts of one extent class and of several)."""
    E, n_t = 4096, len(numels)
    n = oracle.plan_pack(numels, E).n_pages
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, 0)
    g = (torch.randn(n * E, device=DEV, generator=torch.Generator(device=DEV).manual_seed(n)) * 1e-2).bfloat16()
    got = []
    for empty in (None, [], "null"):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
        apm.apm_pool_set_layout(pool, apm.make_tensors(numels, apm.APM_F32, [0] * n_t), n_t)
        apm.apm_step_delayed(pool, None, n, g.data_ptr(), hyper)
        if empty is not None:
            pages = None if empty == "null" else empty
            apm.apm_step_delayed(pool, pages, 0, g.data_ptr(), hyper)
            apm.apm_delayed_accumulate(pool, pages, 0, g.data_ptr())
        apm.apm_step_delayed(pool, None, n, None, hyper)
        out = [torch.zeros(m, device=DEV) for m in numels]
        apm.apm_unpack(pool, apm.APM_M32, apm.make_tensors(numels, apm.APM_F32, [o.data_ptr() for o in out]), n_t)
        torch.cuda.synchronize()
        got.append(torch.cat(out))
        pool.destroy()
    assert got[0].any() and torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


class _Region:
    """A class region of a pool as an array of half words that torch can wrap."""

    def __init__(self, pool, state, numel):
        self.__cuda_array_interface__ = {"shape": (numel,), "typestr": "<i2", "data": (apm.apm_pool_state_ptr(pool, state), False), "version": 3}


@pytest.mark.parametrize("dead", ["none", "all", "most", "first"])
@pytest.mark.parametrize("form", ["run", "reversed", "fused", "noalloc"])
@pytest.mark.parametrize("E,n_t,per", [(8, 40, 8), (4104, 30, 4103), (1 << 20, 6, 3 << 19), (1 << 20, 40, 5000),
                                     (4104, 1500, 4103), (512, 5000, 500), (1 << 20, 18, 3 << 19)])
def test_skipping_updates_the_touched_pages_and_no_others(E, n_t, per, form, dead):
    """The grid over the noted pages: none, all, few live pages, several extent classes, and (the last size) so many slices a
    wavefront that state is stored non-temporal only.  Same bits as a step without skipping on the live pages; the
    others keep theirs."""
    numels = [per if k % 7 else max(1, per // 600) for k in range(n_t)]
    off = [0]
    for m in numels:
        off.append(off[-1] + (m + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(E + n_t)
    g = (torch.rand(off[-1], device=DEV, generator=gen) + 1e-3).bfloat16()
    alive = {"none": lambda t: True, "all": lambda t: False, "most": lambda t: t % 9 == 4, "first": lambda t: t > 1}[dead]
    for t in range(n_t):
        if not alive(t):
            g[off[t]:off[t + 1]] = 0
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    plan = oracle.plan_pack(numels, E)
    n = plan.n_pages
    live = torch.zeros(n, dtype=torch.bool)
    for s in plan.segments:
        live[s.page] |= alive(s.tensor)
    pages = list(range(n))[::-1] if form == "reversed" else None
    got, mask = [], torch.full((n,), 9, device=DEV, dtype=torch.uint8)
    for skip in (0, 1):
        hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, skip)
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n + 1)
        for st in (apm.APM_P32, apm.APM_M32):
            apm.apm_pack_tensors(pool, st, lst(p0), n_t)
        apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        q = torch.zeros_like(g)
        if form == "fused":
            apm.apm_page_adamw_step_fused(pool, pages, n, 3, hyper, lst(g), lst(q), n_t, None, mask if skip else None)
        elif form == "noalloc":
            apm.apm_page_adamw_step_noalloc(pool, n, 3, hyper, None, mask if skip else None)
        else:
            apm.apm_page_adamw_step(pool, pages, n, 3, hyper, None, mask if skip else None)
        out = [torch.zeros_like(p0) for _ in range(3)]
        for st, o in zip((apm.APM_P32, apm.APM_M32, apm.APM_V32), out):
            apm.apm_unpack(pool, st, lst(o), n_t)
        torch.cuda.synchronize()
        got.append(out + [q])
        pool.destroy()
    assert torch.equal(mask.cpu() == 1, ~(live.flip(0) if form == "reversed" else live)) and (mask < 2).all()
    for s in plan.segments:
        at = slice(off[s.tensor] + s.tensor_off, off[s.tensor] + s.tensor_off + s.n)
        if live[s.page]:
            assert all(torch.equal(a[at], b[at]) for a, b in zip(*got))
        else:
            assert torch.equal(got[1][0][at], p0[at]) and torch.equal(got[1][1][at], p0[at])
            assert not got[1][2][at].any() and not got[1][3][at].any()


@pytest.mark.parametrize("cap", [1, 7, 1000])
@pytest.mark.parametrize("skip", [0, 1])
@pytest.mark.parametrize("form", ["run", "reversed", "fused", "delayed", "delayed reversed"])
def test_updates_in_several_launches_equal_one_launch(form, skip, cap):
    """Page counts beyond what one grid holds are launched in pieces; a low cap on the workgroups of a
    launch gives several pieces per extent class at a small size (packing, sums, hand-overs, updates).  Same bits as
    without the cap."""
    E, numels = 1 << 18, [3, (1 << 18) * 5 + 77, 100, 1, 2000] + [40] * 300
    n_t, off = len(numels), [0]
    for m in numels:
        off.append(off[-1] + (m + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(cap)
    g = (torch.randn(off[-1], device=DEV, generator=gen) * 1e-2).bfloat16()
    g[off[7]:off[100]] = 0
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.05, skip)
    got = []
    for c in (0, cap):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, oracle.plan_pack(numels, E).n_pages)
        assert apm.lib().apm_test_set_max_workgroups(ctypes.c_void_p(pool.handle), ctypes.c_int64(c)) == 0
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)
        apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        n = apm.lib().apm_pool_pages_in_use(pool.handle)
        norm, q = torch.full((n,), -1.0, device=DEV), torch.zeros_like(g)
        pages = list(range(n))[::-1] if "reversed" in form else None
        if form == "fused":
            apm.apm_page_adamw_step_fused(pool, pages, n, 3, hyper, lst(g), lst(q), n_t, norm, None)
        elif "delayed" in form:
            g_pages = torch.as_tensor(_Region(pool, apm.APM_G16, n * E), device=DEV)
            apm.apm_delayed_set_outputs(pool, norm, None)
            apm.apm_step_delayed(pool, pages, n, g_pages.data_ptr(), hyper)
            apm.apm_delayed_accumulate(pool, pages, n, g_pages.data_ptr())
            apm.apm_step_delayed(pool, pages, n, None, hyper)
            apm.apm_unpack(pool, apm.APM_P16, lst(q), n_t)
        else:
            apm.apm_page_adamw_step(pool, pages, n, 3, hyper, norm, None)
            apm.apm_unpack(pool, apm.APM_P16, lst(q), n_t)
        out = [norm, q]
        for st in (apm.APM_P32, apm.APM_M32, apm.APM_V32):
            out.append(torch.zeros_like(p0))
            apm.apm_unpack(pool, st, lst(out[-1]), n_t)
        torch.cuda.synchronize()
        got.append(out)
        pool.destroy()
    assert (got[0][0] >= 0).all() and got[0][2].ne(p0).any()
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("clip,skip", [(0.0, 0), (0.05, 0), (0.05, 1)])
@pytest.mark.parametrize("form", ["whole", "reversed", "fused", "fused reversed", "delayed"])
def test_extents_of_every_class_in_one_grid_equal_steps_page_by_page(form, clip, skip):
    """Full, quarter, small and nearly empty pages, as many of each as make a class of their own in the common
    grid.  Same bits as one call for every page, which has no classes."""
    E = 1 << 18
    numels = [E * 2 + 9, 8000, 500] + [60000] * 12 + [8001] * 60 + [7, 500] * 250 + [E]
    n_t, off, plan = len(numels), [0], oracle.plan_pack(numels, E)
    for m in numels:
        off.append(off[-1] + (m + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(7)
    g = (torch.randn(off[-1], device=DEV, generator=gen) * 1e-2).bfloat16()
    g[off[5]:off[9]] = 0
    g[off[100]:off[300]] = 0
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, skip)
    got = []
    for each in (True, False):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, plan.n_pages)
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)
        apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        n = plan.n_pages
        norm, mask, q = torch.full((n,), -1.0, device=DEV), torch.full((n,), 9, device=DEV, dtype=torch.uint8), torch.zeros_like(g)
        pages = list(range(n))[::-1] if "reversed" in form else None
        if each:
            for k in range(n):
                at = n - 1 - k if pages else k
                apm.apm_page_adamw_step(pool, [k], 1, 1, hyper, norm[at:], mask[at:])
        elif "fused" in form:
            apm.apm_page_adamw_step_fused(pool, pages, n, 1, hyper, lst(g), lst(q), n_t, norm, mask)
        elif form == "delayed":
            g_pages = torch.as_tensor(_Region(pool, apm.APM_G16, n * E), device=DEV)
            apm.apm_delayed_set_outputs(pool, norm, mask)
            apm.apm_step_delayed(pool, None, n, g_pages.data_ptr(), hyper)
            apm.apm_step_delayed(pool, None, n, None, hyper)
        else:
            apm.apm_page_adamw_step(pool, pages, n, 1, hyper, norm, mask)
        if each or "fused" not in form:
            apm.apm_unpack(pool, apm.APM_P16, lst(q), n_t)
        out = [norm, mask, q]
        for st in (apm.APM_P32, apm.APM_M32, apm.APM_V32):
            out.append(torch.zeros_like(p0))
            apm.apm_unpack(pool, st, lst(out[-1]), n_t)
        torch.cuda.synchronize()
        got.append(out)
        pool.destroy()
    assert (got[0][1].sum() > 0) == bool(skip)
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), k


@pytest.mark.parametrize("listed", ["all", "reversed"])
@pytest.mark.parametrize("n_t,apart", [(300, 0), (300, 66 << 30), (439, 0), (441, 0), (441, 66 << 30), (2000, 0)])
def test_fused_step_with_tensors_near_and_far_apart(n_t, apart, listed):
    """Addresses travel as half words where a list's tensors lie within 64 GiB, as whole words elsewhere; tensor counts
    around what one launch carries either way, and empty tensors with any address.  Same bits as the page step."""
    if apart and torch.cuda.mem_get_info()[0] < apart + (8 << 30):
        pytest.skip("not enough free device memory")
    E = 64
    numels = [(0, 3, E, 2 * E + 5, 17)[k % 5] for k in range(n_t)]
    off = [sum((m + 7) // 8 * 8 for m in numels[:k]) for k in range(n_t)]
    room = off[-1] + 256
    gen = torch.Generator(device=DEV).manual_seed(n_t)
    raw = torch.empty(apart + 8 * room + 64, dtype=torch.uint8, device=DEV)
    at = [(apart if k % 3 == 1 else 0) + 2 * o for k, o in enumerate(off)]  # every third tensor at the far end
    place = lambda base: apm.make_tensors(numels, apm.APM_BF16, [base + x if m else 7 for x, m in zip(at, numels)])  # noqa: E731
    g_flat = (torch.randn(room, device=DEV, generator=gen) * 1e-2).bfloat16()
    near = raw[:2 * room].view(torch.bfloat16), raw[apart:apart + 2 * room].view(torch.bfloat16)
    for part in near:
        part.copy_(g_flat)
    q_near = [raw[a + 2 * room:a + 4 * room].view(torch.bfloat16) for a in (0, apart)]
    for part in q_near:
        part.zero_()
    n = oracle.plan_pack(numels, E).n_pages
    pages = list(range(n))[::-1] if listed == "reversed" else None
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.05, 0)
    p0, out = torch.randn(room, device=DEV, generator=gen), []
    for fused in (False, True):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
        apm.apm_pack_tensors(pool, apm.APM_P32, apm.make_tensors(numels, apm.APM_F32, [p0.data_ptr() + 4 * o if m else 0 for o, m in zip(off, numels)]), n_t)
        norm, q = torch.zeros(n, device=DEV), torch.zeros_like(g_flat)
        if fused:
            apm.apm_page_adamw_step_fused(pool, pages, n, 1, hyper, place(raw.data_ptr()), place(raw.data_ptr() + 2 * room), n_t, norm, None)
            for k, (o, m) in enumerate(zip(off, numels)):
                q[o:o + m] = q_near[k % 3 == 1][o:o + m]
        else:
            tight = lambda t: apm.make_tensors(numels, apm.APM_BF16, [t.data_ptr() + 2 * o if m else 0 for o, m in zip(off, numels)])  # noqa: E731
            apm.apm_pack_tensors(pool, apm.APM_G16, tight(g_flat), n_t)
            apm.apm_page_adamw_step(pool, pages, n, 1, hyper, norm, None)
            apm.apm_unpack(pool, apm.APM_P16, tight(q), n_t)
        torch.cuda.synchronize()
        out.append((norm, q))
        pool.destroy()
    assert (out[0][0] > 0).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    if apart:  # 66 GiB that no later test needs
        del raw, near, q_near, part
        torch.cuda.empty_cache()


def _us(f, n):
    """Best of five batches of n calls, microseconds a call."""
    best = float("inf")
    f()
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(n):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / n)
    return best * 1e6


@pytest.mark.parametrize("E,n", [(64, 131072), (512, 32768)])
def test_skipping_costs_little_where_every_small_page_has_a_gradient(E, n):
    """Finding that no page is skipped is a few percent of a step with norms, however many pages: noting
    each with an atomic of its own made it four times such a step (bound: twice)."""
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
    torch.as_tensor(_Region(pool, apm.APM_G16, n * E), device=DEV).fill_(0x3a00)
    norm = torch.zeros(n, device=DEV)
    step = lambda skip: apm.apm_page_adamw_step(pool, None, n, 3, apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, skip), norm, None)  # noqa: E731
    plain, skipping = _us(lambda: step(0), 20), _us(lambda: step(1), 20)
    pool.destroy()
    assert skipping < 2 * plain, (skipping, plain)


def test_gradients_of_many_small_pages_are_taken_over_without_a_list_or_sums_each():
    """A gradient added over 65536 consecutive pages of 512 elements, given as a list or with a page beyond
    the layout, costs about what it costs over all pages; carried as lists in launch after launch it was four
    times as slow, and with sums for the update 3.5 times as slow as without (bounds: 2.5 and 1.5)."""
    E, n = 512, 65536
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n + 1)
    L = apm.lib()
    L.apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
    g = torch.zeros((n + 1) * E, device=DEV, dtype=torch.bfloat16)
    lst = (ctypes.c_int64 * n)(*range(n))
    best = {}
    for clip in (0.0, 1.0):
        hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, 0)
        for name, pages, count in (("all", None, n), ("beyond", None, n + 1), ("list", lst, n)):
            assert L.apm_step_delayed(pool.handle, pages, count, ctypes.c_void_p(g.data_ptr()), ctypes.byref(hyper), None) == 0

            def add():
                assert L.apm_delayed_accumulate(pool.handle, pages, count, ctypes.c_void_p(g.data_ptr()), None) == 0
            best[name, clip] = _us(add, 50)
    L.apm_step_delayed(pool.handle, None, n, None, ctypes.byref(hyper), None)
    torch.cuda.synchronize()
    pool.destroy()
    for clip in (0.0, 1.0):
        assert best["beyond", clip] < 2.5 * best["all", clip] and best["list", clip] < 2.5 * best["all", clip], best
    assert best["all", 1.0] < 1.5 * best["all", 0.0], best


def test_short_segments_do_not_wait_for_idle_wavefronts():
    """65536 segments of 512 elements out of their pages: 2 bytes each cost less than 4 (in workgroups of which three
    wavefronts in four had nothing to do they took 1.2 times as long; half now; bound 0.9)."""
    E, n, us = 512, 65536, []
    out = torch.zeros(n * E, device=DEV)
    for st, kind in ((apm.APM_P16, apm.APM_BF16), (apm.APM_P32, apm.APM_F32)):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n, state_mask=1 << st)
        lst = apm.make_tensors([n * E], kind, [out.data_ptr()])
        apm.apm_pool_set_layout(pool, lst, 1)
        us.append(_us(lambda: apm.apm_unpack(pool, st, lst, 1), 50))
        pool.destroy()
    assert us[0] < 0.9 * us[1], us


def test_a_list_of_many_small_pages_is_grouped_quickly():
    """A page beyond the layout takes the general path, whose host time is the grouping of the pages by
    extent: 131072 pages of 64 elements within three times the path with the layout's own order (four and
    a half times with a function call per page, 1.8 with arrays)."""
    E, n = 64, 131072
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n + 1)
    apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, 0)
    whole, general = (_us(lambda: apm.apm_page_adamw_step(pool, None, k, 3, hyper, None, None), 30) for k in (n, n + 1))
    pool.destroy()
    assert general < 3 * whole, (general, whole)


def test_a_list_that_is_no_run_is_grouped_once():
    """131072 pages of 64 elements in reverse, bound by the host: the step on the page classes, which would take a
    run in coarser classes, costs about what the step from a tensor does (grouped for both 1.5 times as much; bound 1.25)."""
    E, n = 64, 131072
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    L = apm.lib()
    L.apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, 0)
    g = torch.zeros(n * E, device=DEV, dtype=torch.bfloat16)
    lst, g_list = (ctypes.c_int64 * n)(*range(n - 1, -1, -1)), apm.make_tensors([n * E], apm.APM_BF16, [g.data_ptr()])

    def pages():
        assert L.apm_page_adamw_step(pool.handle, lst, n, 3, ctypes.byref(hyper), None, None, None) == 0

    def fused():
        assert L.apm_page_adamw_step_fused(pool.handle, lst, n, 3, ctypes.byref(hyper), g_list, None, 1, None, None, None) == 0
    us = [_us(f, 20) for f in (pages, fused)]
    pool.destroy()
    assert us[0] < 1.25 * us[1], us


@pytest.mark.parametrize("listed", ["all", "reversed", "odd"])
@pytest.mark.parametrize("n", [2047, 2048, 2049, 4100])
@pytest.mark.parametrize("E", [8, 520, 4088, 4096])
def test_clipped_steps_around_the_rule_for_one_grid_agree(E, n, listed):
    """Clipped steps in one grid and as passes (page sizes and page counts on both sides of the rule; lists in
    kernel arguments and in the ring): norms against 64 bits (one fp32 rounding), p16 and moments against the
    same pages stepped through tensors."""
    tot = (n - 1) * E + E // 2 + 3
    gen = torch.Generator(device=DEV).manual_seed(n)
    g = (torch.randn(n * E, device=DEV, generator=gen) * 1e-2).bfloat16()
    g[tot:] = 0
    p0 = torch.randn(n * E, device=DEV, generator=gen) * 0.02
    one = lambda t: apm.make_tensors([tot], apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16, [t.data_ptr()])  # noqa: E731
    pages = {"all": None, "reversed": list(range(n))[::-1], "odd": list(range(1, n, 2))}[listed]
    at = list(range(n)) if pages is None else pages
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.05, apm.APM_SKIP_NONE)
    got = []
    for fused in (False, True):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
        apm.apm_pack_tensors(pool, apm.APM_P32, one(p0), 1)
        norm, q = torch.full((len(at),), -1.0, device=DEV), torch.zeros_like(g)
        if fused:
            apm.apm_page_adamw_step_fused(pool, pages, len(at), 3, hyper, one(g), one(q), 1, norm, None)
        else:
            apm.apm_pack_tensors(pool, apm.APM_G16, one(g), 1)
            apm.apm_page_adamw_step(pool, pages, len(at), 3, hyper, norm, None)
            apm.apm_unpack(pool, apm.APM_P16, one(q), 1)
        out = [norm, q] + [torch.zeros_like(p0) for _ in range(3)]
        for st, o in zip((apm.APM_P32, apm.APM_M32, apm.APM_V32), out[2:]):
            apm.apm_unpack(pool, st, one(o), 1)
        torch.cuda.synchronize()
        got.append(out)
        pool.destroy()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    want = g.view(n, E).double().square().sum(1).sqrt()[torch.tensor(at, device=DEV)]
    assert torch.allclose(got[0][0].double(), want, rtol=2.0 ** -23, atol=0.0)


def test_norms_of_small_pages_cost_no_more_than_finding_skipped_ones():
    """131072 pages of 512 elements: a step with norms in one grid, three wavefronts a page, took 1.55 times the
    passes that a skipping step runs (bound 1.25)."""
    E, n = 512, 131072
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
    torch.as_tensor(_Region(pool, apm.APM_G16, n * E), device=DEV).fill_(0x3a00)
    norm = torch.zeros(n, device=DEV)
    step = lambda skip: apm.apm_page_adamw_step(pool, None, n, 3, apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, skip), norm, None)  # noqa: E731
    norms, skipping = _us(lambda: step(0), 20), _us(lambda: step(1), 20)
    pool.destroy()
    assert norms < 1.25 * skipping, (norms, skipping)


@pytest.mark.parametrize("clip,skip,norms", [(0.0, 0, False), (0.02, 0, True), (0.02, 1, True)])
@pytest.mark.parametrize("E,numels", [(1 << 19, [3, 1 << 19, 700, 1025, 5]), (1 << 19, [(1 << 19) + 9, 1 << 19, 3]), (8192, [4097] + [100] * 9),
                                      (4096, [1] * 5)])
def test_noalloc_step_over_nearly_empty_pages_equals_the_step(E, numels, clip, skip, norms):
    """Pages launched with a full page's grid in larger slices where most of it is idle (both sides of the
    rule): the bits of the step that sizes its grids by extent."""
    n_t, off = len(numels), [0]
    for m in numels:
        off.append(off[-1] + (m + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(n_t)
    g = (torch.randn(off[-1], device=DEV, generator=gen) * 1e-2).bfloat16()
    g[off[n_t - 2]:off[n_t - 1]] = 0
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    n, got = oracle.plan_pack(numels, E).n_pages, []
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, skip)
    for noalloc in (False, True):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)
        apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        norm = torch.full((n,), -1.0, device=DEV) if norms else None
        if noalloc:
            apm.apm_page_adamw_step_noalloc(pool, n, 3, hyper, norm, None)
        else:
            apm.apm_page_adamw_step(pool, None, n, 3, hyper, norm, None)
        out = [torch.zeros_like(p0) for _ in range(3)] + [torch.zeros_like(g)]
        for st, o in zip((apm.APM_P32, apm.APM_M32, apm.APM_V32, apm.APM_P16), out):
            apm.apm_unpack(pool, st, lst(o), n_t)
        torch.cuda.synchronize()
        got.append(out + ([norm] if norms else []))
        pool.destroy()
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_nearly_empty_pages_cost_the_noalloc_step_little():
    """Two full pages of 2^20 elements and 60 nearly empty ones: four times the idle workgroups took 6.6 times the
    two pages' time (larger slices 2.2; bound 3)."""
    E, us = 1 << 20, []
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, 0)
    for empty in (0, 60):
        numels = [E, E] + [100] * empty
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, len(numels))
        apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors(numels, apm.APM_F32, [0] * len(numels)), len(numels), None, None, None, None, None)
        us.append(_us(lambda: apm.apm_page_adamw_step_noalloc(pool, len(numels), 3, hyper, None, None), 100))
        pool.destroy()
    assert us[1] < 3 * us[0], us


def test_a_buffered_gradient_is_not_applied_beyond_what_was_handed_over():
    """The hand-over takes the used extents of its layout.  A layout with larger extents installed before the
    update: an error and no update, once, instead of an older gradient's bytes; one with smaller extents: the
    same bits as a synchronous step."""
    E, gen = 1024, torch.Generator(device=DEV).manual_seed(5)
    lists = {name: [n, n] for name, n in (("small", 40), ("large", 600))}
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, 0)
    g = (torch.randn(2 * E, device=DEV, generator=gen) * 1e-2).bfloat16().view(2, E)

    def lay(pool, name):
        torch.cuda.synchronize()
        apm.apm_pool_set_layout(pool, apm.make_tensors(lists[name], apm.APM_F32, [0, 0]), 2)

    def moments(pool, name):
        out = torch.zeros(2, E, device=DEV)
        apm.apm_unpack(pool, apm.APM_M32, apm.make_tensors(lists[name], apm.APM_F32, [out.data_ptr(), out.data_ptr() + 4 * E]), 2)
        torch.cuda.synchronize()
        return out

    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, 2)
    lay(pool, "large")
    apm.apm_step_delayed(pool, None, 2, g.data_ptr(), hyper)
    apm.apm_step_delayed(pool, None, 2, None, hyper)     # leaves an older gradient in one half
    lay(pool, "small")
    for _ in range(2):                                   # and small extents of a newer one in both
        apm.apm_step_delayed(pool, None, 2, g.data_ptr(), hyper)
    lay(pool, "large")
    for call in (lambda: apm.apm_delayed_accumulate(pool, None, 2, g.data_ptr()), lambda: apm.apm_step_delayed(pool, None, 2, None, hyper)):
        with pytest.raises(apm.ApmError) as e:
            call()
        assert e.value.code == apm.APM_ESTATE
    assert not moments(pool, "large").any()
    apm.apm_step_delayed(pool, None, 2, None, hyper)     # nothing is left to apply
    assert not moments(pool, "large").any()
    apm.apm_step_delayed(pool, None, 2, g.data_ptr(), hyper)
    lay(pool, "small")
    apm.apm_step_delayed(pool, None, 2, None, hyper)
    got = moments(pool, "small")
    assert torch.equal(got[:, :40], g[:, :40].float() * 0.1)
    pool.destroy()


def test_unused_pool_flags_do_not_change_the_update():
    """Bits that the interface does not define have no effect; the highest one used to make every wavefront of
    a clipped update sum its page by itself, hundreds of times the work (bound: three times)."""
    E, n, us = 1 << 20, 8, []
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 1.0, 0)
    for flags in (0, 1 << 31 | 1 << 17):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n, flags=flags)
        apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
        us.append(_us(lambda: apm.apm_page_adamw_step(pool, None, n, 3, hyper, None, None), 10))
        pool.destroy()
    assert us[1] < 3 * us[0], us


def test_wavefronts_that_stop_waiting_do_not_all_sum_the_whole_page():
    """A wait that ends after one look, large pages: wavefronts of a clipped update sum their page by themselves
    only until its scale is there, 16 times the update's time; each summing the whole page, 58 times (bound 35)."""
    E, n, us = 1 << 24, 4, []
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 1.0, 0)
    for limit in (4096, 1):
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
        assert apm.lib().apm_test_set_wait_limit(ctypes.c_void_p(pool.handle), limit) == 0
        apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors([n * E], apm.APM_F32, [0]), 1, None, None, None, None, None)
        us.append(_us(lambda: apm.apm_page_adamw_step(pool, None, n, 3, hyper, None, None), 5))
        pool.destroy()
    assert us[1] < 35 * us[0], us


@pytest.mark.parametrize("clip,skip", [(0.0, 0), (0.05, 0), (0.05, 1)])
@pytest.mark.parametrize("E,numels", [(8, [5, 8, 3] * 9), (512, [300] * 5000), (1 << 20, [(1 << 20) * 2 + 77, 100, 1 << 20, 5]), (1 << 19, [9] * 6)])
def test_noalloc_step_in_a_replayed_graph_equals_the_eager_call(E, numels, clip, skip):
    """Every form of the step that may be captured (plain, passes, one grid, noted pages, larger slices): each of
    several replays, with eager work and new gradients between them, gives the eager call's bits."""
    n_t, off = len(numels), [0]
    for m in numels:
        off.append(off[-1] + (m + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(E)
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    n = oracle.plan_pack(numels, E).n_pages
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, skip)
    pools = [apm.apm_pool_create(apm.APM_DEV_GPU, E, n) for _ in range(2)]
    norm = [torch.full((n,), -1.0, device=DEV) for _ in range(2)]
    outs = [t if clip else None for t in norm]

    def gradients():
        g = (torch.randn(off[-1], device=DEV, generator=gen) * 1e-2).bfloat16()
        g[off[1]:off[2]] = 0
        for pool in pools:
            apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        torch.cuda.synchronize()
    for pool in pools:
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)
    gradients()
    for pool, out in zip(pools, outs):
        apm.apm_page_adamw_step_noalloc(pool, n, 2, hyper, out, None)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        apm.apm_page_adamw_step_noalloc(pools[1], n, 3, hyper, outs[1], None, torch.cuda.current_stream())
    for _ in range(4):
        gradients()
        apm.apm_page_adamw_step_noalloc(pools[0], n, 3, hyper, outs[0], None)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(norm[0], norm[1])
        for st in (apm.APM_P32, apm.APM_M32, apm.APM_V32, apm.APM_P16):
            got = [torch.zeros(off[-1], device=DEV, dtype=torch.float32 if st < 3 else torch.bfloat16) for _ in range(2)]
            for pool, t in zip(pools, got):
                apm.apm_unpack(pool, st, lst(t), n_t)
            torch.cuda.synchronize()
            assert torch.equal(*got)
    for pool in pools:
        pool.destroy()


@pytest.mark.parametrize("skip", [0, 1])
def test_a_small_tensor_alone_in_its_page_costs_the_steps_little(skip):
    """30000 tensors of 300 elements in pages of 8192, every norm wanted: neither the step that launches all pages
    alike (a full page's grid each: 4.5 times the other step's time) nor three wavefronts a page in one grid."""
    E, n, us = 8192, 30000, []
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    apm.lib().apm_pool_set_layout(pool.handle, apm.make_tensors([300] * n, apm.APM_F32, [0] * n), n, None, None, None, None, None)
    torch.as_tensor(_Region(pool, apm.APM_G16, n * E), device=DEV).view(n, E)[:, :300] = 0x3a00
    norm = torch.zeros(n, device=DEV)
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, skip)
    us.append(_us(lambda: apm.apm_page_adamw_step(pool, None, n, 3, hyper, norm, None), 20))
    us.append(_us(lambda: apm.apm_page_adamw_step_noalloc(pool, n, 3, hyper, norm, None), 20))
    pool.destroy()
    assert us[1] < 2 * us[0], us


@pytest.mark.parametrize("bits", [0x0001, 0x7F80, 0xFFC1, 0x8000])
@pytest.mark.parametrize("form", ["pages", "tensors"])
def test_one_element_decides_whether_a_page_is_skipped(form, bits):
    """Skipping without norms looks at an eighth of a tile first: one element in or behind it, at a tile's or tensor's end, the smallest subnormal,
    infinity and NaN count, minus zero does not."""
    E, T = 40960, 16384
    at = [0, 2047, 2048, T - 1, T, T + 2047, T + 2048, 2 * T, E - 1]
    n_t = len(at) + 2
    numels = [E] * len(at) + [5, 2 * E + 3]     # the last tensors: all zero; one element in its last, partial vector
    flat = torch.zeros(n_t, 2 * E + 8, dtype=torch.int16, device=DEV)
    for k, e in enumerate(at):
        flat[k, e] = bits - 65536 * (bits >> 15)
    flat[n_t - 1, 2 * E + 2] = bits - 65536 * (bits >> 15)
    assert flat.stride(0) % 8 == 0
    g = apm.make_tensors(numels, apm.APM_BF16, [flat[k].data_ptr() for k in range(n_t)])
    n = len(at) + 1 + 3
    hy = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, apm.APM_SKIP_UNTOUCHED)
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    apm.apm_pack_tensors(pool, apm.APM_G16, g, n_t)
    skip = torch.full((n,), 9, dtype=torch.uint8, device=DEV)
    if form == "pages":
        apm.apm_page_adamw_step(pool, None, n, 1, hy, None, skip)
    else:
        apm.apm_page_adamw_step_fused(pool, None, n, 1, hy, g, None, n_t, None, skip)
    torch.cuda.synchronize()
    want = [int(bits == 0x8000)] * len(at) + [1, 1, 1, int(bits == 0x8000)]
    assert skip.tolist() == want
    pool.destroy()


def _pages_and_tensors(E, numels, seed, n_pools):
    """Pools with the same masters, the tensors' lists, and a function that draws a gradient, into the tensors and the pages."""
    n_t, off = len(numels), [0]
    for m in numels:
        off.append(off[-1] + (m + 7) // 8 * 8)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    p0 = torch.randn(off[-1], device=DEV, generator=gen) * 0.02
    lst = lambda t: apm.make_tensors(numels, apm.APM_F32 if t.dtype == torch.float32 else apm.APM_BF16,  # noqa: E731
                                     [t.data_ptr() + t.element_size() * o for o in off[:-1]])
    n = oracle.plan_pack(numels, E).n_pages
    pools = [apm.apm_pool_create(apm.APM_DEV_GPU, E, n) for _ in range(n_pools)]
    g = torch.zeros(off[-1], device=DEV, dtype=torch.bfloat16)
    for pool in pools:
        apm.apm_pack_tensors(pool, apm.APM_P32, lst(p0), n_t)

    def draw():
        g.copy_(torch.randn(off[-1], device=DEV, generator=gen) * 1e-2)
        for pool in pools:
            apm.apm_pack_tensors(pool, apm.APM_G16, lst(g), n_t)
        torch.cuda.synchronize()

    def state(pool):
        out = [torch.zeros(off[-1], device=DEV, dtype=torch.float32 if st < 3 else torch.bfloat16) for st in (0, 1, 2, apm.APM_P16)]
        for st, t in zip((0, 1, 2, apm.APM_P16), out):
            apm.apm_unpack(pool, st, lst(t), n_t)
        torch.cuda.synchronize()
        return out
    return pools, n, g, lst, draw, state


@pytest.mark.parametrize("clip", [0.0, 0.05])
@pytest.mark.parametrize("form", ["run", "reversed", "fused", "fused odd"])
def test_captured_steps_replay_as_they_run(form, clip):
    """A step that makes its own records hands results on under a number that a replay would repeat: captured, the words are
    marked instead.  Replays with eager steps of the same pool between them, against eager steps."""
    E, numels = 4104, [(3, 4104, 9000, 17, 2051)[(3 * k) % 5] for k in range(40)]
    pools, n, g, lst, draw, state = _pages_and_tensors(E, numels, 3, 2)
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, 0)
    pages = {"reversed": list(range(n))[::-1], "fused odd": list(range(1, n, 2))}.get(form)
    count = len(pages) if pages else n
    norm = [torch.zeros(n, device=DEV) for _ in range(2)]

    def step(k, stream=None):
        out = norm[k] if clip else None
        if form.startswith("fused"):
            apm.apm_page_adamw_step_fused(pools[k], pages, count, 3, hyper, lst(g), None, len(numels), out, None, stream)
        else:
            apm.apm_page_adamw_step(pools[k], pages, count, 3, hyper, out, None, stream)
    draw()
    for k in range(2):
        step(k)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(1, torch.cuda.current_stream())
    for r in range(4):
        draw()
        step(0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(*norm)
        for a, b in zip(state(pools[0]), state(pools[1])):
            assert torch.equal(a, b)
        if r % 2:
            draw()
            for k in range(2):
                step(k)
    for pool in pools:
        pool.destroy()


@pytest.mark.parametrize("form", ["run", "listed", "tensors"])
@pytest.mark.parametrize("E", [520, 16384, 40968])
def test_norms_handed_on_in_parts_equal_the_marked_ones(E, form):
    """A tile's four parts (512 elements in turn), ends of tensors and pages in each of them, two tenants in one part; against the
    step whose wavefronts take whole tiles; across the call numbers' end."""
    ends = [1, 7, 511, 513, 1024 + 9, 1536 - 1, 2048 + 1, 8 * 2048 - 3, 8 * 2048 + 515]
    numels = [min(m, E - 1) for m in ends] + [E + m for m in ends] + [2 * E]
    pools, n, g, lst, draw, state = _pages_and_tensors(E, numels, E, 2)
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.05, 0)
    norm = [torch.zeros(n, device=DEV) for _ in range(2)]
    pages = list(range(n))[::-1] if form == "listed" else None
    for t in range(1, 6):
        if t == 3:
            assert apm.lib().apm_test_set_call_number(ctypes.c_void_p(pools[0].handle), ctypes.c_uint32(0xFFFFFFFE)) == 0
        draw()
        if form == "tensors":
            apm.apm_page_adamw_step_fused(pools[0], None, n, t, hyper, lst(g), None, len(numels), norm[0], None)
        else:
            apm.apm_page_adamw_step(pools[0], pages, n, t, hyper, norm[0], None)
        apm.apm_page_adamw_step_noalloc(pools[1], n, t, hyper, norm[1], None)
        torch.cuda.synchronize()
        assert torch.equal(norm[0].flip(0) if pages else norm[0], norm[1])
        for a, b in zip(state(pools[0]), state(pools[1])):
            assert torch.equal(a, b)
    for pool in pools:
        pool.destroy()


@pytest.mark.parametrize("clip,skip", [(0.0, 0), (0.05, 0), (0.05, 1), (0.0, 1)])
@pytest.mark.parametrize("n_small", [20, 5000])
def test_noalloc_step_by_launch_order_equals_the_step(n_small, clip, skip):
    """Full and nearly empty pages: with 20 small tensors the no-alloc step goes through the layout's launch order, with 5000 its records
    would not fit the scratch; per-page outputs in the caller's order either way."""
    E = 1 << 19
    numels = [E + 11, 300, 4 * E + 9] + [(7, 900, 20000)[k % 3] for k in range(n_small)] + [3 * E]
    pools, n, g, lst, draw, state = _pages_and_tensors(E, numels, 5, 2) if n_small < 1000 else _pages_and_tensors(16384, numels, 5, 2)
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, skip)
    norm = [torch.full((n,), -1.0, device=DEV) for _ in range(2)]
    mask = [torch.full((n,), 9, dtype=torch.uint8, device=DEV) for _ in range(2)]
    for t in (1, 2):
        draw()
        if skip:
            for pool in pools:
                page = torch.as_tensor(_Region(pool, apm.APM_G16, n * pool.desc.page_elems), device=DEV).view(n, -1)
                page[::3] = 0
        out = [x if clip or skip else None for x in norm]
        apm.apm_page_adamw_step(pools[0], None, n, t, hyper, out[0], mask[0] if skip else None)
        apm.apm_page_adamw_step_noalloc(pools[1], n, t, hyper, out[1], mask[1] if skip else None)
        torch.cuda.synchronize()
        assert torch.equal(*norm) and torch.equal(*mask)
        for a, b in zip(state(pools[0]), state(pools[1])):
            assert torch.equal(a, b)
    for pool in pools:
        pool.destroy()


@pytest.mark.parametrize("clip", [0.0, 0.05])
@pytest.mark.parametrize("form", ["pages", "tensors"])
@pytest.mark.parametrize("listed", ["down", "up and down", "pieces", "many pieces", "alternating"])
def test_long_lists_as_runs_equal_the_whole_step(listed, form, clip):
    """Lists beyond what a launch carries word by word: runs upwards and downwards, runs of one and two pages, more runs than a launch
    carries, hardly any runs; outputs by list position."""
    E, numels = 520, [(3, 1040, 519, 520 * 9 + 7)[k % 4] for k in range(600)]
    pools, n, g, lst, draw, state = _pages_and_tensors(E, numels, 9, 2)
    pages = {"down": list(range(n))[::-1], "up and down": list(range(n // 2, n)) + list(range(n // 2))[::-1],
             "pieces": [p for k in range(0, n - 40, 40) for p in ([k + 30, k + 31] + list(range(k, k + 20))[::-1] + [k + 39])],
             "many pieces": [p for k in range(0, n - 5, 5) for p in (k + 3, k + 2, k)],
             "alternating": [p ^ 1 for p in range(n // 2 * 2)]}[listed]
    assert len(pages) > 440
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, clip, 0)
    draw()
    before = state(pools[0])
    norm = [torch.zeros(len(pages), device=DEV), torch.zeros(n, device=DEV)]
    q = [torch.zeros_like(g) for _ in range(2)]
    for pool, lst_, m, out, qq in zip(pools, (pages, None), (len(pages), n), norm, q):
        out = out if clip else None
        if form == "tensors":
            apm.apm_page_adamw_step_fused(pool, lst_, m, 3, hyper, lst(g), lst(qq), len(numels), out, None)
        else:
            apm.apm_page_adamw_step(pool, lst_, m, 3, hyper, out, None)
    torch.cuda.synchronize()
    at = torch.tensor(pages, device=DEV)
    if clip:
        assert torch.equal(norm[0], norm[1][at])
    touched = torch.zeros(n, E, device=DEV)
    touched[at] = 1
    mask = apm.apm_pool_create(apm.APM_DEV_GPU, E, n, state_mask=1)
    apm.apm_pool_set_layout(mask, lst(before[0]), len(numels))
    torch.as_tensor(_Region(mask, apm.APM_P32, 2 * n * E), device=DEV).view(torch.float32).copy_(touched.flatten())
    on = torch.zeros_like(before[0])
    apm.apm_unpack(mask, apm.APM_P32, lst(on), len(numels))
    torch.cuda.synchronize()
    want = [torch.where(on > 0, new, old) for new, old in zip(state(pools[1]), before)]
    got = state(pools[0])
    if form == "tensors":
        got, want = got[:3] + [q[0]], want[:3] + [torch.where(on > 0, q[1], torch.zeros_like(q[1]))]
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    for pool in pools + [mask]:
        pool.destroy()


def test_a_later_step_with_norms_takes_no_more_memory():
    """What small steps with norms hand results on through comes with the pool's first call and is sized by the pages such a step
    can list: a pool of very many small pages, the first such step after others."""
    E, n = 64, 1 << 20
    numels = [40 + k % 20 for k in range(300)]
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    apm.apm_pool_set_layout(pool, apm.make_tensors(numels, apm.APM_BF16, None), len(numels))
    apm.apm_page_adamw_step(pool, None, 300, 1, apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, 0))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    norm = torch.full((300,), -1.0, device=DEV)
    apm.apm_page_adamw_step(pool, None, 300, 2, apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 1.0, 0), norm)
    torch.cuda.synchronize()
    assert (norm == 0).all()
    assert before - torch.cuda.mem_get_info()[0] < 32 << 20   # of the pool's pages: 128 bytes each, 128 MiB
    pool.destroy()


@pytest.mark.parametrize("listed", ["all", "head", "odd"])
@pytest.mark.parametrize("E,numels", [(4104, [1 + k * 7919 % 4100 for k in range(90)]), (49160, [49001] + [1600 + k for k in range(40)])])
def test_hand_overs_of_pages_that_hold_little_equal_the_synchronous_step(E, numels, listed):
    """Additions and copies without sums by four wavefronts a workgroup: pages well below their class's largest, ends in each wavefront's part."""
    pools, n, g, lst, draw, state = _pages_and_tensors(E, numels, E, 2)
    pages = {"all": None, "head": list(range(n - 1)), "odd": list(range(1, n, 2))}[listed]
    count = len(pages) if pages else n
    hyper = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 0.0, 0)
    for t in (1, 2, 3):
        parts = []
        for _ in range(2):
            draw()
            parts.append((torch.as_tensor(_Region(pools[0], apm.APM_G16, n * E), device=DEV).clone(), g.clone()))
        g.copy_((parts[0][1].float() + parts[1][1].float()).bfloat16())
        apm.apm_pack_tensors(pools[0], apm.APM_G16, lst(g), len(numels))
        apm.apm_page_adamw_step(pools[0], pages, count, t, hyper)
        apm.apm_step_delayed(pools[1], pages, count, parts[0][0].data_ptr(), hyper)
        apm.apm_delayed_accumulate(pools[1], pages, count, parts[1][0].data_ptr())
        torch.cuda.synchronize()
    apm.apm_step_delayed(pools[1], pages, count, None, hyper)
    torch.cuda.synchronize()
    for a, b in zip(state(pools[0]), state(pools[1])):
        assert torch.equal(a, b)
    for pool in pools:
        pool.destroy()


def test_norms_of_thousands_of_pages_cost_what_they_do_with_marked_words():
    """Beyond some pages, handing results on under the call's number costs more than the kernel that it saves (11 % here); the no-alloc step
    takes the marked form at every size."""
    E, n = 4096, 7168
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, E, n)
    g, q = (torch.full((n * E,), 1e-3, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    gl, ql = (apm.make_tensors([n * E], apm.APM_BF16, [t.data_ptr()]) for t in (g, q))
    apm.apm_pack_tensors(pool, apm.APM_G16, gl, 1)
    hyper, norm = apm.make_hyper(1e-3, 0.9, 0.999, 1e-8, 0.01, 1.0, 0), torch.zeros(n, device=DEV)
    fused = _us(lambda: apm.apm_page_adamw_step_fused(pool, None, n, 1, hyper, gl, ql, 1, norm, None), 50)
    marked = _us(lambda: apm.apm_page_adamw_step_noalloc(pool, n, 1, hyper, norm, None), 50)
    assert fused < 1.08 * marked, (fused, marked)
    pool.destroy()
