"""Calls of one record and of longer lists run different kernels (different
lanes per tile, different instruction order): the same records must give the
same bits through either, on every kind of last tile, in and out of place and
on shards; and the long-list kernel is checked against the oracle on the same
sizes."""
import numpy as np
import pytest

from paper_2306_10015_amd import synth
from gpu_util import assert_theta_close, to_device, to_host

pytestmark = pytest.mark.gpu

#: Around a lane's groups (4 and 8 elements), its share of a tile (16), a
#: wave's and a workgroup's pass over it, and the tiles (1024 fp32, 2048 bf16
#: and NF4 elements).
SIZES = [1, 3, 5, 8, 15, 17, 255, 257, 511, 1023, 1024, 1025, 1279, 2047, 2048, 2049, 3071, 4095, 4097, 6145]


@pytest.fixture(scope="module")
def mz():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2306_10015_amd import mezo
    return mezo


def records(n, seed):
    rng = np.random.default_rng(seed)
    out = np.zeros(n, dtype=synth.SEED_DTYPE)
    out["machine"] = np.sort(rng.integers(0, 2**63, size=n, dtype=np.int64))
    out["step"] = rng.integers(0, 2**32, size=n, dtype=np.int64)
    out["sample"] = rng.integers(0, 2**32, size=n, dtype=np.int64)
    return out, (rng.normal(size=n) * 1e-2).astype(np.float32)


def hosts(dtype, seed=3):
    return [synth.theta0_tensor((n,), dtype, 7 + i, seed) for i, n in enumerate(SIZES)]


def assert_few_codes_differ(a, b, sizes, n_rec):
    """4-bit storage in fast mode: calls of one record round the quantizer
    differently from lists, so a code may differ where x lies within about 2^-22
    of a midpoint. At 15 midpoints and a density of x below 0.8 that is at most
    5.7e-6 of the elements in each of the n_rec steps (twice that and 4 blocks
    are allowed; an element that becomes its block's largest takes the block
    along). All other blocks: every code equal, the absmax within 2^-22 a
    step."""
    import torch

    def blocks_of(t, n):
        c = torch.stack([t.codes & 15, t.codes >> 4], dim=1).reshape(-1)
        return torch.nn.functional.pad(c[:n], (0, -n % 64)).reshape(-1, 64)

    differing = 0
    for x, y, n in zip(a, b, sizes):
        same = (blocks_of(x, n) == blocks_of(y, n)).all(dim=1)
        differing += int((~same).sum())
        assert bool((((x.absmax - y.absmax).abs() <= n_rec * 2.0**-22 * y.absmax) | ~same).all()), n
    assert differing <= 4 + 2 * 5.7e-6 * n_rec * sum(sizes)


@pytest.mark.parametrize("gaussian", ["fast", "portable"])
@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16, synth.NF4])
@pytest.mark.parametrize("n_rec", [3, 40])
def test_list_kernel_matches_single_record_calls(mz, dtype, n_rec, gaussian):
    import torch
    g = mz.GAUSS_PORTABLE if gaussian == "portable" else mz.GAUSS_FAST
    ids = [5 * i + 1 for i in range(len(SIZES))]

    def fresh():
        if dtype == synth.NF4:
            ts = []
            for i, n in enumerate(SIZES):
                p, a = synth.nf4_theta0_tensor(n, i, 2)
                ts.append(mz.NF4Tensor(torch.from_numpy(p).cuda(), torch.from_numpy(a).cuda(), n))
            return ts
        return [to_device(h) for h in hosts(dtype)]

    seeds, scales = records(n_rec, 11 + n_rec)
    a, b = fresh(), fresh()
    pa, pb = mz.ParamSet(a, ids, gaussian=g), mz.ParamSet(b, ids, gaussian=g)
    pa.perturb_multi(seeds, scales)
    for s, c in zip(seeds, scales):
        pb.perturb(s, c)
    torch.cuda.synchronize()
    if dtype == synth.NF4 and gaussian == "fast":
        assert_few_codes_differ(a, b, SIZES, n_rec)
        pa.close()
        pb.close()
        return
    for n, x, y in zip(SIZES, a, b):
        if dtype == synth.NF4:
            assert torch.equal(x.codes, y.codes) and torch.equal(x.absmax, y.absmax), n
        else:
            assert np.array_equal(to_host(x).view(np.uint8), to_host(y).view(np.uint8)), n
    pa.close()
    pb.close()


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("K", [2, 5, 33])
def test_list_kernel_against_the_oracle(mz, orc, dtype, K):
    """One step of K records from a backup, on shards (first > 0) too."""
    seeds, _ = records(K, 70 + K)
    q = synth.grads_int8(K, seed=K)
    src_h = hosts(dtype, seed=9)
    # padded allocations: nothing outside the tensors may be written
    src = [to_device(h) for h in src_h]
    pads = [to_device(np.full(len(h) + 16, 1, dtype=h.dtype)) for h in src_h]
    dst = [p[: len(h)] for p, h in zip(pads, src_h)]
    firsts = [8 * i for i in range(len(SIZES))]
    ps, pd = mz.ParamSet(src, firsts=firsts), mz.ParamSet(dst, firsts=firsts)
    lr = 1e-3
    pd.update_multi_from(ps, seeds, q, lr)
    for i, h in enumerate(src_h):
        assert np.array_equal(to_host(src[i]).view(np.uint8), h.view(np.uint8))
        ref = np.zeros(firsts[i] + len(h), dtype=h.dtype)
        ref[firsts[i]:] = h
        full_in = ref.copy()
        orc.update(ref, i, seeds, q, lr)
        assert_theta_close(to_host(dst[i]), ref[firsts[i]:], f"n={len(h)}", inp=full_in[firsts[i]:])
        assert np.array_equal(to_host(pads[i][len(h):]), np.full(16, 1, dtype=h.dtype)), len(h)
    ps.close()
    pd.close()


@pytest.mark.parametrize("dtype,tiles,gaussian", [
    # one set on each side of the sizes at which the kernel changes: issue
    # phases, more blocks per lane
    (synth.F32, 257, "fast"), (synth.BF16, 257, "fast"), (synth.NF4, 257, "fast"),
    (synth.F32, 24 * 1024, "fast"), (synth.F32, 96 * 1024, "fast"), (synth.BF16, 8 * 1024, "fast"),
    (synth.F32, 64 * 1024, "portable"), (synth.NF4, 12 * 1024, "fast"), (synth.NF4, 48 * 1024, "portable")])
def test_list_kernels_of_large_sets(mz, dtype, tiles, gaussian):
    """Ragged tensors beside a large one that makes the set's tile count cross
    the line: three records in one pass against three calls."""
    import torch
    g = mz.GAUSS_PORTABLE if gaussian == "portable" else mz.GAUSS_FAST
    per = 1024 if dtype == synth.F32 else 2048
    small_tiles = sum((n + per - 1) // per for n in SIZES)
    seeds, scales = records(3, 23)
    for big_tiles in (tiles - small_tiles - 1, tiles - small_tiles):
        sizes = SIZES + [big_tiles * per - 5]
        ids = [3 * i + 2 for i in range(len(sizes))]

        def fresh():
            gen = torch.Generator(device="cuda")
            gen.manual_seed(5)
            out = []
            for n in sizes:
                if dtype == synth.NF4:
                    t = mz.NF4Tensor.empty(n)
                    t.codes.random_(0, 256, generator=gen)
                    if n % 2:
                        t.codes[-1] &= 15
                    t.absmax.uniform_(0.04, 0.06, generator=gen)
                    out.append(t)
                else:
                    x = torch.empty(n, device="cuda").normal_(0.0, 0.02, generator=gen)
                    out.append(x if dtype == synth.F32 else x.bfloat16())
            return out

        a, b = fresh(), fresh()
        pa, pb = mz.ParamSet(a, ids, gaussian=g), mz.ParamSet(b, ids, gaussian=g)
        pa.perturb_multi(seeds, scales)
        for s, c in zip(seeds, scales):
            pb.perturb(s, c)
        for n, x, y in zip(sizes, a, b):
            if dtype != synth.NF4:
                same = torch.int32 if dtype == synth.F32 else torch.int16
                assert torch.equal(x.view(same), y.view(same)), (big_tiles, n)
            elif gaussian == "portable":
                assert torch.equal(x.codes, y.codes) and torch.equal(x.absmax, y.absmax), (big_tiles, n)
        if dtype == synth.NF4 and gaussian == "fast":
            assert_few_codes_differ(a, b, sizes, 3)
        pa.close()
        pb.close()


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("spread", [1, 6, 7, 8, 11, 13, 14])
def test_checksum_runs_across_tensor_ends(mz, orc, dtype, spread):
    """A workgroup's run of tiles in groups of eight: short tensors one after
    another, in one group or several, between tensors of many tiles, and a
    shard's chunk numbers. The 512 workgroups' runs are of 0 to 1, 4 to 7, 10
    to 11 and 13 to 16 tiles: short ones taken a tile at a time or in a group,
    and long ones' last 2 to 8."""
    per = 1024 if dtype == synth.F32 else 2048
    sizes = list(SIZES)
    for i in range(spread):
        sizes += [(37 * i + 300) * per + [0, 1, 5, per - 1][i % 4], 3, per + 2, 9, 2 * per, per - 3]
    hs = [synth.theta0_tensor((n,), dtype, i, 9) for i, n in enumerate(sizes)]
    ids = [4 * i + 3 for i in range(len(sizes))]
    want = orc.checksum(hs, ids)
    devs = [to_device(h) for h in hs]
    ps = mz.ParamSet(devs, ids)
    assert ps.checksum() == want and ps.checksum() == want
    ps.close()
    # every tensor's rest after its first 16 elements, or all of a short one
    cuts = [16 if n > 16 else 0 for n in sizes]
    heads = [(d[:16], i) for d, i, c in zip(devs, ids, cuts) if c]
    a = mz.ParamSet([d for d, _ in heads], [i for _, i in heads])
    b = mz.ParamSet([to_device(h[c:]) for h, c in zip(hs, cuts)], ids, firsts=cuts)
    assert (a.checksum() + b.checksum()) & 0xFFFFFFFFFFFFFFFF == want
    a.close()
    b.close()


@pytest.mark.parametrize("types", [[synth.F32], [synth.F32, synth.BF16], [synth.BF16, synth.NF4]])
@pytest.mark.parametrize("n_rec,n", [(1, 1 << 22), (2, 1 << 24), (30, 1 << 22), (30, 1 << 24)])
def test_destroy_with_queued_calls(mz, types, n_rec, n):
    """Sets, destination and source, destroyed with a queue of short calls on two
    streams still running: nothing they use goes first, and the streams are
    drained. (Freeing device memory waits for the device by itself, so this
    cannot tell whether destroy's own waits are right: the host check on the
    CPU does, tests/sanitize/abi_host_check.c, check_waits.)"""
    import torch

    def fresh():
        return mz.ParamSet([mz.NF4Tensor.empty(n) if d == synth.NF4 else
                            torch.zeros(n, device="cuda", dtype=torch.float32 if d == synth.F32 else torch.bfloat16)
                            for d in types])

    a, b = fresh(), fresh()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    seeds, scales = records(n_rec, 31)
    out = torch.zeros(1, dtype=torch.int64, device="cuda")
    a.checksum(), b.checksum()
    torch.cuda.synchronize()
    for _ in range(100):
        for s in streams:
            a.perturb_multi(seeds, scales, stream=s)
    b.perturb_from(a, (1, 2, 3), 1e-3, stream=streams[0])
    a.checksum_into(out, stream=streams[1])
    a.close()
    assert streams[0].query() and streams[1].query()
    b.close()


@pytest.mark.parametrize("n", [1 << 20, (1 << 24) + 1029])
@pytest.mark.parametrize("last", ["checksum", "perturb"])
@pytest.mark.parametrize("dtypes", [[synth.F32], [synth.BF16, synth.F32]])
def test_a_taken_over_entry_waits_for_its_work(mz, orc, dtypes, last, n):
    """The first stream's last call on a set, a checksum or a perturbation, waits
    behind a long queue of another set's work; fifteen more streams use the set;
    the seventeenth takes the first one's entry and its running sum, and must
    wait on the host for that call: its own checksum then sees the perturbed
    weights, and what it leaves on its stream the first stream's result. On both
    routes of the entry's event: recorded behind the call, or completed by the
    call's last launch (2^24 elements on)."""
    import torch
    src_h = [synth.theta0_tensor((n if i == 0 else 5001,), d, i, 4) for i, d in enumerate(dtypes)]
    devs = [to_device(h) for h in src_h]
    ps = mz.ParamSet(devs)
    seed, scale = (3, 1, 4), 1e-3
    other = mz.ParamSet([torch.zeros(1 << 26, device="cuda")])
    seeds, _ = records(30, 5)
    q = synth.grads_int8(30, seed=5)
    streams = [torch.cuda.Stream() for _ in range(17)]
    outs = torch.zeros(17, dtype=torch.int64, device="cuda")
    # the tables and every stream's queue are made before the clock runs
    other.update_multi(seeds, q, 1e-3)
    ps.checksum_into(outs[:1], stream=streams[0])
    for s in streams:
        s.wait_stream(streams[0])
        with torch.cuda.stream(s):
            outs.zero_()
    torch.cuda.synchronize()
    for _ in range(60):  # tens of milliseconds
        other.update_multi(seeds, q, 1e-3, stream=streams[0])
    if last == "checksum":
        ps.checksum_into(outs[:1], stream=streams[0])
    else:
        ps.perturb(seed, scale, stream=streams[0])
    for i in range(1, 16):
        ps.checksum_into(outs[i:i + 1], stream=streams[i])
    assert not streams[0].query()
    ps.checksum_into(outs[16:], stream=streams[16])
    with torch.cuda.stream(streams[16]):
        got = [int(v) & 0xFFFFFFFFFFFFFFFF for v in outs[::16].tolist()]
    torch.cuda.synchronize()
    want = orc.checksum([to_host(t) for t in devs])
    assert got == [want if last == "checksum" else 0, want]
    assert ps.checksum() == want
    ps.close()
    other.close()
