"""N = 2048 and 4096 with few ciphertexts, where two workgroups share each: against the kernels with one workgroup per ciphertext (which larger
batches, captured calls and calls beside another stream's take) bit for bit; those are compared with the oracle elsewhere."""
import ctypes
import threading

import numpy as np
import pytest

import synth
from tests.test_gpu_fft import _inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slz():
    import paper_2504_17785_amd as m
    return m


def _case(slz, N, batch, n):
    p = synth.CONFIGS[2].with_(name="pairs", N=N, n=n, pbs_level=1, pbs_base_log=22, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", n * 4 * N).reshape(n, 2, 1, 2, N)
    luts = synth.raw_words(p, "misc", 2 * N).reshape(2, N)
    cts = synth.raw_words(p, "raw_ct", batch * (n + 1)).reshape(batch, n + 1)
    ctx = slz.Context(p, batch)
    d_bsk = ctx.bsk_prepare(slz.to_device_u64(bsk))
    return ctx, [slz.to_device_u64(cts), slz.to_device_u64(luts), torch.from_numpy((np.arange(batch) % 2).astype(np.int32)).cuda(), d_bsk]


def _driver(slz, N):
    """The launch with any number of workgroups and any patience (an internal function, by its mangled name)."""
    run = getattr(slz.lib(), "_Z16slz_fft%d_pairP7slz_ctxPKmS2_PKjPKvjPmS7_jjjP12ihipStream_t" % N)
    run.argtypes = [ctypes.c_void_p] * 5 + [ctypes.c_uint32] + [ctypes.c_void_p] * 2 + [ctypes.c_uint32] * 3 + [ctypes.c_void_p]
    run.restype = ctypes.c_int
    return run


@pytest.mark.parametrize("N", [2048, 4096])
def test_pairs_of_workgroups_match_one_workgroup(slz, N):
    # 129 ciphertexts are one past the pairs' last; 8 and 9: one pair per XCD and a second on each; odd and even numbers of steps, from the fewest on that
    # pairs take (N = 2048: 8; N = 4096: 8 up to 64 ciphertexts, 32 up to 100, 64 above) and below
    ctx, d = _case(slz, N, 129, 65)
    for steps in (1, 7, 8, 9, 31, 32, 41, 63, 64, 65):
        every = ctx.blind_rotate_batch(*d, steps)
        for count in (1, 2, 8, 9, 63, 100, 127, 128):
            part = ctx.blind_rotate_batch(d[0][:count], d[1], d[2][:count], d[3], steps)
            assert torch.equal(part, every[:count]), (steps, count)
    every = ctx.pbs_batch(*d)
    for _ in range(3):
        assert torch.equal(ctx.pbs_batch(d[0][:100], d[1], d[2][:100], d[3]), every[:100])


@pytest.mark.parametrize("N,batch,beta,extreme", [(2048, 1, 23, False), (2048, 5, 12, True), (2048, 37, 1, False), (2048, 100, 23, True), (2048, 128, 8, True),
                                                   (4096, 1, 22, True), (4096, 37, 1, False), (4096, 64, 13, True)])
def test_pairs_of_workgroups_match_generic_path_and_oracle(slz, N, batch, beta, extreme):
    import oracle as orc
    n = 9
    p, ctx, bsk, luts, cts, idx, d = _inputs(slz, batch, beta, n=n, extreme=extreme, N=N)
    got = {s: ctx.blind_rotate_batch(*d, s) for s in (8, 9)}
    out, out0 = ctx.pbs_batch(*d), ctx.pbs_batch(d[0], d[1], None, d[3])
    ctx.set_option(slz.SLZ_OPT_FORCE_GENERIC, 1)                       # the same prepared key
    for s, acc in got.items():
        assert torch.equal(acc, ctx.blind_rotate_batch(*d, s)), s
    assert torch.equal(out, ctx.pbs_batch(*d))
    assert torch.equal(out0, ctx.pbs_batch(d[0], d[1], None, d[3]))
    sample = np.unique([0, batch // 2, batch - 1])
    assert np.array_equal(slz.to_host_u64(out)[sample], orc.pbs_batch(p, cts[sample], luts, idx[sample], bsk))


@pytest.mark.parametrize("N", [2048, 4096])
def test_pairs_of_workgroups_beside_other_streams_and_in_graphs(slz, N):
    ctx, d = _case(slz, N, 129, 40)
    every = ctx.pbs_batch(*d)
    count = 100
    few = [d[0][:count].clone(), d[1], d[2][:count].clone(), d[3]]
    outs = [torch.empty_like(every[:count]) for _ in range(6)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for i, out in enumerate(outs):                      # calls of one context on two streams at once
        with torch.cuda.stream(streams[i % 2]):
            ctx.pbs_batch(*few, out=out)
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        assert torch.equal(out, every[:count]), i
    def calls(i):                                       # and by two threads
        with torch.cuda.stream(streams[i]):
            for _ in range(20):
                ctx.pbs_batch(*few, out=outs[i])
    threads = [threading.Thread(target=calls, args=(i,)) for i in range(2)]
    for out in outs:
        out.zero_()
    torch.cuda.synchronize()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert torch.equal(outs[0], every[:count]) and torch.equal(outs[1], every[:count])
    graph, out = torch.cuda.CUDAGraph(), torch.empty_like(outs[0])
    with torch.cuda.graph(graph):
        ctx.pbs_batch(*few, out=out)
    for rep in range(3):                                # replays beside eager calls on another stream
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        with torch.cuda.stream(streams[0]):
            ctx.pbs_batch(*few, out=outs[0])
        torch.cuda.synchronize()
        assert torch.equal(out, every[:count]) and torch.equal(outs[0], every[:count]), rep


@pytest.mark.parametrize("N", [2048, 4096])
def test_pairs_of_workgroups_of_several_contexts_at_once(slz, N):
    # 2 x 64 ciphertexts have room for their pairs together, 3 x 80 and 2 x 128 have not: those that do not find all their places leave the ciphertexts to
    # the kernel with one workgroup on each
    cases = [_case(slz, N, 128, 65) for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in cases]
    d = cases[0][1]
    want = _case(slz, N, 129, 65)[0].pbs_batch(torch.cat([d[0], d[0][:1]]), d[1], torch.cat([d[2], d[2][:1]]), d[3])[:128]
    for contexts, count in ((2, 64), (3, 80), (2, 128)):
        outs = [torch.zeros_like(want[:count]) for _ in range(4 * contexts)]
        torch.cuda.synchronize()
        for i, out in enumerate(outs):
            with torch.cuda.stream(streams[i % contexts]):
                cases[i % contexts][0].pbs_batch(d[0][:count], d[1], d[2][:count], d[3], out=out)
        torch.cuda.synchronize()
        assert all(torch.equal(out, want[:count]) for out in outs), (contexts, count)


@pytest.mark.parametrize("N", [2048, 4096])
def test_pairs_memory_comes_with_the_first_call_and_may_be_refused(slz, N):
    def pairs_ran(ctx, d):
        out = torch.zeros((100, 2, N), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        rc = _driver(slz, N)(ctx._h, d[0].data_ptr(), d[1].data_ptr(), d[2].data_ptr(), d[3].data_ptr() + 33 * 2 * 4 * N * 8, 33, out.data_ptr(), None, 100,
                             208, 200000, None)
        torch.cuda.synchronize()
        assert rc == slz.SLZ_E_INVALID_ARG or torch.equal(out, ctx.blind_rotate_batch(*d, 33)[:100])
        return rc == slz.SLZ_OK

    ctx, d = _case(slz, N, 129, 33)
    few = [d[0][:100].clone(), d[1], d[2][:100].clone(), d[3]]
    ctx.set_option(slz.SLZ_OPT_FAIL_ALLOC_AFTER, 0)     # the first call's allocation: that call and all after it run without pairs
    every = ctx.pbs_batch(*d)
    assert torch.equal(ctx.pbs_batch(*few), every[:100]) and not pairs_ran(ctx, d)
    other, e = _case(slz, N, 129, 33)                   # a batch that makes no pairs brings their memory, and later calls ask for none
    other.pbs_batch(*e)
    assert pairs_ran(other, e)
    other.set_option(slz.SLZ_OPT_FAIL_ALLOC_AFTER, 0)
    assert torch.equal(other.pbs_batch(*few), every[:100])
    with pytest.raises(slz.SlzError) as err:            # still armed: the keyswitch's digit scratch meets it
        other.keyswitch_batch(every, torch.zeros((N, other.p.ks_level, 34), dtype=torch.int64, device="cuda"))
    assert err.value.code == slz.SLZ_E_NOMEM
    # a first call beside another stream's capture, which may allocate nothing itself
    third, e = _case(slz, N, 129, 33)
    side, graph, out, again = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.empty_like(every), torch.empty_like(every)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        other.pbs_batch(*d, out=out)
        with torch.cuda.stream(side):
            third.pbs_batch(*e, out=again)
    torch.cuda.synchronize()
    assert torch.equal(again, every) and pairs_ran(third, e)
    out.zero_()
    for rep in range(2):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, every), rep


@pytest.mark.parametrize("N", [2048, 4096])
def test_pairs_of_workgroups_do_every_ciphertext_whatever_their_number_and_patience(slz, N):
    # A workgroup per XCD or fewer: nobody has a partner, all leave and the launch
    # behind takes everything.  16 to 40: two to five of an XCD, so pairs with many ciphertexts each and workgroups left over.  Without
    # patience the first one to come finds that not all have, and all leave.
    count, n = 100, 33
    ctx, d = _case(slz, N, 129, n)
    run = _driver(slz, N)
    key = d[3].data_ptr() + n * 2 * 4 * N * 8            # the transform form, behind the residues
    ctx.blind_rotate_batch(d[0][:1], d[1], d[2][:1], d[3], n)         # allocates what pairs need
    for steps in (1, 5, 6):
        want = ctx.blind_rotate_batch(*d, steps)[:count]
        for workgroups in (1, 7, 8, 16, 17, 18, 31, 40, 208, 256):
            for patience in (200000, 0):
                out = torch.full_like(want, -1)
                torch.cuda.synchronize()
                assert run(ctx._h, d[0].data_ptr(), d[1].data_ptr(), d[2].data_ptr(), key, steps, out.data_ptr(), None, count, workgroups, patience,
                           None) == 0
                torch.cuda.synchronize()
                assert torch.equal(out, want), (steps, workgroups, patience)
    assert run(ctx._h, d[0].data_ptr(), d[1].data_ptr(), d[2].data_ptr(), key, 1, want.data_ptr(), None, count, 257, 0, None) == slz.SLZ_E_INVALID_ARG


@pytest.mark.parametrize("N", [2048, 4096])
def test_lookups_on_streams_limited_to_some_compute_units(slz, N):
    # one, two and eight compute units of every XCD; 7 ciphertexts make 8 pairs at most, which fit the last two, 100 fit none of them
    ctx, d = _case(slz, N, 129, 33)
    every = ctx.pbs_batch(*d)
    fits = slz.lib()._Z13slz_pairs_fitjP12ihipStream_t
    fits.argtypes, fits.restype = [ctypes.c_uint32, ctypes.c_void_p], ctypes.c_int
    assert fits(128, None) and not fits(129, None)
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    for units in (8, 16, 64):
        handle = ctypes.c_void_p()
        mask = (ctypes.c_uint32 * 8)(*[min(0xffffffff, (1 << max(0, units - 32 * i)) - 1) for i in range(8)])
        assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
        assert [bool(fits(count, handle)) for count in (1, 7, 32, 33)] == [units >= 16, units >= 16, units >= 64, False]
        with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
            for count in (1, 7, 100):
                got = ctx.pbs_batch(d[0][:count], d[1], d[2][:count], d[3])
                torch.cuda.synchronize()
                assert torch.equal(got, every[:count]), (units, count)
