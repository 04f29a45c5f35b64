"""N = 512 (two levels), 1024 and 2048 through exact floating-point transforms, and how the large-N path cuts its batches: bit for bit
against the oracle and the generic path or one lane."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slz():
    import paper_2504_17785_amd as m
    return m


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


def _inputs(slz, batch, beta, n=3, extreme=False, N=2048):
    l = 2 if N == 512 else 1
    p = synth.CONFIGS[2].with_(name="fft", N=N, n=n, pbs_level=l, pbs_base_log=beta, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", n * 4 * l * N)
    luts = synth.raw_words(p, "misc", 2 * N).reshape(2, N)
    cts = synth.raw_words(p, "raw_ct", batch * (n + 1)).reshape(batch, n + 1)
    if extreme:
        # key words whose pieces are all of the largest magnitude and sign patterns that line their spectra up, digits at
        # -B/2 and B/2 - 1, rotations by N (X^N = -1: every difference is -2 ACC) and by odd amounts
        bsk[:2 * N] = np.uint64(0x7FFF7FFBFFDFFEFF)
        bsk[2 * N:4 * N:2] = np.uint64(1 << 63)
        bsk[4 * N:8 * N:3] = np.uint64(0xF001800C00600300)
        bsk[8 * N:] = np.uint64(0x0010008004002001) * np.uint64(0xFFF)
        luts[0] = np.uint64(1 << 62)
        luts[1, 0::2] = np.uint64((1 << 63) - (1 << 40))
        luts[1, 1::2] = np.uint64(1 << 63)
        cts[0::3] = np.uint64(1 << 63)
        cts[1::3, 0] = np.uint64(1 << 63)
    idx = (np.arange(batch) % 2).astype(np.uint32)
    ctx = slz.Context(p, batch)
    assert ctx.path == "fused_n%d" % N
    # the prepared key: the residue form, and behind it the transform form where the error bound holds
    steps = {4096: 5 * 4 * 8 * 4 * 64, 2048: 5 * 2 * 8 * 4 * 64, 1024: 5 * 8 * 4 * 64, 512: 3 * 4 * 8 * 64}
    transform = n * steps[N] * 16 if beta <= {4096: 22, 2048: 23, 1024: 23, 512: 14}[N] else 0
    assert ctx.bsk_prepared_bytes() == n * 2 * 4 * l * N * 8 + transform
    d = [slz.to_device_u64(cts), slz.to_device_u64(luts), torch.from_numpy(idx.astype(np.int32)).cuda(),
         ctx.bsk_prepare(slz.to_device_u64(bsk.reshape(n, 2, l, 2, N)))]
    return p, ctx, bsk.reshape(n, 2, l, 2, N), luts, cts, idx, d


# N = 2048: 2^23 is the largest base a context takes; 256 and 257 ciphertexts are the two sides of the line between the two forms of
# the kernel, 1025 and 1300 give some pairs of waves a second ciphertext.  N = 1024: the lines are at 256, 512 and 1024, 2100 gives some
# waves a second ciphertext; 2^23 is the largest base whose error bound holds (2^24 stays on residues).  N = 512: the lines are at 256
# and 512; 2^14 is the largest base whose bound holds.
@pytest.mark.parametrize("N,batch,beta,extreme", [
    (2048, 1, 23, False), (2048, 5, 12, True), (2048, 37, 1, False), (2048, 256, 23, True), (2048, 257, 23, False),
    (2048, 300, 23, True), (2048, 300, 1, True), (2048, 260, 12, False), (2048, 1025, 23, False), (2048, 1300, 22, True),
    (1024, 1, 23, False), (1024, 3, 12, True), (1024, 256, 23, True), (1024, 257, 23, True), (1024, 512, 23, False), (1024, 513, 23, True), (1024, 600, 1, False),
    (1024, 1024, 23, False), (1024, 1025, 23, True), (1024, 2100, 22, True), (1024, 40, 24, True),
    (512, 1, 8, False), (512, 7, 14, True), (512, 256, 1, False), (512, 257, 14, True), (512, 512, 8, False), (512, 513, 8, True),
    (512, 1024, 14, False), (512, 1025, 14, True), (512, 2100, 8, False), (512, 40, 15, True)])
def test_fft_states_and_outputs_match_generic_path_and_oracle(slz, orc, N, batch, beta, extreme):
    p, ctx, bsk, luts, cts, idx, d = _inputs(slz, batch, beta, extreme=extreme, N=N)
    sample = np.unique(np.minimum([0, 1, 2, 255, 256, batch - 1], batch - 1))
    got = {s: ctx.blind_rotate_batch(*d, s) for s in (0, 1, p.n)}
    out, out0 = ctx.pbs_batch(*d), ctx.pbs_batch(d[0], d[1], None, d[3])
    # which of the two kernels behind one path name ran: without the residue form only the transform kernel gives the same
    other = d[3].clone()
    other[:bsk.size * 2] = 0
    assert torch.equal(ctx.pbs_batch(*d[:3], other), out) == (other.numel() > bsk.size * 2)
    ctx.set_option(slz.SLZ_OPT_FORCE_GENERIC, 1)                       # the same prepared key
    for s, acc in got.items():
        assert torch.equal(acc, ctx.blind_rotate_batch(*d, s)), s
        want = orc.blind_rotate_batch(p, cts[sample], luts, idx[sample], bsk, s)
        assert np.array_equal(slz.to_host_u64(acc)[sample], want), s
    assert torch.equal(out, ctx.pbs_batch(*d))
    assert torch.equal(out0, ctx.pbs_batch(d[0], d[1], None, d[3]))
    assert np.array_equal(slz.to_host_u64(out)[sample], orc.pbs_batch(p, cts[sample], luts, idx[sample], bsk))


# N = 2048, 200 and 256 ciphertexts with eight waves on each, 257, 511 and 512 with four (an odd count leaves one half of a workgroup
# idle), 513 with two: a ciphertext's result does not depend on which
def test_fft2048_forms_agree(slz):
    p, ctx, bsk, luts, cts, idx, d = _inputs(slz, 513, 23, n=4)
    want = ctx.blind_rotate_batch(*d, p.n)
    for count in (512, 511, 257, 256, 200, 1):
        assert torch.equal(ctx.blind_rotate_batch(d[0][:count], d[1], d[2][:count], d[3], p.n), want[:count]), count


# N = 4096: one ciphertext, all workgroups busy, a second round for one and for 44 of them; the largest base a context takes is 2^22
@pytest.mark.parametrize("batch,beta,extreme", [(1, 22, False), (5, 22, True), (256, 1, False), (257, 22, True), (300, 13, True)])
def test_fft4096_states_and_outputs_match_generic_path_and_oracle(slz, orc, batch, beta, extreme):
    N, n = 4096, 2
    p = synth.CONFIGS[2].with_(name="fft", N=N, n=n, pbs_base_log=beta, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", n * 4 * N)
    luts = synth.raw_words(p, "misc", 2 * N).reshape(2, N)
    cts = synth.raw_words(p, "raw_ct", batch * (n + 1)).reshape(batch, n + 1)
    if extreme:                                 # as above: pieces of the largest magnitude, digits at the ends, rotations by N
        bsk[:2 * N] = np.uint64(0x7FFF7FFBFFDFFEFF)
        bsk[2 * N:4 * N:2] = np.uint64(1 << 63)
        bsk[4 * N:8 * N:3] = np.uint64(0xF001800C00600300)
        luts[0] = np.uint64(1 << 62)
        luts[1, 0::2] = np.uint64((1 << 63) - (1 << (63 - beta)))
        luts[1, 1::2] = np.uint64(1 << 63)
        cts[0::3] = np.uint64(1 << 63)
        cts[1::3, 0] = np.uint64(1 << 63)
    idx = (np.arange(batch) % 2).astype(np.uint32)
    ctx = slz.Context(p, batch)
    assert ctx.path == "fused_n4096"
    assert ctx.bsk_prepared_bytes() == n * 2 * 4 * N * 8 + n * 5 * 4 * 8 * 4 * 64 * 16
    bsk = bsk.reshape(n, 2, 1, 2, N)
    d = [slz.to_device_u64(cts), slz.to_device_u64(luts), torch.from_numpy(idx.astype(np.int32)).cuda(), ctx.bsk_prepare(slz.to_device_u64(bsk))]
    sample = np.unique(np.minimum([0, 1, 2, 255, 256, batch - 1], batch - 1))
    got = {s: ctx.blind_rotate_batch(*d, s) for s in (0, 1, n)}
    out, out0 = ctx.pbs_batch(*d), ctx.pbs_batch(d[0], d[1], None, d[3])
    other = d[3].clone()
    other[:bsk.size * 2] = 0                    # without the residue form: the transform kernel ran
    assert torch.equal(ctx.pbs_batch(*d[:3], other), out)
    ctx.set_option(slz.SLZ_OPT_FORCE_GENERIC, 1)
    for s, acc in got.items():
        assert torch.equal(acc, ctx.blind_rotate_batch(*d, s)), s
    want = orc.blind_rotate_batch(p, cts[sample], luts, idx[sample], bsk, n)
    assert np.array_equal(slz.to_host_u64(got[n])[sample], want)
    assert torch.equal(out, ctx.pbs_batch(*d))
    assert torch.equal(out0, ctx.pbs_batch(d[0], d[1], None, d[3]))


# Three launches per step.  N = 16384: one lane up to 32 ciphertexts, two even halves from 33 to 128, halves of 64 past that.  N = 8192: even
# lanes from 65 to 160 and from 208 to 256, a lane of 128 and the rest in between; N = 4096: even lanes from 129 to 320, then a lane of 256 and
# the rest.  By default up to 56 ciphertexts of N = 16384 and 96 of N = 8192 take two launches per step, so every size runs without them as well.
@pytest.mark.parametrize("N,batch", [(16384, 32), (16384, 33), (16384, 49), (16384, 128), (16384, 129), (8192, 66), (8192, 67), (8192, 98), (8192, 99), (8192, 161),
                                     (8192, 208), (4096, 129), (4096, 134), (4096, 321)])
def test_large_n_halves_match_one_lane_and_oracle(slz, orc, N, batch):
    p = synth.CONFIGS[2].with_(name="halves", N=N, n=2, pbs_level=2, pbs_base_log=15, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", p.n * 8 * p.N).reshape(p.n, 2, 2, 2, p.N)
    luts = synth.raw_words(p, "misc", p.N).reshape(1, p.N)
    cts = synth.raw_words(p, "raw_ct", batch * (p.n + 1)).reshape(batch, p.n + 1)
    ctx = slz.Context(p, batch)
    assert ctx.path == "three_pass_large_n"
    d = [slz.to_device_u64(cts), slz.to_device_u64(luts), None, ctx.bsk_prepare(slz.to_device_u64(bsk))]
    got = [ctx.pbs_batch(*d) for _ in range(3)]
    ctx.set_option(slz.SLZ_OPT_LARGE_N_LATENCY, 0)
    got += [ctx.pbs_batch(*d) for _ in range(3)]
    ctx.set_option(slz.SLZ_OPT_LARGE_N_LANES, 1)
    want = ctx.pbs_batch(*d)
    assert all(torch.equal(g, want) for g in got)
    idx = np.array([0, batch // 2 - 1, (batch + 1) // 2, batch - 1])
    assert np.array_equal(slz.to_host_u64(want)[idx], orc.pbs_batch(p, cts[idx], luts, np.zeros(4, np.uint32), bsk))


# One lane up to 32 ciphertexts, so a context that has only seen 20 has no lane streams when the capture begins.  Kernels a lane: 49 ciphertexts
# take two a step and one at the end, 65 three a step.
@pytest.mark.parametrize("batch,kernels", [(49, 5), (65, 6)])
def test_large_n_graph_gets_both_lanes_whatever_the_context_ran_before(slz, batch, kernels):
    import ctypes
    p = synth.CONFIGS[2].with_(name="halves", N=16384, n=2, pbs_level=2, pbs_base_log=15, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", p.n * 8 * p.N).reshape(p.n, 2, 2, 2, p.N)
    d_luts = slz.to_device_u64(synth.raw_words(p, "misc", p.N).reshape(1, p.N))
    d_in = slz.to_device_u64(synth.raw_words(p, "raw_ct", batch * (p.n + 1)).reshape(batch, p.n + 1))
    out = torch.empty((batch, p.N + 1), dtype=torch.int64, device="cuda")
    nodes = {}
    for warm in (batch, 20):
        ctx = slz.Context(p, batch)
        d_key = ctx.bsk_prepare(slz.to_device_u64(bsk))
        ctx.pbs_batch(d_in[:warm], d_luts, None, d_key)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            ctx.pbs_batch(d_in, d_luts, None, d_key, out=out)
        count = ctypes.c_size_t(0)
        assert slz.lib().hipGraphGetNodes(ctypes.c_void_p(int(graph.raw_cuda_graph())), None, ctypes.byref(count)) == 0
        nodes[warm] = count.value
        graph.instantiate()
        for rep in range(3):
            d_in.copy_(slz.to_device_u64(synth.raw_words(p, "raw_ct", batch * (p.n + 1), offset=999 * rep + warm).reshape(batch, p.n + 1)))
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ctx.pbs_batch(d_in, d_luts, None, d_key)), (warm, rep)
    assert nodes[20] == nodes[batch] == 2 * kernels + 2      # two lanes, the accumulators' start and extraction


# Without the two-launch steps 33 to 56 ciphertexts of N = 16384 (and 17 to 32 of 32768, 65 to 96 of 8192) are two even halves on the two lanes
@pytest.mark.parametrize("N,batch,lanes", [(16384, 32, 1), (16384, 33, 2), (16384, 49, 2), (32768, 17, 2), (8192, 66, 2)])
def test_large_n_three_launch_steps_get_both_lanes_at_every_batch_that_had_them(slz, N, batch, lanes):
    import ctypes
    p = synth.CONFIGS[2].with_(name="halves", N=N, n=2, pbs_level=2, pbs_base_log=15, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", p.n * 8 * p.N).reshape(p.n, 2, 2, 2, p.N)
    d_luts = slz.to_device_u64(synth.raw_words(p, "misc", p.N).reshape(1, p.N))
    d_in = slz.to_device_u64(synth.raw_words(p, "raw_ct", batch * (p.n + 1)).reshape(batch, p.n + 1))
    ctx = slz.Context(p, batch)
    d_key = ctx.bsk_prepare(slz.to_device_u64(bsk))
    want = ctx.pbs_batch(d_in, d_luts, None, d_key)
    out = torch.empty_like(want)
    ctx.set_option(slz.SLZ_OPT_LARGE_N_LATENCY, 0)
    nodes = {}
    for option in (1, 2):
        ctx.set_option(slz.SLZ_OPT_LARGE_N_LANES, option)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            ctx.pbs_batch(d_in, d_luts, None, d_key, out=out)
        count = ctypes.c_size_t(0)
        assert slz.lib().hipGraphGetNodes(ctypes.c_void_p(int(graph.raw_cuda_graph())), None, ctypes.byref(count)) == 0
        nodes[option] = count.value
        graph.instantiate()
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            assert torch.equal(ctx.pbs_batch(d_in, d_luts, None, d_key), want)
    assert nodes[2] - nodes[1] == (lanes - 1) * 3 * p.n


# The largest batch of the two-launch steps and one past it, by the kernels of a captured call: 2 n + 1 a lane against 3 n, and the accumulators'
# start and extraction
@pytest.mark.parametrize("N,l,beta,last,lanes", [(2048, 3, 12, 128, 1), (2048, 4, 12, 192, 1), (4096, 3, 12, 64, 1), (4096, 4, 12, 96, 1), (8192, 1, 20, 96, 1),
                                                 (8192, 3, 12, 32, 1), (8192, 4, 10, 48, 1), (16384, 1, 20, 49, 2), (16384, 2, 15, 56, 2), (16384, 3, 12, 40, 2),
                                                 (32768, 3, 12, 22, 2), (32768, 4, 10, 22, 2)])
def test_large_n_two_launch_steps_up_to_their_line(slz, N, l, beta, last, lanes):
    import ctypes
    n, batch = 3, last + 1
    p = synth.CONFIGS[2].with_(name="line", N=N, n=n, pbs_level=l, pbs_base_log=beta, msg_bits=3, batch=batch)
    bsk = synth.raw_words(p, "raw_bsk", n * 4 * l * N).reshape(n, 2, l, 2, N)
    d_luts = slz.to_device_u64(synth.raw_words(p, "misc", N).reshape(1, N))
    d_in = slz.to_device_u64(synth.raw_words(p, "raw_ct", batch * (n + 1)).reshape(batch, n + 1))
    ctx = slz.Context(p, batch)
    d_key = ctx.bsk_prepare(slz.to_device_u64(bsk))
    ctx.set_option(slz.SLZ_OPT_FORCE_GENERIC, 1)
    want = ctx.pbs_batch(d_in, d_luts, None, d_key)
    ctx.set_option(slz.SLZ_OPT_FORCE_GENERIC, 0)
    past = 2 if batch > 512 // (N // 1024) else 1                      # lanes of the three-launch steps
    for count, kernels in ((last, lanes * (2 * n + 1)), (last + 1, past * 3 * n)):
        out = torch.empty((count, N + 1), dtype=torch.int64, device="cuda")
        ctx.pbs_batch(d_in[:count], d_luts, None, d_key, out=out)
        assert torch.equal(out, want[:count]), count
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            ctx.pbs_batch(d_in[:count], d_luts, None, d_key, out=out)
        nodes = ctypes.c_size_t(0)
        assert slz.lib().hipGraphGetNodes(ctypes.c_void_p(int(graph.raw_cuda_graph())), None, ctypes.byref(nodes)) == 0
        assert nodes.value == kernels + 2, count


# N = 32768 with two levels, by the kernels of a captured call: the one launch (behind a kernel that clears its words) up to 16, 22 to 24 and 31 to 40, the
# two-launch steps between on two lanes, three launches past it
def test_large_n_one_launch_and_two_launch_steps_take_turns(slz):
    import ctypes
    N, l, n, batch = 32768, 2, 3, 41
    p = synth.CONFIGS[2].with_(name="turns", N=N, n=n, pbs_level=l, pbs_base_log=15, msg_bits=3, batch=batch)
    d_key = synth.raw_words(p, "raw_bsk", n * 4 * l * N).reshape(n, 2, l, 2, N)
    d_luts = slz.to_device_u64(synth.raw_words(p, "misc", N).reshape(1, N))
    d_in = slz.to_device_u64(synth.raw_words(p, "raw_ct", batch * (n + 1)).reshape(batch, n + 1))
    ctx = slz.Context(p, batch)
    d_key = ctx.bsk_prepare(slz.to_device_u64(d_key))
    want = ctx.pbs_batch(d_in, d_luts, None, d_key)
    one, two, three = 2, 2 * (2 * n + 1), 2 * 3 * n
    for count, kernels in ((16, one), (17, two), (21, two), (22, one), (24, one), (25, two), (30, two), (31, one), (40, one), (41, three)):
        out = torch.empty((count, N + 1), dtype=torch.int64, device="cuda")
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            ctx.pbs_batch(d_in[:count], d_luts, None, d_key, out=out)
        nodes = ctypes.c_size_t(0)
        assert slz.lib().hipGraphGetNodes(ctypes.c_void_p(int(graph.raw_cuda_graph())), None, ctypes.byref(nodes)) == 0
        assert nodes.value == kernels + 2, count
        graph.instantiate()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[:count]), count
