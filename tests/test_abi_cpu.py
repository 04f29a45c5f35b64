"""Host-only checks of the C-ABI library (no GPU): it loads, exports every symbol the header declares,
its pure host function slz_lut_encode agrees with the oracle, and argument errors are reported."""
import ctypes
import decimal
import os
import re

import numpy as np
import pytest

import synth
import paper_2504_17785_amd as slz

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_loads_and_exports_header_symbols():
    L = slz.lib()
    header = "".join(open(os.path.join(ROOT, "include", h)).read() for h in sorted(os.listdir(os.path.join(ROOT, "include"))))
    declared = set(re.findall(r"\b(slz_[a-z_0-9]+)\s*\(", header))
    declared -= {"slz_params", "slz_ctx", "slz_matmul_rns_shape", "slz_rns_shape", "slz_shift_shape"}
    assert {"slz_pbs_batch", "slz_keyswitch_batch", "slz_lut_encode"} <= declared
    for name in sorted(declared):
        assert hasattr(L, name), name
    assert declared == set(slz.EXPORTS)


@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5])
def test_lut_encode_matches_oracle(orc, cfg):
    p = synth.CONFIGS[cfg]
    tables = synth.config_tables(cfg)
    assert np.array_equal(slz.lut_encode(p, tables), orc.lut_encode(p, tables))


def test_lut_encode_small_shapes_match_oracle(orc):
    for N, bits in [(8, 1), (8, 2), (64, 5), (32, 3), (1024, 9)]:
        p = synth.CONFIGS[1].with_(N=N, msg_bits=bits)
        tables = synth.random_tables(p, 3)
        assert np.array_equal(slz.lut_encode(p, tables), orc.lut_encode(p, tables))


def test_lut_encode_rejects_bad_arguments():
    L = slz.lib()
    p = synth.CONFIGS[1]
    cp = slz.make_params(p)
    tab = np.zeros(p.t, dtype=np.uint64)
    out = np.zeros(p.N, dtype=np.uint64)
    assert L.slz_lut_encode(ctypes.byref(cp), None, 1, out.ctypes.data) == -1
    assert L.slz_lut_encode(ctypes.byref(cp), tab.ctypes.data, 0, out.ctypes.data) == -1
    assert L.slz_lut_encode(None, tab.ctypes.data, 1, out.ctypes.data) == -1
    tab[3] = p.t                                           # entry out of range
    assert L.slz_lut_encode(ctypes.byref(cp), tab.ctypes.data, 1, out.ctypes.data) == -1
    small = slz.make_params(p.with_(N=8, msg_bits=3))      # N < 2t
    assert L.slz_lut_encode(ctypes.byref(small), tab.ctypes.data, 1, out.ctypes.data) == -1
    bad = slz.make_params(p.with_(N=500))                  # not a power of two
    assert L.slz_lut_encode(ctypes.byref(bad), tab.ctypes.data, 1, out.ctypes.data) == -1
    assert L.slz_strerror(-1) == b"invalid argument"
    assert L.slz_strerror(0) == b"success"


def test_null_context_calls_are_errors_not_crashes():
    L = slz.lib()
    assert L.slz_ctx_destroy(None) == -1
    assert L.slz_ctx_set_option(None, 1, 1) == -1
    assert L.slz_pbs_batch(None, None, None, None, 0, None, None, 0, None) == -1
    assert L.slz_keyswitch_batch(None, None, None, None, 0, None) == -1
    assert L.slz_blind_rotate_batch(None, None, None, None, 0, None, 0, None, 0, None) == -1
    assert L.slz_lwe_lincomb_batch(None, None, None, None, 0, 0, 0, None) == -1
    need = ctypes.c_size_t(0)
    assert L.slz_bsk_prepare(None, None, None, ctypes.byref(need), None) == -1
    assert L.slz_ksk_prepare(None, None, None, ctypes.byref(need), None) == -1
    assert L.slz_keyswitch_batch_prepared(None, None, None, None, 0, None) == -1
    assert L.slz_keyswitch_batch_static(None, None, None, None, 0, None) == -1
    out = ctypes.c_void_p()
    assert L.slz_ctx_create(None, 1, ctypes.byref(out)) == -1


def test_bench_refuses_more_than_one_gpu():
    # one GPU per box: the bench says so instead of launching anything (no GPU is touched before the check)
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=300)
    assert r.returncode != 0
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


def test_matmul_rns_luts_match_oracle_tables(orc):
    from oracle import gadgets
    p = synth.Params(name="t", n=4, k=1, N=2048, pbs_base_log=23, pbs_level=1, ks_base_log=4, ks_level=8, msg_bits=8,
                     sigma_lwe=2.0 ** -40, sigma_bsk=2.0 ** -50, batch=1, n_luts=1, seed=1)
    for m in gadgets.RNS_BASES.values():
        want = orc.lut_encode(p, np.concatenate(gadgets.lookup_tables(p, m)))
        assert np.array_equal(slz.matmul_rns_luts(p, m, 2, 3, 4), want)
    with pytest.raises(slz.SlzError):
        slz.matmul_rns_luts(p, (17, 3), 1, 1, 1)           # not a 4-bit modulus
    with pytest.raises(slz.SlzError):
        slz.matmul_rns_luts(p.with_(msg_bits=4), (7, 8), 1, 1, 1)
    with pytest.raises(slz.SlzError):
        slz.matmul_rns_luts(p, (7, 8), 0, 1, 1)


def test_rns_luts_match_oracle_tables(orc):
    from oracle import gadgets
    p = synth.Params(name="t", n=4, k=1, N=2048, pbs_base_log=23, pbs_level=1, ks_base_log=4, ks_level=8, msg_bits=8,
                     sigma_lwe=2.0 ** -40, sigma_bsk=2.0 ** -50, batch=1, n_luts=1, seed=1)
    for m in list(gadgets.RNS_BASES.values()) + [(5, 7, 8)]:
        for nzp in ((-1, 0, 1), (-1, 1, 1), (3, 0, -128)):
            want = orc.lut_encode(p, np.concatenate([gadgets.rns2mrns_tables(p, m), gadgets.sign_tables(p, m, *nzp)]))
            assert np.array_equal(slz.rns_luts(p, m, *nzp), want)
    with pytest.raises(slz.SlzError):
        slz.rns_luts(p, (6, 15, 14))                       # not pairwise coprime
    with pytest.raises(slz.SlzError):
        slz.rns_luts(p, (15, 14), 200, 0, 1)               # result out of the signed byte range
    with pytest.raises(slz.SlzError):
        slz.rns_luts(p.with_(msg_bits=5), (15, 14))


def test_shift2msbs_luts_match_oracle_tables(orc):
    from oracle import gadgets
    p = synth.Params(name="t", n=4, k=1, N=2048, pbs_base_log=23, pbs_level=1, ks_base_log=4, ks_level=8, msg_bits=8,
                     sigma_lwe=2.0 ** -40, sigma_bsk=2.0 ** -50, batch=1, n_luts=1, seed=1)
    for m in gadgets.RNS_BASES.values():
        for gamma in (1, 5, 7):
            want = orc.lut_encode(p, np.concatenate([gadgets.rns2mrns_tables(p, m), gadgets.sign_tables(p, m, 1, 0, 0),
                                                     gadgets.shift_tables(p, m, 4, gamma), gadgets.pm_tables(p, m)]))
            assert np.array_equal(slz.shift2msbs_luts(p, m, 4, gamma), want)
    with pytest.raises(slz.SlzError):
        slz.shift2msbs_luts(p, (15, 14), 5, 5)            # only 4-bit digits
    with pytest.raises(slz.SlzError):
        slz.shift2msbs_luts(p, (15, 14), 4, 8)            # the output must fit 7 bits


def test_loss_and_weight_update_luts_match_oracle_tables(orc):
    from oracle import loss
    base = dict(n=4, k=1, N=2048, pbs_base_log=23, pbs_level=1, ks_base_log=4, ks_level=8, sigma_lwe=2.0 ** -40, sigma_bsk=2.0 ** -50,
                batch=1, n_luts=1, seed=1)
    for bits, cases in ((8, ((7, 7, 2), (2, 7, 2), (16, 7, 1), (3, 4, 2), (5, 8, 2))), (9, ((3, 7, 3), (2, 9, 2))), (6, ((3, 5, 1),))):
        p = synth.Params(name="t", msg_bits=bits, **base)
        for b, Gamma, kappa in cases:
            assert np.array_equal(slz.loss_luts(p, b, Gamma, kappa), orc.lut_encode(p, loss.loss_tables(p, b, Gamma, kappa)))
        for alpha in range(2, bits - 1):
            assert np.array_equal(slz.weight_update_luts(p, alpha), orc.lut_encode(p, loss.weight_update_table(p, alpha)))
        with pytest.raises(slz.SlzError):
            slz.weight_update_luts(p, bits - 1)
    p = synth.Params(name="t", msg_bits=8, **base)
    for bad in ((3, 7, 4), (17, 7, 1), (3, 9, 2), (3, 1, 2), (3, 7, 0)):       # too wide, too many classes, Gamma out of range, kappa 0
        with pytest.raises(slz.SlzError):
            slz.loss_luts(p, *bad)


def test_matmul_highres_luts_match_oracle_tables(orc):
    from oracle import gadgets
    p = synth.Params(name="t", n=4, k=1, N=2048, pbs_base_log=23, pbs_level=1, ks_base_log=4, ks_level=8, msg_bits=8,
                     sigma_lwe=2.0 ** -40, sigma_bsk=2.0 ** -50, batch=1, n_luts=1, seed=1)
    for m in gadgets.RNS_BASES_5BIT.values():
        assert np.array_equal(slz.matmul_highres_luts(p, m, 1, 1, 1), orc.lut_encode(p, gadgets.highres_tables(p, m)))
    with pytest.raises(slz.SlzError):
        slz.matmul_highres_luts(p, (33, 31), 1, 1, 1)               # moduli are at most 5 bits wide
    with pytest.raises(slz.SlzError):
        slz.matmul_highres_luts(p.with_(msg_bits=7), (31, 30), 1, 1, 1)


def test_headers_are_plain_c():
    """The boundary is a C ABI: both headers must compile as C99 on their own."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include")
    for h in ("silenzio_pbs.h", "silenzio_gadgets.h"):
        r = subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-fsyntax-only", "-x", "c", os.path.join(inc, h)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr


def test_transform_error_bound_and_the_bases_it_admits():
    # internal host functions, by their mangled names.  The sum is written out again: rounding of the layers (a radix-4 layer 2 for the
    # product, sqrt(1/2) for its twiddle, 2 for two additions; a radix-2 layer 4), of the products (one per fused multiply-add, the
    # partial results of a row counted as often as they are rounded), of the key spectrum, of the inverse's stages and the constant
    # sqrt(1/2) in two of them, and for every table
    # twiddle what its computation in long double leaves, 26 * 2^-64 of angle, functions and second rounding.
    L = slz.lib()
    bound, supported = L._Z19slz_fft_error_boundjjj, L._Z17slz_fft_supportedPK10slz_params
    bound.argtypes, bound.restype = [ctypes.c_uint32] * 3, ctypes.c_double
    table = 26 * 2.0 ** -11
    half = 0.5 ** 0.5                                                 # as a double; its relative error in units of 2^-53:
    root = decimal.Context(prec=40).sqrt(decimal.Decimal("0.5"))
    constant = float(abs(decimal.Decimal(half) / root - 1)) * 2.0 ** 53
    shapes = {(2048, 1): (23, 5, 13, 5 * (4 + half + table) + 3 + 1.05 + 2 + (2 + constant) + 7 * (4 + table) + 1 + constant),
              (1024, 1): (23, 5, 13, 9 * (4 + table) + 3 + 1.05 + 2 + (2 + constant) + 6 * (4 + table) + 1 + constant),
              (512, 2): (14, 3, 22, 8 * (4 + table) + 5 + 1.05 + 2 + 6 * (4 + table) + 1 + constant)}
    # N = 2048 with eight waves per ciphertext: half-sizes 4 and 8 are one radix-4 layer (the same terms as forward); it rounds less, so the
    # bound is that of the other kernel
    team = 5 * (4 + half + table) + 3 + 1.05 + 2 + (4 + half + table) + 6 * (4 + table) + 1 + constant
    assert shapes[2048, 1][3] - 2 < team < shapes[2048, 1][3]
    for (N, level), (top, pieces, bits, units) in shapes.items():
        assert pieces * bits >= 64                                    # the pieces make up a key word
        rows = 2 * level
        for beta in range(1, top + 2):
            want = units * 2.0 ** -53 * rows * N * 2.0 ** (beta - 1) * 2.0 ** (bits - 1)
            got = bound(N, rows, beta)
            assert want <= got <= 1.01 * want, (N, beta)
            assert bool(supported(ctypes.byref(slz.make_params(synth.CONFIGS[2].with_(N=N, pbs_level=level, pbs_base_log=beta))))) == \
                (got < 0.499) == (beta <= top), (N, beta)
    for kw in (dict(N=2048, pbs_level=2), dict(N=1024, pbs_level=2), dict(N=512, pbs_level=1), dict(N=4096), dict(N=1024, k=2), dict(N=256)):
        q = synth.CONFIGS[2].with_(pbs_base_log=kw.pop("beta", 8), **kw)
        assert not supported(ctypes.byref(slz.make_params(q))), kw


def test_transform_error_bound_of_n4096():
    # N = 4096: forward a radix-2 layer on integers with the constant sqrt(1/2), radix 4, radix 8 twice (product, two additions, an addition
    # whose odd part is a sum times the constant), radix 4; inverse 1, 2, 4, then radix 4 and radix 2 twice, 512, 1024 and the turn
    L = slz.lib()
    bound, supported = L._Z19slz_fft_error_boundjjj, L._Z21slz_fft4096_supportedPK10slz_params
    bound.argtypes, bound.restype = [ctypes.c_uint32] * 3, ctypes.c_double
    table, half = 26 * 2.0 ** -11, 0.5 ** 0.5
    root = decimal.Context(prec=40).sqrt(decimal.Decimal("0.5"))
    constant = float(abs(decimal.Decimal(half) / root - 1)) * 2.0 ** 53
    radix4, radix8, radix2 = 4 + half + table, 2 + half + table + 2 + 2 + constant, 4 + table
    units = 1 + constant + 2 * radix4 + 2 * radix8 + 3 + 1.05 + 2 + (2 + constant) + 2 * (radix4 + radix2) + 2 * radix2 + 1 + constant
    for beta in range(1, 24):
        want = units * 2.0 ** -53 * 2 * 4096 * 2.0 ** (beta - 1) * 2.0 ** 12
        assert want <= bound(4096, 2, beta) <= 1.01 * want, beta
        q = synth.CONFIGS[2].with_(N=4096, pbs_base_log=beta)
        assert bool(supported(ctypes.byref(slz.make_params(q)))) == (want < 0.499) == (beta <= 22), beta
    for kw in (dict(N=4096, pbs_level=2), dict(N=4096, k=2), dict(N=2048), dict(N=8192)):
        assert not supported(ctypes.byref(slz.make_params(synth.CONFIGS[2].with_(pbs_base_log=8, **kw)))), kw


@pytest.mark.parametrize("G,half", [(2, 512), (4, 256), (8, 128), (16, 64), (32, 32)])
def test_large_n_lanes_are_cut_where_it_wins_and_keep_the_order_of_the_row_pass(G, half):
    # an internal host function, by its mangled name: ciphertexts of the first lane for a batch past half / 2, 0: not even
    f = slz.lib()._Z28slz_bign_first_of_even_lanesjjj
    f.argtypes, f.restype = [ctypes.c_uint32] * 3, ctypes.c_uint32
    assert not any(f(G, b, half) for b in range(1, 512 // G + 1)) and half // 2 == 512 // G
    unit = 16 // G if G in (4, 8) else 1                    # what the XCD-aware order takes: batch * 2 G a multiple of 32
    got = {b: f(G, b, half) for b in range(half // 2 + 1, 2 * half + 8)}
    for b, first in got.items():
        if first:
            rest = b - first
            assert b <= 2 * half and rest % unit == 0 and rest <= first < rest + 2 * unit
            assert first % unit == 0 or b % unit            # both lanes in that order where the batch allows it
            assert (b + first - 1) // first <= 2            # the two lanes take everything in one round
    last = half + half // (8 if G == 2 else 4)              # measured: a full lane and the rest are faster past this ...
    assert all(got[b] for b in got if b <= last)
    if G < 16:
        again = {8: half + half * 5 // 8}.get(G, 2 * half + 1)
        assert not any(got[b] for b in range(last + 1, again))
        assert all(got[b] for b in range(again, 2 * half + 1))
    else:                                                   # ... and never here
        assert all(got[b] for b in got if b <= 2 * half)
    assert not any(got[b] for b in got if b > 2 * half)


def test_large_n_two_launch_steps_end_where_they_stop_winning():
    # by G = N / 1024 and levels; a step of more levels has fewer and larger workgroups, which stop winning earlier
    f = slz.lib()._Z26slz_bign_latency_max_batchjj
    f.argtypes, f.restype = [ctypes.c_uint32] * 2, ctypes.c_uint32
    want = {1: {8: 96, 16: 49, 32: 32}, 2: {2: 256, 4: 128, 8: 96, 16: 56, 32: 32}, 3: {2: 128, 4: 64, 8: 32, 16: 40, 32: 22},
            4: {2: 192, 4: 96, 8: 48, 16: 40, 32: 22}}
    assert {l: {G: f(G, l) for G in row} for l, row in want.items()} == want


def test_large_n_one_launch_is_taken_where_it_wins():
    # rounds of eight ciphertexts: the first two, and the fuller part of the next three
    f = slz.lib()._Z18slz_bign_xcd_takesjjj
    f.argtypes, f.restype = [ctypes.c_uint32] * 3, ctypes.c_uint32
    assert [b for b in range(1, 300) if f(32, 2, b)] == list(range(1, 17)) + list(range(22, 25)) + list(range(31, 41))
    assert not any(f(G, l, b) for G in (2, 4, 8, 16, 32, 64) for l in (1, 2, 3, 4) for b in range(1, 65) if (G, l) != (32, 2))


def test_n4096_pairs_take_as_many_steps_as_win_back_their_launches():
    f = slz.lib()._Z22slz_fft4096_pair_stepsj
    f.argtypes, f.restype = [ctypes.c_uint32], ctypes.c_uint32
    assert [f(b) for b in (1, 64, 65, 100, 101, 128)] == [8, 8, 32, 32, 64, 64]


def test_keyswitch_takes_ranges_where_they_win():
    # (words, n, levels): groups of 256 ciphertexts up to 20 with the standard and with the prepared key; segments win by 4 to 13 % at the groups left out
    # up to the limits of 8 and 16, and by 15 to 30 % past the latter
    f = slz.lib()._Z20slz_ksm_takes_rangesPK10slz_paramsji
    f.argtypes, f.restype = [ctypes.POINTER(slz.SlzParams), ctypes.c_uint32, ctypes.c_int], ctypes.c_int
    to8, to16 = list(range(1, 9)), list(range(1, 17))
    want = {(2048, 742, 5): (to8, to16), (1024, 630, 5): (to8, to16), (2048, 300, 3): (to8[1:], to16[1:]), (512, 500, 4): (to8[2:], to16[2:]),
            (256, 128, 2): ([], []), (4096, 800, 5): (to8, to16[:10] + [14, 15, 16]), (8192, 900, 4): (to8, to16[:10] + [14, 15, 16]),
            (32768, 1024, 5): ([], to16[:6] + [8, 16])}
    for (kN, n, l), groups in want.items():
        cp = slz.make_params(synth.CONFIGS[2].with_(N=kN, n=n, k=1, ks_base_log=4, ks_level=l))
        got = tuple([g for g in range(1, 21) if f(ctypes.byref(cp), 256 * g, prepared)] for prepared in (0, 1))
        assert got == groups, (kN, n, l)
        assert all(f(ctypes.byref(cp), 256 * g - 255, q) == f(ctypes.byref(cp), 256 * g, q) for g in range(1, 21) for q in (0, 1))


def test_bench_counts_the_key_form_and_the_operations_of_the_path_that_runs():
    import sys
    sys.path.insert(0, ROOT)
    import bench
    p = synth.CONFIGS[2]
    residue, transform = 742 * 2 * 4 * 2048 * 8, 742 * 5 * 2 * 8 * 4 * 64 * 16          # 97 and 243 MB
    assert bench.residue_key_bytes(p) == residue
    assert bench.key_bytes_read(p, residue + transform) == (transform, True)
    assert bench.key_bytes_read(p, residue + transform, generic=True) == (residue, False)
    assert bench.key_bytes_read(p, residue) == (residue, False)
    assert bench.alu_model_ops_per_pbs(p, True) == 742 * 550912.0
    assert bench.alu_model_ops_per_pbs(p, False) == bench.alu_model_ops_per_pbs(p) > 1.8 * 742 * 550912.0
    # what changes the traffic of a kernel is in the hash of its sources: the header holds the piece count and the key's step size
    for path in ("fused_n2048", "fused_n512"):
        assert "slz_fft.h" in bench.PATH_SOURCES[path]


def test_stored_traffic_figures_belong_to_the_current_kernel_sources():
    # bench.py reports a stored FETCH_SIZE / WRITE_SIZE figure only when the kernel's sources still hash to the value recorded
    # with it; a line that has gone stale is dropped silently there, so it is caught here
    import os
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    sys.path.insert(0, root)
    import bench
    rows = [l.split() for l in open(os.path.join(root, "profiles", "hbm_traffic.txt")) if l.strip() and not l.startswith("#")]
    assert len(rows) >= 3
    for path, workload, fetch, write, commit, digest in rows:
        assert bench.kernel_source_hash(path) == digest, "%s %s: re-measure and update profiles/hbm_traffic.txt" % (path, workload)
        assert bench.stored_traffic(path, workload) == float(fetch) + float(write)
