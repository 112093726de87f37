"""The walk's launch plan (CPU): launch shape, tally path and workspace for any
size, without a launch."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2507_23189_amd import _capi as K
from paper_2507_23189_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
CU_LDS, GRANULE = 160 * 1024, 1280     # LDS is handed out in granules


class Request(C.Structure):
    _fields_ = [("batch", C.c_bool), ("phase", C.c_int), ("n_cdf", C.c_int), ("n_inst", C.c_uint32), ("n_pix", C.c_uint64),
                ("flags", C.c_uint32), ("photons", C.c_uint64), ("path_photons", C.c_uint64), ("block_size", C.c_int), ("grid_blocks", C.c_int),
                ("chunk", C.c_uint32), ("tau_z", C.c_double), ("cus", C.c_int), ("max_copies", C.c_uint64),
                ("ws_bytes", C.c_uint64)]


class Plan(C.Structure):
    _fields_ = [("use_log", C.c_bool), ("block", C.c_int), ("grid", C.c_int), ("cache_bits", C.c_int), ("lds", C.c_size_t),
                ("bits", C.c_uint32), ("rbits", C.c_uint32), ("parts", C.c_uint32), ("copies", C.c_uint64),
                ("n_cleared", C.c_uint64), ("permuted", C.c_bool), ("ws_words", C.c_uint64), ("log_at", C.c_uint64),
                ("log_cap", C.c_uint32), ("chunk", C.c_uint64), ("refill_min", C.c_uint32)]

    @property
    def path(self):
        """What decides which kernels run on which memory, launch shape apart."""
        return (self.use_log, self.copies, self.n_cleared, self.permuted, self.cache_bits, self.log_at)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{B.INCLUDE}", f"-I{B.CSRC}",
                    os.path.join(HERE, "walk_plan_driver.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    lib.words.restype = C.c_uint64
    lib.words.argtypes = [C.POINTER(K.Detector), C.c_uint64]
    assert lib.walk_plan_sizes(0) == C.sizeof(Request) and lib.walk_plan_sizes(1) == C.sizeof(Plan)
    return lib


def plan(lib, photons, shape=(512, 512, 512, 512), *, media=0, flags=0, n_cdf=16384, tau=4.0, log_photons=None, **kw):
    """The plan of a walk (or, with media, of a batch) in a workspace of the size
    the library asks for."""
    det = K.Detector(*shape, flags)
    n = max(media, 1)
    if flags & K.MC_EXIT_LOG:
        size = photons if log_photons is None else log_photons
        ws = K.mc_workspace_bytes_batch_log(det, media, size) if media else K.mc_workspace_bytes_log(det, size)
    else:
        ws = K.mc_workspace_bytes_batch(det, media) if media else K.mc_workspace_bytes(det)
    q = dict(batch=bool(media), phase=K.MC_PHASE_MIE, n_cdf=n_cdf, n_inst=n, n_pix=shape[0] * shape[1] + shape[2] * shape[3],
             flags=flags, photons=photons, path_photons=photons, tau_z=-1.0 if media else tau, cus=256, max_copies=8, ws_bytes=ws)
    q.update(kw)
    p = Plan()
    lib.walk_plan(C.byref(Request(**q)), C.byref(p))
    return p


def test_the_headline_plan(lib):
    p = plan(lib, 100_000_000, flags=K.MC_EXIT_LOG)
    assert p.use_log and (p.block, p.grid) == (1024, 512) and p.lds <= CU_LDS // 2
    # Every region holds half as many exits again as an even share of the photons.
    assert p.log_cap * (1 << p.rbits) * p.grid >= 150_000_000
    assert not plan(lib, 100_000_000).use_log and plan(lib, 100_000_000).copies == 8


@pytest.mark.parametrize("px", [16, 64, 100, 150], ids=str)
@pytest.mark.parametrize("log", [False, True], ids=["", "log"])
def test_every_batch_has_the_blocks_its_tallies_leave_room_for(lib, px, log):
    """A batch's block needs 16 scalar words a medium, 16 queues of 1 KB and, with the
    log, its append counters: two fill a CU up to half its LDS, to the byte (512
    media, or 384, 448 and 480 with 2^12, 2^11 and 2^10 counters)."""
    for media in range(1, 513):
        p = plan(lib, 10_000_000, (px,) * 4, media=media, flags=K.MC_EXIT_LOG if log else 0, n_cdf=0, grid_blocks=0)
        need = 128 * media + 16 * 1024 + ((4 << p.rbits) if p.use_log else 0)
        assert p.grid == 256 * (2 if need <= CU_LDS // 2 else 1), (media, p.lds)
        assert p.lds >= need


@pytest.mark.parametrize("sigma", [False, True], ids=["", "sigma"])
def test_the_cache_under_the_log_costs_no_block(lib, sigma):
    """It takes only LDS that no further block could have, in whole granules."""
    flags = K.MC_EXIT_LOG | (K.MC_SIGMA if sigma else 0)
    cached = 0
    for block in range(64, 1025, 64):
        for n_cdf in (0, 2, 1000, 1024, 2048, 4096, 5000, 8192, 12345, 16384):
            p = plan(lib, 100_000_000, flags=flags, n_cdf=n_cdf, block_size=block)
            waves = block // 64
            fixed = 4 * ((n_cdf + 3) & ~3) + 160 + 768 * waves + (4 << p.rbits)
            assert p.use_log and p.lds == fixed + ((20 if sigma else 12) << p.cache_bits if p.cache_bits else 0)
            fits = lambda lds: max(1, min(CU_LDS // GRANULE // -(-lds // GRANULE), 32 // waves))
            assert fits(p.lds) == fits(fixed), (block, n_cdf, p.lds)
            assert p.grid == 256 * max(1, min(CU_LDS // fixed, 32 // waves))
            cached += p.cache_bits > 0
    assert cached > 50


def _room(p, photons):
    """Entries of the log for each photon."""
    return (p.log_cap << p.rbits) * p.grid / photons


@pytest.mark.parametrize("sigma", [False, True], ids=["", "sigma"])
def test_a_log_beside_the_copies_where_it_pays(lib, sigma):
    """Without the flag: with room for three exits of five; where the log's counters
    cost the second block of every CU, and no squares are tallied, for nine of ten."""
    flags = K.MC_SIGMA if sigma else 0
    seen = set()
    for media in (64, 256, 384, 385, 450, 480, 481, 511, 512):
        for px in (40, 64, 91, 100, 113, 128, 150, 207, 256):
            for each in (20_000, 60_000, 200_000, 400_000):
                n = media * each
                p = plan(lib, n, (px,) * 4, media=media, flags=flags, n_cdf=0)
                two = 128 * media + 16 * 1024 <= CU_LDS // 2
                log_two = 128 * media + 16 * 1024 + (4 << p.rbits) <= CU_LDS // 2
                least = 0.9 if two and not log_two and not sigma else 0.6
                if p.use_log:
                    assert n > max(1 << 21, p.ws_words // 8 // (2 if sigma else 1) - 32 * media)
                    assert _room(p, n) >= least, (media, px, each)
                    assert p.grid == 256 * (2 if log_two else 1)
                    assert p.log_at + ((p.grid << p.rbits) + 1) // 2 + (p.log_cap << p.rbits) * p.grid <= p.ws_words
                else:
                    assert p.grid == 256 * (2 if two else 1)
                seen.add((p.use_log, least))
    assert seen == {(True, 0.6), (False, 0.6)} | (set() if sigma else {(True, 0.9), (False, 0.9)})


@pytest.mark.parametrize("flags", [0, K.MC_EXIT_LOG, K.MC_SIGMA, K.MC_EXIT_LOG | K.MC_SIGMA], ids=["", "log", "sigma", "log-sigma"])
def test_a_sample_takes_the_path_of_its_launch(lib, flags):
    """The tuner's sample, a sixteenth of the photons: the log, the copies and their
    order are those of the launch it is timed for, at every block size it tries."""
    for media in (2, 32, 256, 500):
        for px in (16, 64, 150, 256):
            for each in (2_000, 20_000, 200_000, 2_000_000):
                n = media * each
                for block in K.AUTOTUNE_BLOCKS:
                    kw = dict(media=media, flags=flags, n_cdf=0, block_size=block, log_photons=n)
                    whole = plan(lib, n, (px,) * 4, **kw)
                    sample = plan(lib, n // 16, (px,) * 4, path_photons=n, **kw)
                    assert sample.path == whole.path and (sample.grid, sample.lds) == (whole.grid, whole.lds)
                    assert (sample.log_cap, sample.rbits) == (whole.log_cap, whole.rbits)


@pytest.mark.parametrize("moments", [False, True], ids=["", "moments"])
def test_the_library_block_set_by_the_caller(lib, moments):
    """A caller who sets the block that the library takes gets the library's plan."""
    for log in (0, K.MC_EXIT_LOG):
        for n in (10_000, 300_000, 1_000_000, 3_000_000, 10_000_000, 50_000_000, 200_000_000):
            for px in (32, 128, 200, 512):
                for tau in (0.5, 4.0, 16.0):
                    kw = dict(flags=log | (K.MC_MOMENTS if moments else 0), tau=tau)
                    a, b = (plan(lib, n, (px,) * 4, block_size=block, **kw) for block in (0, 768 if moments else 1024))
                    assert bytes(a) == bytes(b), (n, px, tau)


@pytest.mark.parametrize("photons, pixels, bits", [
    (1 << 20, 64, 8), ((1 << 20) + 1, 1024, 10), ((1 << 23) - 1, 1 << 18, 10),
    (1 << 23, 1 << 16, 10), (1 << 23, (1 << 16) + 2, 11), ((1 << 24) - 1, 1 << 16, 10), ((1 << 24) - 1, 1 << 19, 11),
    (1 << 24, 1 << 13, 10), (1 << 24, (1 << 13) + 2, 11), ((1 << 25) - 1, 1 << 18, 11), ((1 << 25) - 1, (1 << 18) + 2, 12), (1 << 25, 1 << 13, 10),
    (1 << 25, 1 << 15, 11), (1 << 25, (1 << 15) + 2, 12), (1 << 30, 1 << 13, 10)], ids=str)
def test_slots_by_photons_and_pixels(lib, photons, pixels, bits):
    shape = (pixels // 2, 1, 1, pixels - pixels // 2)
    p = plan(lib, photons, shape, n_cdf=0)
    assert not p.use_log and p.cache_bits == bits
    assert plan(lib, photons, shape, n_cdf=16384).cache_bits == min(bits, 8)    # what the LDS beside the table holds


def test_the_countdown_to_the_next_look_never_wraps(lib):
    """A wave whose photons may always meet roulette, for as many rounds as a walk of
    2^31 photons by one wave could have."""
    most = 1 << 24          # steps between two rounds: a photon takes no more
    calm = 0
    for _ in range(1000):
        calm -= most
        assert calm >= -(1 << 31)
        calm = lib.calm(calm, 0)
        assert calm == 0    # (no look is skipped for it)
    assert lib.calm(17, 0) == 17 and lib.calm(17, 1) == 0 and lib.calm(-3, 1) == 0
