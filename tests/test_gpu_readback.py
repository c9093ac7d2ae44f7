"""Read-back of the macroscopic fields (pond_moments): in one pinned piece, in pieces shared
by threads, and straight into the caller's arrays when another read-back has the staging.
Every value comes from the same device buffer, so all must be the same bits."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2002_09217_amd import pond, workloads as W
from tests.common import pond_config

pytestmark = pytest.mark.gpu


def lattice(nx, ny, seed, stream=None):
    case = W.perturbed(nx, ny, seed=seed)
    return pond.Lattice(pond_config(case, tile=0, stream=stream)).init_fields(case.rho, case.u, case.T)


def read(lat, wanted):
    """pond_moments with NULL for the fields not in `wanted`."""
    N = lat.cfg.N
    out = {k: np.full(2 * N if k == "u" else N, np.nan) for k in ("rho", "u", "T", "p", "E")}
    rc = pond.load().pond_moments(lat._h, *(pond._dp(v) if k in wanted else ctypes.POINTER(ctypes.c_double)()
                                            for k, v in out.items()))
    assert rc == pond.POND_OK
    return {k: v for k, v in out.items() if k in wanted}


# 6 N doubles in all (48 N bytes): the smallest lattice, just within one 2 MiB piece and just over, just
# within the 16 MiB staging and just over, several rounds of all eight pieces
@pytest.mark.parametrize("n", [(4, 4), (257, 170), (241, 183), (607, 575), (700, 501), (1500, 1401)])
def test_subsets_of_the_fields_are_the_same_bits(n):
    print(f"readback {n}", flush=True)
    with lattice(*n, seed=4) as lat:
        one = {}
        for k in ("rho", "u", "T", "p", "E"):
            one.update(read(lat, (k,)))
        for wanted in (("rho", "u", "T", "p", "E"), ("rho", "T", "E"), ("u", "T"), ()):
            got = read(lat, wanted)
            assert all(np.array_equal(got[k], one[k]) for k in wanted)
        assert all(np.isfinite(v).all() for v in one.values())


def test_pieces_on_the_per_thread_stream():
    """hipStreamPerThread (handle 2) names another stream in each helper thread: its pieces
    still hold what the caller's thread computed."""
    with lattice(1500, 1401, seed=4) as own, lattice(1500, 1401, seed=4, stream=2) as lat:
        for _ in range(3):
            ref, got = own.step(2).moments(), lat.step(2).moments()
            assert all(np.array_equal(got[k], ref[k]) for k in ref)


def test_read_backs_side_by_side():
    lats = [lattice(900, 701, seed=s) for s in (1, 2, 3)]
    alone = [lat.moments() for lat in lats]
    bad = []

    def loop(lat, ref):
        for _ in range(6):
            got = lat.moments()
            if not all(np.array_equal(got[k], ref[k]) for k in ref):
                bad.append(lat)

    threads = [threading.Thread(target=loop, args=a) for a in zip(lats, alone)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for lat in lats:
        lat.close()
    assert not bad


@pytest.mark.parametrize("where", ["page-locked", "device"])
@pytest.mark.parametrize("n", [(30, 30), (241, 183), (900, 701)])
def test_arrays_in_other_memory(n, where):
    """Page-locked arrays, and arrays on the device, hold the bits that pageable ones do."""
    torch = pytest.importorskip("torch")
    print(f"readback {n} into {where} memory", flush=True)
    with lattice(*n, seed=4) as lat:
        ref = read(lat, ("rho", "u", "T", "p", "E"))
        kw = dict(pin_memory=True) if where == "page-locked" else dict(device="cuda")
        out = {k: torch.full((v.size,), float("nan"), dtype=torch.float64, **kw) for k, v in ref.items()}
        torch.cuda.synchronize()
        dp = ctypes.POINTER(ctypes.c_double)
        assert pond.load().pond_moments(lat._h, *(ctypes.cast(v.data_ptr(), dp) for v in out.values())) == pond.POND_OK
        assert all(np.array_equal(v.cpu().numpy(), ref[k]) for k, v in out.items())
