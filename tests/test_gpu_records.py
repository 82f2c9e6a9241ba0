"""Records that the device hands to the host from several threads, each with its
lattice and stream: every call gets its own."""
import threading

import pytest

pytestmark = pytest.mark.gpu

from paper_2409_02964_amd import workloads as W  # noqa: E402

RATES = dict(s_c=1.2, s_e=1.2, s_eps=1.2, s_q=1.2, s_nu=0.8)


def test_records_of_several_threads():
    import torch
    from paper_2409_02964_amd.vanse import Lattice, VanseError
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, reps = 12, 40
    lats, phis, streams = [], [], [torch.cuda.Stream() for _ in range(n)]
    for k in range(n):
        nx, ny = 40 + 7 * k, 33 + 5 * k
        phis.append(torch.from_numpy(W.channel_phi(nx, ny, seed=k, noise=0.05)).cuda())
        lat = Lattice(nx, ny, precision=["f64", "f32", "f32s", "f16s"][k % 4]).set_params(0.5, RATES)
        lats.append(lat.set_void_fraction(phis[k]).set_populations(W.random_populations(nx, ny, seed=k)).step(3))
    wrong = [p.clone() for p in phis]
    for p in wrong:
        p[2, 3] = 1.5
    want = [lat.observe() for lat in lats]
    assert len({w["mass"] for w in want}) == n
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(streams[k]):
                for r in range(reps):
                    assert lats[k].observe() == want[k]
                    lats[k].set_void_fraction(phis[k])
                    if r % 8 == k % 8:
                        with pytest.raises(VanseError, match="1 void-fraction values"):
                            lats[k].set_void_fraction(wrong[k])
                    assert lats[k].residual()[1] == want[k]["u2"]
        except BaseException as e:  # noqa: BLE001
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
