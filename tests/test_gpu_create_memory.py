"""hdg_create's host memory: the tables of a large mesh are held once."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rss():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * 4096


def test_tables_are_not_copied_on_the_host():
    from paper_2608_27863_amd import hdg, synth
    mesh = synth.box_mesh((22, 20, 20), p=4)
    wl = synth.make_state(synth.box_mesh((2, 2, 2), p=1), lambda x: synth.tgv_state(x, 1.25), mach=1.25)
    hdg.Context(synth.box_mesh((2, 2, 2), p=1), wl)  # the library and the device are loaded
    # geometry at the quadrature points, the largest tables: 10 values at 6^3 points and 4 at 6^2 of each face
    tables = mesh.n_elem * 8 * (10 * 216 + 6 * 4 * 36)
    print(f"[create] {mesh.n_elem} elements at p=4, {tables / 2**20:.0f} MiB of geometry", flush=True)
    start, peak, stop = _rss(), [0], threading.Event()

    def sample():
        while not stop.wait(0.0005):
            peak[0] = max(peak[0], _rss())

    t = threading.Thread(target=sample)
    t.start()
    ctx = hdg.Context(mesh, wl)
    stop.set()
    t.join()
    grown = peak[0] - start
    print(f"  grown by {grown / 2**20:.0f} MiB at most", flush=True)
    assert ctx.n_elem == mesh.n_elem
    assert 0.5 * tables < grown < 1.75 * tables
