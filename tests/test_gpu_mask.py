"""The mask read on demand (mask_kernel): exact 3x3 median, foreground count and raw labels, on the host and into
device buffers of any alignment, at widths with and without the four-pixel path, before and after a frame."""
import numpy as np
import pytest

from oracle import prost_oracle as O

pytestmark = pytest.mark.gpu


def _orth(m, k, seed):
    return np.linalg.qr(np.random.default_rng(seed).standard_normal((m, k)))[0]


@pytest.mark.parametrize("width,height", [(1, 1), (3, 1), (1, 7), (4, 1), (4, 3), (5, 4), (6, 171), (8, 128), (64, 16),
                                          (68, 61), (1023, 3), (1024, 2)])
def test_mask_of_given_labels(width, height):
    import torch
    from paper_1302_2073_amd.tracker import Tracker
    P = width * height
    rng = np.random.default_rng([width, height])
    with Tracker(width, height, 1, 1) as t:
        for density in (0.0, 0.3, 0.55, 1.0):
            lab = (rng.random(P) < density).astype(np.uint8)
            want = O.median3x3(lab, height, width).astype(np.uint8).ravel()
            store = torch.full((P + 8,), 7, dtype=torch.uint8, device="cuda")
            for shift in (0, 1):
                t.set_state(_orth(P, 1, 1), labels=lab, n=3)
                t.mask(out=store[shift:shift + P])             # the median itself writes it
                torch.cuda.synchronize()
                got = store.cpu().numpy()
                assert np.array_equal(got[shift:shift + P], want) and np.all(got[shift + P:] == 7)
                t.mask(out=store[shift:shift + P])             # again: a copy of the finished mask
                assert np.array_equal(t.mask(), want)
                assert np.array_equal(t.mask(filtered=False), lab)
                assert t.stats()["fg_pixels"] == int(lab.sum())
            t.set_state(_orth(P, 1, 1), labels=lab, n=3)
            assert t.stats()["fg_pixels"] == int(lab.sum())    # the statistics first
            assert np.array_equal(t.mask(), want)


@pytest.mark.parametrize("storage,rows", [("f32", 0), ("bf16", 0), ("f32", -1)])
def test_mask_read_every_frame_changes_nothing(storage, rows):
    """Reading each mask (on the device or the host) leaves labels, masks and state as when none is read."""
    import torch
    from paper_1302_2073_amd.tracker import Tracker
    w, h, k, frames = 52, 36, 4, 5
    m = 3 * w * h
    U = _orth(m, k, 5)
    rng = np.random.default_rng(9)
    xs = [torch.tensor(0.2 * (U @ rng.standard_normal(k)) + 0.02 * rng.standard_normal(m), dtype=torch.float32,
                       device="cuda").to(torch.float32 if storage == "f32" else torch.bfloat16) for _ in range(frames)]
    for filtered_weights in (False, True):
        runs = []
        for read in (0, 1, 2):
            with Tracker(w, h, 3, k, storage=storage, weights_from_filtered=filtered_weights) as t:
                if rows:
                    t.set_launch(rows)
                t.set_state(U, None, None, 0)
                out = torch.zeros(w * h, dtype=torch.uint8, device="cuda")
                for x in xs:
                    t.track(x)
                    if read == 1:
                        t.mask(out=out)
                    elif read == 2:
                        labels = t.mask(filtered=False)
                        assert np.array_equal(t.mask(), O.median3x3(labels, h, w).astype(np.uint8).ravel())
                        assert t.stats()["fg_pixels"] == int(labels.sum())
                runs.append((*t.get_state(), t.mask()))
        for other in runs[1:]:
            for a, b in zip(runs[0], other):
                assert np.array_equal(a, b)
