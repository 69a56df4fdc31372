"""Kernels stay inside the memory that the library asks for: every allocation
lies between guard words, without slack."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GUARD = 4096


@pytest.fixture(scope="module")
def mp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_11878_amd import mpcd
    return mpcd


def _guarded(mp, blocks):
    """The context's allocator with GUARD bytes of 0xA5 before and behind each block."""
    class Guarded(mp._TorchAllocator):
        def _alloc(self, nbytes, user):
            try:
                with self._torch.cuda.stream(self.stream):
                    t = self._torch.full((int(nbytes) + 2 * GUARD,), 0xA5, dtype=self._torch.uint8,
                                         device=self.device)
            except Exception:
                return None
            p = t.data_ptr() + GUARD
            self.blocks[p] = t
            blocks.append(t)
            return p
    return Guarded


@pytest.mark.parametrize("tiles", [1025, 1056, 2080])
def test_observing_a_large_box_stays_inside_it(mp, monkeypatch, tiles):
    """Boxes of so many tiles of 4096 particles that their exact sums are folded
    in two levels.  Of 1056 and 2080 tiles, folded by fives and nines, the last
    run would hold one tile, and the partial sums end on the last byte of the
    box's allocation: a record of sums over a run of one would end 56 bytes
    behind it."""
    import torch
    blocks = []
    monkeypatch.setattr(mp, "_TorchAllocator", _guarded(mp, blocks))
    n = 4096 * tiles
    with mp.Context(binning=mp.MPCD_BIN_SORT) as ctx:
        slot = ctx.admit(mp.make_desc((128, 128, 64), n, seed=2, unordered=True))
        for _ in range(2):
            ctx.step(1)
            obs = ctx.observe(slot)
            assert obs["status"] == 0 and abs(obs["T"] - 1.0) < 1e-6
        torch.cuda.synchronize()
        assert len(blocks) >= 2
        for t in blocks:
            assert bool((t[:GUARD] == 0xA5).all()) and bool((t[-GUARD:] == 0xA5).all()), t.numel()


@pytest.mark.parametrize("more", [{}, dict(unordered=True), dict(particle_mass=True), dict(conserve_l=True),
                                  dict(vacf_stride=2)])
@pytest.mark.parametrize("binning", [1, 2])
def test_a_box_stays_inside_its_memory(mp, monkeypatch, binning, more):
    """A ragged box that is set, stepped with full buckets, read and set again."""
    import torch
    blocks = []
    monkeypatch.setattr(mp, "_TorchAllocator", _guarded(mp, blocks))
    L, n = (17, 9, 13), 20011
    g = np.random.default_rng(4)
    pos = (g.uniform(0.0, 1.0, (3, n)) * np.array([[3.0], [9.0], [13.0]])).astype(np.float32)
    vel = g.standard_normal((3, n)).astype(np.float32)
    vel[0] += np.float32(4.0)
    with mp.Context(binning=binning, brick=4 if binning == 1 else 0) as ctx:
        slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, **more), (pos, vel))
        for steps in (1, 5, 20):
            ctx.step(steps)
            ctx.observe(slot)
            state = ctx.get_state(slot)
            ctx.set_state(slot, state[:2], state[2])
        torch.cuda.synchronize()
        for t in blocks:
            assert bool((t[:GUARD] == 0xA5).all()) and bool((t[-GUARD:] == 0xA5).all()), t.numel()
