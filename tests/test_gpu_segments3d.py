"""Segments of a 3-D rollout: their ends are checkpoints that steps read and
write in place, and a recomputed segment's last step stops at its grid."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS, FRAMES = 7, [2, 4, 6, 7]


# segments of one step, with a remainder, that fit, and longer than the rollout
@pytest.mark.parametrize("transfer", [W.APIC, W.FLIP])
def test_segments_do_not_change_the_gradient(transfer):
    """Every split of the rollout gives the same end state bit for bit, the
    same loss up to the order in which four waves add to it in four frames (16
    sums of positive terms), and the same gradient up to the order of the
    reverse step's binary64 atomics, from the tape and recomputed (a second
    sweep)."""
    from paper_2507_04192_amd.native import Solver
    cfg = W.SimConfig(dim=3, n=(20, 16, 12), dx=0.01, dt=1e-4, material=W.FLUID, ppc=8, gravity=(0, 0, -9.81),
                      bulk=1e4, gamma=1.0, transfer=transfer, flip_alpha=0.9)
    n = 3001
    rng = np.random.default_rng(7)
    x = rng.uniform(0.02, 0.1, size=(3, n))
    v = rng.normal(0, 0.5, size=(3, n))
    tr = W.pick_tracers(n, 200, 8)
    tgt = rng.normal(0, 0.3, size=(len(FRAMES), 3, 200)).astype(np.float32).astype(np.float64)
    plain = Solver(cfg, "f64", capacity=n)
    plain.mpm_init_particles(x, v)
    plain.mpm_step(STEPS)
    ref = None
    for every, taped in ((1, 0), (1, 7), (2, 1), (3, 2), (3, 3), (7, 1), (9, 1)):
        print(f"[case] segments of {every}, {taped} taped, transfer {transfer}", flush=True)
        s = Solver(cfg, "f64", capacity=n, tape_steps=STEPS, ckpt_every=every, tape_segments=taped)
        s.mpm_init_particles(x, v)
        s.mpm_set_observations(frames=FRAMES, tracer_pid=tr, lag_field="v", lag_target=tgt)
        loss = s.mpm_forward_loss(STEPS)
        for f in ("x", "v", "C", "stress", "pid"):
            assert np.array_equal(s.mpm_read_state(f).cpu().numpy(), plain.mpm_read_state(f).cpu().numpy()), f
        grads = [s.mpm_backward(True, False)[0].cpu().numpy() for _ in range(2)]
        s.mpm_step(2)
        after = s.mpm_read_state("x", "pid").cpu().numpy()
        assert s.mpm_sync_status()[0] == 0
        s.close()
        ref = ref or (loss, grads[0], after)
        assert abs(loss - ref[0]) <= 16 * 2.0 ** -53 * ref[0] and np.array_equal(after, ref[2])
        for g in grads:
            assert np.linalg.norm(g - ref[1]) <= 1e-12 * np.linalg.norm(ref[1])
    plain.close()
