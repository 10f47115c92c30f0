"""The local solve's headers on the host (host_solve.cpp): what the bracket
refinement accepts, where coarse sweeps and iteration caps leave it little to
go by."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_26108_amd")

# a strongly attenuating layer-like medium and a strongly anisotropic one, both
# with sweep intervals of 22.5 degrees that span more than a right angle of ray
# directions (qSV, opposite-end velocity)
COARSE = np.array([
    [5907509.213320775, 2918469.166620558, 5341460.524536856, 1631421.5936059605,
     2060605.3945572022, 12.941943652162367, 2.9667210365482743, 8.509536873357579,
     3.948429015215527, 5.893121311447293, 2300.0, -0.17949259425881514, 0.0],
    [4102158.950271772, 1775638.28687719, 1090284.6187087786, 46382.89533621889,
     36164.636058535085, 906.4433285547342, 14.095390222235016, 153.98735066119715,
     647.9902803100911, 48.10317854220429, 2300.0, 0.0010491099580471897, 0.0]])


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_solve") / "host_solve")
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off",
                    "-I", os.path.join(PKG, "opcount"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "host_solve.cpp"), "-o", exe, "-lm"],
                   check=True, capture_output=True, text=True)

    def run(classes, mode, kernel, n_sweep=1440, n_dirs=360, newton=12, bisect=200, extra=()):
        text = "\n".join(" ".join(repr(float(x)) for x in r) for r in classes) + "\n"
        out = subprocess.run([exe] + [str(x) for x in (mode, kernel, n_sweep, n_dirs, newton, bisect, *extra)],
                             input=text, check=True, capture_output=True, text=True).stdout
        return np.array([[float(x) for x in line.split()] for line in out.splitlines()])
    return run


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("n_sweep", [16, 17, 20, 90])
def test_newton_keeps_only_the_targets_own_direction(host, n_sweep, kernel):
    """The iteration's direction equation also vanishes at the reverse of the
    target and at right angles to it; a bracket that holds such a zero goes to
    the bisection.  An accepted root's ray is the target's to far below any
    residual bound (1e-6 rad against the last step's 1e-10)."""
    b = host(COARSE, 1, kernel, n_sweep=n_sweep)
    ok = b[:, 2] == 1
    assert ok.any()
    assert b[ok, 3].max() < 1e-6


def layer_classes(n, seed):
    """Thomsen media in the ranges of the layered models, a quality factor per modulus."""
    rng = np.random.default_rng(seed)
    rows = []
    for _ in range(n):
        vp = rng.uniform(2000.0, 4500.0)
        a33, a44 = vp * vp, (vp / rng.uniform(1.6, 2.0)) ** 2
        delta = rng.uniform(-0.1, 0.2)
        a13 = np.sqrt((a33 - a44) * (a33 - a44 + 2.0 * delta * a33)) - a44
        rows.append([a33 * (1.0 + 2.0 * rng.uniform(0.0, 0.3)), a13, a33, a44,
                     a44 * (1.0 + 2.0 * rng.uniform(0.0, 0.2)), *rng.uniform(15.0, 150.0, 5),
                     2300.0, rng.uniform(-np.pi / 4, np.pi / 4), 0.0])
    return np.array(rows)


@pytest.mark.parametrize("cap", [3, 12, 30, 200])
def test_a_converged_root_survives_a_small_iteration_cap(host, cap):
    """Entries whose attenuation cancels are bisected again for their last
    digits; with few halvings allowed (or where the bisection closes on a jump)
    a converged Newton root must not be given up for that."""
    b = host(layer_classes(60, 5), 1, 1, newton=max(cap, 12), bisect=cap)
    solved = (b[:, 2] == 1) & (b[:, 4] <= 1e-9)
    assert solved.sum() > 5000
    assert (b[solved, 5] == 1).all()
    assert b[solved, 6].max() <= 1e-9


def test_surrogate_start_leaves_cancelled_attenuation_to_the_plain_search(host):
    """Both builds store the same digits of an attenuation that has cancelled:
    the surrogate start accepts no such entry, and what it accepts is the plain
    search's entry within the cache bar."""
    cls = layer_classes(60, 6)
    b = host(cls, 1, 1, extra=("warm",))
    im = [cls[:, i] / cls[:, 5 + i] for i in range(5)]  # imaginary parts of the moduli
    loss = np.minimum.reduce([im[0] / cls[:, 0], im[2] / cls[:, 2], im[3] / cls[:, 3]])
    ok = b[:, 5] == 0
    assert ok.sum() > 5000
    a_v = np.abs(b[ok, 7]) * b[ok, 6]
    assert (a_v >= 1e-3 * loss[b[ok, 0].astype(int)]).all()
    same = ok & (b[:, 2] == 0) & (np.abs(b[:, 6] - b[:, 3]) < 1e-6 * b[:, 3])
    assert same.sum() > 5000
    assert (np.abs(b[same, 7] - b[same, 4]) / np.abs(b[same, 4])).max() <= 1e-10


@pytest.mark.parametrize("power", [-200, -50, -13, 13, 50, 200])
@pytest.mark.parametrize("mode,kernel", [(0, 0), (1, 0), (1, 1), (2, 1)])
def test_the_unit_of_the_moduli_does_not_matter(host, mode, kernel, power):
    """Moduli times a power of four: the same angles and residuals to the last
    bit, so the same brackets, roots and misses, whatever the unit."""
    cls = layer_classes(6, 7)
    scaled = cls.copy()
    scaled[:, :5] = np.ldexp(cls[:, :5], 2 * power)
    a = host(cls, mode, kernel, n_dirs=72)
    assert len(a) > 200
    np.testing.assert_array_equal(a, host(scaled, mode, kernel, n_dirs=72))
