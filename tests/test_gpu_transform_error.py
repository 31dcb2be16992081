"""Rounding of the nonlinear term's transforms, in both forms, against the same
term in long double.  The limits are the errors of plain passes (radices 8, 4
or 2, 3, 5 in this order, powers of one twiddle by products) on these inputs,
measured on an MI355X; the mean over four inputs repeats within a few per cent,
so 1.1 times the limit is allowed."""
import numpy as np
import pytest
import scipy.fft as sf

import oracle
import tc_inputs
from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu

LD, CLD = np.longdouble, np.clongdouble

# azimuthal length: relative l2 error of the plain passes
ROTATIONAL = {16: 8.42e-16, 32: 1.13e-15, 40: 1.31e-15, 80: 1.52e-15, 144: 1.66e-15, 160: 2.10e-15, 288: 2.78e-15,
              480: 5.47e-15, 640: 9.43e-15, 1152: 1.83e-14}
CONVECTIVE = {144: 3.65e-16, 240: 4.06e-16, 288: 4.18e-16, 480: 4.52e-16}


class Exact:
    """N(u) by long double transforms on (p_z, p_theta)."""

    def __init__(self, P, u):
        self.P, self.u = P, u.astype(CLD)
        self.mz, self.mt = u.shape[2:]
        self.pz, self.pt = P.p_z, P.p_theta
        self.slots = [s for s in range(self.mz) if s != P.nyq]
        self.l = [s if s < P.nyq else s - self.mz for s in self.slots]
        self.r = P.r.astype(LD)[:, None, None]
        self.a, self.b = P.a.astype(LD)[None, None, :], P.b.astype(LD)[None, :, None]
        self.du = [np.tensordot(P.D1.astype(LD), f, axes=(1, 0)) for f in self.u]

    def spectrum(self, fp, fm):
        """Full spectrum of v_r + i v_theta from (v+, v-), or twice the same
        real field; both stored halves of n = 0 averaged."""
        G = np.zeros(fp.shape[:1] + (self.pz, self.pt), dtype=CLD)
        for s, l in zip(self.slots, self.l):
            G[:, l % self.pz, :self.mt] = fp[:, s]
            G[:, l % self.pz, 0] = (fp[:, s, 0] + np.conj(fm[:, -l % self.mz, 0])) / 2
            G[:, -l % self.pz, self.pt - np.arange(1, self.mt)] = np.conj(fm[:, s, 1:])
        return G

    @staticmethod
    def signed(n):
        k = np.arange(n)
        return np.where(k <= n // 2, k, k - n)

    def physical(self, fp, fm, factor=1):
        return sf.ifft2(factor * self.spectrum(fp, fm), axes=(-2, -1), norm="forward")

    def real(self, f, factor=1):
        return self.physical(f, f, factor).real

    def truncate(self, hn, nz):
        H, Z = (sf.fft2(x, axes=(-2, -1), norm="forward") for x in (hn, nz))
        N = np.zeros((3,) + self.u.shape[1:], dtype=CLD)
        for s, l in zip(self.slots, self.l):
            N[0][:, s] = H[:, l % self.pz, :self.mt]
            N[1][:, s] = np.conj(H[:, -l % self.pz, -np.arange(self.mt) % self.pt])
            N[2][:, s] = Z[:, l % self.pz, :self.mt]
        return N

    def rotational(self):
        (up, um, uz), (dp, dm, dz), a, b, r = self.u, self.du, self.a, self.b, self.r
        hw = self.physical(1j * (a / r * uz - dz) - b * up, 1j * (a / r * uz + dz) + b * um)
        wz = self.real(-0.5j * ((dp + (1 + a) / r * up) - (dm + (1 - a) / r * um)))
        hu, uz = self.physical(up, um), self.real(uz)
        return self.truncate((hw.imag * uz - wz * hu.imag) + 1j * (wz * hu.real - hw.real * uz),
                             hw.real * hu.imag - hw.imag * hu.real)

    def convective(self):
        (up, um, uz), (dp, dm, dz), r = self.u, self.du, self.r
        dth, dax = 1j * self.signed(self.pt), 1j * self.signed(self.pz)[:, None]
        hu, w = self.physical(up, um), self.real(uz)
        ur, ut = hu.real, hu.imag
        hn = (ur * self.physical(dp, dm) + ut * self.physical(up, um, dth) / r + w * self.physical(up, um, dax)
              + 1j * ut / r * hu)
        return self.truncate(hn, ur * self.real(dz) + ut * self.real(uz, dth) / r + w * self.real(uz, dax))


@pytest.mark.parametrize("form,p_theta", [("rot", L) for L in ROTATIONAL] + [("conv", L) for L in CONVECTIVE])
def test_transforms_as_accurate_as_plain_passes(form, p_theta):
    from paper_1311_2481_amd import Solver
    n_r, m_theta, m_z, p_z = 9, (p_theta + 2) // 3, 6, 16
    args = (n_r, m_theta, m_z, 0.5, 100.0, 0.0, 1e-4)
    P = oracle.Problem(*args, p_theta=p_theta, p_z=p_z)
    S = Solver(*args, p_theta=p_theta, p_z=p_z, form=form)
    errs = []
    for seed in range(4):
        u = tc_inputs.random_state((3, n_r, m_z, m_theta), 100 + seed)
        E = Exact(P, u)
        ref = E.rotational() if form == "rot" else E.convective()
        d = np.abs(to_host(S.nonlinear(to_dev(u))) - ref)
        errs.append(float(np.sqrt((d ** 2).sum() / (np.abs(ref) ** 2).sum())))
    S.close()
    limit = (ROTATIONAL if form == "rot" else CONVECTIVE)[p_theta]
    print(f"{form} p_theta={p_theta}: rel_l2 against long double {np.mean(errs):.2e} (plain passes {limit:.2e})")
    assert np.mean(errs) <= 1.1 * limit
