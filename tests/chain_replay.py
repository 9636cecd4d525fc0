"""Host replay of how far the evaluator's first pass and its first continuation pass take a pipeline
(whole numbers in float64, as there), so that tests can state which pass their plans end in."""
import numpy as np

CONT_BUDGET, POWER_MIN, CONT_FEW = 48, 16, 12288


class Chains:
    """N pipelines of S stages as chains on potentials: forward, backward (input-gradient) and
    weight-gradient times and hops [N, S], micro-batches [N]."""

    def __init__(self, f, b, w, c, M):
        self.w, self.M, self.S = w, M, f.shape[1]
        self.a = f + b + w
        self.d = np.zeros_like(f)
        self.d[:, :-1] = 2 * c[:, :-1] + f[:, 1:] + b[:, 1:]
        s = np.arange(self.S)
        self.F = np.minimum(self.S - 1 - s[None, :], M[:, None] - 1) * np.maximum.accumulate(f, axis=1)

    def step(self, on, i=None):
        """One steady iteration of the pipelines `on`; i < S - 1: an early one of the zero-bubble order."""
        F, a = self.F[on], self.a[on]
        B = None
        for s in range(self.S - 1, -1, -1):
            B = F[:, s] if s == self.S - 1 else np.maximum(F[:, s], B + self.d[on, s])
            x = B + a[:, s] - (self.w[on, s] if i is not None and i < s else 0)
            F[:, s] = np.maximum(x, F[:, s - 1]) if s else x
        self.F[on] = F

    def rate_step(self, on, r):
        """One iteration with the rates r of the state: the new rates, and for how many steps every max
        keeps its argument."""
        F, J = self.F[on], np.full(int(on.sum()), 1e9)
        B = rB = None

        def pick(x, rx, y, ry):
            dx, dr = x - y, rx - ry
            ahead = (dx > 0) | ((dx == 0) & (dr > 0))
            meets = np.sign(dx) * np.sign(dr) < 0
            J[meets] = np.minimum(J[meets], -dx[meets] / dr[meets])
            return np.maximum(x, y), np.where(ahead, rx, ry)
        r = r.copy()
        for s in range(self.S - 1, -1, -1):
            if s == self.S - 1:
                B, rB = F[:, s].copy(), r[:, s].copy()
            else:
                B, rB = pick(F[:, s], r[:, s], B + self.d[on, s], rB)
            if s:
                F[:, s], r[:, s] = pick(B + self.a[on, s], rB, F[:, s - 1].copy(), r[:, s - 1].copy())
            else:
                F[:, 0], r[:, 0] = B + self.a[on, 0], rB
        self.F[on] = F
        return r, J

    def first_pass(self, zero_bubble=False):
        """Steady iterations left after the first pass's budget (0: the pipeline ends there)."""
        left = self.M - self.S
        if zero_bubble:
            for i in range(self.S - 1):
                on = left > 0
                self.step(on, i)
                left = left - on
        budget = self.S + 8
        while budget > 0 and np.any(left >= 2):
            on = left >= 2
            self.step(on)
            old = self.F.copy()
            self.step(on)
            adv = self.F - old
            same = on & np.all(adv == adv[:, -1:], axis=1)
            left = np.where(on, left - 2, left)
            left[same] = 0
            budget -= 2
        return np.where(left == 1, 0, np.maximum(left, 0))

    def cont_pass(self, left):
        """Of pipelines with `left` iterations to go, those left after the first continuation pass."""
        left, budget, q = left.copy(), np.full(left.size, CONT_BUDGET), 1
        while True:
            on = (left >= 3 * q) & (budget > 0)
            if not np.any(on):
                return left
            old = self.F.copy()
            for _ in range(q):
                self.step(on)
            D = self.F - old
            left, budget = left - q * on, budget - q * on
            same = on & np.all(D == D[:, :1], axis=1)
            left[same] = left[same] % q
            go = on & ~same
            old = self.F.copy()
            for _ in range(q):
                self.step(go)
            left, budget = left - q * go, budget - q * go
            go &= np.all(self.F - old == D, axis=1)
            if np.any(go):
                old, r, J = self.F.copy(), D[go], np.full(int(go.sum()), 1e9)
                for _ in range(q):
                    r, j = self.rate_step(go, r)
                    J = np.minimum(J, j)
                left, budget = left - q * go, budget - q * go
                ok = np.all(r == D[go], axis=1) & np.all((self.F - old == D)[go], axis=1)
                k = np.where(ok, np.minimum(np.floor(J * 0.99999), left[go] // q), 0).astype(np.int64)
                self.F[go] += k[:, None] * D[go]
                left[go] -= k * q
            q = 3 - q


def chains(oracle, p, plans, S, zero_bubble=False):
    """The S-stage pipelines of those of `plans` that are valid."""
    f, b, w, c, M = [], [], [], [], []
    for i in plans:
        d = oracle.detail(p, int(i))
        for g in range(d["G"] if d else 0):
            if d["S_class"][g] == S:
                for v, key in ((f, "f"), (b, "b"), (w, "w"), (c, "c")):
                    v.append(d[key][g])
                M.append(d["M"][g])
    f, b, w, c = (np.array(v, np.float64) for v in (f, b, w, c))
    if not zero_bubble:
        w = np.zeros_like(b)
    return Chains(f, b - w, w, c, np.array(M, np.int64))
