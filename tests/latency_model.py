"""A model of the range search of csrc/latency_dp.hip for one shared search: the same
ranges in the same order, one Python pass at a time.  It tells how many passes the
kernel takes and whether it swept a range threshold by threshold, so that a test can
pick searches that do and check that the kernel did."""
import numpy as np

BIG = 1 << 62
NODES = 24   # open ranges a search keeps


def weight(c):
    return c + (c + 2) // 3


def cost(w):
    return 3 * (w >> 2) + (((w & 3) + 1) >> 1)


def bands(lo, hi, n):
    """First end layer and width of every stage's band under its windows."""
    cl, ch = np.cumsum(lo), np.cumsum(hi)
    first = np.maximum(cl, n - (ch[-1] - ch))
    return first.tolist(), (np.minimum(ch, n - (cl[-1] - cl)) - first + 1).tolist()


class Search:
    def __init__(self, cost_tensor, lo, hi, micro):
        """cost_tensor [pp][n + 1][n + 1] (stage, from, to), micro: the members' B, all
        above the depth, in order."""
        self.pp, w1, _ = cost_tensor.shape
        n = w1 - 1
        self.micro = list(micro)
        first, width = bands(lo, hi, n)
        prev = (0, 1)
        self.rows = []   # [stage][end layer of the band]: (split point of the band before, weight), costs rising
        for s in range(self.pp):
            rows = []
            for b in range(first[s], first[s] + width[s]):
                row = [(a - prev[0], weight(int(cost_tensor[s, a, b])))
                       for a in range(b - lo[s], b - hi[s] - 1, -1)
                       if prev[0] <= a < prev[0] + prev[1] and cost_tensor[s, a, b] < BIG // 4]
                assert all(x[1] <= y[1] for x, y in zip(row, row[1:]))
                rows.append(row)
            self.rows.append(rows)
            prev = (first[s], width[s])
        self.weights = sorted({w for rows in self.rows for row in rows for _, w in row})
        widest = max(width)
        self.slots = 2 * (4 if widest <= 24 else 2 if widest <= 48 else 1)   # with LDS to spare

    def least_largest(self):
        f = [0]
        for rows in self.rows:
            f = [min((max(f[q], w) for q, w in row), default=BIG) for row in rows]
        return f[0]

    def one_pass(self, lo, hi, micro):
        """(least V, its bottleneck, largest stage twice plus a tie flag) of a range."""
        state = [(0, 0, BIG, 0, 0)]
        for s, rows in enumerate(self.rows):
            steady = max(0, micro - s - 2)
            new = []
            for row in rows:
                b0, m0, b1, t1, m1 = BIG, 0, BIG, 0, 0
                for q, w in row:
                    if w > hi:
                        break
                    v0, n0, v1, u1, n1 = state[q]
                    c, mm, x0 = cost(w), max(n0, w), v0 + w
                    if not (lo == hi and w == hi) and (x0 < b0 or (x0 == b0 and mm < m0)):
                        b0, m0 = x0, mm
                    x1 = x0 + steady * c
                    if w >= lo and v0 < BIG and (x1 < b1 or (x1 == b1 and w < t1)):
                        b1, t1, m1 = x1, w, 2 * mm + (n0 >= w)
                    y = v1 + c
                    if y < b1 or (y == b1 and u1 < t1 and v1 < BIG):
                        b1, t1, m1 = y, u1, max(n1, 2 * w)
                new.append((b0, m0, b1, t1, m1))
            state = new
        return state[0][2:]

    def run(self):
        """Members' (latency, largest stage), passes, and the passes of threshold sweeps."""
        slots, top, t = self.slots, self.weights[-1], self.least_largest()
        best = [(BIG, BIG)] * len(self.micro)
        edges = [(t, t)] + [(t + (0 if k == 1 else t >> (9 - k)) + 1, top if k == 7 else t + (t >> (8 - k)))
                            for k in range(1, 8)]
        nodes = [(a, min(z, top), 0 if a <= min(z, top) else BIG, self.micro[0]) for a, z in edges]
        passes = swept = 0

        def gain(a, z, v, bb):
            """Whether a member may gain in [a, z], and the B to run it at."""
            is_open, be = False, self.micro[0]
            for bu, (lat, tl) in zip(self.micro, best):
                d = bu - bb
                low = v + d * (cost(a) if d >= 0 else cost(z))
                if v < BIG and (low < lat or (low == lat and a < tl)):
                    if not is_open or (v > 0 and abs(d) > abs(be - bb)):
                        be = bu
                    is_open = True
            return is_open, be

        def evaluate(jobs):
            out = [self.one_pass(*j) for j in jobs]
            for (_, _, bb), (v, tau, m) in zip(jobs, out):
                if v < BIG and m == 2 * tau:
                    for j, bu in enumerate(self.micro):
                        best[j] = min(best[j], (v + (bu - bb) * cost(tau), tau))
            return out

        while True:
            kept = [(nd, gain(*nd)) for nd in nodes]
            kept = [(nd, be) for nd, (is_open, be) in kept if is_open]
            nodes = [nd for nd, _ in kept]
            if not nodes:
                return best, passes, swept
            if len(nodes) > NODES - 2 * slots:   # the first one threshold by threshold
                (a, z, v, bb), be = kept[0]
                todo = [w for w in self.weights if a <= w <= z]
                while todo:
                    part, todo = todo[:slots], todo[slots:]
                    evaluate([(w, w, be) for w in part])
                    passes, swept, a = passes + len(part), swept + len(part), part[-1] + 1
                nodes = nodes[1:]
                continue
            count = min(len(nodes), slots)
            lg = 0
            while count << (lg + 1) <= slots:
                lg += 1
            jobs = []
            for (a, z, _, _), be in kept[:count]:
                step = ((z - a) >> lg) + 1
                jobs += [(a + k * step, min(a + (k + 1) * step - 1, z), be) for k in range(1 << lg)]
            passes += len(jobs)
            children = []
            for (a, z, bb), (v, tau, m) in zip(jobs, evaluate(jobs)):
                if v >= BIG:
                    continue
                m2 = m >> 1
                if m == 2 * tau:
                    part = [(a, tau - 1, v + 1), (tau + 1, z, v)] if len(self.micro) > 1 else []
                elif m2 > tau:
                    mid = tau + ((m2 - 1 - tau) >> 1)
                    part = [(a, mid, v), (mid + 1, z, v)]
                else:
                    part = [(a, tau - 1, v + 1), (tau, tau, v), (tau + 1, z, v)]
                children += [(x, y, u, bb) for x, y, u in part if x <= y]
            nodes = children + nodes[count:]
