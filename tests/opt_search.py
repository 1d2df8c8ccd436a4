"""The hindsight optimum's one-wave search in plain Python: what the first launch does
with an instance that does not fit a 64-step memory profile, and how many start steps
it tests (64 at a time, in order, each level ended by the first one that reaches the
best total)."""


def one_wave_search(inst, M, cap):
    """(best total, start steps tested, whether the search ended within `cap` of them)."""
    o0, s0 = [int(x) for x in inst["output"]], [int(x) for x in inst["prompt"]]
    n = len(o0)
    a0 = [int(x) for x in inst["arrival"]] if inst.get("arrival") is not None else [0] * n
    horizon = max(a0) + sum(x + 1 for x in o0) + 1
    best, t = 0, 0
    for i in range(n):  # one request at a time
        start = max(t, a0[i])
        best += start + o0[i] - a0[i]
        t = start + o0[i] + 1
    order = sorted(range(n), key=lambda i: (a0[i], -(s0[i] + o0[i]), -o0[i]))
    a, s, o = ([v[i] for i in order] for v in (a0, s0, o0))
    rem = [sum(o[i:]) for i in range(n + 1)]
    state = {"best": best, "nodes": 0, "stop": False}
    placed = []  # (start, completion, request)

    def fits(d, p):
        runs = placed + [(p, p + o[d], d)]
        return all(sum(s[i] + e - q for q, f, i in runs if q <= e <= f) <= M
                   for e in {f for q, f, i in runs if p <= f <= p + o[d]})

    def level(d, cost):
        same = d > 0 and (a[d], s[d], o[d]) == (a[d - 1], s[d - 1], o[d - 1])
        base = placed[d - 1][0] if same else a[d]
        while base <= horizon:
            # live starts of this chunk come first
            live = min(64, horizon + 1 - base, state["best"] - (cost + base + o[d] - a[d] + rem[d + 1]))
            live = max(live, 0)
            state["nodes"] += live + (1 if live < 64 else 0)
            if state["nodes"] > cap:
                state["stop"] = True
                return
            for p in range(base, base + live):
                if not fits(d, p):
                    continue
                c = cost + p + o[d] - a[d]
                if c + rem[d + 1] >= state["best"]:
                    return
                if d == n - 1:
                    state["best"] = c
                    return
                placed.append((p, p + o[d], d))
                level(d + 1, c)
                placed.pop()
                if state["stop"]:
                    return
            if live < 64:
                return
            base += 64

    level(0, 0)
    return state["best"], state["nodes"], not state["stop"]
