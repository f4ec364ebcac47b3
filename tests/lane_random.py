"""Random programs over a forest, for the generated lanes: functions f(v, c, k) of a node, fuel and an integer that call
one another with less fuel, with switches inside each other, calls in any order of readiness, arguments from the forest and
from other calls, and EMBEDs and cells where the tag has room for one.  `evaluate` is a plain evaluator of the node
tables: values, DEAD, and what fired."""
from paper_2410_20225_amd import tdf as T
from paper_2410_20225_amd.programs import _Fn

DEAD = object()


class Skip(Exception):
    """An instance that the lanes leave to the step machine (a call with some arguments dead), or a large one."""


def program(rng, vector):
    """Kinds of functions: N gives a node, I an integer, V a vector value; function 1 is what `result` calls."""
    n_fn = rng.randint(1, 3)
    kinds = ["V" if vector else "I"] + [rng.choice("NIV" if vector else "NII") for _ in range(n_fn - 1)]
    fns = []
    for kind in kinds:
        F = _Fn("f", 3)
        v, c, k = (F.add(T.OP_IN, imm=i) for i in range(3))
        const, calls, most = {}, [0], rng.randint(1, 4)

        def C(x):
            if x not in const:
                const[x] = F.add(T.OP_CONST, imm=x)
            return const[x]

        def call(env, typ, depth, fuel):
            calls[0] += 1
            less = F.add(T.OP_SUB, [fuel, C(rng.choice([1, 1, 2, 3]))])
            g = rng.choice([i + 1 for i in range(n_fn) if kinds[i] == typ])
            return F.add(T.OP_CALLFN, [expr(env, "N", depth - 1, fuel), less, expr(env, "I", depth - 1, fuel)], imm=g)

        def other_side(p, env, fuel, port):
            return ({t: [(F.add(T.OP_SWITCH, [p, r])[0], port) for r in env[t][-3:]] for t in "NI"},
                    None if fuel is None else (F.add(T.OP_SWITCH, [p, fuel])[0], port))

        def merge(a, b):
            return F.add(T.OP_MERGE, [a, b] if rng.random() < .5 else [b, a])

        def expr(env, typ, depth, fuel):   # env: values by kind, all of them on the same sides of the same switches
            can_call = fuel is not None and depth > 0 and calls[0] < most and typ in kinds
            ops = {"N": ["var", "var", "right", "next"], "V": ["embed", "embed"],
                   "I": ["var", "var", "const"] + (["token", "isleaf", "left", "cmp", "arith", "arith"] if depth > 0 else ["token0"])}[typ]
            ops = ops + (["switch"] if depth > 0 else []) + (["call"] * 4 if can_call else [])
            if typ == "V" and can_call:
                ops += ["cell"] * 4 + ["early"] * 2
            op = rng.choice(ops)
            sub = lambda t: expr(env, t, depth - 1, fuel)  # noqa: E731
            if op == "var":
                return rng.choice(env[typ])
            if op == "const":
                return F.add(T.OP_ADD, [rng.choice(env["I"]), C(rng.randint(-3, 3))])
            if op == "right":
                return F.add(T.OP_TREE_RIGHT, [rng.choice(env["N"])])
            if op == "next":   # right child of a leaf, left child of another node (both are nodes in these forests)
                n = rng.choice(env["N"])
                s = F.add(T.OP_SWITCH, [F.add(T.OP_TREE_ISLEAF, [n]), n])
                return merge(F.add(T.OP_TREE_RIGHT, [(s[0], 0)]), F.add(T.OP_TREE_LEFT, [(s[0], 1)]))
            if op == "token0":
                return F.add(T.OP_TREE_TOKEN, [rng.choice(env["N"])])
            if op in ("token", "isleaf", "left"):
                return F.add({"token": T.OP_TREE_TOKEN, "isleaf": T.OP_TREE_ISLEAF, "left": T.OP_TREE_LEFT}[op], [sub("N")])
            if op == "arith":
                return F.add(rng.choice([T.OP_ADD, T.OP_SUB, T.OP_MUL]), [sub("I"), sub("I")])
            if op == "cmp":
                return F.add(rng.choice([T.OP_EQ, T.OP_LT]), [sub("I"), sub("I")])
            if op == "call":
                return call(env, typ, depth, fuel)
            if op == "embed":
                return F.add(T.OP_EMBED, [F.add(T.OP_TREE_TOKEN, [sub("N")])])
            if op == "cell":
                return F.add(T.OP_RNN_CELL, [call(env, "V", depth, fuel), call(env, "V", depth, fuel)])
            p = F.add(T.OP_LT, [expr(env, "I", min(depth - 1, 2), fuel), C(rng.randint(-2, 15))])
            if op == "early":   # the EMBED fires under every tag, one side of the switch takes it
                e = F.add(T.OP_SWITCH, [p, F.add(T.OP_EMBED, [F.add(T.OP_TREE_TOKEN, [sub("N")])])])
                env2, fuel2 = other_side(p, env, fuel, 1)
                return merge((e[0], 0), call(env2, "V", 1, fuel2))
            (env0, fuel0), (env1, fuel1) = other_side(p, env, fuel, 0), other_side(p, env, fuel, 1)
            return merge(expr(env0, typ, depth - 1, fuel0), expr(env1, typ, depth - 1, fuel1))

        p = F.add(T.OP_LT, [c, C(1)])
        sv, sc, sk = (F.add(T.OP_SWITCH, [p, x])[0] for x in (v, c, k))
        base = expr({"N": [(sv, 0)], "I": [(sk, 0), (sc, 0)]}, kind, rng.randint(0, 3), None)
        rest = expr({"N": [(sv, 1)], "I": [(sk, 1), (sc, 1)]}, kind, rng.randint(2, 4), (sc, 1))
        F.add(T.OP_OUT, [F.add(T.OP_MERGE, [base, rest])])
        fns.append(F.desc())
    r = _Fn("result", 3)
    r.add(T.OP_OUT, [r.add(T.OP_CALLFN, [r.add(T.OP_IN, imm=i) for i in range(3)], imm=1)])
    return [r.desc()] + fns, 0


def forest(rng, n=12):
    """Not a tree: every right child is a node, and every left child but the leaves'."""
    return dict(left=[rng.randrange(n) if rng.random() < .6 else -1 for _ in range(n)], right=[rng.randrange(n) for _ in range(n)],
                token=[rng.randrange(9) for _ in range(n)])


def evaluate(prog, forest, args, most=4000):
    """(value, tags, EMBED firings, cell firings); a vector value is ("E", token) or ("C", left, right)."""
    fns, result = prog
    left, right, token = forest["left"], forest["right"], forest["token"]
    n = [-1, 0, 0]
    wrap = lambda x: (x + 2 ** 63) % 2 ** 64 - 2 ** 63  # noqa: E731

    def call(f, a):
        n[0] += 1
        if n[0] > most:
            raise Skip
        V = []
        for op, ins, imm in fns[f][2]:
            x = [V[i][port] if fns[f][2][i][0] == T.OP_SWITCH else V[i] for i, port in ins]
            dead = [y is DEAD for y in x]
            if op == T.OP_IN:
                y = a[imm]
            elif op == T.OP_CONST:
                y = imm
            elif op == T.OP_MERGE:
                live = [z for z in x if z is not DEAD]
                y = live[0] if live else DEAD
            elif op == T.OP_CALLFN and any(dead) and not all(dead):
                raise Skip
            elif any(dead):
                y = (DEAD, DEAD) if op == T.OP_SWITCH else DEAD
            elif op == T.OP_CALLFN:
                y = call(imm, x)
            elif op == T.OP_SWITCH:
                y = (x[1], DEAD) if x[0] else (DEAD, x[1])
            elif op == T.OP_OUT:
                return x[0]
            elif op == T.OP_EMBED:
                n[1] += 1
                y = ("E", x[0])
            elif op == T.OP_RNN_CELL:
                n[2] += 1
                y = ("C", x[0], x[1])
            else:
                y = {T.OP_ADD: lambda: wrap(x[0] + x[1]), T.OP_SUB: lambda: wrap(x[0] - x[1]), T.OP_MUL: lambda: wrap(x[0] * x[1]),
                     T.OP_EQ: lambda: int(x[0] == x[1]), T.OP_LT: lambda: int(x[0] < x[1]), T.OP_TREE_ISLEAF: lambda: int(left[x[0]] < 0),
                     T.OP_TREE_LEFT: lambda: left[x[0]], T.OP_TREE_RIGHT: lambda: right[x[0]], T.OP_TREE_TOKEN: lambda: token[x[0]]}[op]()
            V.append(y)
        return DEAD
    value = call(result, args)
    if value is DEAD:
        raise Skip
    return (value, *n)
