"""Programs over a forest whose generated lanes are easy to get wrong, each with a small forest, arguments and a plain
Python function that says what an instance gives: the value, or for vector results the token whose row it is."""
from paper_2410_20225_amd import programs, tdf as T
from paper_2410_20225_amd.programs import _Fn


def _result(n_params, callee):
    r = _Fn("result", n_params)
    r.add(T.OP_OUT, [r.add(T.OP_CALLFN, [r.add(T.OP_IN, imm=k) for k in range(n_params)], imm=callee)])
    return r


class Forest:
    """Children as pairs, None at a leaf."""
    def __init__(self, children, token):
        self.left = [c[0] if c else -1 for c in children]
        self.right = [c[1] if c else -1 for c in children]
        self.token = list(token)

    def arrays(self):
        return dict(left=self.left, right=self.right, token=self.token)


def _chain(n):
    """n inner nodes 0 .. n - 1, each the left child of the one before; their right children and the end are leaves."""
    children = [(k + 1, n + 1 + k) for k in range(n)] + [None] * (n + 1)
    return Forest(children, [(7 * k + 3) % 50 for k in range(2 * n + 1)])


def embed_under_every_tag():
    """f(v) = let e = E[token(v)] in if isleaf(v) then e else f(left(v)): the EMBED fires in callees that are not
    complete yet, in which it must not have fired before."""
    f = _Fn("f", 1)
    v = f.add(T.OP_IN)
    e = f.add(T.OP_EMBED, [f.add(T.OP_TREE_TOKEN, [v])])
    p = f.add(T.OP_TREE_ISLEAF, [v])
    se, sv = f.add(T.OP_SWITCH, [p, e]), f.add(T.OP_SWITCH, [p, v])
    call = f.add(T.OP_CALLFN, [f.add(T.OP_TREE_LEFT, [(sv[0], 1)])], imm=1)
    f.add(T.OP_OUT, [f.add(T.OP_MERGE, [(se[0], 0), call])])
    F = _chain(9)

    def ref(v):
        return F.token[v] if F.left[v] < 0 else ref(F.left[v])
    return ([_result(1, 1).desc(), f.desc()], 0), F, [(v,) for v in range(19)], ref


def one_of_two_entries():
    """result(v, c) = if c < 1 then left(v) else right(v)"""
    r = _Fn("result", 2)
    v, c = r.add(T.OP_IN, imm=0), r.add(T.OP_IN, imm=1)
    s = r.add(T.OP_SWITCH, [r.add(T.OP_LT, [c, r.add(T.OP_CONST, imm=1)]), v])
    r.add(T.OP_OUT, [r.add(T.OP_MERGE, [r.add(T.OP_TREE_LEFT, [(s[0], 0)]), r.add(T.OP_TREE_RIGHT, [(s[0], 1)])])])
    F = _chain(9)
    return ([r.desc()], 0), F, [(v, c) for v in range(19) for c in (0, 1)], lambda v, c: F.right[v] if c else F.left[v]


def entries_under_an_argument():
    """f(v, c) = if c < 1 then k(c) + k(c) + k(c) + f(v, c + 1) else token(v), k(c) = c + 1: f(v, 0) is tried in place
    and does not look at its node, whose entries must not count as read in f(v, 1) (the fourth call is not tried)."""
    f = _Fn("f", 2)
    v, c = f.add(T.OP_IN, imm=0), f.add(T.OP_IN, imm=1)
    p = f.add(T.OP_LT, [c, f.add(T.OP_CONST, imm=1)])
    sv, sc = f.add(T.OP_SWITCH, [p, v]), f.add(T.OP_SWITCH, [p, c])
    one = f.add(T.OP_CONST, imm=1)
    k1, k2, k3 = (f.add(T.OP_CALLFN, [(sc[0], 0)], imm=2) for _ in range(3))
    y = f.add(T.OP_CALLFN, [(sv[0], 0), f.add(T.OP_ADD, [(sc[0], 0), one])], imm=1)
    for k in (k1, k2, k3):
        y = f.add(T.OP_ADD, [y, k])
    f.add(T.OP_OUT, [f.add(T.OP_MERGE, [y, f.add(T.OP_TREE_TOKEN, [(sv[0], 1)])])])
    k = _Fn("k", 1)
    k.add(T.OP_OUT, [k.add(T.OP_ADD, [k.add(T.OP_IN), k.add(T.OP_CONST, imm=1)])])
    F = _chain(9)
    return ([_result(2, 1).desc(), f.desc(), k.desc()], 0), F, [(v, c) for v in range(19) for c in range(2)], \
        lambda v, c: F.token[v] + (0 if c else 3)


def constant_nodes():
    """result(n) = token(6) - token(3) + n"""
    r = _Fn("result", 1)
    n = r.add(T.OP_IN)
    b, a = (r.add(T.OP_TREE_TOKEN, [r.add(T.OP_CONST, imm=k)]) for k in (6, 3))
    r.add(T.OP_OUT, [r.add(T.OP_ADD, [r.add(T.OP_SUB, [b, a]), n])])
    F = _chain(9)
    return ([r.desc()], 0), F, [(n,) for n in range(3)], lambda n: F.token[6] - F.token[3] + n
def _framed(name, index, add):
    """name(x) = x + add for x below 1000, in a call of its own, so that it is not done in the caller's sweep."""
    q = _Fn(name, 1)
    x, k = q.add(T.OP_IN), q.add(T.OP_CONST, imm=1000)
    s = q.add(T.OP_SWITCH, [q.add(T.OP_LT, [x, k]), x])
    again = q.add(T.OP_CALLFN, [q.add(T.OP_ADD, [(s[0], 0), q.add(T.OP_CONST, imm=1000 + add)])], imm=index)
    q.add(T.OP_OUT, [q.add(T.OP_MERGE, [again, q.add(T.OP_SUB, [(s[0], 1), k])])])
    return q


def entry_of_a_calls_result():
    """f(n) = h(left(g(n))) + token(g(n)): the argument of h is not there when g is called."""
    f = _Fn("f", 1)
    g = f.add(T.OP_CALLFN, [f.add(T.OP_IN)], imm=2)
    h = f.add(T.OP_CALLFN, [f.add(T.OP_TREE_LEFT, [g])], imm=3)
    f.add(T.OP_OUT, [f.add(T.OP_ADD, [h, f.add(T.OP_TREE_TOKEN, [g])])])
    F = _chain(9)
    return ([_result(1, 1).desc(), f.desc(), _framed("g", 2, 1).desc(), _framed("h", 3, 50).desc()], 0), F, \
        [(n,) for n in range(18)], lambda n: F.left[n + 1] + 50 + F.token[n + 1]


def entry_behind_a_switch_on_a_call():
    """f(n) = let s = g(n) < 5 in (if s then h(right(n)) else h(n)) + k(token(n)): the argument of h waits for g."""
    f = _Fn("f", 1)
    n = f.add(T.OP_IN)
    p = f.add(T.OP_LT, [f.add(T.OP_CALLFN, [n], imm=2), f.add(T.OP_CONST, imm=5)])
    s = f.add(T.OP_SWITCH, [p, n])
    a = f.add(T.OP_CALLFN, [f.add(T.OP_TREE_RIGHT, [(s[0], 0)])], imm=3)
    b = f.add(T.OP_CALLFN, [(s[0], 1)], imm=3)
    k = f.add(T.OP_CALLFN, [f.add(T.OP_TREE_TOKEN, [n])], imm=2)
    f.add(T.OP_OUT, [f.add(T.OP_ADD, [f.add(T.OP_MERGE, [a, b]), k])])
    F = _chain(9)
    return ([_result(1, 1).desc(), f.desc(), _framed("g", 2, 1).desc(), _framed("h", 3, 50).desc()], 0), F, \
        [(n,) for n in range(19)], lambda n: (F.right[n] if n + 1 < 5 else n) + 50 + F.token[n] + 1


def entry_of_what_may_be_a_call():
    """f(v, c) = h(left(if c < 1 then v else g(v))): the argument of h is there at once, or waits for g."""
    f = _Fn("f", 2)
    v, c = f.add(T.OP_IN, imm=0), f.add(T.OP_IN, imm=1)
    s = f.add(T.OP_SWITCH, [f.add(T.OP_LT, [c, f.add(T.OP_CONST, imm=1)]), v])
    w = f.add(T.OP_MERGE, [(s[0], 0), f.add(T.OP_CALLFN, [(s[0], 1)], imm=2)])
    f.add(T.OP_OUT, [f.add(T.OP_CALLFN, [f.add(T.OP_TREE_LEFT, [w])], imm=3)])
    F = _chain(9)
    return ([_result(2, 1).desc(), f.desc(), _framed("g", 2, 1).desc(), _framed("h", 3, 50).desc()], 0), F, \
        [(v, c) for v in range(18) for c in (0, 1)], lambda v, c: F.left[v + c] + 50


def waiting_calls_with_entries_as_arguments():
    """f(n) = g(n) + g(left(n)) + h(left(n)) + h(isleaf(n)) + h(right(n)): calls that wait, two of them with the same
    argument, one with an entry that is a truth value; g(x) is done in place for x >= 1000 only."""
    f = _Fn("f", 1)
    n = f.add(T.OP_IN)
    left = f.add(T.OP_TREE_LEFT, [n])
    y = f.add(T.OP_CALLFN, [n], imm=2)
    for callee, arg in ((2, left), (3, left), (3, f.add(T.OP_TREE_ISLEAF, [n])), (3, f.add(T.OP_TREE_RIGHT, [n]))):
        y = f.add(T.OP_ADD, [y, f.add(T.OP_CALLFN, [arg], imm=callee)])
    f.add(T.OP_OUT, [y])
    F = _chain(9)
    return ([_result(1, 1).desc(), f.desc(), _framed("g", 2, 1).desc(), _framed("h", 3, 50).desc()], 0), F, \
        [(n,) for n in range(19)], lambda n: n + 1 + F.left[n] + 1 + F.left[n] + 50 + (F.left[n] < 0) + 50 + F.right[n] + 50


def bad_index_in_result():
    """result(n) = token(n): the instance that names no node is also the last to end."""
    r = _Fn("result", 1)
    r.add(T.OP_OUT, [r.add(T.OP_TREE_TOKEN, [r.add(T.OP_IN)])])
    return ([r.desc()], 0), _chain(9), [-1, -1000, -2, 19, 500]


def bad_index_from_a_call():
    """entry_of_a_calls_result with nodes that do not exist, which the sweep after the call of g meets first."""
    prog, F, _, _ = entry_of_a_calls_result()
    return prog, F, [18, 19, 500, 998]


def bad_index_through_calls():
    """waiting_calls_with_entries_as_arguments with nodes that do not exist: every sweep reads their entries."""
    prog, F, _, _ = waiting_calls_with_entries_as_arguments()
    return prog, F, [-1000, -2, 19, 500]


def fib_value(n):
    a, b = 0, 1
    for _ in range(n):
        a, b = b, a + b
    return a


def _fib_as(index):
    """fib as the function of that number."""
    (_, (name, n_params, nodes)), _ = programs.fib()
    return (name, n_params, [(op, ins, index if op == T.OP_CALLFN else imm) for op, ins, imm in nodes])


def fib_below_a_chain():
    """f(n, m) = if n < 1 then fib(m - 6) + fib(m) else 1 + f(n - 1, m): a program and its reference."""
    f = _Fn("f", 2)
    n, m, one = f.add(T.OP_IN, imm=0), f.add(T.OP_IN, imm=1), f.add(T.OP_CONST, imm=1)
    p = f.add(T.OP_LT, [n, one])
    sn, sm = f.add(T.OP_SWITCH, [p, n]), f.add(T.OP_SWITCH, [p, m])
    a = f.add(T.OP_CALLFN, [f.add(T.OP_SUB, [(sm[0], 0), f.add(T.OP_CONST, imm=6)])], imm=2)
    b = f.add(T.OP_CALLFN, [(sm[0], 0)], imm=2)
    c = f.add(T.OP_ADD, [one, f.add(T.OP_CALLFN, [f.add(T.OP_SUB, [(sn[0], 1), one]), (sm[0], 1)], imm=1)])
    f.add(T.OP_OUT, [f.add(T.OP_MERGE, [f.add(T.OP_ADD, [a, b]), c])])
    return ([_result(2, 1).desc(), f.desc(), _fib_as(2)], 0), lambda n, m: n + (m - 6 if m < 6 else fib_value(m - 6)) + fib_value(m)


def fibs_along_a_chain():
    """f(n, c, m) = if n < 1 then fib(m) else if c < 1 then f(n - 1, 2, m) + fib(m) else 1 + f(n - 1, c - 1, m): every third
    frame of a chain has a second call; a program and its reference."""
    f = _Fn("f", 3)
    n, c, m = (f.add(T.OP_IN, imm=k) for k in range(3))
    one, two = f.add(T.OP_CONST, imm=1), f.add(T.OP_CONST, imm=2)
    sn, sc, sm = (f.add(T.OP_SWITCH, [f.add(T.OP_LT, [n, one]), v]) for v in (n, c, m))
    base = f.add(T.OP_CALLFN, [(sm[0], 0)], imm=2)
    tn, tc, tm = (f.add(T.OP_SWITCH, [f.add(T.OP_LT, [(sc[0], 1), one]), (s[0], 1)]) for s in (sn, sc, sm))
    a = f.add(T.OP_CALLFN, [f.add(T.OP_SUB, [(tn[0], 0), one]), f.add(T.OP_ADD, [(tc[0], 0), two]), (tm[0], 0)], imm=1)
    b = f.add(T.OP_CALLFN, [(tm[0], 0)], imm=2)
    d = f.add(T.OP_CALLFN, [f.add(T.OP_SUB, [(tn[0], 1), one]), f.add(T.OP_SUB, [(tc[0], 1), one]), (tm[0], 1)], imm=1)
    f.add(T.OP_OUT, [f.add(T.OP_MERGE, [base, f.add(T.OP_ADD, [a, b]), f.add(T.OP_ADD, [one, d])])])

    def ref(n, c, m):
        total = fib_value(m)
        for _ in range(n):
            total, c = (total + fib_value(m), 2) if c < 1 else (total + 1, c - 1)
        return total
    return ([_result(3, 1).desc(), f.desc(), _fib_as(2)], 0), ref


# name -> program, forest, arguments, reference; the vector results are rows of E
VECTOR = {"embed_under_every_tag": embed_under_every_tag}
INTEGER = {p.__name__: p for p in (one_of_two_entries, entries_under_an_argument, constant_nodes, entry_of_a_calls_result,
                                   entry_behind_a_switch_on_a_call, entry_of_what_may_be_a_call,
                                   waiting_calls_with_entries_as_arguments)}
# name -> program, forest, arguments that name a node that does not exist
BAD_INDEX = {p.__name__: p for p in (bad_index_in_result, bad_index_from_a_call, bad_index_through_calls)}


def fib_at_every_frame_of_a_chain(fib_first):
    """f(n, m) = fib(m) + f(n - 1, m) down to f(0, m) = fib(m), either call first: a program and its reference."""
    f = _Fn("f", 2)
    n, m, one = f.add(T.OP_IN, imm=0), f.add(T.OP_IN, imm=1), f.add(T.OP_CONST, imm=1)
    sn, sm = (f.add(T.OP_SWITCH, [f.add(T.OP_LT, [n, one]), v]) for v in (n, m))
    base = f.add(T.OP_CALLFN, [(sm[0], 0)], imm=2)
    two = {}
    for first in (fib_first, not fib_first):
        two[first] = f.add(T.OP_CALLFN, [(sm[0], 1)], imm=2) if first else \
            f.add(T.OP_CALLFN, [f.add(T.OP_SUB, [(sn[0], 1), one]), (sm[0], 1)], imm=1)
    f.add(T.OP_OUT, [f.add(T.OP_MERGE, [base, f.add(T.OP_ADD, [two[True], two[False]])])])
    return ([_result(2, 1).desc(), f.desc(), _fib_as(2)], 0), lambda n, m: (n + 1) * fib_value(m)
