"""Programs over a forest whose generated lanes are easy to get wrong, each with a small forest, arguments and a plain
Python function that says what an instance gives: the value, or for vector results the token whose row it is."""
from paper_2410_20225_amd import tdf as T
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


# name -> program, forest, arguments, reference; the vector results are rows of E
VECTOR = {"embed_under_every_tag": embed_under_every_tag}
