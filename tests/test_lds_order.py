"""The order of memory accesses in the step kernels, read from the source.

Shared memory: in the loop over the stages, as it stands in
the source, every two accesses that different waves may make to one array, one
of them a write, have a barrier between them, also across the end of a stage
and the start of the next.  A missing barrier shows in no result reliably (a
wave would have to fall behind by most of a stage), so the order is read here.

The loop's text is taken as straight-line code: `if constexpr` and the collision
switch are resolved for each kind of kernel, other branches count as taken.

Populations stepped in place (App. A): lanes without a point of their own read
another lane's, so that lane has to be of the same wave."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_1708_03249_amd", "csrc")
LOOP = "for (int it = 0; it < A.nsteps * A.nst; ++it) {"


def closing(text, i, pair="{}"):
    """Index of the bracket that closes the one at i."""
    depth = 0
    for k in range(i, len(text)):
        depth += (text[k] == pair[0]) - (text[k] == pair[1])
        if depth == 0:
            return k
    raise ValueError("unbalanced")


def statement(text, i):
    """End of the statement that starts at i (a block, or up to a semicolon)."""
    while text[i].isspace():
        i += 1
    return closing(text, i) + 1 if text[i] == "{" else text.index(";", i) + 1


def resolve(text, env):
    """The text without the branches that `env` rules out."""
    out, pos = [], 0
    for m in iter(lambda: re.compile(r"\bif (?:constexpr )?\(").search(text, pos), None):
        par = m.end() - 1
        end = closing(text, par, "()")
        cond = text[par + 1:end]
        if "constexpr" not in m.group() and cond.strip() != "collide":
            out.append(text[pos:end + 1])
            pos = end + 1
            continue
        expr = re.sub(r"\w+<[^<>]*>\(\)", lambda c: c.group().split("<")[0], cond)
        expr = re.sub(r"!(?!=)", " not ", expr).replace("&&", " and ").replace("||", " or ").replace("PREC", "'PREC'")
        taken = bool(eval(expr, {}, env))
        yes_end = statement(text, end + 1)
        out.append(text[pos:m.start()])
        if taken:
            out.append(resolve(text[end + 1:yes_end], env))
        pos = yes_end
        other = re.compile(r"\s*else\b").match(text, pos)
        if other:
            no_end = statement(text, other.end())
            if re.compile(r"\s*if\b").match(text, other.end()):   # else if: the whole chain
                chain = other.end()
                while True:
                    e = statement(text, closing(text, text.index("(", chain), "()") + 1)
                    nxt = re.compile(r"\s*else\b").match(text, e)
                    if not nxt:
                        break
                    chain = nxt.end()
                    if not re.compile(r"\s*if\b").match(text, chain):
                        e = statement(text, chain)
                        break
                no_end = e
            if not taken:
                out.append(resolve(text[other.end():no_end], env))
            pos = no_end
    out.append(text[pos:])
    return "".join(out)


ACCESS = re.compile(r"__syncthreads\(\)|\b(s_y|s_nw|s_geq|ge|s_tile)\[|\bpart\(|mfma_(?:tile|force)<[^;]*\bs_tile\b")


def events(text):
    for m in ACCESS.finditer(text):
        word = m.group()
        if word.startswith("__"):
            yield "barrier", ""
        elif word.startswith("mfma") or word == "s_tile[":
            yield "tile", "own"
        else:
            pair = "()" if word == "part(" else "[]"
            rest = text[closing(text, m.end() - 1, pair) + 1:].lstrip()
            kind = "write" if rest.startswith("=") and not rest.startswith("==") else "read"
            if word == "part(":   # one array per sum, the second argument
                which = text[m.end():closing(text, m.end() - 1, pair)].split(",")[1]
                for q in re.findall(r"\d", which):
                    yield "part" + q, kind
            else:
                yield {"ge[": "s_geq"}.get(word, word[:-1]), kind


def conflicts(loop, alias, collide):
    """Pairs of accesses of two consecutive stages with no barrier between."""
    def clash(a, b):
        if a[0] == b[0]:
            return a[0] != "tile" and {a[1], b[1]} == {"read", "write"}
        return alias and {a[0][:4], b[0][:4]} == {"part", "tile"}
    found, open_ = set(), []
    once = list(events(loop))
    assert ("part0", "write") in once and any(e[0] == "barrier" for e in once)
    for e in once + once:
        if e[0] == "barrier":
            open_ = []
            continue
        if e[0] == "s_geq" and not collide:
            continue   # zeros from both waves of a half, read by the lane that wrote them
        found |= {(a, e) for a in open_ if clash(a, e)}
        open_.append(e)
    return found


def stage_loop(name):
    with open(os.path.join(CSRC, name)) as fh:
        text = re.sub(r"//[^\n]*", "", fh.read())
    i = text.index(LOOP) + len(LOOP) - 1
    return text[i:closing(text, i) + 1]


def fp64_env(quad, mfma, nfun, slots, collide):
    own = mfma and nfun == 1 and slots == 1
    return dict(H=16 if mfma else 8, QUAD=quad, kMfma=mfma, NFUN=nfun, SLOTS=slots, collide=collide, kOwnEq=own, kAlias=mfma and not own,
                kDefer=mfma and slots == 2)


@pytest.mark.parametrize("collide", [True, False])
@pytest.mark.parametrize("slots", [1, 2])
@pytest.mark.parametrize("nfun", [1, 2])
@pytest.mark.parametrize("quad,mfma", [(0, False), (0, True), (1, False)])
def test_fp64_step_kernel(quad, mfma, nfun, slots, collide):
    env = fp64_env(quad, mfma, nfun, slots, collide)
    assert not conflicts(resolve(stage_loop("fused_kernels.hpp"), env), env["kAlias"], collide)


@pytest.mark.parametrize("collide", [True, False])
@pytest.mark.parametrize("slots", [1, 2])
@pytest.mark.parametrize("nfun", [1, 2])
@pytest.mark.parametrize("mfma_k,alias", [(False, False), (True, False), (True, True)])
def test_mixed_step_kernel(mfma_k, alias, nfun, slots, collide):
    env = dict(H=16 if alias else 8, NFUN=nfun, SLOTS=slots, kMfmaEq=False, kMfmaK=mfma_k, kAlias=alias, collide=collide)
    assert not conflicts(resolve(stage_loop("mixed_kernels.hpp"), env), alias, collide)


def test_a_removed_barrier_is_found():
    env = fp64_env(1, False, 2, 2, True)
    loop = resolve(stage_loop("fused_kernels.hpp"), env)
    for m in re.finditer(r"__syncthreads\(\);", loop):
        assert conflicts(loop[:m.start()] + loop[m.end():], False, True), loop[m.start() - 200:m.end()]


def test_waves_without_a_point_read_none():
    with open(os.path.join(CSRC, "multi_steps.hpp")) as fh:
        text = re.sub(r"//[^\n]*", "", fh.read())
    body = text[text.index("multi_steps_kernel(MultiArgs A)"):]
    load = body.index("A.in + pt * V")
    assert "pt0 < A.npts ? pt0 : A.npts - 1" in body[:load]   # the last point stands in
    leave = body.index("if (pt_wave >= A.npts) return;")
    last_barrier = max(m.start() for m in re.finditer(r"__syncthreads\(\)", body[:body.index("inline size_t")]))
    assert last_barrier < leave < load
