"""Arrays in LDS with a slot per wavefront of a block: a block of T threads has
ceil(T / 64) wavefronts, the last of them perhaps part of one, and each writes its
slot.  Read from the sources: every ``__shared__`` array whose size is a number of
threads over 64 is compared with the block its kernel is bounded to."""
import glob
import os
import re

import paper_1803_07491_amd as P

CSRC = os.path.join(os.path.dirname(os.path.abspath(P.__file__)), "csrc")


def _constants(texts):
    """Integer constants of the sources, as far as they evaluate."""
    pairs = []
    for text in texts:
        for decl in re.findall(r"constexpr\s+(?:int|long|unsigned)\s+([^;{}()]*(?:\([^;{}]*\)[^;{}]*)?);", text):
            pairs += re.findall(r"(\w+)\s*=\s*([^,=]+)", decl)
    known = {}
    for _ in range(4):
        for name, expr in pairs:
            value = _value(expr, known)
            if value is not None:
                known[name] = value
    return known


def _value(expr, known):
    try:
        return int(eval(expr.replace("/", "//"), {"__builtins__": {}}, dict(known)))
    except Exception:
        return None


def _kernels(text):
    """(bound expression, name, text from the bound to the end of the kernel)."""
    for m in re.finditer(r"__launch_bounds__\(", text):
        start, depth = m.end(), 1
        end = start
        while depth:
            depth += {"(": 1, ")": -1}.get(text[end], 0)
            end += 1
        stop = text.find("\n}\n", end)
        body = text[end:stop if stop > 0 else len(text)]
        yield text[start:end - 1], (re.search(r"\b(k_\w+|scan_\w+)\s*\(", body) or [None, "?"])[1], body


def test_every_wave_has_a_slot():
    headers = [open(f).read() for f in sorted(glob.glob(os.path.join(CSRC, "*.h")))]
    short, seen = [], 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        known = _constants(headers + [text])
        for bound, name, body in _kernels(text):
            threads = _value(bound, known)
            for decl in re.findall(r"__shared__[^;]*;", body):
                for array, size in re.findall(r"(\w+)\[([^\]]*/ 64\)?)\]", decl):
                    slots = _value(size, known)
                    if threads is None or slots is None:
                        continue
                    seen += 1
                    if slots < -(-threads // 64):
                        short.append((os.path.basename(path), name, array, slots, threads))
    assert seen >= 20
    assert not short, short


def test_block_reductions_run_on_whole_waves():
    """block_combine adds the slots of blockDim.x / 64 wavefronts: its kernels' blocks
    are whole ones."""
    headers = [open(f).read() for f in sorted(glob.glob(os.path.join(CSRC, "*.h")))]
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        known = _constants(headers + [text])
        for bound, name, body in _kernels(text):
            if re.search(r"\b(block_combine|partials_combine|block_sum\w*)\b", body):
                threads = _value(bound, known)
                assert threads is not None and threads % 64 == 0, (os.path.basename(path), name, bound, threads)
                seen += 1
    assert seen >= 8
