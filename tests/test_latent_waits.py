"""Result distance of the latent kernel's matrix products, in the compiled code.

The products are written as instructions, so the compiler does not see that
their accumulators arrive late: every read of one must lie behind the
product_wait() (two `s_nop 15`) that follows the last product on its way. The
kernel is compiled to assembly here (no GPU) and each path that ends in a read
is followed backwards until the wait."""
import re
import subprocess

import pytest

from paper_2606_04415_amd import build as B

READ = re.compile(r"v_accvgpr_(?:read|mov)\w* \w+, (?:a(\d+)|\\reg)$")   # \reg: the accumulators of a repeated line
PRODUCT = re.compile(r"v_mfma\S+ a\[(\d+):(\d+)\]")
BRANCH = re.compile(r"s_(c?branch)\w* (\.L\w+)")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "latent.s"
    subprocess.run([B.hipcc()] + B.common_flags() + ["--cuda-device-only", "-S", B.CSRC + "/latent.hip", "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    found, name = {}, None
    for line in out.read_text().splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"_ZN\S*latent_kernel\S*:$", line):
            name = line[:-1]
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line and (not line.startswith(".") or line.startswith(".L")):
            found[name].append(line)
    return found


def early_reads(lines):
    """Reads of a product's accumulator that some path reaches without a wait."""
    at = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    before = [[] for _ in lines]
    for i, l in enumerate(lines):
        m = BRANCH.match(l)
        if m:
            before[at[m[2]]].append(i)
        if i + 1 < len(lines) and not l.startswith("s_branch") and not l.startswith("s_endpgm"):
            before[i + 1].append(i)
    results = {r for l in lines for m in [PRODUCT.match(l)] if m for r in range(int(m[1]), int(m[2]) + 1)}
    assert len(results) == 256, "the accumulators of 512 value columns"
    reads = [i for i, l in enumerate(lines) for m in [READ.match(l)] if m and (m[1] is None or int(m[1]) in results)]
    assert reads
    early = []
    for i in reads:
        seen, todo = set(), list(before[i])
        while todo:
            j = todo.pop()
            if j in seen:
                continue
            seen.add(j)
            if lines[j] == "s_nop 15" and j and lines[j - 1] == "s_nop 15":
                continue
            if PRODUCT.match(lines[j]):
                early.append((i, lines[i], lines[j]))
                break
            todo += before[j]
    return early


def test_every_read_of_an_accumulator_is_behind_the_wait(kernels):
    assert len(kernels) == 4   # decode and prefill, pages of 16 and 64
    for name, lines in kernels.items():
        assert not early_reads(lines), name


def test_a_read_ahead_of_the_wait_is_found(kernels):
    """The check itself: the first wait of a kernel taken out of the text."""
    lines = list(next(iter(kernels.values())))
    last = max(i for i, l in enumerate(lines) if l == "s_nop 15" and lines[i - 1] == "s_nop 15")
    assert early_reads(lines[:last - 1] + lines[last + 1:])


def test_latent_kernels_hold_everything_in_registers(tmp_path):
    """A spilled register that is read back inside the tile loop waits for every
    load in flight, which undoes the loads ahead."""
    spills = {}
    for src in ("attention.hip", "latent.hip"):
        out = tmp_path / "k.s"
        subprocess.run([B.hipcc()] + B.common_flags() + ["--cuda-device-only", "-S", f"{B.CSRC}/{src}", "-o", str(out)],
                       check=True, capture_output=True, timeout=300)
        for m in re.finditer(r"^(_ZN\S*(?:rowpar_kernelILi576|latent_kernel)\S*):.*?; ScratchSize: (\d+)", out.read_text(),
                             re.S | re.M):
            spills[m[1]] = int(m[2])
    assert len(spills) == 8   # 64 and 128 rows, decode and prefill, pages of 16 and 64
    assert not any(spills.values()), spills
