"""Properties of the compiled kernels that no numerical test can see, checked on the
assembly hipcc emits for gfx950 (no GPU needed).

* The prompt-scoring passes and the prompt attention run two wave groups one phase apart: a step
  is `matrix phase, barrier, vector phase, barrier`.  Pass 1's vector phase touches no
  memory, so only a data dependence on the closing barrier keeps the compiler from
  scheduling its arithmetic behind that barrier (a build did exactly that: the
  results stay right, the two groups then take turns and the pass is ~10 % slower).
  Every steady-state loop must therefore have its exponentials between its barriers.
* The kernels the benchmark times must not spill registers to scratch memory.
* A step's output sums halve the columns a lane is left with at every exchange between lanes;
  with all columns in all lanes they take three times the instructions, which steps of many
  heads and few slots pay for.
"""
import os
import re
import subprocess
from collections import Counter

import pytest

from paper_2306_14048_amd import build as hb


def device_asm(src: str, tmp_path) -> str:
    out = os.path.join(str(tmp_path), src.replace(".hip", ".s"))
    cmd = ["hipcc", *hb.FLAGS, "--cuda-device-only", "-S", os.path.join(hb.CSRC, src), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return open(out).read()


def functions(asm: str):
    """name -> list of basic blocks, each a list of instruction lines"""
    lines = asm.split("\n")
    fns = {}
    for i, l in enumerate(lines):
        m = re.match(r"^(_Z\S+):", l)
        if not m:
            continue
        blocks, cur = [], []
        for x in lines[i + 1:]:
            if x.startswith(".Lfunc_end"):
                break
            if re.match(r"^\.LBB\d+_\d+:", x):
                if cur:
                    blocks.append(cur)
                cur = []
                continue
            t = x.strip()
            if t and not t.startswith(";") and not t.startswith("."):
                cur.append(t)
        if cur:
            blocks.append(cur)
        fns[m.group(1)] = blocks
    return fns


def metadata(asm: str):
    """name -> {vgpr_count, vgpr_spill_count, ...} from the code object metadata"""
    meta, name = {}, None
    for l in asm.split("\n"):
        m = re.match(r"^\s+\.name:\s+(\S+)", l)
        if m:
            name = m.group(1)
            meta[name] = {}
        m = re.match(r"^\s+\.(vgpr_count|vgpr_spill_count|sgpr_spill_count|private_segment_fixed_size):\s+(\d+)", l)
        if m and name:
            meta[name][m.group(1)] = int(m.group(2))
    return meta


@pytest.fixture(scope="module")
def scores_asm(tmp_path_factory):
    return device_asm("prefill_scores.hip", tmp_path_factory.mktemp("isa"))


@pytest.fixture(scope="module")
def attention_asm(tmp_path_factory):
    return device_asm("prefill_attention.hip", tmp_path_factory.mktemp("isa"))


def test_vector_phase_of_the_scoring_passes_sits_between_the_barriers(scores_asm):
    # eight waves: 3 element types x 2 head dims x 2 passes; two groups of four waves one phase apart (16-bit,
    # d = 128, last template argument set): 2 types x (column sums, statistics with keys in one and in two places)
    fns = {n: b for n, b in functions(scores_asm).items()
           if "prefill_pass_kernel" in n or re.search(r"prefill_pass4_kernelI\w+?Lb1EEEv", n)}
    assert len(fns) == 12 + 6
    for name, blocks in fns.items():
        loops = 0
        for ins in blocks:
            ops = [x.split()[0] for x in ins]
            if ops.count("s_barrier") != 2 or not any("mfma" in o for o in ops):
                continue
            loops += 1
            first = ops.index("s_barrier")
            second = len(ops) - 1 - ops[::-1].index("s_barrier")
            last_mfma = max(i for i, o in enumerate(ops) if "mfma" in o)
            exps = [i for i, o in enumerate(ops) if o.startswith("v_exp_f32")]
            assert last_mfma < first, name
            between = [i for i in exps if first < i < second]
            assert len(between) >= 16 and not [i for i in exps if i > second], \
                "%s: %d exponentials between the barriers, %d behind the second" % (
                    name, len(between), len([i for i in exps if i > second]))
        assert loops >= 1, name                             # the unmasked steady-state loop was found


def test_phases_of_the_attention_groups_sit_between_their_barriers(attention_asm):
    """The attention with its groups one phase apart: all matrix instructions of a step in front of its
    middle barrier, the softmax behind it and in front of the closing one."""
    fns = {n: b for n, b in functions(attention_asm).items() if re.search(r"prefill_attn_kernelI\w+?ELb1EEEv", n)}
    assert len(fns) == 2 * 2 * 2                            # types, head dims, keys in one and in two places
    for name, blocks in fns.items():
        middle = closing = 0
        for ins in blocks:
            ops = [x.split()[0] for x in ins]
            bars, mfmas, exps = ([i for i, o in enumerate(ops) if f(o)] for f in
                                 (lambda o: o == "s_barrier", lambda o: "mfma" in o, lambda o: o.startswith("v_exp_f32")))
            assert len(bars) <= 1 or not (mfmas or len(exps) >= 32), name
            if mfmas and bars:
                assert max(mfmas) < bars[0] and all(i > bars[0] for i in exps), name
                middle += 1
            elif mfmas:
                assert not exps, name
            elif len(exps) >= 32:                           # a tile's exponentials
                assert len(exps) == 32 and (not bars or max(exps) < bars[0]), name
                closing += len(bars)                        # (a masked tile's barrier is in the next block)
        assert middle >= 1 and closing >= 1, (name, middle, closing)


def test_benchmarked_kernels_do_not_spill(scores_asm, tmp_path):
    meta = metadata(scores_asm)
    checked = 0
    for name, m in meta.items():
        # 16-bit element types (1 = f16, 2 = bf16): the shapes of every workload in the benchmark
        if "prefill_pass_kernel" in name and ("ILi1E" in name or "ILi2E" in name):
            assert m["vgpr_spill_count"] == 0 and m["vgpr_count"] <= 128, (name, m)
            checked += 1
    assert checked == 8
    meta = metadata(device_asm("decode_step.hip", tmp_path))
    checked = 0
    for name, m in meta.items():
        if "decode_resident_kernel" in name:
            # two workgroups of eight waves per CU need <= 128 registers per lane
            assert m["vgpr_spill_count"] == 0 and m["vgpr_count"] <= 128, (name, m)
            checked += 1
    assert checked >= 8


def test_builds_of_the_selection_do_not_spill(tmp_path):
    """Nor do those of a compression (a chunked prompt's is one with several workgroups per head inside the cache)."""
    checked = Counter()
    for name, m in metadata(device_asm("select_gather.hip", tmp_path)).items():
        # row bytes, 4-bit type, pattern, keys, in place (0 no, 1 by one workgroup, 2 by columns), threads
        shape = re.search(r"select_gather_kernelILi\d+ELi\w+ELb\dELi\d+ELi(\d)ELi(\d+)E", name)
        if shape:
            assert m["vgpr_spill_count"] == 0 and m["private_segment_fixed_size"] == 0, (name, m)
            checked[shape[1]] += 1
    assert checked["0"] >= 60 and checked["1"] == checked["2"] >= 27, checked


def test_output_sums_halve_their_columns(tmp_path):
    checked = 0
    for src in ("decode_step.hip", "decode_split.hip"):
        for name, blocks in functions(device_asm(src, tmp_path)).items():
            m = re.search(r"decode_(?:resident|chunked|part)_kernelILi(\d)ELi(\d+)E", name)
            if not m:
                continue
            f32, d = m[1] == "0", int(m[2])
            # columns of a lane: 4 or 8; exchanges over 16 lanes (rows of up to 16 lanes) and over 32
            want = {(True, 64): 2 + 1, (True, 128): 2, (False, 64): 4 + 2, (False, 128): 4 + 2}[(f32, d)]
            ops = [x.split()[0] for ins in blocks for x in ins]
            assert sum(o.startswith("v_permlane") for o in ops) == want, name
            checked += 1
    assert checked >= 100


def test_masks_of_the_column_sums_take_one_comparison_per_product(scores_asm):
    """A masked tile tests both ends of the stream as one range."""
    checked = 0
    for name, blocks in functions(scores_asm).items():
        # (name ends: G, TWO, COLSUM, SKEW / COLSUM)
        if not re.search(r"prefill_pass_kernelILi\dELi\d+ELi\dELb1EEE|prefill_pass4_kernelILi\dELi\d+ELi\dELi\dELb0ELb1ELb\dE", name):
            continue
        f32_128 = "ILi0ELi128E" in name
        for ins in blocks:
            ops = [x.split()[0] for x in ins]
            exps, cmps = (sum(o.startswith(p) for o in ops) for p in ("v_exp_f32", "v_cmp"))
            if exps >= 16:
                assert cmps <= (16 if f32_128 else 32) + 2, (name, cmps, exps)
                checked += 1
    assert checked >= 40
