"""Waits that a kernel's source has to state itself, read from the gfx950 assembly
that the sources compile to (no GPU needed)."""
import functools
import os
import re
import subprocess
import tempfile

from paper_2608_07814_amd import build as B


@functools.lru_cache(maxsize=None)
def _asm(src):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, src + ".s")
        subprocess.run([B.HIPCC, *B.CFLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", out],
                       check=True, stderr=subprocess.DEVNULL)
        return open(out).read()


def _functions(asm):
    """Name -> lines of every function."""
    out, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            out[name].append(line)
    return out


def test_fp32_ring_waits_for_lds_reads_before_freeing_a_stage():
    """The K loop's barrier frees the stage of the slab before it for direct
    loads of every wavefront, so each wavefront's LDS reads have to be
    complete when it arrives: the wait stands right before the barrier."""
    kernels = {n: f for n, f in _functions(_asm("k_gemm.hip")).items() if "k_gemm_f32m" in n}
    assert len(kernels) == 2
    for name, lines in kernels.items():
        in_loop, block, seen = False, [], 0
        for line in lines:
            if line.startswith(".LBB"):
                in_loop, block = "Loop" in line, []
                continue
            block.append(line.split(";")[0].strip())
            if block[-1] == "s_barrier" and in_loop:
                waits = [b for b in block[:-1] if b.startswith("s_waitcnt")]
                assert waits and "lgkmcnt(0)" in waits[-1], (name, block)
                seen += 1
        assert seen == 1, (name, seen)


def test_swiglu_divides():
    """SiLU in full fp32, whatever format the rows have: every exponential of a
    SwiGLU kernel has its range reduction, and its division the IEEE fix-up
    (a bare hardware exponential and reciprocal are off by 8e-7 at g = -25)."""
    kernels = {n: "\n".join(f) for n, f in _functions(_asm("k_token.hip")).items() if "k_swiglu" in n}
    assert len(kernels) >= 10
    for name, code in kernels.items():
        n = len(re.findall(r"\bv_exp_f32", code))
        assert n > 0 and n == len(re.findall(r"\bv_div_fixup_f32", code)), name
        assert n <= len(re.findall(r"\bv_rndne_f32", code)), name


def test_two_slab_kernels_add_a_half_at_a_time():
    """The skinny kernels that hold a hi/lo pair's fragments at once add the hi
    half's K steps of a slab, then the lo half's, as the kernels that take one
    half per step do, so a product's sum does not depend on which of them runs:
    no two MFMAs in a row read the same weight fragment."""
    kernels = {n: f for n, f in _functions(_asm("k_gemm2.hip")).items()
               if "k_gemm_skinny_mix" in n or "k_gemm_skinnyILi2ELi2E" in n}
    assert len(kernels) == 4
    for name, lines in kernels.items():
        weights = [re.split(r"[\s,]+", line.strip())[3] for line in lines if "v_mfma_f32_32x32x16_bf16" in line]
        assert len(weights) >= 8
        assert all(a != b for a, b in zip(weights, weights[1:])), (name, weights)


def test_large_kmedoids_loads_members_only():
    """Past 128 experts the member sums of the k-medoids read the distance matrix
    from memory: a distance is loaded under its membership branch, right before
    it is added (loading all of a row in batches took 2.5 times as long at 1024
    experts)."""
    kernels = {n: f for n, f in _functions(_asm("k_cluster.hip")).items() if "k_kmedoidsILi1024E" in n}
    assert len(kernels) == 1
    (lines,) = kernels.values()
    code = [c for c in (line.split(";")[0].strip() for line in lines) if c and not c.startswith(".")]
    sums = 0
    for i, c in enumerate(code):
        if c.startswith("v_add_f64") and code[i - 2].startswith("global_load_dwordx2"):
            assert code[i - 1].startswith("s_waitcnt vmcnt(0)")
            assert any(b.startswith("s_cbranch_execz") for b in code[max(0, i - 12):i]), code[i - 12:i]
            sums += 1
        elif c.startswith("v_add_f64"):  # (1 - D: the sum follows its subtraction)
            assert code[i - 1].startswith("v_add_f64") and code[i - 3].startswith("global_load_dwordx2"), code[i - 4:i + 1]
    assert sums >= 2


def test_skinny_kernels_load_shared_weights_plainly():
    """Which weight loads carry the non-temporal hint. Router (its row tiles all
    read the same weights): none, and one step of 6 loads waited for at a time,
    three further ones in flight. Batches of at most 32 tokens (no node has a
    second row tile): each. Else: both kinds, by the node's tiles."""
    kernels = {n: "\n".join(f) for n, f in _functions(_asm("k_gemm2.hip")).items() if "k_gemm_skinny" in n}
    use = {n: int(re.search(r"WeightUseE(\d)E", n).group(1)) for n in kernels}
    assert sorted(use.values()).count(2) == 3 and set(use.values()) == {0, 1, 2}
    for name, code in kernels.items():
        hinted = len(re.findall(r"global_load_lds_dwordx4.* nt", code))
        plain = len(re.findall(r"global_load_lds_dwordx4", code)) - hinted
        # (activations are always plain; a weight slab is 64 rows, an activation slab 32)
        if use[name] == 2:
            assert hinted == 0 and plain > 0, name
        elif use[name] == 0:
            assert hinted >= plain > 0, (name, hinted, plain)
        else:
            assert plain > hinted > 0, (name, hinted, plain)
    (ring,) = [c for n, c in kernels.items() if use[n] == 2 and "k_gemm_skinnyILi4ELi1E" in n]
    assert "s_waitcnt vmcnt(18)" in ring


def test_topk_keeps_eight_wavefronts_per_simd():
    """The top-k of many tokens is bound by instructions that other wavefronts
    hide: at most 64 VGPRs (of 512 per SIMD lane) and nothing in scratch, for
    every number of experts."""
    asm = _asm("k_route.hip")
    vgprs = {m[0]: int(m[1]) for m in re.findall(r"\.set (_Z\w*k_topk\w*)\.num_vgpr, (\d+)", asm)}
    scratch = {m[0]: int(m[1]) for m in re.findall(r"\.set (_Z\w*k_topk\w*)\.private_seg_size, (\d+)", asm)}
    assert len(vgprs) >= 8 and vgprs.keys() == scratch.keys()
    assert max(vgprs.values()) <= 64 and max(scratch.values()) == 0, vgprs
