"""CPU-only checks of the C boundary: the library loads, exports every symbol the header declares, and its host-side
logic (configuration checks, workspace sizing, dropout keys) behaves.  No kernel is launched here."""
import ctypes as C
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def T():
    import paper_1904_01038_amd as T
    if not os.path.exists(T.lib_path()):
        from paper_1904_01038_amd import build
        build.build(verbose=False)
    return T


def declared_functions():
    text = open(os.path.join(ROOT, "include", "tfm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tfm_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(T):
    names = declared_functions()
    assert len(names) >= 25 and "tfm_train_step" in names and "tfm_apply_update" in names and "tfm_create" in names
    lib = C.CDLL(T.lib_path())
    missing = [n for n in names if not hasattr(lib, n)]
    assert not missing, missing


def test_workspace_sizing_and_config_validation(T):
    from synth import PRESETS, count_params
    L = T.lib()
    n = C.c_size_t()
    sizes = {}
    for name, prec in [("tiny", T.FP32), ("base", T.BF16), ("big", T.FP16), ("lm16", T.FP16)]:
        cfg = T.make_config(PRESETS[name], precision=prec, max_sentences=256, max_len=128, max_tokens=4096)
        assert L.tfm_workspace_bytes(C.byref(cfg), C.byref(n)) == 0
        sizes[name] = n.value
        # at least master + two moments + accumulator in fp32
        assert n.value >= 16 * count_params(PRESETS[name])
    assert sizes["tiny"] < sizes["base"] < sizes["big"]
    assert sizes["big"] < 12 * 2 ** 30              # a small fraction of 288 GB
    bad = [dict(d_model=100), dict(n_heads=3), dict(dec_layers=0), dict(vocab=2), dict(dropout=1.0), dict(precision=7),
           dict(max_tokens=0), dict(label_smoothing=-0.1), dict(init_loss_scale=0.0), dict(scale_window=0), dict(pad_id=-1)]
    for change in bad:
        cfg = T.make_config(PRESETS["tiny"], precision=T.FP32, max_sentences=8, max_len=16, max_tokens=128)
        for k, v in change.items():
            setattr(cfg, k, v)
        assert L.tfm_workspace_bytes(C.byref(cfg), C.byref(n)) == -1, change
        assert L.tfm_last_error(None)
    # a null workspace is rejected before anything touches the GPU
    cfg = T.make_config(PRESETS["tiny"], precision=T.FP32, max_sentences=8, max_len=16, max_tokens=128)
    h = C.c_void_p()
    assert L.tfm_create(C.byref(cfg), None, 0, None, C.byref(h)) == -1


def test_dropout_site_keys_match_the_oracle(T):
    from oracle.transformer import dropout_key, site_id
    L = T.lib()
    rng = np.random.default_rng(0)
    for _ in range(50):
        seed, step = int(rng.integers(0, 2 ** 62)), int(rng.integers(0, 2 ** 40))
        stream, layer, sub = int(rng.integers(0, 2)), int(rng.integers(-1, 16)), int(rng.integers(0, 3))
        assert L.tfm_dropout_key(seed, step, stream, layer, sub) == int(dropout_key(seed, step, site_id(stream, layer, sub)))


def test_parameter_list_matches_the_shared_shape_module(T):
    # the C side enumerates its parameters only for a live context; compare the count it needs with the shape module
    from synth import PRESETS, param_specs
    for name in ("tiny", "big", "lm16"):
        specs = param_specs(PRESETS[name])
        assert len({n for n, _ in specs}) == len(specs)
        assert specs[0][0] == "embed"


def assembly(source):
    from paper_1904_01038_amd import build
    r = subprocess.run(["hipcc", *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_decoding_scores_are_formed_by_32_bit_multiply_adds():
    """v_dot2_f32_f16 truncates small terms against a fixed floor (1.6e-5 of a result with subnormal keys, where 32-bit FMAs are
    off by 6e-8), and the compiler forms it by itself from FMAs whose factors it sees as halves."""
    text = assembly("decode.hip")
    assert "decode_attention64_kernel" in text and "v_dot2" not in text


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_no_instance_of_the_few_row_product_spills_registers():
    """An instance that no call reaches is not built: those are the ones that would not fit."""
    spills = re.findall(r"\.name: +(\S*gemm_thin_kernel\S*).*?\.vgpr_spill_count: +(\d+)", assembly("gemm_thin.hip"), flags=re.S)
    assert len(spills) >= 50
    assert [name for name, n in spills if int(n)] == []


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_decoding_attention_fetches_the_rows_of_a_chunk_together():
    """The rows' places in the caches come from a table: 4 or 8 words, asked for one after the other and waited for once.  (A wait
    behind every word made a chunk of 64 positions nine trips to memory.)"""
    kernels = re.findall(r"^(\S*decode_attention64_kernel\S*):(.*?)s_endpgm", assembly("decode.hip"), flags=re.S | re.M)
    assert len(kernels) == 4
    for name, body in kernels:
        lines = [l.strip() for l in body.splitlines() if l.strip() and not l.strip().startswith((";", "."))]
        waits = sum(a.startswith("global_load_dword v") and b.startswith("s_waitcnt vmcnt(0)") for a, b in zip(lines, lines[1:]))
        assert waits <= 1, (name, waits)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_masks_of_a_product_are_fetched_together():
    """Input gradients behind a ReLU: a wavefront of the 192x256 tile reads back 12 pieces, whose masks are asked for ahead of the
    first store (between the stores, which may alias them, each would be waited for: 39.8 us against 36.6)."""
    kernels = re.findall(r"^(\S*gemm_mfma_kernel\S*Li192ELi256E\S*):(.*?)s_endpgm", assembly("gemm_mfma.hip"), flags=re.S | re.M)
    assert len(kernels) >= 4
    for name, body in kernels:
        runs = [len(re.findall("global_load_dwordx4", part)) for part in body.split("global_store")]
        assert max(runs) >= 12, (name, max(runs))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_layernorm_backward_fetches_a_row_with_its_slices_together():
    """512 or 1024 columns in 2-byte types: the row's operands and slices (2 x 16 bytes each, `add` apart) are asked for ahead of the first wait.  (In bf16
    they came in up to 20 groups of loads.)"""
    kernels = re.findall(r"^\S*layernorm_bwd_row_kernelI(\S*?)Li([12])ELi4ELi([248])EEE\S*:(.*?)s_endpgm", assembly("norm.hip"), flags=re.S | re.M)
    assert len(kernels) == 12
    for dtype, chunks, slices, body in kernels:
        ahead = body.split("s_waitcnt vmcnt", 1)[0]
        assert len(re.findall("global_load_dwordx4", ahead)) >= int(chunks) * (3 + 2 * int(slices)), (dtype, chunks, slices)
