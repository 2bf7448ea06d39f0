"""CPU checks of the boundary: the library loads, exports every symbol include/mdn.h declares,
and the host-side entry points (no device access) validate their arguments."""
import ctypes
import os
import re

import pytest

from paper_2605_05838_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "mdn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mdn_[a-z_]+)\s*\(", text)))


def test_header_and_binding_agree_on_the_export_list():
    assert declared_symbols() == sorted(binding.EXPORTS)


def test_library_exports_every_declared_symbol():
    lib = binding.load_library()
    for name in declared_symbols():
        assert hasattr(lib, name), name
    assert lib.mdn_version() >= 100
    assert lib.mdn_strerror(0) == b"ok"
    assert b"workspace" in lib.mdn_strerror(-4)


def shape(**kw):
    base = dict(B=2, T=128, H=3, dk=128, dv=128, C=64, dtype=0, scale=0.1)
    base.update(kw)
    return binding.MdnShape(**base)


def test_workspace_query_validates_shapes():
    lib = binding.load_library()
    n = ctypes.c_size_t(0)
    assert lib.mdn_workspace_bytes(ctypes.byref(shape()), 0, ctypes.byref(n)) == 0 and n.value > 0
    fwd = n.value
    assert lib.mdn_workspace_bytes(ctypes.byref(shape()), 1, ctypes.byref(n)) == 0 and n.value > fwd
    # a partial last chunk has chunk blocks like a whole one: more workspace than the full chunks alone
    assert lib.mdn_workspace_bytes(ctypes.byref(shape(T=100)), 0, ctypes.byref(n)) == 0
    ragged = n.value
    assert lib.mdn_workspace_bytes(ctypes.byref(shape(T=64)), 0, ctypes.byref(n)) == 0 and ragged > n.value
    assert lib.mdn_workspace_bytes(ctypes.byref(shape(T=0)), 0, ctypes.byref(n)) == -2
    assert lib.mdn_saved_states_bytes(ctypes.byref(shape(T=100)), ctypes.byref(n)) == 0
    assert n.value == 2 * 3 * 2 * 2 * 128 * 128 * 2                                           # ceil(100 / 64) chunks
    assert lib.mdn_workspace_bytes(ctypes.byref(shape(dk=96, dv=96)), 0, ctypes.byref(n)) == -2
    assert lib.mdn_workspace_bytes(ctypes.byref(shape(C=48)), 0, ctypes.byref(n)) == -2
    # chunk sizes 32 and 16 (Algorithm 1): every chunk runs as a 64-token tile, so 2x / 4x the chunks' workspace plus
    # the padded copies of the tokens; the kept states follow the number of chunks
    for C in (32, 16):
        assert lib.mdn_workspace_bytes(ctypes.byref(shape(C=C)), 0, ctypes.byref(n)) == 0 and n.value > (64 // C) * fwd
        assert lib.mdn_saved_states_bytes(ctypes.byref(shape(C=C)), ctypes.byref(n)) == 0
        assert n.value == 2 * 3 * (128 // C) * 2 * 128 * 128 * 2
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(shape(B=1, C=32)), (ctypes.c_int32 * 2)(0, 128), 1, 0, ctypes.byref(n)) == -2
    assert lib.mdn_workspace_bytes(ctypes.byref(shape(dtype=7)), 0, ctypes.byref(n)) == -3
    assert lib.mdn_workspace_bytes(ctypes.byref(shape()), 0, None) == -1
    assert lib.mdn_workspace_bytes(None, 0, ctypes.byref(n)) == -1
    assert lib.mdn_saved_states_bytes(ctypes.byref(shape()), ctypes.byref(n)) == 0
    assert n.value == 2 * 3 * 2 * 2 * 128 * 128 * 2
    assert lib.mdn_saved_operands_bytes(ctypes.byref(shape()), ctypes.byref(n)) == 0 and n.value > 0
    # fp32 storage doubles every stored intermediate; the coefficient block and the two state buffers that
    # carry S, M between segments of a split call are fp32 in both modes
    fixed = 4 * 8 * 64 * 2 * 3 * 2 + 2 * (3 * 2 * 128 * 128 * 4 + 256)
    assert binding.workspace_bytes(shape(dtype=1), 0) > 1.9 * (fwd - fixed)


def test_entry_points_reject_null_and_misaligned_pointers_before_touching_a_device():
    lib = binding.load_library()
    s = shape()
    null = [None] * 17
    assert lib.mdn_chunk_fwd(ctypes.byref(s), *null[:15], None, 0, None) == -1
    assert lib.mdn_recurrent_step(ctypes.byref(s), *[None] * 10, None) == -1
    good = ctypes.c_void_p(4096)
    bad = ctypes.c_void_p(4098)
    args = [good, good, good, good, good, good, None, None, None, bad, None, None, None, None, None, good, 1 << 40,
            None]
    assert lib.mdn_chunk_fwd(ctypes.byref(s), *args) == -5
    args[9] = good
    args[16] = 16
    assert lib.mdn_chunk_fwd(ctypes.byref(s), *args) == -4


def test_cpu_tensors_are_refused():
    import torch
    x = torch.zeros(1, 64, 1, 64)
    g = torch.zeros(1, 64, 1)
    with pytest.raises(binding.MdnError):
        binding.mdn_chunk_fwd(x, x, x, g, g, g)


def test_varlen_workspace_query_validates_the_offsets():
    lib = binding.load_library()
    n = ctypes.c_size_t(0)
    cu = lambda *v: (ctypes.c_int32 * len(v))(*v)
    s1 = shape(B=1, T=300)
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s1), cu(0, 100, 300), 2, 0, ctypes.byref(n)) == 0 and n.value > 0
    # enough for whatever the call brings in: 6 chunks, where one sequence of all T tokens has 5 and needs no table
    whole = ctypes.c_size_t(0)
    assert lib.mdn_workspace_bytes(ctypes.byref(s1), 0, ctypes.byref(whole)) == 0
    assert n.value >= whole.value + 2 * 300 * s1.H * 4
    first = n.value
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s1), cu(0, 150, 300), 2, 0, ctypes.byref(n)) == 0 and n.value <= first
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s1), cu(0, 100, 299), 2, 0, ctypes.byref(n)) == -2   # does not end at T
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s1), cu(0, 100, 100, 300), 3, 0, ctypes.byref(n)) == -2   # empty sequence
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s1), cu(1, 100, 300), 2, 0, ctypes.byref(n)) == -2   # does not start at 0
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(shape(B=2, T=300)), cu(0, 100, 300), 2, 0, ctypes.byref(n)) == -2
    assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s1), None, 2, 0, ctypes.byref(n)) == -1


@pytest.mark.parametrize("n", [1, 2, 8, 64, 512, 4096])
def test_varlen_workspace_follows_what_the_call_brings_in_and_stays_bounded(n):
    """32 768 tokens of 16 heads of 128 in n sequences.  Calls without adjoints of the final states need what one unbroken sequence
    does, up to a quarter more for partial chunks and 64 bytes a token for tables and copies of the gates; so do calls with
    adjoints, unless one long sequence by itself needs more (it also keeps the rounding remainders of its states)."""
    T, H = 32768, 16
    s = shape(B=1, T=T, H=H)
    w = [1 + (7 * i) % 13 for i in range(n)]
    at = lambda i: sum(w[:i]) * (T - n) // sum(w) + i
    cu = (ctypes.c_int32 * (n + 1))(*[at(i) for i in range(n)], T)
    lib = binding.load_library()

    def need(which):
        b = ctypes.c_size_t(0)
        assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s), cu, n, which, ctypes.byref(b)) == 0
        return b.value
    whole = binding.workspace_bytes(s, binding.MDN_WS_BWD)
    extra = 64 * T
    assert need(binding.MDN_WS_BWD_NO_STATES) <= 5 * whole // 4 + extra
    assert need(binding.MDN_WS_BWD_NO_STATES) <= need(binding.MDN_WS_BWD_NO_STATE_ADJOINTS) <= 5 * whole // 4 + extra
    longest = shape(B=1, T=max(cu[i + 1] - cu[i] for i in range(n)), H=H)
    most = max(5 * whole // 4, binding.workspace_bytes(longest, binding.MDN_WS_BWD_STATE_ADJOINTS))
    assert need(binding.MDN_WS_BWD_NO_STATE_ADJOINTS) <= need(binding.MDN_WS_BWD) <= most + extra
    assert need(binding.MDN_WS_FWD_NO_STATES) <= need(binding.MDN_WS_FWD)
    bytes_out = ctypes.c_size_t(0)
    for which in (2, 6, -1):
        assert lib.mdn_workspace_bytes_varlen(ctypes.byref(s), cu, n, which, ctypes.byref(bytes_out)) == -2
    g = ctypes.c_void_p(4096)
    inputs = [g] * 6 + [None]                             # q k v beta alpha mu eta
    for state, adjoint in ((None, None), (g, None), (g, g)):
        assert lib.mdn_chunk_fwd_varlen(ctypes.byref(s), cu, n, *inputs, state, None, g, None, None, None, g, 1 << 20, None) == -4
        assert lib.mdn_chunk_bwd_varlen(ctypes.byref(s), cu, n, *inputs, state, None, g, g, adjoint, None, *[g] * 6, None, None, None,
                                        g, 1 << 20, None) == -4


def _cpu_inputs(B=1, T=64, H=2, d=64, dtype=None):
    import torch
    dtype = dtype or torch.float32
    q = torch.zeros(B, T, H, d, dtype=dtype)
    g = torch.zeros(B, T, H)
    return dict(q=q, k=q.clone(), v=q.clone(), beta=g, alpha=g.clone(), mu=g.clone())


@pytest.mark.parametrize("bad", ["k_shape", "v_dtype", "gate_shape", "gate_dtype", "S0_shape", "eta_shape", "out_o",
                                 "workspace_small", "states_small"])
def test_binding_refuses_tensors_that_do_not_fit_q_before_any_launch(bad):
    """The C ABI trusts raw pointers, so the binding checks every tensor's shape, dtype and device against what q
    implies; the checks run before a pointer is taken (they fire on CPU tensors, with no device in reach)."""
    import torch
    t = _cpu_inputs()
    kw = {}
    if bad == "k_shape":
        t["k"] = torch.zeros(1, 64, 2, 32)
    elif bad == "v_dtype":
        t["v"] = t["v"].to(torch.bfloat16)
    elif bad == "gate_shape":
        t["alpha"] = torch.zeros(1, 63, 2)
    elif bad == "gate_dtype":
        t["mu"] = t["mu"].double()
    elif bad == "S0_shape":
        kw["S0"] = torch.zeros(1, 2, 64, 32)
    elif bad == "eta_shape":
        kw["eta"] = torch.zeros(1, 64)
    elif bad == "out_o":
        kw["out"] = {"o": torch.zeros(1, 32, 2, 64)}
    elif bad == "workspace_small":
        kw["workspace"] = torch.zeros(1024, dtype=torch.uint8)
    elif bad == "states_small":
        kw.update(save_states=True, out={"states": torch.zeros(16)})
    with pytest.raises(binding.MdnError) as e:
        binding.mdn_chunk_fwd(t["q"], t["k"], t["v"], t["beta"], t["alpha"], t["mu"], **kw)
    assert "GPU" not in str(e.value), str(e.value)      # refused for what is wrong with it, not for being a CPU tensor


def test_binding_checks_the_backward_and_the_other_entry_points_too():
    import torch
    t = _cpu_inputs()
    names = ("q", "k", "v", "beta", "alpha", "mu")
    vt = torch.zeros(1, 64, 2, 64)
    with pytest.raises(binding.MdnError, match="dO"):
        binding.mdn_chunk_bwd(*(t[k] for k in names), vt, torch.zeros(1, 64, 2, 32))
    with pytest.raises(binding.MdnError, match="dS_final"):
        binding.mdn_chunk_bwd(*(t[k] for k in names), vt, vt.clone(), dS_final=torch.zeros(1, 2, 64, 64, dtype=torch.float64))
    with pytest.raises(binding.MdnError, match=r"out\['dq'\]"):
        binding.mdn_chunk_bwd(*(t[k] for k in names), vt, vt.clone(), out={"dq": torch.zeros(1, 64, 2, 32)})
    S = torch.zeros(1, 2, 64, 64)
    with pytest.raises(binding.MdnError, match="M0"):     # the states of the recurrent step go through the same check
        binding.mdn_recurrent_step(*(t[k] for k in names), S, torch.zeros(1, 2, 64, 32))
    with pytest.raises(binding.MdnError, match="cu_seqlens"):
        binding.mdn_chunk_fwd_varlen(*(t[k] for k in names), [0, 40, 63])
    with pytest.raises(binding.MdnError, match="cu_seqlens"):
        binding.mdn_chunk_fwd_varlen(*(t[k] for k in names), [0, 40, 40, 64])
    for huge in ([0, 40, 2 ** 70], [-2 ** 70, 64], [0, 2 ** 31 + 64]):
        with pytest.raises(binding.MdnError, match="cu_seqlens"):
            binding.mdn_chunk_fwd_varlen(*(t[k] for k in names), huge)
    with pytest.raises(binding.MdnError, match="S0"):     # per-sequence states: [n_seq, H, dk, dv]
        binding.mdn_chunk_fwd_varlen(*(t[k] for k in names), [0, 40, 64], S0=torch.zeros(1, 2, 64, 64))
    for scale in ("0.125", 1, torch.tensor(0.125)):       # whatever float() takes
        with pytest.raises(binding.MdnError, match="GPU"):
            binding.mdn_chunk_fwd(*(t[k] for k in names), scale=scale)
    x = torch.zeros(1, 64, 2)
    h = torch.zeros(2)
    with pytest.raises(binding.MdnError, match="b_mu"):
        binding.mdn_gates_fwd(x, x, x, x, h, h, h, torch.zeros(3), 1.0, 1.0)
    with pytest.raises(binding.MdnError, match="x_beta"):
        binding.mdn_gates_fwd(x, x, torch.zeros(1, 64, 3), x, h, h, h, h, 1.0, 1.0)
    with pytest.raises(binding.MdnError, match="x_k"):
        binding.mdn_frontend_fwd(t["q"], torch.zeros(1, 64, 2, 32), t["v"], h)
    with pytest.raises(binding.MdnError, match="w"):
        binding.mdn_epilogue_fwd(t["q"], t["q"], torch.zeros(32))


def test_backward_workspace_for_calls_with_adjoints_of_the_final_states():
    """Such a call keeps the rounding remainders of the chunk states and chunk adjoints (16-bit storage): two more
    state-sized tensors; with 32-bit storage nothing changes."""
    plain = binding.workspace_bytes(shape(), binding.MDN_WS_BWD)
    more = binding.workspace_bytes(shape(), binding.MDN_WS_BWD_STATE_ADJOINTS)
    states = 2 * 3 * 2 * 2 * 128 * 128 * 2
    assert more == plain + 2 * states
    f32 = shape(dtype=1)
    assert binding.workspace_bytes(f32, binding.MDN_WS_BWD) == binding.workspace_bytes(f32, binding.MDN_WS_BWD_STATE_ADJOINTS)
    lib = binding.load_library()
    n = ctypes.c_size_t(0)
    assert lib.mdn_workspace_bytes(ctypes.byref(shape()), 3, ctypes.byref(n)) == -2


def test_host_side_entry_points_from_several_threads():
    """mdn_set_segments is one atomic exchange for the process and the size queries touch no shared state: threads that
    call them at the same time see consistent values (every value a call returns is one that some call has set)."""
    import threading
    lib = binding.load_library()
    want = binding.workspace_bytes(shape(), binding.MDN_WS_BWD)
    old = lib.mdn_set_segments(0)
    seen, wrong = [set() for _ in range(8)], []

    def work(i):
        n = ctypes.c_size_t(0)
        for it in range(3000):
            seen[i].add(lib.mdn_set_segments(1 + (i + it) % 7))
            if lib.mdn_workspace_bytes(ctypes.byref(shape()), 1, ctypes.byref(n)) != 0 or n.value != want:
                wrong.append(n.value)
            if lib.mdn_strerror(-4 - i % 3) is None:
                wrong.append("strerror")

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    last = lib.mdn_set_segments(old)
    assert not wrong
    assert set().union(*seen) <= set(range(0, 8)) and 1 <= last <= 7
    assert lib.mdn_set_segments(old) == old


# stand-ins for the four device queries on the way to a call's stream, so that a call gets as far as its pointers without
# a device; the library refuses the null pointers of the unwrapped call before it launches anything
STUB = """
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { return d != 0; }
int hipDeviceGetStreamPriorityRange(int *least, int *greatest) { *least = *greatest = 0; return 0; }
"""
NO_STORAGE = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
import torch
import torch._subclasses.fake_tensor as fake
from paper_2605_05838_amd import binding
fake.init_gpu_context = lambda device: None
with fake.FakeTensorMode():
    x, g, S = (torch.empty(s, device="cuda:0") for s in ((3, 1, 1, 1, 64), (3, 1, 1, 1), (3, 1, 1, 64, 64)))
    one = [torch.empty(t.shape[1:], device="cuda:0") for t in (x, g, S)]
step = lambda x, g, S: binding.mdn_recurrent_step(x, x, x, g, g, g, S, S, out=x)
for f, args, error, text in ((step, one, binding.MdnError, "NULL"), (torch.vmap(step), (x, g, S), RuntimeError, "storage")):
    try:
        f(*args)
    except error as e:
        assert text in str(e), e
    else:
        raise AssertionError("accepted")
print("raised")
"""


def test_a_tensor_without_storage_raises_and_the_interpreter_goes_on(tmp_path):
    """Inside torch.vmap the tensors have no storage: taking their pointers raises, which has to happen while the binding
    holds the interpreter lock."""
    import subprocess
    import sys
    (tmp_path / "stub.c").write_text(STUB)
    stub = str(tmp_path / "stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", stub, str(tmp_path / "stub.c")], check=True)
    p = subprocess.run([sys.executable, "-c", NO_STORAGE, stub], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.strip() == "raised", (p.returncode, p.stderr[-2000:])


def test_no_kernel_spills_vector_registers(tmp_path):
    """The kernels are laid out to fit the register file: what the compiler puts into scratch memory instead is stored and
    loaded again by every lane.  Read from the metadata of the kernels as built here."""
    import glob
    import subprocess
    objs = sorted(glob.glob(os.path.join(ROOT, "paper_2605_05838_amd", "_build", "mdn_*.o")))
    tools = "/opt/rocm/llvm/bin/"
    if not objs or not os.path.exists(tools + "llvm-readelf"):
        pytest.skip("needs the objects of a build and the LLVM tools")
    kernels = {}
    for obj in objs:
        bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
        if subprocess.run([tools + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, obj, "/dev/null"],
                          capture_output=True).returncode:
            continue                                          # (the binding's module holds no kernels)
        subprocess.run([tools + "clang-offload-bundler", "--unbundle", "--type=o", "--input=" + bundle, "--output=" + code,
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True, capture_output=True)
        notes = subprocess.run([tools + "llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
        for k in notes.split("- .agpr_count:")[1:]:
            field = lambda name: re.search(rf"\.{name}:\s+(\S+)", k)[1]
            kernels[field("name")] = int(field("private_segment_fixed_size")), int(field("vgpr_spill_count"))
    assert len(kernels) > 50 and any("grad_kernel" in k for k in kernels)
    assert not [k for k, v in kernels.items() if v != (0, 0)]


# a runtime that accepts everything and an allocator that can be told to fail
NO_MEMORY_STUB = """
#include <new>
#include <cstdlib>
extern "C" {
int no_memory = 0;
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipFuncGetAttributes(void *, const void *) { return 1; }
int hipEventCreate(void **e) { *e = &no_memory; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = &no_memory; return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventDestroy(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = &no_memory; return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipLaunchKernel(const void *, unsigned long, unsigned, unsigned long, unsigned, void **, unsigned long, void *) { return 0; }
int hipGetLastError() { return 0; }
}
void *operator new(std::size_t n) {
    if (no_memory) throw std::bad_alloc();
    return std::malloc(n);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
"""
NO_MEMORY = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
fail = ctypes.c_int.in_dll(stub, "no_memory")
class Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in "BTHdvCt"] + [("scale", ctypes.c_float)]
s, g, none = Shape(1, 1, 1, 64, 64, 64, 0, 0.1), ctypes.c_void_p(4096), ctypes.c_void_p(None)
step = lambda: lib.mdn_recurrent_step(ctypes.byref(s), g, g, g, g, g, g, none, g, g, g, none)
codes = [step()]
lib.mdn_profile_begin()
fail.value = 1
codes.append(step())
fail.value = 0
lib.mdn_profile_end(None, None, 0)
s.T = 1024
cu = (ctypes.c_int32 * 3)(0, 500, 1024)
fwd = lambda: lib.mdn_chunk_fwd(ctypes.byref(s), g, g, g, g, g, g, none, none, none, g, none, none, none, none, none, g, ctypes.c_size_t(1 << 40), none)
packed = lambda: lib.mdn_chunk_fwd_varlen(ctypes.byref(s), cu, 2, g, g, g, g, g, g, none, none, none, g, none, none, none, g, ctypes.c_size_t(1 << 40), none)
lib.mdn_set_segments(2)
fail.value = 1
codes += [fwd(), packed()]
fail.value = 0
codes += [fwd(), packed()]
print(codes)
"""


def test_running_out_of_host_memory_is_an_error_code(tmp_path):
    """No C++ exception leaves an entry point: the event list of the timing facility, the second stream's events, the offsets
    of a packed batch.  (The pointers given are no memory: only where there is no device that could read them.)"""
    import subprocess
    import sys
    import torch
    if torch.cuda.device_count():
        pytest.skip("for machines without a GPU")
    (tmp_path / "stub.cpp").write_text(NO_MEMORY_STUB)
    stub = str(tmp_path / "stub.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-w", "-o", stub, str(tmp_path / "stub.cpp")], check=True)
    p = subprocess.run([sys.executable, "-c", NO_MEMORY, stub, binding.LIB_PATH], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.split("\n")[0] == "[0, -6, -6, -6, 0, 0]", (p.returncode, p.stdout, p.stderr[-2000:])
