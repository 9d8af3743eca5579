"""GPU parity at the edges of the kernels' dispatch: the smallest and largest
size of a variant, and sizes just off its tiles.  Same oracle, metric and
tolerances as test_gpu_parity.py."""
import pytest

from _gpu_helpers import announce
from test_gpu_parity import check_layer, layer_case, oracle_layer, run_layer_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def run_case(T, B, I, H, Hp, dtype, reverse, scale, states=True):
    label = f"edge T{T} B{B} I{I} H{H} Hp{Hp} {dtype} rev{int(reverse)} states{int(states)}"
    announce(label)
    c = layer_case(T, B, I, H, Hp, dtype, reverse, seed=T * 1000 + B + H, states=states, final_grads=states,
                   scale=scale)
    gpu = run_layer_gpu(c, T, B, I, H, Hp, dtype, reverse)
    check_layer(gpu, oracle_layer(c, Hp, reverse), dtype, label)
    return gpu


# XCD-local kernels at widths padded to the next of 256, 512 and 1024:
# (T, B, H, reverse, states); weights U(+-1/sqrt(H)), the usual LSTM range
XCD_PAD_CASES = [
    (3, 5, 8, False, True),       # one workgroup per XCD, one wave's worth of k
    (3, 130, 248, True, True),    # one row of cells short of 256; two row blocks
    (2, 264, 120, False, False),  # four row blocks
    (4, 9, 264, False, True),     # just past 256
    (3, 140, 504, True, False),
    (3, 40, 520, True, True),     # just past 512: half of the workgroups idle
    (4, 130, 648, False, True),   # the last workgroup with a quarter of its cells
    (2, 257, 1016, True, True),   # one workgroup short of full; four row blocks
    (1, 1, 776, False, True),
]


@pytest.mark.parametrize("T,B,H,reverse,states", XCD_PAD_CASES)
def test_padded_xcd_widths(T, B, H, reverse, states):
    gpu = run_case(T, B, 40, H, 0, "bf16", reverse, H ** -0.5, states)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert gpu["tiling"][3] == 1001 and gpu["tiling"][7] == 1001, gpu["tiling"]
