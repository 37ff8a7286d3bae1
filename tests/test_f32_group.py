"""CPU: what the fp32 launch of dX with the weight gradients takes (gemm_f32_group, called through its own header).  Its tile for the weight
gradients is chosen once, from the first of them, so a second one of other extents is refused before anything is launched: 64-wide
tiles of split products begin before the end of an extent and would begin before an operand of less than 64."""
import ctypes
import os
import subprocess

import pytest
import torch

from paper_2507_09029_amd import build

SOURCE = '''#include "sdp_internal.h"
extern "C" int group(int m0, int n0, int k0, int m1, int n1, int k1) {
    sdp::GemmDesc d[3];
    char* const at = (char*)4096; // never read: refused before a launch
    d[0].M = 512, d[0].N = 512, d[0].K = 512, d[0].lda = 512, d[0].A = at, d[0].B = at, d[0].ldb = 512, d[0].b_km = 1, d[0].C = at, d[0].ldc = 512;
    const int e[2][3] = {{m0, n0, k0}, {m1, n1, k1}};
    for (int i = 0; i < 2; ++i) {
        sdp::GemmDesc& w = d[1 + i];
        w.M = e[i][0], w.N = e[i][1], w.K = e[i][2], w.lda = w.ldb = w.ldc = 512, w.a_km = w.b_km = 1, w.A = w.B = at, w.C = at;
    }
    d[1].nbatch = 3;
    for (int i = 0; i < 3; ++i) d[1].Ab[i] = d[1].Bb[i] = at, d[1].Cb[i] = at;
    return sdp::gemm_f32_group(d, 3, "test", nullptr);
}
'''


@pytest.fixture(scope="module")
def group(tmp_path_factory):
    if torch.cuda.is_available():
        pytest.skip("made-up addresses: a call that is not refused ends at the first HIP call where there is no GPU")
    d = tmp_path_factory.mktemp("group")
    (d / "group.hip").write_text(SOURCE)
    if not os.path.exists(build.LIB):
        build.build_library()
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-host-only", "-shared", str(d / "group.hip"), "-o", str(d / "group.so"), "-L", build.HERE,
                    "-l:" + os.path.basename(build.LIB), f"-Wl,-rpath,{build.HERE}"], check=True)
    return ctypes.CDLL(str(d / "group.so")).group


@pytest.mark.parametrize("second", [(32, 512, 512), (512, 32, 512), (512, 512, 40), (448, 512, 512), (512, 576, 512)])
def test_weight_gradients_of_other_extents_are_refused(group, second):
    assert group(512, 512, 512, *second) == -5  # SDP_ERR_UNSUPPORTED
