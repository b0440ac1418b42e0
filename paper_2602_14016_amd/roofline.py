"""Byte models of the hot kernels and the HBM-traffic record.

Kernel classes are those the library's launch timer knows (pa_profile_start):
0 the right-hand-side row pass, 1 the forward-stage column pass, 2 the
adjoint-product row pass, 3 the adjoint-stage column pass.

kernel_bytes counts what a kernel must move per member and launch, with every
field read or written once: Yb is one field in the Y layout restricted to the
retained band, N rows of Kc + 1 complex values; Cb is one compact spectral
state, (2 Kc + 1) x (Kc + 1) complex values.  Padding columns and repeated
reads are not counted, so kernel_bytes / time is a lower bound on the
bandwidth a kernel actually draws.

algorithmic_bytes is the same count for the passes in advective form (u, v,
w_x, w_y in physical space), which the kernels computed before they worked on
velocities only.  It is the yardstick of the profiles taken on those kernels
(row_nl_kernel, row_adj_kernel, col_kernel).
"""

import hashlib
import os

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HBM_PEAK_GBS = 8000.0   # MI355X HBM3E

CLASS_NAMES = {0: "row_sq_kernel", 1: "col_pass_kernel (forward stages)", 2: "row_mul_kernel",
               3: "col_pass_kernel (adjoint stages)"}


def field_bytes(N):
    """(Yb, Cb) for grid size N."""
    Kc = (N - 1) // 3
    return N * (Kc + 1) * 16, (2 * Kc + 1) * (Kc + 1) * 16


def algorithmic_bytes(cls, N):
    """Bytes per member of one launch of class cls in the advective form."""
    Yb, Cb = field_bytes(N)
    return {0: 5 * Yb,                  # read U, V, Wx, Wy; write q
            1: 5 * Yb + 2.75 * Cb,      # read q; write U, V, Wx, Wy; state and accumulator (mean over stages A-D)
            2: 8 * Yb,                  # read U, V, Wx, Wy, Lambda, Lambda_y; write the two products
            3: 4 * Yb + 2.5 * Cb}[cls]  # read the two products; write Lambda, Lambda_y; adjoint accumulators


def kernel_bytes(cls, N):
    """Bytes per member of one launch of kernel class cls: each input and output once."""
    Yb, Cb = field_bytes(N)
    return {0: 4 * Yb,                  # read the velocity pair; write the pair of products
            1: 4 * Yb + 2.75 * Cb,      # read the products; write the velocity pair; state and accumulator
            2: 6 * Yb,                  # read the velocity and cotangent pairs; write the products
            3: 4 * Yb + 2.5 * Cb}[cls]  # read the products; write the cotangent pair; adjoint accumulators


# the sources that define and instantiate the row and column kernels, and the
# build flags they are compiled with (host-side files do not change them)
KERNEL_SOURCES = ("csrc/fft.hpp", "csrc/kernels.hpp", "csrc/kernels_impl.hpp", "csrc/kernels.hip",
                  "csrc/kern_8.hip", "csrc/kern_16.hip", "csrc/kern_32.hip", "csrc/kern_64.hip",
                  "csrc/kern_128.hip", "csrc/kern_256.hip", "csrc/kern_512.hip", "csrc/kern_1024.hip", "csrc/small.hpp", "csrc/kern_small.hip",
                  "build.py")


def kernel_source_sha():
    """Hash of the row/column kernel sources and build flags: a traffic record
    applies only to the kernels it was taken on."""
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(HERE, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


TRAFFIC_PATH = os.path.join(ROOT, "profiles", "traffic_counters.txt")


def read_traffic(cls, N, members, kernel=None, path=TRAFFIC_PATH):
    """HBM bytes per launch of class cls from the committed counter record, or
    None if the record is missing or was taken on other sources, another
    class or shape, or (if given) holds no such kernel instantiation: the record's
    own, or one that its launch lines name."""
    if not os.path.exists(path):
        return None
    kv, launches = {}, {}
    with open(path) as fh:
        for line in fh:
            if ":" in line and not line.startswith("#"):
                k, v = line.split(":", 1)
                if k == "launch":
                    name, _, value = v.strip().rpartition(" ")
                    launches[name] = value
                kv[k.strip()] = v.strip()
    if kv.get("source_sha") != kernel_source_sha():
        return None
    try:
        if int(kv.get("class", -1)) != cls or int(kv.get("N", -1)) != N or int(kv.get("members", -1)) != members:
            return None
        if kernel is not None and kv.get("kernel") != kernel:
            return float(launches[kernel])
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None
