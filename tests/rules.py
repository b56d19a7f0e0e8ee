"""csrc/sgn_rules.h (host rules that need neither device nor runtime), compiled by itself."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_01997_amd", "csrc")

SHIM = r"""
#include "sgn_rules.h"
struct Kf { int32_t n_items, n_nbr, item_base; };
extern "C" {
void cut_shares(int nq, const Kf* kfs, int n, double fixed, int32_t* out) {
    sgn::cut_shares(nq, kfs, n, fixed, (sgn::QueueDev*)out);
}
int item_blocks(int nq, const int32_t* queues, int items, int wpb) {
    return sgn::item_blocks(nq, (const sgn::QueueDev*)queues, items, wpb);
}
size_t tap_reach(int w, int h, size_t pitch_b, int elem) { return sgn::tap_reach(w, h, pitch_b, elem); }
size_t image_end(int w, int h, size_t pitch_b, int elem) { return sgn::image_end(w, h, pitch_b, elem); }
int rows_by_index_safe(uint64_t data, int w, int h, size_t pitch_b, int elem, uint64_t next, uint64_t mapped) {
    return sgn::rows_by_index_safe(data, w, h, pitch_b, elem, next, [&](uintptr_t) { return (uintptr_t)mapped; });
}
int bin_in_lds(int keyframes, int64_t tiles, int64_t surfels) { return sgn::bin_in_lds(keyframes, tiles, surfels); }
int damped_one_frame(double w, int patch, double pixels, double bytes, double frames, int far_taps) {
    return sgn::damped_one_frame(w, patch, pixels, bytes, frames, far_taps != 0);
}
int init_reach(float beta_r, int patch) { return sgn::init_reach(beta_r, patch); }
int raster_pixels(int64_t tiles, double mean, int cus) { return sgn::raster_pixels(tiles, mean, cus); }
double mean_tiles(double radius, int tile) { return sgn::mean_tiles(radius, tile); }
int disc_form(double w, double slots, int f32, int damped) {
    const sgn::DiscForm f = sgn::disc_form(w, slots, f32, damped);
    return f.waves * 100 + f.deep * 10 + f.shared;
}
}
"""


@functools.lru_cache(maxsize=None)
def lib():
    d = tempfile.mkdtemp(prefix="sgn_rules_")
    src, out = os.path.join(d, "shim.cpp"), os.path.join(d, "libshim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, src, "-o", out],
                   check=True)
    L = C.CDLL(out)
    for n in ("tap_reach", "image_end"):
        getattr(L, n).restype = C.c_size_t
        getattr(L, n).argtypes = [C.c_int, C.c_int, C.c_size_t, C.c_int]
    L.rows_by_index_safe.argtypes = [C.c_uint64, C.c_int, C.c_int, C.c_size_t, C.c_int, C.c_uint64, C.c_uint64]
    L.cut_shares.argtypes = [C.c_int, C.c_void_p, C.c_int, C.c_double, C.c_void_p]
    L.cut_shares.restype = None
    L.item_blocks.argtypes = [C.c_int, C.c_void_p, C.c_int, C.c_int]
    L.bin_in_lds.argtypes = [C.c_int, C.c_int64, C.c_int64]
    L.damped_one_frame.argtypes = [C.c_double, C.c_int, C.c_double, C.c_double, C.c_double, C.c_int]
    L.init_reach.argtypes = [C.c_float, C.c_int]
    L.raster_pixels.argtypes = [C.c_int64, C.c_double, C.c_int]
    L.mean_tiles.argtypes = [C.c_double, C.c_int]
    L.mean_tiles.restype = C.c_double
    L.disc_form.argtypes = [C.c_double, C.c_double, C.c_int, C.c_int]
    return L
