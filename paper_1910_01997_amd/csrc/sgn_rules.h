// Rules of the host side that need neither the device nor the runtime (plain
// C++, so that tests compile them by themselves).
#pragma once

#include <cstddef>
#include <cstdint>

namespace sgn {

// One past the last byte, from an image's first, that the taps of a sample can
// touch when rows are read by index: corners reach x0 = width - 2 and the
// second row is the last.  Float taps are the pair itself; halves and bytes
// come as eight bytes from the aligned dword below the pair, which at the
// row's end is up to four bytes more than the row's last dword.
inline size_t tap_reach(int width, int height, size_t pitch_b, int elem_bytes) {
    const size_t col = (size_t)(width - 2) * elem_bytes;
    return (size_t)(height - 1) * pitch_b + (elem_bytes == 4 ? col : col & ~size_t(3)) + 8;
}
// One past the image's last dword.
inline size_t image_end(int width, int height, size_t pitch_b, int elem_bytes) {
    return (size_t)(height - 1) * pitch_b + (((size_t)width * elem_bytes + 3) & ~size_t(3));
}

// Whether an image's rows may be read by index.  Those loads check the row
// only, so where taps reach past the image the bytes there have to be mapped:
// they are in the page of the image's last byte, or the next image starts
// there (next: its address, or 0), or the memory's owner says so
// (mapped_end(address of the last byte): one past the last mapped byte).
// Otherwise the rows are read by byte offset, which the hardware checks
// against the image's size.
template <class MappedEnd>
bool rows_by_index_safe(uintptr_t data, int width, int height, size_t pitch_b, int elem_bytes, uintptr_t next,
                        MappedEnd&& mapped_end) {
    constexpr uintptr_t kPage = 4096;              // the smallest page
    const uintptr_t end = data + image_end(width, height, pitch_b, elem_bytes);
    const uintptr_t reach = data + tap_reach(width, height, pitch_b, elem_bytes);
    if (reach <= end || end % kPage != 0 || next == end) return true;
    return reach <= mapped_end(end - 1);
}

}  // namespace sgn
