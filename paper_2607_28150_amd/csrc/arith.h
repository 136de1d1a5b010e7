// Launch and sampling arithmetic.  Nothing here needs HIP, so the host tests
// compile this file by itself.
#pragma once

#include <stdint.h>

namespace sg {

// Workgroups of `threads` threads that one grid dimension may hold: its
// threads are counted in 32 bits (a larger launch is refused).
constexpr int64_t max_workgroups(int64_t threads) { return 0xffffffffll / threads; }

// Workgroups of a grid-stride kernel over `total` items, `per` items per
// workgroup and pass: one pass where the launch may be that large, else the
// kernel's stride loop takes the rest.
constexpr int64_t stride_grid(int64_t total, int64_t per, int threads) {
    const int64_t need = (total + per - 1) / per, most = max_workgroups(threads);
    return need < 1 ? 1 : need < most ? need : most;
}

// launch(first, n) for the pieces [first, first + n) of `count` that one launch
// of `threads` threads each may hold.
template <typename F>
void launch_slices(int64_t count, int64_t threads, F &&launch) {
    const int64_t most = max_workgroups(threads);
    for (int64_t first = 0; first < count; first += most)
        launch(first, count - first < most ? count - first : most);
}

// Sampled key i of `ns` among `seen` keys (0 <= i < ns <= seen): one in each of
// ns equal stretches of all of them, at a hashed place.  (At one fixed place of
// stretches of whole keys, keys whose logits repeat with the stretch were
// sampled at one phase only, and up to ns - 1 keys at the end, the newest, not
// at all: 900 keys of a prompt whose logits rise took 278 us, random ones 103.)
constexpr int sample_key(int i, int ns, int seen) {
    if (ns == seen) return i;
    uint32_t h = (uint32_t)i * 0x9e3779b1u;
    h = (h ^ (h >> 15)) * 0x85ebca77u;
    h ^= h >> 13;
    const float place = (float)i + (float)(h >> 8) * 0x1p-24f;
    const int key = (int)(place * ((float)seen / (float)ns));
    return key < seen - 1 ? key : seen - 1;
}

}  // namespace sg
