// Index arithmetic at the edges of the tensors and launches that the entry points accept: up to 2^31 - 1 elements, counted in int.
#pragma once

namespace dwc {

// Whether the ve elements from a on lie inside a tensor of `total` elements; a + ve may be 2^31 and more.
constexpr bool vector_inside(int a, int ve, int total) { return a <= total - ve; }

// Four elements from p on are read from run_start(p, total) on, so that the read stays inside a tensor of total >= 4 elements wherever p lies in
// it; they are then the ones from element p - run_start of the read on.  runs_past: whether that is not 0 for some p before `end`.
constexpr unsigned run_start(unsigned p, unsigned total) { return p < total - 4 ? p : total - 4; }
constexpr bool runs_past(unsigned end, unsigned total) { return end > total - 3; }

// ceil(a / b) for a >= 1, b >= 1 (a + b - 1 may be 2^31 and more)
constexpr int cdiv(int a, int b) { return (a - 1) / b + 1; }

// End of part `part` of `items` dealt `per` at a time; part * per < items.
constexpr int part_end(int items, int per, int part) { return items - part * per < per ? items : part * per + per; }

// Whether a launch has fewer than 2^32 lanes, which the runtime asks for.
constexpr bool launchable(long long blocks, int threads) { return blocks * threads < 1LL << 32; }

}  // namespace dwc
