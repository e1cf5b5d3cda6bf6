// Index arithmetic at the edges of the tensors and launches that the entry points accept: up to 2^31 - 1 elements, counted in int.
#pragma once

namespace dwc {

// Whether the ve elements from a on lie inside a tensor of `total` elements; a + ve may be 2^31 and more.
constexpr bool vector_inside(int a, int ve, int total) { return a <= total - ve; }

}  // namespace dwc
