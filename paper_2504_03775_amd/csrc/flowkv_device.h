// What the library's launches ask of the current device.
#pragma once

namespace flowkv {

// Writes the current device's number of CUs to *out (looked up once per
// device).  Returns FLOWKV_OK, or records FLOWKV_EHIP and returns it.
int cu_count(int* out);

}  // namespace flowkv
