// Test helper (a shared library loaded with ctypes beside libxg.so): what
// the planner and the emitters made of a loaded program, without a GPU.
#include <fstream>
#include <string>
#include <vector>

#include "xg_program.h"

extern "C" {

// The source of the persistent kernel over k programs, written to `path`.
int probe_batch_source(xg_program** ps, int k, const char* path) {
  std::string src;
  const xg_status st = xg::batch_source(std::vector<xg_program*>(ps, ps + k), src);
  if (st == XG_OK) std::ofstream(path) << src;
  return (int)st;
}

}  // extern "C"
