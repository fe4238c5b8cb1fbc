// gn::LdsLimit against a stand-in of the two HIP calls it makes.
#include "lds_limit.h"

static int g_device = 0, g_calls = 0, g_last = 0;
static hipError_t g_result = hipSuccess;

extern "C" hipError_t hipGetDevice(int *d) {
  *d = g_device;
  return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int value) {
  ++g_calls;
  if (g_result == hipSuccess) g_last = value;
  return g_result;
}

extern "C" {
void *l_create() { return new gn::LdsLimit(); }
void l_destroy(void *p) { delete (gn::LdsLimit *)p; }
int l_raise(void *p, int device, int fail, int bytes) {
  g_device = device;
  g_result = fail ? hipErrorInvalidValue : hipSuccess;
  return ((gn::LdsLimit *)p)->raise(nullptr, (size_t)bytes) == hipSuccess ? 0 : -1;
}
int l_calls() { return g_calls; }
int l_last() { return g_last; }
}
