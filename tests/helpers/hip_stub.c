/* Stand-ins for the HIP calls a convolution makes on the host, loaded before
 * libdfp.so: a current device that the test sets, counts of what was asked of
 * each, and attribute calls that fail where the test says so. */
int stub_device = 0, stub_attribute_fails = 0, stub_attributes[64], stub_launches[64];

int hipGetDevice(int* d) {
  *d = stub_device;
  return 0;
}
int hipDeviceGetAttribute(int* v, int attr, int dev) {
  (void)attr, (void)dev;
  *v = 256;
  return 0;
}
int hipFuncSetAttribute(const void* f, int attr, int value) {
  (void)f, (void)attr, (void)value;
  if (stub_attribute_fails) return 1;
  ++stub_attributes[stub_device];
  return 0;
}
int hipFuncGetAttributes(void* attr, const void* f) {
  (void)attr, (void)f;
  return 1;
}
int hipLaunchKernel(const void* f, ...) {
  (void)f;
  ++stub_launches[stub_device];
  return 0;
}
typedef struct {
  unsigned x, y, z;
} dim3_t;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, unsigned long shared, void* stream) {
  (void)grid, (void)block, (void)shared, (void)stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, unsigned long* shared, void** stream) {
  const dim3_t one = {1, 1, 1};
  *grid = *block = one;
  *shared = 0;
  *stream = 0;
  return 0;
}
int hipGetLastError(void) { return 0; }
