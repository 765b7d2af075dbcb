// lba_wide_conv.hip -- lba_wide.hip for im2col rows of an NHWC tensor.
#define LBA_WIDE_CONV 1
#include "lba_wide.hip"
