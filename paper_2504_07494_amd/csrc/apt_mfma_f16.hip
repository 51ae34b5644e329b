#define APT_MFMA_DT 1
#include "apt_mfma.inc"
