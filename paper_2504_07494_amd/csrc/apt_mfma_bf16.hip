#define APT_MFMA_DT 2
#include "apt_mfma.inc"
